// The atomic NNs in FP64: every layer of one element's NN in one launch, on the FP64 matrix
// instruction, with the density before it and its adjoint behind it.
//
// One workgroup takes 16 rows, one wave per 16 columns of a layer's output (H / 16 waves).  The
// activations stay in LDS, each layer in place of the one before.  Instruction and layout:
//   v_mfma_f64_16x16x4  lane l supplies A[l % 16][l / 16] (activations) and B[l / 16][l % 16]
//   (weights); D[l / 16 + 4 r][l % 16] is register r
// K advances in chunks of 8: a lane holds the pair k = 8 kc + 2 (l / 16) + {0, 1} of both operands
// (one 16-byte load each) and feeds its two values to two instructions.  The weights are packed so
// that a wave's fragment is one contiguous KB (pack_operands64).  The row stride of every LDS array is
// 4 banks mod 16 banks, odd multiples of 4: the 16 rows a fragment load touches fall into different
// banks.
//
// Bound: the matrix unit (a 16x16x4 instruction takes 64 cycles of a SIMD, 124 of them per wave in
// the forward of 3 x 128 hidden units on 234 features: 8 us a tile at the clock it sustains), and with
// few tiles a CU the phases between the layers, where all of a tile's waves wait for each other
// (SiLU 3.3 us, density 3.5, operand streams 2-11 of a 32 us launch).  16 rows a tile, so that a CU
// holds three workgroups (47 KB of LDS each) that fill each other's gaps; 32 rows halve the
// weights read but leave one workgroup a CU.  us per forward / adjoint, 16- against 32-row tiles, 3 x
// 128: 864 atoms 18.7 / 21.9 against 30.3 / 34.6, 6,336 32.4 / 35.5 against 34.3 / 37.5, 20,736 86 /
// 99 against 94 / 110.  Layer by layer with the vector units, density apart, 6,864 atoms took 172 + 20
// and 194 + 38 us; the evaluation (T = 3, E + F + W) went from 1,391 to 450 us.
#include "mfma.hpp"

namespace reann {

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kBM64 = 16;   // rows per workgroup
constexpr int kKC64 = 8;    // k per chunk

// Row stride of the activations (doubles) for F features and width H.
constexpr int ld64(int F, int H) { return (ceil_div(F, kKC64) * kKC64 > H ? ceil_div(F, kKC64) * kKC64 : H) + 2; }

__device__ inline double sigm64(double z) { return 1.0 / (1.0 + exp(-z)); }
__device__ inline double silu64(double z) { return z / (1.0 + exp(-z)); }
__device__ inline double dsilu64(double z) {
    const double sg = sigm64(z);
    return sg * (1.0 + z * (1.0 - sg));
}

// D = sum_k X[l % 16][k] W[16 jb + l % 16][k] over NCK chunks, W packed with NBLK blocks of 16
// rows; a block at or past NBLK reads the last one (the caller never stores it).
template <int NCK, int NBLK>
__device__ inline d4 layer64(const double *X, int ldx, const double *__restrict__ W, int jb, int lane) {
    constexpr int NS = NCK < 4 ? NCK : 4;   // register sets of weight fragments (2, 4 and 7 take the same)
    const d2 *wl = reinterpret_cast<const d2 *>(W) + min(jb, NBLK - 1) * 64 + lane;
    const double *xl = X + (lane & 15) * ldx + 2 * (lane >> 4);
    d2 w[NS], x[2];
    d4 acc0 = d4{0., 0., 0., 0.}, acc1 = d4{0., 0., 0., 0.};
#pragma unroll
    for (int q = 0; q < NS - 1; ++q) w[q] = wl[q * NBLK * 64];
    if (NS == 1) w[0] = wl[0];
    x[0] = *reinterpret_cast<const d2 *>(xl);
#pragma unroll
    for (int kc = 0; kc < NCK; ++kc) {
        if (NS > 1 && kc + NS - 1 < NCK) w[(kc + NS - 1) % NS] = wl[(kc + NS - 1) * NBLK * 64];
        if (kc + 1 < NCK) x[(kc + 1) & 1] = *reinterpret_cast<const d2 *>(xl + (kc + 1) * kKC64);
        __builtin_amdgcn_sched_barrier(0);   // the requests stay ahead of the instructions
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kc & 1][0], w[kc % NS][0], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kc & 1][1], w[kc % NS][1], acc1, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc0 + acc1;
}

// The tile's orbital sums into LDS; rows past the segment's end take its last row (their results
// are never stored).
template <int NLK, int NT>
__device__ inline void load_sums(const FusedNN64 &p, double *Ssh, int64_t m0, int tid) {
    static_assert(NLK % 2 == 0, "pairs");
    for (int e = tid; e < kBM64 * (NLK / 2); e += NT) {
        const int r = e / (NLK / 2), q = e % (NLK / 2);
        const int64_t row = min(m0 + r, p.rows - 1);
        *reinterpret_cast<d2 *>(Ssh + r * (NLK + 2) + 2 * q) = reinterpret_cast<const d2 *>(p.S + row * NLK)[q];
    }
}

template <int H, int L, int K> __device__ __forceinline__ void fwd64_body(const FusedNN64 &p, const int64_t m0) {
    constexpr int NT = 4 * H, NW = H / 16;
    constexpr int F = fused_features(L, K), NCK0 = ceil_div(F, kKC64), Fk = NCK0 * kKC64, ldx = ld64(F, H);
    constexpr int NLK = n_lambda(L) * K, lds = NLK + 2, P = K * (K + 1) / 2;
    constexpr int NPART = kBM64 * lds > NW * 256 ? kBM64 * lds : NW * 256;
    __shared__ __attribute__((aligned(16))) double X[kBM64 * ldx];
    __shared__ __attribute__((aligned(16))) double Ssh[NPART];   // orbital sums, then the output layer's partial sums
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    load_sums<NLK, NT>(p, Ssh, m0, tid);
    __syncthreads();
    if constexpr (L == 0) {
        for (int it = tid; it < kBM64 * K; it += NT) X[(it & 15) * ldx + (it >> 4)] = Ssh[(it & 15) * lds + (it >> 4)];
    } else {   // one task per (row, pair a <= b): that pair's features of every order
        for (int it = tid; it < kBM64 * P; it += NT) {
            const int r = it & 15, pr = it >> 4;
            int a = 0, b = pr;
            while (b >= K - a) { b -= K - a; ++a; }
            b += a;
            const double *s = Ssh + r * lds;
#pragma unroll
            for (int l = 0; l <= L; ++l) {
                double acc = 0.0;
#pragma unroll
                for (int q = l * (l + 1) * (l + 2) / 6; q < (l + 1) * (l + 2) * (l + 3) / 6; ++q)
                    acc += (double)lambda_weight(L, q) * s[q * K + a] * s[q * K + b];
                X[r * ldx + l * P + pr] = acc;
            }
        }
    }
    if constexpr (Fk > F)
        for (int it = tid; it < kBM64 * (Fk - F); it += NT) X[(it & 15) * ldx + F + (it >> 4)] = 0.0;
    __syncthreads();
    const int col = 16 * wave + li;
    for (int k = 0; k < p.nh; ++k) {
        const double bias = p.b[k][col];
        const d4 acc = k == 0 ? layer64<NCK0, NW>(X, ldx, (const double *)p.W[0], wave, lane)
                              : layer64<H / kKC64, NW>(X, ldx, (const double *)p.W[k], wave, lane);
        __syncthreads();   // every wave has read this layer's input
        double *Zk = p.Z[k];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = lg + 4 * r;
            const double z = acc[r] + bias;
            if (m0 + rr < p.rows) Zk[(m0 + rr) * H + col] = z;
            X[rr * ldx + col] = silu64(z);
        }
        __syncthreads();
    }
    {   // output layer: one block of columns, its K split over the waves
        d4 acc = d4{0., 0., 0., 0.};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = 16 * wave + 4 * s + lg;
            const double w = p.Wout[min(li, p.dout - 1) * H + k];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[li * ldx + k], w, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) Ssh[wave * 256 + (lg + 4 * r) * 16 + li] = acc[r];
    }
    __syncthreads();
    for (int it = tid; it < kBM64 * p.dout; it += NT) {
        const int r = it / p.dout, o = it % p.dout;
        const int64_t row = m0 + r;
        if (row >= p.rows) break;
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += Ssh[w * 256 + r * 16 + o];
        v += p.bout[o];
        if (p.resid) v += p.resid[row * p.dout + o];
        p.C[row * p.dout + o] = v;
        if (p.copy_rng) {
            const int2 c = p.copy_rng[row];
            for (int q = c.x; q < c.y; ++q) p.Cg[(int64_t)p.copy_idx[q] * p.dout + o] = v;
        }
    }
}

// Output layer of the adjoint: Ga[r][q] = (sum_o G[r][o] Wout[o][q]) SiLU'(z) for column q = tid % H of
// rows tid / H + 4 i.
template <int DOUT, int H>
__device__ inline void out_adjoint64(const FusedNN64 &p, const double *gs, double *Ga, int ldg, int64_t m0, int tid) {
    const int q = tid % H, r0 = tid / H;
    double wq[DOUT], z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = p.Z[p.nh - 1][min(m0 + r0 + 4 * i, p.rows - 1) * H + q];
#pragma unroll
    for (int o = 0; o < DOUT; ++o) wq[o] = p.Wout[o * H + q];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + 4 * i;
        double s = 0.0;
#pragma unroll
        for (int o = 0; o < DOUT; ++o) s += gs[r * DOUT + o] * wq[o];
        Ga[r * ldg + q] = m0 + r < p.rows ? s * dsilu64(z[i]) : 0.0;
    }
}

template <int H, int L, int K> __device__ __forceinline__ void bwd64_body(const FusedNN64 &p, const int64_t m0) {
    constexpr int NT = 4 * H, NW = H / 16;
    constexpr int F = fused_features(L, K), NBF = ceil_div(F, 16), NCBF = ceil_div(NBF, NW), ldg = ld64(F, H);
    constexpr int NL = n_lambda(L), NLK = NL * K, lds = NLK + 2, P = K * (K + 1) / 2;
    __shared__ __attribute__((aligned(16))) double Ga[kBM64 * ldg];   // the adjoint tile, in the end dE/drho
    __shared__ __attribute__((aligned(16))) double Ssh[kBM64 * lds];
    __shared__ double gs[kBM64 * K];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    if constexpr (L > 0) load_sums<NLK, NT>(p, Ssh, m0, tid);
    if (p.dout == 1) {   // the energy NN: the seed of the reverse sweep
        if (tid < kBM64) {
            const int64_t row = m0 + tid;
            gs[tid] = row < p.rows ? p.seed_scale * (p.seed_g ? *p.seed_g : 1.0) * (p.seed_w ? p.seed_w[p.perm[row]] : 1.0)
                                   : 0.0;
        }
    } else {
        for (int e = tid; e < kBM64 * K; e += NT) {
            const int64_t row = m0 + e / K;
            const int o = e % K;
            double g = 0.0;
            if (row < p.rows) {
                g = p.G[row * K + o];
                if (p.copy_rng) {   // the ghost copies' message adjoints
                    const int2 c = p.copy_rng[row];
                    for (int q = c.x; q < c.y; ++q) g += p.Gg[(int64_t)p.copy_idx[q] * K + o];
                }
                if (p.next_in) g += p.next_in[row * K + o];
                if (p.next_out) p.next_out[row * K + o] = g;
            }
            gs[e] = g;
        }
    }
    __syncthreads();
    if (p.dout == 1) out_adjoint64<1, H>(p, gs, Ga, ldg, m0, tid);
    else out_adjoint64<K, H>(p, gs, Ga, ldg, m0, tid);
    __syncthreads();
    const int col = 16 * wave + li;
    for (int k = p.nh - 1; k >= 1; --k) {
        double z[4];   // requested before the matrix loop
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = p.Z[k - 1][min(m0 + lg + 4 * r, p.rows - 1) * H + col];
        const d4 acc = layer64<H / kKC64, NW>(Ga, ldg, (const double *)p.W[k], wave, lane);
        __syncthreads();   // every wave has read the tile
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = lg + 4 * r;
            Ga[rr * ldg + col] = m0 + rr < p.rows ? acc[r] * dsilu64(z[r]) : 0.0;
        }
        __syncthreads();
    }
    d4 acc[NCBF];   // first layer: dE/drho = zbar_0 W_0
#pragma unroll
    for (int cb = 0; cb < NCBF; ++cb)
        acc[cb] = layer64<H / kKC64, NBF>(Ga, ldg, (const double *)p.W[0], wave + NW * cb, lane);
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCBF; ++cb) {
        const int f = col + H * cb;
        if (f >= F) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) Ga[(lg + 4 * r) * ldg + f] = acc[cb][r];
    }
    __syncthreads();
    if constexpr (L == 0) {   // the radial form: dE/dS = dE/dx
        for (int it = tid; it < kBM64 * K; it += NT) {
            const int r = it / K, f = it % K;
            if (m0 + r < p.rows) p.C[(m0 + r) * K + f] = Ga[r * ldg + f];
        }
    } else {
        // density adjoint: dE/dS[lambda][a] = w_lambda sum_b M_l[a][b] S[lambda][b], M_l the symmetric
        // matrix of dE/drho[l], doubled on the diagonal; one task per (row, lambda, 4 channels a)
        for (int it = tid; it < kBM64 * NL * (K / 4); it += NT) {
            const int r = it & 15, rest = it >> 4, lam = rest % NL, a0 = rest / NL * 4;
            const int64_t row = m0 + r;
            if (row >= p.rows) continue;
            const int l = lam == 0 ? 0 : (lam < 4 ? 1 : 2);
            const double wl = (lam == 5 || lam == 6 || lam == 8) ? 2.0 : 1.0;   // lambda_weight
            const double *M = Ga + r * ldg + l * P, *sl = Ssh + r * lds + lam * K;
            double s[K], out[4];
#pragma unroll
            for (int b = 0; b < K; ++b) s[b] = sl[b];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = a0 + j, rowa = a * K - a * (a - 1) / 2 - a;   // (a, b >= a) at rowa + b
                double t = 0.0;
#pragma unroll
                for (int b = 0; b < K; ++b) {
                    const double m = M[b < a ? b * K - b * (b - 1) / 2 - b + a : rowa + b];
                    t += (a == b ? 2.0 * m : m) * s[b];
                }
                out[j] = wl * t;
            }
            d2 *C = reinterpret_cast<d2 *>(p.C + row * NLK + lam * K + a0);
            C[0] = d2{out[0], out[1]};
            C[1] = d2{out[2], out[3]};
        }
    }
}

__device__ __forceinline__ int segment64(const FusedMultiT<double> &pm) {
    int s = 0;
    while (s + 1 < pm.n && (int64_t)blockIdx.x >= pm.tile0[s + 1]) ++s;
    return s;
}
template <int H, int L, int K> __global__ __launch_bounds__(4 * H) void k_mlp64_fwd(FusedMultiT<double> pm) {
    const int s = segment64(pm);
    fwd64_body<H, L, K>(pm.seg[s], ((int64_t)blockIdx.x - pm.tile0[s]) * kBM64);
}
template <int H, int L, int K> __global__ __launch_bounds__(4 * H) void k_mlp64_bwd(FusedMultiT<double> pm) {
    const int s = segment64(pm);
    bwd64_body<H, L, K>(pm.seg[s], ((int64_t)blockIdx.x - pm.tile0[s]) * kBM64);
}

// block (x, matrix, NN)
__global__ void k_pack64(Pack64 pk, const double *__restrict__ src, double *__restrict__ dst) {
    const Pack64Matrix m = pk.m[blockIdx.y];
    const int nblk = (m.rows + 15) / 16, nck = (m.cols + kKC64 - 1) / kKC64;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nblk * nck * 128) return;
    const int e = (int)(t & 1), l = (int)(t >> 1 & 63);
    const int64_t frag = t >> 7;
    const int r = (int)(frag % nblk) * 16 + l % 16, c = (int)(frag / nblk) * kKC64 + 2 * (l / 16) + e;
    const double *W = src + blockIdx.z * pk.src_stride + m.src;
    dst[blockIdx.z * pk.dst_stride + m.dst + t] =
        r < m.rows && c < m.cols ? W[(int64_t)r * m.ld_row + (int64_t)c * m.ld_col] : 0.0;
}

template <int H> bool launch_lk(hipStream_t st, bool fwd, unsigned tiles, const FusedMultiT<double> &pm) {
    const int L = pm.seg[0].L, K = pm.seg[0].K;
#define MLP64(LL, KK)                                                                                         \
    if (L == LL && K == KK) {                                                                                 \
        if (fwd) hipLaunchKernelGGL((k_mlp64_fwd<H, LL, KK>), dim3(tiles), dim3(4 * H), 0, st, pm);           \
        else hipLaunchKernelGGL((k_mlp64_bwd<H, LL, KK>), dim3(tiles), dim3(4 * H), 0, st, pm);               \
        return true;                                                                                          \
    }
    MLP64(2, 12) MLP64(2, 8) MLP64(2, 4) MLP64(1, 4) MLP64(0, 12) MLP64(0, 8)
#undef MLP64
    return false;
}

}  // namespace

bool fused64_ok(int L, int K, int F, int H, int nh) {
    const bool lk = (L == 2 && (K == 12 || K == 8 || K == 4)) || (L == 1 && K == 4) || (L == 0 && (K == 12 || K == 8));
    return lk && F == fused_features(L, K) && fused_nn_ok(F, H, nh, K, n_lambda(L) * K);
}

size_t packed64_elems(int rows, int cols) {
    return (size_t)((rows + 15) / 16 * 16) * (size_t)((cols + kKC64 - 1) / kKC64 * kKC64);
}

void pack_operands64(hipStream_t st, const Pack64 &pk, int count, const double *src, double *dst) {
    size_t most = 0;
    for (int k = 0; k < pk.n; ++k) most = std::max(most, packed64_elems(pk.m[k].rows, pk.m[k].cols));
    hipLaunchKernelGGL(k_pack64, dim3(grid_for(most, 256), pk.n, count), dim3(256), 0, st, pk, src, dst);
    LAUNCH_OK("k_pack64");
}

int mlp64_segments(hipStream_t st, bool fwd, const FusedNN64 *segs, int nseg) {
    int launches = 0;
    for (int s0 = 0; s0 < nseg; s0 += kFuseMaxSeg) {
        FusedMultiT<double> pm{};
        pm.n = std::min(kFuseMaxSeg, nseg - s0);
        const FusedNN64 &p = segs[s0];
        if (!fused64_ok(p.L, p.K, p.F, p.H, p.nh) || (p.dout != p.K && p.dout != 1))
            fail(REANN_E_DEVICE, "mlp64: unsupported layer shape");
        int64_t tiles = 0;
        for (int s = 0; s < pm.n; ++s) {
            const FusedNN64 &q = segs[s0 + s];
            if (q.F != p.F || q.H != p.H || q.nh != p.nh || q.dout != p.dout || q.L != p.L || q.K != p.K)
                fail(REANN_E_DEVICE, "mlp64: segments of different shapes");
            pm.seg[s] = q;
            pm.tile0[s] = tiles;
            tiles += (q.rows + kBM64 - 1) / kBM64;
        }
        pm.tile0[pm.n] = tiles;
        const bool ok = p.H == 128 ? launch_lk<128>(st, fwd, (unsigned)tiles, pm) : launch_lk<64>(st, fwd, (unsigned)tiles, pm);
        if (!ok) fail(REANN_E_DEVICE, "mlp64: no kernel compiled for this (L, K)");
        LAUNCH_OK(fwd ? "k_mlp64_fwd" : "k_mlp64_bwd");
        ++launches;
    }
    return launches;
}

}  // namespace reann
