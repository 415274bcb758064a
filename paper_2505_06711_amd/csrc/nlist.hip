// GPU neighbour-list build for the subdomain-extended system.
//
// Every FP64 position operation here is written without contraction so that the pair
// predicate is exactly  d = y_j - w_i,  fma(dz,dz, fma(dy,dy, dx*dx)) < (r_c+skin)^2,
// with w the wrapped position and y = w + shift*L the copy position.
#include "nlist.hpp"

#include <cstring>

#include <algorithm>
#include <cmath>

#pragma clang fp contract(off)

namespace reann {

// ------------------------------------------------------------------ geometry --

void geom_init(Geom &g, const double cell[9], const int32_t pbc[3], const int32_t P[3], double r_c, double skin) {
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            if (a != b && cell[3 * a + b] != 0.0) fail(REANN_E_UNSUPPORTED, "only orthorhombic cells are supported");
    g.ndom = 1;
    for (int a = 0; a < 3; ++a) {
        g.L[a] = cell[4 * a];
        g.per[a] = pbc[a] ? 1 : 0;
        g.P[a] = P ? (P[a] > 0 ? P[a] : 1) : 1;
        if (g.P[a] > kMaxSplit) fail(REANN_E_UNSUPPORTED, "at most 16 subdomains per axis");
        if (!g.per[a] && g.P[a] != 1) fail(REANN_E_INVALID, "a non-periodic axis cannot be split");
        if (g.per[a] && !(g.L[a] > 0.0 && std::isfinite(g.L[a]))) fail(REANN_E_INVALID, "periodic cell length must be > 0");
        g.ndom *= g.P[a];
        if (g.per[a]) {
            double h = g.L[a] / g.P[a];
            for (int k = 0; k < g.P[a]; ++k) {
                g.lo[a][k] = k * h;
                g.hi[a][k] = (k == g.P[a] - 1) ? g.L[a] : (k + 1) * h;
            }
        } else {
            g.lo[a][0] = -INFINITY;
            g.hi[a][0] = INFINITY;
        }
    }
    g.rcut = r_c + skin;
    g.rc2 = g.rcut * g.rcut;
    g.shell = g.rcut + 1e-6;
    for (int a = 0; a < 3; ++a) g.nm[a] = g.per[a] ? (int)std::floor(g.shell / g.L[a]) + 1 : 0;
}

__device__ inline double wrap_coord(double x, double L, int &qe) {
    double q = floor(x / L);
    double t = q * L;
    double w = x - t;
    int k = (int)q;
    if (w < 0.0) { w = w + L; k -= 1; }
    if (w >= L) { w = w - L; k += 1; }
    qe = k;
    return w;
}

// Domains along axis a whose shell contains coordinate y: bitmask (P <= 16).
__device__ inline unsigned axis_domains(const Geom &g, int a, double y) {
    if (!g.per[a]) return 1u;
    unsigned m = 0;
    for (int k = 0; k < g.P[a]; ++k)
        if (y >= g.lo[a][k] - g.shell && y < g.hi[a][k] + g.shell) m |= 1u << k;
    return m;
}

__global__ void k_wrap_count(Geom g, int64_t n, const double *__restrict__ pos, double *__restrict__ w,
                             int32_t *__restrict__ q, int32_t *__restrict__ dom, int64_t *__restrict__ gcount,
                             int32_t *__restrict__ bad) {
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    int c[3];
    double wu[3];
    bool finite = true;
    for (int a = 0; a < 3; ++a) finite = finite && isfinite(pos[3 * u + a]) && fabs(pos[3 * u + a]) < 1e9;
    if (!finite) {
        // flagged for the host; the atom gets no copies so every offset stays in range
        atomicOr(bad, 1);
        for (int a = 0; a < 3; ++a) { w[3 * u + a] = 0.0; q[3 * u + a] = 0; }
        dom[u] = 0;
        gcount[u] = 0;
        return;
    }
    for (int a = 0; a < 3; ++a) {
        double x = pos[3 * u + a];
        int qe = 0;
        double ww = g.per[a] ? wrap_coord(x, g.L[a], qe) : x;
        wu[a] = ww;
        w[3 * u + a] = ww;
        q[3 * u + a] = qe;
        c[a] = 0;
        for (int k = 0; k < g.P[a]; ++k)
            if (ww >= g.lo[a][k] && ww < g.hi[a][k]) c[a] = k;
    }
    dom[u] = (c[0] * g.P[1] + c[1]) * g.P[2] + c[2];
    // copies = (shift, subdomain) combinations whose shell holds the shifted atom, less the atom
    // itself in its own subdomain; the axes are independent, so the count is a product
    int64_t cnt = 1;
    for (int a = 0; a < 3; ++a) {
        int k = 0;
        for (int s = -g.nm[a]; s <= g.nm[a]; ++s)
            k += __popc(axis_domains(g, a, g.per[a] ? wu[a] + (double)s * g.L[a] : wu[a]));
        cnt *= k;
    }
    gcount[u] = cnt - 1;
}

// The copies of every atom in the order (shift, subdomain), from goff[u]; each axis' shift is
// tested before the axes inside it, so an atom far from every boundary tests few of them.  The
// same launch clears the key counts (count[0 .. ncount)).
__global__ void k_ghost_gen(Geom g, int64_t n, const double *__restrict__ w, const int32_t *__restrict__ dom,
                            const int64_t *__restrict__ goff, int32_t *__restrict__ g_owner, int32_t *__restrict__ g_shift,
                            int32_t *__restrict__ g_dom, double *__restrict__ g_pos, int32_t *__restrict__ count,
                            int64_t ncount) {
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u < ncount) count[u] = 0;
    if (u >= n) return;
    int64_t o = goff[u];
    if (goff[u + 1] == o) return;   // no copies (also the case of a flagged atom)
    const double wu[3] = {w[3 * u], w[3 * u + 1], w[3 * u + 2]};
    const int own = dom[u];
    auto at = [&](int a, int s) { return g.per[a] ? wu[a] + (double)s * g.L[a] : wu[a]; };
    for (int s0 = -g.nm[0]; s0 <= g.nm[0]; ++s0) {
        const double y0 = at(0, s0);
        const unsigned m0 = axis_domains(g, 0, y0);
        if (!m0) continue;
        for (int s1 = -g.nm[1]; s1 <= g.nm[1]; ++s1) {
            const double y1 = at(1, s1);
            const unsigned m1 = axis_domains(g, 1, y1);
            if (!m1) continue;
            for (int s2 = -g.nm[2]; s2 <= g.nm[2]; ++s2) {
                const double y2 = at(2, s2);
                const unsigned m2 = axis_domains(g, 2, y2);
                for (int k0 = 0; k0 < g.P[0]; ++k0) {
                    if (!(m0 >> k0 & 1u)) continue;
                    for (int k1 = 0; k1 < g.P[1]; ++k1) {
                        if (!(m1 >> k1 & 1u)) continue;
                        for (int k2 = 0; k2 < g.P[2]; ++k2) {
                            if (!(m2 >> k2 & 1u)) continue;
                            int p = (k0 * g.P[1] + k1) * g.P[2] + k2;
                            if (s0 == 0 && s1 == 0 && s2 == 0 && p == own) continue;
                            g_owner[o] = (int32_t)u;
                            g_shift[3 * o] = s0; g_shift[3 * o + 1] = s1; g_shift[3 * o + 2] = s2;
                            g_dom[o] = p;
                            g_pos[3 * o] = y0; g_pos[3 * o + 1] = y1; g_pos[3 * o + 2] = y2;
                            ++o;
                        }
                    }
                }
            }
        }
    }
}

struct Bins {
    double mn[3], bs[3];
    int nb[3];
    int64_t nbin;
};

__device__ inline int bin_of(const Bins &b, const double *y) {
    int c[3];
    for (int a = 0; a < 3; ++a) {
        int k = (int)((y[a] - b.mn[a]) / b.bs[a]);
        c[a] = k < 0 ? 0 : (k >= b.nb[a] ? b.nb[a] - 1 : k);
    }
    return (c[0] * b.nb[1] + c[1]) * b.nb[2] + c[2];
}

// Key of a pre-ext element: locals (slot = species) then ghosts (slot = n_species, or with
// ghosts_by_species n_species + the owner's species).
__global__ void k_keys(Bins b, int ndom, int n_species, int64_t n, int64_t n_gh, const double *__restrict__ w,
                       const int32_t *__restrict__ dom, const int32_t *__restrict__ species, const double *__restrict__ g_pos,
                       const int32_t *__restrict__ g_dom, const int32_t *__restrict__ g_owner, int ghosts_by_species,
                       int64_t *__restrict__ key, int32_t *__restrict__ count) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n + n_gh) return;
    int slot, p;
    int bn;
    if (e < n) {
        slot = species[e]; p = dom[e]; bn = bin_of(b, w + 3 * e);
    } else {
        int64_t gi = e - n;
        slot = n_species + (ghosts_by_species ? species[g_owner[gi]] : 0);
        p = g_dom[gi];
        bn = bin_of(b, g_pos + 3 * gi);
    }
    int64_t k = ((int64_t)slot * ndom + p) * b.nbin + bn;
    key[e] = k;
    atomicAdd(&count[k], 1);
}

__global__ void k_scatter(int64_t m, const int64_t *__restrict__ key, const int64_t *__restrict__ kstart,
                          int32_t *__restrict__ cursor, int32_t *__restrict__ order) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= m) return;
    int64_t k = key[e];
    int64_t pos = kstart[k] + atomicAdd(&cursor[k], 1);
    order[pos] = (int32_t)e;
}

// Sort each segment [start[k], start[k+1]) of distinct values ascending.  One wave per
// segment: every value's rank is the number of smaller values in the segment, taken against
// an LDS copy; a segment longer than kSegLds is sorted by one lane (insertion sort) instead.
constexpr int kSegLds = 1024;

__global__ __launch_bounds__(256) void k_sort_segments(int64_t nseg, const int64_t *__restrict__ start,
                                                       int32_t *__restrict__ v) {
    __shared__ int32_t sv[4][kSegLds];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t k = (int64_t)blockIdx.x * 4 + w;
    const bool valid = k < nseg;
    const int64_t a = valid ? start[k] : 0;
    const int m = valid ? (int)(start[k + 1] - a) : 0;
    const bool in_lds = m <= kSegLds;
    if (in_lds)
        for (int e = lane; e < m; e += 64) sv[w][e] = v[a + e];
    __syncthreads();
    if (in_lds) {
        for (int e = lane; e < m; e += 64) {
            const int32_t x = sv[w][e];
            int rank = 0;
            for (int q = 0; q < m; ++q) rank += sv[w][q] < x;
            v[a + rank] = x;
        }
    } else if (lane == 0) {
        for (int64_t i = a + 1; i < a + m; ++i) {
            const int32_t x = v[i];
            int64_t j = i - 1;
            while (j >= a && v[j] > x) { v[j + 1] = v[j]; --j; }
            v[j + 1] = x;
        }
    }
}

// rev[f] for the entry f = (x -> j) of a sorted list: the slot of (j -> x) in row j.  Every
// entry has one: rows of locals list every ext atom in range, rows of ghosts every local in
// range, and a row of a ghost only holds locals.  Each pair is resolved once, from its entry
// with x < j (a binary search for x in row j), which writes both slots; rev starts at -1 (k_rows), and
// k_reverse_check then sets *bad if a slot was not written (an entry without its reverse).
__global__ void k_reverse(int64_t n_ext, const int64_t *__restrict__ row, const int32_t *__restrict__ col,
                          int32_t *__restrict__ rev, int32_t *__restrict__ bad) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t x = t >> 4;
    const int g = (int)(t & 15);
    if (x >= n_ext) return;
    const int64_t hi = row[x + 1];
    for (int64_t f = row[x] + g; f < hi; f += 16) {
        const int32_t j = col[f];
        if (j < x) continue;   // resolved from (j -> x)
        int64_t a = row[j], b = row[j + 1];
        const int64_t end = b;
        while (a < b) {
            const int64_t mid = (a + b) >> 1;
            if (col[mid] < x) a = mid + 1;
            else b = mid;
        }
        if (a < end && col[a] == (int32_t)x) {
            rev[f] = (int32_t)a;
            rev[a] = (int32_t)f;
        } else {
            atomicOr(bad, 1);
        }
    }
}

__global__ void k_reverse_check(int64_t n_pairs, const int32_t *__restrict__ rev, int32_t *__restrict__ bad) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f < n_pairs && rev[f] < 0) atomicOr(bad, 1);
}

// The ext atoms in key order.  An owner's ghost copies were generated one after another (goff),
// so its copy list is that range, with each copy's final ghost index at its place.
__global__ void k_build_ext(Bins b, int64_t n, int64_t n_ext, const int32_t *__restrict__ order,
                            const double *__restrict__ pos, const double *__restrict__ w,
                            const int32_t *__restrict__ dom, const int32_t *__restrict__ species,
                            const int64_t *__restrict__ goff, const double *__restrict__ g_pos,
                            const int32_t *__restrict__ g_dom, const int32_t *__restrict__ g_owner_user,
                            const int32_t *__restrict__ g_shift_in, int32_t *__restrict__ perm,
                            int32_t *__restrict__ inv_perm, double *__restrict__ pext, int32_t *__restrict__ dom_ext,
                            int32_t *__restrict__ bin_ext, int8_t *__restrict__ spec_ext,
                            int32_t *__restrict__ gh_owner_user, int32_t *__restrict__ gh_shift,
                            int2 *__restrict__ copy_rng, int32_t *__restrict__ copy_idx, double *__restrict__ xref) {
    int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n_ext) return;
    int64_t pre = order[x];
    const double *y;
    if (pre < n) {
        perm[x] = (int32_t)pre;
        inv_perm[pre] = (int32_t)x;
        y = w + 3 * pre;
        dom_ext[x] = dom[pre];
        spec_ext[x] = (int8_t)species[pre];
        copy_rng[x] = make_int2((int)goff[pre], (int)goff[pre + 1]);
        for (int a = 0; a < 3; ++a) xref[3 * x + a] = pos[3 * pre + a];
    } else {
        int64_t gi = pre - n, go = x - n;
        y = g_pos + 3 * gi;
        dom_ext[x] = g_dom[gi];
        int32_t ou = g_owner_user[gi];
        gh_owner_user[go] = ou;
        copy_idx[gi] = (int32_t)go;
        spec_ext[x] = (int8_t)species[ou];
        for (int a = 0; a < 3; ++a) gh_shift[3 * go + a] = g_shift_in[3 * gi + a];
    }
    pext[x] = y[0];
    pext[n_ext + x] = y[1];
    pext[2 * n_ext + x] = y[2];
    bin_ext[x] = bin_of(b, y);
}

// Candidate scan over the 27 bins around atom x of its subdomain.  Locals see every ext atom
// of the subdomain; ghosts see only locals.  Keys number a bin column's bins consecutively, so
// the three bins of a stencil column hold one run of ext atoms: a row's candidates are 9 runs
// per slot.  A half-wave (32 lanes) takes a row; for up to 3 slots at a time (27 runs) its
// lanes read the runs' bounds together, sum their lengths, and then walk the runs end to end,
// 32 candidates a word, so that short runs (small bins, several elements) leave no lanes idle
// and a lane's position loads do not wait for one another.  Runs are in key order and ext atoms
// are numbered in key order, so the row comes out with its columns ascending.  The count pass
// keeps each word's hits (up to cap_words words a row) and the fill replays them; a row with
// more words is measured again by the fill.
//
// Bound by load latency (few rows) and FP64 issue (many).  Before, rows whose keys held under 24
// atoms on average took a thread each and the others a half-wave that walked its runs one bin at
// a time.  Count + fill, before -> now: 3,000-atom water box (8,600 rows) 297 + 187 -> 15 + 20 us;
// 100,800-atom crystal 305 + 161 -> 167 + 140 us; 1.2M-atom water split 2x2x2 (1.68M rows)
// 1,715 + 1,471 -> 1,571 + 1,769 us, the fill now also clearing the reverse slots (a 0.42 GB
// memset before).  Batches whose candidates end before the unrolled words do load no more (with 64
// elements a batch has about 22): a rebuild of 400,000 atoms of 64 elements takes 5,930 us, 6,670 with
// those loads and 6,190 with a thread a row; the 1.2M-atom box 5,920, 6,130 and 6,260.
constexpr int kRowsPerBlk = 8;   // 256 threads, a half-wave per row
constexpr int kRunSlots = 3;     // slots whose runs (9 each) are walked together
constexpr int kRowUnroll = 4;    // words whose positions are loaded together

template <bool FILL>
__global__ __launch_bounds__(256) void k_rows(Bins b, Geom g, int n_species, int n_ghost_slots, int64_t n, int64_t n_ext,
                                              const double *__restrict__ pext, const int32_t *__restrict__ dom_ext,
                                              const int32_t *__restrict__ bin_ext, const int64_t *__restrict__ kstart,
                                              int64_t *__restrict__ rowcnt, const int64_t *__restrict__ row,
                                              int32_t *__restrict__ col, int32_t *__restrict__ rev,
                                              int32_t *__restrict__ coincident, uint32_t *__restrict__ mask,
                                              int32_t *__restrict__ nwords, int cap_words,
                                              const int32_t *__restrict__ gh_owner_user,
                                              const int32_t *__restrict__ inv_perm, int32_t *__restrict__ gh_owner) {
    __shared__ int32_t s_off[kRowsPerBlk][33], s_beg[kRowsPerBlk][32];
    const int hw = threadIdx.x >> 5;
    const int64_t x = (int64_t)blockIdx.x * kRowsPerBlk + hw;
    const int lane = threadIdx.x & 31, half = threadIdx.x & 32;
    if (x >= n_ext) return;   // the whole half-wave
    // a ghost's owner in local numbering (every inv_perm entry is in place by now)
    if (!FILL && lane == 0 && x >= n) gh_owner[x - n] = inv_perm[gh_owner_user[x - n]];
    const double xi = pext[x], yi = pext[n_ext + x], zi = pext[2 * n_ext + x];
    const int p = dom_ext[x];
    const int bx = bin_ext[x];
    const int c2 = bx % b.nb[2], c1 = (bx / b.nb[2]) % b.nb[1], c0 = bx / (b.nb[2] * b.nb[1]);
    const int lo2 = max(c2 - 1, 0), hi2 = min(c2 + 1, b.nb[2] - 1);
    const int nslot = (x < n) ? n_species + n_ghost_slots : n_species;
    uint32_t *mrow = mask + x * cap_words;
    const int nkept = FILL ? nwords[x] : 0;
    const bool replay = FILL && nkept <= cap_words;
    int64_t o = FILL ? row[x] : 0;
    int cnt = 0;
    int q = 0;   // words so far
    // replay: the row's words are read 32 at a time, one per lane, and passed round by shuffles
    uint32_t wbuf = 0;
    int wbase = -32;
    int32_t *off = s_off[hw], *beg = s_beg[hw];
    for (int s0 = 0; s0 < nslot; s0 += kRunSlots) {
        // lane r: run r of the batch (slot s0 + r / 9, column r % 9), its first atom and length
        const int sl = s0 + lane / 9, dd = lane % 9;
        const int a0 = c0 + dd / 3 - 1, a1 = c1 + dd % 3 - 1;
        int first = 0, len = 0;
        if (lane < 9 * kRunSlots && sl < nslot && a0 >= 0 && a0 < b.nb[0] && a1 >= 0 && a1 < b.nb[1]) {
            const int64_t k = ((int64_t)sl * g.ndom + p) * b.nbin + ((int64_t)a0 * b.nb[1] + a1) * b.nb[2];
            first = (int)kstart[k + lo2];
            len = (int)(kstart[k + hi2 + 1] - first);
        }
        int end = len;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const int t = __shfl_up(end, d, 32);
            if (lane >= d) end += t;
        }
        const int total = __shfl(end, 31, 32);
        // the half-wave's own table (LDS accesses of a wave complete in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        off[lane + 1] = end;
        if (lane == 0) off[0] = 0;
        beg[lane] = first;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int r = 0;   // run of this lane's candidate
        auto atom = [&](int c) -> int {   // c < total, not below the last one asked for
            while (c >= off[r + 1]) ++r;
            return beg[r] + (c - off[r]);
        };
        if (replay) {
            for (int w0 = 0; w0 < total; w0 += 32, ++q) {
                if (q >= wbase + 32) {
                    wbase = q;
                    wbuf = q + lane < nkept ? mrow[q + lane] : 0u;
                }
                const uint32_t bits = (uint32_t)__shfl((int)wbuf, q - wbase, 32);
                if ((bits >> lane) & 1u) {
                    const int64_t d = o + __popc(bits & ((1u << lane) - 1u));
                    col[d] = atom(w0 + lane);
                    rev[d] = -1;   // not resolved yet
                }
                o += __popc(bits);
            }
            continue;
        }
        for (int w0 = 0; w0 < total; w0 += 32 * kRowUnroll) {
            int e[kRowUnroll];
            double ex[kRowUnroll], ey[kRowUnroll], ez[kRowUnroll];
#pragma unroll
            for (int u = 0; u < kRowUnroll; ++u) {
                if (w0 + 32 * u >= total) break;   // uniform over the half-wave
                const int c = w0 + 32 * u + lane;
                e[u] = c < total ? atom(c) : (int)x;   // past the end: the atom itself, never a hit
            }
#pragma unroll
            for (int u = 0; u < kRowUnroll; ++u) {
                if (w0 + 32 * u >= total) break;
                ex[u] = pext[e[u]]; ey[u] = pext[n_ext + e[u]]; ez[u] = pext[2 * n_ext + e[u]];
            }
#pragma unroll
            for (int u = 0; u < kRowUnroll; ++u) {
                if (w0 + 32 * u >= total) break;
                const double dx = ex[u] - xi, dy = ey[u] - yi, dz = ez[u] - zi;
                const double dd2 = fma(dz, dz, fma(dy, dy, dx * dx));
                const bool hit = e[u] != (int)x && dd2 < g.rc2;
                // two copies closer than 1e-6 A: the pair direction is undefined
                if (!FILL && e[u] != (int)x && dd2 < 1e-12) atomicOr(coincident, 1);
                const uint32_t bits = (uint32_t)(__ballot(hit) >> half);
                if (FILL) {
                    if (hit) {
                        const int64_t d = o + __popc(bits & ((1u << lane) - 1u));
                        col[d] = e[u];
                        rev[d] = -1;
                    }
                    o += __popc(bits);
                } else {
                    cnt += __popc(bits);
                    if (lane == 0 && q < cap_words) mrow[q] = bits;
                }
                ++q;
            }
        }
    }
    if (!FILL && lane == 0) {
        rowcnt[x] = cnt;
        nwords[x] = q;
    }
}

// Bounds of the wrapped positions (needed along open axes only): per-block minima and maxima of
// the three coordinates over a grid-strided share of the atoms (stride = blocks x 256), then
// one block combines the blocks' values.  Min and max do not depend on the order.
constexpr int kMinmaxBlocks = 256;

__global__ __launch_bounds__(256) void k_minmax_part(int64_t n, const double *__restrict__ w, double *__restrict__ part) {
    __shared__ double smin[3][256], smax[3][256];
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        for (int a = 0; a < 3; ++a) {
            double v = w[3 * i + a];
            mn[a] = fmin(mn[a], v);
            mx[a] = fmax(mx[a], v);
        }
    for (int a = 0; a < 3; ++a) { smin[a][threadIdx.x] = mn[a]; smax[a][threadIdx.x] = mx[a]; }
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) {
                smin[a][threadIdx.x] = fmin(smin[a][threadIdx.x], smin[a][threadIdx.x + s]);
                smax[a][threadIdx.x] = fmax(smax[a][threadIdx.x], smax[a][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; ++a) { part[6 * blockIdx.x + a] = smin[a][0]; part[6 * blockIdx.x + 3 + a] = smax[a][0]; }
}

__global__ __launch_bounds__(256) void k_minmax(int nb, const double *__restrict__ part, double *__restrict__ out) {
    __shared__ double smin[3][256], smax[3][256];
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += 256)
        for (int a = 0; a < 3; ++a) {
            mn[a] = fmin(mn[a], part[6 * b + a]);
            mx[a] = fmax(mx[a], part[6 * b + 3 + a]);
        }
    for (int a = 0; a < 3; ++a) { smin[a][threadIdx.x] = mn[a]; smax[a][threadIdx.x] = mx[a]; }
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) {
                smin[a][threadIdx.x] = fmin(smin[a][threadIdx.x], smin[a][threadIdx.x + s]);
                smax[a][threadIdx.x] = fmax(smax[a][threadIdx.x], smax[a][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; ++a) { out[a] = smin[a][0]; out[3 + a] = smax[a][0]; }
}

// ---------------------------------------------------------------------- scan --

// Exclusive scans of n counts (32- or 64-bit) into 64-bit offsets out[0 .. n], out[n] = total
// (in and out may be the same array).  A thread takes kScanItems consecutive counts; the
// block's threads are combined by shuffles and one LDS word per wave.  zero_in clears the
// counts behind the scan (they are used as cursors next).
constexpr int kScanThreads = 1024, kScanItems = 4, kScanTile = kScanThreads * kScanItems;

// Exclusive prefix of v over the block (kScanThreads threads); total receives the block's sum.
__device__ inline int64_t block_exclusive(int64_t v, int64_t &total) {
    __shared__ int64_t s_wave[kScanThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    __syncthreads();   // the previous call's readers are done
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    int64_t before = 0, sum = 0;
    for (int q = 0; q < kScanThreads / 64; ++q) {
        const int64_t t = s_wave[q];
        if (q < w) before += t;
        sum += t;
    }
    total = sum;
    return before + inc - v;
}

template <typename In>
__device__ inline int64_t scan_tile(const In *in, int64_t *out, int64_t n, int64_t base, int64_t carry, In *zero_in) {
    int64_t v[kScanItems], mine = 0;
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
        v[u] = i0 + u < n ? (int64_t)in[i0 + u] : 0;
        mine += v[u];
    }
    int64_t total;
    int64_t o = carry + block_exclusive(mine, total);
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
        if (i0 + u < n) {
            out[i0 + u] = o;
            if (zero_in) zero_in[i0 + u] = In(0);
        }
        o += v[u];
    }
    return total;
}

// the whole scan in one block, tile after tile
template <typename In>
__global__ __launch_bounds__(kScanThreads) void k_scan_one(const In *in, int64_t *out, int64_t n, In *zero_in) {
    int64_t carry = 0;
    for (int64_t base = 0; base < n; base += kScanTile) carry += scan_tile(in, out, n, base, carry, zero_in);
    if (threadIdx.x == 0) out[n] = carry;
}

// one tile per block, its sum to sums[block]; k_scan_add then adds the scanned sums
template <typename In>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const In *in, int64_t *out, int64_t n, In *zero_in,
                                                             int64_t *__restrict__ sums) {
    const int64_t total = scan_tile(in, out, n, (int64_t)blockIdx.x * kScanTile, (int64_t)0, zero_in);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(int64_t *__restrict__ out, int64_t n,
                                                           const int64_t *__restrict__ sums) {
    const int64_t add = sums[blockIdx.x];
    const int64_t i0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
        const int64_t i = i0 + u * kScanThreads;
        if (i < n) out[i] += add;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = sums[gridDim.x];
}

// Up to kScanOne counts take one block (a tile is about 1 us, a launch about 3 us with its gap;
// the 8,600 rows of a 3,000-atom box take 5.4 us in one block, 11 us in three launches), more take
// the three launches.  Enqueued only: the total stays on the device.
constexpr int64_t kScanOne = 4 * kScanTile;

template <typename In>
static void scan_exclusive_async(hipStream_t st, const In *in, int64_t *out, int64_t n, DevBuf &tmp,
                                 In *zero_in = nullptr) {
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one<In>, dim3(1), dim3(kScanThreads), 0, st, in, out, n, zero_in);
        LAUNCH_OK("k_scan_one");
        return;
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    int64_t *sums = static_cast<int64_t *>(tmp.ensure((size_t)(nb + 1) * sizeof(int64_t)));
    hipLaunchKernelGGL(k_scan_tiles<In>, dim3((unsigned)nb), dim3(kScanThreads), 0, st, in, out, n, zero_in, sums);
    LAUNCH_OK("k_scan_tiles");
    hipLaunchKernelGGL(k_scan_one<int64_t>, dim3(1), dim3(kScanThreads), 0, st, sums, sums, nb, (int64_t *)nullptr);
    LAUNCH_OK("k_scan_one");
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, st, out, n, sums);
    LAUNCH_OK("k_scan_add");
}

// Scattered device scalars the host needs (counts for allocation sizes, bounds, check flags),
// gathered by one tiny kernel into one block of pinned host memory and read after one wait for
// the stream (behind other streams' work sharing a hardware queue a wait can take far longer
// than the work itself).
constexpr int kPickMax = 160;
struct Pick {
    const void *p[kPickMax];
    int8_t is32[kPickMax];   // 1: int32 (sign-extended); 0: eight bytes (int64, or a double's bits)
    int n;
};

__global__ void k_pick(Pick pk, int64_t *__restrict__ out) {
    for (int t = threadIdx.x; t < pk.n; t += blockDim.x)
        out[t] = pk.is32[t] ? (int64_t) * static_cast<const int32_t *>(pk.p[t]) : *static_cast<const int64_t *>(pk.p[t]);
}

struct Picker {
    Pick pk{};
    int add(const void *p, bool is32) {
        if (pk.n >= kPickMax) fail(REANN_E_UNSUPPORTED, "neighbour build: too many values to read back");
        pk.p[pk.n] = p;
        pk.is32[pk.n] = is32 ? 1 : 0;
        return pk.n++;
    }
    // enqueue the gather into pinned memory and wait; the values stay valid until the next read
    const int64_t *read(hipStream_t st, NListScratch &s) {
        if (current_arena()) {   // the allocation-free entry point: no pinned allocation, a copy instead
            int64_t *d = static_cast<int64_t *>(s.chk.ensure(kPickMax * sizeof(int64_t)));
            s.values.resize(kPickMax);
            hipLaunchKernelGGL(k_pick, dim3(1), dim3(128), 0, st, pk, d);
            LAUNCH_OK("k_pick");
            HIP_OK(hipMemcpyAsync(s.values.data(), d, pk.n * sizeof(int64_t), hipMemcpyDeviceToHost, st));
            HIP_OK(hipStreamSynchronize(st));
            return s.values.data();
        }
        int64_t *h = s.pick.get(kPickMax * sizeof(int64_t));
        hipLaunchKernelGGL(k_pick, dim3(1), dim3(128), 0, st, pk, h);
        LAUNCH_OK("k_pick");
        HIP_OK(hipStreamSynchronize(st));
        return h;
    }
};

// --------------------------------------------------------------------- build --

void build_nlist(hipStream_t st, const double *d_pos, const int32_t *d_species, int64_t n, int n_species,
                 const Geom &g, double r_c, double skin, NList &nl, NListScratch &s, bool ghosts_by_species,
                 bool defer_check) {
    if (n <= 0) fail(REANN_E_INVALID, "n must be > 0");
    if (n >= (int64_t)1 << 30) fail(REANN_E_UNSUPPORTED, "too many atoms");
    const int B = 256;
    nl.g = g;
    nl.n = n;
    nl.n_species = n_species;
    nl.skin = skin;
    nl.r_c = r_c;
    double *w = static_cast<double *>(s.a.ensure(n * 3 * sizeof(double)));
    int32_t *q = nl.q.resize(n * 3);
    int32_t *dom = static_cast<int32_t *>(s.b.ensure(n * sizeof(int32_t)));
    int64_t *goff = static_cast<int64_t *>(s.c.ensure((n + 1) * sizeof(int64_t)));
    // check flags: invalid positions, coincident copies, entries without their reverse
    int32_t *flags = static_cast<int32_t *>(s.flag.ensure(64));
    int32_t *bad = flags, *coinc = flags + 1, *asym = flags + 2;
    HIP_OK(hipMemsetAsync(flags, 0, 64, st));
    hipLaunchKernelGGL(k_wrap_count, dim3(grid_for(n, B)), dim3(B), 0, st, g, n, d_pos, w, q, dom, goff, bad);
    LAUNCH_OK("k_wrap_count");
    scan_exclusive_async(st, goff, goff, n, s.m);
    // the bounds of the wrapped locals set the bins along open axes only
    const bool open_axis = !(g.per[0] && g.per[1] && g.per[2]);
    double *d_mm = static_cast<double *>(s.mm.ensure((6 + 6 * kMinmaxBlocks) * sizeof(double)));
    if (open_axis) {
        const int nb = (int)std::min<int64_t>(kMinmaxBlocks, (n + 255) / 256);
        hipLaunchKernelGGL(k_minmax_part, dim3(nb), dim3(256), 0, st, n, w, d_mm + 6);
        LAUNCH_OK("k_minmax_part");
        hipLaunchKernelGGL(k_minmax, dim3(1), dim3(256), 0, st, nb, d_mm + 6, d_mm);
        LAUNCH_OK("k_minmax");
    }
    // first read: ghost count, the invalid-position flag and (open axes) the bounds
    double bb[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t n_gh, any_bad;
    {
        Picker pk;
        pk.add(goff + n, false);
        pk.add(bad, true);
        if (open_axis)
            for (int a = 0; a < 6; ++a) pk.add(d_mm + a, false);
        const int64_t *hv = pk.read(st, s);
        n_gh = hv[0];
        any_bad = hv[1];
        if (open_axis) std::memcpy(bb, hv + 2, sizeof bb);
    }
    check_deferred(s);   // a previous build's deferred check (the wait above covered its copy)
    if (any_bad) fail(REANN_E_INVALID, "positions contain NaN, Inf or |x| >= 1e9");
    if (n + n_gh >= ((int64_t)1 << 31) - 1) fail(REANN_E_UNSUPPORTED, "extended system too large");
    nl.n_gh = n_gh;
    nl.n_ext = n + n_gh;
    const int64_t n_ext = nl.n_ext;

    // spatial bins of size >= r_c + skin over the region holding every copy
    Bins b{};
    b.nbin = 1;
    for (int a = 0; a < 3; ++a) {
        double lo = g.per[a] ? -g.shell : bb[a];
        double hi = g.per[a] ? g.L[a] + g.shell : bb[3 + a];
        double ext = hi - lo;
        if (!(ext >= 0.0 && ext < 1e8)) fail(REANN_E_INVALID, "system extent out of range");
        int nb = (int)std::floor(ext / (g.rcut * 1.000000001));
        nb = std::max(1, std::min(nb, 1024));
        b.nb[a] = nb;
        b.mn[a] = lo;
        b.bs[a] = nb > 1 ? ext / nb : 1.0;
        b.nbin *= nb;
    }
    const int nghs = ghosts_by_species ? n_species : 1;   // ghost key slots
    const int64_t nkeys = (int64_t)(n_species + nghs) * g.ndom * b.nbin;
    if (nkeys > ((int64_t)1 << 28)) fail(REANN_E_UNSUPPORTED, "bin table too large");

    int32_t *g_owner = static_cast<int32_t *>(s.d.ensure((n_gh + 1) * sizeof(int32_t)));
    int32_t *g_shift = static_cast<int32_t *>(s.e.ensure((n_gh + 1) * 3 * sizeof(int32_t)));
    int32_t *g_dom = static_cast<int32_t *>(s.f.ensure((n_gh + 1) * sizeof(int32_t)));
    double *g_pos = static_cast<double *>(s.g.ensure((n_gh + 1) * 3 * sizeof(double)));
    int64_t *key = static_cast<int64_t *>(s.h.ensure(n_ext * sizeof(int64_t)));
    int32_t *cnt32 = static_cast<int32_t *>(s.i.ensure((nkeys + 1) * sizeof(int32_t)));
    int64_t *kstart = static_cast<int64_t *>(s.j.ensure((nkeys + 1) * sizeof(int64_t)));
    hipLaunchKernelGGL(k_ghost_gen, dim3(grid_for(std::max(n, nkeys), B)), dim3(B), 0, st, g, n, w, dom, goff, g_owner,
                       g_shift, g_dom, g_pos, cnt32, nkeys);
    LAUNCH_OK("k_ghost_gen");
    hipLaunchKernelGGL(k_keys, dim3(grid_for(n_ext, B)), dim3(B), 0, st, b, g.ndom, n_species, n, n_gh, w, dom,
                       d_species, g_pos, g_dom, g_owner, ghosts_by_species ? 1 : 0, key, cnt32);
    LAUNCH_OK("k_keys");
    // every ext atom adds one to exactly one key, so the total is n_ext by construction; it is
    // read back (and checked) with the pair count below.  The counts are cleared for the scatter.
    scan_exclusive_async(st, cnt32, kstart, nkeys, s.m, cnt32);
    int32_t *order = static_cast<int32_t *>(s.k.ensure(n_ext * sizeof(int32_t)));
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(n_ext, B)), dim3(B), 0, st, n_ext, key, kstart, cnt32, order);
    LAUNCH_OK("k_scatter");
    hipLaunchKernelGGL(k_sort_segments, dim3(grid_for(nkeys, 4)), dim3(256), 0, st, nkeys, kstart, order);
    LAUNCH_OK("k_sort_segments");

    int32_t *perm = nl.perm.resize(n);
    int32_t *inv_perm = nl.inv_perm.resize(n);
    double *pext = static_cast<double *>(s.l.ensure(3 * n_ext * sizeof(double)));
    int32_t *d_dom_ext = static_cast<int32_t *>(s.dext.ensure(n_ext * sizeof(int32_t)));
    int32_t *d_bin_ext = static_cast<int32_t *>(s.bext.ensure(n_ext * sizeof(int32_t)));
    int32_t *gh_owner_user = static_cast<int32_t *>(s.gou.ensure((n_gh + 1) * sizeof(int32_t)));
    int8_t *spec_ext = nl.spec_ext.resize(n_ext);
    int32_t *gh_shift = nl.gh_shift.resize((n_gh + 1) * 3);
    int32_t *gh_owner = nl.gh_owner.resize(n_gh + 1);
    int2 *copy_rng = nl.copy_rng.resize(n);
    int32_t *copy_idx = nl.copy_idx.resize(n_gh + 1);
    double *xref = nl.xref.resize(n * 3);
    hipLaunchKernelGGL(k_build_ext, dim3(grid_for(n_ext, B)), dim3(B), 0, st, b, n, n_ext, order, d_pos, w, dom,
                       d_species, goff, g_pos, g_dom, g_owner, g_shift, perm, inv_perm, pext, d_dom_ext, d_bin_ext,
                       spec_ext, gh_owner_user, gh_shift, copy_rng, copy_idx, xref);
    LAUNCH_OK("k_build_ext");

    // rows: count (keeping the hits), scan, fill.  A bin holds about n_ext / nbin atoms (a
    // subdomain's atoms fill about its own share of the bins), so a row has about
    // 27 n_ext / nbin candidates; the hits are kept for up to about twice that.
    int64_t *row = nl.row.resize(n_ext + 1);
    const double mean_cand = 27.0 * (double)n_ext / (double)b.nbin;
    const int cap_words = (int)std::min<double>(4096.0, std::ceil(2.0 * mean_cand / 32.0) + 2.0);
    uint32_t *mask = static_cast<uint32_t *>(s.mask.ensure((size_t)n_ext * cap_words * sizeof(uint32_t)));
    int32_t *nkept = static_cast<int32_t *>(s.ncand.ensure((size_t)n_ext * sizeof(int32_t)));
    hipLaunchKernelGGL(k_rows<false>, dim3(grid_for(n_ext, kRowsPerBlk)), dim3(256), 0, st, b, g, n_species, nghs, n,
                       n_ext, pext, d_dom_ext, d_bin_ext, kstart, row, nullptr, nullptr, nullptr, coinc, mask, nkept,
                       cap_words, gh_owner_user, inv_perm, gh_owner);
    LAUNCH_OK("k_rows<count>");
    scan_exclusive_async(st, row, row, n_ext, s.m);
    // second read: pair counts, the key total and the species segments of the locals
    int64_t n_pairs;
    {
        Picker pk;
        pk.add(row + n_ext, false);
        pk.add(row + n, false);
        pk.add(kstart + nkeys, false);
        pk.add(coinc, true);
        for (int sp = 0; sp <= n_species; ++sp) pk.add(kstart + (int64_t)sp * g.ndom * b.nbin, false);
        if (ghosts_by_species)
            for (int sp = 1; sp <= n_species; ++sp) pk.add(kstart + (int64_t)(n_species + sp) * g.ndom * b.nbin, false);
        const int64_t *hv = pk.read(st, s);
        n_pairs = hv[0];
        if (hv[2] != n_ext) fail(REANN_E_DEVICE, "neighbour build: key count mismatch");
        if (hv[3]) fail(REANN_E_INVALID, "two atoms (or an atom and a periodic copy) closer than 1e-6 A");
        nl.n_local_pairs = hv[1];
        nl.seg.assign(hv + 4, hv + 4 + n_species + 1);
        // ghost species segments: [gseg[s], gseg[s+1]) are the ghosts of element s
        // (ghosts_by_species), else one segment of every ghost
        if (ghosts_by_species) {
            nl.gseg.assign(1, n);
            nl.gseg.insert(nl.gseg.end(), hv + 4 + n_species + 1, hv + 4 + 2 * n_species + 1);
        } else {
            nl.gseg = {n, n_ext};
        }
    }
    if (nl.gseg.back() != n_ext) fail(REANN_E_DEVICE, "neighbour build: ghost segments mismatch");
    if (nl.seg[n_species] != n) fail(REANN_E_DEVICE, "neighbour build: species segments mismatch");
    if (n_pairs >= ((int64_t)1 << 31) - 1) fail(REANN_E_UNSUPPORTED, "too many neighbour pairs");
    nl.n_pairs = n_pairs;
    int32_t *col = nl.col.resize(n_pairs + 1);
    int32_t *rev = nl.rev.resize(n_pairs + 1);
    hipLaunchKernelGGL(k_rows<true>, dim3(grid_for(n_ext, kRowsPerBlk)), dim3(256), 0, st, b, g, n_species, nghs, n,
                       n_ext, pext, d_dom_ext, d_bin_ext, kstart, nullptr, row, col, rev, nullptr, mask, nkept,
                       cap_words, nullptr, nullptr, nullptr);
    LAUNCH_OK("k_rows<fill>");
    // the rows are ascending as filled; the reverse slot of every entry
    hipLaunchKernelGGL(k_reverse, dim3(grid_for(n_ext * 16, B)), dim3(B), 0, st, n_ext, row, col, rev, asym);
    LAUNCH_OK("k_reverse");
    if (n_pairs > 0) {
        hipLaunchKernelGGL(k_reverse_check, dim3(grid_for(n_pairs, B)), dim3(B), 0, st, n_pairs, rev, asym);
        LAUNCH_OK("k_reverse_check");
    }
    // last read (the list is complete when it returns): the symmetry check of the reverse slots
    if (defer_check) {
        HIP_OK(hipMemcpyAsync(s.sym.get(), asym, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        s.sym_pending = true;
        return;
    }
    Picker pk;
    pk.add(asym, true);
    if (pk.read(st, s)[0]) fail(REANN_E_DEVICE, "neighbour build: list is not symmetric");
}

void check_deferred(NListScratch &s) {
    if (!s.sym_pending) return;
    s.sym_pending = false;
    if (*s.sym.get()) fail(REANN_E_DEVICE, "neighbour build: list is not symmetric");
}

// ------------------------------------------------------------ per-step work --

// With disp, the skin check rides along: the largest displacement since the list build.  A block
// raises the maximum only if its own is larger than what it reads there, so that few blocks meet
// at the word.
__global__ __launch_bounds__(256) void k_refresh(Geom g, int64_t n, int64_t n_ext, const double *__restrict__ pos,
                                                 const int32_t *__restrict__ perm, const int32_t *__restrict__ q,
                                                 const int32_t *__restrict__ gh_owner,
                                                 const int32_t *__restrict__ gh_shift, double4 *__restrict__ p4,
                                                 const double *__restrict__ xref, unsigned long long *disp) {
    __shared__ unsigned long long sm[4];
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long d2bits = 0;
    if (x < n_ext) {
        int64_t i = x < n ? x : gh_owner[x - n];
        int64_t u = perm[i];
        double w[3], d2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            double v = pos[3 * u + a];
            if (disp && x < n) {
                const double d = v - xref[3 * x + a];
                d2 += d * d;
            }
            if (g.per[a]) {
                double t = (double)q[3 * u + a] * g.L[a];   // q is stored per caller index
                v = v - t;
            }
            w[a] = v;
        }
        d2bits = (unsigned long long)__double_as_longlong(d2) & 0x7fffffffffffffffull;
        if (x >= n) {
            int64_t gi = x - n;
            for (int a = 0; a < 3; ++a)
                if (g.per[a]) w[a] = w[a] + (double)gh_shift[3 * gi + a] * g.L[a];
        }
        p4[x] = make_double4(w[0], w[1], w[2], 0.0);
    }
    if (!disp) return;   // uniform over the grid
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long t = __shfl_xor(d2bits, o, 64);
        d2bits = t > d2bits ? t : d2bits;
    }
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = d2bits;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < 4; ++v) d2bits = sm[v] > d2bits ? sm[v] : d2bits;
        if (d2bits > __hip_atomic_load(disp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(disp, d2bits);
    }
}

void refresh_positions(hipStream_t st, const NList &nl, const double *d_pos, double4 *p4, unsigned long long *disp) {
    hipLaunchKernelGGL(k_refresh, dim3(grid_for(nl.n_ext, 256)), dim3(256), 0, st, nl.g, nl.n, nl.n_ext, d_pos,
                       nl.perm.ptr(), nl.q.ptr(), nl.gh_owner.ptr(), nl.gh_shift.ptr(), p4, nl.xref.ptr(), disp);
    LAUNCH_OK("k_refresh");
}

__device__ inline double nan_max(double a, double b) { return (b > a || b != b) ? b : a; }

// Per-block maxima of |x_i - xref_i|^2 (NaN counts as too far), then one block combines them.
__global__ void k_maxdisp_part(int64_t n, const double *__restrict__ pos, const int32_t *__restrict__ perm,
                               const double *__restrict__ xref, double *__restrict__ part) {
    __shared__ double sm[256];
    double m = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = perm[i];
        const double dx = pos[3 * u] - xref[3 * i], dy = pos[3 * u + 1] - xref[3 * i + 1],
                     dz = pos[3 * u + 2] - xref[3 * i + 2];
        m = nan_max(m, dx * dx + dy * dy + dz * dz);
    }
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sm[threadIdx.x] = nan_max(sm[threadIdx.x], sm[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sm[0];
}

__global__ void k_maxdisp_final(int nb, const double *__restrict__ part, double *__restrict__ out) {
    __shared__ double sm[256];
    double m = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) m = nan_max(m, part[i]);
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sm[threadIdx.x] = nan_max(sm[threadIdx.x], sm[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sm[0];
}

// d_out must hold 1 + 1024 doubles (result, then per-block partials).
void max_displacement2(hipStream_t st, const NList &nl, const double *d_pos, double *d_out) {
    const int nb = (int)std::min<int64_t>(1024, std::max<int64_t>(1, (nl.n + 255) / 256));
    hipLaunchKernelGGL(k_maxdisp_part, dim3(nb), dim3(256), 0, st, nl.n, d_pos, nl.perm.ptr(), nl.xref.ptr(),
                       d_out + 1);
    LAUNCH_OK("k_maxdisp_part");
    hipLaunchKernelGGL(k_maxdisp_final, dim3(1), dim3(256), 0, st, nb, d_out + 1, d_out);
    LAUNCH_OK("k_maxdisp_final");
}

}  // namespace reann
