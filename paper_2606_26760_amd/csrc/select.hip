// Selection steps around the subspace solve (Sec. 2.2): the classical
// expansion of Eq. 2 (every determinant outside B that H connects to one of
// the largest-|c| determinants of B), the PT2 importance of Eq. 3 (the
// numerator sum_i c_i <x|H|x_i> of a candidate x over B, its diagonal H_xx
// and the score), and a stable top-k over a vector of scores, used both for
// the cold-start ranking by H_xx and for keeping the best-scored candidates.
//
// Both the expansion and the PT2 numerator reach into B only through its
// sorted string tables: alpha groups (distinct alpha strings ua, rows
// ga[g] .. ga[g+1] with ascending beta strings sb) and beta groups (distinct
// beta strings ub, entries gb[g] .. gb[g+1] of the beta-major listing bperm
// with their alpha strings bm_alpha).  A determinant is found by two binary
// searches; every partner of a candidate lies in one of at most
// 2 + na (norb - na) groups, which are scanned, or, for the groups one alpha move
// away, looked up in tables of their members by the candidate's own beta moves.
// Matrix elements follow slater.hpp, with the packed integrals in LDS when they
// fit.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "common.hpp"
#include "slater.hpp"

namespace hinqs {

namespace {

constexpr int EX_NT = 1024; // expansion: one workgroup per chosen determinant at a time
constexpr int PT_NT = 1024; // PT2: one wave per candidate at a time
constexpr int NPAIR32 = 32 * 31 / 2;

struct BTables {
    int32_t nua, nub;
    const uint32_t *ua, *ub;      // distinct strings, ascending
    const uint32_t *sa, *sb;      // strings in sorted order
    const int32_t *ga, *gb;       // group offsets
    const int32_t *bperm;         // beta-major listing of sorted positions
    const uint32_t *bm_alpha;     // alpha string of bperm[u]
};

BTables tables_of(const Ctx &c) {
    return BTables{c.nua, c.nub, c.ua.p, c.ub.p, c.sa.p, c.sb.p, c.ga.p, c.gb.p, c.bperm.p, c.bm_alpha.p};
}

// Index of x in the ascending array v[0..n), or -1.
__device__ inline int32_t find_u32(const uint32_t *v, int32_t n, uint32_t x) {
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (v[mid] < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return (lo < n && v[lo] == x) ? lo : -1;
}

// Sorted position of the determinant (a, b) in B, or -1.
__device__ inline int64_t find_det(const BTables &t, uint32_t a, uint32_t b) {
    const int32_t g = find_u32(t.ua, t.nua, a);
    if (g < 0) return -1;
    const int32_t lo = t.ga[g], hi = t.ga[g + 1];
    const int32_t r = find_u32(t.sb + lo, hi - lo, b);
    return r < 0 ? -1 : (int64_t)lo + r;
}

// Orbital of the n-th set bit (from the lowest) of m; m has more than n bits.
__device__ inline int nth_bit(uint32_t m, int n) {
    for (int i = 0; i < n; ++i) m &= m - 1;
    return lowbit(m);
}

__device__ inline double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Stage the packed integrals and h in LDS (USE_LDS) or point at them.
template <bool USE_LDS>
__device__ inline void stage_integrals(double *smem, const double *eri_g, const double *h_g, int npack, int norb,
                                       const double *&eri, const double *&h) {
    eri = eri_g;
    h = h_g;
    if (USE_LDS) {
        for (int t = threadIdx.x; t < npack; t += blockDim.x) smem[t] = eri_g[t];
        for (int t = threadIdx.x; t < norb * norb; t += blockDim.x) smem[npack + t] = h_g[t];
        __syncthreads();
        eri = smem;
        h = smem + npack;
    }
}

// ------------------------------------------------------------ top-k keys
// Order-preserving unsigned image of a double (ascending values give
// ascending keys; -0 is taken as +0, so equal values tie); with `largest`
// the order is reversed.  NaN raises the flag.
__global__ void k_order_keys(const double *v, int64_t n, bool largest, uint64_t *keys, int32_t *vals,
                             unsigned *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x = v[i];
    if (x != x) atomicOr(bad, 1u);
    if (x == 0.0) x = 0.0;
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    uint64_t k = (b >> 63) ? ~b : (b | 0x8000000000000000ull);
    keys[i] = largest ? ~k : k;
    vals[i] = (int32_t)i;
}

// Keys ordering |c| descending; non-finite c raises the flag.
__global__ void k_mag_keys(const double *c, int64_t n, uint64_t *keys, int32_t *vals, unsigned *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = c[i];
    if (!isfinite(x)) atomicOr(bad, 1u);
    keys[i] = 0x7fffffffffffffffull - (uint64_t)__double_as_longlong(fabs(x));
    vals[i] = (int32_t)i;
}

// top_out[t] = vals[t] (index in the caller's order of the vector); pos[t] =
// its sorted position.
__global__ void k_take_top(const int32_t *vals, int64_t ntop, const int32_t *inv, int32_t *top_out,
                           int32_t *pos) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntop) return;
    const int32_t v = vals[t];
    if (top_out) top_out[t] = v;
    if (pos) pos[t] = inv ? inv[v] : v;
}

// ------------------------------------------------------ classical expansion
struct ExpArgs {
    BTables B;
    int norb, npack, na, nb;
    int64_t ntop;
    const int32_t *pos;  // sorted positions of the chosen determinants
    const double *eri, *h;
    uint64_t *keys;      // ntop * (excitations per determinant) entries
    unsigned long long *count;
};

// Every single and double excitation y of a chosen determinant x, indexed
// r = 0 .. nexc-1 in five ranges: alpha singles, beta singles, alpha-alpha
// doubles, beta-beta doubles, alpha-beta doubles.  y is kept when
// <y|H|x> != 0 and y is not in B; kept keys (alpha << norb | beta) are
// appended with one atomic per workgroup pass (one per wave, on the one
// counter, took 1.1 ms for 1,000 determinants of 5,545 excitations;
// 0.20 ms).
template <bool USE_LDS>
__global__ __launch_bounds__(EX_NT) void k_expand(ExpArgs a) {
    extern __shared__ double smem[];
    __shared__ uint16_t pairs[NPAIR32];      // k = j (j - 1) / 2 + i  ->  i | j << 8, i < j
    __shared__ uint8_t occ[2][32], vir[2][32];
    __shared__ int wcnt[EX_NT / 64];
    __shared__ unsigned long long wbase[EX_NT / 64];
    const double *eri, *h;
    stage_integrals<USE_LDS>(smem, a.eri, a.h, a.npack, a.norb, eri, h);
    for (int k = threadIdx.x; k < NPAIR32; k += blockDim.x) {
        int j = 1;
        while ((j + 1) * j / 2 <= k) ++j;
        pairs[k] = (uint16_t)((k - j * (j - 1) / 2) | (j << 8));
    }
    const int norb = a.norb, na = a.na, nb = a.nb, nva = norb - na, nvb = norb - nb;
    const uint32_t full = norb >= 32 ? 0xffffffffu : ((1u << norb) - 1u);
    const int64_t sA = (int64_t)na * nva, sB = (int64_t)nb * nvb;
    const int64_t cva = (int64_t)nva * (nva - 1) / 2, cvb = (int64_t)nvb * (nvb - 1) / 2;
    const int64_t dAA = (int64_t)na * (na - 1) / 2 * cva, dBB = (int64_t)nb * (nb - 1) / 2 * cvb;
    const int64_t total = sA + sB + dAA + dBB + sA * sB;
    const int lane = threadIdx.x & 63;
    for (int64_t t = blockIdx.x; t < a.ntop; t += gridDim.x) {
        const int32_t p = a.pos[t];
        const uint32_t xa = a.B.sa[p], xb = a.B.sb[p];
        __syncthreads();  // the previous determinant's lists are no longer read
        if (threadIdx.x < 2) {
            const uint32_t s = threadIdx.x == 0 ? xa : xb;
            int no = 0, nv = 0;
            for (int q = 0; q < norb; ++q) {
                if ((s >> q) & 1u)
                    occ[threadIdx.x][no++] = (uint8_t)q;
                else
                    vir[threadIdx.x][nv++] = (uint8_t)q;
            }
        }
        __syncthreads();
        for (int64_t r0 = 0; r0 < total; r0 += EX_NT) {
            int64_t r = r0 + threadIdx.x;
            bool keep = false;
            uint64_t key = 0;
            if (r < total) {
                uint32_t ya = xa, yb = xb;
                if (r < sA) {
                    ya ^= (1u << occ[0][r / nva]) | (1u << vir[0][r % nva]);
                } else if ((r -= sA) < sB) {
                    yb ^= (1u << occ[1][r / nvb]) | (1u << vir[1][r % nvb]);
                } else if ((r -= sB) < dAA) {
                    const int po = pairs[r / cva], pv = pairs[r % cva];
                    ya ^= (1u << occ[0][po & 255]) | (1u << occ[0][po >> 8]) | (1u << vir[0][pv & 255]) |
                          (1u << vir[0][pv >> 8]);
                } else if ((r -= dAA) < dBB) {
                    const int po = pairs[r / cvb], pv = pairs[r % cvb];
                    yb ^= (1u << occ[1][po & 255]) | (1u << occ[1][po >> 8]) | (1u << vir[1][pv & 255]) |
                          (1u << vir[1][pv >> 8]);
                } else {
                    r -= dBB;
                    const int64_t s1 = r / sB, s2 = r % sB;
                    ya ^= (1u << occ[0][s1 / nva]) | (1u << vir[0][s1 % nva]);
                    yb ^= (1u << occ[1][s2 / nvb]) | (1u << vir[1][s2 % nvb]);
                }
                const double v = coupling_value(eri, h, norb, pair_desc(ya, yb, xa, xb), ya, yb);
                if (v != 0.0 && find_det(a.B, ya, yb) < 0) {
                    keep = true;
                    key = ((uint64_t)ya << norb) | (uint64_t)(yb & full);
                }
            }
            const uint64_t m = __ballot(keep);
            if (lane == 0) wcnt[threadIdx.x >> 6] = __popcll(m);
            __syncthreads();
            if (threadIdx.x < 64) {
                const int n = threadIdx.x < EX_NT / 64 ? wcnt[threadIdx.x] : 0;
                int incl = n;
#pragma unroll
                for (int off = 1; off < EX_NT / 64; off <<= 1) {
                    const int x = __shfl_up(incl, off, 64);
                    if (lane >= off) incl += x;
                }
                unsigned long long base = 0;
                if (threadIdx.x == EX_NT / 64 - 1 && incl > 0) base = atomicAdd(a.count, (unsigned long long)incl);
                base = __shfl(base, EX_NT / 64 - 1, 64);
                if (threadIdx.x < EX_NT / 64) wbase[threadIdx.x] = base + (unsigned long long)(incl - n);
            }
            __syncthreads();
            if (keep) a.keys[wbase[threadIdx.x >> 6] + __popcll(m & ((1ull << lane) - 1ull))] = key;
        }
    }
}

__global__ void k_unique_flags(const uint64_t *keys, int64_t n, int32_t *flag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

__global__ void k_unique_write(const uint64_t *keys, const int32_t *flag, const int32_t *pos, int64_t n,
                               int norb, int64_t cap, uint64_t *out_a, uint64_t *out_b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !flag[i]) return;
    const int64_t p = pos[i];
    if (p >= cap) return;
    const uint64_t lo = norb >= 64 ? ~0ull : ((1ull << norb) - 1ull);
    out_a[p] = keys[i] >> norb;
    out_b[p] = keys[i] & lo;
}

// ------------------------------------------------------------------- PT2
struct Pt2Args {
    BTables B;
    int norb, npack, na, nb;
    int alink_max;
    const int32_t *alink_ptr, *alink;  // single alpha moves between strings of B
    double ecore, e0;
    int64_t ncand;
    const uint64_t *ca, *cb;
    const double *cs;  // coefficients in sorted order
    const double *eri, *h;
    double *numer, *hxx, *score;
    unsigned *bad;
    // per candidate in key order: H_xx, and (links done elsewhere) the same-spin numerator
    double *dval, *part;
};

constexpr int SCAN_U = 8;  // group entries in flight per lane

// <x|H|x_j> for strings si (of x) and sj that differ by two electrons of one
// spin, the other spin's string being the same.
__device__ inline double same_spin_double(const double *eri, uint32_t si, uint32_t sj) {
    const uint32_t holes = sj & ~si, parts = si & ~sj;
    const int h1 = lowbit(holes), h2 = highbit(holes), p1 = lowbit(parts), p2 = highbit(parts);
    const double v = eri[eri_index(p1, h1, p2, h2)] - eri[eri_index(p1, h2, p2, h1)];
    return double_parity(sj, h1, h2, p1, p2) ? -v : v;
}

// ... by one electron; other: the string of the other spin.
__device__ inline double same_spin_single(const double *eri, const double *h, int norb, uint32_t si, uint32_t sj,
                                          uint32_t other) {
    const int q = lowbit(sj & ~si), p = lowbit(si & ~sj);
    const double v = single_value(eri, h, norb, p, q, si & sj, other);
    return single_parity(sj, q, p) ? -v : v;
}

// acc += c_j <x|H|x_j> over the members at [lo, hi) of one group that share
// the other spin's string: str their strings of this spin, own that of x, pos
// their place in cs (null: the same, and a member equal to x takes the diagonal
// d).  Doubles and singles are summed in passes of their own: a single costs
// a sum over every electron, which each lane would otherwise wait for at nearly
// every step.
__device__ inline void scan_same_spin(const Pt2Args &a, const double *eri, const double *h, const uint32_t *str,
                                      const int32_t *pos, int32_t lo, int32_t hi, uint32_t own, uint32_t other,
                                      double d, int lane, double &acc) {
    for (int32_t j0 = lo + lane; j0 < hi; j0 += 64 * SCAN_U) {
        uint32_t sj[SCAN_U];
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            const int32_t j = j0 + 64 * u;
            sj[u] = j < hi ? str[j] : ~own;
        }
        uint32_t m2 = 0, m1 = 0, m0 = 0;
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            const int n = popc32(own ^ sj[u]);
            m2 |= n == 4 ? 1u << u : 0u;
            m1 |= n == 2 ? 1u << u : 0u;
            m0 |= n == 0 ? 1u << u : 0u;
        }
        for (; m2; m2 &= m2 - 1) {
            const int32_t j = j0 + 64 * lowbit(m2);
            acc += a.cs[pos ? pos[j] : j] * same_spin_double(eri, own, str[j]);
        }
        for (; m1; m1 &= m1 - 1) {
            const int32_t j = j0 + 64 * lowbit(m1);
            acc += a.cs[pos ? pos[j] : j] * same_spin_single(eri, h, a.norb, own, str[j], other);
        }
        if (m0 && !pos) acc += a.cs[j0 + 64 * lowbit(m0)] * d;
    }
}

// acc += c_j <x|H|x_j> over the rows j in [lo, hi) of the alpha group of aj, one
// move from xa, whose beta string is one move from xb.
__device__ inline void scan_alpha_group(const Pt2Args &a, const double *eri, const double *h, int32_t lo, int32_t hi,
                                        uint32_t xa, uint32_t xb, uint32_t aj, int lane, double &acc) {
    for (int32_t j0 = lo + lane; j0 < hi; j0 += 64 * SCAN_U) {
        uint32_t bj[SCAN_U];
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            const int32_t j = j0 + 64 * u;
            bj[u] = j < hi ? a.B.sb[j] : ~xb;
        }
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) m |= popc32(xb ^ bj[u]) == 2 ? 1u << u : 0u;
        // the hits in ascending order, so every lane sums its entries in group order
        for (; m; m &= m - 1) {
            const int32_t j = j0 + 64 * lowbit(m);
            acc += a.cs[j] * coupling_value(eri, h, a.norb, pair_desc(xa, xb, aj, a.B.sb[j]), xa, xb);
        }
    }
}

// Linked alpha groups of at most PT2_GL * SCAN_U rows are scanned 64 / PT2_GL
// at a time, PT2_GL lanes each and in a single step, so the chain of
// dependent loads per candidate runs over a few batches of groups instead of
// every group one after another.
constexpr int PT2_GL = 32;
constexpr int PT2_SMALL = PT2_GL * SCAN_U;

// acc += c_j <x|H|x_j> over the rows j in [lo, hi) (at most PT2_SMALL of them)
// of one alpha group (alpha string aj) whose beta string is one electron from
// xb; sl is this lane's index among the PT2_GL lanes sharing the group.
__device__ inline void scan_small_group(const Pt2Args &a, const double *eri, const double *h, int32_t lo,
                                        int32_t hi, uint32_t xa, uint32_t xb, uint32_t aj, int sl, double &acc) {
    uint32_t bj[SCAN_U];
#pragma unroll
    for (int u = 0; u < SCAN_U; ++u) {
        const int32_t j = lo + sl + PT2_GL * u;
        bj[u] = j < hi ? a.B.sb[j] : ~xb;
    }
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < SCAN_U; ++u) m |= popc32(xb ^ bj[u]) == 2 ? 1u << u : 0u;
    for (; m; m &= m - 1) {
        const int32_t j = lo + sl + PT2_GL * lowbit(m);
        acc += a.cs[j] * coupling_value(eri, h, a.norb, pair_desc(xa, xb, aj, a.B.sb[j]), xa, xb);
    }
}

// Candidate order for PT2: key (alpha << norb | beta) of each candidate
// (0 for a malformed one; the main kernel checks every candidate itself).
__global__ void k_pt2_keys(const uint64_t *ca, const uint64_t *cb, int64_t n, int norb, uint64_t *keys,
                           int32_t *vals) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const uint64_t a = ca[t], b = cb[t];
    keys[t] = ((a >> norb) | (b >> norb)) ? 0ull : ((a << norb) | b);
    vals[t] = (int32_t)t;
}

// Groups of each candidate (in key order): its alpha group and beta group in
// B, or -1.  One thread per candidate, so the searches overlap.
__global__ void k_pt2_groups(const BTables B, const uint64_t *ca, const uint64_t *cb, const int32_t *order, int64_t n,
                             int norb, int32_t *ga_of, int32_t *gb_of) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const int32_t t = order[u];
    const uint64_t a = ca[t], b = cb[t];
    const bool ok = ((a >> norb) | (b >> norb)) == 0;
    ga_of[u] = ok ? find_u32(B.ua, B.nua, (uint32_t)a) : -1;
    gb_of[u] = ok ? find_u32(B.ub, B.nub, (uint32_t)b) : -1;
}

// H_xx of every candidate, one thread each; malformed candidates get NaN
// outputs and raise the flag.  (With all 64 lanes of a candidate's wave
// computing the same sum this took 5.1 of 21.3 ms on 8.8e5 candidates.)
template <bool USE_LDS>
__global__ __launch_bounds__(256) void k_pt2_diag(Pt2Args a, const int32_t *order) {
    extern __shared__ double smem[];
    const double *eri, *h;
    stage_integrals<USE_LDS>(smem, a.eri, a.h, a.npack, a.norb, eri, h);
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < a.ncand;
         u += (int64_t)gridDim.x * blockDim.x) {
        const int32_t t = order[u];
        const uint64_t a64 = a.ca[t], b64 = a.cb[t];
        if ((a64 >> a.norb) != 0 || (b64 >> a.norb) != 0 || (int)__popcll(a64) != a.na ||
            (int)__popcll(b64) != a.nb) {
            atomicOr(a.bad, 1u);
            const double nan = __longlong_as_double(0x7ff8000000000000ll);
            if (a.numer) a.numer[t] = nan;
            if (a.hxx) a.hxx[t] = nan;
            if (a.score) a.score[t] = nan;
            a.dval[u] = a.part[u] = nan;
            continue;
        }
        const double d = diag_value(eri, h, a.norb, a.ecore, (uint32_t)a64, (uint32_t)b64);
        a.dval[u] = d;
        if (a.hxx) a.hxx[t] = d;
    }
}

// Waves take runs of PT2_RUN consecutive candidates in key order from a
// shared counter (every wave stops once the counter passes ncand), one
// candidate at a time.  Its partners in B fall into three disjoint classes, each read from
// one kind of group:
//   same alpha string        the alpha group of xa (beta differs by 0, 1 or 2)
//   same beta string         the beta group of xb (alpha differs by 1 or 2)
//   one move in each spin    the alpha groups of the strings one move from xa
//                            (link table when xa is an alpha string of B, else
//                            searched), keeping beta strings one move from xb
//                            (LINKS; otherwise k_pt2_links adds this class)
// The diagonal enters through the first class when x lies in B.  Candidates
// of a run mostly share xa, so the bounds of its alpha groups are loaded once
// per distinct xa and kept in the lanes (slot r of lane l: move 64 r + l;
// SLOTS * 64 >= na (norb - na)).
constexpr int PT2_RUN = 16;

template <bool USE_LDS, int SLOTS, bool LINKS>
__global__ __launch_bounds__(PT_NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_pt2(
    Pt2Args a, const int32_t *order, const int32_t *ga_of, const int32_t *gb_of, unsigned long long *next) {
    extern __shared__ double smem[];
    const double *eri, *h;
    stage_integrals<USE_LDS>(smem, a.eri, a.h, a.npack, a.norb, eri, h);
    const int lane = threadIdx.x & 63;
    const int norb = a.norb, nva = norb - a.na, nmov = a.na * nva;
    const uint32_t full = norb >= 32 ? 0xffffffffu : ((1u << norb) - 1u);
    uint32_t cur_a = 0;
    bool have = false;
    int nlink = 0;
    int32_t lo_m[SLOTS], hi_m[SLOTS];
    uint32_t aj_m[SLOTS];
    int64_t u = 0, u_end = 0;
    for (;;) {
        if (u == u_end) {  // next run of PT2_RUN candidates from the shared counter
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(next, (unsigned long long)PT2_RUN);
            base = __shfl(base, 0, 64);
            if ((int64_t)base >= a.ncand) break;
            u = (int64_t)base;
            u_end = min(a.ncand, u + PT2_RUN);
        }
        const int32_t t = order[u];
        const uint64_t a64 = a.ca[t], b64 = a.cb[t];
        const int32_t g = ga_of[u], gbx = gb_of[u];
        const double d = a.dval[u];
        double *const part = LINKS ? nullptr : a.part + u;
        ++u;
        if ((a64 >> norb) != 0 || (b64 >> norb) != 0 || (int)__popcll(a64) != a.na || (int)__popcll(b64) != a.nb)
            continue;
        const uint32_t xa = (uint32_t)a64, xb = (uint32_t)b64;
        if (LINKS && (!have || xa != cur_a)) {  // alpha groups one move from xa
            have = true;
            cur_a = xa;
            nlink = g >= 0 ? a.alink_ptr[g] : nmov;
#pragma unroll
            for (int r = 0; r < SLOTS; ++r) {
                const int m = 64 * r + lane;
                int32_t gm = -1;
                if (m < nlink) {
                    if (g >= 0) {
                        gm = a.alink[(int64_t)g * a.alink_max + m];
                    } else {
                        const uint32_t am =
                            xa ^ (1u << nth_bit(xa, m / nva)) ^ (1u << nth_bit(~xa & full, m % nva));
                        gm = find_u32(a.B.ua, a.B.nua, am);
                    }
                }
                lo_m[r] = gm >= 0 ? a.B.ga[gm] : 0;
                hi_m[r] = gm >= 0 ? a.B.ga[gm + 1] : 0;
                aj_m[r] = gm >= 0 ? a.B.ua[gm] : 0u;
            }
        }
        double acc = 0.0;
        if (g >= 0)
            scan_same_spin(a, eri, h, a.B.sb, nullptr, a.B.ga[g], a.B.ga[g + 1], xb, xa, d, lane, acc);
        if (gbx >= 0)
            scan_same_spin(a, eri, h, a.B.bm_alpha, a.B.bperm, a.B.gb[gbx], a.B.gb[gbx + 1], xa, xb, 0.0, lane, acc);
#pragma unroll
        for (int r = 0; r < (LINKS ? SLOTS : 0); ++r) {
            const int32_t sz = hi_m[r] - lo_m[r];
            uint64_t found = __ballot(sz > PT2_SMALL);  // large groups: the whole wave, one at a time
            while (found) {
                const int src = __builtin_ctzll(found);
                found &= found - 1;
                const int32_t lo = __shfl(lo_m[r], src, 64), hi = __shfl(hi_m[r], src, 64);
                const uint32_t aj = (uint32_t)__shfl((int)aj_m[r], src, 64);
                scan_alpha_group(a, eri, h, lo, hi, xa, xb, aj, lane, acc);
            }
            found = __ballot(sz > 0 && sz <= PT2_SMALL);  // small groups: 64 / PT2_GL at a time
            while (found) {
                int src = -1;
#pragma unroll
                for (int k = 0; k < 64 / PT2_GL; ++k) {
                    if (found) {
                        const int f = __builtin_ctzll(found);
                        found &= found - 1;
                        if (k == lane / PT2_GL) src = f;
                    }
                }
                const int sidx = src < 0 ? 0 : src;
                const int32_t lo = __shfl(lo_m[r], sidx, 64), hi = __shfl(hi_m[r], sidx, 64);
                const uint32_t aj = (uint32_t)__shfl((int)aj_m[r], sidx, 64);
                scan_small_group(a, eri, h, lo, src < 0 ? lo : hi, xa, xb, aj, lane % PT2_GL, acc);
            }
        }
        acc = wave_sum_d(acc);
        if (lane == 0) {
            if (!LINKS) {
                *part = acc;
            } else {
                if (a.numer) a.numer[t] = acc;
                if (a.score) a.score[t] = acc * acc / fabs(a.e0 - d);
            }
        }
    }
}

// ------------------------------------- one move in each spin, through tables
// Members of each alpha group as a bit per distinct beta string: word w of a
// group holds strings 32 w .. 32 w + 31 (x: the bits, y: members before them).
// The partners of a candidate in a group are then looked up by its own beta
// moves (na (norb - na) tests) instead of read past (the group's rows).
constexpr int PT2_MAX_WORDS = 1024;            // 32,768 distinct beta strings
constexpr int64_t PT2_MAX_TABLE = 256 << 20;   // bytes
constexpr int PT2_CS = 2304;                   // members of a group whose coefficients are staged
constexpr int PT2_CPW = 4;                     // candidates of a wave
constexpr int PT2_TILE = PT2_CPW * PT_NT / 64; // and of a workgroup
constexpr int PT2_MAX_MOVES = 256;
constexpr int PT2_MAX_PAIRS = 32 * 33 / 2;
static_assert(PT2_MAX_PAIRS <= PT_NT && PT2_MAX_WORDS <= PT_NT && PT2_CS <= 3 * PT_NT, "staging");

__global__ void k_pt2_bits(int64_t ndet, const int32_t *aidx, const int32_t *bidx, int words, uint2 *tab) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ndet) return;
    const int32_t b = bidx[i];
    atomicOr(&tab[(int64_t)aidx[i] * words + (b >> 5)].x, 1u << (b & 31));
}

// Members before each word, one wave per group.
__global__ __launch_bounds__(256) void k_pt2_ranks(int32_t nua, int words, uint2 *tab) {
    const int lane = threadIdx.x & 63;
    const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (g >= nua) return;
    uint2 *row = tab + g * words;
    int before = 0;
    for (int w0 = 0; w0 < words; w0 += 64) {
        const int w = w0 + lane;
        const int n = w < words ? popc32(row[w].x) : 0;
        int incl = n;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int x = __shfl_up(incl, off, 64);
            if (lane >= off) incl += x;
        }
        if (w < words) row[w].y = (uint32_t)(before + incl - n);
        before += __shfl(incl, 63, 64);
    }
}

// flag[u] = 1 where a tile starts: every PT2_TILE candidates of a run that shares its alpha string.
__global__ void k_pt2_tile_flags(const uint64_t *keys, int64_t n, int norb, int32_t *flag) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const uint64_t first = (keys[u] >> norb) << norb;
    int64_t lo = 0, hi = u;  // first candidate of the run
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < first) lo = mid + 1;
        else hi = mid;
    }
    flag[u] = (u - lo) % PT2_TILE == 0 ? 1 : 0;
}

__global__ void k_pt2_tile_list(const int32_t *flag, const int32_t *pos, int64_t n, int32_t *tiles, int32_t *ntiles) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    if (flag[u]) tiles[pos[u]] = (int32_t)u;
    if (u == n - 1) *ntiles = pos[u] + flag[u];
}

// Numerators over the alpha groups one move from the candidates' common alpha
// string, added to the same-spin part.  A workgroup owns one tile and walks the
// groups: the group's bits, its members' coefficients and the row of integrals
// (pa ha|..) of the alpha move are staged in LDS (the next group's while this
// one is used); lane l of a wave holds beta move 64 s + l of each of the wave's
// four candidates -- the index of the string it leads to, its integral and its
// sign -- tests the bit and, on a hit, adds coefficient times integral.
// What bounds it: scanning the groups read every member for every candidate
// through L1 (8.8e5 candidates, 1e6 rows: 13.4 of 21.3 ms); here a group is read
// once for up to 64 candidates, and a test covers 64 moves where a scan step
// covered 64 members, most of them not coupled: 4.1 ms.
template <int SLOTS>
__global__ __launch_bounds__(PT_NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_pt2_links(
    Pt2Args a, const uint64_t *keys, const int32_t *order, const int32_t *tiles, const int32_t *ntiles, int words,
    const uint2 *tab) {
    __shared__ uint2 s_bits[2][PT2_MAX_WORDS + 1];  // the word after the last is empty
    __shared__ double s_cs[2][PT2_CS];
    __shared__ double s_row[2][PT2_MAX_PAIRS];
    __shared__ int32_t s_g[PT2_MAX_MOVES], s_lo[PT2_MAX_MOVES], s_sz[PT2_MAX_MOVES], s_mv[PT2_MAX_MOVES];
    __shared__ int s_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int norb = a.norb, nva = norb - a.na, nvb = norb - a.nb, nma = a.na * nva, nmb = a.nb * nvb;
    const int npair = norb * (norb + 1) / 2;
    const uint32_t full = norb >= 32 ? 0xffffffffu : ((1u << norb) - 1u);
    const int nt = *ntiles;
    if (tid < 2) s_bits[tid][words] = make_uint2(0, 0);
    for (int tile = blockIdx.x; tile < nt; tile += gridDim.x) {
        const int64_t u0 = tiles[tile];
        const uint32_t xa = (uint32_t)(keys[u0] >> norb);
        if (popc32(xa) != a.na) continue;  // malformed candidates (uniform over the workgroup)
        __syncthreads();                   // the previous tile's lists are no longer read
        if (wave == 0) {  // the groups one move away, in the order of the moves
            int at = 0;
            for (int m0 = 0; m0 < nma; m0 += 64) {
                const int m = m0 + lane;
                int32_t g = -1;
                int r = 0, q = 0;
                if (m < nma) {
                    r = nth_bit(xa, m / nva);
                    q = nth_bit(~xa & full, m % nva);
                    g = find_u32(a.B.ua, a.B.nua, xa ^ (1u << r) ^ (1u << q));
                }
                const uint64_t on = __ballot(g >= 0);
                if (g >= 0) {
                    const int k = at + __popcll(on & ((1ull << lane) - 1ull));
                    s_g[k] = g;
                    s_lo[k] = a.B.ga[g];
                    s_sz[k] = a.B.ga[g + 1] - a.B.ga[g];
                    s_mv[k] = pair_index(r, q) | (int)(single_parity(xa ^ (1u << r) ^ (1u << q), q, r) << 16);
                }
                at += __popcll(on);
            }
            if (lane == 0) s_n = at;
        }
        // this wave's candidates: word | bit << 16 of the string each beta move
        // leads to (the empty word: none), integral | sign << 31
        int32_t at[PT2_CPW][SLOTS], mv[PT2_CPW][SLOTS];
        double acc[PT2_CPW];
        int mine = 0;
#pragma unroll
        for (int c = 0; c < PT2_CPW; ++c) {
            acc[c] = 0.0;
            const int64_t u = u0 + wave * PT2_CPW + c;
            const uint64_t key = u < a.ncand ? keys[u] : ~0ull;
            const uint32_t xb = (uint32_t)key & full;
            const bool ok = u < a.ncand && (uint32_t)(key >> norb) == xa && popc32(xb) == a.nb;
            mine |= ok ? 1 << c : 0;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const int m = 64 * s + lane;
                at[c][s] = words;
                mv[c][s] = 0;
                if (ok && m < nmb) {
                    const int r = nth_bit(xb, m / nvb), q = nth_bit(~xb & full, m % nvb);
                    const uint32_t bj = xb ^ (1u << r) ^ (1u << q);
                    const int32_t b = find_u32(a.B.ub, a.B.nub, bj);
                    if (b >= 0) at[c][s] = (b >> 5) | (b & 31) << 16;
                    mv[c][s] = pair_index(r, q) | (int)(single_parity(bj, q, r) << 31);
                }
            }
        }
        __syncthreads();
        const int nl = s_n;
        uint2 rb = {};
        double rc[3] = {}, rr = 0.0;
        auto fetch = [&](int l) {
            const int32_t lo = s_lo[l], sz = s_sz[l] <= PT2_CS ? s_sz[l] : 0, m = s_mv[l], A = m & 0xffff;
            if (tid < words) rb = tab[(int64_t)s_g[l] * words + tid];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (tid + i * PT_NT < sz) rc[i] = a.cs[lo + tid + i * PT_NT];
            if (tid < npair) {
                const double v = a.eri[A >= tid ? A * (A + 1) / 2 + tid : tid * (tid + 1) / 2 + A];
                rr = m >> 16 ? -v : v;
            }
        };
        auto store = [&](int l, int buf) {
            const int32_t sz = s_sz[l] <= PT2_CS ? s_sz[l] : 0;
            if (tid < words) s_bits[buf][tid] = rb;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (tid + i * PT_NT < sz) s_cs[buf][tid + i * PT_NT] = rc[i];
            if (tid < npair) s_row[buf][tid] = rr;
        };
        if (nl > 0) {
            fetch(0);
            store(0, 0);
        }
        __syncthreads();
        for (int l = 0; l < nl; ++l) {
            const int buf = l & 1;
            if (l + 1 < nl) fetch(l + 1);
            auto test = [&](auto staged) {
                const double *gcs = a.cs + s_lo[l];
#pragma unroll
                for (int s = 0; s < SLOTS; ++s) {
                    uint2 w[PT2_CPW];
#pragma unroll
                    for (int c = 0; c < PT2_CPW; ++c) w[c] = s_bits[buf][at[c][s] & 0xffff];
#pragma unroll
                    for (int c = 0; c < PT2_CPW; ++c) {
                        const uint32_t below = w[c].x & ((1u << (at[c][s] >> 16)) - 1u);
                        if ((w[c].x >> (at[c][s] >> 16)) & 1u) {
                            const int pos = (int)w[c].y + popc32(below);
                            double v;
                            if constexpr (decltype(staged)::value) v = s_cs[buf][pos];
                            else v = gcs[pos];
                            v *= s_row[buf][mv[c][s] & 0xffff];
                            acc[c] += mv[c][s] < 0 ? -v : v;
                        }
                    }
                }
            };
            if (mine) {
                if (s_sz[l] <= PT2_CS) test(std::true_type{});
                else test(std::false_type{});
            }
            if (l + 1 < nl) store(l + 1, buf ^ 1);
            __syncthreads();
        }
#pragma unroll
        for (int c = 0; c < PT2_CPW; ++c) {
            if (!((mine >> c) & 1)) continue;
            const int64_t u = u0 + wave * PT2_CPW + c;
            const double sum = wave_sum_d(acc[c]) + a.part[u];
            if (lane == 0) {
                const int32_t t = order[u];
                if (a.numer) a.numer[t] = sum;
                if (a.score) a.score[t] = sum * sum / fabs(a.e0 - a.dval[u]);
            }
        }
    }
}

int device_cus(const Ctx &c) {
    int n = 256;
    (void)hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, c.device);
    return n;
}

size_t integral_lds(const Ctx &c) {
    return sizeof(double) * ((size_t)neri_packed(c.norb) + (size_t)c.norb * c.norb);
}

}  // namespace

int64_t excitations_per_det(int norb, int na, int nb) {
    const int64_t nva = norb - na, nvb = norb - nb;
    const int64_t sA = na * nva, sB = nb * nvb;
    return sA + sB + (int64_t)na * (na - 1) / 2 * (nva * (nva - 1) / 2) +
           (int64_t)nb * (nb - 1) / 2 * (nvb * (nvb - 1) / 2) + sA * sB;
}

void top_k(Ctx &c, int64_t n, const double *v, int64_t k, bool largest, int32_t *idx) {
    hipStream_t s = c.stream;
    uint64_t *keys = c.cs.get<uint64_t>(0, n);
    int32_t *vals = c.cs.get<int32_t>(1, n);
    unsigned *bad = (unsigned *)c.cs.words(1);
    HQ_CHECK(hipMemsetAsync(bad, 0, sizeof(unsigned), s));
    hipLaunchKernelGGL(k_order_keys, dim3(grid_for(n, 256)), dim3(256), 0, s, v, n, largest, keys, vals, bad);
    HQ_LAUNCH_CHECK();
    radix_sort_u64(s, keys, vals, n, 64, c.work);
    unsigned hbad = 0;
    HQ_CHECK(hipMemcpyAsync(&hbad, bad, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HQ_CHECK(hipStreamSynchronize(s));
    if (hbad) throw Error(HINQS_E_NONFINITE, "values contain NaN");
    hipLaunchKernelGGL(k_take_top, dim3(grid_for(k, 256)), dim3(256), 0, s, vals, k, (const int32_t *)nullptr,
                       idx, (int32_t *)nullptr);
    HQ_LAUNCH_CHECK();
    HQ_CHECK(hipStreamSynchronize(s));
}

int64_t expand(Ctx &c, const double *coeffs, bool sorted, int64_t ntop, int64_t capacity, uint64_t *out_a,
               uint64_t *out_b, int32_t *top) {
    hipStream_t s = c.stream;
    const int64_t n = c.ndet;
    if (ntop > n) ntop = n;
    // the ntop largest |c| (stable: ties keep the lower index first).  Scratch
    // slots 0 and 1 hold the sort keys and values, then (stream-ordered after
    // the top ntop have been taken) the raw excitations and their sort values.
    uint64_t *keys = c.cs.get<uint64_t>(0, n);
    int32_t *vals = c.cs.get<int32_t>(1, n);
    int32_t *pos = c.cs.get<int32_t>(2, ntop);
    unsigned long long *words = c.cs.words(2);
    unsigned *bad = (unsigned *)words;
    unsigned long long *cnt = words + 1;
    HQ_CHECK(hipMemsetAsync(bad, 0, sizeof(unsigned), s));
    hipLaunchKernelGGL(k_mag_keys, dim3(grid_for(n, 256)), dim3(256), 0, s, coeffs, n, keys, vals, bad);
    HQ_LAUNCH_CHECK();
    radix_sort_u64(s, keys, vals, n, 63, c.work);
    unsigned hbad = 0;
    HQ_CHECK(hipMemcpyAsync(&hbad, bad, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HQ_CHECK(hipStreamSynchronize(s));
    if (hbad) throw Error(HINQS_E_NONFINITE, "coefficients contain NaN/Inf");
    hipLaunchKernelGGL(k_take_top, dim3(grid_for(ntop, 256)), dim3(256), 0, s, vals, ntop,
                       sorted ? (const int32_t *)nullptr : (const int32_t *)c.inv.p, top, pos);
    HQ_LAUNCH_CHECK();

    // every single and double of the chosen determinants, kept when coupled and outside B
    const int64_t nexc = excitations_per_det(c.norb, c.na, c.nb);
    const int64_t cap = ntop * nexc;
    if (cap >= ((int64_t)1 << 31))
        throw Error(HINQS_E_UNSUPPORTED, "expansion of " + std::to_string(ntop) +
                                             " determinants exceeds 2^31 excitations; expand fewer at once");
    uint64_t *raw = c.cs.get<uint64_t>(0, cap);
    HQ_CHECK(hipMemsetAsync(cnt, 0, sizeof(unsigned long long), s));
    ExpArgs ea{tables_of(c), c.norb, neri_packed(c.norb), c.na, c.nb, ntop, pos, c.d_eri.p, c.d_h.p, raw, cnt};
    const size_t lds = integral_lds(c);
    const int cus = device_cus(c);
    if (lds <= 150 * 1024) {
        HQ_CHECK(hipFuncSetAttribute((const void *)k_expand<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
        const unsigned grid = (unsigned)std::min<int64_t>(ntop, (int64_t)cus * 2);
        hipLaunchKernelGGL(k_expand<true>, dim3(grid), dim3(EX_NT), lds, s, ea);
    } else {
        const unsigned grid = (unsigned)std::min<int64_t>(ntop, (int64_t)cus * 2);
        hipLaunchKernelGGL(k_expand<false>, dim3(grid), dim3(EX_NT), 0, s, ea);
    }
    HQ_LAUNCH_CHECK();
    unsigned long long hcnt = 0;
    HQ_CHECK(hipMemcpyAsync(&hcnt, cnt, sizeof(hcnt), hipMemcpyDeviceToHost, s));
    HQ_CHECK(hipStreamSynchronize(s));
    const int64_t nraw = (int64_t)hcnt;
    if (nraw == 0) return 0;

    // sort and drop repeats: ascending (alpha, beta)
    int32_t *rv = c.cs.get<int32_t>(1, nraw);
    radix_sort_u64(s, raw, rv, nraw, 2 * c.norb, c.work);
    int32_t *flag = c.cs.get<int32_t>(3, nraw);
    int32_t *fpos = c.cs.get<int32_t>(4, nraw);
    hipLaunchKernelGGL(k_unique_flags, dim3(grid_for(nraw, 256)), dim3(256), 0, s, raw, nraw, flag);
    HQ_LAUNCH_CHECK();
    exclusive_scan_i32(s, flag, fpos, nraw, c.work);
    int32_t last[2] = {0, 0};
    HQ_CHECK(hipMemcpyAsync(&last[0], fpos + nraw - 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HQ_CHECK(hipMemcpyAsync(&last[1], flag + nraw - 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    if (capacity > 0) {
        hipLaunchKernelGGL(k_unique_write, dim3(grid_for(nraw, 256)), dim3(256), 0, s, raw, flag, fpos,
                           nraw, c.norb, capacity, out_a, out_b);
        HQ_LAUNCH_CHECK();
    }
    HQ_CHECK(hipStreamSynchronize(s));
    return (int64_t)last[0] + last[1];
}

namespace {

// Strings of n among norb orbitals (at most 6e8).
int64_t strings(int norb, int n) {
    int64_t s = 1;
    for (int i = 1; i <= n; ++i) s = s * (norb - n + i) / i;
    return s;
}

// Times (us) of the linked class alone: scanning the groups, and through the
// tables.  The scan's waves take PT2_RUN candidates one after another, 8,192 of
// them at a time, and wait for each group in turn: about 0.4 us for a few
// members, 0.95 from about 64 on.  The tables cost their building, then 1.4 us
// per group and 512 tiles at a time, whatever a tile holds.
// Whole calls, scan / tables in us: 1e6 rows, groups of 87, 1 candidate 135 / 260,
// 100 candidates 1028 / 409, 8,000 in as many tiles 1287 / 1685, 1e5 in 11,000
// 2410 / 2780, 5.4e5 in 18,000 6536 / 5124; 1e5 rows, groups of 9, 2,000 in as
// many 538 / 569, 30,000 in 8,600 823 / 1810, 5.3e6 in 88,000 25,900 / 23,250;
// 1,000 rows, 1 candidate 82 / 127, 3,000 in 250 tiles 411 / 250.  Lists of more than
// a few hundred candidates are mostly excitations of the set's leading members, near
// its large groups, and wait for the longest of their waves: half again (1e6 rows,
// 54,500 excitations in 5,961 tiles 1823 / 1682, 1.6e5 in 10,900 2838 / 2850).
double link_scan_us(const Ctx &c, int moves, int64_t ncand) {
    const double group = (double)c.ndet / c.nua;
    const double per_wave = ncand <= 8192 * PT2_RUN ? (double)std::min<int64_t>(ncand, PT2_RUN) : ncand / 8192.0;
    const double list = ncand > 256 ? 1.5 : 1.0;
    return list * per_wave * moves * (0.4 + 0.55 * std::min(1.0, group / 64.0));
}
double link_table_us(size_t bytes, int moves, int64_t tiles) {
    return 40.0 + 0.5e-6 * bytes + moves * 1.4 * std::max(1.0, tiles / 512.0);
}

}  // namespace

void pt2(Ctx &c, const double *coeffs, bool sorted, double e0, int64_t ncand, const uint64_t *ca,
         const uint64_t *cb, double *numer, double *hxx, double *score) {
    hipStream_t s = c.stream;
    const double *csp = coeffs;
    if (!sorted) {
        double *cs = c.cs.get<double>(0, c.ndet);
        gather_rows(s, coeffs, cs, c.perm.p, c.ndet, 8);
        csp = cs;
    }
    unsigned long long *words = c.cs.words(2);
    unsigned *bad = (unsigned *)words;
    unsigned long long *next = words + 1;
    HQ_CHECK(hipMemsetAsync(bad, 0, sizeof(unsigned), s));
    Pt2Args pa{tables_of(c), c.norb, neri_packed(c.norb), c.na, c.nb, c.alink_max, c.alink_ptr.p, c.alink.p,
               c.ecore, e0, ncand, ca, cb, csp, c.d_eri.p, c.d_h.p, numer, hxx, score, bad, nullptr, nullptr};
    // candidates in key order, and their groups in B
    uint64_t *keys = c.cs.get<uint64_t>(1, ncand);
    int32_t *order = c.cs.get<int32_t>(2, ncand);
    int32_t *ga_of = c.cs.get<int32_t>(3, ncand);
    int32_t *gb_of = c.cs.get<int32_t>(4, ncand);
    hipLaunchKernelGGL(k_pt2_keys, dim3(grid_for(ncand, 256)), dim3(256), 0, s, ca, cb, ncand, c.norb, keys,
                       order);
    HQ_LAUNCH_CHECK();
    radix_sort_u64(s, keys, order, ncand, 2 * c.norb, c.work);
    hipLaunchKernelGGL(k_pt2_groups, dim3(grid_for(ncand, 256)), dim3(256), 0, s, pa.B, ca, cb, order, ncand,
                       c.norb, ga_of, gb_of);
    HQ_LAUNCH_CHECK();
    const size_t lds = integral_lds(c);
    const int cus = device_cus(c);
    const bool use_lds = lds <= 150 * 1024;
    pa.dval = c.cs.get<double>(5, 2 * ncand);
    pa.part = pa.dval + ncand;
    const unsigned dgrid = (unsigned)std::min<int64_t>((ncand + 255) / 256, (int64_t)cus * 8);
    if (use_lds) {
        HQ_CHECK(hipFuncSetAttribute((const void *)k_pt2_diag<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
        hipLaunchKernelGGL(k_pt2_diag<true>, dim3(dgrid), dim3(256), lds, s, pa, order);
    } else {
        hipLaunchKernelGGL(k_pt2_diag<false>, dim3(dgrid), dim3(256), 0, s, pa, order);
    }
    HQ_LAUNCH_CHECK();
    // lookups by the candidates' own moves while the tables stay small (sets of very
    // many distinct strings keep the scan) and the candidates share alpha strings
    const int nwords = (c.nub + 31) / 32;
    const int moves = c.na * (c.norb - c.na), moves_b = c.nb * (c.norb - c.nb);
    const bool fits = nwords <= PT2_MAX_WORDS && (int64_t)c.nua * nwords * (int64_t)sizeof(uint2) <= PT2_MAX_TABLE &&
                      moves <= PT2_MAX_MOVES && moves_b <= PT2_MAX_MOVES;
    const size_t table = sizeof(uint2) * (size_t)c.nua * nwords;
    const double scan = link_scan_us(c, moves, ncand);
    const char *env = std::getenv("HINQS_PT2_TABLES");  // 0: scan, 1: tables wherever they fit
    const int asked = env && *env ? std::atoi(env) : -1;
    // fewest and most tiles that the list can have: a partly filled one per alpha string
    const int64_t fewest = (ncand + PT2_TILE - 1) / PT2_TILE;
    const int64_t most = std::min(ncand, (int64_t)(ncand / PT2_TILE + strings(c.norb, c.na)));
    bool lookup = fits && (asked >= 0 ? asked != 0 : link_table_us(table, moves, fewest) <= scan);
    // the scan needs none of the tables' memory: where there is none, it runs
    auto room = [&](auto &&get) {
        try {
            get();
            return true;
        } catch (const Error &e) {
            if (e.code != HINQS_E_OOM) throw;
            (void)hipGetLastError();
            return false;
        }
    };
    int32_t *flag = nullptr, *tiles = nullptr, *ntiles = nullptr;
    uint2 *tab = nullptr;
    lookup = lookup && room([&] { flag = c.cs.get<int32_t>(7, 3 * ncand + 1); });
    if (lookup) {
        int32_t *fpos = flag + ncand;
        tiles = fpos + ncand;
        ntiles = tiles + ncand;
        hipLaunchKernelGGL(k_pt2_tile_flags, dim3(grid_for(ncand, 256)), dim3(256), 0, s, keys, ncand, c.norb, flag);
        HQ_LAUNCH_CHECK();
        exclusive_scan_i32(s, flag, fpos, ncand, c.work);
        hipLaunchKernelGGL(k_pt2_tile_list, dim3(grid_for(ncand, 256)), dim3(256), 0, s, flag, fpos, ncand, tiles,
                           ntiles);
        HQ_LAUNCH_CHECK();
        // the number of tiles is read back where it decides
        if (asked < 0 && link_table_us(table, moves, most) > scan) {
            int32_t nt = 0;
            HQ_CHECK(hipMemcpyAsync(&nt, ntiles, sizeof(int32_t), hipMemcpyDeviceToHost, s));
            HQ_CHECK(hipStreamSynchronize(s));
            lookup = link_table_us(table, moves, nt) <= scan;
        }
    }
    lookup = lookup && room([&] { tab = c.cs.get<uint2>(6, (size_t)c.nua * nwords); });
    // resident workgroups only (two per CU); they share the candidates through a counter
    const int64_t runs = (ncand + PT2_RUN - 1) / PT2_RUN;
    const unsigned grid =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)cus * 2, (runs + PT_NT / 64 - 1) / (PT_NT / 64)));
    HQ_CHECK(hipMemsetAsync(next, 0, sizeof(unsigned long long), s));
    auto launch = [&](auto lds_tag, auto slots_tag, auto links_tag) {
        constexpr bool L = decltype(lds_tag)::value;
        constexpr int S = decltype(slots_tag)::value;
        constexpr bool K = decltype(links_tag)::value;
        if (L)
            HQ_CHECK(hipFuncSetAttribute((const void *)k_pt2<L, S, K>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)lds));
        hipLaunchKernelGGL((k_pt2<L, S, K>), dim3(grid), dim3(PT_NT), L ? lds : 0, s, pa, order, ga_of, gb_of, next);
        HQ_LAUNCH_CHECK();
    };
    using T = std::true_type;
    using F = std::false_type;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S4 = std::integral_constant<int, 4>;
    if (lookup) {
        HQ_CHECK(hipMemsetAsync(tab, 0, table, s));
        hipLaunchKernelGGL(k_pt2_bits, dim3(grid_for(c.ndet, 256)), dim3(256), 0, s, c.ndet, c.aidx.p, c.bidx.p,
                           nwords, tab);
        HQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_pt2_ranks, dim3(grid_for((int64_t)c.nua * 64, 256)), dim3(256), 0, s, c.nua, nwords, tab);
        HQ_LAUNCH_CHECK();
        if (use_lds) launch(T{}, S1{}, F{});
        else launch(F{}, S1{}, F{});
        const dim3 lg((unsigned)std::min<int64_t>((int64_t)cus * 2, ncand)), lb(PT_NT);
        if (moves_b <= 64)
            hipLaunchKernelGGL(k_pt2_links<1>, lg, lb, 0, s, pa, keys, order, tiles, ntiles, nwords, tab);
        else if (moves_b <= 128)
            hipLaunchKernelGGL(k_pt2_links<2>, lg, lb, 0, s, pa, keys, order, tiles, ntiles, nwords, tab);
        else hipLaunchKernelGGL(k_pt2_links<4>, lg, lb, 0, s, pa, keys, order, tiles, ntiles, nwords, tab);
    } else if (use_lds) {
        if (moves <= 64) launch(T{}, S1{}, T{});
        else if (moves <= 128) launch(T{}, S2{}, T{});
        else launch(T{}, S4{}, T{});
    } else {
        if (moves <= 64) launch(F{}, S1{}, T{});
        else if (moves <= 128) launch(F{}, S2{}, T{});
        else launch(F{}, S4{}, T{});
    }
    HQ_LAUNCH_CHECK();
    unsigned hbad = 0;
    HQ_CHECK(hipMemcpyAsync(&hbad, bad, sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HQ_CHECK(hipStreamSynchronize(s));
    if (hbad)
        throw Error(HINQS_E_BAD_OCCUPATION,
                    "a candidate has bits at or above norb or the wrong electron count (its outputs are NaN)");
}

namespace {

// PT2 quantities of the members of B from (H_B c) in sorted order (diagonal
// included); outputs in caller order through perm (null: sorted order).
__global__ void k_pt2_members(int64_t n, const double *hc, const double *diag, double e0, const int32_t *perm,
                              double *numer, double *hxx, double *score) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = perm ? (int64_t)perm[i] : i;
    const double v = hc[i], d = diag[i];
    if (numer) numer[o] = v;
    if (hxx) hxx[o] = d;
    if (score) score[o] = v * v / fabs(e0 - d);
}

}  // namespace

void pt2_members(Ctx &c, const double *coeffs, bool sorted, double e0, double *numer, double *hxx,
                 double *score) {
    hipStream_t s = c.stream;
    const int64_t n = c.ndet;
    const double *cs = coeffs;
    if (!sorted) {
        double *g = c.cs.get<double>(0, n);
        gather_rows(s, coeffs, g, c.perm.p, n, 8);
        cs = g;
    }
    double *hc = c.cs.get<double>(1, n);
    sigma_sorted(c, 1, cs, 1, hc, 1, HINQS_FP64, s);
    hipLaunchKernelGGL(k_pt2_members, dim3(grid_for(n, 256)), dim3(256), 0, s, n, (const double *)hc,
                       (const double *)c.diag.p, e0, sorted ? (const int32_t *)nullptr : (const int32_t *)c.perm.p,
                       numer, hxx, score);
    HQ_LAUNCH_CHECK();
}

}  // namespace hinqs

// ------------------------------------------------------------ product space
namespace hinqs {
namespace {

// missing[g] = number of distinct beta strings absent from alpha group g.
__global__ void k_missing_counts(const int32_t *ga, int32_t nua, int32_t nub, int64_t *missing) {
    const int32_t g = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (g < nua) missing[g] = (int64_t)nub - (ga[g + 1] - ga[g]);
}

// One wave per alpha group: the distinct beta strings absent from the group,
// ascending, written as (alpha, beta) pairs from off[g] (first `cap` only).
__global__ void k_missing_list(const uint32_t *ua, const uint32_t *ub, const uint32_t *sb, const int32_t *ga,
                               int32_t nua, int32_t nub, const int64_t *off, int64_t cap, uint64_t *oa,
                               uint64_t *ob) {
    const int lane = threadIdx.x & 63;
    const int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (g >= nua) return;
    const int32_t lo = ga[g], n = ga[g + 1] - lo;
    int64_t pos = off[g];
    for (int32_t t0 = 0; t0 < nub; t0 += 64) {
        const int32_t t = t0 + lane;
        bool miss = false;
        uint32_t b = 0;
        if (t < nub) {
            b = ub[t];
            int32_t l = 0, h = n;  // is b among the group's beta strings?
            while (l < h) {
                const int32_t m = (l + h) >> 1;
                if (sb[lo + m] < b)
                    l = m + 1;
                else
                    h = m;
            }
            miss = !(l < n && sb[lo + l] == b);
        }
        const uint64_t m = __ballot(miss);
        if (miss) {
            const int64_t k = pos + __popcll(m & ((1ull << lane) - 1ull));
            if (k < cap) {
                oa[k] = ua[g];
                ob[k] = b;
            }
        }
        pos += __popcll(m);
    }
}

}  // namespace

int64_t product_closure(Ctx &c, int64_t cap, uint64_t *out_a, uint64_t *out_b) {
    hipStream_t s = c.stream;
    const int64_t total = (int64_t)c.nua * c.nub - c.ndet;
    if (cap <= 0 || total <= 0) return total;
    int64_t *miss = c.cs.get<int64_t>(0, c.nua + 1);
    int64_t *off = c.cs.get<int64_t>(1, c.nua + 1);
    HQ_CHECK(hipMemsetAsync(miss + c.nua, 0, sizeof(int64_t), s));
    hipLaunchKernelGGL(k_missing_counts, dim3(grid_for(c.nua, 256)), dim3(256), 0, s, c.ga.p, c.nua, c.nub, miss);
    HQ_LAUNCH_CHECK();
    exclusive_scan_i64(s, miss, off, c.nua + 1, c.work);
    hipLaunchKernelGGL(k_missing_list, dim3(grid_for((int64_t)c.nua * 64, 256)), dim3(256), 0, s, c.ua.p, c.ub.p,
                       c.sb.p, c.ga.p, c.nua, c.nub, off, cap, out_a, out_b);
    HQ_LAUNCH_CHECK();
    HQ_CHECK(hipStreamSynchronize(s));
    return total;
}

}  // namespace hinqs
