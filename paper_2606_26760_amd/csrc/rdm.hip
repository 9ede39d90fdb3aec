// One- and two-particle density matrices of a vector over B, and the energy
// gradient with respect to the integrals built from them.
//
//   rdm1[p,q]     = sum_s  <c| a+_{ps} a_{qs} |c>
//   rdm2[p,q,r,s] = sum_st <c| a+_{ps} a+_{rt} a_{st} a_{qs} |c>
//
// Every stored coupling (i <- j) contributes c_i c_j times its canonical sign
// to a few entries; the diagonal contributes c_i^2 times occupation products.
//   * diagonal: G[x][y] = sum_i c_i^2 n_x n_y over spin orbitals x, y, a Gram
//     product of the occupation bits (FP64 MFMA);
//   * singles q -> p: rdm1[p][q] += w;  Sc[pq][k] += w for every electron k
//     the two determinants share (Coulomb-like terms rdm2[p,q,k,k] and
//     rdm2[k,k,p,q]); Sx[pq][k] += w for the same-spin ones (exchange-like
//     rdm2[p,k,k,q], rdm2[k,q,p,k] with a minus sign);
//   * doubles: rdm2[p1,h1,p2,h2] += w, same-spin ones rdm2[p1,h2,p2,h1] -= w.
// The coupling set is symmetric and the vector real, so (j <- i) contributes
// to the index-transposed entries exactly what (i <- j) does, and a double adds
// the same to its pair swap: one of each mirror pair is visited, and everything
// is summed per class of entries that must be equal -- an unordered orbital
// pair for rdm1 / Sc / Sx, and for the doubles two unordered pairs and their
// relative orientation (n (n - 1) / 2 = P pairs give P (P + 1) classes).
//
// Up to 16 orbitals one set of these sums (148 KB at 16) fits the LDS of a
// workgroup: every double is one LDS add (two same-spin), and each workgroup
// writes its table once.  The lanes of a wave hold couplings of one row, whose
// moves differ, so their adds hardly ever meet.  What bounds it: the gathers
// of c_j, one per visited coupling.  2e5 rows, 12 orbitals: 0.44 ms, against
// 2.37 ms with the doubles added to 32 copies of rdm2 in global memory and the
// diagonal's pairs added one by one; 1e6 rows, 16 orbitals, 1.57e8 couplings: 1.06 ms,
// the whole call 1.13 against 4.9.
// Above 16 orbitals the global copies stay.  The floating-point atomics make
// the result reproducible to rounding, not bitwise.
#include <algorithm>

#include "common.hpp"

namespace hinqs {

namespace {

constexpr int NCOPY = 32;

struct RdmArgs {
    int64_t ndet;
    int norb;
    const uint32_t *sa, *sb;
    const int64_t *rowptr;
    const int32_t *col;
    const uint32_t *desc;
    const double *c;
    double *g2;      // NCOPY x norb^4
    double *tab;     // per-copy tables when not in LDS: NCOPY x ntab
    int ntab;        // doubles per table set
};

// Table layout (one set): Sc[norb^3] | Sx[norb^3] | rdm1[norb^2] | Psame[norb^2] | Pab[norb^2] | occ[norb]
__host__ __device__ inline int tab_size(int n) { return 2 * n * n * n + 3 * n * n + n; }

template <bool LDS>
__global__ __launch_bounds__(256) void k_rdm(RdmArgs a) {
    extern __shared__ double sm[];
    const int n = a.norb, n2 = n * n, n3 = n2 * n;
    const int copy = blockIdx.x % NCOPY;
    double *tab = LDS ? sm : a.tab + (int64_t)copy * a.ntab;
    if (LDS) {
        for (int t = threadIdx.x; t < a.ntab; t += blockDim.x) tab[t] = 0.0;
        __syncthreads();
    }
    double *Sc = tab, *Sx = tab + n3, *g1 = tab + 2 * n3, *Ps = g1 + n2, *Pab = Ps + n2, *occ = Pab + n2;
    double *g2 = a.g2 + (int64_t)copy * n2 * n2;
    auto G2 = [&](int p, int q, int r, int s, double v) {
        atomicAdd(&g2[((p * n + q) * n + r) * n + s], v);
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int64_t row = (int64_t)blockIdx.x * nw + wave; row < a.ndet; row += (int64_t)gridDim.x * nw) {
        const double ci = a.c[row];
        const uint32_t ai = a.sa[row], bi = a.sb[row];
        if (ci != 0.0) {
            // diagonal: occupied pairs spread over lanes
            const double w = ci * ci;
            const int na = popc32(ai), nb = popc32(bi);
            const int ntot = na + nb;
            for (int t = lane; t < ntot * ntot; t += 64) {
                const int x = t / ntot, y = t % ntot;
                // x-th and y-th occupied spin-orbital (alpha first)
                uint32_t sx = x < na ? ai : bi, sy = y < na ? ai : bi;
                int ix = x < na ? x : x - na, iy = y < na ? y : y - na;
                for (int q = 0; q < ix; ++q) sx &= sx - 1;
                for (int q = 0; q < iy; ++q) sy &= sy - 1;
                const int k = lowbit(sx), l = lowbit(sy);
                const bool xa = x < na, ya = y < na;
                if (x == y) {
                    atomicAdd(&occ[k], w);
                } else if (xa == ya) {
                    atomicAdd(&Ps[k * n + l], w);
                } else if (xa) {
                    atomicAdd(&Pab[k * n + l], w);
                }
            }
        }
        const int64_t beg = a.rowptr[row], end = a.rowptr[row + 1];
        for (int64_t e = beg + lane; e < end; e += 64) {
            const int32_t j = a.col[e];
            if (j > row) continue;  // its mirror (row <- j) is the transpose
            const double cj = a.c[j];
            const uint32_t d = a.desc[e];
            double w = ci * cj;
            if (w == 0.0) continue;
            if (desc_neg(d)) w = -w;
            const uint32_t type = desc_type(d);
            const int h1 = desc_h1(d), h2 = desc_h2(d), p1 = desc_p1(d), p2 = desc_p2(d);
            if (type == HINQS_EXC_1A || type == HINQS_EXC_1B) {
                const int p = p1, q = h1;
                const uint32_t same = (type == HINQS_EXC_1A ? ai : bi) & ~(1u << p);
                const uint32_t other = (type == HINQS_EXC_1A ? bi : ai);
                atomicAdd(&g1[p * n + q], w);
                for (uint32_t m = same; m; m &= m - 1) {
                    const int k = lowbit(m);
                    atomicAdd(&Sc[(p * n + q) * n + k], w);
                    atomicAdd(&Sx[(p * n + q) * n + k], w);
                }
                for (uint32_t m = other; m; m &= m - 1) {
                    const int k = lowbit(m);
                    atomicAdd(&Sc[(p * n + q) * n + k], w);
                }
            } else if (type == HINQS_EXC_2AB) {
                G2(p1, h1, p2, h2, w);  // + pair swap (p2, h2, p1, h1) at assembly
            } else {
                G2(p1, h1, p2, h2, w);  // + (p2, h2, p1, h1)
                G2(p1, h2, p2, h1, -w);  // + (p2, h1, p1, h2)
            }
        }
    }
    if (LDS) {
        __syncthreads();
        double *dst = a.tab + (int64_t)copy * a.ntab;
        for (int t = threadIdx.x; t < a.ntab; t += blockDim.x) atomicAdd(&dst[t], tab[t]);
    }
}

// rdm1 / rdm2 from the copies and tables (fixed summation order over copies).
__global__ void k_rdm_assemble(int norb, const double *g2c, const double *tabc, int ntab, double *rdm1,
                               double *rdm2) {
    const int n = norb, n2 = n * n, n3 = n2 * n;
    const int64_t n4 = (int64_t)n2 * n2;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n4) return;
    const int s = (int)(t % n), r = (int)((t / n) % n), q = (int)((t / n2) % n), p = (int)(t / n3);
    const int64_t tt = ((int64_t)(q * n + p) * n + s) * n + r;  // transpose (q, p, s, r)
    const int64_t tp = ((int64_t)(r * n + s) * n + p) * n + q;  // pair swap (r, s, p, q)
    const int64_t tq = ((int64_t)(s * n + r) * n + q) * n + p;  // both (s, r, q, p)
    double v = 0.0;
    for (int cpy = 0; cpy < NCOPY; ++cpy) {
        const double *g = g2c + (int64_t)cpy * n4;
        v += (g[t] + g[tt]) + (g[tp] + g[tq]);
    }
    double sc1 = 0, sc2 = 0, sx1 = 0, sx2 = 0, ps = 0, pab = 0, pba = 0, pex = 0;
    for (int cpy = 0; cpy < NCOPY; ++cpy) {
        const double *tb = tabc + (int64_t)cpy * ntab;
        const double *Sc = tb, *Sx = tb + n3, *Ps = tb + 2 * n3 + n2, *Pab = Ps + n2;
        if (r == s) sc1 += Sc[(p * n + q) * n + r] + Sc[(q * n + p) * n + r];
        if (p == q) sc2 += Sc[(r * n + s) * n + p] + Sc[(s * n + r) * n + p];
        if (q == r) sx1 += Sx[(p * n + s) * n + q] + Sx[(s * n + p) * n + q];
        if (p == s) sx2 += Sx[(r * n + q) * n + p] + Sx[(q * n + r) * n + p];
        if (p == q && r == s) {
            if (p != r) ps += Ps[p * n + r];
            pab += Pab[p * n + r];
            pba += Pab[r * n + p];
        }
        if (q == r && p == s && p != q) pex += Ps[p * n + q];
    }
    v += sc1 + sc2 - sx1 - sx2 + ps + pab + pba - pex;
    rdm2[t] = v;
    if (t < n2) {
        const int pp = (int)(t / n), qq = (int)(t % n);
        double g = 0.0;
        for (int cpy = 0; cpy < NCOPY; ++cpy) {
            const double *tb = tabc + (int64_t)cpy * ntab;
            g += tb[2 * n3 + pp * n + qq] + tb[2 * n3 + qq * n + pp];
            if (pp == qq) g += tb[2 * n3 + 3 * n2 + pp];
        }
        rdm1[t] = g;
    }
}

// ------------------------------------------------- tables in LDS (norb <= 16)
constexpr int RDM_LDS_NORB = 16;
constexpr int RDM_NT = 1024;
constexpr int RDM_UNR = 4;   // couplings in flight per lane

__host__ __device__ inline int orb_pairs(int n) { return n * (n - 1) / 2; }
// Unordered pair of p != q.
__host__ __device__ inline int orb_pair(int p, int q) { return p > q ? p * (p - 1) / 2 + q : q * (q - 1) / 2 + p; }
// Class of the two-body entry (p, q, r, s), p != q, r != s.
__host__ __device__ inline int two_class(int p, int q, int r, int s) {
    const int u = orb_pair(p, q), v = orb_pair(r, s);
    const int hi = u > v ? u : v, lo = u > v ? v : u;
    return (hi * (hi + 1) / 2 + lo) * 2 + ((p > q) != (r > s) ? 1 : 0);
}
// Table: doubles[P (P + 1)] | Sc[P n] | Sx[P n] | rdm1[P]
__host__ __device__ inline int class_size(int n) {
    const int P = orb_pairs(n);
    return P * (P + 1) + 2 * P * n + P;
}

struct RdmRows {
    int64_t b[9];  // rows of each XCD
};

__global__ __launch_bounds__(RDM_NT) void k_rdm_lds(RdmArgs a, RdmRows xr, double *parts) {
    extern __shared__ double sm[];
    const int n = a.norb, P = orb_pairs(n);
    for (int t = threadIdx.x; t < a.ntab; t += RDM_NT) sm[t] = 0.0;
    __syncthreads();
    double *D = sm, *Sc = sm + P * (P + 1), *Sx = Sc + P * n, *g1 = Sx + P * n;
    const int lane = threadIdx.x & 63;
    const int xcd = blockIdx.x & 7;
    const int64_t r1 = xr.b[xcd + 1], stride = (int64_t)(gridDim.x >> 3) * (RDM_NT / 64);
    int64_t row = xr.b[xcd] + (int64_t)(blockIdx.x >> 3) * (RDM_NT / 64) + (threadIdx.x >> 6);
    int64_t beg = 0, end = 0;
    double ci = 0.0;
    uint32_t ai = 0, bi = 0;
    if (row < r1) {
        beg = a.rowptr[row];
        end = a.rowptr[row + 1];
        ci = a.c[row];
        ai = a.sa[row];
        bi = a.sb[row];
    }
    while (row < r1) {
        // the next row's data, in flight during this one
        const int64_t nrow = row + stride, at = nrow < r1 ? nrow : row;
        const int64_t nbeg = a.rowptr[at], nend = a.rowptr[at + 1];
        const double nci = a.c[at];
        const uint32_t nai = a.sa[at], nbi = a.sb[at];
        for (int64_t e0 = beg + lane; e0 < end; e0 += 64 * RDM_UNR) {
            int32_t j[RDM_UNR];
            uint32_t d[RDM_UNR];
            double w[RDM_UNR];
#pragma unroll
            for (int u = 0; u < RDM_UNR; ++u) {
                const int64_t e = e0 + 64 * u;
                j[u] = e < end ? a.col[e] : (int32_t)row;
                d[u] = e < end ? a.desc[e] : 0u;
            }
#pragma unroll
            for (int u = 0; u < RDM_UNR; ++u) {
                // one of (row, j) and (j, row), half of every row's couplings
                const bool mine = (j[u] < row) != ((((int32_t)row ^ j[u]) & 1) != 0) && j[u] != row;
                w[u] = mine ? ci * a.c[j[u]] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < RDM_UNR; ++u) {
                if (w[u] == 0.0) continue;
                const double v = desc_neg(d[u]) ? -w[u] : w[u];
                const uint32_t type = desc_type(d[u]);
                const int h1 = desc_h1(d[u]), h2 = desc_h2(d[u]), p1 = desc_p1(d[u]), p2 = desc_p2(d[u]);
                if (type == HINQS_EXC_1A || type == HINQS_EXC_1B) {
                    const int pq = orb_pair(p1, h1);
                    const uint32_t same = (type == HINQS_EXC_1A ? ai : bi) & ~(1u << p1);
                    const uint32_t other = type == HINQS_EXC_1A ? bi : ai;
                    unsafeAtomicAdd(&g1[pq], v);
                    for (uint32_t m = same; m; m &= m - 1) {
                        const int k = lowbit(m);
                        unsafeAtomicAdd(&Sc[pq * n + k], v);
                        unsafeAtomicAdd(&Sx[pq * n + k], v);
                    }
                    for (uint32_t m = other; m; m &= m - 1) unsafeAtomicAdd(&Sc[pq * n + lowbit(m)], v);
                } else {
                    unsafeAtomicAdd(&D[two_class(p1, h1, p2, h2)], v);
                    if (type != HINQS_EXC_2AB) unsafeAtomicAdd(&D[two_class(p1, h2, p2, h1)], -v);
                }
            }
        }
        row = nrow;
        beg = nbeg;
        end = nend;
        ci = nci;
        ai = nai;
        bi = nbi;
    }
    __syncthreads();
    double *dst = parts + (int64_t)blockIdx.x * a.ntab;
    for (int t = threadIdx.x; t < a.ntab; t += RDM_NT) dst[t] = sm[t];
}

// Occupation products of the diagonal: with w_i = c_i^2 and the 2 * 16
// occupation bits of row i, tile (s, t) of parts[block] is
// sum_i w_i n_{s k} n_{t l} for spins s <= t (aa, ab, bb), on
// v_mfma_f64_16x16x4f64: lane l supplies orbital l % 16 of row l / 16 in each
// step, element r of lane l is entry (l / 16 + 4 r, l % 16).
using v4d = __attribute__((__vector_size__(4 * sizeof(double)))) double;
__global__ __launch_bounds__(256) void k_rdm_occ(int64_t ndet, const uint32_t *sa, const uint32_t *sb,
                                                 const double *c, double *parts) {
    __shared__ double sm[3 * 256];
    const int lane = threadIdx.x & 63, orb = lane & 15, sub = lane >> 4;
    v4d t[3] = {};
    const int64_t nw = (int64_t)gridDim.x * 4;
    for (int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64; base < ndet; base += nw * 64) {
        const int64_t r = base + lane;
        const double ci = r < ndet ? c[r] : 0.0;
        const int ra = r < ndet ? (int)sa[r] : 0, rb = r < ndet ? (int)sb[r] : 0;
        double wi = ci * ci;
        // a weight that is not finite reaches only the pairs its row occupies
        for (uint64_t m = __ballot(!(fabs(wi) <= 1.7976931348623157e308)); m; m &= m - 1) {
            const int src = __builtin_ctzll(m);
            const double w = __shfl(wi, src, 64);
            const int a = __shfl(ra, src, 64), b = __shfl(rb, src, 64);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int k = sub + 4 * x;
                if ((a >> k) & (a >> orb) & 1) t[0][x] += w;
                if ((a >> k) & (b >> orb) & 1) t[1][x] += w;
                if ((b >> k) & (b >> orb) & 1) t[2][x] += w;
            }
            if (lane == src) wi = 0.0;
        }
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const double w = __shfl(wi, 4 * s + sub, 64);
            const double na = (__shfl(ra, 4 * s + sub, 64) >> orb) & 1 ? 1.0 : 0.0;
            const double nb = (__shfl(rb, 4 * s + sub, 64) >> orb) & 1 ? 1.0 : 0.0;
            t[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(na != 0.0 ? w : 0.0, na, t[0], 0, 0, 0);
            t[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(na != 0.0 ? w : 0.0, nb, t[1], 0, 0, 0);
            t[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(nb != 0.0 ? w : 0.0, nb, t[2], 0, 0, 0);
        }
    }
    // the four waves one after another, so the sum has a fixed order
    for (int w = 0; w < 4; ++w) {
        if ((threadIdx.x >> 6) == w) {
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = m * 256 + (sub + 4 * r) * 16 + orb;
                    sm[at] = w == 0 ? t[m][r] : sm[at] + t[m][r];
                }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < 3 * 256; i += 256) parts[(int64_t)blockIdx.x * 768 + i] = sm[i];
}

// out[i] = sum of parts[b][i], b < nb, in a fixed order: 64 entries and 16
// slices of the parts per workgroup.
__global__ __launch_bounds__(1024) void k_rdm_fold(const double *parts, int nb, int n, double *out) {
    __shared__ double sm[16][64];
    const int x = threadIdx.x & 63, slice = threadIdx.x >> 6;
    const int i = (int)blockIdx.x * 64 + x;
    double v = 0.0;
    if (i < n)
        for (int b = slice; b < nb; b += 16) v += parts[(int64_t)b * n + i];
    sm[slice][x] = v;
    __syncthreads();
    if (slice == 0 && i < n) {
        for (int s = 1; s < 16; ++s) v += sm[s][x];
        out[i] = v;
    }
}

// rdm1 / rdm2 from the class sums (tab) and the occupation products (occ).
__global__ __launch_bounds__(256) void k_rdm_expand(int norb, const double *tab, const double *occ, double *rdm1,
                                                    double *rdm2) {
    const int n = norb, n2 = n * n, P = orb_pairs(n);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n2 * n2) return;
    const int s = (int)(t % n), r = (int)((t / n) % n), q = (int)((t / n2) % n), p = (int)(t / ((int64_t)n2 * n));
    const double *D = tab, *Sc = tab + P * (P + 1), *Sx = Sc + P * n, *g1 = Sx + P * n;
    auto same = [&](int k, int l) { return occ[k * 16 + l] + occ[512 + k * 16 + l]; };  // aa + bb
    auto ab = [&](int k, int l) { return occ[256 + k * 16 + l]; };
    double v = 0.0;
    if (p != q && r != s) v = D[two_class(p, q, r, s)] * (orb_pair(p, q) == orb_pair(r, s) ? 2.0 : 1.0);
    double sc = 0.0, sx = 0.0, dg = 0.0;
    if (r == s && p != q) sc += Sc[orb_pair(p, q) * n + r];
    if (p == q && r != s) sc += Sc[orb_pair(r, s) * n + p];
    if (q == r && p != s) sx += Sx[orb_pair(p, s) * n + q];
    if (p == s && q != r) sx += Sx[orb_pair(q, r) * n + p];
    if (p == q && r == s) dg += (p != r ? same(p, r) : 0.0) + ab(p, r) + ab(r, p);
    if (q == r && p == s && p != q) dg -= same(p, q);
    rdm2[t] = v + sc - sx + dg;
    if (t < n2) {
        const int pp = (int)(t / n), qq = (int)(t % n);
        rdm1[t] = pp == qq ? same(pp, pp) : g1[orb_pair(pp, qq)];
    }
}

__global__ void k_grad(int norb, const double *rdm1, const double *rdm2, double scale, double *gh,
                       double *geri) {
    const int n = norb, n2 = n * n, n3 = n2 * n;
    const int64_t n4 = (int64_t)n2 * n2;
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n4) return;
    const int s = (int)(t % n), r = (int)((t / n) % n), q = (int)((t / n2) % n), p = (int)(t / n3);
    auto R = [&](int a, int b, int c, int d) { return rdm2[((a * n + b) * n + c) * n + d]; };
    double v = R(p, q, r, s) + R(q, p, r, s) + R(p, q, s, r) + R(q, p, s, r) + R(r, s, p, q) +
               R(s, r, p, q) + R(r, s, q, p) + R(s, r, q, p);
    geri[t] = scale * 0.5 * v / 8.0;
    if (t < n2) {
        const int pp = (int)(t / n), qq = (int)(t % n);
        gh[t] = scale * 0.5 * (rdm1[pp * n + qq] + rdm1[qq * n + pp]);
    }
}

}  // namespace

void rdm12_sorted(Ctx &c, const double *cs, double *rdm1, double *rdm2) {
    hipStream_t s = c.stream;
    const int n = c.norb;
    const int64_t n4 = (int64_t)n * n * n * n;
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c.device);
    if (n <= RDM_LDS_NORB) {
        // as many workgroups as stay resident, a multiple of 8 (one row range
        // per XCD), and no more than give every wave four rows
        const int nt = class_size(n);
        const size_t lds = sizeof(double) * (size_t)nt;
        const int per_cu = std::max(1, std::min<int>(2, (int)(160 * 1024 / (lds + 1024))));
        const int64_t want = (c.ndet + 4 * (RDM_NT / 64) - 1) / (4 * (RDM_NT / 64));
        const int nb = (int)std::max<int64_t>(8, (std::min<int64_t>((int64_t)cus * per_cu, want) + 7) / 8 * 8);
        const int nbo = (int)std::max<int64_t>(1, std::min<int64_t>((c.ndet + 1023) / 1024, cus));
        double *parts = c.cs.get<double>(2, (size_t)nb * nt + (size_t)nbo * 768);
        double *occp = parts + (size_t)nb * nt;
        double *sums = c.cs.get<double>(3, (size_t)nt + 768);
        RdmRows xr;
        for (int x = 0; x <= 8; ++x) xr.b[x] = c.xcd_rows[x];
        RdmArgs a{c.ndet, n, c.sa.p, c.sb.p, c.rowptr.p, c.col.p, c.desc.p, cs, nullptr, nullptr, nt};
        if (nt > 0) {  // two orbitals or more
            HQ_CHECK(hipFuncSetAttribute((const void *)k_rdm_lds, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)lds));
            hipLaunchKernelGGL(k_rdm_lds, dim3(nb), dim3(RDM_NT), lds, s, a, xr, parts);
            HQ_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_rdm_fold, dim3((nt + 63) / 64), dim3(1024), 0, s, parts, nb, nt, sums);
            HQ_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL(k_rdm_occ, dim3(nbo), dim3(256), 0, s, c.ndet, c.sa.p, c.sb.p, cs, occp);
        HQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_rdm_fold, dim3(12), dim3(1024), 0, s, occp, nbo, 768, sums + nt);
        HQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_rdm_expand, dim3(grid_for(n4, 256)), dim3(256), 0, s, n, sums, sums + nt, rdm1, rdm2);
        HQ_LAUNCH_CHECK();
        return;
    }
    const int ntab = tab_size(n);
    // accumulation copies in the context's call scratch (slots 2 and 3; slot
    // 0 may hold the gathered coefficients), kept for the next call
    double *g2c = c.cs.get<double>(2, (size_t)NCOPY * n4);
    double *tabc = c.cs.get<double>(3, (size_t)NCOPY * ntab);
    HQ_CHECK(hipMemsetAsync(g2c, 0, sizeof(double) * NCOPY * n4, s));
    HQ_CHECK(hipMemsetAsync(tabc, 0, sizeof(double) * NCOPY * ntab, s));
    RdmArgs a{c.ndet, n, c.sa.p, c.sb.p, c.rowptr.p, c.col.p, c.desc.p, cs, g2c, tabc, ntab};
    const size_t lds = sizeof(double) * (size_t)ntab;
    unsigned grid = (unsigned)std::min<int64_t>((c.ndet + 3) / 4, (int64_t)cus * 4);
    if (grid < 1) grid = 1;
    if (lds <= 150 * 1024) {
        HQ_CHECK(hipFuncSetAttribute((const void *)k_rdm<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds));
        hipLaunchKernelGGL(k_rdm<true>, dim3(grid), dim3(256), lds, s, a);
    } else {
        hipLaunchKernelGGL(k_rdm<false>, dim3(grid), dim3(256), 0, s, a);
    }
    HQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_rdm_assemble, dim3(grid_for(n4, 256)), dim3(256), 0, s, n, g2c, tabc, ntab,
                       rdm1, rdm2);
    HQ_LAUNCH_CHECK();
}

void integral_grad_sorted(Ctx &c, const double *cs, double scale, double *gh, double *geri) {
    hipStream_t s = c.stream;
    const int n = c.norb;
    const int64_t n4 = (int64_t)n * n * n * n;
    double *r1 = c.cs.get<double>(4, (size_t)n * n + (size_t)n4);  // rdm1, then rdm2
    double *r2 = r1 + (size_t)n * n;
    rdm12_sorted(c, cs, r1, r2);
    hipLaunchKernelGGL(k_grad, dim3(grid_for(n4, 256)), dim3(256), 0, s, n, r1, r2, scale, gh, geri);
    HQ_LAUNCH_CHECK();
}

}  // namespace hinqs
