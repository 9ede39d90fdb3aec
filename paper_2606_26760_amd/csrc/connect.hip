// Coupling enumeration: for every determinant x_i of B, every x_j of B that
// differs from it by one or two electrons, i.e. every pair with a possibly
// nonzero <x_i|H|x_j> (Slater-Condon rules; paper Sec. 2.2, Step 3 builds
// [H_B]_ij over exactly these pairs).
//
// The three classes are found without an O(|B|^2) scan:
//   alpha-only moves   x_j shares beta_i: scan the beta group of beta_i;
//   beta-only moves    x_j shares alpha_i: scan the alpha group of alpha_i;
//   alpha+beta moves   alpha_j is a single move of alpha_i present in B (alpha
//                      link table): scan that alpha group for beta strings one
//                      move away or, in groups of at least lookup_min rows
//                      (dense sets, e.g. product spaces), look each beta
//                      string one move away up by binary search.
// Each candidate is tested with XOR + popcount; the sign comes from masked
// popcounts (common.hpp).  The alpha-only class runs one thread per entry of
// the beta-major listing and the other two one thread per sorted row, so in
// both kernels neighbouring threads share the string whose groups they walk,
// which turns the string loads into scalar ones.  Small sets run one wave per
// row instead.  A counting pass sizes each
// row; a fill pass writes (col, desc), alpha-only entries first.  What bounds
// both: the tests, four vector instructions per pair of strings, and in the
// filling pass the descriptors of the hits (1e6 rows, 16 orbitals, 1.56e8
// couplings: counting 1.8 ms, filling 3.6; before the buffered stores, the
// scalar loads and the 32-string steps 2.7 and 5.0).
#include <chrono>
#include <cstdlib>

#include "common.hpp"

namespace hinqs {

namespace {

// Group scans test CONNECT_W candidates without branching, then emit the hits of
// that step from a bit mask: the emission code (descriptor and two stores)
// then runs about once per step instead of on every candidate where some lane
// of the wave happens to hit.  Entries keep their order.
struct ConnArgs {
    int64_t ndet;
    const uint32_t *sa, *sb;
    const int32_t *aidx, *bidx, *ga, *gb, *bperm;
    const uint32_t *bm_alpha;
    const int32_t *alink_cnt, *alink;
    const uint32_t *alink_info;
    int alink_max;
    int norb;
    int32_t lookup_min;  // alpha groups at least this long are searched, not scanned
};

// Alpha+beta couplings of a row with beta string bi into the alpha group
// [g0, g1) (rows sorted by beta string) by lookup: every beta string one move
// away from bi, generated in ascending order, is located by binary search in
// the part of the group not passed yet, so the hits come out with j ascending,
// as from the scan.  Ascending order: first the moves that lower the value
// (hole h from the highest occupied orbital down, then particle p < h
// upwards), then those that raise it (particle p from the lowest empty
// orbital up, then hole h < p downwards).
template <typename Emit>
__device__ inline void ab_lookup(const uint32_t *__restrict__ sb, int32_t g0, int32_t g1, uint32_t bi, int norb,
                                 Emit &&emit) {
    const uint32_t full = norb >= 32 ? 0xffffffffu : ((1u << norb) - 1u);
    const uint32_t emp = ~bi & full;
    int32_t lo = g0;
    auto find = [&](uint32_t v) {
        int32_t l = lo, h = g1;  // first position in [lo, g1) with sb >= v
        while (l < h) {
            const int32_t m = (l + h) >> 1;
            if (sb[m] < v) l = m + 1;
            else h = m;
        }
        lo = l;
        if (l < g1 && sb[l] == v) {
            emit(l);
            lo = l + 1;
        }
    };
    for (uint32_t hs = bi; hs;) {
        const int h = 31 - __builtin_clz(hs);
        hs &= ~(1u << h);
        for (uint32_t ps = emp & ((1u << h) - 1u); ps; ps &= ps - 1) find(bi ^ (1u << h) ^ (1u << lowbit(ps)));
    }
    for (uint32_t ps = emp; ps; ps &= ps - 1) {
        const int p = lowbit(ps);
        for (uint32_t hs = bi & ((1u << p) - 1u); hs;) {
            const int h = 31 - __builtin_clz(hs);
            hs &= ~(1u << h);
            find(bi ^ (1u << h) ^ (1u << p));
        }
    }
}

// Couplings a wave has found and not written yet: up to EMIT_CAP per lane (one
// row per lane) in LDS.  Written straight from the lanes, every 4-byte store of
// a wave went to 64 different rows (1.56e8 couplings: 5.0 ms, against 2.7 ms
// for the same tests without the stores); a flush writes up to sixteen
// consecutive couplings of a row with sixteen neighbouring lanes.
constexpr int CONNECT_W = 32;  // strings tested per step of a scan
constexpr int EMIT_CAP = 16;
constexpr int EMIT_STRIDE = EMIT_CAP + 1;  // keeps the lanes' slots in different banks
struct EmitBuf {
    int32_t col[64 * EMIT_STRIDE];
    uint32_t desc[64 * EMIT_STRIDE];
};

// out: the lane's next place in the matrix; n: couplings it holds.  Called by
// the whole wave.
__device__ inline void emit_flush(EmitBuf &b, int64_t &out, int &n, int lane, int32_t *col, uint32_t *desc) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int r0 = 0; r0 < 64; r0 += 64 / EMIT_CAP) {
        const int r = r0 + lane / EMIT_CAP, k = lane % EMIT_CAP;
        const int nr = __shfl(n, r, 64);
        const int64_t at = __shfl(out, r, 64) + k;
        if (k < nr) {
            col[at] = b.col[r * EMIT_STRIDE + k];
            desc[at] = b.desc[r * EMIT_STRIDE + k];
        }
    }
    __builtin_amdgcn_wave_barrier();
    out += n;
    n = 0;
}

// Tests every string in str[lo, hi) (per lane) against own, CONNECT_W at a
// time: hits(j0, mask) with bit u of the mask set where accept(bits that differ)
// of str[j0 + u] holds, at most EMIT_CAP of them.  Lanes that share the range
// (rows of one group) read it through the scalar cache.  Called by the whole
// wave; str is readable CONNECT_W strings past its end.
template <typename Accept, typename Hits>
__device__ inline void scan_strings(const uint32_t *__restrict__ str, int32_t lo, int32_t hi, uint32_t own,
                                    Accept &&accept, Hits &&hits) {
    auto test = [&](int32_t j0, int32_t end) {
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < CONNECT_W; ++u) m |= accept(popc32(own ^ str[j0 + u])) ? 1u << u : 0u;
        return end - j0 < CONNECT_W ? m & ((1u << (end - j0)) - 1u) : m;
    };
    auto report = [&](int32_t j0, uint32_t m) {
        if (__any(popc32(m) > EMIT_CAP)) {
            hits(j0, m & 0xffffu);
            hits(j0 + 16, m >> 16);
        } else {
            hits(j0, m);
        }
    };
    static_assert(CONNECT_W == 32 && EMIT_CAP >= 16, "halves fit");
    const int32_t ulo = __builtin_amdgcn_readfirstlane(lo), uhi = __builtin_amdgcn_readfirstlane(hi);
    if (__all(lo == ulo && hi == uhi)) {
        for (int32_t j0 = ulo; j0 < uhi; j0 += CONNECT_W) report(j0, test(j0, uhi));
    } else {
        for (int32_t j0 = lo; __any(j0 < hi); j0 += CONNECT_W) report(j0, j0 < hi ? test(j0, hi) : 0u);
    }
}

// Alpha-only moves (x_j shares beta_i), one thread per entry of the
// beta-major listing: neighbouring threads share beta_i and scan the same
// beta group, where one thread per sorted row would scan a different beta group
// on every lane.  Counting pass: n1[i]; filling pass: the row's first n1[i]
// entries.
template <bool FILL>
__global__ __launch_bounds__(256) void k_connect_beta(ConnArgs a, int32_t *n1, const int64_t *rowptr,
                                                      int32_t *col, uint32_t *desc) {
    __shared__ EmitBuf bufs[FILL ? 4 : 1];
    EmitBuf &buf = bufs[FILL ? threadIdx.x >> 6 : 0];
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = t < a.ndet;
    const int32_t i = live ? a.bperm[t] : 0;
    const uint32_t ai = live ? a.bm_alpha[t] : 0u;
    const int32_t bg = a.bidx[i];
    int64_t out = FILL ? rowptr[i] : 0;
    int n = 0;
    scan_strings(
        a.bm_alpha, live ? a.gb[bg] : 0, live ? a.gb[bg + 1] : 0, ai, [](int d) { return d == 2 || d == 4; },
        [&](int32_t t0, uint32_t m) {
            if (!FILL) {
                n += popc32(m);
                return;
            }
            if (__any(n + popc32(m) > EMIT_CAP)) emit_flush(buf, out, n, lane, col, desc);
            for (; m; m &= m - 1) {
                const int32_t u = t0 + lowbit(m);
                buf.col[lane * EMIT_STRIDE + n] = a.bperm[u];
                buf.desc[lane * EMIT_STRIDE + n] = same_spin_desc(ai, a.bm_alpha[u], HINQS_EXC_1A, HINQS_EXC_2AA);
                ++n;
            }
        });
    if (FILL) emit_flush(buf, out, n, lane, col, desc);
    else if (live) n1[i] = n;
}

// Beta-only and alpha+beta moves, one thread per sorted row (neighbouring
// rows share alpha_i and scan the same groups).  Counting
// pass: counts[i] = n1[i] + these; filling pass: after the row's n1[i]
// alpha-only entries.
template <bool FILL>
__global__ __launch_bounds__(256) void k_connect(ConnArgs a, const int32_t *n1, int64_t *counts,
                                                 const int64_t *rowptr, int32_t *col, uint32_t *desc) {
    __shared__ EmitBuf bufs[FILL ? 4 : 1];
    EmitBuf &buf = bufs[FILL ? threadIdx.x >> 6 : 0];
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = i < a.ndet;
    const int64_t at = live ? i : 0;
    const uint32_t bi = a.sb[at];
    const int32_t ag = a.aidx[at];
    int64_t out = FILL ? rowptr[at] + n1[at] : 0;
    int held = 0;   // filling: couplings in the buffer
    int64_t n = 0;  // counting
    auto found = [&](uint32_t m) {  // counts; or makes room for the hits
        if (!FILL) n += popc32(m);
        else if (__any(held + popc32(m) > EMIT_CAP)) emit_flush(buf, out, held, lane, col, desc);
    };
    auto put = [&](int32_t j, uint32_t d) {
        buf.col[lane * EMIT_STRIDE + held] = j;
        buf.desc[lane * EMIT_STRIDE + held] = d;
        ++held;
    };
    // beta-only: determinants with the same alpha string
    scan_strings(
        a.sb, live ? a.ga[ag] : 0, live ? a.ga[ag + 1] : 0, bi, [](int d) { return d == 2 || d == 4; },
        [&](int32_t j0, uint32_t m) {
            found(m);
            if (FILL)
                for (; m; m &= m - 1) {
                    const int32_t j = j0 + lowbit(m);
                    put(j, same_spin_desc(bi, a.sb[j], HINQS_EXC_1B, HINQS_EXC_2BB));
                }
        });
    // alpha + beta: alpha string one move away, beta string one move away
    const int64_t lbase = (int64_t)ag * a.alink_max;
    const int32_t le = live ? a.alink_cnt[ag] : 0;
    for (int32_t l = 0; __any(l < le); ++l) {
        int32_t t0 = 0, t1 = 0;
        int ha = 0, pa = 0;
        uint32_t npar = 0;
        if (l < le) {
            const int32_t tgt = a.alink[lbase + l];
            const uint32_t info = a.alink_info[lbase + l];
            ha = info & 31;
            pa = (info >> 5) & 31;
            npar = (info >> 10) & 1u;
            t0 = a.ga[tgt];
            t1 = a.ga[tgt + 1];
        }
        const bool search = t1 - t0 >= a.lookup_min;
        if (__any(search)) {
            if (FILL) emit_flush(buf, out, held, lane, col, desc);
            if (search) {
                ab_lookup(a.sb, t0, t1, bi, a.norb, [&](int32_t j) {
                    if (FILL) {
                        col[out] = j;
                        desc[out] = ab_desc(ha, pa, npar, bi, a.sb[j]);
                        ++out;
                    } else {
                        ++n;
                    }
                });
                t1 = t0;
            }
        }
        scan_strings(
            a.sb, t0, t1, bi, [](int d) { return d == 2; },
            [&](int32_t j0, uint32_t m) {
                found(m);
                if (FILL)
                    for (; m; m &= m - 1) {
                        const int32_t j = j0 + lowbit(m);
                        put(j, ab_desc(ha, pa, npar, bi, a.sb[j]));
                    }
            });
    }
    if (FILL) emit_flush(buf, out, held, lane, col, desc);
    else if (live) counts[i] = n1[i] + n;
}

// Every coupling of a row by one wave, for sets with too few rows to fill the
// chip one per lane (CONNECT_ROWS_MAX).  The lanes stride each group; the groups
// one move away are looked up 64 at a time, one per lane, so that only a group's
// strings are on the path of the loop.  Same order of the entries as above.
template <bool FILL>
__global__ __launch_bounds__(256) void k_connect_rows(ConnArgs a, int64_t *counts, const int64_t *rowptr,
                                                      int32_t *col, uint32_t *desc) {
    const int lane = threadIdx.x & 63;
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (i >= a.ndet) return;
    const uint32_t ai = a.sa[i], bi = a.sb[i];
    const int32_t ag = a.aidx[i], bg = a.bidx[i];
    int64_t out = FILL ? rowptr[i] : 0;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    auto emit = [&](bool keep, int32_t j, uint32_t d) {
        const uint64_t m = __ballot(keep);
        if (FILL && keep) {
            const int64_t k = out + __popcll(m & below);
            col[k] = j;
            desc[k] = d;
        }
        out += __popcll(m);
    };
    for (int32_t u0 = a.gb[bg], e = a.gb[bg + 1]; u0 < e; u0 += 64) {
        const int32_t u = u0 + lane;
        const uint32_t aj = u < e ? a.bm_alpha[u] : ai;
        const int d = popc32(ai ^ aj);
        const bool k = d == 2 || d == 4;
        emit(k, FILL && k ? a.bperm[u] : 0, FILL && k ? same_spin_desc(ai, aj, HINQS_EXC_1A, HINQS_EXC_2AA) : 0u);
    }
    for (int32_t j0 = a.ga[ag], e = a.ga[ag + 1]; j0 < e; j0 += 64) {
        const int32_t j = j0 + lane;
        const uint32_t bj = j < e ? a.sb[j] : bi;
        const int d = popc32(bi ^ bj);
        const bool k = d == 2 || d == 4;
        emit(k, j, FILL && k ? same_spin_desc(bi, bj, HINQS_EXC_1B, HINQS_EXC_2BB) : 0u);
    }
    const int64_t lbase = (int64_t)ag * a.alink_max;
    const int32_t le = a.alink_cnt[ag];
    for (int32_t l0 = 0; l0 < le; l0 += 64) {
        int32_t lo = 0, hi = 0;
        uint32_t info = 0;
        if (l0 + lane < le) {
            const int32_t tgt = a.alink[lbase + l0 + lane];
            info = a.alink_info[lbase + l0 + lane];
            lo = a.ga[tgt];
            hi = a.ga[tgt + 1];
        }
        const int nl = min(64, le - l0);
        // the first 64 strings of the next group are in flight while this one's are tested
        int32_t t0 = __shfl(lo, 0, 64), t1 = __shfl(hi, 0, 64);
        uint32_t b0 = t0 + lane < t1 ? a.sb[t0 + lane] : bi;
        for (int l = 0; l < nl; ++l) {
            const int32_t s0 = t0, s1 = t1;
            uint32_t bj = b0;
            const uint32_t inf = __shfl(info, l, 64);
            if (l + 1 < nl) {
                t0 = __shfl(lo, l + 1, 64);
                t1 = __shfl(hi, l + 1, 64);
                b0 = t0 + lane < t1 ? a.sb[t0 + lane] : bi;
            }
            for (int32_t j0 = s0;;) {
                const bool k = popc32(bi ^ bj) == 2;
                emit(k, j0 + lane, FILL && k ? ab_desc(inf & 31, (inf >> 5) & 31, (inf >> 10) & 1u, bi, bj) : 0u);
                j0 += 64;
                if (j0 >= s1) break;
                bj = j0 + lane < s1 ? a.sb[j0 + lane] : bi;
            }
        }
    }
    if (!FILL && lane == 0) counts[i] = out;
}

// bounds[x] = first row whose couplings start at or after x * total / 8 (x = 0..8).
__global__ void k_balance_bounds(int64_t n, const int64_t *rowptr, int64_t *bounds) {
    const int x = threadIdx.x;
    if (x > 8) return;
    const int64_t total = rowptr[n];
    if (x == 8) { bounds[8] = n; return; }
    const int64_t target = (total / 8) * x + (total % 8) * x / 8;
    int64_t lo = 0, hi = n;  // smallest r in [0, n] with rowptr[r] >= target
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (rowptr[mid] < target) lo = mid + 1;
        else hi = mid;
    }
    bounds[x] = lo;
}

__global__ void k_caller_counts(int64_t n, const int64_t *rowptr, const int32_t *perm, int64_t *counts) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    counts[perm[i]] = rowptr[i + 1] - rowptr[i];
}

// One wave per sorted row: copy its couplings to the caller-order position,
// translating column indices to caller indices.
__global__ void k_caller_copy(int64_t n, const int64_t *rowptr, const int32_t *col, const uint32_t *desc,
                              const int32_t *perm, const int64_t *rowptr_c, int32_t *col_c,
                              uint32_t *desc_c) {
    const int lane = threadIdx.x & 63;
    const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (row >= n) return;
    const int64_t beg = rowptr[row], end = rowptr[row + 1];
    const int64_t dst = rowptr_c[perm[row]];
    for (int64_t e = beg + lane; e < end; e += 64) {
        if (col_c) col_c[dst + (e - beg)] = perm[col[e]];
        if (desc_c) desc_c[dst + (e - beg)] = desc[e];
    }
}

// One wave per row up to here: with one row per lane, fewer rows leave most
// of the chip idle (both passes, one row per lane against one wave per row: 5,000 rows
// 166 / 82 us, 20,000 558 / 185, 60,000 797 / 484; 100,000 506 / 730, 200,000
// 909 / 1608, 1e6 5.7 / 16.3 ms).
constexpr int64_t CONNECT_ROWS_MAX = 65536;

int32_t env_i32(const char *name, int32_t dflt) {
    const char *v = std::getenv(name);
    return (v && *v) ? (int32_t)std::atoi(v) : dflt;
}

}  // namespace

void export_connectivity(Ctx &c, int64_t *rowptr_c, int32_t *col_c, uint32_t *desc_c) {
    hipStream_t s = c.stream;
    const int64_t n = c.ndet;
    DBuf<int64_t> counts;
    counts.ensure(n + 1);
    HQ_CHECK(hipMemsetAsync(counts.p + n, 0, sizeof(int64_t), s));
    hipLaunchKernelGGL(k_caller_counts, dim3(grid_for(n, 256)), dim3(256), 0, s, n, c.rowptr.p, c.perm.p,
                       counts.p);
    HQ_LAUNCH_CHECK();
    exclusive_scan_i64(s, counts.p, rowptr_c, n + 1, c.work);
    if (col_c || desc_c) {
        hipLaunchKernelGGL(k_caller_copy, dim3(grid_for(n * 64, 256)), dim3(256), 0, s, n, c.rowptr.p,
                           c.col.p, c.desc.p, c.perm.p, rowptr_c, col_c, desc_c);
        HQ_LAUNCH_CHECK();
    }
    wait_stream(s);
}

void compute_xcd_rows(Ctx &c) {
    hipStream_t s = c.stream;
    DBuf<int64_t> bnd;
    bnd.ensure(9);
    hipLaunchKernelGGL(k_balance_bounds, dim3(1), dim3(64), 0, s, c.ndet, c.rowptr.p, bnd.p);
    HQ_LAUNCH_CHECK();
    HQ_CHECK(hipMemcpyAsync(c.xcd_rows, bnd.p, sizeof(c.xcd_rows), hipMemcpyDeviceToHost, s));
    wait_stream(s);
}

void build_connectivity(Ctx &c, bool xcd_rows) {
    auto t0 = std::chrono::steady_clock::now();
    hipStream_t s = c.stream;
    const int64_t n = c.ndet;
    // lookups replace the scan only where a group is very long next to the
    // number of beta moves: a lookup is a binary search whose loads differ
    // from lane to lane, while a scan step tests 16 candidates with loads that
    // neighbouring threads share (measured: lookups in every group 4x slower
    // on the sampled 1e6 set, and no faster on product spaces with groups of
    // 1,716 and 3,432 rows)
    const int32_t nmoves = c.nb * (c.norb - c.nb);
    const int32_t lookup_min = env_i32("HINQS_CONNECT_LOOKUP_MIN", std::max<int32_t>(4096, 64 * nmoves));
    ConnArgs a{n,          c.sa.p,        c.sb.p,        c.aidx.p,  c.bidx.p,
               c.ga.p,     c.gb.p,        c.bperm.p, c.bm_alpha.p,  c.alink_ptr.p,
               c.alink.p,  c.alink_info.p, c.alink_max, c.norb, lookup_min};
    auto &counts = c.bs.counts;
    auto &n1 = c.bs.gidx;  // alpha-only couplings per row (free once the tables are built)
    counts.ensure(n + 1);
    n1.ensure(n);
    // the per-lane kernel keeps the lookup of very long groups (a set of at most
    // CONNECT_ROWS_MAX rows has one only if HINQS_CONNECT_LOOKUP_MIN asks)
    const bool by_rows = n <= CONNECT_ROWS_MAX && env_i32("HINQS_CONNECT_LOOKUP_MIN", 0) == 0;
    const dim3 g(grid_for(by_rows ? 64 * n : n, 256)), b(256);
    if (by_rows) {
        hipLaunchKernelGGL(k_connect_rows<false>, g, b, 0, s, a, counts.p, (const int64_t *)nullptr,
                           (int32_t *)nullptr, (uint32_t *)nullptr);
        HQ_LAUNCH_CHECK();
    } else {
        hipLaunchKernelGGL(k_connect_beta<false>, g, b, 0, s, a, n1.p, (const int64_t *)nullptr, (int32_t *)nullptr,
                           (uint32_t *)nullptr);
        HQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_connect<false>, g, b, 0, s, a, (const int32_t *)n1.p, counts.p,
                           (const int64_t *)nullptr, (int32_t *)nullptr, (uint32_t *)nullptr);
        HQ_LAUNCH_CHECK();
    }
    HQ_CHECK(hipMemsetAsync(counts.p + n, 0, sizeof(int64_t), s));
    c.rowptr.ensure(n + 1);
    exclusive_scan_i64(s, counts.p, c.rowptr.p, n + 1, c.work);
    int64_t nnz = 0;
    HQ_CHECK(hipMemcpyAsync(&nnz, c.rowptr.p + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    wait_stream(s);
    if (nnz >= ((int64_t)1 << 40)) throw Error(HINQS_E_UNSUPPORTED, "too many couplings");
    c.nnz = nnz;
    c.col.ensure(nnz);
    c.desc.ensure(nnz);
    if (by_rows) {
        hipLaunchKernelGGL(k_connect_rows<true>, g, b, 0, s, a, (int64_t *)nullptr, c.rowptr.p, c.col.p, c.desc.p);
        HQ_LAUNCH_CHECK();
    } else {
        hipLaunchKernelGGL(k_connect_beta<true>, g, b, 0, s, a, (int32_t *)nullptr, c.rowptr.p, c.col.p, c.desc.p);
        HQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_connect<true>, g, b, 0, s, a, (const int32_t *)n1.p, (int64_t *)nullptr, c.rowptr.p,
                           c.col.p, c.desc.p);
        HQ_LAUNCH_CHECK();
    }
    if (xcd_rows) compute_xcd_rows(c);
    for (auto &row : c.sigma_cfg)
        for (auto &g : row) g = SigmaCfg{};
    c.ms_connect =
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

}  // namespace hinqs
