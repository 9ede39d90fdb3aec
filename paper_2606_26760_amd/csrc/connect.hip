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
#include "enumerate.hpp"

namespace hinqs {

namespace {

constexpr int CONNECT_W = 32;  // strings tested per step of a scan

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
    const int32_t *rows = nullptr;  // k_connect_rows: the ndet rows to enumerate, nullptr: all
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
    scan_strings<CONNECT_W>(
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
    scan_strings<CONNECT_W>(
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
        scan_strings<CONNECT_W>(
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

// Hits of RW rows on their way to the matrix, a ring per row.
template <int RW>
struct RowQueue {
    int32_t j[RW][128];
    uint32_t str[RW][128], info[RW][128];
};

// Every coupling of RW rows by one wave, for sets with too few rows to fill the
// chip one per lane (CONNECT_ROWS_MAX) and for listed rows, which share their
// strings with few others of the list.  The lanes stride each group; the groups
// one move away are looked up 64 at a time, one per lane, and the next group's
// strings are on their way while one's are tested.  Rows of the wave with the same
// alpha string are tested against a group's strings together.  Bound by the
// instructions of a step, so hits, two or three per row and group, only go to a
// queue: their descriptors are computed 64 at a time, and stored next to each
// other (75,000 rows of 1e6, 1.2e7 couplings, counting / filling: row by row with
// the descriptors in each step 0.54 / 0.85 ms, RW = 1 0.55 / 0.69, RW = 4 0.44 /
// 0.64, RW = 8 0.58 / 1.03).
// Same order of the entries as above.
template <bool FILL, int RW>
__global__ __launch_bounds__(256) void k_connect_rows(ConnArgs a, int64_t *counts, const int64_t *rowptr,
                                                      int32_t *col, uint32_t *desc) {
    constexpr uint32_t ALPHA = 0xffffffffu, BETA = 0xfffffffeu;  // info of same-spin hits
    __shared__ RowQueue<FILL ? RW : 1> queues[FILL ? 4 : 1];
    RowQueue<FILL ? RW : 1> &queue = queues[FILL ? threadIdx.x >> 6 : 0];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6));
    const int64_t t0 = wave * (int64_t)RW;
    if (t0 >= a.ndet) return;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    int64_t row[RW], out[RW];
    uint32_t ai[RW], bi[RW];
    int32_t ag[RW], bg[RW], held[RW], head[RW];
    int64_t n[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const bool live = t0 + r < a.ndet;
        row[r] = live ? (a.rows ? (int64_t)a.rows[t0 + r] : t0 + r) : -1;
        const int64_t i = live ? row[r] : 0;
        ai[r] = a.sa[i];
        bi[r] = a.sb[i];
        ag[r] = live ? a.aidx[i] : -1;
        bg[r] = a.bidx[i];
        out[r] = FILL ? rowptr[i] : 0;
        n[r] = 0;
        held[r] = head[r] = 0;
    }
    auto flush = [&](int r, int cnt) {  // the oldest cnt hits of row r
        __builtin_amdgcn_wave_barrier();
        if (lane < cnt) {
            const int at = (head[r] + lane) & 127;
            const int32_t j = queue.j[r][at];
            const uint32_t s = queue.str[r][at], inf = queue.info[r][at];
            uint32_t d;
            if (inf == ALPHA) d = same_spin_desc(ai[r], s, HINQS_EXC_1A, HINQS_EXC_2AA);
            else if (inf == BETA) d = same_spin_desc(bi[r], s, HINQS_EXC_1B, HINQS_EXC_2BB);
            else d = ab_desc(inf & 31, (inf >> 5) & 31, (inf >> 10) & 1u, bi[r], s);
            col[out[r] + lane] = inf == ALPHA ? a.bperm[j] : j;
            desc[out[r] + lane] = d;
        }
        __builtin_amdgcn_wave_barrier();
        out[r] += cnt;
        held[r] -= cnt;
        head[r] = (head[r] + cnt) & 127;
    };
    auto emit = [&](int r, bool keep, int32_t j, uint32_t s, uint32_t inf) {
        const uint64_t m = __ballot(keep);
        if (!FILL) {
            n[r] += __popcll(m);
        } else if (m) {
            if (keep) {
                const int at = (head[r] + held[r] + __popcll(m & below)) & 127;
                queue.j[r][at] = j;
                queue.str[r][at] = s;
                queue.info[r][at] = inf;
            }
            held[r] += __popcll(m);
            if (held[r] >= 64) flush(r, 64);
        }
    };
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        if (ag[r] < 0) continue;
        for (int32_t u0 = a.gb[bg[r]], e = a.gb[bg[r] + 1]; u0 < e; u0 += 64) {
            const int32_t u = u0 + lane;
            const uint32_t aj = u < e ? a.bm_alpha[u] : ai[r];
            const int d = popc32(ai[r] ^ aj);
            emit(r, d == 2 || d == 4, u, aj, ALPHA);
        }
    }
    // runs of rows with one alpha string
    for (int r0 = 0; r0 < RW;) {
        int32_t g = -1;
        bool in[RW];
        int next = RW;
#pragma unroll
        for (int r = RW - 1; r >= 0; --r)
            if (r == r0) g = ag[r];
        if (g < 0) break;
#pragma unroll
        for (int r = RW - 1; r >= 0; --r)
            if (r > r0 && ag[r] != g) next = r;
#pragma unroll
        for (int r = 0; r < RW; ++r) in[r] = r >= r0 && r < next;
        for (int32_t j0 = a.ga[g], e = a.ga[g + 1]; j0 < e; j0 += 64) {
            const int32_t j = j0 + lane;
            const uint32_t sj = j < e ? a.sb[j] : 0u;
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (in[r]) {
                    const int d = popc32(bi[r] ^ sj);
                    emit(r, j < e && (d == 2 || d == 4), j, sj, BETA);
                }
        }
        const int64_t lbase = (int64_t)g * a.alink_max;
        const int32_t le = a.alink_cnt[g];
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
            int32_t s0 = __builtin_amdgcn_readlane(lo, 0), s1 = __builtin_amdgcn_readlane(hi, 0);
            uint32_t b0 = s0 + lane < s1 ? a.sb[s0 + lane] : 0u;
            for (int l = 0; l < nl; ++l) {
                const int32_t g0 = s0, g1 = s1;
                uint32_t bj = b0;
                const uint32_t inf = __builtin_amdgcn_readlane(info, l) & 0x7ffu;
                if (l + 1 < nl) {
                    s0 = __builtin_amdgcn_readlane(lo, l + 1);
                    s1 = __builtin_amdgcn_readlane(hi, l + 1);
                    b0 = s0 + lane < s1 ? a.sb[s0 + lane] : 0u;
                }
                for (int32_t j0 = g0;;) {
                    const bool ok = j0 + lane < g1;
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        if (in[r]) emit(r, ok && popc32(bi[r] ^ bj) == 2, j0 + lane, bj, inf);
                    j0 += 64;
                    if (j0 >= g1) break;
                    bj = j0 + lane < g1 ? a.sb[j0 + lane] : 0u;
                }
            }
        }
        r0 = next;
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        if (row[r] < 0) continue;
        if (FILL) flush(r, held[r]);
        else if (lane == 0) counts[row[r]] = n[r];
    }
}

// RW = 4 needs enough rows to leave several waves per SIMD (both passes of a whole
// set, RW = 1 / 4: 20,000 rows 142 / 151 us, 60,000 rows 375 / 298 us).
constexpr int64_t CONNECT_RW4_MIN = 32768;
template <bool FILL>
void launch_connect_rows(hipStream_t s, const ConnArgs &a, int64_t *counts, const int64_t *rowptr, int32_t *col,
                         uint32_t *desc) {
    if (a.ndet >= CONNECT_RW4_MIN)
        hipLaunchKernelGGL((k_connect_rows<FILL, 4>), dim3(grid_for((a.ndet + 3) / 4 * 64, 256)), dim3(256), 0, s, a,
                           counts, rowptr, col, desc);
    else
        hipLaunchKernelGGL((k_connect_rows<FILL, 1>), dim3(grid_for(a.ndet * 64, 256)), dim3(256), 0, s, a, counts,
                           rowptr, col, desc);
    HQ_LAUNCH_CHECK();
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

// One wave for a row, or four, up to here: with one row per lane, fewer rows leave
// most of the chip idle, and past it groups of thousands of rows are looked up
// (both passes, one row per lane against this: 5,000 rows 166 / 70 us, 20,000
// 558 / 147, 60,000 797 / 298; 100,000 513 / 481, 200,000 907 / 899 and, with
// longer groups, 2074 / 1673; 3 groups of 60,000 rows 8.3 / 16.7 ms).
constexpr int64_t CONNECT_ROWS_MAX = 65536;

int32_t env_i32(const char *name, int32_t dflt) {
    const char *v = std::getenv(name);
    return (v && *v) ? (int32_t)std::atoi(v) : dflt;
}

}  // namespace

void connect_listed_rows(Ctx &c, const int32_t *rows, int64_t nrows, int64_t *counts, bool fill) {
    const ConnArgs a{nrows,      c.sa.p,        c.sb.p,        c.aidx.p,    c.bidx.p, c.ga.p, c.gb.p,
                     c.bperm.p,  c.bm_alpha.p,  c.alink_ptr.p, c.alink.p,   c.alink_info.p,
                     c.alink_max, c.norb,       0,             rows};
    if (fill) launch_connect_rows<true>(c.stream, a, nullptr, c.rowptr.p, c.col.p, c.desc.p);
    else launch_connect_rows<false>(c.stream, a, counts, nullptr, nullptr, nullptr);
}

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
    // from lane to lane, while a scan step tests CONNECT_W candidates with loads
    // that neighbouring threads share (against steps of 16 strings: lookups in
    // every group 4x slower on the sampled 1e6 set, and no faster on product
    // spaces with groups of 1,716 and 3,432 rows)
    const int32_t nmoves = c.nb * (c.norb - c.nb);
    const int32_t lookup_min = env_i32("HINQS_CONNECT_LOOKUP_MIN", std::max<int32_t>(4096, 64 * nmoves));
    ConnArgs a{n,          c.sa.p,        c.sb.p,        c.aidx.p,  c.bidx.p,
               c.ga.p,     c.gb.p,        c.bperm.p, c.bm_alpha.p,  c.alink_ptr.p,
               c.alink.p,  c.alink_info.p, c.alink_max, c.norb, lookup_min};
    auto &counts = c.bs.counts;
    auto &n1 = c.bs.gidx;  // alpha-only couplings per row (free once the tables are built)
    counts.ensure(n + 1);
    n1.ensure(n);
    // very long groups are scanned too where a wave takes a row (5 alpha strings with
    // 12,870 rows each: 2.4 ms, looked up one row per lane 4.2), unless
    // HINQS_CONNECT_LOOKUP_MIN asks for the lookup
    const bool by_rows = n <= CONNECT_ROWS_MAX && env_i32("HINQS_CONNECT_LOOKUP_MIN", 0) == 0;
    const dim3 g(grid_for(n, 256)), b(256);
    if (by_rows) {
        launch_connect_rows<false>(s, a, counts.p, nullptr, nullptr, nullptr);
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
        launch_connect_rows<true>(s, a, nullptr, c.rowptr.p, c.col.p, c.desc.p);
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
