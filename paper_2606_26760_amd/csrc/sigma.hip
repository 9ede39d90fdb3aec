// Block sigma product S = H_B X over the stored couplings (paper Sec. 2.2,
// Step 3: the product the Davidson iteration repeats).
//
// Layout: CSR over sorted rows (rowptr int64, col int32, val fp64/fp32) plus
// the diagonal; X and S are ndet x K row-major with leading dimensions, so a
// row of X for K = 8 doubles is one 64-byte segment.  A team of lanes owns
// one row; groups of lanes inside the team share one coupling and gather its
// X row as one contiguous segment (16 bytes per lane), while the CSR stream is
// read with non-temporal loads so it does not evict X from the caches.  The
// partial sums are combined with a butterfly of cross-lane shuffles.  Every
// row is written by exactly one team, so the result is deterministic and
// atomic-free.
//
// Workgroups are remapped so each XCD (8 on MI355X, round-robin dispatch)
// receives a contiguous range of rows: rows with the same alpha string gather
// the same X rows, and keeping them on one XCD keeps those X rows in its L2.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <utility>

#include "common.hpp"

namespace hinqs {

namespace {

constexpr int SIGMA_BLOCK = 256;
constexpr int NUM_XCD = 8;

// One 16-byte vector of T (2 doubles or 4 floats).
template <typename T>
struct Vec16;
template <>
struct Vec16<double> { using type = double2; static constexpr int n = 2; };
template <>
struct Vec16<float> { using type = float4; static constexpr int n = 4; };

// A value known to be equal on all lanes of the wave, moved to a scalar register
// so that loops over it branch on the scalar unit.
template <bool UNIFORM>
__device__ inline int64_t uniform_if(int64_t v) {
    if constexpr (UNIFORM) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    } else {
        return v;
    }
}

template <typename T, int N>
__device__ inline void load_vec(const T *p, T (&x)[N]) {
    if constexpr (N * sizeof(T) == 16) {
        using V = typename Vec16<T>::type;
        V v = *(const V *)p;
        if constexpr (N == 2) { x[0] = v.x; x[1] = v.y; }
        else { x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w; }
    } else {
#pragma unroll
        for (int c = 0; c < N; ++c) x[c] = p[c];
    }
}

template <typename T, int N>
__device__ inline void store_vec(T *p, const T (&x)[N]) {
    if constexpr (N * sizeof(T) == 16) {
        using V = typename Vec16<T>::type;
        V v;
        if constexpr (N == 2) { v.x = x[0]; v.y = x[1]; }
        else { v.x = x[0]; v.y = x[1]; v.z = x[2]; v.w = x[3]; }
        *(V *)p = v;
    } else {
#pragma unroll
        for (int c = 0; c < N; ++c) p[c] = x[c];
    }
}

// The entries of a row of S that one lane holds, columns c0 .. c0 + N - 1, to the
// caller's row: whole vectors, or the columns that there are, one by one.
template <typename T, int N>
__device__ inline void store_row(T *S, int64_t row, int lds, int c0, const SigmaOut &out, const T (&x)[N]) {
    T *p = S + row * lds + c0;
    if (out.cols == 0) {
        store_vec<T, N>(p, x);
    } else {
#pragma unroll
        for (int c = 0; c < N; ++c)
            if (c0 + c < out.cols) p[c] = x[c];
    }
}

// The 32 bits that lane U of each group of LPN neighbouring lanes holds, on every
// lane of the group (DPP moves; LPN in {1, 2, 4, 8}).
template <int LPN, int U>
__device__ inline int group_bcast(int x) {
    if constexpr (LPN == 1) return x;
    else if constexpr (LPN == 2) return __builtin_amdgcn_update_dpp(x, x, U == 0 ? 0xa0 : 0xf5, 0xf, 0xf, false);
    else if constexpr (LPN == 4) return __builtin_amdgcn_update_dpp(x, x, U * 0x55, 0xf, 0xf, false);
    else {  // lane U of a row of 16 to its first half, lane 8 + U to its second
        const int lo = __builtin_amdgcn_update_dpp(x, x, 0x150 + U, 0xf, 0x3, false);
        return __builtin_amdgcn_update_dpp(lo, x, 0x158 + U, 0xf, 0xc, false);
    }
}
template <int LPN, int U>
__device__ inline float group_bcast(float x) {
    return __int_as_float(group_bcast<LPN, U>(__float_as_int(x)));
}
template <int LPN, int U>
__device__ inline double group_bcast(double x) {
    return __hiloint2double(group_bcast<LPN, U>(__double2hiint(x)), group_bcast<LPN, U>(__double2loint(x)));
}
template <int... I, typename F>
__device__ inline void static_for_seq(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ inline void static_for(F &&f) {
    static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

// Persistent teams: TEAM lanes own one row at a time and walk a strided list
// of rows.  Rows are split into 8 contiguous ranges holding equal numbers of
// couplings, one per XCD (hardware block b runs on XCD b % 8; the coupling
// count per row varies several-fold along the sorted order, so equal row
// counts would leave most XCDs idle behind the densest one), and inside a
// range consecutive teams take
// consecutive rows, so the rows in flight on an XCD are neighbours in the
// sorted order and gather overlapping X rows from that XCD's L2.  LPN lanes
// share one coupling: each loads EPL consecutive entries (16 bytes) of the
// gathered X row, so one load instruction touches 64 / LPN distinct rows and
// every row is read as one contiguous segment.
// What bounds the product is the return path of a CU's loads: about 20 clk per
// load instruction whatever it brings, 75 % busy when the LPN lanes of a coupling
// each fetched its column and value.  So every lane fetches the column and value
// of a coupling of its own, and the group takes its LPN couplings in turn, handing
// each around by DPP: half the load instructions per coupling for k = 8 (FP64,
// 20,000 rows, 7.1e6 couplings 69 -> 53 us, 1e6 rows, 1.56e8 1750 -> 1500).  Past
// that it is the lines that miss L1, 0.8 per coupling at 2.4 clk from L2 and 10 from
// beyond it (1e6 rows: 40 % of them).  Larger workgroups, the first fetch of the
// next row ahead of a row's end and its diagonal element ahead were within 8 %
// either way.
// The CSR stream is software-pipelined: while the X rows of one step (CH
// couplings per lane) are in flight, the (col, val) of the next step and the
// bounds of the team's next row are already being fetched, so the dependent
// load chain rowptr -> col -> X costs one memory latency per step, not three.
struct XcdRows {
    int64_t b[NUM_XCD + 1];
};

// MASK (batched instances): the XCD row ranges come from device memory and the
// rows of finished instances are skipped; a team jumps over a finished
// instance in one step, so the cost does not grow with its size.
// Row counters (ctr, not for MASK; sets above SIGMA_STATIC_NNZ couplings, see
// row_run): instead of a fixed stride, the team leader takes the XCD's next run
// of `run` rows from a counter, so the teams of an XCD stay on neighbouring rows
// however unequal the rows are; with fixed strides the
// teams drift apart and the X rows in flight no longer share the XCD's L2
// (a trace-driven model of the gathers gives 53 % L2 hits for strides and
// 80 % for a shared counter).  The next run is requested when a run starts,
// so the atomic's latency hides behind the current rows; runs of several
// rows keep the counters from becoming a hot spot in their L2 channels.  The
// last team of an XCD to finish puts its counters back to zero for the next
// launch.  ctr: CTR_STRIDE words per XCD, word 0 = next row, word
// CTR_DONE = teams finished.
constexpr int CTR_STRIDE = SIGMA_CTR_WORDS / NUM_XCD;
constexpr int CTR_DONE = 16;

template <typename T, int K, int TEAM, int UNR, bool MASK>
__global__ __launch_bounds__(SIGMA_BLOCK) void k_sigma(XcdRows ranges, SigmaMask mk, int xcd_map,
                                                       const int64_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ col,
                                                       const T *__restrict__ val,
                                                       const T *__restrict__ diag,
                                                       const T *__restrict__ X, int ldx,
                                                       T *__restrict__ S, int lds, SigmaOut out,
                                                       unsigned long long *ctr, int run) {
    constexpr int VW = Vec16<T>::n;
    constexpr int LPN = (K >= VW) ? K / VW : 1;   // lanes per coupling
    constexpr int EPL = K / LPN;                   // entries of X per lane
    constexpr int CH = (UNR + LPN - 1) / LPN;      // couplings that a lane fetches per step
    constexpr int STEP = CH * TEAM;                // couplings per team step
    constexpr int TPB = SIGMA_BLOCK / TEAM;        // teams per block
    static_assert(TEAM % LPN == 0 && TEAM <= 64, "team shape");
    const int64_t blocks_per_xcd = gridDim.x / NUM_XCD;
    const int xcd = xcd_map ? blockIdx.x % NUM_XCD : blockIdx.x / blocks_per_xcd;
    const int64_t bix = xcd_map ? blockIdx.x / NUM_XCD : blockIdx.x % blocks_per_xcd;
    const int64_t team0 = bix * TPB + threadIdx.x / TEAM;
    const int64_t nteams = blocks_per_xcd * TPB;
    const int64_t r0 = MASK ? mk.ranges[xcd] : ranges.b[xcd];
    const int64_t r1 = MASK ? mk.ranges[xcd + 1] : ranges.b[xcd + 1];
    const int sub = threadIdx.x % TEAM;
    const int q = sub % LPN, g = sub / LPN;
    const T *Xq = X + q * EPL;
    // MASK: instance of the last row looked up (rows only increase)
    int64_t inst_end = -1;
    bool inst_done = false;
    auto live_row = [&](int64_t rw) -> int64_t {
        if constexpr (MASK) {
            while (rw < r1) {
                if (rw >= inst_end) {
                    const int32_t b = mk.row_inst[rw];
                    inst_end = mk.inst_row[b + 1];
                    inst_done = mk.done[b] != 0;
                }
                if (!inst_done) break;
                rw += (inst_end - rw + nteams - 1) / nteams * nteams;
            }
        }
        return rw;
    };
    const bool dyn = !MASK && ctr != nullptr;
    unsigned long long *const myctr = dyn ? ctr + xcd * CTR_STRIDE : nullptr;
    auto take = [&]() -> unsigned long long {  // result valid on the team leader only
        unsigned long long v = 0;
        if (sub == 0) v = atomicAdd(myctr, (unsigned long long)run);
        return v;
    };
    auto first_row = [&](unsigned long long v) -> int64_t { return r0 + (int64_t)__shfl(v, 0, TEAM); };
    int64_t run_end = 0;  // end of the run of rows taken last
    auto finish = [&]() {
        if (dyn && sub == 0) {
            const unsigned long long d = atomicAdd(myctr + CTR_DONE, 1ull);
            if (d + 1 == (unsigned long long)nteams) {
                atomicExch(myctr, 0ull);
                atomicExch(myctr + CTR_DONE, 0ull);
            }
        }
    };
    unsigned long long pend = 0;
    int64_t row;
    if (dyn) {
        row = first_row(take());
        run_end = min(row + run, r1);
        if (row < r1) pend = take();
    } else {
        row = live_row(r0 + team0);
    }
    if (row >= r1) {  // uniform across the team
        finish();
        return;
    }
    int64_t beg = uniform_if<TEAM == 64>(rowptr[row]), end = uniform_if<TEAM == 64>(rowptr[row + 1]);
    int32_t srow = !MASK && out.row ? out.row[row] : (int32_t)row;
    for (;;) {
        int64_t nrow;
        if (dyn) {
            if (row + 1 < run_end) {
                nrow = row + 1;
            } else {
                nrow = first_row(pend);
                run_end = min(nrow + run, r1);
                if (nrow < r1) pend = take();
            }
        } else {
            nrow = live_row(row + nteams);
        }
        // next row's bounds, in flight during this row (clamped, not predicated)
        const int64_t nrc = nrow < r1 ? nrow : row;
        const int64_t nbeg = rowptr[nrc], nend = rowptr[nrc + 1];
        const int32_t nsrow = !MASK && out.row ? out.row[nrc] : (int32_t)nrc;
        T acc[EPL];
#pragma unroll
        for (int c = 0; c < EPL; ++c) acc[c] = T(0);
        // Software pipeline with two register sets (a, b): while the X rows of
        // one step are in flight, the (col, val) of the next step are fetched
        // into the other set, so no loop-carried copy has to wait for a load.
        // Loads are never predicated: indices past the row are clamped to a
        // valid entry and their value is replaced by 0 at the point of use.
        const int64_t last = end > 0 ? end - 1 : 0;
        int32_t ja[CH], jb[CH];
        T va[CH], vb[CH];
        bool oka[CH], okb[CH];
        auto fetch = [&](int64_t eb, int32_t (&jj)[CH], T (&vv)[CH], bool (&ok)[CH]) {
#pragma unroll
            for (int v = 0; v < CH; ++v) {
                const int64_t idx = eb + v * TEAM + sub;
                ok[v] = idx < end;
                const int64_t idc = ok[v] ? idx : last;
                jj[v] = __builtin_nontemporal_load(col + idc);
                vv[v] = __builtin_nontemporal_load(val + idc);
            }
        };
        auto step = [&](const int32_t (&jj)[CH], const T (&vv)[CH], const bool (&ok)[CH],
                        int64_t eb_next, int32_t (&jn)[CH], T (&vn)[CH], bool (&okn)[CH]) {
            T x[CH][LPN][EPL], w[CH];
#pragma unroll
            for (int v = 0; v < CH; ++v) {
                const int32_t jr = ok[v] ? jj[v] : (int32_t)row;
                w[v] = ok[v] ? vv[v] : T(0);
                static_for<LPN>([&](auto u) {
                    load_vec<T, EPL>(Xq + (int64_t)group_bcast<LPN, u>(jr) * ldx, x[v][u]);
                });
            }
            fetch(eb_next, jn, vn, okn);
#pragma unroll
            for (int v = 0; v < CH; ++v)
                static_for<LPN>([&](auto u) {
                    const T wu = group_bcast<LPN, u>(w[v]);
#pragma unroll
                    for (int c = 0; c < EPL; ++c) acc[c] += wu * x[v][u][c];
                });
        };
        int64_t eb = beg;
        fetch(eb, ja, va, oka);
        while (eb < end) {  // same trip count on every lane of the team
            step(ja, va, oka, eb + STEP, jb, vb, okb);
            eb += STEP;
            if (eb >= end) break;
            step(jb, vb, okb, eb + STEP, ja, va, oka);
            eb += STEP;
        }
#pragma unroll
        for (int off = LPN; off < TEAM; off <<= 1) {
#pragma unroll
            for (int c = 0; c < EPL; ++c) acc[c] += __shfl_xor(acc[c], off, TEAM);
        }
        if (g == 0) {
            if (diag) {   // null: off-diagonal part only (the caller adds the diagonal itself)
                const T d = diag[row];
                T xr[EPL];
                load_vec<T, EPL>(Xq + row * ldx, xr);
#pragma unroll
                for (int c = 0; c < EPL; ++c) acc[c] += d * xr[c];
            }
            store_row<T, EPL>(S, srow, lds, q * EPL, out, acc);
        }
        if (nrow >= r1) break;
        row = nrow;
        srow = nsrow;
        beg = uniform_if<TEAM == 64>(nbeg);
        end = uniform_if<TEAM == 64>(nend);
    }
    finish();
}

// Small sets (at most SIGMA_SMALL_ROWS rows): one wave per row, in whatever
// order the caller's vectors are (perm: sorted position -> caller index; null:
// sorted), any k up to K and any alignment (VEC: k == K and 16-byte aligned
// rows).  Such a product is bound by launches, not by its gathers: staging
// caller-order vectors took two more kernels (400 rows, k = 1: 12.8 us per call
// with them, 5 us for this kernel alone), and the lookup perm[col] stays in L1.
// Couplings are fetched one per lane and handed around as in k_sigma (8,192 rows of
// 165 couplings, caller order, k = 8 / 16: 14.6 / 24.3 us with a fetch on every lane
// of a coupling, 10.4 / 12.9 us).
template <typename T, int K, bool VEC>
__global__ __launch_bounds__(SIGMA_BLOCK) void k_sigma_small(int64_t ndet, const int64_t *__restrict__ rowptr,
                                                             const int32_t *__restrict__ col,
                                                             const T *__restrict__ val, const T *__restrict__ diag,
                                                             const int32_t *__restrict__ perm,
                                                             const T *__restrict__ X, int k, T *__restrict__ S) {
    constexpr int VW = Vec16<T>::n;
    constexpr int LPN = (K >= VW) ? K / VW : 1;
    constexpr int EPL = K / LPN;
    constexpr int CH = LPN >= 4 ? 1 : 4 / LPN;  // couplings that a lane fetches per step
    const int lane = threadIdx.x & 63, q = lane % LPN, g = lane / LPN;
    const int64_t row = uniform_if<true>((int64_t)blockIdx.x * (SIGMA_BLOCK / 64) + (threadIdx.x >> 6));
    if (row >= ndet) return;
    const int c0 = q * EPL;
    auto load = [&](int64_t r, T (&x)[EPL]) {
        if constexpr (VEC) {
            load_vec<T, EPL>(X + r * K + c0, x);
        } else {
#pragma unroll
            for (int c = 0; c < EPL; ++c) x[c] = c0 + c < k ? X[r * k + c0 + c] : T(0);
        }
    };
    const int64_t beg = uniform_if<true>(rowptr[row]), end = uniform_if<true>(rowptr[row + 1]);
    const int64_t orow = perm ? perm[row] : row;
    T acc[EPL], own[EPL];
#pragma unroll
    for (int c = 0; c < EPL; ++c) acc[c] = T(0);
    load(orow, own);
    const T d = diag ? diag[row] : T(0);
    for (int64_t e0 = beg; e0 + g * LPN < end; e0 += CH * 64) {  // a group with a coupling stays whole
        int32_t j[CH];
        T w[CH], x[CH][LPN][EPL];
        // past the row's end: the row itself with value 0
#pragma unroll
        for (int v = 0; v < CH; ++v) {
            const int64_t e = e0 + v * 64 + lane;
            const bool ok = e < end;
            const int64_t i = ok ? e : beg;
            const int32_t ji = col[i];
            const T wi = val[i];
            j[v] = ok ? ji : (int32_t)row;
            w[v] = ok ? wi : T(0);
        }
        if (perm) {
#pragma unroll
            for (int v = 0; v < CH; ++v) j[v] = perm[j[v]];
        }
#pragma unroll
        for (int v = 0; v < CH; ++v)
            static_for<LPN>([&](auto u) { load(group_bcast<LPN, u>(j[v]), x[v][u]); });
#pragma unroll
        for (int v = 0; v < CH; ++v)
            static_for<LPN>([&](auto u) {
                const T wu = group_bcast<LPN, u>(w[v]);
#pragma unroll
                for (int c = 0; c < EPL; ++c) acc[c] += wu * x[v][u][c];
            });
    }
#pragma unroll
    for (int off = LPN; off < 64; off <<= 1) {
#pragma unroll
        for (int c = 0; c < EPL; ++c) acc[c] += __shfl_xor(acc[c], off, 64);
    }
    if (g != 0) return;
    if (diag) {
#pragma unroll
        for (int c = 0; c < EPL; ++c) acc[c] += d * own[c];
    }
    if constexpr (VEC) {
        store_vec<T, EPL>(S + orow * K + c0, acc);
    } else {
#pragma unroll
        for (int c = 0; c < EPL; ++c)
            if (c0 + c < k) S[orow * k + c0 + c] = acc[c];
    }
}

template <typename T, int K>
void launch_small(const Ctx &c, const T *val, const T *diag, const T *X, int k, T *S, bool sorted, hipStream_t s) {
    const bool vec = k == K && (uintptr_t)X % 16 == 0 && (uintptr_t)S % 16 == 0;
    const dim3 grid((unsigned)((c.ndet + SIGMA_BLOCK / 64 - 1) / (SIGMA_BLOCK / 64))), block(SIGMA_BLOCK);
    const int32_t *perm = sorted ? (const int32_t *)nullptr : (const int32_t *)c.perm.p;
    if (vec)
        hipLaunchKernelGGL((k_sigma_small<T, K, true>), grid, block, 0, s, c.ndet, c.rowptr.p, c.col.p, val, diag,
                           perm, X, k, S);
    else
        hipLaunchKernelGGL((k_sigma_small<T, K, false>), grid, block, 0, s, c.ndet, c.rowptr.p, c.col.p, val, diag,
                           perm, X, k, S);
    HQ_LAUNCH_CHECK();
}

template <typename T>
void dispatch_small(const Ctx &c, const T *val, const T *diag, const T *X, int k, T *S, bool sorted, hipStream_t s) {
    if (k <= 1) launch_small<T, 1>(c, val, diag, X, k, S, sorted, s);
    else if (k <= 2) launch_small<T, 2>(c, val, diag, X, k, S, sorted, s);
    else if (k <= 4) launch_small<T, 4>(c, val, diag, X, k, S, sorted, s);
    else if (k <= 8) launch_small<T, 8>(c, val, diag, X, k, S, sorted, s);
    else launch_small<T, 16>(c, val, diag, X, k, S, sorted, s);
}

int env_int(const char *name, int dflt) {
    const char *v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : dflt;
}

int kindex(int k) { return k <= 1 ? 0 : k <= 2 ? 1 : k <= 4 ? 2 : k <= 8 ? 3 : 4; }

template <typename T, int K>
constexpr int lanes_per_coupling() {
    return (K >= Vec16<T>::n) ? K / Vec16<T>::n : 1;
}

// Rows a team takes from its XCD's counter at a time; 0: fixed strides.  The
// atomics on one counter come through at about 24 ns each (1e6 rows, runs of
// one row: 3.0 ms, all of it the counters), so they pay only where X is large
// against the L2s (32 MB) and a row's work against its atomic: strides / counters
// in us, k = 1 and 8, 20,000 rows with 356 couplings 33 / 170 and 54 / 140, 5e5
// with 85 333 / 350 and 457 / 463, 2e5 with 615 565 / 601 and 962 / 938, 1e6 with
// 156 1087 / 1086 and 1648 / 1506, 4e6 with 171 4425 / 4250 and 8321 / 6332, 1e7
// with 13.5 1327 / 1664 and 2200 / 2554, 6e6 with 23.6 1264 / 1376 and 2110 / 2079,
// 2e7 with 27 5718 / 5569 and 9390 / 8859.  By the bytes of X: 1e6 with 157, FP32, k = 1
// (4 MB) 823 / 851, FP64, k = 1 (8 MB) 1093 / 1087; 1.5e6 with 236, k = 1 (12 MB) 2393 /
// 2346; long rows keep their XCD's X together by themselves for longer, 3e5 with 856,
// k = 4 (9.6 MB) 1553 / 1619, 7e5 with 870, k = 2 and 4 (11.2, 22.4 MB) 3203 / 3259 and
// 4077 / 4083.
constexpr int64_t SIGMA_STATIC_NNZ = 130000000;
constexpr double SIGMA_COUNTER_ROW = 25.0;  // mean couplings
constexpr double SIGMA_LONG_ROW = 256.0;    // mean couplings from which two rows make a run
constexpr int64_t SIGMA_COUNTER_X = 6 << 20, SIGMA_COUNTER_X_LONG = 16 << 20;  // bytes of X

int row_run(const Ctx &c, const SigmaCfg &cfg, int64_t xbytes) {
    if (cfg.run >= 0) return cfg.run;
    const double avg = (double)c.nnz / (double)c.ndet;
    const bool long_rows = avg >= SIGMA_LONG_ROW;
    if (c.nnz <= SIGMA_STATIC_NNZ || avg < SIGMA_COUNTER_ROW ||
        xbytes < (long_rows ? SIGMA_COUNTER_X_LONG : SIGMA_COUNTER_X))
        return 0;
    return long_rows ? 2 : 4;
}

template <typename T, int K, int TEAM, int UNR, bool MASK>
void launch_sigma_u(const Ctx &c, const SigmaCfg &cfg, const SigmaMask &mk, const T *val, const T *diag,
                    const T *X, int ldx, T *S, int lds, const SigmaOut &out, hipStream_t s, unsigned long long *ctr) {
    static int cus = 0;
    if (!cus) {
        cus = 256;
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c.device);
    }
    // workgroups resident per CU (4 waves each), capped by the number of row teams
    int64_t nblk = (int64_t)cus * std::max(1, cfg.occ);
    const int64_t max_blk = (c.ndet + SIGMA_BLOCK / TEAM - 1) / (SIGMA_BLOCK / TEAM);
    nblk = std::min(nblk, std::max<int64_t>(max_blk, 1));
    nblk = (nblk + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    XcdRows ranges;
    for (int x = 0; x <= NUM_XCD; ++x) ranges.b[x] = c.xcd_rows[x];
    const int xmap = env_int("HINQS_SIGMA_XCDMAP", 1);
    const int run = MASK ? 0 : row_run(c, cfg, c.ndet * K * (int64_t)sizeof(T));
    hipLaunchKernelGGL((k_sigma<T, K, TEAM, UNR, MASK>), dim3((unsigned)nblk), dim3(SIGMA_BLOCK), 0, s, ranges, mk,
                       xmap, c.rowptr.p, c.col.p, val, diag, X, ldx, S, lds, out,
                       run > 0 ? (ctr ? ctr : c.sigma_ctr.p) : (unsigned long long *)nullptr, std::max(1, run));
    HQ_LAUNCH_CHECK();
}

template <typename T, int K, int TEAM, bool MASK>
void launch_sigma(const Ctx &c, const SigmaCfg &cfg, const SigmaMask &mk, const T *val, const T *diag,
                  const T *X, int ldx, T *S, int lds, const SigmaOut &out, hipStream_t s, unsigned long long *ctr) {
    // cfg.unr pairs of gathers in flight per lane; a step has at least the couplings
    // that the lanes of one fetch
    constexpr int U4 = lanes_per_coupling<T, K>() < 8 ? 4 : 8;
    if (cfg.unr <= 2) launch_sigma_u<T, K, TEAM, U4, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr);
    else launch_sigma_u<T, K, TEAM, 8, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr);
}

template <typename T, int K, bool MASK>
void dispatch_team(const Ctx &c, const SigmaCfg &cfg, const SigmaMask &mk, const T *val, const T *diag,
                   const T *X, int ldx, T *S, int lds, const SigmaOut &out, hipStream_t s, unsigned long long *ctr) {
    constexpr int LPN = lanes_per_coupling<T, K>();
    const int team = std::max(cfg.team, LPN);
#define HQ_TEAM(n) launch_sigma<T, K, n, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr)
    switch (team) {
        case 1: if constexpr (LPN <= 1) { HQ_TEAM(1); break; } [[fallthrough]];
        case 2: if constexpr (LPN <= 2) { HQ_TEAM(2); break; } [[fallthrough]];
        case 4: if constexpr (LPN <= 4) { HQ_TEAM(4); break; } [[fallthrough]];
        case 8: if constexpr (LPN <= 8) { HQ_TEAM(8); break; } [[fallthrough]];
        case 16: HQ_TEAM(16); break;
        case 32: HQ_TEAM(32); break;
        default: HQ_TEAM(64); break;
    }
#undef HQ_TEAM
}

template <typename T, bool MASK = false>
void dispatch_k(const Ctx &c, int k, const SigmaCfg &cfg, const T *val, const T *diag, const T *X, int ldx,
                T *S, int lds, hipStream_t s, const SigmaMask &mk = SigmaMask{},
                unsigned long long *ctr = nullptr, const SigmaOut &out = SigmaOut{}) {
    switch (k) {
        case 1: dispatch_team<T, 1, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr); break;
        case 2: dispatch_team<T, 2, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr); break;
        case 4: dispatch_team<T, 4, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr); break;
        case 8: dispatch_team<T, 8, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr); break;
        case 16: dispatch_team<T, 16, MASK>(c, cfg, mk, val, diag, X, ldx, S, lds, out, s, ctr); break;
        default: throw Error(HINQS_E_UNSUPPORTED, "sigma block size must be 1, 2, 4, 8 or 16");
    }
}

}  // namespace

// Default shape before tuning, from the mean row and the lanes that share a
// coupling (times in us, FP64).  Lanes: a step takes one or two couplings per
// lane, and a row should be a few steps (k = 1: rows of 19 couplings 8 lanes 21.3,
// of 73 16 lanes 16.1, of 356 32 lanes 31.3 and 64 lanes 32.4; k = 8: 36 couplings 16
// lanes 94, 230 and 356 32 lanes 113 and 54, 64 lanes 117 and 53; k = 16, eight
// lanes per coupling: 19 couplings 16 lanes 43 and 32 lanes 55, 356 64 lanes 67 and
// 32 lanes 75), and the rows' teams fill the chip (5,000 rows of 13: 16 lanes
// 5.9, 8 lanes 7.2).  The same holds for large sets (1e7 rows of 13.5, 8 / 16 / 32 /
// 64 lanes: k = 1 1327 / 1579 / 2755 / 5527, k = 8 2361 / 2200 / 2460 / 3702; 2e7 of
// 27, k = 8, 16 / 32 / 64 lanes 8859 / 9148 / 10568), but for their rows of 64 and
// more (16 / 32 / 64 lanes, k = 1: 2e6 of 86 1372 / 1169 / 1460; k = 8: 2e6 of 86 1920 /
// 1738 / 1682, 1e6 of 156 1665 / 1499 / 1506, 4e6 of 171 7780 / 6471 / 6332).
// Gathers in flight: eight per lane where the row has them
// (k = 8, 356 couplings 52 against 59 with four).  Workgroups per CU: more than are
// resident even out rows of different length (60,000 rows, k = 8, 8 / 4: 114 / 117)
// until the rows per team are many (4.9e7 couplings: 4 386, 8 400).
constexpr int64_t SIGMA_EVEN_NNZ = 32000000;
constexpr double SIGMA_WIDE_ROW = 240.0;  // mean couplings times lanes per coupling
SigmaCfg default_cfg(const Ctx &c, int k, int precision) {
    const int vw = precision == HINQS_FP64 ? 2 : 4;
    const int lpn = k >= vw ? k / vw : 1;
    const double avg = c.ndet > 0 ? (double)c.nnz / (double)c.ndet : 0.0;
    const double want = avg / 8.0 * lpn;
    SigmaCfg g;
    g.unr = avg * lpn >= SIGMA_WIDE_ROW ? 4 : 2;
    g.occ = c.nnz <= SIGMA_EVEN_NNZ ? 8 : 4;
    if (lpn >= 8) g.team = avg < 32 ? 16 : avg < 100 ? 32 : 64;
    else g.team = want <= 3 ? 8 : want <= 16 ? 16 : 32;
    if (c.nnz > SIGMA_STATIC_NNZ && avg >= 64.0) g.team = lpn >= 4 ? 64 : 32;
    while (g.team < 64 && c.ndet * g.team < (int64_t)256 * 1024) g.team *= 2;
    if (c.ndet <= SIGMA_SMALL_ROWS) g.pipe = 2;
    return g;
}

SigmaCfg sigma_config(const Ctx &c, int k, int precision) {
    SigmaCfg g = c.sigma_cfg[precision == HINQS_FP64 ? 0 : 1][kindex(k)];
    if (g.team == 0) g = default_cfg(c, k, precision);
    // explicit overrides for experiments
    if (std::getenv("HINQS_SIGMA_TEAM") && g.pipe == 2) g.pipe = 0;
    g.team = env_int("HINQS_SIGMA_TEAM", g.team);
    g.unr = env_int("HINQS_SIGMA_UNR", g.unr);
    g.occ = env_int("HINQS_SIGMA_OCC", g.occ);
    g.pipe = env_int("HINQS_SIGMA_PIPE", g.pipe);
    g.run = env_int("HINQS_SIGMA_RUN", g.run);
    return g;
}

namespace {

void launch_shape(const Ctx &c, int k, int precision, const SigmaCfg &cfg, const void *X, int ldx, void *S, int lds,
                  hipStream_t s, unsigned long long *ctr, const SigmaOut &out = SigmaOut{}) {
    const bool small = cfg.pipe == 2 && ldx == k && lds == k && !out.row && !out.cols;
    if (precision == HINQS_FP64) {
        if (small) dispatch_small<double>(c, c.val.p, c.diag.p, (const double *)X, k, (double *)S, true, s);
        else dispatch_k<double>(c, k, cfg, c.val.p, c.diag.p, (const double *)X, ldx, (double *)S, lds, s,
                                SigmaMask{}, ctr, out);
    } else if (precision == HINQS_FP32) {
        if (small) dispatch_small<float>(c, c.val32.p, c.diag32.p, (const float *)X, k, (float *)S, true, s);
        else dispatch_k<float>(c, k, cfg, c.val32.p, c.diag32.p, (const float *)X, ldx, (float *)S, lds, s,
                               SigmaMask{}, ctr, out);
    } else {
        throw Error(HINQS_E_INVALID_ARG, "precision must be HINQS_FP64 or HINQS_FP32");
    }
}

}  // namespace

// X in sorted order; k in {1,2,4,8,16}; leading dimensions keep 16-byte
// alignment of every row (ldx, lds multiples of 16 / sizeof(T) when k >= that).
// S in sorted order as well, or where out says.
void sigma_sorted(Ctx &c, int k, const void *X, int ldx, void *S, int lds, int precision,
                  hipStream_t s, unsigned long long *ctr, const SigmaOut &out) {
    if (!c.have_elements) throw Error(HINQS_E_NOT_READY, "matrix elements are not built");
    launch_shape(c, k, precision, sigma_config(c, k, precision), X, ldx, S, lds, s, ctr, out);
}

bool sigma_small(const Ctx &c, int k, const void *X, void *S, int precision, bool sorted, hipStream_t s) {
    const int K = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : 16;
    // A tuned shape was timed on products in sorted order, aligned and of K columns.
    // Any other product of a small set would be staged first, which this launch
    // saves (caller order, one launch / staged: 400 rows, k = 1 4.6 / 8.2 us, 8,192
    // rows, k = 8 11.1 / 16.3), so no tuned shape takes it away.
    const bool direct = sorted && K == k && (uintptr_t)X % 16 == 0 && (uintptr_t)S % 16 == 0;
    const bool asked = std::getenv("HINQS_SIGMA_TEAM") || std::getenv("HINQS_SIGMA_PIPE");
    if ((direct || asked || c.ndet > SIGMA_SMALL_ROWS) && sigma_config(c, K, precision).pipe != 2) return false;
    // the launch reads X while others of its waves write S: arrays that share
    // memory take the path that copies X first
    const size_t bytes = (size_t)c.ndet * k * (precision == HINQS_FP64 ? 8 : 4);
    const uintptr_t x = (uintptr_t)X, y = (uintptr_t)S;
    if (x < y + bytes && y < x + bytes) return false;
    if (precision == HINQS_FP64)
        dispatch_small<double>(c, c.val.p, c.diag.p, (const double *)X, k, (double *)S, sorted, s);
    else
        dispatch_small<float>(c, c.val32.p, c.diag32.p, (const float *)X, k, (float *)S, sorted, s);
    return true;
}

void sigma_offdiag_fp32(const Ctx &c, int k, const float *X, float *S, hipStream_t s) {
    if (!c.have_elements) throw Error(HINQS_E_NOT_READY, "matrix elements are not built");
    const SigmaCfg cfg = sigma_config(c, k, HINQS_FP32);
    if (cfg.pipe == 2) return dispatch_small<float>(c, c.val32.p, (const float *)nullptr, X, k, S, true, s);
    dispatch_k<float>(c, k, cfg, c.val32.p, (const float *)nullptr, X, k, S, k, s);
}

void sigma_masked_fp64(const Ctx &c, int k, const double *X, double *S, const SigmaMask &mk, hipStream_t s) {
    if (!c.have_elements) throw Error(HINQS_E_NOT_READY, "matrix elements are not built");
    const SigmaCfg cfg = sigma_config(c, k, HINQS_FP64);
    dispatch_k<double, true>(c, k, cfg, c.val.p, c.diag.p, X, k, S, k, s, mk);
}

void sigma_launch(const Ctx &c, int k, int precision, const SigmaCfg &cfg, const void *X, int ldx, void *S,
                  int lds, hipStream_t s) {
    if (!c.have_elements) throw Error(HINQS_E_NOT_READY, "matrix elements are not built");
    launch_shape(c, k, precision, cfg, X, ldx, S, lds, s, nullptr);
}

}  // namespace hinqs
