// Scans of string groups and buffered stores of the couplings found, shared by
// the full enumeration and the incremental update.
#pragma once

#include "common.hpp"

namespace hinqs {
namespace {

// Couplings a wave has found and not written yet: up to EMIT_CAP per lane (one
// row per lane) in LDS.  Written straight from the lanes, every 4-byte store of
// a wave went to 64 different rows (1.56e8 couplings: 5.0 ms, against 2.7 ms
// for the same tests without the stores); a flush writes up to sixteen
// consecutive couplings of a row with sixteen neighbouring lanes.
constexpr int EMIT_CAP = 16;
constexpr int EMIT_STRIDE = EMIT_CAP + 1;  // keeps the lanes' slots in different banks
struct EmitBuf {
    int32_t col[64 * EMIT_STRIDE];
    uint32_t desc[64 * EMIT_STRIDE];
};

// out: the lane's next place in the matrix; n: couplings it holds; map: column of
// a buffered one, nullptr: itself.  Called by the whole wave.
__device__ inline void emit_flush(EmitBuf &b, int64_t &out, int &n, int lane, int32_t *col, uint32_t *desc,
                                  const int32_t *map = nullptr) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int r0 = 0; r0 < 64; r0 += 64 / EMIT_CAP) {
        const int r = r0 + lane / EMIT_CAP, k = lane % EMIT_CAP;
        const int nr = __shfl(n, r, 64);
        const int64_t at = __shfl(out, r, 64) + k;
        if (k < nr) {
            const int32_t j = b.col[r * EMIT_STRIDE + k];
            col[at] = map ? map[j] : j;
            desc[at] = b.desc[r * EMIT_STRIDE + k];
        }
    }
    __builtin_amdgcn_wave_barrier();
    out += n;
    n = 0;
}

// Tests every string in str[lo, hi) (per lane) against own, W (16 or 32) at a
// time: hits(j0, mask) with bit u of the mask set where accept(bits that differ)
// of str[j0 + u] holds, at most EMIT_CAP of them.  Lanes that share the range
// (rows of one group) read it through the scalar cache.  Called by the whole
// wave; str is readable W strings past its end.
template <int W, typename Accept, typename Hits>
__device__ inline void scan_strings(const uint32_t *__restrict__ str, int32_t lo, int32_t hi, uint32_t own,
                                    Accept &&accept, Hits &&hits) {
    auto test = [&](int32_t j0, int32_t end) {
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < W; ++u) m |= accept(popc32(own ^ str[j0 + u])) ? 1u << u : 0u;
        return end - j0 < W ? m & ((1u << (end - j0)) - 1u) : m;
    };
    auto report = [&](int32_t j0, uint32_t m) {
        if (W > EMIT_CAP && __any(popc32(m) > EMIT_CAP)) {
            hits(j0, m & 0xffffu);
            hits(j0 + 16, m >> 16);
        } else {
            hits(j0, m);
        }
    };
    static_assert((W == 16 || W == 32) && EMIT_CAP >= 16, "halves fit");
    const int32_t ulo = __builtin_amdgcn_readfirstlane(lo), uhi = __builtin_amdgcn_readfirstlane(hi);
    if (__all(lo == ulo && hi == uhi)) {
        for (int32_t j0 = ulo; j0 < uhi; j0 += W) report(j0, test(j0, uhi));
    } else {
        for (int32_t j0 = lo; __any(j0 < hi); j0 += W) report(j0, j0 < hi ? test(j0, hi) : 0u);
    }
}

}  // namespace
}  // namespace hinqs
