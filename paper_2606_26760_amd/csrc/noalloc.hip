// Sigma product S = H_B X without any device allocation (the repeated product
// of the Davidson iteration, Sec. 2.2, Step 3), for callers that cannot
// allocate: the kernel's row counters and the sorted-order copy of X live in
// one static device array per GPU instead of context buffers.  The staging
// kernel (caller order and k padded to K in one pass; the product writes S's
// rows and columns itself) serves hinqs_sigma too, with the context's buffer.
//
// Layout of the array: [0, 4096) row counters (SIGMA_CTR_WORDS words, cleared
// by a fill kernel on every call; no memset, so the call can be captured in a
// graph); [4096, 4096 + B) staged X, where B = ndet * K * element size rounded
// up to 256 bytes.  Calls with 4096 + 2B beyond the array are refused.
#include <mutex>

#include "common.hpp"

namespace hinqs {

constexpr size_t NOALLOC_BYTES = HINQS_NOALLOC_SCRATCH_BYTES;
constexpr size_t NOALLOC_CTR_BYTES = 4096;
static_assert(SIGMA_CTR_WORDS * sizeof(unsigned long long) <= NOALLOC_CTR_BYTES, "counter region");

// In host code `scratch` only names the host-side shadow of the array; its
// device address comes from hipGetSymbolAddress (noalloc_setup) and only that
// address is ever passed to kernels.
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_mu;
unsigned char *g_ptr[MAX_DEVICES] = {};

unsigned char *device_scratch(int device) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (device < 0 || device >= MAX_DEVICES || !g_ptr[device])
        throw Error(HINQS_E_NOT_READY, "the no-allocation scratch of this device is not set up");
    return g_ptr[device];
}

__global__ void k_clear_words(unsigned long long *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// xs (sorted order, K wide) from X (k wide; caller order through perm, or
// sorted when perm is null); columns k..K-1 are zero.  Bound by memory; VEC: X is
// K wide and aligned, 16 bytes per thread (1e6 rows of 8 doubles: 30 us, element
// by element with the row divided out 40 us).
template <typename T, int K, bool VEC>
__global__ __launch_bounds__(256) void k_stage_in(const T *__restrict__ X, int k, const int32_t *__restrict__ perm,
                                                  int64_t D, T *__restrict__ xs) {
    constexpr int N = VEC ? 16 / sizeof(T) : 1, PER = K / N;  // elements per thread, threads per row
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t / PER;
    const int col = (int)(t % PER) * N;
    if (i >= D) return;
    const int64_t r = perm ? (int64_t)perm[i] : i;
    if constexpr (VEC) {
        typedef float vec4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<vec4 *>(xs + i * K + col) = *reinterpret_cast<const vec4 *>(X + r * K + col);
    } else {
        xs[i * K + col] = col < k ? X[r * k + col] : T(0);
    }
}

template <typename T, int K>
void staged(Ctx &c, int k, const T *X, T *S, bool sorted, T *xs, unsigned long long *ctr) {
    hipStream_t s = c.stream;
    const int64_t D = c.ndet;
    const int32_t *perm = sorted ? nullptr : c.perm.p;
    constexpr int N = 16 / sizeof(T);
    if constexpr (K >= N) {
        if (k == K && (uintptr_t)X % 16 == 0)
            hipLaunchKernelGGL((k_stage_in<T, K, true>), dim3(grid_for(D * (K / N), 256)), dim3(256), 0, s, X, k, perm,
                               D, xs);
        else
            hipLaunchKernelGGL((k_stage_in<T, K, false>), dim3(grid_for(D * K, 256)), dim3(256), 0, s, X, k, perm, D,
                               xs);
    } else {
        hipLaunchKernelGGL((k_stage_in<T, K, false>), dim3(grid_for(D * K, 256)), dim3(256), 0, s, X, k, perm, D, xs);
    }
    HQ_LAUNCH_CHECK();
    // whole vectors where S's rows keep their alignment
    const bool vec = k == K && (K < N || (uintptr_t)S % 16 == 0);
    sigma_sorted(c, K, xs, K, S, k, sizeof(T) == 8 ? HINQS_FP64 : HINQS_FP32, s, ctr, SigmaOut{perm, vec ? 0 : k});
}

template <typename T>
void staged_k(Ctx &c, int k, const T *X, T *S, bool sorted, T *xs, unsigned long long *ctr) {
    if (k <= 1) staged<T, 1>(c, k, X, S, sorted, xs, ctr);
    else if (k <= 2) staged<T, 2>(c, k, X, S, sorted, xs, ctr);
    else if (k <= 4) staged<T, 4>(c, k, X, S, sorted, xs, ctr);
    else if (k <= 8) staged<T, 8>(c, k, X, S, sorted, xs, ctr);
    else staged<T, 16>(c, k, X, S, sorted, xs, ctr);
}

}  // namespace

void sigma_staged(Ctx &c, int k, const void *X, void *S, int precision, bool sorted, void *xs,
                  unsigned long long *ctr) {
    if (precision == HINQS_FP64) staged_k<double>(c, k, (const double *)X, (double *)S, sorted, (double *)xs, ctr);
    else staged_k<float>(c, k, (const float *)X, (float *)S, sorted, (float *)xs, ctr);
}

void noalloc_setup(int device) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (device < 0 || device >= MAX_DEVICES) throw Error(HINQS_E_UNSUPPORTED, "device index above 63");
    if (g_ptr[device]) return;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
        throw Error(HINQS_E_HIP, std::string("hipGetSymbolAddress of the no-allocation scratch failed: ") +
                                     hipGetErrorString(e));
    g_ptr[device] = (unsigned char *)p;
}

void sigma_noalloc(Ctx &c, int k, const void *X, void *S, int precision, bool sorted) {
    struct Forbid {  // any device allocation below is an internal error
        bool prev = g_no_alloc;
        Forbid() { g_no_alloc = true; }
        ~Forbid() { g_no_alloc = prev; }
    } forbid;
    unsigned char *base = device_scratch(c.device);
    const size_t esz = precision == HINQS_FP64 ? 8 : 4;
    const int K = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : 16;
    const bool aligned = ((uintptr_t)X % 16 == 0) && ((uintptr_t)S % 16 == 0);
    const bool direct = sorted && K == k && aligned;
    const size_t blk = ((size_t)c.ndet * K * esz + 255) / 256 * 256;
    // the limit that the entry point has always had, two blocks; one is used
    const size_t need = NOALLOC_CTR_BYTES + (direct ? 0 : 2 * blk);
    if (need > NOALLOC_BYTES)
        throw Error(HINQS_E_UNSUPPORTED, "the no-allocation sigma needs " + std::to_string(need) +
                                             " bytes of scratch for ndet = " + std::to_string(c.ndet) +
                                             " and k = " + std::to_string(k) + "; its limit is " +
                                             std::to_string(NOALLOC_BYTES) +
                                             " (sorted-order, 16-byte aligned X and S with k in {1,2,4,8,16} "
                                             "need no staging)");
    hipStream_t s = c.stream;
    if (sigma_small(c, k, X, S, precision, sorted, s)) return;
    hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(SIGMA_CTR_WORDS), 0, s, (unsigned long long *)base,
                       SIGMA_CTR_WORDS);
    HQ_LAUNCH_CHECK();
    if (direct)
        sigma_sorted(c, K, X, K, S, K, precision, s, (unsigned long long *)base);
    else
        sigma_staged(c, k, X, S, precision, sorted, base + NOALLOC_CTR_BYTES, (unsigned long long *)base);
}

}  // namespace hinqs
