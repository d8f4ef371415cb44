// Compares the kernels' square root, reciprocal and quotient with correctly rounded ones
// (formed in double precision and rounded once more, which is exact for these operations),
// and the reciprocal root's estimate with rsqrtf.  Built by build(), run by
// tests/test_gpu_rounding.py; prints the number of floats and of differences of each.
#include "rounding.h"

#include <cstdint>
#include <cstdio>

using namespace dsdp;

static __device__ __forceinline__ uint32_t mix(uint64_t k)
{
    k = (k ^ (k >> 30)) * 0xBF58476D1CE4E5B9ull;   // splitmix64's finaliser
    k = (k ^ (k >> 27)) * 0x94D049BB133111EBull;
    return (uint32_t)((k ^ (k >> 31)) >> 16);
}

// roots and reciprocals of the floats with bits [lo, hi)
__global__ void every_float(uint32_t lo, uint32_t hi, uint32_t normal_lo, unsigned long long *bad)
{
    unsigned long long b[3] = {0, 0, 0};
    for (uint64_t i = (uint64_t)lo + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < hi;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const float x = __uint_as_float((uint32_t)i);
        b[0] += __float_as_uint(sqrt_normal(x)) != __float_as_uint((float)sqrt((double)x));
        b[1] += __float_as_uint(rcp_normal(x)) != __float_as_uint((float)(1.0 / (double)x));
        if (i >= normal_lo) b[2] += __float_as_uint(__builtin_amdgcn_rsqf(x)) != __float_as_uint(rsqrtf(x));
    }
    for (int k = 0; k < 3; k++)
        if (b[k]) atomicAdd(&bad[k], b[k]);
}

// quotients a / b of n pairs with b in the normal range and a / b too
__global__ void quotients(uint64_t n, uint64_t seed, unsigned long long *bad)
{
    const uint32_t lo = __float_as_uint(kNormalLo), span = __float_as_uint(kNormalHi) - lo;
    unsigned long long b = 0, used = 0;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const float den = __uint_as_float(lo + mix(seed + 2 * i) % span);
        const float want = __uint_as_float(lo + mix(seed + 2 * i + 1) % span);
        const float num = want * den;   // any float near a quotient in range
        if (!in_normal(num)) continue;
        used++;
        b += __float_as_uint(div_normal(num, den)) != __float_as_uint((float)((double)num / (double)den));
    }
    if (b) atomicAdd(&bad[3], b);
    atomicAdd(&bad[4], used);
}

#define TRY(x)                                                             \
    do {                                                                   \
        const hipError_t e = (x);                                          \
        if (e != hipSuccess) {                                             \
            std::fprintf(stderr, "%s: %s\n", #x, hipGetErrorString(e));    \
            return 2;                                                      \
        }                                                                  \
    } while (0)

int main()
{
    unsigned long long *bad = nullptr, h[5] = {0, 0, 0, 0, 0};
    TRY(hipMalloc(&bad, sizeof h));
    TRY(hipMemcpy(bad, h, sizeof h, hipMemcpyHostToDevice));
    // bits of 2^-96, 2^-80 and 64
    const uint32_t lo = (127u - 96u) << 23, normal = (127u - 80u) << 23, hi = (127u + 6u) << 23;
    const uint64_t pairs = 1ull << 30;
    every_float<<<4096, 256>>>(lo, hi, normal, bad);
    TRY(hipGetLastError());
    quotients<<<4096, 256>>>(pairs, 12345, bad);
    TRY(hipGetLastError());
    TRY(hipMemcpy(h, bad, sizeof h, hipMemcpyDeviceToHost));
    TRY(hipFree(bad));
    std::printf("floats %u roots %llu reciprocals %llu inverse_roots %llu\n", hi - lo, h[0], h[1], h[2]);
    std::printf("pairs %llu quotients %llu\n", h[4], h[3]);
    return h[0] || h[1] || h[2] || h[3] ? 1 : 0;
}
