// Binding-site points from a site predictor's score volume on gfx950.
//
// Paper: Section 2, site-prediction paragraph (the score voxels are extracted
// and clustered, the top 200 points describe the site for the docking stage,
// the maximum-score position is the sampling centre).
//
// One workgroup of 1024 threads.  The points are the top_n largest 64-bit keys
// (orderable score bits, then the inverted voxel index, so ties go to the lower
// index).  Two passes over the volume find them: the first keeps the maximum of
// each of 4096 strips of voxels (four per thread, one for each component of its
// 16-byte loads); the top_n-th largest maximum, cut to its upper 16 bits, is a
// lower bound of the top_n-th largest score, and the second pass collects the keys
// at or above it into LDS (about 1.2 to 2 top_n of them), where one bitonic sort
// orders them.  A volume with more keys there than LDS holds (a plateau) takes a
// radix selection over the volume instead (eight 8-bit digits).  Single-linkage
// clusters are the connected components of "integer voxel offset within the link
// distance": a union-find in LDS in which a root is only ever hooked under a
// smaller one, so every label is the rank of its component's best point
// whatever the thread schedule.
//
// Bound by latency: one compute unit reads 187 KB (36^3) twice in about 3 us, and
// the rest is a chain of barriers.
#include "dsdp_internal.h"

namespace dsdp {
namespace {

constexpr int kSiteThreads = 1024;

constexpr int kSiteCand = 4096;   // candidate keys held in LDS (32 KB)
constexpr int kTopBits = 16;

__device__ __forceinline__ uint32_t score_order(float v)
{
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ uint64_t site_key(float v, int i)
{
    return ((uint64_t)score_order(v) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i);
}

// Voxels 4 g to 4 g + 3 (those below n; VEC: the volume is 16-byte aligned).
template <bool VEC>
__device__ __forceinline__ float4 load4(const float *scores, int n, int g)
{
    if (VEC && 4 * g + 3 < n) return reinterpret_cast<const float4 *>(scores)[g];
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (4 * g + 0 < n) v.x = scores[4 * g + 0];
    if (4 * g + 1 < n) v.y = scores[4 * g + 1];
    if (4 * g + 2 < n) v.z = scores[4 * g + 2];
    if (4 * g + 3 < n) v.w = scores[4 * g + 3];
    return v;
}

// Root of a in the union-find forest (parents only ever decrease).
__device__ __forceinline__ int find_root(volatile int *parent, int a)
{
    int p = parent[a];
    while (p != a) {
        a = p;
        p = parent[a];
    }
    return a;
}

template <bool VEC>
__global__ __launch_bounds__(kSiteThreads) void site_extract_kernel(const float *scores, int nx, int ny, int nz,
                                                                     int k, int lim, int *out_index,
                                                                     int *out_label)
{
    __shared__ uint64_t cand[kSiteCand];
    __shared__ unsigned int hist[256];
    __shared__ int lab[kMaxSitePoints];
    __shared__ int ci[kMaxSitePoints], cj[kMaxSitePoints], ck[kMaxSitePoints];
    __shared__ uint64_t prefix_s;
    __shared__ int remain_s, count_s, votes_s[kTopBits];
    const int t = (int)threadIdx.x, lane = t & 63;
    const int n = nx * ny * nz, groups = (n + 3) / 4;

    // (1) strip maxima, and their k-th largest cut to its upper bits (every strip
    //     holds a voxel, or the volume has at most 4096 and each its own strip, so
    //     at least k maxima are voxels' scores)
    if (t < kTopBits) votes_s[t] = 0;
    if (t == 0) count_s = 0;
    uint32_t m[4] = {0u, 0u, 0u, 0u};
#pragma unroll 4
    for (int g = t; g < groups; g += kSiteThreads) {
        const float4 v = load4<VEC>(scores, n, g);
        m[0] = max(m[0], score_order(v.x));   // voxel 4 g is below n
        m[1] = max(m[1], 4 * g + 1 < n ? score_order(v.y) : 0u);
        m[2] = max(m[2], 4 * g + 2 < n ? score_order(v.z) : 0u);
        m[3] = max(m[3], 4 * g + 3 < n ? score_order(v.w) : 0u);
    }
    __syncthreads();
    uint32_t cut = 0u;
    for (int b = 0; b < kTopBits; b++) {
        const uint32_t tryout = cut | (0x80000000u >> b);
        int votes = 0;
#pragma unroll
        for (int c = 0; c < 4; c++) votes += __popcll(__ballot(m[c] >= tryout));
        if (lane == 0 && votes) atomicAdd(&votes_s[b], votes);
        __syncthreads();
        if (votes_s[b] >= k) cut = tryout;
    }

    // (2) collect the keys at or above the cut
#pragma unroll 4
    for (int g = t; g < groups; g += kSiteThreads) {
        const float4 v = load4<VEC>(scores, n, g);
        const float q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int c = 0; c < 4; c++) {
            if (4 * g + c < n && score_order(q[c]) >= cut) {
                const int at = atomicAdd(&count_s, 1);
                if (at < kSiteCand) cand[at] = site_key(q[c], 4 * g + c);
            }
        }
    }
    __syncthreads();
    int count = count_s;

    if (count > kSiteCand) {
        // radix selection of the k-th largest key, most significant digit first
        __syncthreads();
        if (t == 0) {
            prefix_s = 0;
            remain_s = k;
            count_s = 0;
        }
        __syncthreads();
        for (int shift = 56; shift >= 0; shift -= 8) {
            if (t < 256) hist[t] = 0u;
            __syncthreads();
            const uint64_t prefix = prefix_s;
            const int remain = remain_s;
            const uint64_t hi_mask = shift == 56 ? 0ull : (~0ull << (shift + 8));
            for (int i = t; i < n; i += kSiteThreads) {
                const uint64_t key = site_key(scores[i], i);
                if ((key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (t < 64) {
                // lane l holds digits 255 - 4 l and the three below: the first digit
                // from the top at which the running count reaches `remain`
                int h[4], sum = 0;
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    h[c] = (int)hist[255 - 4 * t - c];
                    sum += h[c];
                }
                int incl = sum;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int v = __shfl_up(incl, o, 64);
                    if (lane >= o) incl += v;
                }
                const int above = incl - sum;
                if (above < remain && incl >= remain) {
                    int rem = remain - above, c = 0;
                    for (; c < 3 && h[c] < rem; c++) rem -= h[c];
                    prefix_s = prefix | ((uint64_t)(255 - 4 * t - c) << shift);
                    remain_s = rem;
                }
            }
            __syncthreads();
        }
        const uint64_t kth = prefix_s;   // every key is distinct: exactly k keys are >= kth
        for (int i = t; i < n; i += kSiteThreads) {
            const uint64_t key = site_key(scores[i], i);
            if (key >= kth) cand[atomicAdd(&count_s, 1)] = key;
        }
        __syncthreads();
        count = count_s;
    }

    // (3) sort the candidates in descending order; the first k are the points
    int size_all = 2;
    while (size_all < count) size_all <<= 1;
    for (int i = count + t; i < size_all; i += kSiteThreads) cand[i] = 0ull;
    __syncthreads();
    for (int size = 2; size <= size_all; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            // pair p: the p-th index with the stride bit clear, and its partner
            for (int p = t; p < size_all / 2; p += kSiteThreads) {
                const int i = 2 * p - (p & (stride - 1)), j = i + stride;
                const bool desc = (i & size) == 0;
                const uint64_t a = cand[i], b = cand[j];
                if ((a < b) == desc) {
                    cand[i] = b;
                    cand[j] = a;
                }
            }
            __syncthreads();
        }

    // (4) voxel coordinates of the points; labels start as their ranks
    for (int a = t; a < k; a += kSiteThreads) {
        const int idx = (int)(0xFFFFFFFFu - (uint32_t)(cand[a] & 0xFFFFFFFFull));
        ci[a] = idx % nx;
        cj[a] = (idx / nx) % ny;
        ck[a] = idx / (nx * ny);
        lab[a] = a;
        out_index[a] = idx;
    }
    __syncthreads();

    // (5) union of every linked pair: a wave takes points a, a lane the points
    //     after a; a root is hooked under a smaller one, retried if another
    //     thread hooked it first
    for (int a = t >> 6; a < k; a += kSiteThreads / 64) {
        const int ai = ci[a], aj = cj[a], ak = ck[a];
        for (int b = a + 1 + lane; b < k; b += 64) {
            const int dx = ai - ci[b], dy = aj - cj[b], dz = ak - ck[b];
            if (dx * dx + dy * dy + dz * dz > lim) continue;
            int u = find_root(lab, a), v = find_root(lab, b);
            while (u != v) {
                if (u < v) {
                    const int w = u;
                    u = v;
                    v = w;
                }
                const int old = atomicCAS(&lab[u], u, v);
                if (old == u) break;
                u = find_root(lab, old);
            }
        }
    }
    __syncthreads();
    for (int a = t; a < k; a += kSiteThreads) out_label[a] = find_root(lab, a);
}

}  // namespace

hipError_t launch_site_extract(const float *scores, const int *dims, int k, int lim, int *out_index, int *out_label,
                               hipStream_t stream)
{
    if (k < 1 || k > kMaxSitePoints) return hipErrorInvalidValue;
    if (((uintptr_t)scores & 15u) == 0)
        site_extract_kernel<true><<<1, kSiteThreads, 0, stream>>>(scores, dims[0], dims[1], dims[2], k, lim, out_index,
                                                                  out_label);
    else
        site_extract_kernel<false><<<1, kSiteThreads, 0, stream>>>(scores, dims[0], dims[1], dims[2], k, lim,
                                                                   out_index, out_label);
    return hipGetLastError();
}

}  // namespace dsdp
