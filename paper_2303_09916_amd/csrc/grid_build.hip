// Receptor grid maps on gfx950: score and gradient per node and per ligand XS type.
//
// Paper: Section 2, "Binding pose search", first modification (every node stores
// the summed interaction with receptor atoms within the cutoff, plus its
// gradient); Appendix eq. 1.  Terms: Vina's (ref. [6]), kept unchanged by the paper.
//
// Design: one workgroup per 8x8x4 tile of nodes; each of its four waves owns a
// 4x4x4 block (one node per lane) and carries all T map types in registers.
// Receptor atoms arrive sorted by 4 A cells (host counting sort); the workgroup
// stages the atoms of the cells within the cutoff of its tile into LDS (rows of
// cells are contiguous in the sorted array).  A wave takes them 64 at a time, one
// per lane, keeps those within the cutoff of its own block (a ballot), and sweeps
// the kept ones in order: the atom's values come from lane reads, so everything
// that depends on the atom alone is uniform over the wave and is branched on
// instead of selected.
//
// Bound by VALU issue.  A node sums each atom's terms in the order of the sorted
// array, so the sums are those of any other tiling; what is saved is work:
//  - the two exponentials and the class-free terms depend on the pair's radius
//    sum only and are formed once for all map types of one XS radius (T maps
//    arrive ordered by radius; 8 types of a usual palette have 4 radii);
//  - the hydrophobic and hydrogen-bond terms are formed only for atoms and maps
//    of that class;
//  - a 4x4x4 block is within the cutoff of 72 atoms at protein density where an
//    8x8x1 slab is of 83, and wastes fewer lanes at the box faces;
//  - the root and the reciprocal are the shortest sequences that still round
//    correctly (rounding.h).
// Measured on MI355X, kernel alone (medians of one box), in the form that evaluated every
// map on its own over 8x8x1 slabs, and in this one: 81^3 nodes, 8 types, 4000 atoms 272 and
// 120 us; 107^3, 9 types, 12000 atoms 589 and 243 us; 43^3, 4 types, 300 atoms 72 and 26 us
// (35 with all maps in one run, see runs_wanted).
#include "dsdp_internal.h"
#include "map_runs.h"
#include "rounding.h"

#include <algorithm>
#include <utility>

namespace dsdp {
namespace {

constexpr int TX = kTileX, TY = kTileY, TZ = kTileZ;
constexpr int kThreads = TX * TY * TZ;
constexpr int BX = 4, BY = 4;        // a wave's block of nodes (x and y; all of TZ)
constexpr int kStageCap = 512;       // atoms staged per pass (8 KB of LDS)
constexpr uint32_t kPolar = 1u << 31;
constexpr long kFillWaves = 12;      // waves per compute unit: three per SIMD

struct BuildArgs {
    const float4 *atoms;      // sorted by cell: x, y, z, XS type bits
    const int *cell_start;    // [ncell + 1]
    int cn[3];
    float clo[3];
    float cell;
    GridView g;
    // the maps ordered by XS radius, in n_parts runs that end on a change of radius;
    // a workgroup builds one run: maps part[p] to part[p + 1] - 1
    int n_parts, part[kNXS + 1];
    float radius[kNXS];       // radius of the k-th map's type
    int slot[kNXS];           // its index in the caller's order
    uint32_t first;           // bit k: the k-th map is the first of its radius
    // per receptor type: its radius, and the maps k with a class term (bit k;
    // kPolar: the term is the hydrogen bond, else the hydrophobic one)
    float rec_radius[kNXS];
    uint32_t rec_class[kNXS];
    float4 *maps;
};

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// f(0), f(1), ..., f(N - 1) with compile-time indices
template <int... I, typename F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F f)
{
    each_of(std::make_integer_sequence<int, N>(), f);
}

template <int TMAX>
__global__ __launch_bounds__(kThreads) void grid_build_kernel(const BuildArgs a)
{
    __shared__ float4 s_atoms[kStageCap];
    __shared__ float s_rad[kNXS];
    __shared__ uint32_t s_cls[kNXS];
    __shared__ int s_row_begin[kMaxRows], s_row_pre[kMaxRows + 1];
    __shared__ int s_half;

    const GridView &g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = blockIdx.z % a.n_parts, k0 = a.part[part], T = a.part[part + 1] - k0;
    const uint32_t first = a.first >> k0;
    const int t0x = blockIdx.x * TX, t0y = blockIdx.y * TY, t0z = blockIdx.z / a.n_parts * TZ;
    const int b0x = t0x + (wave & 1) * BX, b0y = t0y + (wave >> 1) * BY;
    const int i = b0x + (lane & 3), j = b0y + ((lane >> 2) & 3), k = t0z + (lane >> 4);
    const float mx = g.origin[0] + g.h * (float)i;
    const float my = g.origin[1] + g.h * (float)j;
    const float mz = g.origin[2] + g.h * (float)k;

    if (tid < kNXS) {
        s_rad[tid] = a.rec_radius[tid];
        s_cls[tid] = ((a.rec_class[tid] & ~kPolar) >> k0) | (a.rec_class[tid] & kPolar);
    }

    // cell rows covering the tile expanded by the cutoff: one row per thread,
    // then an exclusive scan of their lengths (two waves hold the rows)
    int lo[3], hi[3];
    const int t0[3] = {t0x, t0y, t0z};
    const int tn[3] = {TX, TY, TZ};
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        const float plo = g.origin[ax] + g.h * (float)t0[ax] - kCutoff;
        const float phi = g.origin[ax] + g.h * (float)(t0[ax] + tn[ax] - 1) + kCutoff;
        lo[ax] = max(0, (int)floorf((plo - a.clo[ax]) / a.cell));
        hi[ax] = min(a.cn[ax] - 1, (int)floorf((phi - a.clo[ax]) / a.cell));
    }
    const int ny = hi[1] - lo[1] + 1, nz = hi[2] - lo[2] + 1;
    const int nrows = lo[0] > hi[0] || ny <= 0 || nz <= 0 ? 0 : min(ny * nz, kMaxRows);   // (the host has checked)
    int begin = 0, len = 0, pre = 0;
    if (tid < nrows) {
        const int base = ((lo[2] + tid / ny) * a.cn[1] + lo[1] + tid % ny) * a.cn[0];
        begin = a.cell_start[base + lo[0]];
        len = a.cell_start[base + hi[0] + 1] - begin;
    }
    if (tid < kMaxRows) {
        pre = len;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(pre, o, 64);
            if (lane >= o) pre += v;
        }
        if (tid == 63) s_half = pre;
    }
    __syncthreads();
    if (tid < kMaxRows) {
        if (tid >= 64) pre += s_half;
        s_row_begin[tid] = begin;
        s_row_pre[tid + 1] = pre;
        if (tid == 0) s_row_pre[0] = 0;
    }
    __syncthreads();
    const int total = s_row_pre[kMaxRows];

    float E[TMAX], Gx[TMAX], Gy[TMAX], Gz[TMAX];
#pragma unroll
    for (int t = 0; t < TMAX; t++) E[t] = Gx[t] = Gy[t] = Gz[t] = 0.0f;

    // the wave's block (node positions are monotonic in the index)
    const bool block_in = b0x < g.n[0] && b0y < g.n[1];
    const float bx0 = g.origin[0] + g.h * (float)b0x, bx1 = g.origin[0] + g.h * (float)(b0x + BX - 1);
    const float by0 = g.origin[1] + g.h * (float)b0y, by1 = g.origin[1] + g.h * (float)(b0y + BY - 1);
    const float bz0 = g.origin[2] + g.h * (float)t0z, bz1 = g.origin[2] + g.h * (float)(t0z + TZ - 1);

    for (int base = 0; base < total; base += kStageCap) {
        const int cnt = min(kStageCap, total - base);
        for (int q = tid; q < cnt; q += kThreads) {
            // the row that holds atom base + q: the last with prefix <= it
            int r = 0;
#pragma unroll
            for (int o = kMaxRows / 2; o > 0; o >>= 1)
                if (s_row_pre[r + o] <= base + q) r += o;
            s_atoms[q] = a.atoms[s_row_begin[r] + (base + q - s_row_pre[r])];
        }
        __syncthreads();
        for (int c = 0; block_in && c < cnt; c += 64) {
            const float4 at = s_atoms[min(c + lane, cnt - 1)];
            // distance to the block; the margin covers the rounding of the
            // squared distances below, so no atom within a node's cutoff is left out
            const float ox = fmaxf(fmaxf(bx0 - at.x, at.x - bx1), 0.f);
            const float oy = fmaxf(fmaxf(by0 - at.y, at.y - by1), 0.f);
            const float oz = fmaxf(fmaxf(bz0 - at.z, at.z - bz1), 0.f);
            const int ta = __float_as_int(at.w);
            const uint32_t cls_l = s_cls[ta];
            float sum_l[TMAX];   // radius sums of the lane's atom
#pragma unroll
            for (int t = 0; t < TMAX; t++) sum_l[t] = a.radius[min(k0 + t, kNXS - 1)] + s_rad[ta];
            uint64_t keep = __ballot(c + lane < cnt && ox * ox + oy * oy + oz * oz < kCutoff2 + 0.01f);
            while (keep) {
#pragma clang fp contract(off)
                const int l = __builtin_ctzll(keep);
                keep &= keep - 1;
                const float dx = mx - lane_value(at.x, l), dy = my - lane_value(at.y, l),
                            dz = mz - lane_value(at.z, l);
                const uint32_t cls = (uint32_t)__builtin_amdgcn_readlane((int)cls_l, l);
                const float r2 = fmaf(dz, dz, fmaf(dx, dx, dy * dy));
                if (r2 < kCutoff2) {
                    // r and 1 / r, correctly rounded.  A distance below 2^-45 is as good as
                    // 0 (every radius sum is above 1).
                    const float r = sqrt_normal(__int_as_float(max(__float_as_int(r2), 0x12800000)));
                    const float inv = rcp_normal(r);
                    const float half_inv = r > 1e-9f ? 0.5f * inv : 0.0f;
                    // Vina's pair term on the surface distance d; the derivative is
                    // carried doubled (de2), which scales every product exactly
                    float d = 0.f, e = 0.f, de2 = 0.f, gs = 0.f;
                    constexpr float kLog2e = 1.44269504088896341f;
                    // unrolled by the template, so that the accumulators are
                    // registers before any branch is seen
                    each<TMAX>([&](auto index) {
#pragma clang fp contract(off)
                        constexpr int t = decltype(index)::value;
                        if (t < T) {
                            if (first & (1u << t)) {
                                d = r - lane_value(sum_l[t], l);
                                const float b = d - 3.0f;
                                const float g1 = __builtin_amdgcn_exp2f((d * d) * (-4.0f * kLog2e));
                                const float g2 = __builtin_amdgcn_exp2f((b * b) * (-0.25f * kLog2e));
                                const float dn = fminf(d, 0.0f);
                                const float m2 = g2 * kWGauss2;
                                e = fmaf(dn, kWRepulsion * dn, fmaf(g1, kWGauss1, m2));
                                de2 = fmaf(d, g1 * (-16.0f * kWGauss1), -(b * m2));
                                de2 = fmaf(kWRepulsion * 4.0f, dn, de2);
                                gs = half_inv * de2;
                            }
                            if (cls & (1u << t)) {
                                // at a kink the left-hand slope is taken
                                float p, h2;
                                if (cls & kPolar) {
                                    p = kWHBond * fminf(fmaxf(d * -(1.0f / 0.7f), 0.0f), 1.0f);
                                    h2 = (d > -0.7f && d <= 0.0f) ? -2.0f * (kWHBond * (1.0f / 0.7f)) : 0.0f;
                                } else {
                                    p = kWHydrophobic * fminf(fmaxf(1.5f - d, 0.0f), 1.0f);
                                    h2 = (d > 0.5f && d <= 1.5f) ? -2.0f * kWHydrophobic : 0.0f;
                                }
                                const float gt = half_inv * (de2 + h2);
                                E[t] += e + p;
                                Gx[t] = fmaf(gt, dx, Gx[t]);
                                Gy[t] = fmaf(gt, dy, Gy[t]);
                                Gz[t] = fmaf(gt, dz, Gz[t]);
                            } else {
                                E[t] += e;
                                Gx[t] = fmaf(gs, dx, Gx[t]);
                                Gy[t] = fmaf(gs, dy, Gy[t]);
                                Gz[t] = fmaf(gs, dz, Gz[t]);
                            }
                        }
                    });
                }
            }
        }
        __syncthreads();
    }

    if (i < g.n[0] && j < g.n[1] && k < g.n[2]) {
        const long nodes = (long)g.n[0] * g.n[1] * g.n[2];
        const long node = ((long)k * g.n[1] + j) * g.n[0] + i;
#pragma unroll
        for (int t = 0; t < TMAX; t++)
            if (t < T) a.maps[(long)a.slot[k0 + t] * nodes + node] = make_float4(E[t], Gx[t], Gy[t], Gz[t]);
    }
}

}  // namespace

hipError_t launch_grid_build(const float4 *atoms, const int *cell_start, const int *cn, const float *clo, float cell,
                             const GridView &g, const int *map_types_host, float4 *maps, long cus, hipStream_t stream)
{
    if (cell_rows(g.h, cell) > kMaxRows) return hipErrorInvalidValue;
    BuildArgs a;
    a.atoms = atoms;
    a.cell_start = cell_start;
    for (int ax = 0; ax < 3; ax++) {
        a.cn[ax] = cn[ax];
        a.clo[ax] = clo[ax];
    }
    a.cell = cell;
    a.g = g;
    // order the maps by radius (stable), so that maps of one radius follow each other
    for (int t = 0; t < kNXS; t++) {
        a.slot[t] = t;
        a.radius[t] = 0.f;
        a.rec_radius[t] = xs_radius(t);
        a.rec_class[t] = 0u;
    }
    std::stable_sort(a.slot, a.slot + g.T, [&](int u, int v) {
        return xs_radius(map_types_host[u]) < xs_radius(map_types_host[v]);
    });
    a.first = 0u;
    for (int k = 0; k < g.T; k++) {
        const int mt = map_types_host[a.slot[k]];
        a.radius[k] = xs_radius(mt);
        if (k == 0 || a.radius[k] != a.radius[k - 1]) a.first |= 1u << k;
        for (int r = 0; r < kNXS; r++) {
            // a receptor type is hydrophobic or polar, never both
            const uint32_t fl = pair_flags(mt, r);
            if (fl) a.rec_class[r] |= (1u << k) | ((fl & kPairHBond) ? kPolar : 0u);
        }
    }
    a.maps = maps;

    const dim3 tiles((g.n[0] + TX - 1) / TX, (g.n[1] + TY - 1) / TY, (g.n[2] + TZ - 1) / TZ);
    const long waves = (long)((g.n[0] + BX - 1) / BX) * ((g.n[1] + BY - 1) / BY) * tiles.z;
    a.n_parts = split_maps(a.first, g.T, runs_wanted(waves, kFillWaves * cus, g.T), a.part);
    int max_maps = 0;
    for (int r = 0; r < a.n_parts; r++) max_maps = std::max(max_maps, a.part[r + 1] - a.part[r]);
    const dim3 grid(tiles.x, tiles.y, tiles.z * a.n_parts);
#define DSDP_BUILD(N) grid_build_kernel<N><<<grid, kThreads, 0, stream>>>(a)
    switch (max_maps) {
    case 1: DSDP_BUILD(1); break;
    case 2: DSDP_BUILD(2); break;
    case 3: case 4: DSDP_BUILD(4); break;
    case 5: case 6: DSDP_BUILD(6); break;
    case 7: case 8: DSDP_BUILD(8); break;
    case 9: DSDP_BUILD(9); break;
    case 10: case 11: case 12: DSDP_BUILD(12); break;
    default: DSDP_BUILD(kNXS); break;
    }
#undef DSDP_BUILD
    return hipGetLastError();
}

}  // namespace dsdp
