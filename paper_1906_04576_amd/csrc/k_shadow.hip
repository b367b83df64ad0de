// Soft shadows (Sec. 2.4: shadow map after Williams 1978, percentage-closer
// filtering after Reeves et al. 1987, PCSS penumbra after Fernando 2005) and
// the one-sample shadow test whose differences add shadow edges to the mask
// (Sec. 3.1).
//
// Light coordinates: P_l = M P (3 x 4 affine, rows summed left to right),
// d_r = -P_l.z, su = c_L + (P_l.x / d_r) f_L, sv = c_L - (P_l.y / d_r) f_L,
// c_L = size / 2.  Outside the light frustum = lit.  Blocker search over a
// disk of half-width R_s = (l (d_r - n_L)) / (d_r n_L), l = f_L (w_L / 2);
// penumbra R_f = (l (d_r - d_b)) / (d_b d_r) from the mean blocker depth d_b;
// visibility = share of PCF taps that are not in front of d_r - bias.
#include "shadow_light.hpp"

namespace mr {

__global__ __launch_bounds__(256) void k_hard(HardArgs a) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= a.W || y >= a.H) return;
    const long long p = (long long)y * a.W + x;
    const float z = a.depth[p];
    uint8_t h = 0;
    if (valid_depth(z)) {
        float px, py, pz;
        view_pos<false>(x, y, z, a.f, 0.5f * (float)a.W, 0.5f * (float)a.H, px, py, pz);
        const LightCoord c = to_light(a.M, a.size, a.fL, px, py, pz);
        if (c.inside) {
            const float thr = c.dr - a.bias;
            h = a.sm[(long long)(int)floorf(c.sv) * a.size + (int)floorf(c.su)] < thr ? 1 : 0;
        }
    }
    a.hard[p] = h;
}

hipError_t launch_hard(const HardArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_hard, dim3((a.W + 63) / 64, (a.H + 3) / 4), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Shadow-map taps whose gathers are in flight together.  (One tap at a time,
// each waiting for its gather, the evaluation was bound by that latency: 150
// us of a 246 us frame at 3840 x 2160 with 16 blocker and 32 PCF taps.)
constexpr int kTaps = 8;

// taps su + R ox, sv + R oy of the map, clamped to it
struct ShadowTaps {
    __amdgpu_buffer_rsrc_t map;
    float su, sv;
    int size;
    template <typename DP>
    __device__ __forceinline__ float operator()(DP disk, int k, float R) const {
        // the floors saturate, NaN gives 0, as the clamp of the float would
        const int x = min(max(floor_i32(su + R * disk[2 * k]), 0), size - 1);
        const int y = min(max(floor_i32(sv + R * disk[2 * k + 1]), 0), size - 1);
        return buf_f1(map, (__umul24((unsigned)y, (unsigned)size) + (unsigned)x) * 4u);
    }
};

// f(s) for every tap's depth s, in order of the taps: groups of kTaps, then of
// half as many and of two, then what is left (naive pass at 1920 x 1080 with 4 +
// 4 taps 51.3 us with single taps after the groups of 8, 40.5 us so)
template <typename DP, typename F>
__device__ __forceinline__ void for_taps(const ShadowTaps& t, DP disk, int n, float R, F&& f) {
    int k = 0;
    auto group = [&](auto count) {
        constexpr int N = decltype(count)::value;
        float s[N];
#pragma unroll
        for (int q = 0; q < N; ++q) s[q] = t(disk, k + q, R);
#pragma unroll
        for (int q = 0; q < N; ++q) f(s[q]);
        k += N;
    };
    while (k + kTaps <= n) group(std::integral_constant<int, kTaps>{});
    if (k + kTaps / 2 <= n) group(std::integral_constant<int, kTaps / 2>{});
    if (k + 2 <= n) group(std::integral_constant<int, 2>{});
    if (k < n) group(std::integral_constant<int, 1>{});
}

// visibility of one texel; BD / PD point to LDS (staged disks) or global memory
template <typename DP>
__device__ __forceinline__ float pcss_texel(const ShadowArgs& a, const EvalLevel& L, DP bd, DP pd, int x, int y,
                                            float z) {
    float px, py, pz;
    view_pos<false>(x, y, z, L.f, L.cx, L.cy, px, py, pz);
    const LightCoord c = to_light(a.M, a.size, a.fL, px, py, pz);
    if (!c.inside) return 1.0f;
    const ShadowTaps taps{buf_rsrc(a.sm, 4u * (unsigned)a.size * (unsigned)a.size), c.su, c.sv, a.size};
    const float lsz = a.fL * (0.5f * a.lsize);
    const float thr = c.dr - a.bias;
    const float Rs = (lsz * (c.dr - a.nL)) / (c.dr * a.nL);
    float bsum = 0.0f;
    int bcnt = 0;
    for_taps(taps, bd, a.nb, Rs, [&](float s) {
        const bool blocks = s < thr;
        bsum = bsum + (blocks ? s : 0.0f);
        bcnt += blocks ? 1 : 0;
    });
    if (bcnt == 0) return 1.0f;
    const float db = bsum / (float)bcnt;
    const float Rf = (lsz * (c.dr - db)) / (db * c.dr);
    int dark = 0;
    for_taps(taps, pd, a.np, Rf, [&](float s) { dark += s < thr ? 1 : 0; });
    return (float)(a.np - dark) / (float)a.np;
}

template <bool LDS, bool AL>
__device__ __forceinline__ void pcss_items(const ShadowArgs& a, const float* bds, const float* pds,
                                           const float* rows) {
    const ItemMap m = make_item_map(a.c);
    const unsigned total = item_total(m), nchunks = (total + 255) / 256;
    const ChunkRange cr = AL ? chunk_range(nchunks) : level_chunks(nchunks);
    for (unsigned c = cr.first; c < cr.end; c += cr.step) {
        const unsigned item = c * 256u + threadIdx.x;
        if (item >= total) continue;
        const int j = item_level(m, item);
        const EvalLevel& L = a.c.lv[j];
        const unsigned local = item_local(m, item, j);
        if (local == ~0u) continue;  // padding of the level's item range
        const unsigned t = L.list ? L.list[local] : local;
        if (t >= L.dense_n) continue;  // malformed list entry
        const int y = (int)(t / (unsigned)L.W), x = (int)(t - (unsigned)y * (unsigned)L.W);
        const float z = L.z[(unsigned)y * L.zpy + (unsigned)x * L.zpx];
        if (AL && L.ac) L.ac[local] = alpha_dispatch(L, rows, j, x, y);
        float vis = 1.0f;
        if (valid_depth(z)) {
            if (LDS)
                vis = pcss_texel(a, L, bds, pds, x, y, z);
            else
                vis = pcss_texel(a, L, a.bd, a.pd, x, y, z);
        }
        store_out(L, L.compact ? local : (unsigned)y * (unsigned)L.W + (unsigned)x, vis);
    }
}

// LDS: the disks are staged in LDS (at most kLdsSamples points each).  The
// multi-resolution instance runs four waves per SIMD: its texels, near shadow
// edges, search a large part of the map, which the L2 caches do not hold, and
// more waves only make it worse (4K frame 230, 233 and 237 us at 4, 6 and 8;
// 119 us with every tap in the same 16 KB).
template <bool AL, bool LDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(AL ? 4 : 1, AL ? 4 : 8)))
void k_pcss(ShadowArgs a) {
    __shared__ float bds[LDS ? 2 * kLdsSamples : 1], pds[LDS ? 2 * kLdsSamples : 1];
    __shared__ float rows[kRowLevels * kRowTable];
    if (AL) stage_rows(a.c, rows);
    if (LDS) {
        for (int i = threadIdx.x; i < 2 * a.nb; i += 256) bds[i] = a.bd[i];
        for (int i = threadIdx.x; i < 2 * a.np; i += 256) pds[i] = a.pd[i];
    }
    __syncthreads();
    pcss_items<LDS, AL>(a, bds, pds, rows);
}

hipError_t launch_shadow(const ShadowArgs& a, unsigned total_hint, hipStream_t s) {
    const bool lds = a.nb <= kLdsSamples && a.np <= kLdsSamples;
    // a tap counts as two samples: with 2 + 2 of them a block per chunk is the
    // faster grid (3840 x 2160 74 us, 85 us with a resident grid), with 1 + 1 not
    // (53 and 47 us)
#define MR_PCSS(AL, LD) \
    hipLaunchKernelGGL((k_pcss<AL, LD>), dim3(eval_grid<k_pcss<AL, LD>>(a.c, total_hint, 2 * (a.nb + a.np))), dim3(256), 0, s, a)
    if (fused_alpha(a.c)) {
        if (lds) MR_PCSS(true, true);
        else MR_PCSS(true, false);
    } else {
        if (lds) MR_PCSS(false, true);
        else MR_PCSS(false, false);
    }
#undef MR_PCSS
    return hipGetLastError();
}

}  // namespace mr
