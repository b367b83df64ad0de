// SSAO evaluated per sub-image (Sec. 3.2 / 4.1) and as the naive full-res
// pass (Sec. 5).  The paper cites Mittring 2007 and Bavoil et al. 2008 for
// SSAO without printing an estimator; this one is a normal-oriented
// hemisphere with a fixed caller-supplied kernel, a hard range check and a
// relative depth bias; output = occluded fraction.
#pragma once
#include "sample_hits.hpp"

namespace mr {


// A staged copy of the level depth around a tile: tw x tw texels from
// (x0, y0), in LDS.  TILE: a sample whose texel lies in it reads it there,
// the others read the depth plane.
struct DepthTile {
    const float* t;
    unsigned x0, y0, tw;
};

// Samples in flight together in the launches with depth tiles: kTileGroup of
// the list levels' texels, kTilePair of a tile's, whose gathers mostly end in
// LDS and which are not tested a group behind.  Frame at 3840 x 2160 with 64
// samples, halos 8, 16, 24: 123.1, 124.8, 125.7 us with groups of 8 for both
// (84 to 89 registers, 5 waves per SIMD); 116.2, 118.0, 118.1 us with groups
// of 4 and 8 waves per SIMD; 115.4, 116.1, 115.7 us with the pairs.
constexpr int kTileGroup = 4, kTilePair = 2;

// gathers from a staged square of on-screen texels, else from the plane
struct TileGather {
    __amdgpu_buffer_rsrc_t rz;
    DepthTile dt;
    unsigned last;
    __device__ __forceinline__ float operator()(unsigned off, int x, int y) const {
        const unsigned dx = (unsigned)x - dt.x0, dy = (unsigned)y - dt.y0;
        if ((dx < dt.tw) & (dy < dt.tw) & (off <= last)) return dt.t[dy * dt.tw + dx];
        return buf_f1(rz, off);
    }
};

// Occluding samples of one texel.  FAST: in groups of N samples, the gathers
// of one group in flight while the one before is tested (kGroup measured on
// multi-resolution frames: 3840 x 2160 104.7 us for groups of 4 and 101.6 us
// for groups of 8, with fewer waves but twice the gathers in flight).
template <bool FAST, int N, typename SA, typename KP, typename GF>
__device__ __forceinline__ int ssao_count(const SA& a, const EvalLevel& L, KP K, const SampleTexel& T,
                                          const GF& gather) {
    const float r = a.r, b = a.b;
    const int S = a.S;
    int occ = 0, s = 0;
    if constexpr (FAST) {
        auto count = [&](const auto& g) { return __popc(test_samples(T, g, r, b, 0u)); };
        if (S >= N) {
            SampleGroup<N> A, B;
            issue_samples(L, K, 0, T, gather, A);
            for (s = N; s + 2 * N <= S; s += 2 * N) {
                issue_samples(L, K, s, T, gather, B);
                occ += count(A);
                issue_samples(L, K, s + N, T, gather, A);
                occ += count(B);
            }
            if (s + N <= S) {
                issue_samples(L, K, s, T, gather, B);
                occ += count(A);
                occ += count(B);
                s += N;
            } else {
                occ += count(A);
            }
        }
        if (N >= 8 && s + N / 2 <= S) {
            SampleGroup<N / 2> A;
            issue_samples(L, K, s, T, gather, A);
            occ += count(A);
            s += N / 2;
        }
        for (; s < S; ++s) {
            SampleGroup<1> A;
            issue_samples(L, K, s, T, gather, A);
            occ += count(A);
        }
    } else {
        constexpr int G = 2;
        for (; s + G <= S; s += G) {
            bool on[G];
            float d[G], zs[G];
#pragma unroll
            for (int k = 0; k < G; ++k) {
                unsigned off;
                int x, y;
                project_any<false>(L, K, s + k, T, on[k], d[k], off, x, y);
                zs[k] = gather(off, x, y);
            }
#pragma unroll
            for (int k = 0; k < G; ++k) occ += occludes_any(on[k], T.z, d[k], zs[k], r, b) ? 1 : 0;
        }
        for (; s < S; ++s) {
            bool on;
            float d;
            unsigned off;
            int x, y;
            project_any<false>(L, K, s, T, on, d, off, x, y);
            occ += occludes_any(on, T.z, d, gather(off, x, y), r, b) ? 1 : 0;
        }
    }
    return occ;
}

// the same count of a tile's texel (fast form): kTilePair projections, then
// their gathers, then their tests
template <typename SA, typename KP>
__device__ __forceinline__ int ssao_count_tile(const SA& a, const EvalLevel& L, KP K, const SampleTexel& T,
                                               const TileGather& gather) {
    int occ = 0, s = 0;
    auto test = [&](auto count) {
        constexpr int N = decltype(count)::value;
        SampleGroup<N> g;
        unsigned off[N];
        int x[N], y[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            project_fast(L, K, s + k, T, g.d[k], off[k], x[k], y[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) g.zs[k] = gather(off[k], x[k], y[k]);
        occ += __popc(test_samples(T, g, a.r, a.b, 0u));
        s += N;
    };
    while (s + kTilePair <= a.S) test(std::integral_constant<int, kTilePair>{});
    while (s < a.S) test(std::integral_constant<int, 1>{});
    return occ;
}

// occlusion of one texel; K points to LDS (staged samples) or global memory;
// kmax as in fast_samples; a holds the sampling parameters r, b and S
// (SsaoArgs or SsaoSampling); dt: TILE, the staged square
template <int N, bool TILE = false, typename SA, typename KP>
__device__ __forceinline__ float ssao_texel(const SA& a, const EvalLevel& L, const Normal& n, KP K, float kmax, int x,
                                            int y, float z, const DepthTile& dt = DepthTile{}) {
    const SampleTexel T = sample_texel(L, n, a.r, x, y, z);
    const unsigned last = last_texel(L);
    const __amdgpu_buffer_rsrc_t rz = buf_rsrc(L.z, last + 4u);
    int occ;
    if constexpr (TILE) {
        const TileGather gather{rz, dt, last};
        occ = fast_samples(T, kmax, a.r) ? ssao_count_tile(a, L, K, T, gather) : ssao_count<false, N>(a, L, K, T, gather);
    } else {
        const PlaneGather gather{rz};
        occ = fast_samples(T, kmax, a.r) ? ssao_count<true, N>(a, L, K, T, gather)
                                         : ssao_count<false, N>(a, L, K, T, gather);
    }
    return (float)occ / (float)a.S;
}

// one item (a listed texel, or a texel of a dense level)
template <typename NT, bool KLDS, bool AL, int N = kGroup>
__device__ __forceinline__ void ssao_item(const SsaoArgs& a, const ItemMap& m, unsigned item, const float* ks,
                                          const float* rows, float kmax) {
    const NT* nrm = static_cast<const NT*>(a.c.normal);
    const unsigned plane = (unsigned)a.c.plane;
    const int j = item_level(m, item);
    const EvalLevel& L = a.c.lv[j];
    const unsigned local = item_local(m, item, j);
    if (local == ~0u) return;  // padding of the level's item range
    const unsigned t = L.list ? L.list[local] : local;
    if (t >= L.dense_n) return;  // malformed list entry
    const int y = (int)(t / (unsigned)L.W), x = (int)(t - (unsigned)y * (unsigned)L.W);
    // depth and normal are on their way while a_i is computed
    const float z = L.z[(unsigned)y * L.zpy + (unsigned)x * L.zpx];
    const Normal n = texel_normal(L, nrm, plane, x, y);
    if (AL && L.ac) L.ac[local] = alpha_dispatch(L, rows, j, x, y);
    float res = 0.0f;
    if (valid_depth(z)) {
        if (KLDS)
            res = ssao_texel<N>(a, L, n, ks, kmax, x, y, z);
        else
            res = ssao_texel<N>(a, L, n, a.kernel, kmax, x, y, z);
    }
    store_out(L, L.compact ? local : (unsigned)y * (unsigned)L.W + (unsigned)x, res);
}

template <typename NT, bool KLDS, bool AL>
__device__ __forceinline__ void ssao_items(const SsaoArgs& a, const float* ks, const float* rows, float kmax) {
    const ItemMap m = make_item_map(a.c);
    const unsigned total = item_total(m), nchunks = (total + 255) / 256;
    const ChunkRange cr = AL ? chunk_range(nchunks) : level_chunks(nchunks);
    for (unsigned c = cr.first; c < cr.end; c += cr.step) {
        const unsigned item = c * 256u + threadIdx.x;
        if (item < total) ssao_item<NT, KLDS, AL>(a, m, item, ks, rows, kmax);
    }
}

// The multi-resolution evaluation with the dense coarsest level in 16 x 16
// texel tiles, each with a halo of H texels of its depth staged in LDS (zt,
// (16 + 2H)^2 floats) before its texels' samples gather: the samples that
// land in the staged square read it there.  Values outside the level are
// staged clamped; only off-screen samples, which never count, can reach
// them.  The list levels' chunks run as in ssao_items; they come first in a
// block's sweep, so that zt takes over the LDS of their row tables.
template <typename NT, int H>
__device__ __forceinline__ void ssao_items_tiled(const SsaoArgs& a, const float* ks, float* zt, float kmax) {
    constexpr int TW = kDenseTile + 2 * H;
    static_assert(TW * TW >= kRowLevels * kRowTable, "the row tables lie in the depth tile's LDS");
    const ItemMap m = make_item_map(a.c);
    const unsigned total = item_total(m);
    const int jd = m.nlev - 1;  // the dense coarsest level
    unsigned dense0 = 0;
#pragma unroll
    for (int k = 0; k < kMaxLevels; ++k) dense0 = k == jd ? m.cum[k] : dense0;
    const NT* nrm = static_cast<const NT*>(a.c.normal);
    const unsigned plane = (unsigned)a.c.plane;
    const ChunkRange cr = chunk_range((total + 255) / 256);
    for (unsigned c = cr.first; c < cr.end; c += cr.step) {
        if (c * 256u < dense0) {
            const unsigned item = c * 256u + threadIdx.x;
            if (item < total) ssao_item<NT, true, true, kTileGroup>(a, m, item, ks, zt, kmax);
            continue;
        }
        const EvalLevel& L = a.c.lv[jd];
        const unsigned tile = c - dense0 / 256u, tx = dense_tiles_x(L.W);
        const int x0 = (int)(tile % tx) * kDenseTile, y0 = (int)(tile / tx) * kDenseTile;
        __syncthreads();  // all reads of the row tables or of the tile before are done
        for (int i = threadIdx.x; i < TW * TW; i += 256) {
            const int ry = i / TW, rx = i - ry * TW;
            const int gx = min(max(x0 - H + rx, 0), L.W - 1), gy = min(max(y0 - H + ry, 0), L.H - 1);
            zt[i] = L.z[(unsigned)gy * (unsigned)L.zpy + (unsigned)gx * (unsigned)L.zpx];
        }
        __syncthreads();
        const int x = x0 + (int)(threadIdx.x % kDenseTile), y = y0 + (int)(threadIdx.x / kDenseTile);
        if (x < L.W && y < L.H) {
            const float z = zt[(y - y0 + H) * TW + (x - x0 + H)];
            float res = 0.0f;
            if (valid_depth(z)) {
                const DepthTile dt{zt, (unsigned)(x0 - H), (unsigned)(y0 - H), (unsigned)TW};
                res = ssao_texel<kTileGroup, true>(a, L, texel_normal(L, nrm, plane, x, y), ks, kmax, x, y, z, dt);
            }
            store_out(L, (unsigned)y * (unsigned)L.W + (unsigned)x, res);
        }
    }
}

// One chunk c of a frame's item space with the dense coarsest level in
// tiles (m built with TILES): a chunk of list items, or one 16 x 16 tile of
// the dense level evaluated from its LDS depth tile as in ssao_items_tiled.
// Every thread of the block takes part (the tile staging ends with
// barriers).  Used by the batch launch, whose frames share the LDS.
template <typename NT, int H>
__device__ __forceinline__ void ssao_chunk_tiled(const SsaoArgs& a, const ItemMap& m, unsigned c, const float* ks,
                                                 const float* rows, float kmax, float* zt) {
    constexpr int TW = kDenseTile + 2 * H;
    const unsigned total = item_total(m);
    const int jd = m.nlev - 1;  // the dense coarsest level
    unsigned dense0 = 0;
#pragma unroll
    for (int k = 0; k < kMaxLevels; ++k) dense0 = k == jd ? m.cum[k] : dense0;
    if (c * 256u < dense0) {
        const unsigned item = c * 256u + threadIdx.x;
        if (item < total) ssao_item<NT, true, true, kTileGroup>(a, m, item, ks, rows, kmax);
        return;
    }
    const NT* nrm = static_cast<const NT*>(a.c.normal);
    const unsigned plane = (unsigned)a.c.plane;
    const EvalLevel& L = a.c.lv[jd];
    const unsigned tile = c - dense0 / 256u, tx = dense_tiles_x(L.W);
    const int x0 = (int)(tile % tx) * kDenseTile, y0 = (int)(tile / tx) * kDenseTile;
    for (int i = threadIdx.x; i < TW * TW; i += 256) {
        const int ry = i / TW, rx = i - ry * TW;
        const int gx = min(max(x0 - H + rx, 0), L.W - 1), gy = min(max(y0 - H + ry, 0), L.H - 1);
        zt[i] = L.z[(unsigned)gy * (unsigned)L.zpy + (unsigned)gx * (unsigned)L.zpx];
    }
    __syncthreads();
    const int x = x0 + (int)(threadIdx.x % kDenseTile), y = y0 + (int)(threadIdx.x / kDenseTile);
    if (x < L.W && y < L.H) {
        const float z = zt[(y - y0 + H) * TW + (x - x0 + H)];
        float res = 0.0f;
        if (valid_depth(z)) {
            const DepthTile dt{zt, (unsigned)(x0 - H), (unsigned)(y0 - H), (unsigned)TW};
            res = ssao_texel<kTileGroup, true>(a, L, texel_normal(L, nrm, plane, x, y), ks, kmax, x, y, z, dt);
        }
        store_out(L, (unsigned)y * (unsigned)L.W + (unsigned)x, res);
    }
    __syncthreads();  // the next tile's staging overwrites zt
}

// samples of the tiled evaluation (staged in LDS with the depth tile)
constexpr int kTiledSamples = 256;

// Per block: the blur's row sums (AL) and, KLDS, the samples in LDS; returns
// the largest |component| of the samples.
template <bool AL, bool KLDS>
__device__ __forceinline__ float ssao_stage(const SsaoArgs& a, float* ks, float* rows) {
    return stage_samples<KLDS>(a.kernel, a.S, ks, [&] {
        if (AL) stage_rows(a.c, rows);
    });
}

}  // namespace mr
