// One-bounce screen-space indirect light (Sec. 2.4, after Ritschel et al.
// 2009).  The SSAO sampling and occlusion test are reused; every occluding
// sample adds the directly lit colour of the texel it hit, weighted as a
// small patch sending light to the receiver:
//   v = X_t - P, dd = dot(v, v), dist2 = max(dd, (0.1 r)^2),
//   v_hat = v / sqrt(dd), g = (max(0, n.v_hat) max(0, -n_t.v_hat)) / dist2,
//   acc += C_t g;  out = acc (r^2 / S).
#pragma once
#include "sample_hits.hpp"

namespace mr {

// element e of a plane of floats or halves, widened
template <typename T>
__device__ __forceinline__ float plane_ld(__amdgpu_buffer_rsrc_t r, unsigned e);
template <>
__device__ __forceinline__ float plane_ld<float>(__amdgpu_buffer_rsrc_t r, unsigned e) {
    return buf_f1(r, e * 4u);
}
template <>
__device__ __forceinline__ float plane_ld<_Float16>(__amdgpu_buffer_rsrc_t r, unsigned e) {
    return (float)__builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r, e * 2u, 0, 0));
}

// the three planes of a normal or colour image
template <typename T>
struct Planes {
    __amdgpu_buffer_rsrc_t r[3];
    __device__ __forceinline__ Planes(const T* p, unsigned plane) {
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = buf_rsrc(p + (size_t)c * plane, plane * (unsigned)sizeof(T));
    }
    __device__ __forceinline__ void load(unsigned e, float (&o)[3]) const {
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = plane_ld<T>(r[c], e);
    }
};

// samples whose depth gathers are in flight together (2, 4 and 8 measured the
// same: the light's six gathers per hit bound the launches)
constexpr int kLightGroup = 4;

// What a texel's light gathers from one occluding sample: the texel it hit.
struct LightHit {
    int x, y;
    float z, n[3], c[3];
};

template <typename NT, typename CT>
__device__ __forceinline__ void light_load(const EvalLevel& L, const Planes<NT>& nrm, const Planes<CT>& col, LightHit& h) {
    const unsigned e = (unsigned)L.goff + (unsigned)h.y * (unsigned)L.gpy + (unsigned)h.x * (unsigned)L.gpx;
    nrm.load(e, h.n);
    col.load(e, h.c);
}

// Whether light_add's fast form holds for the wave's texels (besides
// fast_samples): with these ranges a hit's position is below 2^28, so that
// d . d of its direction is 0 or in [2^-84, 2^60): either the depths differ,
// by an ulp of z at least, or the texels do, by about z / f.
__device__ __forceinline__ bool fast_light(const EvalLevel& L, const SampleTexel& T, float r) {
    const float rmin = 0.1f * r;
    const bool safe = (L.f >= kFocalLo) & (L.f < kFocalHi) & (rmin * rmin >= 0x1p-40f) & (r < 0x1p28f) &
                      (T.z + r < 0x1p11f * L.f);
    return __ballot(!safe) == 0;
}

// FAST: the three quotients and the square root by fused multiply-adds from
// reciprocals (rcf = 1/f); same bits.  About three samples in four light some
// lane of a wave, and the light is then most of its instructions: with the
// IEEE sequences the naive pass at 1080p took 228 us and the multi-resolution
// frame at 1440p 135 us, now 206 us and 126 us.
template <bool FAST>
__device__ __forceinline__ void light_add(const EvalLevel& L, const SampleTexel& T, const Normal& n, const LightHit& h,
                                          float rmin2, float rcf, float (&acc)[3]) {
    float hx, hy, hz;
    if constexpr (FAST) {
        hx = quotient(((float)h.x + 0.5f) - L.cx, L.f, rcf) * h.z;
        hy = quotient(L.cy - ((float)h.y + 0.5f), L.f, rcf) * h.z;
        hz = -h.z;
    } else {
        view_pos(h.x, h.y, h.z, L.f, L.cx, L.cy, hx, hy, hz);
    }
    const float vx = hx - T.px, vy = hy - T.py, vz = hz - T.pz;
    const float dd = ((vx * vx) + (vy * vy)) + (vz * vz);
    if (!(dd > 0.0f)) return;
    const float dist2 = fmaxf(dd, rmin2);
    const float il = FAST ? rsqrt_fast(dd) : rsqrt_pos(dd);  // = 1.0f / sqrtf(dd) (dd > 0)
    const float vhx = vx * il, vhy = vy * il, vhz = vz * il;
    const float cr = fmaxf(0.0f, ((n.x * vhx) + (n.y * vhy)) + (n.z * vhz));
    const float ce = fmaxf(0.0f, -(((h.n[0] * vhx) + (h.n[1] * vhy)) + (h.n[2] * vhz)));
    const float cc = cr * ce;
    float w;
    if constexpr (FAST) {
        // 2^-40 <= dist2 < 2^60; the square of cc is normal for cc in about
        // [2^-63, 2^64)
        constexpr int kZero = 0x60, kDenormal = 0x90, kInf = 0x204;  // v_cmp_class
        w = quotient(cc, dist2, recip_fast(dist2));
        const bool odd = __builtin_amdgcn_classf(cc * cc, kZero | kDenormal | kInf) & (cc != 0.0f);
        if (__builtin_expect(__ballot(odd) != 0, 0)) {
            if (odd) w = cc / dist2;
        }
    } else {
        w = cc / dist2;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = acc[c] + h.c[c] * w;
}

// The light of N samples from s: which of them occlude, the depth gathers of
// all in flight together, then sample by sample the light by the lanes that
// it occludes, the gathers of two samples in flight together.  All lanes are
// at the same sample, so that their gathers stay close together: lanes that
// each worked through their own hits (found for 32 samples before) gathered
// all over the image and ran the multi-resolution launches 12 % slower.
template <bool FAST, int N, typename NT, typename CT, typename KP>
__device__ __forceinline__ void light_group(const SsgiArgs& a, const EvalLevel& L, const SampleTexel& T, const Normal& n,
                                            KP K, int s, __amdgpu_buffer_rsrc_t rz, const Planes<NT>& np,
                                            const Planes<CT>& cp, float rmin2, float rcf, float (&acc)[3]) {
    float zs[N], d[N];
    unsigned xy[N];
    bool hit[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        unsigned off;
        int x, y;
        if constexpr (FAST)
            project_fast(L, K, s + k, T, d[k], off, x, y);
        else
            project_any<true>(L, K, s + k, T, hit[k], d[k], off, x, y);
        zs[k] = buf_f1(rz, off);
        xy[k] = __builtin_amdgcn_perm((unsigned)y, (unsigned)x, 0x05040100u);  // on screen both fit 16 bits
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
        hit[k] = FAST ? (int)occludes_fast(T.z, d[k], zs[k], a.r, a.b) < 0
                      : occludes_any(hit[k], T.z, d[k], zs[k], a.r, a.b);
#pragma unroll
    for (int k = 0; k < N; k += 2) {
        constexpr int P = N > 1 ? 2 : 1;  // samples at a time
        LightHit h[P];
#pragma unroll
        for (int q = 0; q < P; ++q)
            if (hit[k + q]) {
                h[q].x = (int)(xy[k + q] & 0xFFFFu), h[q].y = (int)(xy[k + q] >> 16), h[q].z = zs[k + q];
                light_load(L, np, cp, h[q]);
            }
#pragma unroll
        for (int q = 0; q < P; ++q)
            if (hit[k + q]) light_add<FAST>(L, T, n, h[q], rmin2, rcf, acc);
    }
}

// N samples at a time.  The general form (waves with a texel nearer than about
// the sampling radius, focal lengths and radii outside fast_light's) takes the
// group in the naive pass, one sample in multi-resolution launches, whose
// registers its group of 4 would take: naive pass at 1280 x 720, 64 samples,
// radius 40, 110 us with groups and 139 us without; frame at 2560 x 1440 154
// and 145 us.
template <bool FAST, int N, typename NT, typename CT, typename KP>
__device__ __forceinline__ void ssgi_texel(const SsgiArgs& a, const EvalLevel& L, const SampleTexel& T, const Normal& n,
                                           KP K, float (&acc)[3]) {
    const Planes<NT> np(static_cast<const NT*>(a.c.normal), (unsigned)a.c.plane);
    const Planes<CT> cp(static_cast<const CT*>(a.c.color), (unsigned)a.c.plane);
    const __amdgpu_buffer_rsrc_t rz = buf_rsrc(L.z, last_texel(L) + 4u);
    const float rmin = 0.1f * a.r;
    const float rmin2 = rmin * rmin;
    const float rcf = recip_fast(L.f);  // read in the fast form only
    int s = 0;
    for (; s + N <= a.S; s += N) light_group<FAST, N>(a, L, T, n, K, s, rz, np, cp, rmin2, rcf, acc);
    for (; N > 1 && s < a.S; ++s) light_group<FAST, 1>(a, L, T, n, K, s, rz, np, cp, rmin2, rcf, acc);
}

// one item (a listed texel, or a texel of a dense level)
template <typename NT, typename CT, bool AL, typename KP>
__device__ __forceinline__ void ssgi_item(const SsgiArgs& a, const ItemMap& m, unsigned item, KP K, float kmax,
                                          const float* rows) {
    const int j = item_level(m, item);
    const EvalLevel& L = a.c.lv[j];
    const unsigned local = item_local(m, item, j);
    if (local == ~0u) return;  // padding of the level's item range
    const unsigned t = L.list ? L.list[local] : local;
    if (t >= L.dense_n) return;  // malformed list entry
    const int y = (int)(t / (unsigned)L.W), x = (int)(t - (unsigned)y * (unsigned)L.W);
    // depth and normal are on their way while a_i is computed
    const float z = L.z[(unsigned)y * L.zpy + (unsigned)x * L.zpx];
    const Normal n = texel_normal(L, static_cast<const NT*>(a.c.normal), (unsigned)a.c.plane, x, y);
    if (AL && L.ac) L.ac[local] = alpha_dispatch(L, rows, j, x, y);
    float acc[3] = {0.0f, 0.0f, 0.0f};
    if (valid_depth(z)) {
        const SampleTexel T = sample_texel(L, n, a.r, x, y, z);
        if (fast_samples(T, kmax, a.r) && fast_light(L, T, a.r))
            ssgi_texel<true, kLightGroup, NT, CT>(a, L, T, n, K, acc);
        else
            ssgi_texel<false, AL ? 1 : kLightGroup, NT, CT>(a, L, T, n, K, acc);
    }
    const float scale = (a.r * a.r) / (float)a.S;
    const unsigned o = L.compact ? local : (unsigned)y * (unsigned)L.W + (unsigned)x;
#pragma unroll
    for (int c = 0; c < 3; ++c) store_out(L, (unsigned)c * (unsigned)L.out_plane + o, acc[c] * scale);
}

template <typename NT, typename CT, bool AL, typename KP>
__device__ __forceinline__ void ssgi_items(const SsgiArgs& a, KP K, float kmax, const float* rows) {
    const ItemMap m = make_item_map(a.c);
    const unsigned total = item_total(m), nchunks = (total + 255) / 256;
    const ChunkRange cr = AL ? chunk_range(nchunks) : level_chunks(nchunks);
    for (unsigned c = cr.first; c < cr.end; c += cr.step) {
        const unsigned item = c * 256u + threadIdx.x;
        if (item < total) ssgi_item<NT, CT, AL>(a, m, item, K, kmax, rows);
    }
}

// Per block: the blur's row sums (AL) and, KLDS, the samples in LDS; returns
// the largest |component| of the samples.
template <bool AL, bool KLDS>
__device__ __forceinline__ float ssgi_stage(const SsgiArgs& a, float* ks, float* rows) {
    return stage_samples<KLDS>(a.kernel, a.S, ks, [&] {
        if (AL) stage_rows(a.c, rows);
    });
}

}  // namespace mr
