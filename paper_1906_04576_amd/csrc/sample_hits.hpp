// The samples of SSAO and SSGI (Sec. 2.4 reading): a texel's sample points,
// the texels they project to, and which of them occlude.
#pragma once
#include "eval_common.hpp"

namespace mr {

// A texel: its view position, depth and scaled tangent frame.
struct SampleTexel {
    float px, py, pz, z;
    float rtx, rty, rtz, rbx, rby, rbz, rnx, rny, rnz;
};

struct Normal {
    float x, y, z;
};

template <typename NT>
__device__ __forceinline__ Normal texel_normal(const EvalLevel& L, const NT* nrm, unsigned plane, int x, int y) {
    const unsigned g = (unsigned)L.goff + (unsigned)y * (unsigned)L.gpy + (unsigned)x * (unsigned)L.gpx;
    return {ld(nrm, g), ld(nrm, plane + g), ld(nrm, 2 * plane + g)};
}

__device__ __forceinline__ SampleTexel sample_texel(const EvalLevel& L, const Normal& n, float r, int x, int y,
                                                    float z) {
    float px, py, pz;
    view_pos(x, y, z, L.f, L.cx, L.cy, px, py, pz);
    float tx, ty, tz, bx, by, bz;
    onb(n.x, n.y, n.z, tx, ty, tz, bx, by, bz);
    return {px, py, pz, z, r * tx, r * ty, r * tz, r * bx, r * by, r * bz, r * n.x, r * n.y, r * n.z};
}

// Whether the fast forms below hold for every sample of the wave's texels;
// kmax = the largest |component| over the samples.
// Every sample's d = z - (kx rtz + ky rbz + kz rnz) (rounded) lies within
// Bz = kmax (|rtz| + |rbz| + |rnz|) of z, up to a relative 2^-21; with these
// margins all d are in [2^-126, 2^126), where recip_fast is exact.  Sample
// points are finite, and z >= r.  NaN fails every comparison.
__device__ __forceinline__ bool fast_samples(const SampleTexel& T, float kmax, float r) {
    const float Bx = kmax * ((fabsf(T.rtx) + fabsf(T.rbx)) + fabsf(T.rnx));
    const float By = kmax * ((fabsf(T.rty) + fabsf(T.rby)) + fabsf(T.rny));
    const float Bz = kmax * ((fabsf(T.rtz) + fabsf(T.rbz)) + fabsf(T.rnz));
    const bool safe = (T.z * 0.999f > Bz * 1.001f + 1e-37f) & ((T.z + Bz) * 1.001f < 0x1p125f) & (T.z >= r) &
                      (fabsf(T.px) + Bx < 0x1p120f) & (fabsf(T.py) + By < 0x1p120f);
    return __ballot(!safe) == 0;
}

// samples whose gathers are in flight together
constexpr int kGroup = 8;

// A vector instruction takes about 4 cycles of a SIMD here, and an FP32 add or
// multiply or a 32-bit integer add or logic operation 2 (measured streams;
// the two kinds overlap), so the fast form's tests are sign bits that adds
// and logic operations combine, in place of compares and selects: 37 of its
// 45 instructions per sample are of the cheap kind (29 of 45 with compares).
//
// Fast form (fast_samples): off is the byte offset of the sample's texel; off
// screen its sign bit is set, which lies past the plane's end, where a load
// returns 0 without an access, and z - 0 >= r fails the range test.
template <typename KP>
__device__ __forceinline__ void project_fast(const EvalLevel& L, KP K, int s, const SampleTexel& T, float& d,
                                             unsigned& off, int& x, int& y) {
    const float kx = K[3 * s], ky = K[3 * s + 1], kz = K[3 * s + 2];
    d = -(((T.pz + kx * T.rtz) + ky * T.rbz) + kz * T.rnz);
    const float qx = ((T.px + kx * T.rtx) + ky * T.rbx) + kz * T.rnx;
    const float qy = ((T.py + kx * T.rty) + ky * T.rby) + kz * T.rny;
    const float inv = recip_fast(d);
    x = floor_i32(L.cx + (qx * inv) * L.f);
    y = floor_i32(L.cy - (qy * inv) * L.f);
    // rows < 2^14 and byte pitches < 2^22 keep the products within 24 bits
    const unsigned ux = (unsigned)x, uy = (unsigned)y;
    const unsigned out = ((((unsigned)L.W - 1u) - ux) | ux) | ((((unsigned)L.H - 1u) - uy) | uy);
    off = ((unsigned)__umul24(uy, 4u * (unsigned)L.zpy) + (unsigned)__umul24(ux, 4u * (unsigned)L.zpx)) |
          (out & 0x80000000u);
}

// Any sample: the bounds by compares, 1/d by recip_pos (RCP) or the division.
// off: the offset of the sample's texel, of texel (0, 0) when it is off screen.
// (RCP pays in SSGI's launches; in SSAO's it takes registers that the fast form
// needs more: batch of three with radius 8 122 us, 120 us with the division.)
template <bool RCP, typename KP>
__device__ __forceinline__ void project_any(const EvalLevel& L, KP K, int s, const SampleTexel& T, bool& on, float& d,
                                            unsigned& off, int& x, int& y) {
    const float Wf = (float)L.W, Hf = (float)L.H;
    const float kx = K[3 * s], ky = K[3 * s + 1], kz = K[3 * s + 2];
    const float qz = ((T.pz + kx * T.rtz) + ky * T.rbz) + kz * T.rnz;
    d = -qz;
    const float qx = ((T.px + kx * T.rtx) + ky * T.rbx) + kz * T.rnx;
    const float qy = ((T.py + kx * T.rty) + ky * T.rby) + kz * T.rny;
    const float inv = RCP ? recip_pos(d) : 1.0f / d;  // the same where d > 0, else unused
    const float u = L.cx + (qx * inv) * L.f;
    const float v = L.cy - (qy * inv) * L.f;
    on = (d > 0.0f) & (u >= 0.0f) & (u < Wf) & (v >= 0.0f) & (v < Hf);
    x = (int)(on ? u : 0.0f);  // u, v >= 0 when on, so truncation is floor
    y = (int)(on ? v : 0.0f);
    off = (unsigned)__umul24((unsigned)y, 4u * (unsigned)L.zpy) + (unsigned)__umul24((unsigned)x, 4u * (unsigned)L.zpx);
}

// Sign set iff a sample of the fast form occludes: z_s < d - b d, and
// |z - z_s| < r on the bit patterns (false for infinities and NaN).
__device__ __forceinline__ unsigned occludes_fast(float z, float d, float zs, float r, float b) {
    const float e = zs - (d - (b * d));
    const unsigned in = (__float_as_uint(z - zs) & 0x7FFFFFFFu) - __float_as_uint(r);  // r > 0
    return __float_as_uint(e) & in;
}

// z_s <= 0 must not count; +inf and NaN fail the depth test
__device__ __forceinline__ bool occludes_any(bool on, float z, float d, float zs, float r, float b) {
    return on & (zs > 0.0f) & (zs < d - (b * d)) & (fabsf(z - zs) < r);
}

// byte offset of the last texel of a level's depth view
__device__ __forceinline__ unsigned last_texel(const EvalLevel& L) {
    return ((unsigned)(L.H - 1) * (unsigned)L.zpy + (unsigned)(L.W - 1) * (unsigned)L.zpx) * 4u;
}

// depths of N samples and what their gathers bring
template <int N>
struct SampleGroup {
    float d[N], zs[N];
};

// a level's depth view as a buffer resource (L is wave-uniform here)
struct PlaneGather {
    __amdgpu_buffer_rsrc_t rz;
    __device__ __forceinline__ float operator()(unsigned off, int, int) const { return buf_f1(rz, off); }
};

// the projections and gathers of N samples from s
template <int N, typename KP, typename GF>
__device__ __forceinline__ void issue_samples(const EvalLevel& L, KP K, int s, const SampleTexel& T, const GF& gather,
                                              SampleGroup<N>& g) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        unsigned off;
        int x, y;
        project_fast(L, K, s + k, T, g.d[k], off, x, y);
        g.zs[k] = gather(off, x, y);
        // one projection at a time: interleaving them buys little and costs
        // registers (occupancy)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// hits << N | one bit per sample of the group, the first one on top
template <int N>
__device__ __forceinline__ unsigned test_samples(const SampleTexel& T, const SampleGroup<N>& g, float r, float b,
                                                 unsigned hits) {
#pragma unroll
    for (int k = 0; k < N; ++k)
        hits = __builtin_amdgcn_alignbit(hits, occludes_fast(T.z, g.d[k], g.zs[k], r, b), 31);
    __builtin_amdgcn_sched_barrier(0);
    return hits;
}

// Per block: the S samples in LDS (KLDS: at most kLdsSamples), and the largest
// |component| of them; ends with its one barrier.  (Without the maximum of a
// set that is not staged, all its waves took the general form: 1025 samples,
// SSGI frame at 1280 x 720 786 us, now 610 us; naive SSAO pass 1031 and 924 us.)
// meanwhile() runs while the samples are on their way.  (With a barrier
// before the loads and the row sums ahead of them the naive pass at 4K, a
// block of which stages for 256 texels, took 238 us, now 233 us.)
template <bool KLDS, typename F>
__device__ __forceinline__ float stage_samples(const float* kernel, int S, float* ks, F meanwhile) {
    __shared__ unsigned wmax[4];  // per wave, as bits: all values >= 0
    const int t = (int)threadIdx.x, n = 3 * S;
    const float v = t < n ? kernel[t] : 0.0f;
    meanwhile();
    unsigned m = __float_as_uint(fabsf(v));
    if (KLDS && t < n) ks[t] = v;
    for (int i = t + 256; i < n; i += 256) {
        const float u = kernel[i];
        if (KLDS) ks[i] = u;
        m = max(m, __float_as_uint(fabsf(u)));
    }
    for (int o = 32; o >= 1; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o, 64));
    if (__lane_id() == 0) wmax[t >> 6] = m;
    __syncthreads();
    return __uint_as_float(max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3])));
}

}  // namespace mr
