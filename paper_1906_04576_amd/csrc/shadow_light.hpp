// Light coordinates of a view-space point and the one-sample shadow test
// (Sec. 3.1): P_l = M P (3 x 4 affine, rows summed left to right),
// d_r = -P_l.z, su = c_L + (P_l.x / d_r) f_L, sv = c_L - (P_l.y / d_r) f_L,
// c_L = size / 2.  Outside the light frustum = lit.
#pragma once
#include "eval_common.hpp"

namespace mr {

struct LightCoord {
    float dr, su, sv;
    bool inside;
};

__device__ __forceinline__ LightCoord to_light(const float* M, int size, float fL, float px,
                                               float py, float pz) {
    const float lx = ((M[0] * px + M[1] * py) + M[2] * pz) + M[3];
    const float ly = ((M[4] * px + M[5] * py) + M[6] * pz) + M[7];
    const float lz = ((M[8] * px + M[9] * py) + M[10] * pz) + M[11];
    LightCoord c;
    const float cL = 0.5f * (float)size;
    c.dr = -lz;
    const float inv = recip_pos(c.dr);  // = 1.0f / d_r (d_r > 0)
    c.su = cL + (lx * inv) * fL;
    c.sv = cL - (ly * inv) * fL;
    const float sz = (float)size;
    c.inside = c.dr > 0.0f && c.su >= 0.0f && c.su < sz && c.sv >= 0.0f && c.sv < sz;
    return c;
}

// One-sample shadow bits of N pixels at view positions (X[k] z[k], Y z[k],
// -z[k]), as bytes of one word; the gathers are in flight together.
template <int N>
__device__ __forceinline__ unsigned hard_bits(const HardArgs& a, __amdgpu_buffer_rsrc_t map, const float (&X)[N], float Y,
                                              const float (&z)[N]) {
    float s[N], thr[N];
    bool inside[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const LightCoord c = to_light(a.M, a.size, a.fL, X[k] * z[k], Y * z[k], -z[k]);
        inside[k] = c.inside & valid_depth(z[k]);
        thr[k] = c.dr - a.bias;
        // inside the map, where truncation is floor; else texel (0, 0)
        const unsigned x = (unsigned)(int)(inside[k] ? c.su : 0.0f), y = (unsigned)(int)(inside[k] ? c.sv : 0.0f);
        s[k] = buf_f1(map, (__umul24(y, (unsigned)a.size) + x) * 4u);
    }
    unsigned h = 0u;
#pragma unroll
    for (int k = 0; k < N; ++k) h |= (inside[k] & (s[k] < thr[k])) ? 1u << (8 * k) : 0u;
    return h;
}

}  // namespace mr
