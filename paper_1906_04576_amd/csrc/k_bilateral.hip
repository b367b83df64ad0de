// Bilateral blur of SSAO sub-images (Sec. 4.1) on the compact frame path.
//
// One thread per rendered texel of every blurred level, the levels' item
// ranges padded to whole waves so that a wave's level is uniform.  A tap's
// value is found from the stencil bits: its rank is the rank of its stencil
// word's first texel plus the set bits before it, so values stay stored by
// rank and the merge reads the blurred values exactly where it read the
// unblurred ones.  Taps outside the level, outside the stencil, with invalid
// depth or with a range weight that is not positive add w = +0 (times a
// finite value) to both sums, which leaves them bit-identical to sums over
// the taking-part taps alone in window order.
//
// A texel's 25 taps were bound by their 25 divisions by one tolerance and by
// the stencil words of a lane, indexed by lane and so kept in LDS: 25 us for
// half values at 2560 x 1440.  With the quotients taken from one reciprocal,
// a row's window bits shifted into place once and all loads before the sums
// it is 10.6 us, in the order of its 50 gathers per wave.
#include "eval_common.hpp"

namespace mr {
namespace {

struct BilateralMap {
    unsigned cum[kMaxLevels + 1];
    int nlev;
};

__device__ __forceinline__ BilateralMap bilateral_map(const BilateralArgs& a) {
    BilateralMap m;
    m.nlev = a.nlev;
    m.cum[0] = 0;
#pragma unroll
    for (int j = 0; j < kMaxLevels; ++j) {
        unsigned n = 0;
        if (j < a.nlev) n = a.lv[j].list ? min(a.counts[a.lv[j].count_idx], a.lv[j].dense_n) : a.lv[j].dense_n;
        m.cum[j + 1] = m.cum[j] + ((n + 63u) & ~63u);
    }
    return m;
}

// The quotient from one reciprocal is the division's for every quotient that
// can change 1 - n/d, i.e. of at least 2^-26, when d is in this range (no
// residual is lost below the smallest float; a quotient that overflows leaves
// a NaN, whose tap takes no part, as the division's does not).
constexpr float kQuotLo = 0x1p-40f, kQuotHi = 0x1p60f;

template <int R, typename VT>
__device__ __forceinline__ void bilateral_item(const BilateralArgs& a, const BilateralMap& m, unsigned item) {
    int j = 0;
    unsigned first = 0;
#pragma unroll
    for (int k = 1; k < kMaxLevels; ++k) {
        const bool past = k < m.nlev && item >= m.cum[k];
        j += past ? 1 : 0;
        first = past ? m.cum[k] : first;
    }
    j = __builtin_amdgcn_readfirstlane(j);
    const BilateralLevel& L = a.lv[j];
    const unsigned local = item - first;
    const unsigned n = L.list ? min(a.counts[L.count_idx], L.dense_n) : L.dense_n;
    if (local >= n) return;  // padding of the level's item range
    const unsigned t = L.list ? L.list[local] : local;
    if (t >= L.dense_n) return;  // malformed list entry
    const int y = (int)(t / (unsigned)L.W), x = (int)(t - (unsigned)y * (unsigned)L.W);
    const unsigned own = L.list ? local : t;
    const VT* c = static_cast<const VT*>(L.c);
    const float zp = L.z[t];
    float res = static_cast<float>(c[own]);
    if (valid_depth(zp)) {
        const float d = a.drel * zp;
        // Branch-free window, all loads issued before the sums: a tap that does
        // not take part reads past the buffers' ends, its depth 0 is invalid
        // and its weight +0.  A row's window bits start at column x - R; they
        // span at most two stencil words (R < 32), whose ranks are not
        // consecutive where the words lie in different ranking tiles.
        constexpr int N = 2 * R + 1;
        constexpr unsigned kNone = 0x3FFFFFFFu;
        const unsigned nz = (unsigned)L.W * (unsigned)L.H;
        const __amdgpu_buffer_rsrc_t rz = buf_rsrc(L.z, nz * 4u);
        const __amdgpu_buffer_rsrc_t rv = buf_rsrc(c, nz * (unsigned)sizeof(VT));
        const int x0 = x - R, wa = max(x0, 0) >> 5, wb = min(x + R, L.W - 1) >> 5;
        const int b0 = x0 - 32 * wa;   // may be negative at the left border
        const int split = 32 - b0;     // first window column of word wb, if it is another
        const unsigned below = b0 > 0 ? (1u << b0) - 1u : 0u;
        unsigned cols = (1u << N) - 1u;  // window columns inside the level
        if (x0 < 0) cols &= ~0u << -x0;
        if (x + R >= L.W) cols &= (1u << (L.W - x0)) - 1u;
        const unsigned in_a = split >= N ? (1u << N) - 1u : (1u << split) - 1u;
        unsigned lo[N], hi[N], off_a[N], off_b[N];
        if (L.list) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const unsigned r0 = (unsigned)min(max(y - R + k, 0), L.H - 1) * (unsigned)L.wpr;
                lo[k] = L.Sb[r0 + (unsigned)wa];
                hi[k] = L.Sb[r0 + (unsigned)wb];
                off_a[k] = L.woff[r0 + (unsigned)wa];
                off_b[k] = L.woff[r0 + (unsigned)wb];
            }
        }
        float zq[N][N], vq[N][N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int qy = y - R + k;
            const unsigned q0 = (unsigned)qy * (unsigned)L.W + (unsigned)x0;
            unsigned win = qy >= 0 && qy < L.H ? cols : 0u;
            unsigned ra = q0, rb = q0;  // rank of window column 0, counted from either word
            if (L.list) {
                win &= b0 >= 0 ? __builtin_amdgcn_alignbit(hi[k], lo[k], (unsigned)b0 & 31u) : lo[k] << -b0;
                ra = off_a[k] + (unsigned)__popc(lo[k] & below);
                rb = off_b[k] - (unsigned)__popc(win & in_a);
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const bool ok = (win >> j) & 1u;
                const unsigned r = L.list ? (j < split ? ra : rb) + (unsigned)__popc(win & ((1u << j) - 1u))
                                          : q0 + (unsigned)j;
                zq[k][j] = buf_f1(rz, (ok ? q0 + (unsigned)j : kNone) * 4u);
                const unsigned e = ok ? r : kNone;
                if constexpr (sizeof(VT) == 4)
                    vq[k][j] = buf_f1(rv, e * 4u);
                else
                    vq[k][j] = (float)__builtin_bit_cast(_Float16,
                                                         __builtin_amdgcn_raw_buffer_load_b16(rv, (int)(e * 2u), 0, 0));
            }
        }
        float num = 0.0f, den = 0.0f;
        const float rc = recip_fast(d);
        auto sums = [&](auto div) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const float wz = 1.0f - div(fabsf(zq[k][j] - zp));
                    const bool ok = valid_depth(zq[k][j]) && wz > 0.0f;
                    const float w = ok ? (a.wb[k] * a.wb[j]) * wz : 0.0f;
                    num = num + w * vq[k][j];
                    den = den + w;
                }
            }
        };
        if (__builtin_expect(__ballot(!(d >= kQuotLo && d <= kQuotHi)) != 0, 0))
            sums([&](float n) { return n / d; });
        else
            sums([&](float n) { return quotient(n, d, rc); });
        res = num / den;
    }
    static_cast<VT*>(L.out)[own] = static_cast<VT>(res);
}

template <int R, typename VT>
__global__ __launch_bounds__(256) void k_bilateral(BilateralArgs a) {
    const BilateralMap m = bilateral_map(a);
    const ChunkRange cr = chunk_range((m.cum[kMaxLevels] + 255u) / 256u);
    for (unsigned ch = cr.first; ch < cr.end; ch += cr.step) {
        const unsigned item = ch * 256u + threadIdx.x;
        if (item < m.cum[kMaxLevels]) bilateral_item<R, VT>(a, m, item);
    }
}

}  // namespace

hipError_t launch_bilateral(const BilateralArgs& a, unsigned total_hint, hipStream_t s) {
#define MR_BL(R, VT) \
    hipLaunchKernelGGL((k_bilateral<R, VT>), dim3(eval_blocks<k_bilateral<R, VT>>(total_hint)), dim3(256), 0, s, a)
    if (a.R == 1) {
        if (a.c16) MR_BL(1, _Float16);
        else MR_BL(1, float);
    } else {
        if (a.c16) MR_BL(2, _Float16);
        else MR_BL(2, float);
    }
#undef MR_BL
    return hipGetLastError();
}

}  // namespace mr
