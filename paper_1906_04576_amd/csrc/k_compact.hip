// Work-list compaction: the stencil test of Sec. 4.1 turned into per-level
// lists of the texels to evaluate, in row-major ascending order, with the
// list lengths left on the device.
//
// Two launches over the stencils of all compacted levels at once (a level's
// stencil is cut into chunks of 4096 texels, 16 per thread):
//   count   - nonzero bytes per chunk (popcount of a byte mask, block sum);
//             further blocks of the same launch write the owner-level map,
//             which reads the same stencils;
//   scatter - each chunk sums the counts of its level's earlier chunks (at
//             most 65536 of them, 256 threads wide), recounts, takes a wave64
//             prefix sum of the per-thread counts plus the wave totals from
//             LDS, and writes its indices; a level's last chunk writes its
//             total.
// (The map, the count, a scan by one workgroup and the scatter were four
// launches of 4 to 5 us each on a 1366 x 768 frame, most of it the launch.)
#include "mr_internal.hpp"

namespace mr {

// number of nonzero bytes of a 32-bit word
__device__ __forceinline__ unsigned nz_bytes(unsigned w) {
    return __popc((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u);
}

__device__ __forceinline__ int find_level(const CompactArgs& a, unsigned c) {
    int l = 0;
    while (l + 1 < a.nlev && c >= a.chunk_base[l + 1]) ++l;
    return l;
}

// 16 stencil bytes of one thread (bytes past the end read as 0)
__device__ __forceinline__ uint4 load16(const uint8_t* S, unsigned n, unsigned off) {
    if (off + 16 <= n) return *reinterpret_cast<const uint4*>(S + off);
    unsigned w[4] = {0, 0, 0, 0};
    for (unsigned b = 0; b < 16 && off + b < n; ++b) w[b >> 2] |= (unsigned)S[off + b] << (8 * (b & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        unsigned o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

__device__ __forceinline__ void count_chunk(const CompactArgs& a, unsigned c, unsigned* wsum) {
    const int l = find_level(a, c);
    const unsigned off = (c - a.chunk_base[l]) * kChunk + threadIdx.x * 16;
    unsigned cnt = 0;
    if (off < a.n[l]) {
        const uint4 v = load16(a.S[l], a.n[l], off);
        cnt = nz_bytes(v.x) + nz_bytes(v.y) + nz_bytes(v.z) + nz_bytes(v.w);
    }
    // wave reduction
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
    if (__lane_id() == 0) wsum[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) a.chunk_count[c] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// owner-level map: the finest enabled level whose stencil covers the pixel;
// a block writes kMapPixels consecutive pixels
constexpr unsigned kMapPixels = 1024;
__device__ __forceinline__ void map_chunk(const LevelMapArgs& a, unsigned c) {
    const unsigned n = (unsigned)a.W * (unsigned)a.H;
#pragma unroll
    for (int q = 0; q < (int)(kMapPixels / 256u); ++q) {
        const unsigned p = c * kMapPixels + 256u * q + threadIdx.x;
        if (p >= n) return;
        const unsigned y = p / (unsigned)a.W, x = p - y * (unsigned)a.W;
        unsigned lvl = (unsigned)a.levels[a.nlev - 1];
        for (int j = a.nlev - 2; j >= 0; --j) {
            const int i = a.levels[j], sh = i - 1;
            if (a.S[j][(y >> sh) * (unsigned)a.Wi[j] + (x >> sh)]) lvl = (unsigned)i;
        }
        a.out[p] = (uint8_t)lvl;
    }
}

// blocks 0 .. nchunks - 1 count, the others write the level map
__global__ __launch_bounds__(256) void k_count_map(CompactArgs a, LevelMapArgs m, unsigned nchunks) {
    __shared__ unsigned wsum[4];
    if (blockIdx.x < nchunks)
        count_chunk(a, blockIdx.x, wsum);
    else
        map_chunk(m, blockIdx.x - nchunks);
}

__global__ __launch_bounds__(256) void k_scatter(CompactArgs a, unsigned nchunks) {
    __shared__ unsigned wtot[4], wpre[4];
    const unsigned c = blockIdx.x;
    if (c == 0 && threadIdx.x < kMaxLevels) {  // levels that are not compacted report 0
        bool listed = false;
        for (int l = 0; l < a.nlev; ++l) listed = listed || a.count_idx[l] == (int)threadIdx.x;
        if (!listed) a.count[threadIdx.x] = 0;
    }
    if (c >= nchunks) return;
    const int l = find_level(a, c);
    unsigned pre = 0;  // entries of the level's earlier chunks
    for (unsigned u = a.chunk_base[l] + threadIdx.x; u < c; u += 256) pre += a.chunk_count[u];
    for (int d = 32; d >= 1; d >>= 1) pre += __shfl_xor(pre, d, 64);
    const unsigned base = (c - a.chunk_base[l]) * kChunk;
    const unsigned off = base + threadIdx.x * 16;
    uint4 v = make_uint4(0, 0, 0, 0);
    unsigned cnt = 0;
    if (off < a.n[l]) {
        v = load16(a.S[l], a.n[l], off);
        cnt = nz_bytes(v.x) + nz_bytes(v.y) + nz_bytes(v.z) + nz_bytes(v.w);
    }
    const unsigned inc = wave_incl_scan(cnt);
    const int wv = threadIdx.x >> 6;
    if (__lane_id() == 63) {
        wtot[wv] = inc;
        wpre[wv] = pre;
    }
    __syncthreads();
    unsigned before = wpre[0] + wpre[1] + wpre[2] + wpre[3];
    if (threadIdx.x == 0 && c + 1u == a.chunk_base[l + 1])
        a.count[a.count_idx[l]] = before + wtot[0] + wtot[1] + wtot[2] + wtot[3];
    for (int w = 0; w < wv; ++w) before += wtot[w];
    unsigned pos = before + inc - cnt;
    if (!cnt) return;
    uint32_t* list = a.list[l];
    const unsigned words[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned w = words[q];
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if ((w >> (8 * b)) & 0xFFu) list[pos++] = off + 4 * q + b;
    }
}

hipError_t launch_compact(const CompactArgs& a, const LevelMapArgs* map, hipStream_t s) {
    const unsigned nchunks = a.chunk_base[a.nlev];
    unsigned maps = 0;
    if (map) maps = ((unsigned)map->W * (unsigned)map->H + kMapPixels - 1u) / kMapPixels;
    if (nchunks + maps)
        hipLaunchKernelGGL(k_count_map, dim3(nchunks + maps), dim3(256), 0, s, a, map ? *map : LevelMapArgs{}, nchunks);
    hipLaunchKernelGGL(k_scatter, dim3(nchunks ? nchunks : 1u), dim3(256), 0, s, a, nchunks);
    return hipGetLastError();
}

}  // namespace mr
