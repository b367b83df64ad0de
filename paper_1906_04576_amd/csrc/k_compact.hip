// Work-list compaction: the stencil test of Sec. 4.1 turned into per-level
// lists of the texels to evaluate, in row-major ascending order, with the
// list lengths left on the device.
//
// Two launches over the stencils of all compacted levels at once (a level's
// stencil is cut into runs of `chunks` chunks of 4096 texels, 16 per thread):
//   count   - nonzero bytes per run (popcount of a byte mask, block sum);
//             further blocks of the same launch write the owner-level map,
//             which reads the same stencils;
//   scatter - each run's block sums the counts of its level's earlier runs,
//             256 threads wide, and then chunk by chunk recounts, takes a
//             wave64 prefix sum of the per-thread counts plus the wave totals
//             from LDS, and writes its indices; a level's last run writes its
//             total.
// (The map, the count, a scan by one workgroup and the scatter were four
// launches of 4 to 5 us each on a 1366 x 768 frame, most of it the launch.)
// A run is one chunk up to kCompactRuns chunks in the finest level, then as
// many as keep to that number: the sums over earlier runs grow with its
// square.  (16384 x 16384, 65536 chunks: scatter 766 us with a run for each
// chunk, 281 us in runs of 16; 1024 to 8192 runs within 3 % of each other.)
#include "mr_internal.hpp"

namespace mr {

// number of nonzero bytes of a 32-bit word
__device__ __forceinline__ unsigned nz_bytes(unsigned w) {
    return __popc((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u);
}

__device__ __forceinline__ int find_level(const CompactArgs& a, unsigned c) {
    int l = 0;
    while (l + 1 < a.nlev && c >= a.run_base[l + 1]) ++l;
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

// 16 stencil bytes of the thread in chunk k of run c of level l, and where they
// start
struct Piece {
    uint4 v;
    unsigned off, cnt;
};

__device__ __forceinline__ Piece load_piece(const CompactArgs& a, int l, unsigned c, unsigned chunks, unsigned k) {
    Piece p{make_uint4(0, 0, 0, 0), ((c - a.run_base[l]) * chunks + k) * kChunk + threadIdx.x * 16, 0u};
    if (p.off < a.n[l]) {
        p.v = load16(a.S[l], a.n[l], p.off);
        p.cnt = nz_bytes(p.v.x) + nz_bytes(p.v.y) + nz_bytes(p.v.z) + nz_bytes(p.v.w);
    }
    return p;
}

template <bool ONE>
__device__ __forceinline__ void count_run(const CompactArgs& a, unsigned c, unsigned* wsum) {
    const unsigned chunks = ONE ? 1u : a.chunks;
    const int l = find_level(a, c);
    unsigned cnt = 0;
    for (unsigned k = 0; k < chunks; ++k) cnt += load_piece(a, l, c, chunks, k).cnt;
    // wave reduction
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
    if (__lane_id() == 0) wsum[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) a.run_count[c] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
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

// blocks 0 .. nruns - 1 count, the others write the level map.  ONE: runs of one
// chunk, without the loops (3840 x 2160: count 4.9 and 5.1 us, scatter 7.7 and
// 8.3 us).
template <bool ONE>
__global__ __launch_bounds__(256) void k_count_map(CompactArgs a, LevelMapArgs m, unsigned nruns) {
    __shared__ unsigned wsum[4];
    if (blockIdx.x < nruns)
        count_run<ONE>(a, blockIdx.x, wsum);
    else
        map_chunk(m, blockIdx.x - nruns);
}

template <bool ONE>
__global__ __launch_bounds__(256) void k_scatter(CompactArgs a, unsigned nruns) {
    __shared__ unsigned wtot[2][4], wpre[4];
    const unsigned c = blockIdx.x;
    if (c == 0 && threadIdx.x < kMaxLevels) {  // levels that are not compacted report 0
        bool listed = false;
        for (int l = 0; l < a.nlev; ++l) listed = listed || a.count_idx[l] == (int)threadIdx.x;
        if (!listed) a.count[threadIdx.x] = 0;
    }
    if (c >= nruns) return;
    const int l = find_level(a, c);
    unsigned pre = 0;  // entries of the level's earlier runs
    for (unsigned u = a.run_base[l] + threadIdx.x; u < c; u += 256) pre += a.run_count[u];
    for (int d = 32; d >= 1; d >>= 1) pre += __shfl_xor(pre, d, 64);
    const int wv = threadIdx.x >> 6;
    if (__lane_id() == 63) wpre[wv] = pre;
    const unsigned chunks = ONE ? 1u : a.chunks;
    uint32_t* list = a.list[l];
    unsigned done = 0;  // entries of the run's earlier chunks
    for (unsigned k = 0; k < chunks; ++k) {
        const Piece p = load_piece(a, l, c, chunks, k);
        const unsigned inc = wave_incl_scan(p.cnt);
        unsigned* tot = wtot[k & 1u];  // two sets: one barrier per chunk
        if (__lane_id() == 63) tot[wv] = inc;
        __syncthreads();
        if (k == 0) done = wpre[0] + wpre[1] + wpre[2] + wpre[3];
        unsigned pos = done + inc - p.cnt;
        for (int w = 0; w < wv; ++w) pos += tot[w];
        done += tot[0] + tot[1] + tot[2] + tot[3];
        if (!p.cnt) continue;
        const unsigned words[4] = {p.v.x, p.v.y, p.v.z, p.v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned w = words[q];
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if ((w >> (8 * b)) & 0xFFu) list[pos++] = p.off + 4 * q + b;
        }
    }
    if (threadIdx.x == 0 && c + 1u == a.run_base[l + 1]) a.count[a.count_idx[l]] = done;
}

hipError_t launch_compact(const CompactArgs& a, const LevelMapArgs* map, hipStream_t s) {
    const unsigned nruns = a.run_base[a.nlev];
    unsigned maps = 0;
    if (map) maps = ((unsigned)map->W * (unsigned)map->H + kMapPixels - 1u) / kMapPixels;
    const LevelMapArgs m = map ? *map : LevelMapArgs{};
    const dim3 count(nruns + maps), scatter(nruns ? nruns : 1u), threads(256);
    if (a.chunks == 1u) {
        if (nruns + maps) hipLaunchKernelGGL(k_count_map<true>, count, threads, 0, s, a, m, nruns);
        hipLaunchKernelGGL(k_scatter<true>, scatter, threads, 0, s, a, nruns);
    } else {
        if (nruns + maps) hipLaunchKernelGGL(k_count_map<false>, count, threads, 0, s, a, m, nruns);
        hipLaunchKernelGGL(k_scatter<false>, scatter, threads, 0, s, a, nruns);
    }
    return hipGetLastError();
}

}  // namespace mr
