// Stable compaction of the particle slots: the live particles of every
// segment that has holes move, in their order, to the front of the other
// copy, and the copies swap.  Run every few steps (the push leaves holes where
// particles were absorbed).
//
// Tiles of 1024 slots (256 threads, 4 slots each), numbered over
// the segments that have holes.  Four plain passes (three in contexts of few
// tiles), no waiting between workgroups (the two tile passes run on persistent
// grids):
//   count:   live particles of every tile
//   scan:    per segment, exclusive scan of its tiles' counts (first slot of
//            every tile), checked against the segment's live count (contexts
//            of few tiles: part of the scatter)
//   scatter: every live particle written to its tile's first slot + its rank
//            in the tile (four groups of 256 neighbouring slots, all in flight)
//   finish:  copies swap, count = live
#include "pic_device.h"
#include "pic_internal.h"
#include "pic_kernels.h"

#include <algorithm>

namespace pic {

namespace {

constexpr int kCT = 256;              // threads per compaction tile
constexpr int kCP = 4;                // slots per thread
constexpr int kCTile = kCT * kCP;

__device__ __forceinline__ bool has_holes(const DevPtrs& d, int g)
{
    return !d.diss[g / d.S].retired && d.segs[g].count != d.segs[g].live;
}

// first tile of every segment with holes (16 segments per lane at most), in LDS
__device__ __forceinline__ void hole_prefix(const DevPtrs& d, int32_t* pref)
{
    const int NS = d.B * d.S, lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        const int per = (NS + 63) >> 6, g0 = lane * per;
        int32_t run = 0;
        for (int j = 0; j < per; ++j) {
            const int g = g0 + j;
            if (g < NS) {
                if (has_holes(d, g)) run += (int32_t)((d.segs[g].count + kCTile - 1) / kCTile);
                pref[g + 1] = run;
            }
        }
        int32_t incl = run;
#pragma unroll
        for (int dd = 1; dd < 64; dd <<= 1) {
            const int32_t o = __shfl_up(incl, dd, 64);
            if (lane >= dd) incl += o;
        }
        const int32_t excl = incl - run;
        if (lane == 0) pref[0] = 0;
        for (int j = 0; j < per; ++j) {
            const int g = g0 + j;
            if (g < NS) pref[g + 1] += excl;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ int seg_of_tile(const int32_t* pref, int NS, int32_t t)
{
    int lo = 0, hi = NS;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pref[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// live flags of this thread's slots
__device__ __forceinline__ uint32_t live_mask(const PIC_GLOBAL int32_t* cell, int64_t base, int64_t n)
{
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < kCP; ++j)
        if (base + j < n && cell[base + j] >= 0) m |= 1u << j;
    return m;
}

// exclusive scan over the workgroup of v; total in *tot
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t* s_w, uint32_t* tot)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan_u32(v);
    if (lane == 63) s_w[wid] = incl;
    __syncthreads();
    uint32_t wex = 0, t = 0;
#pragma unroll
    for (int w = 0; w < kCT / 64; ++w) {
        if (w < wid) wex += s_w[w];
        t += s_w[w];
    }
    *tot = t;
    return wex + incl - v;
}

__global__ __launch_bounds__(kCT) void compact_count_kernel(DevPtrs d)
{
    __shared__ int32_t pref[kMaxSeg + 1];
    __shared__ uint32_t s_w[kCT / 64];
    hole_prefix(d, pref);
    const int NS = d.B * d.S;
    for (int32_t t = (int32_t)blockIdx.x; t < pref[NS]; t += (int32_t)gridDim.x) {
        const int g = __builtin_amdgcn_readfirstlane(seg_of_tile(pref, NS, t));
        const PIC_CONST SegState& st = const_state(d, g);
        const int64_t base = (int64_t)(t - pref[g]) * kCTile + (int64_t)threadIdx.x * kCP;
        const uint32_t m =
            live_mask((const PIC_GLOBAL int32_t*)const_seg(d, g).cell[st.parity], base, st.count);
        uint32_t tot;
        (void)block_excl((uint32_t)__popc(m), s_w, &tot);
        if (threadIdx.x == 0) d.ccnt[t] = tot;
        __syncthreads();                           // s_w is reused
    }
}

__global__ __launch_bounds__(1024) void compact_scan_kernel(DevPtrs d)
{
    __shared__ int32_t pref[kMaxSeg + 1];
    __shared__ uint32_t s_w[16];
    hole_prefix(d, pref);
    const int g = blockIdx.x;
    if (g >= d.B * d.S || !has_holes(d, g)) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t t0 = pref[g], nt = pref[g + 1] - pref[g];
    uint32_t run = 0;
    for (int32_t r0 = 0; r0 < nt; r0 += 1024) {
        const int32_t i = r0 + (int32_t)threadIdx.x;
        const uint32_t v = i < nt ? d.ccnt[t0 + i] : 0u;
        const uint32_t incl = wave_incl_scan_u32(v);
        if (lane == 63) s_w[wid] = incl;
        __syncthreads();
        uint32_t wex = 0, tot = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wid) wex += s_w[w];
            tot += s_w[w];
        }
        if (i < nt) d.ccnt[t0 + i] = run + wex + incl - v;
        run += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && (int64_t)run != d.segs[g].live) atomicOr(&d.diss[g / d.S].flags, kFlagCell);
}

// A tile's slots, four per thread, are read together, their ranks come from one
// barrier, and all the live particles' arrays are in flight at once: a small
// compaction is a chain of these latencies (four rounds of them, one after the
// other, took 13 us for one discharge of 4e5 particles), a large one wants the
// bytes in flight.  Per step, compaction every 16 or 32 steps, before and now: 64
// discharges of 4.9e7 particles 450 and 443 us, of 1.77e7 sampled 262 and 256;
// one of 4e5 20.5 and 20.3, sampled 31.2 and 30.9.  SCANNED: the scan kernel has
// turned the counts into first slots; otherwise the workgroup adds up the counts of the tiles before its own.
template <bool SCANNED>
__global__ __launch_bounds__(kCT) void compact_scatter_kernel(DevPtrs d)
{
    constexpr int kW = kCT / 64;
    __shared__ int32_t pref[kMaxSeg + 1];
    __shared__ uint32_t s_w[kCP][kW], s_p[kW];
    hole_prefix(d, pref);
    const int NS = d.B * d.S, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    for (int32_t t = (int32_t)blockIdx.x; t < pref[NS]; t += (int32_t)gridDim.x) {
        const int g = __builtin_amdgcn_readfirstlane(seg_of_tile(pref, NS, t));
        CSeg& sc = const_seg(d, g);
        const PIC_CONST SegState& st = const_state(d, g);
        const int in = st.parity, out = in ^ 1;
        const int64_t count = st.count, live_n = st.live;
        const int32_t t0 = pref[g];
        const int64_t base = (int64_t)(t - t0) * kCTile;
        const PIC_GLOBAL int32_t* cell = (const PIC_GLOBAL int32_t*)sc.cell[in];
        // groups of 256 consecutive slots: lanes read and write neighbours
        int32_t c[kCP];
#pragma unroll
        for (int r = 0; r < kCP; ++r) {
            const int64_t i = base + r * kCT + tid;
            c[r] = i < count ? cell[i] : -1;
        }
        uint32_t before = 0;                       // live particles of the tiles before
        if (SCANNED) {
            before = d.ccnt[t];
        } else {
            for (int32_t k = t0 + tid; k < t; k += kCT) before += d.ccnt[k];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) before += (uint32_t)__shfl_xor((int)before, m, 64);
            if (lane == 0) s_p[wid] = before;
        }
        uint64_t m[kCP];
#pragma unroll
        for (int r = 0; r < kCP; ++r) {
            m[r] = __ballot(c[r] >= 0);
            if (lane == 0) s_w[r][wid] = (uint32_t)__popcll(m[r]);
        }
        __syncthreads();
        int64_t first = before;
        if (!SCANNED) {
            first = 0;
#pragma unroll
            for (int w = 0; w < kW; ++w) first += s_p[w];
        }
        int64_t dst[kCP];
        bool bad = false;
#pragma unroll
        for (int r = 0; r < kCP; ++r) {
            uint32_t wex = 0, tot = 0;
#pragma unroll
            for (int w = 0; w < kW; ++w) {
                if (w < wid) wex += s_w[r][w];
                tot += s_w[r][w];
            }
            dst[r] = first + wex +
                     __builtin_amdgcn_mbcnt_hi((uint32_t)(m[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[r], 0u));
            first += tot;
            bad |= c[r] >= 0 && dst[r] >= live_n;   // cannot happen when the counts agree
            if (dst[r] >= live_n) c[r] = -1;
        }
        if (!SCANNED) bad |= t + 1 == pref[g + 1] && first != live_n;
        if (bad) atomicOr(&d.diss[g / d.S].flags, kFlagCell);
        uint32_t v[5][kCP];
        const PIC_GLOBAL uint32_t* from[5] = {
            (const PIC_GLOBAL uint32_t*)sc.off[in], (const PIC_GLOBAL uint32_t*)sc.vx[in],
            (const PIC_GLOBAL uint32_t*)sc.vy[in], (const PIC_GLOBAL uint32_t*)sc.vz[in],
            (const PIC_GLOBAL uint32_t*)sc.id[in]};
        PIC_GLOBAL uint32_t* to[5] = {(PIC_GLOBAL uint32_t*)sc.off[out], (PIC_GLOBAL uint32_t*)sc.vx[out],
                                      (PIC_GLOBAL uint32_t*)sc.vy[out], (PIC_GLOBAL uint32_t*)sc.vz[out],
                                      (PIC_GLOBAL uint32_t*)sc.id[out]};
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
            for (int r = 0; r < kCP; ++r) v[k][r] = c[r] >= 0 ? from[k][base + r * kCT + tid] : 0u;
        PIC_GLOBAL int32_t* cell_to = (PIC_GLOBAL int32_t*)sc.cell[out];
#pragma unroll
        for (int r = 0; r < kCP; ++r) {
            if (c[r] < 0) continue;
            cell_to[dst[r]] = c[r];
#pragma unroll
            for (int k = 0; k < 5; ++k) to[k][dst[r]] = v[k][r];
            if (sc.z[0])
                ((PIC_GLOBAL double*)sc.z[out])[dst[r]] = ((const PIC_GLOBAL double*)sc.z[in])[base + r * kCT + tid];
        }
        __syncthreads();                           // s_w is reused
    }
}

__global__ __launch_bounds__(256) void compact_finish_kernel(DevPtrs d)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= d.B * d.S || !has_holes(d, g)) return;
    SegState& st = d.segs[g];
    st.parity ^= 1;
    st.count = st.live;
}

// Population control of one species over every discharge (the swarm's
// replicas): where the species holds more than `above` live particles, each
// is kept with probability keep / live, by an integer test on a Philox draw
// keyed by its id and the step (call 7); a removed particle becomes a hole,
// counted in the segment's dead count (zero between steps), which
// thin_finish takes off the live count before the compaction.  The live
// count is only read here, so every workgroup uses the same probability.
__global__ __launch_bounds__(256) void thin_mark_kernel(DevPtrs d, int32_t s, int64_t above, int64_t keep)
{
    const int b = (int)blockIdx.y;
    const int g = b * d.S + s;
    if (d.diss[b].retired) return;
    const SegState& st = d.segs[g];
    const int64_t live = st.live;
    if (live <= above || live <= keep) return;
    const uint32_t t24 = (uint32_t)(((uint64_t)keep << 24) / (uint64_t)live);   // < 2^24
    const SegConst& sc = d.segc[g];
    const DisConst& dc = d.disc[b];
    const uint32_t step = (uint32_t)d.diss[b].step;
    int32_t* cell = sc.cell[st.parity];
    const uint32_t* id = sc.id[st.parity];
    const int64_t n = st.count;
    uint32_t removed = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        if (cell[i] < 0) continue;
        const uint4 r = philox10(id[i], step, ((uint32_t)s << 24) | 7u, 0u, dc.key0, dc.key1);
        if (!(odd24(r.x) < t24)) {
            cell[i] = -1;
            ++removed;
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) removed += (uint32_t)__shfl_xor((int)removed, m, 64);
    if ((threadIdx.x & 63) == 0 && removed)
        atomicAdd(reinterpret_cast<unsigned long long*>(&d.segs[g].dead), (unsigned long long)removed);
}

__global__ __launch_bounds__(256) void thin_finish_kernel(DevPtrs d, int32_t s)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= d.B) return;
    SegState& st = d.segs[b * d.S + s];
    if (st.dead > 0) {
        st.live -= st.dead;
        st.dead = 0;
    }
}

}  // namespace

hipError_t launch_thin(const DevPtrs& d, int32_t species, int64_t above, int64_t keep, int64_t max_count,
                       int64_t max_tiles, int n_cu, hipStream_t st)
{
    const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((max_count + 255) / 256, 1024));
    hipLaunchKernelGGL(thin_mark_kernel, dim3(gx, (unsigned)d.B), dim3(256), 0, st, d, species, above, keep);
    hipLaunchKernelGGL(thin_finish_kernel, dim3((unsigned)((d.B + 255) / 256)), dim3(256), 0, st, d, species);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_compact(d, max_tiles, n_cu, st);
}

hipError_t launch_compact(const DevPtrs& d, int64_t max_tiles, int n_cu, hipStream_t st)
{
    const int NS = d.B * d.S;
    // persistent grids: every workgroup builds the segment prefix once and
    // strides over the tiles
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(max_tiles, (int64_t)n_cu * 8));
    hipLaunchKernelGGL(compact_count_kernel, dim3(grid), dim3(kCT), 0, st, d);
    // up to kAddTiles tiles a workgroup adds up the counts before each of its
    // tiles itself (at most 32 a thread and tile, one round of reads in flight
    // together, out of the L2), which is less than a launch of the scan and its
    // gap.  Measured, us per compaction, adding / scanning, one discharge (two
    // segments) of 512 tiles 14.6 / 16.8, 2048 27.0 / 29.9, 4096 38.9 / 43.3,
    // 8192 85 to 89 / 91 to 99; 64 discharges of 2048 tiles in all 18.7 / 24.1,
    // 8192 49.4 / 52.4.  Adding still wins at 32768 (346 / 366), but its reads
    // grow with the square of a segment's tiles, so the line lies well inside.
    constexpr int64_t kAddTiles = 8192;
    if (max_tiles <= kAddTiles) {
        hipLaunchKernelGGL(compact_scatter_kernel<false>, dim3(grid), dim3(kCT), 0, st, d);
    } else {
        hipLaunchKernelGGL(compact_scan_kernel, dim3((unsigned)NS), dim3(1024), 0, st, d);
        hipLaunchKernelGGL(compact_scatter_kernel<true>, dim3(grid), dim3(kCT), 0, st, d);
    }
    hipLaunchKernelGGL(compact_finish_kernel, dim3((unsigned)((NS + 255) / 256)), dim3(256), 0, st, d);
    return hipGetLastError();
}

int64_t compact_tiles_for(int64_t padded_count) { return (padded_count + kCTile - 1) / kCTile; }

}  // namespace pic
