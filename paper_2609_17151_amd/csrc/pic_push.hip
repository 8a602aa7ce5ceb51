#include "pic_push_kernel.h"

namespace pic {

// The events of a step, after the push: chunks of 64 consecutive events of
// one push workgroup's list (in any order: its waves claim places as they go),
// fully packed but for the last of each list, strided over all the waves of
// the grid.  Each lane one event: the renewal (a fresh velocity from the
// species' initial distribution, call 6), the collision of a candidate, or the
// secondary-emission test of an absorbed ion, all in FP64, with the new
// velocity rounded to binary32 once and written to the particle's slot.  The
// push has sampled the particle with the velocity of the record; a sampled
// step adds what the new one changes.  A birth (ionization pair, secondary electron) claims a
// slot of its tile's staging area with an atomic and carries its parent's
// slot, by which the finalize orders the tile's births; its charge goes
// straight into the discharge's fixed-point sums.  Counters come from
// ballots, per segment of the chunk.
// The segments' first tiles and the push workgroups' ranges come from the push,
// which left them in memory (forming them again from the segments' counts took
// 2.7 us of a launch of 54; 64 sampled discharges 262 -> 260 us per step).
template <int BS>
__global__ __launch_bounds__(BS) void events_kernel(EvArgs a)
{
    const DevPtrs& d = a.d;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    constexpr int kW = BS / 64;
    __shared__ uint32_t s_cp[kMaxPushGrid + 1];   // chunks of the push workgroups before each
    __shared__ uint32_t s_ne[kMaxPushGrid];       // events of each push workgroup
    __shared__ uint32_t s_w[kW];
    const int32_t chunk_t = (int32_t)d.evg[kMaxPushGrid];   // the push workgroups' tile ranges
    const int G = a.push_grid;
    uint32_t run = 0;
    for (int r = 0; r < G; r += BS) {
        const int g = r + tid;
        const uint32_t ne = g < G ? d.evg[g] : 0u;
        const uint32_t c = (ne + 63u) >> 6;
        if (g < G) s_ne[g] = ne;
        const uint32_t incl = wave_incl_scan_u32(c);
        if (lane == 63) s_w[wid] = incl;
        __syncthreads();
        uint32_t before = 0, tot = 0;
#pragma unroll
        for (int k = 0; k < kW; ++k) {
            const uint32_t v = s_w[k];
            if (k < wid) before += v;
            tot += v;
        }
        if (g < G) s_cp[g] = run + before + incl - c;
        run += tot;
        __syncthreads();
    }
    if (tid == 0) s_cp[G] = run;
    __syncthreads();
    const uint32_t bpt = (uint32_t)a.births_per_tile;
    const uint32_t nchunk = s_cp[G];
    const uint32_t stride = gridDim.x * kW;

    const EvPass e{a.T, chunk_t, bpt, a.diag, a.eepf_inv_bin, a.vm};
    // the records of chunk ck, for the lanes that hold one; the push
    // workgroup of chunk ck is the last g with s_cp[g] <= ck
    auto records = [&](uint32_t ck, uint4& rec, uint4& rq) -> bool {
        int glo = 0, ghi = G;
        while (ghi - glo > 1) {
            const int mid = (glo + ghi) >> 1;
            if (s_cp[mid] <= ck) glo = mid; else ghi = mid;
        }
        return event_record(d, e, glo, s_ne[glo], ck - s_cp[glo], rec, rq);
    };
    // each wave's next chunk's records are loaded before it works on the
    // current one, so that their latency overlaps the current chunk's loads
    uint32_t ck = blockIdx.x * kW + wid;
    uint4 rec = make_uint4(0u, 0u, 0u, 0u), rq = rec;
    bool act = ck < nchunk && records(ck, rec, rq);
    while (ck < nchunk) {
        const uint32_t nx = ck + stride;
        uint4 rec_n = make_uint4(0u, 0u, 0u, 0u), rq_n = rec_n;
        const bool act_n = nx < nchunk && records(nx, rec_n, rq_n);
        event_chunk(d, nullptr, e, act, rec, rq, -1, 0, nullptr, 0);
        rec = rec_n;
        rq = rq_n;
        act = act_n;
        ck = nx;
    }
}

size_t push_lds_bytes(int n_nodes, int n_cells, int diag)
{
    size_t b = (size_t)n_nodes * 8;
    if (diag) b += (size_t)n_nodes * 8 * 3 + kEepfBins * 4;
    b = (b + 15) & ~(size_t)15;
    b += (size_t)n_cells * 8;
    return b;
}

// nearest instantiated shape (1024 threads: four particles per thread; 512:
// four, or eight in the general kernel; 256: one to eight)
void push_shape(int& ppt, int& threads, bool general)
{
    if (threads >= 1024) {
        threads = 1024;
        ppt = 4;
    } else if (threads >= 512) {
        threads = 512;
        ppt = (general && ppt >= 8) ? 8 : 4;
    } else {
        threads = 256;
        ppt = ppt >= 8 ? 8 : (ppt >= 4 ? 4 : (ppt >= 2 ? 2 : 1));
    }
}

bool push_fusable(int ppt, int threads, bool general) { return general && threads == 256 && ppt <= 4; }

hipError_t launch_push(const PushArgs& a, int ppt, int threads, bool general, bool fuse, int vm, int64_t grid,
                       hipStream_t st)
{
    switch (vm) {
        case 0: return launch_push_vm<0>(a, ppt, threads, general, fuse, grid, st);
        case kUseY: return launch_push_vm<kUseY>(a, ppt, threads, general, fuse, grid, st);
        case kUseZ: return launch_push_vm<kUseZ>(a, ppt, threads, general, fuse, grid, st);
        case kUseY | kUseZ: return launch_push_vm<kUseY | kUseZ>(a, ppt, threads, general, fuse, grid, st);
        default: return hipErrorInvalidValue;
    }
}

int push_occupancy(int ppt, int threads, bool general, bool fuse, int vm, bool diag, size_t lds)
{
    switch (vm) {
        case 0: return push_occupancy_vm<0>(ppt, threads, general, fuse, diag, lds);
        case kUseY: return push_occupancy_vm<kUseY>(ppt, threads, general, fuse, diag, lds);
        case kUseZ: return push_occupancy_vm<kUseZ>(ppt, threads, general, fuse, diag, lds);
        default: return push_occupancy_vm<kUseY | kUseZ>(ppt, threads, general, fuse, diag, lds);
    }
}

template __global__ void events_kernel<kEvThreads>(EvArgs);

hipError_t launch_events(const EvArgs& a, int64_t grid, hipStream_t st)
{
    hipLaunchKernelGGL((events_kernel<kEvThreads>), dim3((unsigned)grid), dim3(kEvThreads), 0, st, a);
    return hipGetLastError();
}

int events_occupancy()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(events_kernel<kEvThreads>),
                                                     kEvThreads, 0) != hipSuccess)
        nb = 0;
    return nb > 0 ? nb : 1;
}

}  // namespace pic
