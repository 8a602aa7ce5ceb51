// Particle kernels of one leapfrog step for every species of every discharge
// of a context (paper Section 1: explicit leapfrog, Boris pusher, walls and
// secondary emission, null-collision Monte Carlo with tabulated cross
// sections; the charge of the particles deposited on the mesh).
//
// The push is one launch over all segments.  Work is cut into tiles of
// T = threads * PPT consecutive particle slots of one (discharge, species)
// segment; tiles are numbered over all segments, discharge-major, and every
// workgroup takes a fixed contiguous range of tiles, so no workgroup ever
// waits for another.  Each thread owns PPT consecutive slots and moves them
// with 16-byte vector loads and stores, in place.  A workgroup stages the
// (E[c], E[c+1]) pairs of a discharge in LDS once per run of tiles of that
// discharge, and zeroes and flushes its deposit histogram once per run of
// tiles of one segment.
//
// Per particle the push does the gather (linear weighting), the Boris push in
// the imposed B, the cell-relative move in FP32, the periodic wrap or the
// absorption at a wall, and the null-collision candidate test (an integer
// test on one Philox draw).  What only a few particles need per step is
// recorded as an event instead: a collision candidate, an axial renewal, the
// secondary-emission test of an absorbed ion.  Each wave appends its events'
// records to its workgroup's packed list at a place one LDS atomic claims
// (ballots and lane counts: no barrier, no queue); the events pass then does
// that work for all of them with full waves, in FP64: in the events kernel,
// or at the end of each push workgroup for its own list (FUSE).
//
// Absorbed particles leave holes (cell = -1) that later steps skip; a stable
// compaction every few steps removes them.  Holes do not change the order of
// the live particles, and births are appended after the last slot in the
// order of their parents, so the particle order after a compaction is the
// order that compacting every step would give.  The events pass stages a
// tile's births in any order, each with a key made of its parent's slot and
// its rank among that parent's births; the finalize writes each birth at the
// rank of its key within its tile, the tiles in order, which also gives their
// ids.
//
// Deposition: LDS histogram in 64-bit fixed point flushed with integer
// atomics (births add theirs with integer atomics too), so sums are exact and
// independent of the order of tiles and runs are bit-reproducible without
// global float atomics.
//
// Streaming instances (GENERAL = false) serve periodic runs without
// collisions or renewal, where nothing can be absorbed or born: no ids,
// holes or events.
#pragma once
#include "pic_device.h"
#include "pic_internal.h"
#include "pic_kernels.h"
#include "pic_solve.h"

namespace pic {

namespace {

// One LDS atomic per particle: with q = f 2^32 its node weights are 2^32 - q
// and q, so a cell's particles need only their number and the sum of their q.
// Both ride in one word: the number in the bits above kDepShift, the sum
// below.  The flush forms the node sums, number 2^32 - sum of the node's cell
// plus the sum of the cell before.  A histogram holds at most kDepMax
// particles, so neither part overflows (2^16 - 1 times 2^32 - 1 is below
// 2^48); a longer run of tiles is flushed in between.  Two 64-bit atomics per
// particle before: an LDS atomic on random cells takes 12 cycles of the
// compute unit per wave.
constexpr int kDepShift = 48;
constexpr int kDepMax = 65535;

__device__ __forceinline__ unsigned long long dep_word(float f)
{
    // f < 1, so f 2^32 fits 32 bits
    return (1ull << kDepShift) | (unsigned long long)(uint32_t)(f * 4294967296.0f);
}

// node i of the histogram of n_cells cells
__device__ __forceinline__ unsigned long long hist_node(const unsigned long long* hist, int i, int n_cells,
                                                        int periodic)
{
    constexpr unsigned long long kSum = (1ull << kDepShift) - 1ull;
    unsigned long long v = 0ull;
    if (i < n_cells) {
        const unsigned long long h = hist[i];
        v = ((h >> kDepShift) << 32) - (h & kSum);
    }
    const int il = i > 0 ? i - 1 : (periodic ? n_cells - 1 : -1);
    if (il >= 0) v += hist[il] & kSum;
    return v;
}

__device__ __forceinline__ void global_deposit(unsigned long long* acc, int c, float f, int n_cells,
                                               int periodic)
{
    uint32_t q = (uint32_t)(f * 4294967296.0f);
    if (f >= 1.0f) q = 0xFFFFFFFFu;
    const int c1 = (periodic && c + 1 == n_cells) ? 0 : c + 1;
    atomicAdd(&acc[c], (unsigned long long)(0x100000000ull - q));
    atomicAdd(&acc[c1], (unsigned long long)q);
}

// NT: non-temporal (streaming) accesses, which leave the caches to the rest
// of the step.  The general push takes them: us per step without / with, 64
// argon discharges of 4.9e7 particles 462 / 396, of 1.77e7 sampled 249 / 231,
// one of 4e5 19.8 / 19.9.  Where the particles would stay in the Infinity Cache
// from step to step they cost: 1.77e7 unsampled 157 / 166, a renewing box of 8e6
// 75.0 / 82.4, forty swarms of 4e6 54.5 / 56.7.  The streaming push, which does
// nothing else with the caches, is 11 % slower with them on an E x B box of 8e6
// and does without.
template <int N, typename V, bool NT = false, typename S>
__device__ __forceinline__ void vload(const PIC_GLOBAL S* p, S* out)
{
    if constexpr (N % 4 == 0) {
        typedef S NV __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            const PIC_GLOBAL NV* q = (const PIC_GLOBAL NV*)(p) + k;
            const NV v = NT ? __builtin_nontemporal_load(q) : *q;
            out[4 * k + 0] = v.x;
            out[4 * k + 1] = v.y;
            out[4 * k + 2] = v.z;
            out[4 * k + 3] = v.w;
        }
    } else {                       // (2-wide vector loads measured 4 % slower here)
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const PIC_GLOBAL S* q = (const PIC_GLOBAL S*)(p) + k;
            out[k] = NT ? __builtin_nontemporal_load(q) : *q;
        }
    }
}

template <int N, typename V, bool NT = false, typename S>
__device__ __forceinline__ void vstore(PIC_GLOBAL S* p, const S* in)
{
    if constexpr (N % 4 == 0) {
        typedef S NV __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            NV v;
            v.x = in[4 * k + 0];
            v.y = in[4 * k + 1];
            v.z = in[4 * k + 2];
            v.w = in[4 * k + 3];
            PIC_GLOBAL NV* q = (PIC_GLOBAL NV*)(p) + k;
            if (NT)
                __builtin_nontemporal_store(v, q);
            else
                *q = v;
        }
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            PIC_GLOBAL S* q = (PIC_GLOBAL S*)(p) + k;
            if (NT)
                __builtin_nontemporal_store(in[k], q);
            else
                *q = in[k];
        }
    }
}

// Events of the step, recorded by the push for the events pass: the slot
// of the particle in its tile and what happens to it there.
constexpr uint32_t kEvSlot = 0xffffu;       // slot in the tile (tiles hold at most 4096 particles)
constexpr uint32_t kEvCand = 1u << 16;      // collision candidate
constexpr uint32_t kEvRenew = 1u << 17;     // axial renewal: a fresh velocity
constexpr uint32_t kEvSee = 1u << 18;       // an emitting ion absorbed at a wall: secondary emission test
constexpr uint32_t kEvWall1 = 1u << 19;     // ... at the wall x = L
constexpr int kEvSegShift = 20;             // the particle's segment (kMaxSeg <= 1024: 10 bits)
static_assert(kMaxSeg <= 1024, "the event word holds the segment in 10 bits");
static_assert(C_N <= 64, "the flush's counters are held by one wave's lanes");

// The constants of a segment that the particle loop reads: loaded with the
// first tile's particles when a workgroup comes to the segment, then held in
// scalar registers (the segment is the same for the whole workgroup) until the
// next one.
struct PushC {
    int nc, periodic, emits, nch;
    uint32_t t32, key0, key1, step;
    float ex, ey, ez, qmh, tx, ty, tz, sx, sy, sz, dtdx;
    float hme, mscale1, mscale2;             // diagnostics
    int bulk_lo, bulk_hi;
    double renew_lz, dt_d;
};

__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t sgpr(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float sgpr(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double sgpr(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)(((uint64_t)sgpr((uint32_t)(u >> 32)) << 32) | sgpr((uint32_t)u)));
}

template <bool GENERAL, int VM, bool DIAG>
__device__ __forceinline__ PushC push_consts(CSeg& sc, CDis& dc, uint32_t step)
{
    PushC k;
    k.nc = dc.n_cells;
    k.periodic = dc.bc == PIC_BC_PERIODIC;
    k.ex = sc.eext[0];
    k.ey = sc.eext[1];
    k.ez = sc.eext[2];
    k.qmh = sc.qmh;
    k.tx = sc.tv[0];
    k.ty = sc.tv[1];
    k.tz = sc.tv[2];
    k.sx = sc.sv[0];
    k.sy = sc.sv[1];
    k.sz = sc.sv[2];
    k.dtdx = sc.dtdx;
    if (GENERAL) {
        k.emits = sc.emits;
        k.nch = sc.nch;
        k.t32 = sc.t32;
        k.key0 = dc.key0;
        k.key1 = dc.key1;
        k.step = step;
        if (VM & kUseZ) {                    // renewal sums vz
            k.renew_lz = sc.renew_lz;
            k.dt_d = sc.dt_d;
        }
    }
    if (DIAG) {
        k.hme = sc.half_m_over_e;
        k.mscale1 = sc.mscale1;
        k.mscale2 = sc.mscale2;
        k.bulk_lo = dc.bulk_lo;
        k.bulk_hi = dc.bulk_hi;
    }
    return k;
}

template <bool GENERAL, int VM, bool DIAG>
__device__ __forceinline__ PushC push_consts_sgpr(const PushC& v)
{
    PushC k;
    k.nc = sgpr(v.nc);
    k.periodic = sgpr(v.periodic);
    k.ex = sgpr(v.ex);
    k.qmh = sgpr(v.qmh);
    k.dtdx = sgpr(v.dtdx);
    if (VM & kUseY) k.ey = sgpr(v.ey);
    if (VM & kUseZ) k.ez = sgpr(v.ez);
    if (VM == (kUseY | kUseZ)) {
        k.tx = sgpr(v.tx);
        k.sx = sgpr(v.sx);
    }
    if (VM & kUseZ) {
        k.ty = sgpr(v.ty);
        k.sy = sgpr(v.sy);
    }
    if (VM & kUseY) {
        k.tz = sgpr(v.tz);
        k.sz = sgpr(v.sz);
    }
    if (GENERAL) {
        k.emits = sgpr(v.emits);
        k.nch = sgpr(v.nch);
        k.t32 = sgpr(v.t32);
        k.key0 = sgpr(v.key0);
        k.key1 = sgpr(v.key1);
        k.step = sgpr(v.step);
        if (VM & kUseZ) {
            k.renew_lz = sgpr(v.renew_lz);
            k.dt_d = sgpr(v.dt_d);
        }
    }
    if (DIAG) {
        k.hme = sgpr(v.hme);
        k.mscale1 = sgpr(v.mscale1);
        k.mscale2 = sgpr(v.mscale2);
        k.bulk_lo = sgpr(v.bulk_lo);
        k.bulk_hi = sgpr(v.bulk_hi);
    }
    return k;
}

// A float that holds an integer, as a 64-bit word: one conversion where it
// fits 32 bits, which the sampled moments and energies do but for extreme
// particles; the general conversion takes ten times as many instructions.
__device__ __forceinline__ unsigned long long fixed_i64(float r)
{
    if (fabsf(r) < 2147483648.0f) return (unsigned long long)(long long)(int)r;
    return (unsigned long long)(long long)r;
}

__device__ __forceinline__ unsigned long long fixed_u64(float r)
{
    if (r < 4294967296.0f) return (unsigned long long)(uint32_t)r;
    return (unsigned long long)r;
}

// Gather, Boris push and cell-relative move of one particle, without a branch:
// the few particles that need more (a wall, a corrupt or non-finite state) are
// found by their results afterwards.  Returns whether the cell was out of
// range (the particle is parked in cell 0).
template <int VM, bool DIAG>
__device__ __forceinline__ bool advance(const PushC& k, const float2* ep, int& c, float& f, float& ux, float& uy,
                                        float& uz, float& ke)
{
    constexpr bool UY = (VM & kUseY) != 0, UZ = (VM & kUseZ) != 0;
    const bool c_bad = (unsigned)c >= (unsigned)k.nc;
    c = c_bad ? 0 : c;
    f = c_bad ? 0.0f : f;
    // gather
    const float2 e2 = ep[c];
    const float ex = e2.x + f * (e2.y - e2.x) + k.ex;
    // Boris: half kick, rotation, half kick.  A component the fields neither
    // change nor read (VM) is left out: its terms in the others' rotation are
    // products with zero, so the rest is the same, bit for bit.
    const float qmh = k.qmh;
    const float vold2 = DIAG ? ux * ux + uy * uy + uz * uz : 0.0f;
    ux += qmh * ex;
    if (UY) uy += qmh * k.ey;
    if (UZ) uz += qmh * k.ez;
    if (UY && UZ) {
        const float tx = k.tx, ty = k.ty, tz = k.tz;
        const float sx = k.sx, sy = k.sy, sz = k.sz;
        const float px = ux + (uy * tz - uz * ty);
        const float py = uy + (uz * tx - ux * tz);
        const float pz = uz + (ux * ty - uy * tx);
        ux += py * sz - pz * sy;
        uy += pz * sx - px * sz;
        uz += px * sy - py * sx;
    } else if (UZ) {                       // B along y
        const float px = ux - uz * k.ty;
        const float pz = uz + ux * k.ty;
        ux -= pz * k.sy;
        uz += px * k.sy;
    } else if (UY) {                       // B along z
        const float px = ux + uy * k.tz;
        const float py = uy - ux * k.tz;
        ux += py * k.sz;
        uy -= px * k.sz;
    }
    ux += qmh * ex;
    if (UY) uy += qmh * k.ey;
    if (UZ) uz += qmh * k.ez;
    ke = DIAG ? vold2 + (ux * ux + uy * uy + uz * uz) : 0.0f;
    // move, relative to the cell
    f += ux * k.dtdx;
    const float fl = floorf(f);
    c += (int)fl;
    f -= fl;
    const bool up = f >= 1.0f;
    f = up ? f - 1.0f : f;
    c += up ? 1 : 0;
    return c_bad;
}

// a particle whose state is not finite after its move: f is in [0, 1) or, for
// an infinite or undefined velocity, undefined
__device__ __forceinline__ bool not_finite(float f, float ux) { return !(f < 1.0f) || !(fabsf(ux) < 3.0e38f); }

// First word of the particle's draw (the candidate test).  The round keys come
// from scalar adds: hidden from the optimiser, which would otherwise hold all
// twenty of them in registers across the loop and spill.
__device__ __forceinline__ uint32_t candidate_draw(uint32_t id, const PushC& k, int s)
{
    uint32_t k0 = k.key0, k1 = k.key1;
    asm volatile("" : "+s"(k0), "+s"(k1));
    return philox10(id, k.step, ((uint32_t)s << 24), 0u, k0, k1).x;
}

// Sampled sums of one or more particles of a cell, fixed point: the velocity
// moments (flux, x-momentum flux) and for electrons the energy, each at the
// cell's two nodes (0 the left one)
struct Sampled {
    unsigned long long f0, f1, m0, m1, e0, e1;
};

// velocity moments of a particle (diagnostics); ms1, ms2 the species'
// fixed-point scales
__device__ __forceinline__ void moment_words(float ms1, float ms2, float f, float ux, Sampled& v)
{
    const float a = ux * ms1, b2 = ux * ux * ms2;
    const float w0 = 1.0f - f;
    v.f0 = fixed_i64(rintf(w0 * a));
    v.f1 = fixed_i64(rintf(f * a));
    v.m0 = fixed_i64(rintf(w0 * b2));
    v.m1 = fixed_i64(rintf(f * b2));
}

__device__ __forceinline__ void energy_words(float eps, float f, Sampled& v)
{
    const float w1 = f * eps, w0 = eps - w1;
    v.e0 = fixed_u64(w0 * 1048576.0f);
    v.e1 = fixed_u64(w1 * 1048576.0f);
}

// fh, mh and ehist are LDS histograms in the push and the discharge's global
// sums in the events pass
__device__ __forceinline__ void add_moments(unsigned long long* fh, unsigned long long* mh, int c, int c1,
                                            const Sampled& v)
{
    atomicAdd(&fh[c], v.f0);
    atomicAdd(&fh[c1], v.f1);
    atomicAdd(&mh[c], v.m0);
    atomicAdd(&mh[c1], v.m1);
}

__device__ __forceinline__ void add_energy(unsigned long long* ehist, int c, int c1, const Sampled& v)
{
    atomicAdd(&ehist[c], v.e0);
    atomicAdd(&ehist[c1], v.e1);
}

__device__ __forceinline__ int right_node(int c, int nc, int periodic) { return (periodic && c + 1 == nc) ? 0 : c + 1; }

// the bulk energy distribution; CT is the bin counter type (32-bit in LDS,
// 64-bit in global memory), [lo, hi) its cells
template <typename CT>
__device__ __forceinline__ void add_bulk(CT* eepf, float eepf_inv_bin, float eps, int c, int lo, int hi)
{
    if (c >= lo && c < hi) {
        const int bin = (int)(eps * eepf_inv_bin);
        if ((unsigned)bin < (unsigned)kEepfBins) atomicAdd(&eepf[bin], (CT)1);
    }
}

// one particle's samples in the events pass: hme = m / 2e
__device__ __forceinline__ void sample_particle(const DevPtrs& d, CSeg& sc, CDis& dc, int b, int sg,
                                                bool electron, float eepf_inv_bin, int c, float f, float ux,
                                                float uy, float uz)
{
    const int c1 = right_node(c, dc.n_cells, dc.bc == PIC_BC_PERIODIC);
    Sampled v;
    moment_words(sc.mscale1, sc.mscale2, f, ux, v);
    unsigned long long* fh = d.macc + (size_t)sg * 2 * d.nodes_max;
    add_moments(fh, fh + d.nodes_max, c, c1, v);
    if (electron) {
        const float eps = sc.half_m_over_e * (ux * ux + uy * uy + uz * uz);
        energy_words(eps, f, v);
        add_energy(d.eacc + (size_t)b * d.nodes_max, c, c1, v);
        add_bulk(d.eepf + (size_t)b * 2 * kEepfBins, eepf_inv_bin, eps, c, dc.bulk_lo, dc.bulk_hi);
    }
}

// What a change of a particle's velocity (o to u) changes in the sums: exact,
// they are whole numbers.  The push samples every particle and the events pass
// adds this for those that did collide, a third of the candidates (one in a
// hundred of the ions').  When it added every candidate's samples itself, up to
// seven atomics on global memory each, a step of 64 sampled discharges with
// 1.77e7 particles took 340 us, now 280.
__device__ __forceinline__ void sample_change(const DevPtrs& d, CSeg& sc, CDis& dc, int b, int sg,
                                              bool electron, float eepf_inv_bin, int c, float f, float ox, float oy,
                                              float oz, float ux, float uy, float uz)
{
    const int c1 = right_node(c, dc.n_cells, dc.bc == PIC_BC_PERIODIC);
    Sampled o, v;
    moment_words(sc.mscale1, sc.mscale2, f, ox, o);
    moment_words(sc.mscale1, sc.mscale2, f, ux, v);
    v.f0 -= o.f0;
    v.f1 -= o.f1;
    v.m0 -= o.m0;
    v.m1 -= o.m1;
    unsigned long long* fh = d.macc + (size_t)sg * 2 * d.nodes_max;
    add_moments(fh, fh + d.nodes_max, c, c1, v);
    if (electron) {
        const float eo = sc.half_m_over_e * (ox * ox + oy * oy + oz * oz);
        const float eps = sc.half_m_over_e * (ux * ux + uy * uy + uz * uz);
        energy_words(eo, f, o);
        energy_words(eps, f, v);
        v.e0 -= o.e0;
        v.e1 -= o.e1;
        add_energy(d.eacc + (size_t)b * d.nodes_max, c, c1, v);
        if (c >= dc.bulk_lo && c < dc.bulk_hi) {
            unsigned long long* eb = d.eepf + (size_t)b * 2 * kEepfBins;
            const int from = (int)(eo * eepf_inv_bin), to = (int)(eps * eepf_inv_bin);
            if (from != to) {
                if ((unsigned)from < (unsigned)kEepfBins) atomicAdd(&eb[from], ~0ull);
                if ((unsigned)to < (unsigned)kEepfBins) atomicAdd(&eb[to], 1ull);
            }
        }
    }
}

// block reduction in a fixed order (deterministic)
template <int BS>
__device__ __forceinline__ double block_sum_f32(float v, float* s_w)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const float w = wave_sum_f32(v);
    __syncthreads();
    if (lane == 0) s_w[wid] = w;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < BS / 64; ++k) t += (double)s_w[k];
    return t;
}

// First tile of every (discharge, species) segment for tiles of T particles,
// from the device-resident counts (retired discharges get none): s_pref[g]
// is the first tile of segment g, s_pref[NS] the number of tiles.  Wave 0,
// up to 16 segments per lane; the caller synchronises.
__device__ __forceinline__ void tile_prefix(const DevPtrs& d, int T, int32_t* s_pref)
{
    const int S = d.S, NS = d.B * d.S;
    const int lane = threadIdx.x & 63;
    if ((threadIdx.x >> 6) != 0) return;
    const int per = (NS + 63) >> 6;
    const int g0 = lane * per;
    int32_t run = 0;
    for (int j = 0; j < per; ++j) {
        const int g = g0 + j;
        if (g < NS) {
            const int64_t n = d.diss[g / S].retired ? 0 : d.segs[g].count;
            run += (int32_t)((n + T - 1) / T);
            s_pref[g + 1] = run;
        }
    }
    int32_t incl = run;
#pragma unroll
    for (int dd = 1; dd < 64; dd <<= 1) {
        const int32_t o = __shfl_up(incl, dd, 64);
        if (lane >= dd) incl += o;
    }
    const int32_t excl = incl - run;
    if (lane == 0) s_pref[0] = 0;
    for (int j = 0; j < per; ++j) {
        const int g = g0 + j;
        if (g < NS) s_pref[g + 1] += excl;
    }
}

// the segment of tile t: the last g with s_pref[g] <= t
__device__ __forceinline__ int tile_segment(const int32_t* s_pref, int NS, int32_t t)
{
    int lo = 0, hi = NS;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_pref[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

}  // namespace

// The events pass over one chunk of 64 events of a push workgroup's list,
// one event per lane (defined with the events kernel below): the records of
// the chunk, then the work on them.
struct EvPass {
    int32_t T;                    // particles of the push's tile
    int32_t chunk_t;              // tiles per push workgroup
    uint32_t bpt;                 // births staged per tile at most
    int32_t diag;
    float eepf_inv_bin;
    int32_t vm;                   // velocity components of the records (the others are read from the particle's slot)
};

__device__ __forceinline__ bool event_record(const DevPtrs& d, const EvPass& ps, int g, uint32_t nev, uint32_t kc,
                                             uint4& rec, uint4& rq);
__device__ __forceinline__ void event_chunk(const DevPtrs& d, const int32_t* s_pref, const EvPass& ps, bool act,
                                            uint4 rec, uint4 rq, int k_sg, int32_t k_first, char* k_base,
                                            int64_t k_stride);

__device__ __forceinline__ int64_t readlane64(int64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The field of a periodic mesh of up to kSolveNodes nodes from the deposit sums
// `acc` of its species, as the finalize kernel forms it (the same operations in
// the same order), straight into the E pairs of the gather; s_a: LDS for nn
// doubles.  The whole workgroup calls it.
template <int BS>
__device__ __forceinline__ void solve_pairs(const DevPtrs& d, CDis& dc, int b,
                                            const unsigned long long* acc, double* s_a, double* s_w, Run* s_run,
                                            float2* ep)
{
    const int S = d.S, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int nn = dc.n_nodes;
    const unsigned long long* ab = acc + (size_t)b * S * kRep * d.nodes_max;
    for (int base = wid * 64; base < nn; base += BS) {
        const int i = base + lane;
        double r = 0.0;
        if (i < nn) {
            unsigned long long v[kMaxSpecies];
#pragma unroll
            for (int s = 0; s < kMaxSpecies; ++s) {
                v[s] = 0ull;
                if (s < S)
                    for (int q = 0; q < kRep; ++q) v[s] += ab[((size_t)s * kRep + q) * d.nodes_max + i];
            }
            r = dc.rho_bg;
#pragma unroll
            for (int s = 0; s < kMaxSpecies; ++s)
                if (s < S) r += dc.q[s] * ((double)v[s] * dc.dens_coef[s]);
            s_a[i] = r;
        }
        const double w = wave_total_f64(r);
        if (lane == 0) s_w[base >> 6] = w;
    }
    lds_barrier();
    constexpr int kN = 4;                                // nodes per thread
    const int i0 = tid * kN;
    const bool active = wid * 64 * kN < nn;
    double g[kN];
    Run inc{0.0, 0.0, 0.0, 0.0};
    if (active) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kSolveNodes / 64; ++w) tot += w * 64 < nn ? s_w[w] : 0.0;
        const double mean = tot / nn, c2 = dc.c2;
        Run loc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            const int i = i0 + j;
            g[j] = 0.0;
            if (i < nn) {
                g[j] = i >= 1 ? (s_a[i] - mean) * c2 : 0.0;
                loc.n += 1.0;
                loc.S += g[j];
                loc.P += loc.S;
                loc.Q += loc.P;
            }
        }
        inc = wave_run_scan(loc);
        if (lane == 63) s_run[wid] = inc;
    }
    lds_barrier();
    if (active) {
        Run before, all;
        few_runs(s_run, (nn + 64 * kN - 1) / (64 * kN), wid, before, all);
        const double d0 = all.P / nn;
        const double pm = (d0 * (0.5 * (double)nn * (double)(nn - 1)) - (all.Q - all.P)) / nn;
        Run lx;
        lx.n = __shfl_up(inc.n, 1, 64);
        lx.S = __shfl_up(inc.S, 1, 64);
        lx.P = __shfl_up(inc.P, 1, 64);
        lx.Q = 0.0;
        if (lane == 0) lx = Run{0.0, 0.0, 0.0, 0.0};
        const Run ex = wid > 0 ? run_combine(before, lx) : lx;
        double G = ex.S, P = ex.P;
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            const int i = i0 + j;
            if (i >= nn) break;
            G += g[j];
            P += G;
            double ph = 0.0 + (double)i * d0 - (P - G);
            if (i == 0) ph = 0.0;
            s_a[i] = ph - pm;
        }
    }
    lds_barrier();
    const double h = dc.inv_2dx;
    for (int c = tid; c < nn; c += BS) {
        const int cm = c == 0 ? nn - 1 : c - 1, c1 = c + 1 == nn ? 0 : c + 1, c2 = c1 + 1 == nn ? 0 : c1 + 1;
        ep[c] = dc.field_solve ? make_float2((float)((s_a[cm] - s_a[c1]) * h), (float)((s_a[c] - s_a[c2]) * h))
                               : make_float2(0.0f, 0.0f);
    }
    lds_barrier();                                       // s_a is free again
}

// FUSE: the workgroup does its own tile range's events after its push (no
// events launch; for workloads too small to fill the GPU twice).
// VM: the velocity components, besides x, that the fields change in some
// segment of the launch (kUseY, kUseZ).  DIAG: the step is sampled.
//
// A small step is a chain of dependent memory latencies, so the start keeps it
// short: contexts of up to 64 segments read every segment's count, step and
// place in one round, a lane each, in every wave (no LDS, no barrier); then the
// first tile's particles, the segment's constants and the discharge's E pairs
// are all in flight together, and one barrier later the particles are pushed.
//
// SOLVE (streaming steps after the first of a run): every workgroup solves for
// the field itself, from the deposit of the step before, so the steps of a run
// are one launch each and the finalize kernel runs once at its end.  A finalize
// in between is one workgroup with the GPU idle around it, 4 to 6 us and two
// launch gaps of 1.2 to 3 us.  Per step, 6.5e4 particles on 128 cells: 11.2
// us with the finalize, 7.9 us with the solve; 8e6 on 1024 cells: 51.8 and
// 47.8 us; 6.4e7: 424 and 418 us.
template <int PPT, int BS, bool GENERAL, bool FUSE, int VM, bool DIAG, bool SOLVE>
__global__ __launch_bounds__(BS) void push_kernel(PushArgs a)
{
    constexpr int kBS = BS;
    constexpr int T = kBS * PPT;
    constexpr bool UY = (VM & kUseY) != 0, UZ = (VM & kUseZ) != 0;
    constexpr bool RY = UY || DIAG, RZ = UZ || DIAG;   // components read
    constexpr int kRunTiles = kDepMax / T;        // tiles one deposit histogram holds
    constexpr int kWavesPerTile = kBS / 64;
    const DevPtrs& d = a.d;
    const int S = d.S, NS = d.B * d.S;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;

    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_pref[kMaxSeg + 1];   // first tile of every segment (discharge-major)
    __shared__ unsigned int s_cnt[C_N];
    __shared__ unsigned long long s_wen[2];   // energy carried into each wall by the run (eV, 2^20)
    __shared__ float s_red[kBS / 64];
    __shared__ uint32_t s_evn;                // events recorded by the workgroup
    // FUSE: the first events' records stay in LDS (the others' go to memory),
    // one round trip less in a step that is little else (with the table rows
    // read together: 4e5 particles of argon 21.5 -> 21.1 us per step, forty
    // swarms 95.2 -> 91.6)
    constexpr uint32_t kEvLds = FUSE ? 128u : 1u;
    __shared__ uint4 s_rec[kEvLds], s_rq[kEvLds];
    __shared__ double s_w[SOLVE ? kSolveNodes / 64 : 1];
    __shared__ Run s_run[SOLVE ? 4 : 1];

    if (SOLVE) {
        const size_t words = (size_t)NS * kRep * d.nodes_max;
        for (size_t i = (size_t)blockIdx.x * kBS + tid; i < words; i += (size_t)gridDim.x * kBS) a.acc_clear[i] = 0ull;
    }

    // the tiles of every segment: lane g holds segment g's row, or (more than
    // 64 segments) the first tiles in LDS
    const bool few = NS <= 64;
    int64_t l_count = 0, l_base = 0, l_stride = 0;
    int32_t l_parity = 0, l_incl = 0, NT;
    if (few) {
        if (lane < NS) {
            const SegState& st = d.segs[lane];
            l_count = st.count;
            l_base = (int64_t)(uintptr_t)st.base;
            l_stride = st.stride;
            l_parity = st.parity;
            const bool off = d.diss[seg_discharge(lane, S)].retired != 0;
            l_incl = off ? 0 : (int32_t)((l_count + T - 1) / T);
        }
        for (int dd = 1; dd < NS; dd <<= 1) {
            const int32_t o = __shfl_up(l_incl, dd, 64);
            if (lane >= dd) l_incl += o;
        }
        if (wid == 0) {
            if (lane < NS) s_pref[lane + 1] = l_incl;
            if (lane == 0) s_pref[0] = 0;
        }
        NT = __builtin_amdgcn_readlane(l_incl, NS - 1);
    } else {
        tile_prefix(d, T, s_pref);
        lds_barrier();
        NT = sgpr(s_pref[NS]);
    }
    if (tid < C_N) s_cnt[tid] = 0;
    if (tid < 2) s_wen[tid] = 0ull;
    if (tid == 0) s_evn = 0u;

    // LDS layout: deposit histogram, [energy, flux and momentum-flux
    // histograms, EEPF], E pairs
    const int nn_max = a.nodes_max_dyn;
    const int dn = DIAG ? nn_max : 0;
    unsigned long long* hist = reinterpret_cast<unsigned long long*>(smem);
    unsigned long long* ehist = hist + nn_max;
    unsigned long long* fhist = ehist + dn;
    unsigned long long* mhist = fhist + dn;
    unsigned int* eepf = reinterpret_cast<unsigned int*>(mhist + dn);
    float2* ep = reinterpret_cast<float2*>(eepf + (DIAG ? kEepfBins : 0));

    // the current segment
    int sg = -1, b = -1, s = 0;
    int32_t seg_first = 0, run_first = 0, hist_end = 0;
    float ke_run = 0.0f;
    int64_t n = 0;
    char* base_p = nullptr;                   // its particle arrays, `stride` bytes apart
    int64_t stride = 0;
    PIC_GLOBAL double* p_z = nullptr;
    PushC k{};
    // a fixed contiguous range of tiles per workgroup
    const int32_t chunk = (NT + (int32_t)gridDim.x - 1) / (int32_t)gridDim.x;
    if (GENERAL && !FUSE && blockIdx.x == 0 && tid == 0) d.evg[kMaxPushGrid] = (uint32_t)chunk;
    const int32_t t_begin = (int32_t)blockIdx.x * chunk;
    const int32_t t_end = t_begin + chunk < NT ? t_begin + chunk : NT;
    if (t_begin >= t_end) {
        if (GENERAL && tid == 0) d.evg[blockIdx.x] = 0u;
        return;
    }
    int32_t seg_end = t_begin;

    // the deposit histogram's node sums go out
    auto flush_nodes = [&](int ft, int nt) {
        unsigned long long* acc_s = a.acc + ((size_t)sg * kRep + blockIdx.x % kRep) * d.nodes_max;
        const int nn = k.nc + (k.periodic ? 0 : 1);
        for (int i = ft; i < nn; i += nt) {
            const unsigned long long v = hist_node(hist, i, k.nc, k.periodic);
            if (v) atomicAdd(&acc_s[i], v);
        }
    };

    // flush the run of tiles of the current segment: deposit, diagnostics,
    // counters, kinetic energy (ranges are fixed, so the grouping of the sums
    // is too).  The first `quiet` threads (whole waves) take part in the
    // barriers only, so that no memory operation of the flush is outstanding
    // in those waves when they go on to the events pass.
    auto flush = [&](int quiet) {
        const int ft = tid - quiet, nt = kBS - quiet;
        if (ft >= 0) {
            flush_nodes(ft, nt);
            const int nn = k.nc + (k.periodic ? 0 : 1);
            if (DIAG) {
                unsigned long long* ma = d.macc + (size_t)sg * 2 * d.nodes_max;
                for (int i = ft; i < nn; i += nt) {
                    const unsigned long long v = fhist[i], w = mhist[i];
                    if (v) atomicAdd(&ma[i], v);
                    if (w) atomicAdd(&ma[d.nodes_max + i], w);
                }
            }
            if (DIAG && s == 0) {
                unsigned long long* ea = d.eacc + (size_t)b * d.nodes_max;
                for (int i = ft; i < nn; i += nt) {
                    const unsigned long long v = ehist[i];
                    if (v) atomicAdd(&ea[i], v);
                }
                unsigned long long* eg = d.eepf + (size_t)b * 2 * kEepfBins;
                for (int i = ft; i < kEepfBins; i += nt) {
                    const unsigned int v = eepf[i];
                    if (v) atomicAdd(&eg[i], (unsigned long long)v);
                }
            }
            if (GENERAL) {
                unsigned long long* cnt = d.cnt + ((size_t)sg * kRep + blockIdx.x % kRep) * C_N;
                if (ft < C_N) {
                    const unsigned int v = s_cnt[ft];
                    if (v) {
                        atomicAdd(&cnt[ft], (unsigned long long)v);
                        if (ft == C_ABS0 || ft == C_ABS1)
                            atomicAdd(reinterpret_cast<unsigned long long*>(&d.segs[sg].dead), (unsigned long long)v);
                    }
                    s_cnt[ft] = 0;
                }
                if (ft < 2) {
                    const unsigned long long v = s_wen[ft];
                    if (v) atomicAdd(&d.wen[(size_t)sg * 2 + ft], v);
                    s_wen[ft] = 0ull;
                }
            }
        }
        if (DIAG) {
            const double kt = block_sum_f32<BS>(ke_run, s_red);
            if (ft == 0) d.ke_part[run_first] = 0.5 * d.segc[sg].mw_half * kt;
            ke_run = 0.0f;
        }
    };

    for (int32_t t = t_begin; t < t_end; ++t) {
        const bool sw = t >= seg_end;                 // the next segment begins
        // the next segment's values: the current ones stay until its flush
        int sg_n = sg, b_n = b;
        int32_t first_n = seg_first;
        char* base_n = base_p;
        PushC kv{};
        if (sw) {
            int64_t count;
            int par;
            if (few) {
                sg_n = (int)__popcll(__ballot(lane < NS && l_incl <= t));
                first_n = sg_n > 0 ? __builtin_amdgcn_readlane(l_incl, sg_n - 1) : 0;
                seg_end = __builtin_amdgcn_readlane(l_incl, sg_n);
                count = readlane64(l_count, sg_n);
                base_n = (char*)(uintptr_t)readlane64(l_base, sg_n);
                stride = readlane64(l_stride, sg_n);
                par = __builtin_amdgcn_readlane(l_parity, sg_n);
            } else {
                if (sg < 0) sg_n = tile_segment(s_pref, NS, t);
                while (s_pref[sg_n + 1] <= t) ++sg_n;
                sg_n = sgpr(sg_n);
                first_n = sgpr(s_pref[sg_n]);
                seg_end = sgpr(s_pref[sg_n + 1]);
                const SegState& st = d.segs[sg_n];
                count = readlane64(st.count, 0);
                base_n = (char*)(uintptr_t)readlane64((int64_t)(uintptr_t)st.base, 0);
                stride = readlane64(st.stride, 0);
                par = sgpr(st.parity);
            }
            n = count;                                // updated in place: the copy in use
            base_n += (int64_t)par * kFields * stride;
            b_n = seg_discharge(sg_n, S);
            CSeg& sc = const_seg(d, sg_n);
            if (GENERAL && UZ) p_z = (PIC_GLOBAL double*)sc.z[par];
            kv = push_consts<GENERAL, VM, DIAG>(sc, const_dis(d, b_n), const_step(d, b_n));   // in flight with the particles
        }
        const int32_t tin = t - first_n;
        const int64_t tile0 = (int64_t)tin * T;
        const int rem = n - tile0 < T ? (int)(n - tile0) : T;     // slots in use
        char* pt = base_n + tile0 * 4;
        PIC_GLOBAL int32_t* p_cell = (PIC_GLOBAL int32_t*)(pt);
        PIC_GLOBAL float* p_off = (PIC_GLOBAL float*)(pt + stride);
        PIC_GLOBAL float* p_vx = (PIC_GLOBAL float*)(pt + 2 * stride);
        PIC_GLOBAL float* p_vy = (PIC_GLOBAL float*)(pt + 3 * stride);
        PIC_GLOBAL float* p_vz = (PIC_GLOBAL float*)(pt + 4 * stride);
        const PIC_GLOBAL uint32_t* p_id = (const PIC_GLOBAL uint32_t*)(pt + 5 * stride);
        const int slot0 = tid * PPT;

        int32_t cell[PPT];
        float off[PPT], vx[PPT], vy[PPT], vz[PPT];
        uint32_t pid[PPT];
        vload<PPT, int4, GENERAL>(p_cell + slot0, cell);
        vload<PPT, float4, GENERAL>(p_off + slot0, off);
        vload<PPT, float4, GENERAL>(p_vx + slot0, vx);
        if (RY) {
            vload<PPT, float4, GENERAL>(p_vy + slot0, vy);
        } else {
#pragma unroll
            for (int j = 0; j < PPT; ++j) vy[j] = 0.0f;
        }
        if (RZ) {
            vload<PPT, float4, GENERAL>(p_vz + slot0, vz);
        } else {
#pragma unroll
            for (int j = 0; j < PPT; ++j) vz[j] = 0.0f;
        }
        // ids only where every particle draws; the events pass reads the
        // others' from their slots
        if (GENERAL && (sw ? const_seg(d, sg_n).nch : k.nch) > 0) {
            vload<PPT, uint4, GENERAL>(p_id + slot0, pid);
        } else {
#pragma unroll
            for (int j = 0; j < PPT; ++j) pid[j] = 0u;
        }

        if (sw) {
            if (sg >= 0) {
                lds_barrier();
                flush(0);
                lds_barrier();
            }
            if (b_n != b) {
                if (SOLVE) {
                    solve_pairs<BS>(d, const_dis(d, b_n), b_n, a.acc_in, reinterpret_cast<double*>(hist), s_w, s_run, ep);
                } else {
                    const float2* epg = d.epair + (size_t)b_n * d.cells_max;
                    for (int i = tid; i < a.cells_max_dyn; i += kBS) ep[i] = epg[i];
                }
            }
            for (int i = tid; i < nn_max; i += kBS) hist[i] = 0ull;
            if (DIAG) {
                for (int i = tid; i < nn_max; i += kBS) {
                    fhist[i] = 0ull;
                    mhist[i] = 0ull;
                }
            }
            sg = sg_n;
            b = b_n;
            s = sg - b * S;
            seg_first = first_n;
            base_p = base_n;
            run_first = t;
            hist_end = t + kRunTiles;
            if (DIAG && s == 0) {
                for (int i = tid; i < nn_max; i += kBS) ehist[i] = 0ull;
                for (int i = tid; i < kEepfBins; i += kBS) eepf[i] = 0u;
            }
            lds_barrier();
            k = push_consts_sgpr<GENERAL, VM, DIAG>(kv);
        } else if (t == hist_end) {
            // a histogram full before its run of tiles ends
            lds_barrier();
            flush_nodes(tid, kBS);
            lds_barrier();
            for (int i = tid; i < k.nc; i += kBS) hist[i] = 0ull;
            lds_barrier();
            hist_end = t + kRunTiles;
        }
        // axial renewal: the displacement along the third axis since
        // injection, summed in FP64 (a slow ion adds only a few binary32
        // spacings of z per step, so a binary32 sum would drift)
        const bool renews = GENERAL && UZ && k.renew_lz > 0.0;
        double zax[PPT];
        if (renews) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) zax[j] = p_z[tile0 + slot0 + j];
        }

        // All of a thread's particles go through each stage together, without
        // branches (their chains overlap); what only few particles need is
        // behind one test per wave.
        uint32_t evw[PPT];
        bool keep[PPT];
        float ke[PPT];
        bool bad = false, odd = false;
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            evw[j] = 0u;
            const int c0 = cell[j];
            keep[j] = slot0 + j < rem && (!GENERAL || c0 >= 0);    // GENERAL: not a hole
            const bool cb = advance<VM, DIAG>(k, ep, cell[j], off[j], vx[j], vy[j], vz[j], ke[j]);
            bad |= keep[j] && cb;
            odd |= keep[j] && not_finite(off[j], vx[j]);
        }
        if (__any(odd)) {
#pragma unroll
            for (int j = 0; j < PPT; ++j)
                if (keep[j] && not_finite(off[j], vx[j])) {
                    atomicOr(&d.diss[b].flags, kFlagNumeric);
                    off[j] = 0.0f;
                    cell[j] = 0;
                    vx[j] = vy[j] = vz[j] = 0.0f;
                    if (!UY) p_vy[slot0 + j] = 0.0f;
                    if (!UZ) p_vz[slot0 + j] = 0.0f;
                }
        }
        if (DIAG) {
            float ke_tile = 0.0f;
#pragma unroll
            for (int j = 0; j < PPT; ++j)
                if (keep[j]) ke_tile += ke[j];
            ke_run += ke_tile;
        }
        const int nc = k.nc;
        if (k.periodic) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                int c = cell[j];
                c += c < 0 ? nc : (c >= nc ? -nc : 0);
                const bool out = (unsigned)c >= (unsigned)nc;       // moved more than the domain
                cell[j] = out ? 0 : c;
                off[j] = out ? 0.0f : off[j];
                bad |= keep[j] && out;
            }
        } else {
            bool walls = false;
#pragma unroll
            for (int j = 0; j < PPT; ++j) walls |= keep[j] && (unsigned)cell[j] >= (unsigned)nc;
            if (__any(walls)) {
                CSeg& sc = const_seg(d, sg);
#pragma unroll
                for (int j = 0; j < PPT; ++j) {
                    if (!(keep[j] && (unsigned)cell[j] >= (unsigned)nc)) continue;
                    const int wall = cell[j] < 0 ? 0 : 1;
                    // components the push does not carry are read for the
                    // few particles that reach a wall
                    const float wy = RY ? vy[j] : p_vy[slot0 + j];
                    const float wz = RZ ? vz[j] : p_vz[slot0 + j];
                    const float vnew2 = vx[j] * vx[j] + wy * wy + wz * wz;
                    const float eps = sc.half_m_over_e * vnew2;
                    atomicAdd(&s_cnt[C_ABS0 + wall], 1u);
                    atomicAdd(&s_wen[wall], fixed_u64(eps * 1048576.0f));
                    if (DIAG) {
                        // impact energy: this species' histogram at this
                        // wall, and for electrons the wall energy distribution
                        const int wb = (int)(eps * sc.wedf_inv_bin);
                        if ((unsigned)wb < (unsigned)kEepfBins)
                            atomicAdd(&d.wedf[((size_t)sg * 2 + wall) * kEepfBins + wb], 1ull);
                        const int bin = (int)(eps * a.eepf_inv_bin);
                        if (s == 0 && (unsigned)bin < (unsigned)kEepfBins)
                            atomicAdd(&d.eepf[((size_t)b * 2 + 1) * kEepfBins + bin], 1ull);
                    }
                    if (GENERAL && k.emits) evw[j] = kEvSee | (wall ? kEvWall1 : 0u);
                    keep[j] = false;
                }
            }
        }
        if (__any(bad)) {
            if (bad) atomicOr(&d.diss[b].flags, kFlagCell);
        }
        if (GENERAL && k.nch > 0) {
            // null-collision Monte Carlo: integer candidate test on the first draw
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const bool cand = candidate_draw(pid[j], k, s) < k.t32;
                evw[j] |= keep[j] && cand ? kEvCand : 0u;
            }
        }
        if (renews) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                if (!keep[j]) continue;
                // past L_z the particle gets a fresh velocity from its
                // species' initial distribution at the same x (events pass)
                const double zz = zax[j] + (double)vz[j] * k.dt_d;
                if (fabs(zz) >= k.renew_lz) {
                    evw[j] |= kEvRenew;
                    zax[j] = 0.0;
                    atomicAdd(&s_cnt[C_REN], 1u);
                } else {
                    zax[j] = zz;
                }
            }
        }
        // Deposit and samples.  A thread's consecutive particles often share a
        // cell where the species is cold or was loaded in order (ions keep
        // their order for long): those add once.  Atomics of one address
        // serialise, so without this a sampled tile of ordered ions takes 17 us
        // on 4 x 1024 tiles where electrons, spread over the mesh, take 7.
        bool same = PPT > 1 && keep[0];
#pragma unroll
        for (int j = 1; j < PPT; ++j) same = same && keep[j] && cell[j] == cell[0];
        if (same) {
            unsigned long long w = 0ull;
#pragma unroll
            for (int j = 0; j < PPT; ++j) w += dep_word(off[j]);
            atomicAdd(&hist[cell[0]], w);
        } else {
#pragma unroll
            for (int j = 0; j < PPT; ++j)
                if (keep[j]) atomicAdd(&hist[cell[j]], dep_word(off[j]));
        }
        if (DIAG) {
            // with the velocity of the push: the events pass adds what a
            // collision changes
            Sampled t{0ull, 0ull, 0ull, 0ull, 0ull, 0ull};
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                if (!keep[j]) continue;
                const int c1 = right_node(cell[j], nc, k.periodic);
                Sampled v;
                moment_words(k.mscale1, k.mscale2, off[j], vx[j], v);
                if (same) {
                    t.f0 += v.f0;
                    t.f1 += v.f1;
                    t.m0 += v.m0;
                    t.m1 += v.m1;
                } else {
                    add_moments(fhist, mhist, cell[j], c1, v);
                }
                if (s == 0) {
                    const float eps = k.hme * (vx[j] * vx[j] + vy[j] * vy[j] + vz[j] * vz[j]);
                    energy_words(eps, off[j], v);
                    if (same) {
                        t.e0 += v.e0;
                        t.e1 += v.e1;
                    } else {
                        add_energy(ehist, cell[j], c1, v);
                    }
                    add_bulk(eepf, a.eepf_inv_bin, eps, cell[j], k.bulk_lo, k.bulk_hi);
                }
            }
            if (same) {
                const int c1 = right_node(cell[0], nc, k.periodic);
                add_moments(fhist, mhist, cell[0], c1, t);
                if (s == 0) add_energy(ehist, cell[0], c1, t);
            }
        }
        // absorbed particles leave holes, holes stay
        if (GENERAL) {
#pragma unroll
            for (int j = 0; j < PPT; ++j) cell[j] = keep[j] ? cell[j] : -1;
        }

        // in place; every particle keeps its slot
        if (slot0 + PPT <= rem) {
            vstore<PPT, int4, GENERAL>(p_cell + slot0, cell);
            vstore<PPT, float4, GENERAL>(p_off + slot0, off);
            vstore<PPT, float4, GENERAL>(p_vx + slot0, vx);
            if (UY) vstore<PPT, float4, GENERAL>(p_vy + slot0, vy);
            if (UZ) vstore<PPT, float4, GENERAL>(p_vz + slot0, vz);
        } else {
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                if (slot0 + j < rem) {
                    p_cell[slot0 + j] = cell[j];
                    p_off[slot0 + j] = off[j];
                    p_vx[slot0 + j] = vx[j];
                    if (UY) p_vy[slot0 + j] = vy[j];
                    if (UZ) p_vz[slot0 + j] = vz[j];
                }
            }
        }
        if (renews) {
#pragma unroll
            for (int j = 0; j < PPT; ++j)
                if (slot0 + j < rem) p_z[tile0 + slot0 + j] = zax[j];
        }
        if (GENERAL) {
            // this wave's events, appended to the workgroup's packed list at
            // a place one LDS atomic per wave claims (no barrier): the order
            // of the records does not matter, each is self-contained and
            // every result of the events pass is independent of it
            uint32_t below = 0, total = 0;
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const uint64_t m = __ballot(evw[j] != 0u);
                below += lanes_below(m);
                total += (uint32_t)__popcll(m);
            }
            if (total) {
                uint32_t wbase = 0;
                if (lane == 0) wbase = atomicAdd(&s_evn, total);
                wbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)wbase);
                // the particle after the push: slot, event bits, id, velocity,
                // position and tile, so the events pass reads the record only
                const size_t r0 = (size_t)t_begin * T;
                uint32_t at = wbase + below;
#pragma unroll
                for (int j = 0; j < PPT; ++j) {
                    if (evw[j]) {
                        const uint4 rec = make_uint4(evw[j] | (uint32_t)(slot0 + j) | ((uint32_t)sg << kEvSegShift),
                                                     pid[j], __float_as_uint(vx[j]), __float_as_uint(vy[j]));
                        const uint4 rq = make_uint4(__float_as_uint(vz[j]), (uint32_t)cell[j],
                                                    __float_as_uint(off[j]), (uint32_t)t);
                        if (FUSE && at < kEvLds) {
                            s_rec[at] = rec;
                            s_rq[at] = rq;
                        } else {
                            d.evr[r0 + at] = rec;
                            d.evq[r0 + at] = rq;
                        }
                        ++at;
                    }
                }
            }
            if (tid == 0) d.bcnt[t] = 0;   // the events pass counts this tile's births
        }
        if (tid == 0 && t == seg_end - 1) {
            d.segs[sg].tile_first = seg_first;
            d.segs[sg].ntiles = seg_end - seg_first;
        }
    }
    if (!GENERAL) {
        lds_barrier();
        flush(0);
        return;
    }
    __syncthreads();                              // every wave's records are written
    const uint32_t nev = s_evn;
    // with fewer chunks of events than waves (FUSE), the first waves run
    // them while the others flush the deposit: each wave waits only on its
    // own memory operations, so the events pass does not wait for the
    // flush's atomics to complete
    const uint32_t nch = FUSE ? (nev + 63u) >> 6 : 0u;
    const int quiet = nch < (uint32_t)kWavesPerTile ? (int)nch * 64 : 0;
    flush(quiet);
    if (tid == kBS - 1) d.evg[blockIdx.x] = nev;  // the events pass's count of this range
    if (FUSE) {
        // this workgroup's own events, in chunks of 64 over its waves:
        // the same pass as the events kernel's, on the records and the
        // tiles this workgroup has just written
        const EvPass ps{T, chunk, (uint32_t)births_per_tile(T, true), DIAG, a.eepf_inv_bin,
                        (RY ? kUseY : 0) | (RZ ? kUseZ : 0)};
        for (uint32_t kc = (uint32_t)wid; kc < nch; kc += (uint32_t)kWavesPerTile) {
            uint4 rec, rq;
            bool act;
            if (kc * 64u + 64u <= kEvLds) {
                const uint32_t e = kc * 64u + (uint32_t)lane;
                act = e < nev;
                if (act) {
                    rec = s_rec[e];
                    rq = s_rq[e];
                }
            } else {
                act = event_record(d, ps, (int)blockIdx.x, nev, kc, rec, rq);
            }
            event_chunk(d, s_pref, ps, act, rec, rq, sg, seg_first, base_p, stride);
        }
    }
}

namespace {

// The collision of a candidate, in FP64: the energy (electrons: target at
// rest; ions: relative to a neutral drawn from the gas), the channel by the
// running sum of the tabulated frequencies against the second word of the
// first draw, then the kinematics of the channel.  Returns the channel (-1:
// null collision); `viol` says whether the summed frequency exceeded the
// bound, `born` whether an ionization filled the velocities of `bb` (the
// ejected electron and the new ion; the caller places them at the parent's
// position).
__device__ __forceinline__ int collide_particle(CSeg& sc, CDis& dc, int s, uint32_t step,
                                                double& ux, double& uy, double& uz, uint32_t pid, Birth& bb,
                                                bool& viol, bool& born)
{
    const uint4 r = philox10(pid, step, ((uint32_t)s << 24), 0u, dc.key0, dc.key1);
    double speed, eps;
    double nvx = 0.0, nvy = 0.0, nvz = 0.0;
    if (!sc.ion_type) {
        const double v2 = ux * ux + uy * uy + uz * uz;
        speed = sqrt(v2);
        eps = sc.half_m_over_e_d * v2;
    } else {
        const uint4 r3 = philox10(pid, step, ((uint32_t)s << 24) | 3u, 0u, dc.key0, dc.key1);
        double g0, g1, g2, g3;
        box_muller_d(u01d(r3.x), u01d(r3.y), g0, g1);
        box_muller_d(u01d(r3.z), u01d(r3.w), g2, g3);
        nvx = sc.vt_gas * g0;
        nvy = sc.vt_gas * g1;
        nvz = sc.vt_gas * g2;
        const double gx = ux - nvx, gy = uy - nvy, gz = uz - nvz;
        const double g2s = gx * gx + gy * gy + gz * gz;
        speed = sqrt(g2s);
        eps = sc.half_m_over_e_d * g2s;
    }
    // channel: the first k whose running sum of n_g sigma_k g / nu_max passes
    // u1, one pass over the table row (the full sum checks the bound).  The
    // row's entries are read four at a time, all in flight together, and the
    // channel's kind and threshold are kept from the pass: no chain of reads.
    const double u1 = u01d(r.y);
    double cum = 0.0, th = 0.0;
    int ch = -1, kind = 0;
    {
        const double lx = (log(fmax(eps, 1e-300)) - sc.xs_ln0) * sc.xs_inv_dln;
        int i;
        double fr;
        if (!(lx > 0.0)) {
            i = 0;
            fr = 0.0;
        } else if (lx >= (double)(sc.xs_n - 1)) {
            i = sc.xs_n - 2;
            fr = 1.0;
        } else {
            i = (int)lx;
            if (i > sc.xs_n - 2) i = sc.xs_n - 2;
            fr = lx - (double)i;
        }
        const PIC_GLOBAL double* r0 = (const PIC_GLOBAL double*)sc.xs + (size_t)i * sc.nch;
        const PIC_GLOBAL double* r1 = r0 + sc.nch;
        const int nch = sc.nch;
        constexpr int kGroup = 4;
        static_assert(kMaxChan % kGroup == 0, "thresholds are read in whole groups");
        for (int k0 = 0; k0 < nch; k0 += kGroup) {
            double a0[kGroup], a1[kGroup], tk[kGroup];
            int kd[kGroup];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const int k = k0 + q < nch ? k0 + q : nch - 1;
                a0[q] = r0[k];
                a1[q] = r1[k];
                tk[q] = sc.th[k0 + q];
                kd[q] = sc.kind[k0 + q];
            }
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                if (k0 + q >= nch) break;                 // uniform
                const double v = a0[q] + fr * (a1[q] - a0[q]);
                cum += ((eps < tk[q]) ? 0.0 : v) * speed;
                if (ch < 0 && u1 < cum) {
                    ch = k0 + q;
                    kind = kd[q];
                    th = tk[q];
                }
            }
        }
    }
    viol = cum > 1.0;
    born = false;
    if (ch < 0) return -1;
    const double cos_chi = 1.0 - 2.0 * u01d(r.z);
    const double u_phi = u01d(r.w);           // azimuth 2 pi u_phi
    if (!sc.ion_type) {
        const double inv = 1.0 / speed;
        const double dx_ = ux * inv, dy_ = uy * inv, dz_ = uz * inv;
        double ndx, ndy, ndz;
        scatter_dir_d(dx_, dy_, dz_, cos_chi, u_phi, ndx, ndy, ndz);
        double enew;
        if (kind == PIC_XS_ELASTIC) {
            enew = eps * (1.0 - sc.mr2 * (1.0 - cos_chi));
        } else if (kind == PIC_XS_EXCITATION) {
            enew = eps - th;
        } else {
            const uint4 r1 = philox10(pid, step, ((uint32_t)s << 24) | 1u, 0u, dc.key0, dc.key1);
            const uint4 r2 = philox10(pid, step, ((uint32_t)s << 24) | 2u, 0u, dc.key0, dc.key1);
            const double avail = eps - th;
            const double eej = u01d(r1.x) * avail;
            enew = avail - eej;
            double edx, edy, edz;
            scatter_dir_d(dx_, dy_, dz_, 1.0 - 2.0 * u01d(r1.y), u01d(r1.z), edx, edy, edz);
            const double vej = sqrt(sc.two_e_over_m * eej);
            double g0, g1, g2, g3;
            box_muller_d(u01d(r2.x), u01d(r2.y), g0, g1);
            box_muller_d(u01d(r2.z), u01d(r2.w), g2, g3);
            bb.vx = (float)(vej * edx);
            bb.vy = (float)(vej * edy);
            bb.vz = (float)(vej * edz);
            bb.ivx = (float)(sc.vt_gas * g0);
            bb.ivy = (float)(sc.vt_gas * g1);
            bb.ivz = (float)(sc.vt_gas * g2);
            born = true;
        }
        enew = fmax(enew, 0.0);
        const double vs = sqrt(sc.two_e_over_m * enew);
        ux = vs * ndx;
        uy = vs * ndy;
        uz = vs * ndz;
    } else if (kind == PIC_XS_ION_CX) {
        ux = nvx;
        uy = nvy;
        uz = nvz;
    } else {
        const double cmx = sc.m_frac * ux + sc.M_frac * nvx;
        const double cmy = sc.m_frac * uy + sc.M_frac * nvy;
        const double cmz = sc.m_frac * uz + sc.M_frac * nvz;
        const double st_ = sqrt(fmax(0.0, 1.0 - cos_chi * cos_chi));
        double sp_, cp_;
        sincospi(2.0 * u_phi, &sp_, &cp_);
        const double gg = sc.M_frac * speed;
        ux = cmx + gg * cos_chi;
        uy = cmy + gg * st_ * cp_;
        uz = cmz + gg * st_ * sp_;
    }
    return ch;
}

// The secondary electron of an ion absorbed at `wall`, in FP64: emitted with
// probability gamma (integer test on the draw), normal speed from the
// flux-weighted half-Maxwellian, tangential components Maxwellian, placed
// u v_n dt into the gap.  Returns 1 with `bb` filled when one is placed,
// -1 when one is emitted but lands beyond the gap, 0 when none is emitted.
__device__ __forceinline__ int secondary(CSeg& sc, CDis& dc, int s, uint32_t step, int wall,
                                         uint32_t pid, Birth& bb)
{
    const uint4 r4 = philox10(pid, step, ((uint32_t)s << 24) | 4u, 0u, dc.key0, dc.key1);
    if (!(odd24(r4.x) < sc.see_k)) return 0;
    const uint4 r5 = philox10(pid, step, ((uint32_t)s << 24) | 5u, 0u, dc.key0, dc.key1);
    const int nc = dc.n_cells;
    const double vn = sc.vsee * sqrt(-2.0 * log(u01d(r4.y)));
    const double adv = u01d(r4.z) * vn * sc.dtdx_e;         // cells
    double g0, g1;
    box_muller_d(u01d(r5.x), u01d(r5.y), g0, g1);
    if (!(adv < (double)nc)) return -1;
    const double pos = wall == 0 ? adv : (double)nc - adv;   // cells from x = 0
    const double cf = floor(pos);
    int cell = (int)cf;
    float off = (float)(pos - cf);
    if (off >= 1.0f) {                   // the edge rule
        off -= 1.0f;
        cell += 1;
    }
    if (cell >= nc) {                    // within rounding of x = L: the last representable offset
        cell = nc - 1;
        off = 0x1.fffffep-1f;
    }
    if (cell < 0) return -1;
    bb.cell = cell;
    bb.off = off;
    bb.vx = (float)(wall == 0 ? vn : -vn);
    bb.vy = (float)(sc.vsee * g0);
    bb.vz = (float)(sc.vsee * g1);
    bb.ivx = bb.ivy = bb.ivz = 0.0f;
    return 1;
}

__device__ __forceinline__ uint32_t popc_ballot(bool p) { return (uint32_t)__popcll(__ballot(p)); }

}  // namespace

// This lane's event of chunk kc (events 64 kc .. 64 kc + 63) of the nev that
// push workgroup g recorded: its two record words; false past the list's end.
__device__ __forceinline__ bool event_record(const DevPtrs& d, const EvPass& ps, int g, uint32_t nev, uint32_t kc,
                                             uint4& rec, uint4& rq)
{
    const uint32_t e = (kc << 6) + (uint32_t)(threadIdx.x & 63);
    if (e >= nev) return false;
    const size_t ri = (size_t)g * ps.chunk_t * ps.T + e;
    rec = d.evr[ri];
    rq = d.evq[ri];
    return true;
}

// The events pass on one chunk: lanes with `act` hold an event's records.  One
// segment at a time (a chunk spans more than one only at a segment's end), so
// its constants are read once for the wave, all in one round.  k_sg: a segment
// the caller knows the place of (first tile, particle arrays and their
// distance), or -1.  s_pref: the segments' first tiles, or null after the push
// has ended, which leaves them in the segments' states.
__device__ __forceinline__ void event_chunk(const DevPtrs& d, const int32_t* s_pref, const EvPass& ps, bool act,
                                            uint4 rec, uint4 rq, int k_sg, int32_t k_first, char* k_base,
                                            int64_t k_stride)
{
    const int S = d.S;
    const int lane = threadIdx.x & 63;
    const uint32_t word = act ? rec.x : 0u;
    uint64_t todo = __ballot(act);
    while (todo) {
        const int sg =
            (int)((uint32_t)__builtin_amdgcn_readlane((int)word, __ffsll((long long)todo) - 1) >> kEvSegShift);
        const bool mine = act && (int)(word >> kEvSegShift) == sg;
        todo &= ~__ballot(mine);
        const int b = seg_discharge(sg, S), s = sg - b * S;
        CDis& dc = const_dis(d, b);
        CSeg& sc = const_seg(d, sg);
        const int nc = dc.n_cells;
        const int periodic = dc.bc == PIC_BC_PERIODIC;
        const uint32_t step = const_step(d, b);
        int64_t stride = k_stride;
        char* base = k_base;
        int32_t first = k_first;
        if (sg != k_sg) {
            const PIC_CONST SegState& st = const_state(d, sg);
            stride = st.stride;
            base = st.base + (int64_t)st.parity * kFields * stride;
            first = s_pref ? s_pref[sg] : (int32_t)st.tile_first;
        }
        const int nch = sc.nch;
        bool hb = false, see = false, cand = false, viol = false, lost = false;
        int wall = 0, ch = -1;
        if (mine) {
            const int32_t t = (int32_t)rq.w;
            const uint32_t key = word & kEvSlot;
            PIC_GLOBAL char* at = (PIC_GLOBAL char*)base + ((int64_t)(t - first) * ps.T + key) * 4;   // the particle's slot
            const uint32_t pid = nch > 0 ? rec.y : *(const PIC_GLOBAL uint32_t*)(at + 5 * stride);
            Birth bb;
            if (word & kEvSee) {
                see = true;
                wall = (word & kEvWall1) ? 1 : 0;
                const int r = secondary(sc, dc, s, step, wall, pid, bb);
                hb = r > 0;
                lost = r < 0;
            } else {
                double ux = __uint_as_float(rec.z);
                double uy = (ps.vm & kUseY) ? __uint_as_float(rec.w) : *(const PIC_GLOBAL float*)(at + 3 * stride);
                double uz = (ps.vm & kUseZ) ? __uint_as_float(rq.x) : *(const PIC_GLOBAL float*)(at + 4 * stride);
                if (word & kEvRenew) {
                    const uint4 r6 = philox10(pid, step, ((uint32_t)s << 24) | 6u, 0u, dc.key0, dc.key1);
                    double g0, g1, g2, g3;
                    box_muller_d(u01d(r6.x), u01d(r6.y), g0, g1);
                    box_muller_d(u01d(r6.z), u01d(r6.w), g2, g3);
                    ux = sc.drift0[0] + sc.vth0 * g0;
                    uy = sc.drift0[1] + sc.vth0 * g1;
                    uz = sc.drift0[2] + sc.vth0 * g2;
                }
                if (word & kEvCand) {
                    cand = true;
                    ch = collide_particle(sc, dc, s, step, ux, uy, uz, pid, bb, viol, hb);
                }
                // the position (the push's, in the record): for an ionization's
                // pair and the diagnostics
                const int c = (int)rq.y;
                const float f = __uint_as_float(rq.z);
                if (hb) {
                    bb.cell = c;
                    bb.off = f;
                }
                const float fx = (float)ux, fy = (float)uy, fz = (float)uz;
                if (ch >= 0 || (word & kEvRenew)) {          // a null collision changes nothing
                    *(PIC_GLOBAL float*)(at + 2 * stride) = fx;
                    *(PIC_GLOBAL float*)(at + 3 * stride) = fy;
                    *(PIC_GLOBAL float*)(at + 4 * stride) = fz;
                    if (ps.diag)                             // the push sampled the velocity of the record
                        sample_change(d, sc, dc, b, sg, s == 0, ps.eepf_inv_bin, c, f, __uint_as_float(rec.z),
                                      __uint_as_float(rec.w), __uint_as_float(rq.x), fx, fy, fz);
                }
            }
            if (hb) {
                const uint32_t pos = atomicAdd(reinterpret_cast<uint32_t*>(&d.bcnt[t]), 1u);
                if (pos < ps.bpt) {
                    bb.key = key;
                    d.births[(size_t)t * ps.bpt + pos] = bb;
                    unsigned long long* acc_e = d.acc + ((size_t)b * S + 0) * kRep * d.nodes_max;
                    global_deposit(acc_e, bb.cell, bb.off, nc, periodic);
                    if (!see && S > 1)          // no ions in a swarm
                        global_deposit(d.acc + ((size_t)b * S + 1) * kRep * d.nodes_max, bb.cell, bb.off, nc,
                                       periodic);
                    if (ps.diag) {
                        // the births' velocity moments and the electron's
                        // energy, with the particles of the step
                        sample_particle(d, const_seg(d, b * S + 0), dc, b, b * S + 0, true, ps.eepf_inv_bin, bb.cell, bb.off,
                                        bb.vx, bb.vy, bb.vz);
                        if (!see && S > 1)
                            sample_particle(d, const_seg(d, b * S + 1), dc, b, b * S + 1, false, ps.eepf_inv_bin, bb.cell,
                                            bb.off, bb.ivx, bb.ivy, bb.ivz);
                    }
                    atomicAdd(reinterpret_cast<unsigned long long*>(&d.segs[sg].staged), 1ull);
                } else {
                    hb = false;
                    lost = true;
                    atomicOr(&d.diss[b].flags, kFlagCapacity);
                }
            }
        }
        // counters of the segment's events: lane i holds counter i
        uint32_t cnt_lane = 0u;
        auto count = [&](int i, bool p) {
            const uint32_t v = popc_ballot(p);
            cnt_lane += lane == i ? v : 0u;
        };
        count(C_CAND, cand);
        count(C_NULL, cand && ch < 0);
        count(C_VIOL, viol);
        for (int q = 0; q < nch; ++q) count(C_COLL + q, ch == q);
        count(C_SEE0, hb && see && wall == 0);
        count(C_SEE1, hb && see && wall == 1);
        count(C_DROP, lost);
        if (lane < C_N && cnt_lane)
            atomicAdd(&d.cnt[((size_t)sg * kRep) * C_N + lane], (unsigned long long)cnt_lane);
    }
}

}  // namespace pic
