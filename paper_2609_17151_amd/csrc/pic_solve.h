// Pieces of the field solve that the finalize kernel and the streaming push
// share: the nested prefix sums of a mesh, in a fixed order, in FP64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pic_device.h"

namespace pic {

// Prefix state of a run of nodes for the nested sums of the solve: n nodes,
// S = sum of g, P = sum over the run of the running sums of g, Q = sum over
// the run of the running sums of those (Q gives the sum of phi, hence the
// zero-mean gauge, without another reduction).  Appending run B after run A:
// n = nA + nB, S = SA + SB, P = PA + PB + nB SA,
// Q = QA + QB + nB PA + SA nB (nB + 1) / 2.  The all-zero run is the identity.
struct Run {
    double n, S, P, Q;
};

__device__ __forceinline__ Run run_combine(const Run& A, const Run& B)
{
    return Run{A.n + B.n, A.S + B.S, A.P + B.P + B.n * A.S,
               A.Q + B.Q + B.n * A.P + A.S * (0.5 * B.n * (B.n + 1.0))};
}

// DPP move of a double within a wave (zero where the source lane is invalid
// or the destination row is masked off)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v)
{
    const unsigned long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffu), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROW_MASK, 0xf, false);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void run_step(Run& v)
{
    Run o;
    o.n = dpp_f64<CTRL, ROW_MASK>(v.n);
    o.S = dpp_f64<CTRL, ROW_MASK>(v.S);
    o.P = dpp_f64<CTRL, ROW_MASK>(v.P);
    o.Q = dpp_f64<CTRL, ROW_MASK>(v.Q);
    v = run_combine(o, v);
}

// inclusive scan of Run over a wave, lanes in order: row shifts 1, 2, 4, 8
// within each row of 16 lanes, then the last lane of row 0 into rows 1 and 3
// and the last lane of row 1 into rows 2 and 3
__device__ __forceinline__ Run wave_run_scan(Run v)
{
    run_step<0x111, 0xf>(v);   // row_shr:1
    run_step<0x112, 0xf>(v);   // row_shr:2
    run_step<0x114, 0xf>(v);   // row_shr:4
    run_step<0x118, 0xf>(v);   // row_shr:8
    run_step<0x142, 0xa>(v);   // row_bcast:15
    run_step<0x143, 0xc>(v);   // row_bcast:31
    return v;
}

// sum over a wave in a fixed order (the same row shifts and broadcasts; the
// last lane ends with the total), returned to every lane.  The whole wave
// must be active.
__device__ __forceinline__ double wave_total_f64(double v)
{
    v += dpp_f64<0x111, 0xf>(v);
    v += dpp_f64<0x112, 0xf>(v);
    v += dpp_f64<0x114, 0xf>(v);
    v += dpp_f64<0x118, 0xf>(v);
    v += dpp_f64<0x142, 0xa>(v);
    v += dpp_f64<0x143, 0xc>(v);
    const unsigned long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffffu), 63);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), 63);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// the runs of up to four waves in their order: all of them together, and those
// before wave w, in the association of the scan over the waves' totals
__device__ __forceinline__ void few_runs(const Run* s_run, int nw, int w, Run& before, Run& all)
{
    const Run zero{0.0, 0.0, 0.0, 0.0};
    const Run r0 = s_run[0], r1 = nw > 1 ? s_run[1] : zero, r2 = nw > 2 ? s_run[2] : zero,
              r3 = nw > 3 ? s_run[3] : zero;
    const Run p1 = run_combine(r0, r1), p2 = run_combine(r0, run_combine(r1, r2));
    all = run_combine(p1, run_combine(r2, r3));
    before = w == 0 ? zero : (w == 1 ? r0 : (w == 2 ? p1 : p2));
}

}  // namespace pic
