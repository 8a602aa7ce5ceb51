// Warm-start network on the matrix cores: every layer, forward and backward,
// is a BF16 product with FP32 accumulation (v_mfma_f32_16x16x32_bf16) whose
// epilogue applies the elementwise work of the layer.
//
// A layer's parameters are the matrix [n_out][n_in + 1] with the bias as the
// last column; the products see the layer input extended by a column of ones,
// so the bias rides in the product both forward (z = [a 1] Wa^T) and backward
// (dWa = dz^T [a 1], whose last column is the bias gradient).
//
// Every product reads both operands along k in fragments of 16 rows by 32: lane
// l of a wave holds k = 8 (l / 16) .. + 7 of row l % 16.  All operands in memory
// are kept fragment by fragment, 64 lanes of 16 bytes (frag_at), so a load is
// 1 KB of whole cache lines, with zeros in the padding of k: the weights as Wa
// (forward) and W^T (backward), the layer inputs and the output gradients of a
// batch by feature, along the samples, for the weight gradients.  The
// writer of an activation or of an output gradient rounds it to BF16 once;
// its only readers are these products, which take BF16 operands.  Sums run
// over k in ascending blocks of 32, so a result does not depend on the tiling
// or on which of the kernels below formed it.
//
// A training step is two launches.  chain_kernel takes 16 (or 32) samples per
// workgroup through all layers and back, the activations in LDS: the layers
// of one sample depend on each other only, so nothing waits on another
// workgroup, and the 1.3 MB of weights come from L2.  grad_kernel forms the
// weight gradients of all layers (a 16 x 16 tile per wave) and applies Adam
// in the epilogue, so the gradient makes no trip through memory.  What bounds
// them for the 5-256-256-256-768 network on batches of 64: the dependent
// chain of seven products through one compute unit's L2 port (64 bytes per
// cycle), and the launch of two kernels.  Measured there: 33 us per training
// step (chain 25, gradients and Adam 9), 313 us with one tiled kernel per
// product that gathered its operands element by element; prediction of 4096
// samples 15 us instead of 122.  Networks with more weights, on batches too
// small for the chain to fill the GPU, and those whose layers do not fit the
// chain's LDS take one layer_kernel per product (operands straight from the
// cache); the rule and both sides' figures are at use_chain.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "pic_device.h"
#include "pic_mlp.h"

namespace {

// between layers: what goes to global memory there is read by no other wave of
// the kernel (the transposed copies), or back by the lane that wrote it (the
// pre-activations)
using pic::lds_barrier;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxL = PIC_MLP_MAX_LAYERS;
constexpr int kChainThreads = 1024;
constexpr int kChainWaves = kChainThreads / 64;
constexpr int kChainLds = 64 * 1024;       // activations of the chain's rows (no more: use_chain)
constexpr int kPad = 8;                    // LDS row padding: rows land on different banks
constexpr int kAhead = 12;                 // weight fragments in flight per wave

__host__ __device__ constexpr int pad16(int n) { return (n + 15) & ~15; }
__host__ __device__ constexpr int pad32(int n) { return (n + 31) & ~31; }

// element (row, k) of an operand whose rows have `ks` blocks of 32 k
__host__ __device__ __forceinline__ int64_t frag_at(int row, int k, int ks)
{
    return (((int64_t)(row >> 4) * ks + (k >> 5)) * 64 + (row & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

struct Layer {
    int32_t ni, no;        // inputs, outputs
    int32_t kf, kb;        // padded lengths of k: forward (ni + 1), backward (no)
    int64_t off;           // first parameter
    __bf16* wf;            // [pad16(no)][kf] Wa, in fragments
    __bf16* wt;            // [pad16(ni)][kb] W^T, in fragments
    __bf16* at;            // [pad32(ni + 1)][ldb] layer input with its ones by feature, in fragments
    __bf16* dzt;           // [pad16(no)][ldb] output gradient by feature, in fragments
    float* z;              // [batch][no] pre-activation (hidden layers)
};

struct Net {
    int32_t L;
    Layer l[kMaxL];
};

__device__ __forceinline__ float gelu(float z)
{
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// acc[i] += A_i B over KS blocks of 32: A_i from LDS (`a` at the lane's row and
// k, blocks of 16 rows lda apart), B from memory (`b` at the lane's part of its
// first fragment), every load issued before the first product.
template <int MT, int KS>
__device__ __forceinline__ void product_blocks(const __bf16* a, int lda, const __bf16* __restrict__ b, f32x4* acc)
{
    bf16x8 f[KS];
#pragma unroll
    for (int u = 0; u < KS; ++u) f[u] = *reinterpret_cast<const bf16x8*>(b + 512 * u);
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
        for (int i = 0; i < MT; ++i)
            acc[i] = mfma(*reinterpret_cast<const bf16x8*>(a + (size_t)i * 16 * lda + 32 * u), f[u], acc[i]);
}

// ... over ks blocks, kAhead at a time
template <int MT>
__device__ __forceinline__ void product(const __bf16* a, int lda, const __bf16* __restrict__ b, int ks, f32x4* acc)
{
    for (; ks >= kAhead; ks -= kAhead, a += 32 * kAhead, b += 512 * kAhead) product_blocks<MT, kAhead>(a, lda, b, acc);
#define PIC_REST(K) case K: product_blocks<MT, K>(a, lda, b, acc); break;
    switch (ks) {
        PIC_REST(1) PIC_REST(2) PIC_REST(3) PIC_REST(4) PIC_REST(5) PIC_REST(6)
        PIC_REST(7) PIC_REST(8) PIC_REST(9) PIC_REST(10) PIC_REST(11) default: break;
    }
#undef PIC_REST
}

struct ChainArgs {
    Net net;
    int32_t M, ld, ldb;    // samples, LDS row, samples padded to 32 (rows of at and dzt)
    const float* x;
    const float* t;        // targets (training)
    float* y;              // outputs (forward only)
    float scale;           // of the output gradient
    float* loss_part;      // one partial sum of squares per workgroup
    int32_t rows_wg;       // workgroups that take samples; the others warm the caches
    const uint4* weights;  // every layer's BF16 weights, n_weights x 16 bytes
    int32_t n_weights;
};

// Workgroups 8 h + x, h >= 1, run beside those that take samples and read the
// weights into the L2 cache of XCD x (workgroups go round the eight XCDs in
// turn).  After an update the weights are in no XCD's L2, and a batch of a few
// row blocks has one workgroup per XCD to fetch 1.4 MB through one compute
// unit's misses.  Only a matter of speed: nothing depends on where a
// workgroup runs.
constexpr int kXcd = 8;
constexpr int kWarmers = 16;                 // workgroups per XCD
constexpr int kWarmRows = 64;                // row blocks up to which they run: with eight per XCD and more the
                                             // blocks warm the cache for each other.  Measured, us per step: 1 block
                                             // 33.5 -> 28.9, 4 blocks 38.1 -> 33.0, 64 blocks 43.3 -> 42.1, 256
                                             // blocks 60.2 -> 61.1

// MT blocks of 16 samples per workgroup through the whole network; TRAIN: and
// back, leaving every layer's input and output gradient in BF16 for
// grad_kernel.  Rows past M carry zero inputs and zero gradients.
template <int MT, bool TRAIN>
__global__ __launch_bounds__(kChainThreads) void chain_kernel(ChainArgs g)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float s_red[kChainWaves];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int fr = lane & 15, fk = (lane >> 4) * 8, rq = (lane >> 4) * 4;
    constexpr int R = 16 * MT;
    const int ld = g.ld, m0 = (int)blockIdx.x * R;
    __bf16* cur = reinterpret_cast<__bf16*>(smem);
    __bf16* nxt = cur + (size_t)R * ld;
    const int L = g.net.L;
    if ((int)blockIdx.x >= g.rows_wg) {
        const int x = (int)blockIdx.x % kXcd, h = (int)blockIdx.x / kXcd - (g.rows_wg + kXcd - 1) / kXcd;
        if (x >= g.rows_wg || h < 0) return;
        uint32_t v = 0u;
        for (int i = h * kChainThreads + tid; i < g.n_weights; i += kWarmers * kChainThreads) v |= g.weights[i].x;
        asm volatile("" ::"v"(v));           // keep the loads
        return;
    }

    // the input rows, their ones and the padding
    {
        const Layer& l0 = g.net.l[0];
        for (int i = tid; i < R * l0.kf; i += kChainThreads) {
            const int r = i / l0.kf, c = i - r * l0.kf;
            float v = 0.0f;
            if (c < l0.ni) {
                if (m0 + r < g.M) v = g.x[(int64_t)(m0 + r) * l0.ni + c];
            } else if (c == l0.ni) {
                v = 1.0f;
            }
            cur[(size_t)r * ld + c] = (__bf16)v;
            if (TRAIN && c <= l0.ni) l0.at[frag_at(c, m0 + r, g.ldb / 32)] = (__bf16)v;
        }
    }
    __syncthreads();

    float sq = 0.0f;
    for (int l = 0; l < L; ++l) {
        const Layer& y = g.net.l[l];
        const bool last = l == L - 1;
        const int no = y.no, kn = last ? (TRAIN ? y.kb : no) : g.net.l[l + 1].kf;
        for (int t = wid; t < pad16(no) / 16; t += kChainWaves) {
            f32x4 acc[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            product<MT>(cur + (size_t)fr * ld + fk, ld, y.wf + (int64_t)t * 16 * y.kf + lane * 8, y.kf / 32, acc);
            const int n = t * 16 + fr;
            if (n >= no) continue;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = i * 16 + rq + r, m = m0 + row;
                    const float v = acc[i][r];
                    float w;
                    if (!last) {
                        if (TRAIN && m < g.M) y.z[(int64_t)m * no + n] = v;
                        w = gelu(v);
                    } else if (TRAIN) {
                        float d = 0.0f;
                        if (m < g.M) {
                            d = v - g.t[(int64_t)m * no + n];
                            sq += d * d;
                        }
                        w = g.scale * d;
                    } else {
                        if (m < g.M) g.y[(int64_t)m * no + n] = v;
                        continue;
                    }
                    o[r] = (__bf16)w;
                    nxt[(size_t)row * ld + n] = o[r];
                }
                if (TRAIN)
                    *reinterpret_cast<bf16x4*>((last ? y.dzt : g.net.l[l + 1].at) +
                                               frag_at(n, m0 + i * 16 + rq, g.ldb / 32)) = o;
            }
        }
        // the ones and the padding of the next product's rows
        for (int i = tid; i < R * (kn - no); i += kChainThreads) {
            const int r = i / (kn - no), c = no + (i - r * (kn - no));
            const __bf16 v = (__bf16)(!last && c == no ? 1.0f : 0.0f);
            nxt[(size_t)r * ld + c] = v;
            if (TRAIN && !last && c == no) g.net.l[l + 1].at[frag_at(c, m0 + r, g.ldb / 32)] = v;
        }
        lds_barrier();
        __bf16* s = cur;
        cur = nxt;
        nxt = s;
    }
    if (!TRAIN) return;

    // the output gradients of the layers below: dz = (dz W) g'(z)
    for (int l = L - 1; l > 0; --l) {
        const Layer& y = g.net.l[l];
        const Layer& p = g.net.l[l - 1];
        const int ni = y.ni;
        for (int t = wid; t < pad16(ni) / 16; t += kChainWaves) {
            const int n = t * 16 + fr;
            float z[MT][4];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = m0 + i * 16 + rq + r;
                    z[i][r] = (n < ni && m < g.M) ? p.z[(int64_t)m * ni + n] : 0.0f;
                }
            f32x4 acc[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            product<MT>(cur + (size_t)fr * ld + fk, ld, y.wt + (int64_t)t * 16 * y.kb + lane * 8, y.kb / 32, acc);
            if (n >= ni) continue;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = i * 16 + rq + r;
                    o[r] = (__bf16)(m0 + row < g.M ? acc[i][r] * gelu_grad(z[i][r]) : 0.0f);
                    nxt[(size_t)row * ld + n] = o[r];
                }
                *reinterpret_cast<bf16x4*>(p.dzt + frag_at(n, m0 + i * 16 + rq, g.ldb / 32)) = o;
            }
        }
        for (int i = tid; i < R * (p.kb - ni); i += kChainThreads) {
            const int r = i / (p.kb - ni);
            nxt[(size_t)r * ld + ni + (i - r * (p.kb - ni))] = (__bf16)0.0f;
        }
        lds_barrier();
        __bf16* s = cur;
        cur = nxt;
        nxt = s;
    }
    // fixed-order reduction of the squares: lanes by butterfly, waves in order
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) s_red[wid] = sq;
    __syncthreads();
    if (tid == 0) {
        float t = 0.0f;
        for (int w = 0; w < kChainWaves; ++w) t += s_red[w];
        g.loss_part[blockIdx.x] = t;
    }
}

enum { LAYER_HIDDEN = 0, LAYER_OUT = 1, LAYER_LOSS = 2, LAYER_BACK = 3 };

struct LayerArgs {
    int32_t epi, M, N, K;  // samples, outputs of the product, padded k
    int32_t train, ldb;
    const __bf16* a;       // [pad64(M)][K] rows of the product, in fragments
    const __bf16* b;       // [pad16(N)][K], in fragments
    __bf16* next;          // rows of the next product, [pad64(M)][kn], in fragments
    __bf16* next_t;        // the same by feature, [kn][ldb], in fragments (training)
    int32_t kn, one;       // its padded k; the column that holds ones (-1: none)
    float* z;              // HIDDEN: pre-activation out; BACK: in; OUT: outputs
    const float* t;
    float scale;
    float* loss_part;
};

// One product, WAVES waves of 16 TM x 16 TN outputs per workgroup, 2 x 2 where
// there are four, with the same epilogues.
template <int TM, int TN, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void layer_kernel(LayerArgs g)
{
    __shared__ float s_red[WAVES];
    constexpr int kG = TM * TN > 1 ? 4 : 8;              // blocks of 32 k in flight
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int fr = lane & 15, rq = (lane >> 4) * 4;
    const int m0 = ((int)blockIdx.y * (WAVES > 1 ? 2 : 1) + (wid >> 1)) * 16 * TM;
    const int n0 = ((int)blockIdx.x * (WAVES > 1 ? 2 : 1) + (wid & 1)) * 16 * TN;
    const int last = pad16(g.N) / 16 - 1;
    const __bf16 *pa[TM], *pb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) pa[i] = g.a + (int64_t)(m0 / 16 + i) * 16 * g.K + lane * 8;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 / 16 + j;                       // columns past N are discarded
        pb[j] = g.b + (int64_t)(n < last ? n : last) * 16 * g.K + lane * 8;
    }
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int ks = g.K / 32;
    bf16x8 fa[kG][TM], fb[kG][TN];
    auto fetch = [&](int u, int k) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[u][i] = *reinterpret_cast<const bf16x8*>(pa[i] + 512 * k);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[u][j] = *reinterpret_cast<const bf16x8*>(pb[j] + 512 * k);
    };
#pragma unroll
    for (int u = 0; u < kG; ++u)
        if (u < ks) fetch(u, u);
    for (int k = 0; k < ks; k += kG) {
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            if (k + u < ks) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = mfma(fa[u][i], fb[u][j], acc[i][j]);
                if (k + u + kG < ks) fetch(u, k + u + kG);
            }
        }
    }
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + j * 16 + fr, mr = m0 + i * 16 + rq;
            bf16x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = mr + r;
                const int64_t ci = (int64_t)m * g.N + n;
                const float v = acc[i][j][r];
                float w = n == g.one ? 1.0f : 0.0f;
                if (m < g.M && n < g.N) {
                    if (g.epi == LAYER_HIDDEN) {
                        if (g.train) g.z[ci] = v;
                        w = gelu(v);
                    } else if (g.epi == LAYER_OUT) {
                        g.z[ci] = v;
                    } else if (g.epi == LAYER_LOSS) {
                        const float d = v - g.t[ci];
                        sq += d * d;
                        w = g.scale * d;
                    } else {
                        w = v * gelu_grad(g.z[ci]);
                    }
                }
                o[r] = (__bf16)w;
                if (g.next && n < g.kn) g.next[frag_at(m, n, g.kn / 32)] = o[r];
            }
            if (g.train && mr < g.ldb && (n < g.N || n == g.one))
                *reinterpret_cast<bf16x4*>(g.next_t + frag_at(n, mr, g.ldb / 32)) = o;
        }
    if (g.epi == LAYER_LOSS) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o, 64);
        if (lane == 0) s_red[wid] = sq;
        __syncthreads();
        if (tid == 0) {
            float t = 0.0f;
            for (int w = 0; w < WAVES; ++w) t += s_red[w];
            g.loss_part[blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// the input rows of the first layer_kernel: BF16 with their ones and padding,
// and the same by feature
__global__ __launch_bounds__(256) void input_kernel(const float* x, int M, int rows, int ni, int kf, __bf16* out,
                                                    __bf16* at, int ldb)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (int64_t)rows * kf; i += (int64_t)gridDim.x * 256) {
        const int m = (int)(i / kf), c = (int)(i - (int64_t)m * kf);
        const float v = c < ni ? (m < M ? x[(int64_t)m * ni + c] : 0.0f) : (c == ni ? 1.0f : 0.0f);
        out[frag_at(m, c, kf / 32)] = (__bf16)v;
        if (at && m < ldb && c <= ni) at[frag_at(c, m, ldb / 32)] = (__bf16)v;
    }
}

struct GradArgs {
    Net net;
    int32_t first[kMaxL + 1];      // first wave of every layer's tiles
    int32_t ldb;
    float *w, *m, *v;              // Adam: master weights and moments
    float* grad;                   // without an update: the gradient
    float lr, b1, b2, eps, c1, c2;
    const float* loss_part;
    int32_t parts;
    float inv_count;
    float *loss, *loss2;
};

// dWa = dz^T [a 1] of every layer, a 16 x 16 tile per wave, and Adam's update
// of its parameters (ADAM) or the gradient itself.  The last workgroup sums
// the loss.
template <bool ADAM>
__global__ __launch_bounds__(256) void grad_kernel(GradArgs g)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        // the loss partials in a fixed order, in FP64
        __shared__ double s[256];
        double t = 0.0;
        for (int i = tid; i < g.parts; i += 256) t += (double)g.loss_part[i];
        s[tid] = t;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if (tid < w) s[tid] += s[tid + w];
            __syncthreads();
        }
        if (tid == 0) {
            const float v = (float)(s[0] * (double)g.inv_count);
            g.loss[0] = v;
            if (g.loss2) g.loss2[0] = v;
        }
        return;
    }
    const int task = (int)blockIdx.x * 4 + wid;
    if (task >= g.first[g.net.L]) return;
    int li = 0;
    while (task >= g.first[li + 1]) ++li;
    const Layer& y = g.net.l[li];
    const int nt = pad16(y.ni + 1) / 16, local = task - g.first[li];
    const int mt = local / nt, m0 = mt * 16, n0 = (local - mt * nt) * 16;
    const int n = n0 + (lane & 15), mr = m0 + (lane >> 4) * 4;
    float w[4], mm[4], vv[4];
    if (ADAM) {                    // in flight with the operands
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (mr + r < y.no && n <= y.ni) {
                const int64_t i = y.off + (int64_t)(mr + r) * (y.ni + 1) + n;
                w[r] = g.w[i];
                mm[r] = g.m[i];
                vv[r] = g.v[i];
            }
        }
    }
    const __bf16* pa = y.dzt + (int64_t)m0 * g.ldb + lane * 8;
    const __bf16* pb = y.at + (int64_t)n0 * g.ldb + lane * 8;
    f32x4 acc{0.0f, 0.0f, 0.0f, 0.0f};
    int ks = g.ldb / 32;
    constexpr int kG = 4;          // blocks of 32 samples in flight
    for (; ks >= kG; ks -= kG, pa += 512 * kG, pb += 512 * kG) {
        bf16x8 fa[kG], fb[kG];
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            fa[u] = *reinterpret_cast<const bf16x8*>(pa + 512 * u);
            fb[u] = *reinterpret_cast<const bf16x8*>(pb + 512 * u);
        }
#pragma unroll
        for (int u = 0; u < kG; ++u) acc = mfma(fa[u], fb[u], acc);
    }
    for (; ks > 0; --ks, pa += 512, pb += 512)
        acc = mfma(*reinterpret_cast<const bf16x8*>(pa), *reinterpret_cast<const bf16x8*>(pb), acc);
    bf16x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = mr + r;
        o[r] = (__bf16)0.0f;
        if (m >= y.no || n > y.ni) continue;
        const int64_t i = y.off + (int64_t)m * (y.ni + 1) + n;
        const float gi = acc[r];
        if (ADAM) {
            const float mi = g.b1 * mm[r] + (1.0f - g.b1) * gi;
            const float vi = g.b2 * vv[r] + (1.0f - g.b2) * gi * gi;
            g.m[i] = mi;
            g.v[i] = vi;
            const float wi = w[r] - g.lr * (mi * g.c1) / (sqrtf(vi * g.c2) + g.eps);
            g.w[i] = wi;
            o[r] = (__bf16)wi;
            y.wf[frag_at(m, n, y.kf / 32)] = o[r];
        } else {
            g.grad[i] = gi;
        }
    }
    // rows past n_out lie in the padding of W^T and stay zero
    if (ADAM && n < y.ni && mr < y.kb) *reinterpret_cast<bf16x4*>(y.wt + frag_at(n, mr, y.kb / 32)) = o;
}

// the BF16 copies of one layer's master weights
__global__ __launch_bounds__(256) void pack_kernel(Layer y, const float* w)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)y.no * (y.ni + 1)) return;
    const int m = (int)(i / (y.ni + 1)), n = (int)(i - (int64_t)m * (y.ni + 1));
    const __bf16 v = (__bf16)w[y.off + i];
    y.wf[frag_at(m, n, y.kf / 32)] = v;
    if (n < y.ni) y.wt[frag_at(n, m, y.kb / 32)] = v;
}

}  // namespace

struct pic_mlp {
    std::vector<int32_t> widths;
    Net net{};
    int64_t P = 0;
    int32_t max_batch = 0;
    int has_alloc = 0;
    pic_allocator alloc{};
    hipStream_t stream = nullptr;
    std::vector<void*> blocks;
    float *w = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
    uint4* weights = nullptr;      // every layer's wf and wt, one block
    size_t weight_bytes = 0;
    size_t forward_bytes = 0, train_bytes = 0;   // of them read by a prediction, by a training step
    bool chain = true;             // the layers of 16 samples fit the chain's LDS
    int kf_max = 0, k_max = 0;     // longest padded k: forward, training
    __bf16* rows[2] = {nullptr, nullptr};   // where the chain is not taken: rows of the current and the next product
    float* loss_part = nullptr;
    float* loss = nullptr;         // [1]
    int64_t max_parts = 0;
    int64_t updates = 0;
};

namespace {

void* net_alloc(pic_mlp* n, size_t bytes)
{
    bytes = (std::max<size_t>(bytes, 256) + 255) & ~(size_t)255;
    void* p = nullptr;
    if (n->has_alloc) p = n->alloc.alloc(bytes, n->alloc.user);
    else if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
    if (p) n->blocks.push_back(p);
    return p;
}

int64_t pad64(int64_t n) { return (n + 63) & ~(int64_t)63; }

size_t chain_lds(int mt, int k) { return (size_t)2 * 16 * mt * (k + kPad) * 2; }

// Whether a call takes the chain.  Its time is that of the weights through one
// compute unit's L2 port, whatever the batch up to 16 samples per compute unit:
// 11 us per MB.  A launch per product takes 5 us for each (6 when training) as
// long as the batch gives it few tiles.  So the chain is left for networks with
// more than kChainBytes of weights in an average product on batches of up to
// kLayerRows samples, and to kHeavyRows above kHeavyBytes.  Measured, us, chain /
// launch per product, hidden layers of h between 5 inputs and 768 outputs,
// batch 64: prediction h = 256 13.0 / 19.8, 448 (0.41 MB per product) 19.7 /
// 19.3, 512 23.3 / 20.2, 960 61.8 / 21.2; training 256 33.4 / 42.2, 384 (0.34
// MB) 48.6 / 45.2, 448 55.6 / 47.8, 512 63.4 / 49.4, 960 145 / 63.7.  By batch:
// h = 512 (0.5 MB), 256 samples 23.6 / 20.3 and 67.4 / 53.5, 1024 24.2 / 29.0 and
// 76.3 / 77.3; seven layers of 512, 256 samples 38.3 / 38.3, 512 38.3 / 41.9; h =
// 640 (0.68 MB), 768 samples 29.6 / 28.4 and 89.7 / 80.0, 1024 29.9 / 33.4.
// Layers that need more than 64 KiB of the compute unit's 160 would only gain
// from the chain above 2048 samples (h = 1024, 512 samples: 65 / 44 and 166 /
// 126; 4096: 72 / 102 and 277 / 337), so they do without.
constexpr size_t kChainBytes = 420000, kHeavyBytes = 600000;
constexpr int kLayerRows = 256, kHeavyRows = 768;

// the batches up to which a launch per product is taken
int layer_rows(const pic_mlp* n, bool train)
{
    if (!n->chain) return n->max_batch;
    const size_t products = train ? 2 * (size_t)n->net.L - 1 : (size_t)n->net.L;
    const size_t bytes = (train ? n->train_bytes : n->forward_bytes) / products;
    return bytes > kHeavyBytes ? kHeavyRows : (bytes > kChainBytes ? kLayerRows : 0);
}

bool use_chain(const pic_mlp* n, int batch, bool train) { return batch > layer_rows(n, train); }

template <bool TRAIN>
hipError_t launch_chain(const pic_mlp* n, ChainArgs& g, int* parts)
{
    const int k = TRAIN ? n->k_max : n->kf_max;
    g.ld = k + kPad;
    const int rows = TRAIN ? g.ldb : g.M;          // training fills its rows of 32
    // 16 samples per workgroup until the batch fills 256 compute units, then
    // 32, which share each weight fragment: the weights cross the L2 ports
    // once per workgroup.  Prediction of 4112 / 16384 samples by
    // 5-200-200-200-300: 18.9 / 39.4 us with 16, 14.1 / 29.0 with 32; training
    // there 72.9 / 176 and 61.3 / 155.  Not 64: its instance spilled
    // registers (16384 samples of 5-200-200-200-768: 51 us, 34 with 32).
    const int mt = rows > 16 * 256 && chain_lds(2, k) <= (size_t)kChainLds ? 2 : 1;
    g.rows_wg = (rows + 16 * mt - 1) / (16 * mt);
    g.weights = n->weights;
    g.n_weights = (int32_t)(n->weight_bytes / 16);
    // with few row blocks, workgroups that bring the weights into L2
    unsigned grid = (unsigned)g.rows_wg;
    if (TRAIN && g.rows_wg <= kWarmRows) grid = ((grid + kXcd - 1) / kXcd + kWarmers) * kXcd;
    const size_t lds = chain_lds(mt, k);
    if (mt == 1) hipLaunchKernelGGL((chain_kernel<1, TRAIN>), dim3(grid), dim3(kChainThreads), lds, n->stream, g);
    else hipLaunchKernelGGL((chain_kernel<2, TRAIN>), dim3(grid), dim3(kChainThreads), lds, n->stream, g);
    if (parts) *parts = g.rows_wg;
    return hipGetLastError();
}

// Tiles of 16 x 16 outputs up to which a layer takes a wave for each: many
// waves for a product that a few workgroups of 64 x 64 would do one after the
// other; above, each operand fragment has to serve more outputs.  Prediction by
// 5-1024-1024-1024-768, wave / workgroup tiles: 1024 of them 26.4 / 40.7 us,
// 2048 32.8 / 42.9, 4096 49.1 / 50.4, 8192 79.2 / 67.3; three layers of 2048:
// 4096 71.8 / 75.9, 8192 125 / 96.
constexpr int kSmallTiles = 4096;

// the layers one launch each (see use_chain)
hipError_t run_layers(pic_mlp* n, int batch, const float* x, float* y, const float* t, float scale, int ldb, int* parts)
{
    const Net& net = n->net;
    const int L = net.L;
    const int64_t rows = pad64(batch);
    const Layer& l0 = net.l[0];
    // a launch has fewer than 2^32 threads
    const int64_t input_wg = std::min<int64_t>((rows * l0.kf + 255) / 256, 1 << 23);
    hipLaunchKernelGGL(input_kernel, dim3((unsigned)input_wg), dim3(256), 0, n->stream, x, batch,
                       (int)rows, l0.ni, l0.kf, n->rows[0], t ? l0.at : nullptr, ldb);
    hipError_t e = hipGetLastError();
    int cur = 0;
    auto go = [&](LayerArgs& a, int cols) {
        a.M = batch;
        a.train = t ? 1 : 0;
        a.ldb = ldb;
        a.a = n->rows[cur];
        dim3 grid((unsigned)((cols + 15) / 16), (unsigned)(rows / 16));
        const bool small = (int64_t)grid.x * grid.y <= kSmallTiles;
        if (!small) grid = dim3((unsigned)((cols + 63) / 64), (unsigned)(rows / 64));
        if (a.epi == LAYER_LOSS && parts) *parts = (int)(grid.x * grid.y);
        if (small) hipLaunchKernelGGL((layer_kernel<1, 1, 1>), grid, dim3(64), 0, n->stream, a);
        else hipLaunchKernelGGL((layer_kernel<2, 2, 4>), grid, dim3(256), 0, n->stream, a);
        cur ^= 1;
        return hipGetLastError();
    };
    for (int l = 0; l < L && e == hipSuccess; ++l) {
        const Layer& p = net.l[l];
        LayerArgs a{};
        a.N = p.no;
        a.K = p.kf;
        a.b = p.wf;
        a.one = -1;
        if (l < L - 1) {
            a.epi = LAYER_HIDDEN;
            a.z = p.z;
            a.next = n->rows[cur ^ 1];
            a.next_t = net.l[l + 1].at;
            a.kn = net.l[l + 1].kf;
            a.one = p.no;
        } else if (t) {
            a.epi = LAYER_LOSS;
            a.t = t;
            a.scale = scale;
            a.loss_part = n->loss_part;
            a.next = n->rows[cur ^ 1];
            a.next_t = p.dzt;
            a.kn = p.kb;
        } else {
            a.epi = LAYER_OUT;
            a.z = y;
        }
        e = go(a, std::max(p.no, a.kn));
    }
    for (int l = L - 1; t && l > 0 && e == hipSuccess; --l) {
        const Layer& p = net.l[l];
        const Layer& q = net.l[l - 1];
        LayerArgs a{};
        a.epi = LAYER_BACK;
        a.N = p.ni;
        a.K = p.kb;
        a.b = p.wt;
        a.one = -1;
        a.z = q.z;
        a.next = n->rows[cur ^ 1];
        a.next_t = q.dzt;
        a.kn = q.kb;
        e = go(a, a.kn);
    }
    return e;
}

hipError_t run_forward(pic_mlp* n, int batch, const float* x, float* y)
{
    if (!use_chain(n, batch, false)) return run_layers(n, batch, x, y, nullptr, 0.0f, pad32(batch), nullptr);
    ChainArgs g{};
    g.net = n->net;
    g.M = batch;
    g.ldb = pad32(batch);
    g.x = x;
    g.y = y;
    return launch_chain<false>(n, g, nullptr);
}

struct AdamArgs {
    float lr, b1, b2, eps, c1, c2;
};

// the batch's loss into n->loss (and loss_out) and its gradient: into n->grad,
// or with `up` into the parameters by Adam
hipError_t run_grad(pic_mlp* n, int batch, const float* x, const float* t, float* loss_out, const AdamArgs* up)
{
    const int L = n->net.L, no = n->widths[L];
    const float scale = 2.0f / ((float)batch * (float)no);
    const int ldb = pad32(batch);
    int parts = 0;
    hipError_t e;
    if (use_chain(n, batch, true)) {
        ChainArgs c{};
        c.net = n->net;
        c.M = batch;
        c.ldb = ldb;
        c.x = x;
        c.t = t;
        c.scale = scale;
        c.loss_part = n->loss_part;
        e = launch_chain<true>(n, c, &parts);
    } else {
        e = run_layers(n, batch, x, nullptr, t, scale, ldb, &parts);
    }
    if (e != hipSuccess) return e;
    GradArgs g{};
    g.net = n->net;
    int tasks = 0;
    for (int l = 0; l < L; ++l) {
        g.first[l] = tasks;
        tasks += pad16(n->net.l[l].no) / 16 * (pad16(n->net.l[l].ni + 1) / 16);
    }
    g.first[L] = tasks;
    g.ldb = ldb;
    g.w = n->w;
    g.m = n->m;
    g.v = n->v;
    g.grad = n->grad;
    g.loss_part = n->loss_part;
    g.parts = parts;
    g.inv_count = 1.0f / ((float)batch * (float)no);
    g.loss = n->loss;
    g.loss2 = loss_out;
    const dim3 grid((unsigned)((tasks + 3) / 4 + 1));
    if (up) {
        g.lr = up->lr;
        g.b1 = up->b1;
        g.b2 = up->b2;
        g.eps = up->eps;
        g.c1 = up->c1;
        g.c2 = up->c2;
        hipLaunchKernelGGL(grad_kernel<true>, grid, dim3(256), 0, n->stream, g);
    } else {
        hipLaunchKernelGGL(grad_kernel<false>, grid, dim3(256), 0, n->stream, g);
    }
    return hipGetLastError();
}

bool batch_ok(const pic_mlp* n, int32_t batch) { return batch >= 1 && batch <= n->max_batch; }

}  // namespace

extern "C" {

pic_status pic_mlp_create(const int32_t* widths, int32_t n_widths, int32_t max_batch, const pic_allocator* alloc,
                          void* hip_stream, pic_mlp** out)
{
    if (!widths || !out || n_widths < 2 || n_widths > PIC_MLP_MAX_LAYERS + 1 || max_batch < 1 ||
        max_batch > (1 << 20))
        return PIC_EINVAL;
    for (int i = 0; i < n_widths; ++i)
        if (widths[i] < 1 || widths[i] > PIC_MLP_MAX_WIDTH) return PIC_EINVAL;
    if (alloc && (!alloc->alloc || !alloc->free)) return PIC_EINVAL;
    pic_mlp* n = new pic_mlp();
    n->widths.assign(widths, widths + n_widths);
    n->max_batch = max_batch;
    n->stream = (hipStream_t)hip_stream;
    if (alloc) {
        n->has_alloc = 1;
        n->alloc = *alloc;
    }
    const int L = n_widths - 1;
    n->net.L = L;
    for (int l = 0; l < L; ++l) {
        Layer& y = n->net.l[l];
        y.ni = widths[l];
        y.no = widths[l + 1];
        y.kf = pad32(y.ni + 1);
        y.kb = pad32(y.no);
        y.off = n->P;
        n->P += (int64_t)y.no * (y.ni + 1);
        n->kf_max = std::max(n->kf_max, y.kf);
        n->k_max = std::max(n->k_max, std::max(y.kf, y.kb));
    }
    n->chain = chain_lds(1, n->k_max) <= (size_t)kChainLds;
    n->max_parts = std::max<int64_t>({kSmallTiles, pad32(max_batch) / 16,
                                      pad64(max_batch) / 64 * ((n->net.l[L - 1].kb + 63) / 64)});
    bool ok = true;
    auto A = [&](size_t bytes) {
        void* p = net_alloc(n, bytes);
        ok = ok && p;
        return p;
    };
    n->w = (float*)A(4 * n->P);
    n->m = (float*)A(4 * n->P);
    n->v = (float*)A(4 * n->P);
    n->grad = (float*)A(4 * n->P);
    // the BF16 weights in the order of their use: forward, then back
    auto wf_bytes = [&](int l) { return 2ull * pad16(n->net.l[l].no) * n->net.l[l].kf; };
    auto wt_bytes = [&](int l) { return 2ull * pad16(n->net.l[l].ni) * n->net.l[l].kb; };
    for (int l = 0; l < L; ++l) n->forward_bytes += wf_bytes(l);
    n->train_bytes = n->forward_bytes;
    for (int l = 1; l < L; ++l) n->train_bytes += wt_bytes(l);
    n->weight_bytes = n->train_bytes + wt_bytes(0);
    n->weights = (uint4*)A(n->weight_bytes);
    {
        char* q = (char*)n->weights;
        for (int l = 0; l < L; ++l) {
            n->net.l[l].wf = (__bf16*)q;
            q += wf_bytes(l);
        }
        for (int l = L - 1; l >= 0; --l) {
            n->net.l[l].wt = (__bf16*)q;
            q += wt_bytes(l);
        }
    }
    const size_t ldb = pad32(max_batch);
    for (int l = 0; l < L; ++l) {
        Layer& y = n->net.l[l];
        y.at = (__bf16*)A(2ull * pad32(y.ni + 1) * ldb);
        y.dzt = (__bf16*)A(2ull * pad16(y.no) * ldb);
        if (l < L - 1) y.z = (float*)A(4ull * max_batch * y.no);
    }
    if (const int64_t rows = std::min(max_batch, std::max(layer_rows(n, false), layer_rows(n, true))))
        for (auto& r : n->rows) r = (__bf16*)A(2ull * pad64(rows) * n->k_max);
    n->loss_part = (float*)A(4ull * n->max_parts);
    n->loss = (float*)A(4);
    if (ok) {
        ok = hipMemsetAsync(n->w, 0, 4 * n->P, n->stream) == hipSuccess &&
             hipMemsetAsync(n->m, 0, 4 * n->P, n->stream) == hipSuccess &&
             hipMemsetAsync(n->v, 0, 4 * n->P, n->stream) == hipSuccess &&
             hipMemsetAsync(n->weights, 0, n->weight_bytes, n->stream) == hipSuccess &&   // padding stays zero
             hipStreamSynchronize(n->stream) == hipSuccess;
        if (!ok) {
            pic_mlp_free(n);
            return PIC_EHIP;
        }
    } else {
        pic_mlp_free(n);
        return PIC_ENOMEM;
    }
    *out = n;
    return PIC_OK;
}

int64_t pic_mlp_n_params(const pic_mlp* net) { return net ? net->P : 0; }

pic_status pic_mlp_set_params(pic_mlp* n, const float* params, int64_t count)
{
    if (!n || !params || count != n->P) return PIC_EINVAL;
    if (hipMemcpyAsync(n->w, params, 4 * n->P, hipMemcpyHostToDevice, n->stream) != hipSuccess) return PIC_EHIP;
    for (int l = 0; l < n->net.L; ++l) {
        const Layer& y = n->net.l[l];
        const int64_t k = (int64_t)y.no * (y.ni + 1);
        hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, n->stream, y, n->w);
        if (hipGetLastError() != hipSuccess) return PIC_EHIP;
    }
    if (hipMemsetAsync(n->m, 0, 4 * n->P, n->stream) != hipSuccess ||
        hipMemsetAsync(n->v, 0, 4 * n->P, n->stream) != hipSuccess)
        return PIC_EHIP;
    n->updates = 0;
    return hipStreamSynchronize(n->stream) == hipSuccess ? PIC_OK : PIC_EHIP;
}

pic_status pic_mlp_get_params(pic_mlp* n, float* params, int64_t count)
{
    if (!n || !params || count != n->P) return PIC_EINVAL;
    if (hipMemcpyAsync(params, n->w, 4 * n->P, hipMemcpyDeviceToHost, n->stream) != hipSuccess) return PIC_EHIP;
    return hipStreamSynchronize(n->stream) == hipSuccess ? PIC_OK : PIC_EHIP;
}

pic_status pic_mlp_forward(pic_mlp* n, int32_t batch, const float* x_dev, float* y_dev)
{
    if (!n || !x_dev || !y_dev || !batch_ok(n, batch)) return PIC_EINVAL;
    return run_forward(n, batch, x_dev, y_dev) == hipSuccess ? PIC_OK : PIC_EHIP;
}

pic_status pic_mlp_train_step(pic_mlp* n, int32_t batch, const float* x_dev, const float* t_dev, float lr,
                              float beta1, float beta2, float eps, float* loss_dev)
{
    if (!n || !x_dev || !t_dev || !batch_ok(n, batch)) return PIC_EINVAL;
    if (!(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
        return PIC_EINVAL;
    const double k = (double)(n->updates + 1);
    AdamArgs up{lr, beta1, beta2, eps, 0.0f, 0.0f};
    up.c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, k)));
    up.c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, k)));
    if (run_grad(n, batch, x_dev, t_dev, loss_dev, &up) != hipSuccess) return PIC_EHIP;
    n->updates += 1;
    return PIC_OK;
}

pic_status pic_mlp_grad(pic_mlp* n, int32_t batch, const float* x_dev, const float* t_dev, float* grad, float* loss)
{
    if (!n || !x_dev || !t_dev || !grad || !loss || !batch_ok(n, batch)) return PIC_EINVAL;
    if (run_grad(n, batch, x_dev, t_dev, nullptr, nullptr) != hipSuccess) return PIC_EHIP;
    if (hipMemcpyAsync(grad, n->grad, 4 * n->P, hipMemcpyDeviceToHost, n->stream) != hipSuccess ||
        hipMemcpyAsync(loss, n->loss, 4, hipMemcpyDeviceToHost, n->stream) != hipSuccess)
        return PIC_EHIP;
    return hipStreamSynchronize(n->stream) == hipSuccess ? PIC_OK : PIC_EHIP;
}

pic_status pic_mlp_sync(pic_mlp* n)
{
    if (!n) return PIC_EINVAL;
    return hipStreamSynchronize(n->stream) == hipSuccess ? PIC_OK : PIC_EHIP;
}

void pic_mlp_free(pic_mlp* n)
{
    if (!n) return;
    (void)hipStreamSynchronize(n->stream);
    for (void* p : n->blocks) {
        if (n->has_alloc) n->alloc.free(p, n->alloc.user);
        else (void)hipFree(p);
    }
    delete n;
}

}  // extern "C"
