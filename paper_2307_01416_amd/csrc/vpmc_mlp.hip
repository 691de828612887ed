// gfx950 kernels of the learned aperture surrogate: a multilayer perceptron
// 8 -> 256 -> 256 -> 256 -> 256 -> 29 (SiLU) with BF16 weights and
// activations and FP32 accumulation on the matrix cores, its loss and
// gradients (transmission cross-entropy + 4-component Gaussian mixture over
// outgoing energy loss / angle / offset) and an Adam optimiser with FP32
// master weights.
#include <math.h>

#include "vpmc_internal.hpp"

namespace vpmc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
    const float s = 1.0f / (1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// Fused inference: one workgroup (4 waves) carries 64 samples through all
// five layers.  The activations stay in LDS (two BF16 buffers of 64 x 256,
// rows padded to 264 to spread the banks); each wave computes 64 output
// columns of a hidden layer as 2 x 2 tiles of v_mfma_f32_32x32x16_bf16, its B
// fragments (eight consecutive K of one output unit, W[out][in] row-major)
// read straight from the L2-resident BF16 weights.  The K order and the
// instruction are those of mlp_chain_kernel, so the outputs equal the training
// pass's bit for bit.  REC: the inputs are computed from
// the deferred-VP records (same encoding as the training data) instead of
// read as FP32 rows of 8.
constexpr int kInfRows = 64;
constexpr int kInfLd = 264;

template <bool REC>
__global__ __launch_bounds__(256) void mlp_infer_kernel(const float *__restrict__ x, const DeferRec *__restrict__ rec,
                                                        int n, const __bf16 *__restrict__ wb,
                                                        const float *__restrict__ wf, float *__restrict__ out) {
    __shared__ __attribute__((aligned(16))) __bf16 H[2][kInfRows][kInfLd];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int row0 = blockIdx.x * kInfRows;
    const __bf16 zero = (__bf16)0.0f;
    if (t < kInfRows) {
        float in[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int r = row0 + t;
        if (r < n) {
            if (REC) {
                const DeferRec q = rec[r];
                in[0] = q.x / 20.0f;
                in[1] = q.y / 20.0f;
                in[2] = q.u / 0.05f;
                in[3] = q.v / 0.05f;
                in[4] = (q.E + q.Elo - 150.0f) / 50.0f;
                in[5] = fminf(q.d_edge, 100.0f) / 10.0f;
                in[6] = q.thick / 30.0f;
                in[7] = 0.0f;   // brass
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) in[j] = x[(size_t)r * 8 + j];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            H[0][t][j] = (__bf16)in[j];
            H[0][t][8 + j] = zero;
        }
    }
    __syncthreads();
    int off = 0;   // parameter offset of the layer
#pragma unroll 1
    for (int l = 0; l < MLP_LAYERS; ++l) {
        const int ni = l == 0 ? MLP_IN : MLP_HIDDEN;
        const int no = l == MLP_LAYERS - 1 ? MLP_OUT : MLP_HIDDEN;
        const int K = l == 0 ? 16 : MLP_HIDDEN;
        const __bf16 *W = wb + off;
        const float *bias = wf + off + no * ni;
        const bool last = l == MLP_LAYERS - 1;
        // hidden layers: wave w owns columns 64w .. 64w+63 (2 x 2 tiles);
        // output layer: waves 0 and 1 each own one 32 x 32 tile (rows 32w)
        const int ntile = last ? 1 : 2, mtile = last ? 1 : 2;
        const int n0 = last ? 0 : 64 * w, m0 = last ? 32 * w : 0;
        if (!last || w < 2) {
            f32x16 acc[2][2];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;
            const __bf16(*in)[kInfLd] = H[l & 1];
            const int kb = 8 * (lane >> 5);
            for (int k0 = 0; k0 < K; k0 += 16) {
                bf16x8 af[2], bfr[2];
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    if (a < mtile) af[a] = *reinterpret_cast<const bf16x8 *>(&in[m0 + 32 * a + (lane & 31)][k0 + kb]);
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (b >= ntile) continue;
                    const int col = n0 + 32 * b + (lane & 31);
                    const int k = k0 + kb;
                    if (col < no && k < ni) {
                        bfr[b] = *reinterpret_cast<const bf16x8 *>(W + (size_t)col * ni + k);
                    } else {
#pragma unroll
                        for (int j = 0; j < 8; ++j) bfr[b][j] = zero;
                    }
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        if (a < mtile && b < ntile)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
            }
            __bf16(*ob)[kInfLd] = H[(l + 1) & 1];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (a >= mtile || b >= ntile) continue;
                    const int col = n0 + 32 * b + (lane & 31);
                    const float bc = col < no ? bias[col] : 0.0f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int r = m0 + 32 * a + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
                        const float z = acc[a][b][i] + bc;
                        if (!last) {
                            ob[r][col] = (__bf16)silu_f(z);
                        } else if (col < no && row0 + r < n) {
                            out[(size_t)(row0 + r) * MLP_OUT + col] = z;
                        }
                    }
                }
        }
        off += no * ni + no;
        __syncthreads();
    }
}

__global__ void to_bf16_kernel(const float *__restrict__ x, __bf16 *__restrict__ y, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        y[i] = (__bf16)x[i];
}

// ---------------------------------------------------------------------------
// Training step: three launches (chain, weight gradients, update).  A layer by
// layer step was 30 launches of 4 to 12 us, 230 us for 4096 samples.
//
// Fragments: 64 lanes x 8 BF16 (16 bytes a lane, 1 KB, one load of a
// wavefront) as v_mfma_f32_32x32x16_bf16 takes an operand: lane & 31 is the
// row (A) or column (B), 8 (lane >> 5) + j the K index.  The weights are kept a
// second time as fragments of both directions (frag_fwd, frag_bwd: layer by
// layer, 32 outputs (inputs) by 16 K); the activations and their gradients are
// written as fragments with the samples along K (per 32 samples: 32 features,
// two halves of 16 samples), which is what the weight gradients contract.
constexpr int kFrag = 512;                          // elements of a fragment
constexpr int kFwdFrags = MLP_FWD_ELEMS / kFrag, kBwdFrags = 3 * 128 + 16;

__host__ __device__ constexpr int fwd_base(int l) { return l == 0 ? 0 : 8 + 128 * (l - 1); }   // in fragments
__host__ __device__ constexpr int bwd_base(int l) { return 128 * (l - 1); }
__device__ __forceinline__ int frag_at(int row, int k, int steps) {
    return (((row >> 5) * steps + (k >> 4)) * 64 + (row & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}
// where the weight W[o][i] of layer l stands in both fragment buffers
__device__ __forceinline__ int frag_fwd(int l, int o, int i) {
    return fwd_base(l) * kFrag + frag_at(o, i, l == 0 ? 1 : 16);
}
__device__ __forceinline__ int frag_bwd(int l, int o, int i) {
    return bwd_base(l) * kFrag + frag_at(i, o, l == MLP_LAYERS - 1 ? 2 : 16);
}

// layer, output and input of the e-th weight (biases not counted), and its
// index among the parameters
__device__ __forceinline__ int weight_at(int e, int &l, int &o, int &i) {
    constexpr int n0 = MLP_HIDDEN * MLP_IN, nh = MLP_HIDDEN * MLP_HIDDEN;
    l = e < n0 ? 0 : 1 + (e - n0) / nh;
    const int r = l == 0 ? e : e - n0 - (l - 1) * nh;
    o = l == 0 ? r / MLP_IN : r / MLP_HIDDEN;
    i = l == 0 ? r % MLP_IN : r % MLP_HIDDEN;
    return e + MLP_HIDDEN * l;
}
constexpr int kWeights = MLP_HIDDEN * (MLP_IN + 3 * MLP_HIDDEN + MLP_OUT);

// both fragment buffers (one behind the other) from the BF16 parameters
__global__ void mlp_pack_kernel(const __bf16 *__restrict__ wb, __bf16 *fwd, __bf16 *bwd) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < kWeights; e += gridDim.x * blockDim.x) {
        int l, o, i;
        const __bf16 w = wb[weight_at(e, l, o, i)];
        fwd[frag_fwd(l, o, i)] = w;
        if (l > 0) bwd[frag_bwd(l, o, i)] = w;
    }
}

// rows of `in` x the fragments b, K in steps of 16
template <int T>
__device__ __forceinline__ f32x16 chain_mm(const __bf16 (*in)[kInfLd], const uint4 (&b)[16]) {
    const int lane = threadIdx.x & 63;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int t = 0; t < T; ++t)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *reinterpret_cast<const bf16x8 *>(&in[lane & 31][16 * t + 8 * (lane >> 5)]),
            __builtin_bit_cast(bf16x8, b[t]), acc, 0, 0, 0);
    return acc;
}

template <int T>
__device__ __forceinline__ void chain_load(uint4 (&b)[16], const __bf16 *frags) {
#pragma unroll
    for (int t = 0; t < T; ++t) b[t] = *((const uint4 *)(frags + (size_t)t * kFrag) + (threadIdx.x & 63));
}

// A 32 x 32 block of values (accumulator layout: sample 8 (i >> 2) + 4 (lane >> 5)
// + (i & 3), feature lane & 31) as two fragments with the samples along K.
__device__ __forceinline__ void put_frags(const unsigned short (&v)[16], __bf16 *to) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        unsigned g[2][2], r[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int k = 0; k < 2; ++k)
                g[q][k] = (unsigned)v[8 * t + 4 * q + 2 * k] | (unsigned)v[8 * t + 4 * q + 2 * k + 1] << 16;
#pragma unroll
        for (int k = 0; k < 2; ++k) r[k] = (unsigned)__shfl_xor((int)(h ? g[0][k] : g[1][k]), 32);
        const uint4 f = h ? make_uint4(r[0], r[1], g[1][0], g[1][1]) : make_uint4(g[0][0], g[0][1], r[0], r[1]);
        *((uint4 *)(to + t * kFrag) + lane) = f;
    }
}

// the same from rows of samples in LDS (features past `cols` are zero)
__device__ __forceinline__ void put_rows(const __bf16 (*in)[kInfLd], int cols, __bf16 *to) {
    const int lane = threadIdx.x & 63, f = lane & 31;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = f < cols ? in[16 * t + 8 * (lane >> 5) + j][f] : (__bf16)0.0f;
        *((uint4 *)(to + t * kFrag) + lane) = __builtin_bit_cast(uint4, v);
    }
}

// Per-sample loss and its gradient with respect to the 29 outputs (scaled by
// inv_n for the batch mean): FP32 in dout (an output every `pitch`), BF16 in db.
__device__ __forceinline__ float loss_head(const float *o, const float (&y)[3], float tr, float inv_n,
                                           float *__restrict__ dout, int pitch, __bf16 *db) {
    float g[29];
#pragma unroll
    for (int j = 0; j < 29; ++j) g[j] = 0.0f;
    const float lt = o[0];
    float L = fmaxf(lt, 0.0f) - lt * tr + log1pf(__expf(-fabsf(lt)));
    g[0] = 1.0f / (1.0f + __expf(-lt)) - tr;
    if (tr > 0.5f) {
        float mw = o[1];
#pragma unroll
        for (int c = 1; c < 4; ++c) mw = fmaxf(mw, o[1 + c]);
        float zs = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) zs += __expf(o[1 + c] - mw);
        const float lz = __logf(zs);
        float lw[4], lp[4], m = -INFINITY;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            lw[c] = o[1 + c] - mw - lz;
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float mu = o[5 + 3 * c + j], ls = o[17 + 3 * c + j];
                const float r = (y[j] - mu) * __expf(-ls);
                acc += -0.5f * r * r - ls - 0.91893853320467274f;
            }
            lp[c] = lw[c] + acc;
            m = fmaxf(m, lp[c]);
        }
        float tot = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) tot += __expf(lp[c] - m);
        const float lse = m + __logf(tot);
        L -= lse;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float gam = __expf(lp[c] - lse), pic = __expf(lw[c]);
            g[1 + c] += pic - gam;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float mu = o[5 + 3 * c + j], ls = o[17 + 3 * c + j];
                const float iv = __expf(-2.0f * ls), d = y[j] - mu;
                g[5 + 3 * c + j] += -gam * d * iv;
                g[17 + 3 * c + j] += -gam * (d * d * iv - 1.0f);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 29; ++j) {
        dout[(size_t)j * pitch] = g[j] * inv_n;
        db[j] = (__bf16)(g[j] * inv_n);
    }
    return L;
}

// Forward, loss and backward of 32 samples by one workgroup of eight
// wavefronts, each on 32 features of every layer.  What bounds it is the chain
// of ten products, not their arithmetic (4096 samples: 128 workgroups): the
// activations stay in LDS, the pre-activations in the registers that the
// backward pass needs them in (the same 32 x 32 block), and the weights of a
// layer, which do not wait for anything, are loaded as fragments while the
// layer before it is finished.  27 us for 4096 samples: the ten products and
// their barriers 14, silu and its derivative 7, loss 2, the fragments' stores
// and loads 4 (25 launches of the layer by layer step: 120 us).  K runs in
// ascending steps of 16 into one accumulator.  Rows past n are zero in all that
// the other kernels read.
__global__ __launch_bounds__(512) void mlp_chain_kernel(MlpStep S) {
    __shared__ __attribute__((aligned(16))) __bf16 H[2][32][kInfLd];
    __shared__ float out[32][MLP_OUT];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), h = lane >> 5;
    const int row0 = blockIdx.x * 32, col = 32 * w + (lane & 31);
    const int rows = min(32, S.n - row0);
    uint4 b[16];
    chain_load<1>(b, S.fwd + (size_t)(fwd_base(0) + w) * kFrag);
    float bias[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) bias[l] = S.w[(l == 0 ? MLP_HIDDEN * MLP_IN : MLP_HIDDEN * (MLP_IN + 1) +
                                               l * MLP_HIDDEN * MLP_HIDDEN + (l - 1) * MLP_HIDDEN) + col];
    float y[3] = {0.0f, 0.0f, 0.0f}, tr = 0.0f;
    if (t < 32) {
        bf16x8 v, zero;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = zero[j] = (__bf16)0.0f;
        if (t < rows) {
            const size_t src = S.idx ? (size_t)S.idx[row0 + t] : (size_t)(row0 + t);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (__bf16)S.x[src * MLP_IN + j];
#pragma unroll
            for (int j = 0; j < 3; ++j) y[j] = S.y[src * 3 + j];
            tr = S.t[src];
        }
        *reinterpret_cast<bf16x8 *>(&H[0][t][0]) = v;
        *reinterpret_cast<bf16x8 *>(&H[0][t][8]) = zero;
    }
    __syncthreads();
    if (w == 7) put_rows(H[0], MLP_IN, S.xf + (size_t)blockIdx.x * 2 * kFrag);
    float z[4][16];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const f32x16 acc = l == 0 ? chain_mm<1>(H[0], b) : chain_mm<16>(H[l & 1], b);
        if (l < 3) chain_load<16>(b, S.fwd + (size_t)(fwd_base(l + 1) + 16 * w) * kFrag);
        else if (w == 0) chain_load<16>(b, S.fwd + (size_t)fwd_base(4) * kFrag);
        else chain_load<2>(b, S.bwd + (size_t)(bwd_base(4) + 2 * w) * kFrag);
        unsigned short v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = 8 * (i >> 2) + 4 * h + (i & 3);
            z[l][i] = acc[i] + bias[l];
            const __bf16 a = m < rows ? (__bf16)silu_f(z[l][i]) : (__bf16)0.0f;
            H[(l + 1) & 1][m][col] = a;
            v[i] = __builtin_bit_cast(unsigned short, a);
        }
        put_frags(v, S.hf[l] + ((size_t)blockIdx.x * 8 + w) * 2 * kFrag);
        __syncthreads();
    }
    if (w == 0) {
        const f32x16 acc = chain_mm<16>(H[0], b);
        chain_load<2>(b, S.bwd + (size_t)bwd_base(4) * kFrag);
        const float bo = lane % 32 < MLP_OUT ? S.w[MLP_HIDDEN * (MLP_IN + 1) + 3 * MLP_HIDDEN * (MLP_HIDDEN + 1) +
                                                   MLP_HIDDEN * MLP_OUT + (lane & 31)] : 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((lane & 31) < MLP_OUT) out[8 * (i >> 2) + 4 * h + (i & 3)][lane & 31] = acc[i] + bo;
    }
    __syncthreads();
    if (t < 32) {
        __bf16 *db = H[1][t];
#pragma unroll
        for (int j = 0; j < 32; j += 8) {
            bf16x8 zero;
#pragma unroll
            for (int k = 0; k < 8; ++k) zero[k] = (__bf16)0.0f;
            *reinterpret_cast<bf16x8 *>(db + j) = zero;
        }
        if (t < rows)
            S.loss[row0 + t] = loss_head(out[t], y, tr, S.inv_n, S.dout + row0 + t, S.n, db);
    }
    __syncthreads();
    if (w == 7) put_rows(H[1], MLP_OUT, S.dof + (size_t)blockIdx.x * 2 * kFrag);
#pragma unroll
    for (int l = 4; l >= 1; --l) {   // dZ of layer l-1 = (dZ of layer l . W_l) * silu'(Z of layer l-1)
        const f32x16 acc = l == 4 ? chain_mm<2>(H[1], b) : chain_mm<16>(H[l & 1 ? 0 : 1], b);
        if (l > 1) chain_load<16>(b, S.bwd + (size_t)(bwd_base(l - 1) + 16 * w) * kFrag);
        unsigned short v[16];
        float csum = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int m = 8 * (i >> 2) + 4 * h + (i & 3);
            __bf16 a = (__bf16)0.0f;
            if (m < rows) {
                const float d = acc[i] * dsilu_f(z[l - 1][i]);
                a = (__bf16)d;
                csum += d;
            }
            if (l > 1) H[l & 1 ? 1 : 0][m][col] = a;
            v[i] = __builtin_bit_cast(unsigned short, a);
        }
        put_frags(v, S.df[l - 1] + ((size_t)blockIdx.x * 8 + w) * 2 * kFrag);
        csum += __shfl_xor(csum, 32, 64);
        if (h == 0) S.bpart[l - 1][(size_t)blockIdx.x * MLP_HIDDEN + col] = csum;
        __syncthreads();
    }
}

// Weight gradients dW = dZ^T . H_in of all layers in one launch: a wavefront per
// 32 x 32 block and K range [z kchunk, ...), partials to part[z][parameter].
// The operands are fragments, read once per wavefront straight from L2 in 1 KB
// loads; a workgroup is 2 x 2 blocks of a hidden layer, or four blocks of the
// first or last.  The K range is the workgroup's number modulo the ranges:
// workgroups go to the XCDs in turn, so each XCD's L2 fetches an eighth of the
// samples (11.8 us with the range as the slow index, 10.5 so).
__global__ __launch_bounds__(256) void mlp_wgrad_kernel(MlpStep S, int kchunk, int split) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kr = (int)blockIdx.x % split, g = (int)blockIdx.x / split;
    int l, mt, nt;
    if (g < 48) {
        l = 1 + g / 16;
        mt = 2 * (g % 16 / 4) + (w >> 1);
        nt = 2 * (g % 4) + (w & 1);
    } else {
        const int k = 4 * (g & 1) + w;
        l = g < 50 ? 0 : 4;
        mt = l == 0 ? k : 0;
        nt = l == 0 ? 0 : k;
    }
    const __bf16 *A = l == 4 ? S.dof : S.df[l] + (size_t)mt * 2 * kFrag;
    const __bf16 *B = l == 0 ? S.xf : S.hf[l - 1] + (size_t)nt * 2 * kFrag;
    const size_t da = (l == 4 ? 2 : 16) * kFrag, db = (l == 0 ? 2 : 16) * kFrag;   // per 32 samples
    const int kbeg = kr * kchunk, kend = min(S.n, kbeg + kchunk);
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    constexpr int kFlight = 4;   // blocks of 32 samples in flight
    for (int k = kbeg; k < kend; k += 32 * kFlight) {
        uint4 a[kFlight][2], b[kFlight][2];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            if (k + 32 * u >= kend) break;
            const uint4 *pa = (const uint4 *)(A + (size_t)((k >> 5) + u) * da) + lane;
            const uint4 *pb = (const uint4 *)(B + (size_t)((k >> 5) + u) * db) + lane;
            a[u][0] = pa[0];
            a[u][1] = pa[64];
            b[u][0] = pb[0];
            b[u][1] = pb[64];
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            if (k + 32 * u >= kend) break;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u][j]),
                                                              __builtin_bit_cast(bf16x8, b[u][j]), acc, 0, 0, 0);
        }
    }
    const int ni = l == 0 ? MLP_IN : MLP_HIDDEN, no = l == 4 ? MLP_OUT : MLP_HIDDEN;
    const int off = l == 0 ? 0 : MLP_HIDDEN * (MLP_IN + 1) + (l - 1) * MLP_HIDDEN * (MLP_HIDDEN + 1);
    float *C = S.part + (size_t)kr * S.np + off;
    const int n = 32 * nt + (lane & 31);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = 32 * mt + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
        if (m < no && n < ni) C[(size_t)m * ni + n] = acc[i];
    }
}

// Sum over x[r * stride], r < n: 256 strided sums, then a tree.  By a workgroup
// (WG, a sum per thread) for a value per sample, by a wavefront (four sums a
// lane) for one per 32 samples; the same bits.  Up to 16 loads of a thread are
// in flight: what the sums cost is the rounds to memory.
template <bool WG>
__device__ __forceinline__ float strided_sum(const float *__restrict__ x, int n, size_t stride, float *red) {
    constexpr int per = WG ? 1 : 4, step = WG ? 256 : 64;
    const int t = WG ? (int)threadIdx.x : (int)(threadIdx.x & 63);
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int r = t; r < n; r += step * 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = r + step * u < n ? x[(size_t)(r + step * u) * stride] : 0.0f;
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (r + step * u < n) s[u % per] += v[u];
    }
    if (WG) {
        red[t] = s[0];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = red[(t & 63) + 64 * q];
    }
    float a = (s[0] + s[2]) + (s[1] + s[3]);
    for (int o = 32; o > 0; o >>= 1) a += __shfl_down(a, o);
    return a;   // lane 0
}

// The gradient of every parameter, finished, and its Adam step (Kingma and Ba)
// on the FP32 master with its BF16 copies refreshed; with S.grad the gradient
// goes there instead.  Workgroups: one for the loss and one per output bias (the
// longest sums, first), a wavefront per hidden bias (sums of dZ), 256 weights
// each (their K ranges' partials in order).
constexpr int kWeightBlocks = (kWeights + 255) / 256;
constexpr int kUpdateBlocks = 1 + MLP_OUT + MLP_HIDDEN + kWeightBlocks;

__global__ __launch_bounds__(256) void mlp_update_kernel(MlpStep S, int parts, float lr, float b1, float b2, float eps,
                                                         float c1, float c2) {
    __shared__ float red[256];
    int l = 0, o = 0, i = -1, p;
    float gi = 0.0f, m = 0.0f, v = 0.0f, w = 0.0f;
    int g = (int)blockIdx.x;
    if (g == 0) {
        const float s = strided_sum<true>(S.loss, S.n, 1, red);
        if (threadIdx.x == 0) *S.loss_acc += (double)s * (1.0 / S.n);
        return;
    }
    g -= 1;
    if (g < MLP_OUT) {
        p = MLP_HIDDEN * (MLP_IN + 1) + 3 * MLP_HIDDEN * (MLP_HIDDEN + 1) + MLP_OUT * MLP_HIDDEN + g;
        gi = strided_sum<true>(S.dout + (size_t)g * S.n, S.n, 1, red);
        if (threadIdx.x) return;
    } else if ((g -= MLP_OUT) < MLP_HIDDEN) {
        const int c = 4 * g + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        l = c / MLP_HIDDEN;
        o = c % MLP_HIDDEN;
        p = l == 0 ? MLP_HIDDEN * MLP_IN + o
                   : MLP_HIDDEN * (MLP_IN + 1) + (l - 1) * MLP_HIDDEN * (MLP_HIDDEN + 1) + MLP_HIDDEN * MLP_HIDDEN + o;
        gi = strided_sum<false>(S.bpart[l] + o, (S.n + 31) / 32, MLP_HIDDEN, red);
        if (threadIdx.x & 63) return;
    } else {
        const int e = (g - MLP_HIDDEN) * 256 + (int)threadIdx.x;
        if (e >= kWeights) return;
        p = weight_at(e, l, o, i);
        float part[kMlpSplit];
#pragma unroll
        for (int k = 0; k < kMlpSplit; ++k) part[k] = k < parts ? S.part[(size_t)k * S.np + p] : 0.0f;
        m = S.m[p];
        v = S.v[p];
        w = S.w[p];
#pragma unroll
        for (int k = 0; k < kMlpSplit; ++k)
            if (k < parts) gi += part[k];
    }
    if (i < 0) {
        m = S.m[p];
        v = S.v[p];
        w = S.w[p];
    }
    if (S.grad) {
        S.grad[p] = gi;
        return;
    }
    const float mi = b1 * m + (1.0f - b1) * gi;
    const float vi = b2 * v + (1.0f - b2) * gi * gi;
    S.m[p] = mi;
    S.v[p] = vi;
    const float pi = w - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    S.w[p] = pi;
    const __bf16 pb = (__bf16)pi;
    S.wb[p] = pb;
    if (i < 0) return;
    S.fwd[frag_fwd(l, o, i)] = pb;
    if (l > 0) S.bwd[frag_bwd(l, o, i)] = pb;
}

int grid_for(size_t n) { return (int)std::min<size_t>((n + 255) / 256, 4096); }

}  // namespace

// ------------------------------------------------------------------ host side
static const int kDims[MLP_LAYERS + 1] = {8, 256, 256, 256, 256, 29};

int mlp_param_count() {
    int n = 0;
    for (int l = 0; l < MLP_LAYERS; ++l) n += kDims[l + 1] * kDims[l] + kDims[l + 1];
    return n;
}

size_t mlp_frag_bytes() { return (size_t)(kFwdFrags + kBwdFrags) * kFrag * sizeof(__bf16); }

hipError_t mlp_pack(const MlpStep &S, hipStream_t s) {
    // the fragments' places past the inputs and outputs hold zeros
    hipError_t e = launch_fill_u64((unsigned long long *)S.fwd, mlp_frag_bytes() / 8, 0ull, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_pack_kernel, dim3(grid_for(kWeights)), dim3(256), 0, s, S.wb, S.fwd, S.bwd);
    return hipGetLastError();
}

// K ranges of the weight gradients: up to kMlpSplit of at least 128 samples
static int wgrad_split(int n, int *kchunk) {
    const int split = n >= 256 ? std::max(1, std::min(kMlpSplit, n / 128)) : 1;
    *kchunk = split > 1 ? ((n + split - 1) / split + 63) / 64 * 64 : (n + 63) / 64 * 64;
    return (n + *kchunk - 1) / *kchunk;
}

hipError_t mlp_step(const MlpStep &S, float lr, int step, hipStream_t s) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    int kchunk;
    const int split = wgrad_split(S.n, &kchunk);
    hipLaunchKernelGGL(mlp_chain_kernel, dim3((S.n + 31) / 32), dim3(512), 0, s, S);
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(52 * split), dim3(256), 0, s, S, kchunk, split);
    hipLaunchKernelGGL(mlp_update_kernel, dim3(kUpdateBlocks), dim3(256), 0, s, S, split, lr, b1, b2, eps,
                       c1, c2);
    return hipGetLastError();
}

hipError_t mlp_infer(const float *x, const DeferRec *rec, int n, const __bf16 *wb, const float *wf, float *out,
                     hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((n + kInfRows - 1) / kInfRows), block(256);
    if (rec) hipLaunchKernelGGL(mlp_infer_kernel<true>, grid, block, 0, s, x, rec, n, wb, wf, out);
    else hipLaunchKernelGGL(mlp_infer_kernel<false>, grid, block, 0, s, x, rec, n, wb, wf, out);
    return hipGetLastError();
}

hipError_t mlp_to_bf16(const float *x, __bf16 *y, size_t n, hipStream_t s) {
    hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(n)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

}  // namespace vpmc
