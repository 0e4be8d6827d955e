// mlp.hip -- the warm-start network on the matrix cores, and the kernels that turn a compiled
// game into network rows and network outputs into initial regrets.
//
// The network maps a 128-wide feature row of an information set through ReLU hidden layers to
// four logits z; p = softplus(z) over the set's legal actions is both the predicted strategy
// (after normalisation) and, scaled, the initial regrets R0 that CFR+ starts from.  Training
// minimises the weighted cross entropy between normalise(p) and the average strategy the solver
// produced, with Adam (Kingma and Ba 2015) on FP32 master weights.  The paper has no learned
// part; these definitions are the project's own.
//
// Arithmetic: every hidden-layer product runs on v_mfma_f32_32x32x16_bf16 with bfloat16
// operands and FP32 accumulation, one accumulator per output over the inputs in ascending order, so
// every kernel that computes a layer gives the same bits.  Stored in bfloat16 (round to nearest even): feature rows,
// the weight copies the matrix cores read (both layouts, refreshed with every parameter update), hidden
// activations, and the gradients of the hidden pre-activations.  FP32: biases, logits, the loss, all
// parameter gradients, Adam state.  The four-wide output layer is a per-row dot product on the vector
// units fused with the loss.  Every reduction has a fixed order (partials, then one sequential pass), so
// a step is bitwise reproducible.
//
// A training step is three launches: k_rows takes a tile of rows through all layers, the loss and back
// (everything that is local to a row) and leaves activations and gradients behind with rows contiguous,
// k_wgrad forms the partial sums over rows, k_finish adds them in order and applies Adam.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/cfr.h"
#include "mlp.hpp"

namespace cfrx {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// round to nearest even, NaN stays NaN (v_cvt_pk_bf16_f32)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ float softplus_f(float z) { return fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))); }
__device__ __forceinline__ float sigmoid_f(float z) { return 1.f / (1.f + expf(-z)); }
constexpr float LOG_CUT = -30.f;  // below: log softplus(z) = z, sigmoid(z) / softplus(z) = 1

// ---- a tile of rows through the network -----------------------------------------------------
// k_rows takes a block's rows through every layer with the activations in LDS, [row][unit], overwritten
// layer by layer.  A layer is computed transposed: the weights are the matrix cores' first operand, the
// activations the second, so that a lane ends up with four consecutive units of one row (accumulator i
// of lane l holds unit 8 (i / 4) + 4 (l / 32) + i % 4 of row l % 32) and stores them as one 8-byte LDS
// write.  A wave owns RT x CT tiles of 32 rows x 32 units and reads its weights straight from L2 into
// registers, PF steps ahead: no wave shares them within the tile except the WR waves of other rows, so
// staging them in LDS would only add barriers.
//
// Tiles (by rows, see rows_tile): 32 rows, one wave per 32 units, for up to 8,192 rows -- there a launch
// has at most a block per compute unit, so the shortest chain per block wins -- and 128 rows beyond, whose
// weight reads (0.3 MB per tile in inference) are shared by more rows.  The line is where the small tile's blocks
// begin to double up, below where the two tiles cost the same.  Both on both sides, us of a call or training step,
// small / large tile: 128 -> 3 x 256 -> 4, inference 8,192 rows 11.4 / 18.2, 10,240 16.0 / 18.2, 16,384
// 16.5 / 18.4, 20,480 21.5 / 18.6, 65,536 51.6 / 24.7; training 8,192 70 / 105, 16,384 103 / 131, 32,768 186 / 185.
// 64 -> 3 x 64 -> 4, inference 4,096 8.1 / 7.2, 8,192 8.2 / 7.2, 10,240 9.5 / 7.4; training 8,192 52 / 86,
// 32,768 115 / 143.  In inference four waves of
// up to 4 x 2 tiles (half an LDS read and a quarter of a KB of weights per MFMA) leave room for two blocks per
// compute unit, which hide each other's loads, stores and output layers.
// Measured: 240,930 rows through 128 -> 3 x 256 -> 4, 377 -> 87 us (920 TFLOP/s; its products alone at the rate of
// a large library GEMM: 66 us).  A training step on 4,096 rows, 190 -> 60 us (23 launches before): this
// kernel 39, k_wgrad 12, k_finish 9.
//
// The bf16 copies of the hidden weights are kept in the order the matrix cores take them, so that a wave's
// load of one operand is 1 KB of consecutive memory: tiles of 32 rows, within a tile steps of 16 inputs, of
// which lane l holds inputs 8 (l / 32) .. + 7 of row l % 32.
struct Weights {
    float *theta;             // FP32 parameters
    uint16_t *fwd, *bwd;      // hidden layer l at wt_off[l]: rows = units (inputs = fan in), and rows = fan in
                              // (inputs = units)
    float *out;               // [HID][4] output weights, rounded to bf16 (FP32, so uniform reads are scalar loads)
    int64_t woff[5], boff[5], wt_off[4];
    int n_hidden, in_dim, hidden;
};

// place of (row, input) in that order, `inputs` inputs per row
__device__ __forceinline__ int64_t operand_at(int row, int input, int inputs) {
    return ((int64_t)(row >> 5) * (inputs >> 4) + (input >> 4)) * 512 + ((row & 31) + 32 * ((input >> 3) & 1)) * 8 +
           (input & 7);
}

struct RowsArgs {
    Weights W;
    const uint16_t *x;        // [.][in_dim] bf16
    int rows;
    float *z;                 // inference: logits [rows][4]
    // training: row r of the minibatch is row idx[r] (clamped into [0, n_data)) of x, T, w, nact
    const int32_t *idx;
    int64_t n_data;
    const float *T, *w;       // [.][4] targets, [.] weights or nullptr
    const uint8_t *nact;      // [.] legal actions (clamped to 1..4)
    const float *inv_wsum;    // 1 / sum of the minibatch's weights, or nullptr: every block sums them itself
    int64_t ld;               // rows of the transposed arrays, a multiple of the tile; rows past the last are zero
    // transposed: units (or input columns) as rows, minibatch rows as inputs, in operand order
    uint16_t *Xt;             // inputs
    uint16_t *H[4], *Ht[4];   // [ld][HID] and transposed activations
    uint16_t *dAt[4];         // transposed gradients of the pre-activations
    float *dz, *ce, *wr;      // [ld][4], [ld], [ld]: logit gradients, cross entropy and weight of each row
    float *bias_part[4];      // [ld / BIAS_ROWS][HID] sums of dA over BIAS_ROWS rows each
};

constexpr int BIAS_ROWS = 16;   // rows per bias partial
constexpr int WSUM_ROWS = 8192; // up to here each block sums the row weights itself

// row of the training arrays that minibatch row r stands for
__device__ __forceinline__ int64_t data_row(const int32_t *idx, int64_t n_data, int r) {
    return idx ? min(max((int64_t)idx[r], (int64_t)0), n_data - 1) : (int64_t)r;
}

// 1 / sum of the row weights (rows when there are none) in fixed order: 256 strided sums, then a tree; red
// holds 256 floats.  Every thread of the block calls it.
__device__ __forceinline__ float inv_weight_sum(const float *w, const int32_t *idx, int64_t n_data, int rows,
                                                float *red) {
    for (int t = threadIdx.x; t < 256; t += blockDim.x) {
        float acc = 0.f;
        if (w) {
            constexpr int U = 16;
            for (int b = t; b < rows; b += 256 * U) {
                int64_t at[U];
                float x[U];
#pragma unroll
                for (int i = 0; i < U; i++) at[i] = data_row(idx, n_data, min(b + i * 256, rows - 1));
#pragma unroll
                for (int i = 0; i < U; i++) x[i] = w[at[i]];
#pragma unroll
                for (int i = 0; i < U; i++) acc = b + i * 256 < rows ? acc + x[i] : acc;
            }
        } else {
            for (int r = t; r < rows; r += 256) acc += 1.f;
        }
        red[t] = acc;
    }
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    const float s = red[0];
    __syncthreads();
    return s > 0.f ? 1.f / s : 0.f;
}

__global__ __launch_bounds__(256) void k_inv_wsum(const float *w, const int32_t *idx, int64_t n_data, int rows,
                                                  float *out) {
    __shared__ float red[256];
    const float x = inv_weight_sum(w, idx, n_data, rows, red);
    if (threadIdx.x == 0) out[0] = x;
}

// acc[r][c] += (32 units at n0 + 32 c) x (32 rows at m0 + 32 r) over K inputs: W in operand order,
// act [.][LDA] in LDS, inputs in ascending steps of 16
// (buffer loads: the weights of the next PF steps are requested while this group is multiplied, and plain
// loads are moved back to their first use).  The buffer ends with the matrix, `units` rows of K inputs.
template <int RT, int CT, int LDA, int PF>
__device__ __forceinline__ void layer_mfma(const uint16_t *W, int units, int K, const uint16_t *act, int m0, int n0,
                                           f32x16 (&acc)[RT][CT]) {
    const int lane = threadIdx.x & 63, row = lane & 31, k8 = (lane >> 5) * 8;
#pragma unroll
    for (int r = 0; r < RT; r++)
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[r][c][i] = 0.f;
    // lane l supplies unit (row) l % 32 and inputs 8 (l / 32) .. + 7 of each step
    constexpr int RAW_32BIT = 0x20000;   // buffer descriptor: untyped 32-bit elements
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, units * K * 2, RAW_32BIT);
    auto weights = [&](int c, int k) {   // byte offsets: 1 KB per tile and step
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                              rsrc, lane * 16, ((n0 >> 5) + c) * K * 64 + k * 64, 0));
    };
    const uint16_t *ap = act + (m0 + row) * LDA + k8;
    bf16x8 w[PF][CT];
#pragma unroll
    for (int p = 0; p < PF; p++)
#pragma unroll
        for (int c = 0; c < CT; c++) w[p][c] = weights(c, p * 16);
    for (int k0 = 0; k0 < K; k0 += 16 * PF) {
        const int kn = k0 + 16 * PF < K ? k0 + 16 * PF : 0;   // the last group requests the first again, unused
#pragma unroll
        for (int p = 0; p < PF; p++) {
            bf16x8 b[RT];
#pragma unroll
            for (int r = 0; r < RT; r++) b[r] = *(const bf16x8 *)(ap + r * 32 * LDA + k0 + p * 16);
            bf16x8 a[CT];
#pragma unroll
            for (int c = 0; c < CT; c++) {
                a[c] = w[p][c];
                w[p][c] = weights(c, kn + p * 16);
            }
#pragma unroll
            for (int r = 0; r < RT; r++)
#pragma unroll
                for (int c = 0; c < CT; c++)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c], b[r], acc[r][c], 0, 0, 0);
        }
    }
}

// The output layer's sums as the 64-lane butterfly adds them: leaf l is the FMA chain over units
// l * HPL .. + HPL - 1, and leaves combine by index bits 5, 4, ..., 0.  One thread takes the leaves of
// residue j = l % 4, l = j + 4 t, and returns their sum (bits 5 .. 2); bits 1 and 0 combine the residues.
struct Four { float c[4]; };
template <int HPL, int BIT, int T>
__device__ __forceinline__ Four head_leaves(const uint16_t *h, const float *w, int j) {
    Four s;
    if constexpr (BIT == 4) {
        const int u = (j + 4 * T) * HPL;
#pragma unroll
        for (int c = 0; c < 4; c++) s.c[c] = 0.f;
#pragma unroll
        for (int q = 0; q < HPL; q++) {
            const float x = from_bf16(h[u + q]);
#pragma unroll
            for (int c = 0; c < 4; c++) s.c[c] = fmaf(x, w[(u + q) * 4 + c], s.c[c]);
        }
    } else {
        const Four a = head_leaves<HPL, BIT + 1, T>(h, w, j);
        const Four b = head_leaves<HPL, BIT + 1, T | (1 << BIT)>(h, w, j);
#pragma unroll
        for (int c = 0; c < 4; c++) s.c[c] = a.c[c] + b.c[c];
    }
    return s;
}

// logits of one row by one wave (every lane returns them): the same sums, lane l holding leaf l
template <int HPL>
__device__ __forceinline__ void head_row(const float (&h)[HPL], const float (&wk)[HPL][4], const float *b, float (&z)[4]) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < HPL; j++) s = fmaf(h[j], wk[j][c], s);
        z[c] = s;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int c = 0; c < 4; c++) z[c] += __shfl_xor(z[c], off, 64);
#pragma unroll
    for (int c = 0; c < 4; c++) z[c] += b[c];
}

// Cross entropy of minibatch row r and its gradient dz by the logits z; with `store`, both and the row's
// weight go to memory.
__device__ __forceinline__ void loss_row(const RowsArgs &f, int r, float invw, const float (&z)[4], bool store,
                                         float (&dz)[4]) {
    const int64_t src = data_row(f.idx, f.n_data, r);
    const int n = min(max((int)f.nact[src], 1), 4);
    const float wr = (f.w ? f.w[src] : 1.f) * invw;
    float T[4];
#pragma unroll
    for (int c = 0; c < 4; c++) T[c] = f.T[src * 4 + c];
    float ls[4], lmax = -INFINITY;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        ls[c] = z[c] < LOG_CUT ? z[c] : logf(softplus_f(z[c]));
        if (c < n) lmax = fmaxf(lmax, ls[c]);
    }
    float se = 0.f;
#pragma unroll
    for (int c = 0; c < 4; c++)
        if (c < n) se += expf(ls[c] - lmax);
    const float lS = lmax + logf(se);
    float tsum = 0.f, ce = 0.f, t[4];
#pragma unroll
    for (int c = 0; c < 4; c++) {
        t[c] = c < n ? T[c] : 0.f;
        tsum += t[c];
        ce -= t[c] * (ls[c] - lS);
    }
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if (c < n) {
            const float ratio = z[c] < LOG_CUT ? 1.f : sigmoid_f(z[c]) / softplus_f(z[c]);
            const float lsig = -softplus_f(-z[c]);
            dz[c] = wr * (-t[c] * ratio + tsum * expf(lsig - lS));
        } else {
            dz[c] = 0.f;
        }
    }
    if (!store) return;
    *(float4 *)(f.dz + (int64_t)r * 4) = make_float4(dz[0], dz[1], dz[2], dz[3]);
    f.ce[r] = ce;
    f.wr[r] = wr;
}

// four consecutive units of a row as bf16, one 8-byte store
__device__ __forceinline__ void store4(uint16_t *p, float a, float b, float c, float d) {
    *(uint2 *)p = make_uint2(to_bf16x2(a, b), to_bf16x2(c, d));
}

// RT x CT tiles per wave, WR waves along the rows, HID / 32 / CT along the units
template <int HID, int K0, int RT, int CT, int WR, bool TRAIN>
__global__ __launch_bounds__(64 * WR * (HID / 32 / CT), TRAIN || RT * WR == 1 ? 1 : 2) void k_rows(RowsArgs f) {
    constexpr int WC = HID / 32 / CT, NW = WR * WC, NT = NW * 64;
    constexpr int ROWS = 32 * RT * WR;
    constexpr int LDA = (K0 > HID ? K0 : HID) + 8;   // rows stay 16-byte aligned and spread over the banks
    constexpr int PF = RT == 1 && CT == 1 ? (K0 < 128 || HID < 128 ? 4 : 8) : 4;
    constexpr int HPL = HID / 64;
    __shared__ __attribute__((aligned(16))) uint16_t act[ROWS * LDA];
    __shared__ __attribute__((aligned(16))) float red[TRAIN ? 256 : ROWS >= 64 ? ROWS * 16 : 1];
    __shared__ __attribute__((aligned(16))) float bias[4 * HID];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = blockIdx.x * ROWS;
    // the tile's input rows (zeros past the last), up to eight loads per thread in flight
    constexpr int PIECES = ROWS * (K0 / 8), IN_FLIGHT = (PIECES + NT - 1) / NT < 8 ? (PIECES + NT - 1) / NT : 8;
    for (int i0 = tid; i0 < PIECES; i0 += NT * IN_FLIGHT) {
        uint4 v[IN_FLIGHT];
#pragma unroll
        for (int p = 0; p < IN_FLIGHT; p++) {
            const int i = min(i0 + p * NT, PIECES - 1), r = min(r0 + i / (K0 / 8), f.rows - 1), c = (i % (K0 / 8)) * 8;
            // (any alignment of x)
            __builtin_memcpy(&v[p], f.x + (TRAIN ? data_row(f.idx, f.n_data, r) : (int64_t)r) * K0 + c, 16);
        }
#pragma unroll
        for (int p = 0; p < IN_FLIGHT; p++) {
            const int i = i0 + p * NT, r = i / (K0 / 8), c = (i % (K0 / 8)) * 8;
            if (i < PIECES) *(uint4 *)&act[r * LDA + c] = r0 + r < f.rows ? v[p] : make_uint4(0, 0, 0, 0);
        }
    }
    for (int l = 0; l < f.W.n_hidden; l++)
        for (int i = tid; i < HID; i += NT) bias[l * HID + i] = f.W.theta[f.W.boff[l] + i];
    // [row][unit] in LDS -> units as rows and rows as inputs in operand order in global memory (eight rows
    // of a unit per store), rows past the last as zeros
    auto put_transposed = [&](uint16_t *dst, int units) {
        for (int i = tid; i < units * (ROWS / 8); i += NT) {
            const int u = i % units, r = i / units * 8;
            uint16_t e[8];
#pragma unroll
            for (int j = 0; j < 8; j++) e[j] = r0 + r + j < f.rows ? act[(r + j) * LDA + u] : (uint16_t)0;
            uint4 v;
            __builtin_memcpy(&v, e, 16);
            *(uint4 *)(dst + operand_at(u, r0 + r, (int)f.ld)) = v;
        }
    };
    const float invw = TRAIN ? (f.inv_wsum ? *f.inv_wsum : inv_weight_sum(f.w, f.idx, f.n_data, f.rows, red)) : 0.f;
    __syncthreads();
    if constexpr (TRAIN) put_transposed(f.Xt, K0);
    const int m0 = wave / WC * (32 * RT), n0 = wave % WC * (32 * CT);
    const int unit4 = (lane >> 5) * 4, mrow = lane & 31;
    f32x16 acc[RT][CT];
    for (int l = 0; l < f.W.n_hidden; l++) {
        layer_mfma<RT, CT, LDA, PF>(f.W.fwd + f.W.wt_off[l], HID, l == 0 ? K0 : HID, act, m0, n0, acc);
        __syncthreads();   // every wave has read this layer's input: overwrite it
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int n = n0 + c * 32 + g * 8 + unit4;
                const float4 b = *(const float4 *)&bias[l * HID + n];
#pragma unroll
                for (int r = 0; r < RT; r++) {
                    const f32x16 &x = acc[r][c];
                    store4(&act[(m0 + r * 32 + mrow) * LDA + n], fmaxf(x[4 * g] + b.x, 0.f), fmaxf(x[4 * g + 1] + b.y, 0.f),
                           fmaxf(x[4 * g + 2] + b.z, 0.f), fmaxf(x[4 * g + 3] + b.w, 0.f));
                }
            }
        __syncthreads();
        if constexpr (TRAIN) {
            for (int i = tid; i < ROWS * (HID / 8); i += NT) {
                const int r = i / (HID / 8), c = (i % (HID / 8)) * 8;
                *(uint4 *)(f.H[l] + (int64_t)(r0 + r) * HID + c) = *(const uint4 *)&act[r * LDA + c];
            }
            put_transposed(f.Ht[l], HID);
        }
    }
    const float *w_out = f.W.out;
    const float *b_out = f.W.theta + f.W.boff[f.W.n_hidden];
    if constexpr (!TRAIN && ROWS >= 64) {
        // 64 rows and one residue per wave at a time, so the output weights are uniform over the wave
#pragma unroll 1
        for (int p = wave; p < ROWS / 16; p += NW) {
            // (a wave's items differ in the residue, so its weights are not kept in registers)
            const int j = p / (ROWS / 64), r = p % (ROWS / 64) * 64 + lane;
            const Four s = head_leaves<HPL, 0, 0>(act + r * LDA, w_out, j);
            *(float4 *)&red[(r * 4 + j) * 4] = make_float4(s.c[0], s.c[1], s.c[2], s.c[3]);
        }
        __syncthreads();
        for (int i = tid; i < ROWS * 4; i += NT) {
            const int r = i / 4, c = i % 4;
            const float *s = &red[r * 16 + c];
            if (r0 + r < f.rows) f.z[(int64_t)(r0 + r) * 4 + c] = ((s[0] + s[8]) + (s[4] + s[12])) + b_out[c];
        }
    } else {
        float wk[HPL][4];
#pragma unroll
        for (int j = 0; j < HPL; j++)
#pragma unroll
            for (int c = 0; c < 4; c++) wk[j][c] = w_out[(lane * HPL + j) * 4 + c];
        constexpr int RPW = ROWS / NW;   // this wave's rows: wave, wave + NW, ...
        static_assert(RPW <= 64, "a lane per row of the wave");
        float zl[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int q = 0; q < RPW; q++) {
            const uint16_t *hr = &act[(wave + q * NW) * LDA + lane * HPL];
            float h[HPL], z[4];
#pragma unroll
            for (int j = 0; j < HPL; j++) h[j] = from_bf16(hr[j]);
            head_row<HPL>(h, wk, b_out, z);
#pragma unroll
            for (int c = 0; c < 4; c++) zl[c] = lane == q ? z[c] : zl[c];
        }
        // lane q holds the logits of the wave's row q
        const int r = r0 + wave + min(lane, RPW - 1) * NW;
        const bool in = lane < RPW && r < f.rows;
        if constexpr (!TRAIN) {
            for (int c = 0; c < 4; c++)
                if (in) f.z[(int64_t)r * 4 + c] = zl[c];
        } else {
            float dz[4];
            loss_row(f, min(r, f.rows - 1), invw, zl, in, dz);
            __syncthreads();   // the last activations are stored before gradients replace them
#pragma unroll 4
            for (int q = 0; q < RPW; q++) {
                uint16_t *hr = &act[(wave + q * NW) * LDA + lane * HPL];
                float g[4];
#pragma unroll
                for (int c = 0; c < 4; c++) g[c] = __shfl(dz[c], q, 64);
                const bool pad = r0 + wave + q * NW >= f.rows;   // no gradient
#pragma unroll
                for (int j = 0; j < HPL; j++) {
                    float d = 0.f;
#pragma unroll
                    for (int c = 0; c < 4; c++) d = fmaf(g[c], wk[j][c], d);
                    hr[j] = to_bf16(!pad && from_bf16(hr[j]) > 0.f ? d : 0.f);
                }
            }
        }
        if constexpr (TRAIN) {
            // act holds the gradient of the last hidden pre-activation: store it, then the one before it is
            // (dA W_l^T) where the activation is positive, and so on
            for (int l = f.W.n_hidden - 1;; l--) {
                __syncthreads();
                put_transposed(f.dAt[l], HID);
                for (int i = tid; i < HID * (ROWS / BIAS_ROWS); i += NT) {
                    const int u = i % HID, q = i / HID;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < BIAS_ROWS; r++)
                        if (r0 + q * BIAS_ROWS + r < f.rows) sum += from_bf16(act[(q * BIAS_ROWS + r) * LDA + u]);
                    f.bias_part[l][(int64_t)(r0 / BIAS_ROWS + q) * HID + u] = sum;
                }
                if (l == 0) break;
                layer_mfma<RT, CT, LDA, PF>(f.W.bwd + f.W.wt_off[l], HID, HID, act, m0, n0, acc);
                __syncthreads();
#pragma unroll
                for (int c = 0; c < CT; c++)
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        const int n = n0 + c * 32 + g * 8 + unit4;
#pragma unroll
                        for (int r = 0; r < RT; r++) {
                            const int m = m0 + r * 32 + mrow;
                            const uint2 k = *(const uint2 *)(f.H[l - 1] + (int64_t)(r0 + m) * HID + n);
                            const f32x16 &x = acc[r][c];
                            store4(&act[m * LDA + n], from_bf16((uint16_t)k.x) > 0.f ? x[4 * g] : 0.f,
                                   from_bf16((uint16_t)(k.x >> 16)) > 0.f ? x[4 * g + 1] : 0.f,
                                   from_bf16((uint16_t)k.y) > 0.f ? x[4 * g + 2] : 0.f,
                                   from_bf16((uint16_t)(k.y >> 16)) > 0.f ? x[4 * g + 3] : 0.f);
                        }
                    }
            }
        }
    }
}

// ---- gradients: sums over rows ---------------------------------------------------------------
constexpr int HEAD_BLOCKS = 256;

// floats from one row of the output layer's partials to the next (HID * 4 weights, 4 biases, the loss): a multiple
// of four, so that every row starts on a 16-byte line for the vector stores
__host__ __device__ constexpr int head_row(int hid) { return hid * 4 + 8; }
static_assert(head_row(64) % 4 == 0 && head_row(128) % 4 == 0 && head_row(256) % 4 == 0, "float4 stores of a partial row");

struct GradArgs {
    Weights W;
    int rows, splits, kchunk, head_blocks;
    int64_t ld;
    const uint16_t *in[4];    // transposed inputs of hidden layer l (operand order, as RowsArgs)
    const uint16_t *dAt[4];   // and gradients
    const uint16_t *H;        // [ld][HID] last activations
    const float *dz, *ce, *wr;
    float *w_part[4];         // [splits][fan in][HID]
    float *bias_part[4];      // [ceil(rows / BIAS_ROWS)][HID]
    float *head_part;         // [head_blocks][head_row(HID)]: output weights, biases, loss
    int task0[5];             // first task of each hidden layer's weight gradient; task0[n_hidden] tasks in all
    float *grad, *loss, *m, *v;
    float lr, b1, b2, eps, c1, c2;   // Adam
};

// Blocks [0, ceil(tasks / 4)): a wave per 64 x 64 tile of a layer's weight gradient and range of kchunk rows,
// in[m][r] dA[n][r] summed over r in ascending steps of 16; both are in operand order, so they go from L2
// straight to the matrix cores, 64 rows requested ahead.  The blocks after that: one each of the output layer's partials,
// rows b * 4 + w, + 4 * head_blocks, ... of wave w in order, then waves 0 to 3.
template <int HID>
__global__ __launch_bounds__(256) void k_wgrad(GradArgs f) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int L = f.W.n_hidden;
    const int mma_blocks = (f.task0[L] + 3) / 4;
    if ((int)blockIdx.x >= mma_blocks) {
        const int b = blockIdx.x - mma_blocks;
        float *out = f.head_part + (int64_t)b * head_row(HID);
        if (tid < HID) {
            float tot[4];
            for (int w = 0; w < 4; w++) {
                float g[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
                for (int r = b * 4 + w; r < f.rows; r += f.head_blocks * 4) {
                    const float h = from_bf16(f.H[(int64_t)r * HID + tid]);
                    const float4 d = *(const float4 *)(f.dz + (int64_t)r * 4);
                    g[0] = fmaf(h, d.x, g[0]); g[1] = fmaf(h, d.y, g[1]);
                    g[2] = fmaf(h, d.z, g[2]); g[3] = fmaf(h, d.w, g[3]);
                }
#pragma unroll
                for (int c = 0; c < 4; c++) tot[c] = w == 0 ? g[c] : tot[c] + g[c];
            }
            *(float4 *)(out + tid * 4) = make_float4(tot[0], tot[1], tot[2], tot[3]);
        }
        if (tid < 5) {
            float tot = 0.f;
            for (int w = 0; w < 4; w++) {
                float g = 0.f;
                for (int r = b * 4 + w; r < f.rows; r += f.head_blocks * 4) {
                    if (tid < 4) g += f.dz[(int64_t)r * 4 + tid];
                    else g = fmaf(f.wr[r], f.ce[r], g);
                }
                tot = w == 0 ? g : tot + g;
            }
            out[HID * 4 + tid] = tot;
        }
        return;
    }
    const int task = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (tid >> 6));
    if (task >= f.task0[L]) return;
    int l = 0;
    while (l + 1 < L && task >= f.task0[l + 1]) l++;
    const int fi = l == 0 ? f.W.in_dim : HID, tiles = (fi / 64) * (HID / 64);
    const int t = task - f.task0[l], split = t / tiles, tile = t % tiles;
    const int m0 = tile / (HID / 64) * 64, n0 = tile % (HID / 64) * 64;
    const int k_beg = split * f.kchunk, k_end = min(k_beg + f.kchunk, (f.rows + 31) / 32 * 32);
    // 32 units x 16 rows are 512 values; the 32 units after them start ld / 16 such pieces later
    const int64_t next = f.ld * 32;
    const uint16_t *ap = f.in[l] + (m0 >> 5) * next + lane * 8, *bp = f.dAt[l] + (n0 >> 5) * next + lane * 8;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 16; i++) acc[0][0][i] = acc[0][1][i] = acc[1][0][i] = acc[1][1][i] = 0.f;
    constexpr int S = 4;
    for (int k = k_beg; k < k_end; k += 16 * S) {
        bf16x8 a[S][2], b[S][2];
#pragma unroll
        for (int s = 0; s < S; s++)
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const int64_t at = (int64_t)min(k + s * 16, k_end - 16) * 32 + i * next;
                a[s][i] = *(const bf16x8 *)(ap + at);
                b[s][i] = *(const bf16x8 *)(bp + at);
            }
#pragma unroll
        for (int s = 0; s < S; s++)
            if (k + s * 16 < k_end) {
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s][i], b[s][j], acc[i][j], 0, 0, 0);
            }
    }
    // accumulator q of lane l holds row 8 (q / 4) + 4 (l / 32) + q % 4, column l % 32
    float *out = f.w_part[l] + (int64_t)split * fi * HID;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const int row = m0 + i * 32 + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3), col = n0 + j * 32 + (lane & 31);
                out[(int64_t)row * HID + col] = acc[i][j][q];
            }
}

// sum over b < nb of part[b * stride], in order of b, U loads in flight
template <int U>
__device__ __forceinline__ float ordered_sum(const float *part, int nb, int64_t stride) {
    float s = 0.f;
    int b = 0;
    for (; b + U <= nb; b += U) {
        float x[U];
#pragma unroll
        for (int i = 0; i < U; i++) x[i] = part[(int64_t)(b + i) * stride];
#pragma unroll
        for (int i = 0; i < U; i++) s += x[i];
    }
    for (; b < nb; b++) s += part[(int64_t)b * stride];
    return s;
}

// the bf16 copies of parameter i
__device__ __forceinline__ void put_bf16(const Weights &W, int64_t i, float x) {
    const uint16_t h = to_bf16(x);
    const int64_t o = i - W.woff[W.n_hidden];
    if (o >= 0 && o < W.hidden * 4) W.out[o] = from_bf16(h);
    for (int l = 0; l < W.n_hidden; l++) {
        const int64_t e = i - W.woff[l];
        const int fin = l == 0 ? W.in_dim : W.hidden;
        if (e >= 0 && e < (int64_t)fin * W.hidden) {
            const int k = (int)(e / W.hidden), n = (int)(e % W.hidden);
            W.fwd[W.wt_off[l] + operand_at(n, k, fin)] = h;
            W.bwd[W.wt_off[l] + operand_at(k, n, W.hidden)] = h;
        }
    }
}

// Adam (Kingma and Ba 2015, Algorithm 1) on the FP32 master copy of one parameter; refreshes the bf16
// copies.  c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t) for step t.
__device__ __forceinline__ void adam_one(const GradArgs &f, int64_t i, float gi) {
    const float mi = fmaf(1.f - f.b1, gi, f.b1 * f.m[i]);
    const float vi = fmaf(gi, (1.f - f.b2) * gi, f.b2 * f.v[i]);
    f.m[i] = mi;
    f.v[i] = vi;
    const float th = f.W.theta[i] - f.lr * (mi * f.c1) / (sqrtf(vi * f.c2) + f.eps);
    f.W.theta[i] = th;
    put_bf16(f.W, i, th);
}

__global__ __launch_bounds__(256) void k_adam(GradArgs f, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) adam_one(f, i, f.grad[i]);
}

// Every parameter's gradient from its partials (and the loss, as element P), then, with ADAM, its update.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_finish(GradArgs f, int64_t P) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > P) return;
    const int L = f.W.n_hidden, HID = f.W.hidden;
    float g;
    if (i >= f.W.woff[L]) {
        // output weights and biases are contiguous in the partial rows as in the parameters, then the loss
        g = ordered_sum<64>(f.head_part + (i - f.W.woff[L]), f.head_blocks, head_row(HID));
        if (i == P) {
            f.loss[0] = g;
            return;
        }
    } else {
        int l = 0;
        while (l + 1 < L && i >= f.W.woff[l + 1]) l++;
        const int fin = l == 0 ? f.W.in_dim : HID;
        if (i < f.W.boff[l]) g = ordered_sum<16>(f.w_part[l] + (i - f.W.woff[l]), f.splits, (int64_t)fin * HID);
        else g = ordered_sum<64>(f.bias_part[l] + (i - f.W.boff[l]), (f.rows + BIAS_ROWS - 1) / BIAS_ROWS, HID);
    }
    f.grad[i] = g;
    if constexpr (ADAM) adam_one(f, i, g);
}

__global__ __launch_bounds__(256) void k_refresh(Weights W, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) put_bf16(W, i, W.theta[i]);
}

// ---- compiled game <-> network rows --------------------------------------------------------
// Columns 120-127 after a probe run: the current strategy (regret matching of the latest regrets)
// and the normalised average strategy over the first four actions (uniform where the sum is 0;
// zero for sets of more than four actions).  One thread per set writes the 16-byte chunk.
template <typename T>
__global__ __launch_bounds__(256) void k_features_probe(FeatureArgs f, const T *sigma, const double *sbar) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= f.I) return;
    const int off = f.canon_off[i], n = f.canon_off[i + 1] - off;
    float col[8];
#pragma unroll
    for (int j = 0; j < 8; j++) col[j] = 0.f;
    if (n <= 4) {
        double sb[4] = {0, 0, 0, 0}, tot = 0.0;
        for (int a = 0; a < n; a++) {
            const int q = f.slot_map ? f.slot_map[off + a] : off + a;
            col[a] = (float)sigma[q];
            sb[a] = sbar[q];
            tot += sb[a];
        }
        for (int a = 0; a < n; a++) col[4 + a] = tot > 0.0 ? (float)(sb[a] / tot) : (float)(1.0 / n);
    }
    uint16_t o[8];
#pragma unroll
    for (int j = 0; j < 8; j++) o[j] = to_bf16(col[j]);
    *(uint4 *)(f.X + i * 128 + 120) = *(const uint4 *)o;
}

// Feature row of information set i (16 threads per row, 8 columns each), and mag[i], the sum of
// the magnitudes of those regrets (the unit of the warm-start regrets):
//   0-63 one-hot hand bucket, 64-95 one-hot public-history code, 96-103 caller scalars,
//   104-107 legal-action mask, 108-111 the first four instantaneous regrets of the uniform
//   strategy over the sum of their magnitudes, 112-115 regret matching (plus) of those regrets,
//   116 acting player (0 / 1), 117-119 zero, 120-127 the strategies of a probe run (uniform here;
//   k_features_probe overwrites them after one).
template <typename T>
__global__ __launch_bounds__(256) void k_features(FeatureArgs f, const T *R) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = t >> 4;
    const int chunk = (int)(t & 15);
    if (i >= f.I) return;
    float col[8];
#pragma unroll
    for (int j = 0; j < 8; j++) col[j] = 0.f;
    const int c0 = chunk * 8;
    if (c0 < 64) {
        const int b = f.bucket[i];
        if (b >= c0 && b < c0 + 8) col[b - c0] = 1.f;
    } else if (c0 < 96) {
        const int hcode = f.history[i];
        if (hcode >= c0 - 64 && hcode < c0 - 56) col[hcode - (c0 - 64)] = 1.f;
    } else if (c0 == 96) {
#pragma unroll
        for (int j = 0; j < 8; j++) col[j] = f.scalars[i * 8 + j];
    } else if (c0 == 104 || c0 == 112) {
        const int off = f.canon_off[i], n = f.canon_off[i + 1] - off;
        const int k = min(n, 4);
        double r[4] = {0, 0, 0, 0}, sa = 0.0, sp = 0.0;
        if (n <= 4)
            for (int a = 0; a < k; a++) {
                const int q = f.slot_map ? f.slot_map[off + a] : off + a;
                r[a] = (double)R[q];
                sa += fabs(r[a]);
                sp += r[a] > 0.0 ? r[a] : 0.0;
            }
        if (c0 == 104) {
            f.mag[i] = n <= 4 ? (float)sa : 0.f;
            for (int a = 0; a < k; a++) col[a] = 1.f;
            if (n <= 4 && sa > 0.0)
                for (int a = 0; a < k; a++) col[4 + a] = (float)(r[a] / sa);
        } else {
            if (n <= 4)
                for (int a = 0; a < k; a++) col[a] = sp > 0.0 ? (float)((r[a] > 0.0 ? r[a] : 0.0) / sp) : (float)(1.0 / k);
            col[4] = f.player[i] == 2 ? 1.f : 0.f;
        }
    } else if (c0 == 120) {
        const int n = f.canon_off[i + 1] - f.canon_off[i];
        if (n <= 4)
            for (int a = 0; a < n; a++) col[a] = col[4 + a] = (float)(1.0 / n);
    }
    uint16_t o[8];
#pragma unroll
    for (int j = 0; j < 8; j++) o[j] = to_bf16(col[j]);
    *(uint4 *)(f.X + i * 128 + c0) = *(const uint4 *)o;
}

// R0 over canonical slots: scale * mag(I) * softplus(z) for the legal actions of sets with <= 4
// actions, 0 (the uniform strategy) for larger sets
__global__ void k_warm_regrets(const int32_t *canon_off, int64_t I, const float *z, const float *mag, float scale,
                               float *R0) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= I) return;
    const int off = canon_off[i], n = canon_off[i + 1] - off;
    const float c = scale * mag[i];
    for (int a = 0; a < n; a++) R0[off + a] = n <= 4 ? c * softplus_f(z[i * 4 + a]) : 0.f;
}

}  // namespace

hipError_t launch_features(const FeatureArgs &f, const void *R, bool fp64, hipStream_t s) {
    if (f.I == 0) return hipSuccess;
    const int64_t threads = f.I * 16;
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    if (fp64) k_features<double><<<blocks, 256, 0, s>>>(f, (const double *)R);
    else k_features<float><<<blocks, 256, 0, s>>>(f, (const float *)R);
    return hipGetLastError();
}

hipError_t launch_features_probe(const FeatureArgs &f, const void *sigma, const double *sbar, bool fp64,
                                 hipStream_t s) {
    if (f.I == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((f.I + 255) / 256);
    if (fp64) k_features_probe<double><<<blocks, 256, 0, s>>>(f, (const double *)sigma, sbar);
    else k_features_probe<float><<<blocks, 256, 0, s>>>(f, (const float *)sigma, sbar);
    return hipGetLastError();
}

hipError_t launch_warm_regrets(const int32_t *canon_off, int64_t I, const float *z, const float *mag, float scale,
                               float *R0, hipStream_t s) {
    if (I == 0) return hipSuccess;
    k_warm_regrets<<<(unsigned)((I + 255) / 256), 256, 0, s>>>(canon_off, I, z, mag, scale, R0);
    return hipGetLastError();
}

}  // namespace cfrx

using namespace cfrx;

// ---- the network handle ---------------------------------------------------------------------
struct cfr_mlp {
    cfr_mlp_desc d{};
    std::vector<int> fin, fout;          // per layer
    std::vector<int64_t> woff, boff;     // offsets into the flat parameter vector
    int64_t P = 0;
    int64_t step = 0;
    float *theta = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr, *inv_w = nullptr, *lossd = nullptr;
    uint16_t *w_fwd = nullptr, *w_bwd = nullptr;   // bf16 weights (see Weights)
    float *w_out = nullptr;
    int64_t wt_off[4] = {0, 0, 0, 0};
    // training, rows padded to a multiple of 32 (zeros): see RowsArgs and GradArgs
    uint16_t *H[4] = {}, *Ht[4] = {}, *dAt[4] = {}, *Xt = nullptr;
    float *dz = nullptr, *ce = nullptr, *wr = nullptr, *bias_part[4] = {}, *w_part[4] = {}, *head_part = nullptr;
    void *memory = nullptr;
};

namespace {
cfr_status mfail(cfr_status s, const std::string &m) {
    set_last_error(m);
    return s;
}

#define MHIP(expr)                                                                                      \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return mfail(CFR_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

// The network's buffers are placed one after another, each on a 256-byte line of its own, in one allocation:
// the device takes 10 to 40 us for each, and a network of three layers has 28.
struct Placement {
    std::vector<std::pair<void **, size_t>> at;
    size_t bytes = 0;
    template <typename T>
    void add(T **p, int64_t count) {
        at.push_back({(void **)p, bytes});
        bytes += ((size_t)(count > 0 ? count : 1) * sizeof(T) + 255) / 256 * 256;
    }
};

void free_mlp(cfr_mlp *n) {
    if (n->memory) (void)hipFree(n->memory);
    delete n;
}

// rows per partial sum of the weight gradients: at most 32 splits of at least 256 rows
int gemm_splits(int rows) { return std::min(std::max((rows + 255) / 256, 1), 32); }

constexpr int SMALL_ROWS = 8192;   // up to here a 32-row tile per block
constexpr int ROW_PAD = 128;       // training rows are padded to the largest training tile

Weights weights_of(const cfr_mlp *n) {
    Weights W{};
    W.theta = n->theta; W.fwd = n->w_fwd; W.bwd = n->w_bwd; W.out = n->w_out;
    for (int l = 0; l <= n->d.n_hidden; l++) { W.woff[l] = n->woff[(size_t)l]; W.boff[l] = n->boff[(size_t)l]; }
    for (int l = 0; l < n->d.n_hidden; l++) W.wt_off[l] = n->wt_off[l];
    W.n_hidden = n->d.n_hidden; W.in_dim = n->d.in_dim; W.hidden = n->d.hidden;
    return W;
}

template <int HID, int K0, bool TRAIN>
hipError_t rows_tile(const RowsArgs &f, hipStream_t s) {
    auto go = [&](auto rt, auto ct, auto wr) {
        constexpr int RT = decltype(rt)::value, CT = decltype(ct)::value, WR = decltype(wr)::value;
        constexpr int ROWS = 32 * RT * WR;
        const unsigned blocks = (unsigned)(((int64_t)f.rows + ROWS - 1) / ROWS);
        k_rows<HID, K0, RT, CT, WR, TRAIN><<<blocks, 64 * WR * (HID / 32 / CT), 0, s>>>(f);
        return hipGetLastError();
    };
    using std::integral_constant;
    using One = integral_constant<int, 1>;
    using Two = integral_constant<int, 2>;
    using Four_ = integral_constant<int, 4>;
    if (f.rows <= SMALL_ROWS) return go(One{}, One{}, One{});
    if constexpr (TRAIN) return go(Four_{}, One{}, One{});
    else if constexpr (HID == 256) return go(Four_{}, Two{}, One{});
    else if constexpr (HID == 128) return go(Two{}, Two{}, Two{});
    else return go(One{}, Two{}, Four_{});
}

template <bool TRAIN>
hipError_t launch_rows(const RowsArgs &f, hipStream_t s) {
#define SHAPE(H_, K_) if (f.W.hidden == H_ && f.W.in_dim == K_) return rows_tile<H_, K_, TRAIN>(f, s);
    SHAPE(64, 64) SHAPE(64, 128) SHAPE(64, 256) SHAPE(128, 64) SHAPE(128, 128) SHAPE(128, 256)
    SHAPE(256, 64) SHAPE(256, 128) SHAPE(256, 256)
#undef SHAPE
    return hipErrorInvalidValue;
}

constexpr int NOALLOC_ROWS = 8192;

// the constants of the next Adam step
void set_adam(cfr_mlp *n, float lr, GradArgs &g) {
    n->step++;
    const double t = (double)n->step;
    g.lr = lr; g.b1 = n->d.beta1; g.b2 = n->d.beta2; g.eps = n->d.eps;
    g.c1 = (float)(1.0 / (1.0 - std::pow((double)n->d.beta1, t)));
    g.c2 = (float)(1.0 / (1.0 - std::pow((double)n->d.beta2, t)));
}

bool valid_desc(const cfr_mlp_desc *d, std::string &why) {
    auto ok_dim = [](int v) { return v == 64 || v == 128 || v == 256; };
    if (!ok_dim(d->in_dim)) { why = "in_dim must be 64, 128 or 256"; return false; }
    if (!ok_dim(d->hidden)) { why = "hidden must be 64, 128 or 256"; return false; }
    if (d->n_hidden < 1 || d->n_hidden > 4) { why = "n_hidden must be in [1, 4]"; return false; }
    if (d->max_rows < 1 || d->max_rows > (1 << 20)) { why = "max_rows must be in [1, 2^20]"; return false; }
    if (!(d->beta1 >= 0.f && d->beta1 < 1.f && d->beta2 >= 0.f && d->beta2 < 1.f && d->eps > 0.f)) {
        why = "Adam constants out of range"; return false;
    }
    return true;
}

}  // namespace

extern "C" {

void cfr_mlp_default_desc(cfr_mlp_desc *d) {
    if (!d) return;
    std::memset(d, 0, sizeof *d);
    d->in_dim = CFR_FEATURES;
    d->hidden = 256;
    d->n_hidden = 3;
    d->max_rows = 4096;
    d->device = 0;
    d->beta1 = 0.9f;
    d->beta2 = 0.999f;
    d->eps = 1e-8f;
}

cfr_status cfr_mlp_create(const cfr_mlp_desc *desc, cfr_mlp **out) {
    if (!out) return mfail(CFR_EINVAL, "out is NULL");
    *out = nullptr;
    cfr_mlp_desc d;
    cfr_mlp_default_desc(&d);
    if (desc) d = *desc;
    std::string why;
    if (!valid_desc(&d, why)) return mfail(CFR_EINVAL, why);
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) return mfail(CFR_EDEVICE, "no HIP device available");
    if (d.device < 0 || d.device >= ndev) return mfail(CFR_EINVAL, "device ordinal out of range");
    MHIP(hipSetDevice(d.device));
    cfr_mlp *n = new cfr_mlp();
    n->d = d;
    int prev = d.in_dim;
    for (int l = 0; l <= d.n_hidden; l++) {
        const int fo = l < d.n_hidden ? d.hidden : CFR_MLP_OUT;
        n->fin.push_back(prev);
        n->fout.push_back(fo);
        n->woff.push_back(n->P);
        n->P += (int64_t)prev * fo;
        n->boff.push_back(n->P);
        n->P += fo;
        prev = fo;
    }
    // rows of the training buffers, a multiple of the largest row tile
    const int64_t R = (d.max_rows + ROW_PAD - 1) / ROW_PAD * ROW_PAD;
    const int64_t hid = d.hidden;
    Placement place;
#define MA(p, c) place.add(&(p), (c))
    MA(n->theta, n->P); MA(n->grad, n->P); MA(n->m, n->P); MA(n->v, n->P);
    {
        int64_t off = 0;
        for (int l = 0; l < d.n_hidden; l++) { n->wt_off[l] = off; off += (int64_t)n->fin[(size_t)l] * hid; }
        MA(n->w_fwd, off); MA(n->w_bwd, off); MA(n->w_out, hid * 4);
    }
    MA(n->inv_w, 1);
    MA(n->lossd, 1);
    for (int l = 0; l < d.n_hidden; l++) {
        MA(n->H[l], R * hid); MA(n->Ht[l], R * hid); MA(n->dAt[l], R * hid);
        MA(n->bias_part[l], (R + BIAS_ROWS - 1) / BIAS_ROWS * hid);
        MA(n->w_part[l], (int64_t)gemm_splits((int)d.max_rows) * n->fin[(size_t)l] * hid);
    }
    MA(n->Xt, R * d.in_dim); MA(n->dz, R * 4); MA(n->ce, R); MA(n->wr, R);
    MA(n->head_part, (int64_t)HEAD_BLOCKS * head_row(d.hidden));
#undef MA
    hipError_t e = hipMalloc(&n->memory, place.bytes);
    if (e != hipSuccess) {
        free_mlp(n);
        return mfail(CFR_ENOMEM, "hipMalloc of " + std::to_string(place.bytes) + " bytes failed");
    }
    for (auto &[p, off] : place.at) *p = (char *)n->memory + off;
    // zero parameters until the caller sets them
    e = hipMemset(n->theta, 0, (size_t)n->P * 4);
    if (e == hipSuccess) {   // and the bf16 copies with them
        k_refresh<<<(unsigned)((n->P + 255) / 256), 256>>>(weights_of(n), n->P);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemset(n->m, 0, (size_t)n->P * 4);
    if (e == hipSuccess) e = hipMemset(n->v, 0, (size_t)n->P * 4);
    if (e == hipSuccess) e = hipMemset(n->grad, 0, (size_t)n->P * 4);
    // the first call may come on a stream that the null stream does not order
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) { free_mlp(n); return mfail(CFR_EDEVICE, std::string("network setup: ") + hipGetErrorString(e)); }
    *out = n;
    return CFR_OK;
}

cfr_status cfr_mlp_num_params(cfr_mlp *n, int64_t *count) {
    if (!n || !count) return mfail(CFR_EINVAL, "NULL argument");
    *count = n->P;
    return CFR_OK;
}

cfr_status cfr_mlp_set_params(cfr_mlp *n, const float *params, int64_t len) {
    if (!n || !params) return mfail(CFR_EINVAL, "NULL argument");
    if (len != n->P) return mfail(CFR_EINVAL, "len must equal the parameter count " + std::to_string(n->P));
    MHIP(hipSetDevice(n->d.device));
    MHIP(hipDeviceSynchronize());
    MHIP(hipMemcpy(n->theta, params, (size_t)len * 4, hipMemcpyHostToDevice));
    MHIP(hipMemset(n->m, 0, (size_t)len * 4));
    MHIP(hipMemset(n->v, 0, (size_t)len * 4));
    k_refresh<<<(unsigned)((len + 255) / 256), 256>>>(weights_of(n), len);
    MHIP(hipGetLastError());
    MHIP(hipDeviceSynchronize());
    n->step = 0;
    return CFR_OK;
}

cfr_status cfr_mlp_get(cfr_mlp *n, int which, float *dst, int64_t len) {
    if (!n || !dst) return mfail(CFR_EINVAL, "NULL argument");
    if (len != n->P) return mfail(CFR_EINVAL, "len must equal the parameter count " + std::to_string(n->P));
    const float *src = which == CFR_MLP_PARAMS ? n->theta : which == CFR_MLP_GRADS ? n->grad
                     : which == CFR_MLP_ADAM_M ? n->m : which == CFR_MLP_ADAM_V ? n->v : nullptr;
    if (!src) return mfail(CFR_EINVAL, "unknown buffer");
    MHIP(hipSetDevice(n->d.device));
    MHIP(hipDeviceSynchronize());
    MHIP(hipMemcpy(dst, src, (size_t)len * 4, hipMemcpyDeviceToHost));
    return CFR_OK;
}

cfr_status cfr_mlp_forward(cfr_mlp *n, const void *x, int64_t rows, float *z, void *stream) {
    if (!n || ((!x || !z) && rows > 0) || rows < 0) return mfail(CFR_EINVAL, "bad argument");
    MHIP(hipSetDevice(n->d.device));
    RowsArgs f{};
    f.W = weights_of(n);
    // launches of at most 2^27 rows keep every row index in int
    const int64_t step = (int64_t)1 << 27;
    for (int64_t r0 = 0; r0 < rows; r0 += step) {
        f.rows = (int)std::min(step, rows - r0);
        f.x = (const uint16_t *)x + r0 * n->d.in_dim;
        f.z = z + r0 * 4;
        MHIP(launch_rows<false>(f, (hipStream_t)stream));
    }
    return CFR_OK;
}

cfr_status cfr_mlp_forward_noalloc(cfr_mlp *n, const void *x, int64_t rows, float *z, void *stream) {
    if (!n || ((!x || !z) && rows > 0) || rows < 0) return mfail(CFR_EINVAL, "bad argument");
    if (rows > NOALLOC_ROWS)
        return mfail(CFR_EINVAL, "cfr_mlp_forward_noalloc takes at most " + std::to_string(NOALLOC_ROWS) +
                                 " rows per call (" + std::to_string(rows) + " given)");
    return cfr_mlp_forward(n, x, rows, z, stream);
}

// gradients of one minibatch into n->grad and the loss into n->lossd, then, with adam, the update of step
// n->step with learning rate lr
static cfr_status gradients(cfr_mlp *n, const void *x, const float *target, const float *weight, const uint8_t *nact,
                            const int32_t *idx, int64_t n_data, int64_t rows, bool adam, float lr, hipStream_t s) {
    if (!n || !x || !target || !nact || rows <= 0) return mfail(CFR_EINVAL, "bad argument");
    if (rows > n->d.max_rows) return mfail(CFR_EINVAL, "rows exceeds max_rows " + std::to_string(n->d.max_rows));
    if (idx && n_data <= 0) return mfail(CFR_EINVAL, "n_data must be positive with an index list");
    MHIP(hipSetDevice(n->d.device));
    const int R = (int)rows, L = n->d.n_hidden, HID = n->d.hidden;
    RowsArgs f{};
    f.W = weights_of(n);
    f.x = (const uint16_t *)x; f.rows = R; f.idx = idx; f.n_data = n_data;
    f.T = target; f.w = weight; f.nact = nact;
    f.ld = (R + ROW_PAD - 1) / ROW_PAD * ROW_PAD;
    f.Xt = n->Xt; f.dz = n->dz; f.ce = n->ce; f.wr = n->wr;
    for (int l = 0; l < L; l++) { f.H[l] = n->H[l]; f.Ht[l] = n->Ht[l]; f.dAt[l] = n->dAt[l]; f.bias_part[l] = n->bias_part[l]; }
    if (R > WSUM_ROWS) {
        k_inv_wsum<<<1, 256, 0, s>>>(weight, idx, n_data, R, n->inv_w);
        MHIP(hipGetLastError());
        f.inv_wsum = n->inv_w;
    }
    MHIP(launch_rows<true>(f, s));
    GradArgs g{};
    g.W = f.W; g.rows = R; g.ld = f.ld;
    const int want = gemm_splits(R);
    g.kchunk = ((R + want - 1) / want + 31) / 32 * 32;
    g.splits = (R + g.kchunk - 1) / g.kchunk;
    g.head_blocks = std::min(HEAD_BLOCKS, (R + 3) / 4);
    g.H = n->H[L - 1]; g.dz = n->dz; g.ce = n->ce; g.wr = n->wr; g.head_part = n->head_part;
    for (int l = 0; l < L; l++) {
        g.in[l] = l == 0 ? n->Xt : n->Ht[l - 1];
        g.dAt[l] = n->dAt[l]; g.w_part[l] = n->w_part[l]; g.bias_part[l] = n->bias_part[l];
        g.task0[l + 1] = g.task0[l] + (n->fin[(size_t)l] / 64) * (HID / 64) * g.splits;
    }
    g.grad = n->grad; g.loss = n->lossd; g.m = n->m; g.v = n->v;
    const unsigned blocks = (unsigned)((g.task0[L] + 3) / 4 + g.head_blocks);
    if (HID == 256) k_wgrad<256><<<blocks, 256, 0, s>>>(g);
    else if (HID == 128) k_wgrad<128><<<blocks, 256, 0, s>>>(g);
    else k_wgrad<64><<<blocks, 256, 0, s>>>(g);
    MHIP(hipGetLastError());
    const unsigned fb = (unsigned)((n->P + 1 + 255) / 256);
    if (adam) {
        set_adam(n, lr, g);
        k_finish<true><<<fb, 256, 0, s>>>(g, n->P);
    } else {
        k_finish<false><<<fb, 256, 0, s>>>(g, n->P);
    }
    MHIP(hipGetLastError());
    return CFR_OK;
}

static cfr_status read_loss(cfr_mlp *n, double *loss, hipStream_t s) {
    if (!loss) return CFR_OK;
    float lh = 0.f;
    MHIP(hipMemcpyAsync(&lh, n->lossd, 4, hipMemcpyDeviceToHost, s));
    MHIP(hipStreamSynchronize(s));
    *loss = lh;
    return CFR_OK;
}

cfr_status cfr_mlp_backward(cfr_mlp *n, const void *x, const float *target, const float *weight,
                            const uint8_t *nact, const int32_t *idx, int64_t n_data, int64_t rows, double *loss,
                            void *stream) {
    cfr_status st = gradients(n, x, target, weight, nact, idx, n_data, rows, false, 0.f, (hipStream_t)stream);
    return st == CFR_OK ? read_loss(n, loss, (hipStream_t)stream) : st;
}

cfr_status cfr_mlp_adam(cfr_mlp *n, float lr, void *stream) {
    if (!n) return mfail(CFR_EINVAL, "NULL argument");
    if (!(lr >= 0.f)) return mfail(CFR_EINVAL, "lr must be >= 0");
    MHIP(hipSetDevice(n->d.device));
    GradArgs g{};
    g.W = weights_of(n); g.grad = n->grad; g.m = n->m; g.v = n->v;
    set_adam(n, lr, g);
    k_adam<<<(unsigned)((n->P + 255) / 256), 256, 0, (hipStream_t)stream>>>(g, n->P);
    MHIP(hipGetLastError());
    return CFR_OK;
}

cfr_status cfr_mlp_train_step(cfr_mlp *n, const void *x, const float *target, const float *weight,
                              const uint8_t *nact, const int32_t *idx, int64_t n_data, int64_t rows, float lr,
                              double *loss, void *stream) {
    // a rejected learning rate leaves the gradients and loss of the minibatch behind, as cfr_mlp_backward would
    const bool ok = lr >= 0.f;
    cfr_status st = gradients(n, x, target, weight, nact, idx, n_data, rows, ok, lr, (hipStream_t)stream);
    if (st == CFR_OK) st = read_loss(n, loss, (hipStream_t)stream);
    return st == CFR_OK && !ok ? mfail(CFR_EINVAL, "lr must be >= 0") : st;
}

void cfr_mlp_destroy(cfr_mlp *n) {
    if (!n) return;
    (void)hipSetDevice(n->d.device);
    (void)hipDeviceSynchronize();
    free_mlp(n);
}

}  // extern "C"

namespace cfrx {
cfr_status mlp_forward_internal(cfr_mlp *n, const void *x, int64_t rows, float *z, hipStream_t s) {
    return cfr_mlp_forward(n, x, rows, z, s);
}
int mlp_in_dim(const cfr_mlp *n) { return n->d.in_dim; }
int mlp_device(const cfr_mlp *n) { return n->d.device; }
}  // namespace cfrx
