// Learned self-distance surrogate: BF16 MFMA kernels for the forward pass,
// the backward pass and Adam, plus the exact-EDT fallback rule.
//
// A training step is six launches; at these sizes (4096 rows, 0.15 M weights,
// 3.6 GFLOP) it is bound by launches and by each one's loads (of k_mlp_forward,
// reading 290 KB of weights per work-group takes 5.7 us, the products 4.4), not by
// the matrix cores:
//   k_mlp_forward  the whole forward pass, a work-group per 16 rows   14.7 us
//   k_bwd_pre      loss partials and dY; W2, W3, W4 transposed         3.9
//   k_bwd_chain    the upstream gradients, 16 rows per work-group     13.4
//   k_dw           weight and bias gradients' partial sums            15.0
//   k_reduce_grad  the partial sums in chunk order, and the loss       4.2
//   k_adam                                                             3.1
// (batch 4096, each kernel alone in the profiler; a step in a stream takes 48 us,
// 143 with a launch per layer and product).
// All products are v_mfma_f32_16x16x32_bf16 over K in ascending steps of 32.
// Lane l of an MFMA holds A[l % 16][8 (l / 16) + i], B[8 (l / 16) + i][l % 16]
// and C[4 (l / 16) + i][l % 16], so an operand whose reduction index is
// contiguous in memory is one 16-byte load.  The gradient products reduce over
// the batch: the activations and upstream gradients they read are kept
// transposed ([feature][row]) by the kernels that make them, which hold four
// consecutive rows of a feature per lane.
#include <algorithm>

#include "common.h"
#include "sdf_mlp.h"

namespace edtmi {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int HID = SDF_MLP_HIDDEN;
constexpr int INP = SDF_MLP_IN_PAD;
constexpr int OUTP = SDF_MLP_OUT_PAD;
constexpr int ROW_ALIGN = 64;
constexpr int TRAIN_ROWS = 8192;   // the most rows that the backward pass takes

__host__ __device__ inline int padded_rows(int b) { return (b + ROW_ALIGN - 1) / ROW_ALIGN * ROW_ALIGN; }

// float -> bfloat16 bits, round to nearest even, one v_cvt_pk_bf16_f32: a NaN
// keeps its sign and the upper bits of its payload.  For values that stay on
// chip, where only being NaN matters (with f2bf there the inference takes 110
// instead of 85 us for 262,144 states).
__device__ __forceinline__ uint16_t cvt_bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// The same for values that go to memory: every NaN is stored as 0x7FC0.
__device__ __forceinline__ uint16_t f2bf(float f) { return f != f ? (uint16_t)0x7FC0u : cvt_bf(f); }

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Workspace layout (bytes) for padded batch P.
struct WsLayout {
    size_t x, h1, h2, h3, y;          // row-major: encoded input, hidden layers, output
    size_t dy;                        // bf16 dY, row-major
    size_t xt, h1t, h2t, h3t;         // the layers' inputs, [feature][row]
    size_t dyt, d1t, d2t, d3t;        // upstream gradients of the layers' outputs, [feature][row]
    size_t w2t, w3t, w4t;             // transposed weights, [input][output]
    size_t part;                      // loss partial sums
    size_t gpart;                     // gradient partial sums, dw_chunks parameter blocks
    size_t total;
};

// Batch chunks of the weight-gradient reduction, in MFMA steps of 32 rows: 16
// chunks of equal length, the last ones shorter or empty.
constexpr int DW_CHUNKS = 16;
__host__ __device__ inline int dw_steps(int P) { return (P / 32 + DW_CHUNKS - 1) / DW_CHUNKS; }
__host__ __device__ inline int dw_chunks(int P) { return (P / 32 + dw_steps(P) - 1) / dw_steps(P); }

__host__ __device__ inline WsLayout ws_layout(int P)
{
    WsLayout w;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t hid = (size_t)P * HID * 2, row_t = (size_t)P * 2;
    w.x = take((size_t)P * INP * 2);
    w.h1 = take(hid);
    w.h2 = take(hid);
    w.h3 = take(hid);
    w.y = take((size_t)P * OUTP * 4);
    if (P > TRAIN_ROWS) {
        // nothing of what only the backward pass reads, but no less than a
        // smaller batch on the same workspace needs
        w.dy = w.xt = w.h1t = w.h2t = w.h3t = w.dyt = w.d1t = w.d2t = w.d3t = w.w2t = w.w3t = w.w4t = w.part = w.gpart = o;
        const size_t train = ws_layout(TRAIN_ROWS).total;
        w.total = o > train ? o : train;
        return w;
    }
    w.dy = take((size_t)P * OUTP * 2);
    w.xt = take(INP * row_t);
    w.h1t = take(HID * row_t);
    w.h2t = take(HID * row_t);
    w.h3t = take(HID * row_t);
    w.dyt = take(OUTP * row_t);
    w.d1t = take(HID * row_t);
    w.d2t = take(HID * row_t);
    w.d3t = take(HID * row_t);
    w.w2t = take((size_t)HID * HID * 2);
    w.w3t = take((size_t)HID * HID * 2);
    w.w4t = take((size_t)HID * OUTP * 2);
    w.part = take(1024 * 4);
    w.gpart = take((size_t)dw_chunks(P) * SDF_MLP_PARAMS * 4);
    w.total = o;
    return w;
}

constexpr int TRAIN_MT = 1;         // 16-row tiles per work-group of the training passes (2: 17.3 against 15.0 us)
constexpr int ACT_LD = HID + 8;   // LDS row stride of activations (bf16): rows 4 banks apart

__device__ __forceinline__ bf16x8 load8(const uint16_t* p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

// The row blocks of a batch, contiguous per XCD (the dispatcher deals
// work-groups to the 8 XCDs round-robin): what one kernel writes for a stretch
// of rows is read by the next one through the same L2, and the four 32-byte
// pieces of a line of a transposed array are written through one.
__device__ __forceinline__ int xcd_block(int b, int blocks)
{
    const int per = (blocks + 7) / 8;
    return (b & 7) * per + (b >> 3);
}

// The B operand of one wave: columns n0 + 16 j + l % 16, j < NT, of a product
// over K = 32 KS, from [column][k] rows of ld elements.
template <int NT, int KS>
__device__ __forceinline__ void load_b(const uint16_t* w, int ld, int n0, bf16x8 (&b)[NT][KS])
{
    const int r = threadIdx.x & 15, kq = ((threadIdx.x & 63) >> 4) * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j][ks] = load8(w + (size_t)(n0 + 16 * j + r) * ld + ks * 32 + kq);
}

// 16 rows of A (LDS, row stride ACT_LD) times the wave's columns.
template <int NT, int KS>
__device__ __forceinline__ void product16(const uint16_t* A, const bf16x8 (&b)[NT][KS], f32x4 (&acc)[NT])
{
    const int r = threadIdx.x & 15, kq = ((threadIdx.x & 63) >> 4) * 8;
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = load8(A + r * ACT_LD + ks * 32 + kq);
#pragma unroll
        for (int j = 0; j < NT; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[j][ks], acc[j], 0, 0, 0);
    }
}

__device__ __forceinline__ uint2 pack4(const uint16_t (&v)[4])
{
    return make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
}

// 32 features of the work-group's rows (LDS, row stride ACT_LD) to [feature][P].
template <int MT>
__device__ __forceinline__ void transpose32(const uint16_t* a, uint16_t* out, int P, int row0)
{
    const int t = threadIdx.x;
    if (t >= 64 * MT) return;
    const int c = t / (2 * MT), h8 = (t % (2 * MT)) * 8;   // 8 rows of a feature each
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = (uint32_t)a[(h8 + 2 * k) * ACT_LD + c] | ((uint32_t)a[(h8 + 2 * k + 1) * ACT_LD + c] << 16);
    *reinterpret_cast<uint4*>(out + (size_t)c * P + row0 + h8) = make_uint4(v[0], v[1], v[2], v[3]);
}

// The forward pass of a training step: a 512-thread work-group per 16 rows
// (256 of them at batch 4096), the activations in LDS.  Wave w owns columns
// [32 w, 32 w + 32) of every hidden layer and loads its weights of all four
// layers at once (150 registers): they depend on nothing, so only the four
// products and their barriers are serial.  Every row's x, h1, h2, h3 (row-major
// and, for the backward pass, transposed) and y go to the workspace.  Batches
// beyond what the backward pass takes: 64 rows per work-group (MT = 4).  A state
// index outside [0, n_rows) gives its row NaN inputs; rows past the batch are zero
// inputs.
struct FwdOut {
    uint16_t *x, *h[3], *xt, *ht[3];
    float* y32;
    float* y;   // nullable, [batch][12]
};

template <int MT>
__global__ __launch_bounds__(512) void k_mlp_forward(const uint16_t* __restrict__ w16,
                                                     const float* __restrict__ master,
                                                     const float* __restrict__ q, int n_rows,
                                                     const int* __restrict__ idx, int batch, int P, FwdOut o)
{
    constexpr bool SAVE_T = MT == TRAIN_MT;   // the transposed copies are the backward pass's
    __shared__ __attribute__((aligned(16))) uint16_t act[2][16 * MT * ACT_LD];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int block = xcd_block(blockIdx.x, P / (16 * MT));
    if (block >= P / (16 * MT)) return;
    const int row0 = block * 16 * MT;
    const int n0 = wave * 32;
    const int r = lane & 15, m4 = 4 * (lane >> 4);
    // the thread's input angles before the weights: loads return in order
    const int em = t >> 5, ec = t & 31;
    float angle[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int b = row0 + 16 * i + em;
        angle[i] = 0.0f;
        if (b < batch && ec < 2 * SDF_MLP_JOINTS) {
            const int row = idx ? idx[b] : b;
            angle[i] = row >= 0 && row < n_rows ? q[(size_t)row * SDF_MLP_JOINTS + (ec >> 1)] : __builtin_nanf("");
        }
    }
    bf16x8 b1[2][1], b2[2][8], b3[2][8], b4[1][8];
    load_b(w16 + SDF_MLP_W1, INP, n0, b1);
    load_b(w16 + SDF_MLP_W2, HID, n0, b2);
    load_b(w16 + SDF_MLP_W3, HID, n0, b3);
    if (wave < OUTP / 16) load_b(w16 + SDF_MLP_W4, HID, 16 * wave, b4);
    float bias[3][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        bias[0][j] = master[SDF_MLP_B1 + n0 + 16 * j + r];
        bias[1][j] = master[SDF_MLP_B2 + n0 + 16 * j + r];
        bias[2][j] = master[SDF_MLP_B3 + n0 + 16 * j + r];
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {   // [sin q1, cos q1, ..., sin q7, cos q7, 0 ...]
        const int m = 16 * i + em;
        const bool real = row0 + m < batch && ec < 2 * SDF_MLP_JOINTS;
        const uint16_t e = f2bf(real ? ((ec & 1) ? cosf(angle[i]) : sinf(angle[i])) : 0.0f);
        act[0][m * ACT_LD + ec] = e;
        o.x[(size_t)(row0 + m) * INP + ec] = e;
    }
    __syncthreads();
    if constexpr (SAVE_T) transpose32<MT>(act[0], o.xt, P, row0);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const uint16_t* A = act[l & 1];
        uint16_t* O = act[(l & 1) ^ 1];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            f32x4 acc[2];
            if (l == 0) product16(A + 16 * i * ACT_LD, b1, acc);
            else if (l == 1) product16(A + 16 * i * ACT_LD, b2, acc);
            else product16(A + 16 * i * ACT_LD, b3, acc);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + 16 * j + r, m = 16 * i + m4;
                uint16_t v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = acc[j][e] + bias[l][j];
                    // ReLU that keeps a NaN (a poisoned row stays visible)
                    v[e] = f2bf((z > 0.0f || z != z) ? z : 0.0f);
                    O[(m + e) * ACT_LD + n] = v[e];
                }
                if constexpr (SAVE_T) *reinterpret_cast<uint2*>(o.ht[l] + (size_t)n * P + row0 + m) = pack4(v);
            }
        }
        __syncthreads();
        // the rows, 16 bytes per thread
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = 16 * i + (t >> 5), c8 = (t & 31) * 8;
            *reinterpret_cast<uint4*>(o.h[l] + (size_t)(row0 + m) * HID + c8) =
                *reinterpret_cast<const uint4*>(O + m * ACT_LD + c8);
        }
    }
    if (wave < OUTP / 16) {
        const int n = 16 * wave + r;
        const float bn = master[SDF_MLP_B4 + n];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            f32x4 acc[1];
            product16(act[1] + 16 * i * ACT_LD, b4, acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int b = row0 + 16 * i + m4 + e;
                const float z = acc[0][e] + bn;
                o.y32[(size_t)b * OUTP + n] = z;
                if (o.y && n < SDF_MLP_OUT && b < batch) o.y[(size_t)b * SDF_MLP_OUT + n] = z;
            }
        }
    }
}

// The upstream gradients of all layers: a 512-thread work-group per 16 rows;
// up_l-1 = bf16((up_l W_l) masked where layer l's input is positive), from dY
// down to layer 1's output.  The same plan as the forward pass: wave w owns 32
// columns and loads its (transposed) weights of all layers at once.
struct BwdChain {
    const uint16_t *dy, *w4t, *w3t, *w2t;
    const uint16_t* ht[3];   // h1, h2, h3 transposed
    uint16_t *dyt, *dt[3];   // dY and the gradients of h1, h2, h3, transposed
};

__global__ __launch_bounds__(512) void k_bwd_chain(BwdChain c, int P)
{
    constexpr int MT = TRAIN_MT, RB = 16 * MT;
    __shared__ __attribute__((aligned(16))) uint16_t up[2][RB * ACT_LD];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int block = xcd_block(blockIdx.x, P / RB);
    if (block >= P / RB) return;
    const int row0 = block * RB;
    const int n0 = wave * 32;
    const int r = lane & 15, m4 = 4 * (lane >> 4);
    uint4 dy = make_uint4(0, 0, 0, 0);   // RB x 32 of dY, before the weights: loads return in order
    if (t < 4 * RB) dy = *reinterpret_cast<const uint4*>(c.dy + (size_t)(row0 + (t >> 2)) * OUTP + (t & 3) * 8);
    bf16x8 b4[2][1], b3[2][8], b2[2][8];
    load_b(c.w4t, OUTP, n0, b4);
    load_b(c.w3t, HID, n0, b3);
    load_b(c.w2t, HID, n0, b2);
    uint2 mask[3][MT][2];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                mask[l][i][j] =
                    *reinterpret_cast<const uint2*>(c.ht[l] + (size_t)(n0 + 16 * j + r) * P + row0 + 16 * i + m4);
    if (t < 4 * RB) *reinterpret_cast<uint4*>(up[0] + (t >> 2) * ACT_LD + (t & 3) * 8) = dy;
    __syncthreads();
    transpose32<MT>(up[0], c.dyt, P, row0);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int l = 2 - s;   // the gradient of h_{l + 1}
        uint16_t* O = up[(s & 1) ^ 1];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            f32x4 acc[2];
            if (s == 0) product16(up[0] + 16 * i * ACT_LD, b4, acc);
            else if (s == 1) product16(up[1] + 16 * i * ACT_LD, b3, acc);
            else product16(up[0] + 16 * i * ACT_LD, b2, acc);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + 16 * j + r, m = 16 * i + m4;
                const uint32_t hm[2] = {mask[l][i][j].x, mask[l][i][j].y};
                uint16_t v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool on = bf2f((uint16_t)(hm[e >> 1] >> (16 * (e & 1)))) > 0.0f;
                    v[e] = f2bf(on ? acc[j][e] : 0.0f);
                    if (s < 2) O[(m + e) * ACT_LD + n] = v[e];
                }
                *reinterpret_cast<uint2*>(c.dt[l] + (size_t)n * P + row0 + m) = pack4(v);
            }
        }
        if (s < 2) __syncthreads();
    }
}

// Gradient partial sums of all four layers: dW_l[m][n] = sum_b up[b][m]
// act[b][n] and db_l[m] = sum_b up[b][m] over the rows b of a chunk,
// from the transposed operands, straight from the caches (no LDS, no barrier):
// a work-group is a 64 x 64 tile, a wave 32 x 32 of it, its loads of 4 steps in
// flight at once.  The bias is one more product, by a column of ones, in the
// waves of the first tile column.  Tiles: W3's 16, W2's 16, W4's 4, W1's 4.  Partial s is a whole parameter block at part + s * SDF_MLP_PARAMS.
struct DwArgs {
    const uint16_t *up[4], *act[4];   // [feature][P]
    float* part;
};
constexpr int DW_TILES = 16 + 16 + 4 + 4;

__global__ __launch_bounds__(256) void k_dw(DwArgs a, int P)
{
    // the tiles of a chunk on the XCD that wrote its rows
    const int KS = dw_chunks(P), per_xcd = (KS + 7) / 8;
    const int j = (int)blockIdx.x >> 3, x = j % DW_TILES, s = (blockIdx.x & 7) * per_xcd + j / DW_TILES;
    if (s >= KS) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int l, M, N, m0, n0, wo, bo;
    if (x < 32) {
        l = x < 16 ? 2 : 1;
        M = N = HID;
        m0 = ((x & 15) >> 2) * 64;
        n0 = (x & 3) * 64;
        wo = l == 2 ? SDF_MLP_W3 : SDF_MLP_W2;
        bo = l == 2 ? SDF_MLP_B3 : SDF_MLP_B2;
    } else if (x < 36) {
        l = 3;
        M = OUTP;
        N = HID;
        m0 = 0;
        n0 = (x - 32) * 64;
        wo = SDF_MLP_W4;
        bo = SDF_MLP_B4;
    } else {
        l = 0;
        M = HID;
        N = INP;
        m0 = (x - 36) * 64;
        n0 = 0;
        wo = SDF_MLP_W1;
        bo = SDF_MLP_B1;
    }
    m0 += (wave >> 1) * 32;
    n0 += (wave & 1) * 32;
    if (m0 >= M || n0 >= N) return;   // M and N are multiples of 32
    const int per = dw_steps(P), k0 = s * per, k1 = min(P / 32, k0 + per);
    const int r = lane & 15, kq = (lane >> 4) * 8;
    const uint16_t* up = a.up[l] + (size_t)(m0 + r) * P + kq;
    const uint16_t* act = a.act[l] + (size_t)(n0 + r) * P + kq;
    f32x4 acc[2][2], accb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        accb[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    bf16x8 one;
#pragma unroll
    for (int e = 0; e < 8; ++e) one[e] = (__bf16)1.0f;
    const bool bias = n0 == 0;
    for (int kb = k0; kb < k1; kb += 4) {
        bf16x8 va[4][2], vb[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t k = 32 * (size_t)min(kb + u, k1 - 1);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                va[u][i] = load8(up + (size_t)(16 * i) * P + k);
                vb[u][i] = load8(act + (size_t)(16 * i) * P + k);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (kb + u >= k1) break;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[u][i], vb[u][j], acc[i][j], 0, 0, 0);
                if (bias) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[u][i], one, accb[i], 0, 0, 0);
            }
        }
    }
    float* out = a.part + (size_t)s * SDF_MLP_PARAMS;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + 16 * i + 4 * (lane >> 4) + e;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) out[wo + m * N + n0 + 16 * jj + r] = acc[i][jj][e];
            if (bias && r == 0) out[bo + m] = accb[i][e];
        }
}

// The whole forward pass for inference.  A 512-thread work-group keeps the
// weights of all four layers in registers (wave w: columns [32 w, 32 w + 32) of
// a hidden layer) and walks over tiles of 16 MTI rows, the activations in LDS:
// the weights (290 KB from the L2 per work-group) are read once instead of
// once per 64 rows.  Products run as weights x activations, so that a lane
// ends with four consecutive features of one row and writes them as 8 bytes.
// While two waves finish a tile (12 outputs), the others encode the next one.
// Every product is the same sequence of v_mfma_f32_16x16x32_bf16 over K in
// steps of 32 as in k_mlp_forward, with the same epilogues, so y is
// bit-identical to sdf_mlp_forward's.  With need given, the work-group also
// applies k_fallback's rule to its rows.  131,072 states: 104 us with the
// weights read per tile and 2-byte LDS writes, 54 us like this (bound by the LDS
// reads of the activations and the matrix cores, 2,048 cycles each per layer
// and 64 rows).
template <int MTI>
__global__ __launch_bounds__(512) void k_mlp_infer(const uint16_t* __restrict__ w16,
                                                   const float* __restrict__ master,
                                                   const float* __restrict__ q, int batch,
                                                   float* __restrict__ y, const float* __restrict__ radii,
                                                   const float* __restrict__ eps, float voxel, float margin,
                                                   int* __restrict__ need)
{
    constexpr int ROWS = 16 * MTI;
    __shared__ __attribute__((aligned(16))) uint16_t act[2][ROWS * ACT_LD];
    __shared__ float yout[ROWS * SDF_MLP_OUT];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n0 = wave * 32;
    const int r = lane & 15, g4 = 4 * (lane >> 4), kq = 8 * (lane >> 4);
    const int tiles = (batch + ROWS - 1) / ROWS;
    // [sin q1, cos q1, ..., sin q7, cos q7, 0 ...] as bf16 (k_mlp_forward's
    // values): item (row, j) is joint j's pair, j = 7 the zeros; rows past the
    // batch are zeros
    auto encode = [&](int tile, int first, int threads) {
        for (int i = first; i < ROWS * 8; i += threads) {
            const int m = i >> 3, j = i & 7, b = tile * ROWS + m;
            uint32_t* o = reinterpret_cast<uint32_t*>(act[0] + m * ACT_LD);
            if (j < SDF_MLP_JOINTS) {
                uint32_t v = 0;
                if (b < batch) {
                    const float a = q[(size_t)b * SDF_MLP_JOINTS + j];
                    v = (uint32_t)cvt_bf(sinf(a)) | ((uint32_t)cvt_bf(cosf(a)) << 16);
                }
                o[j] = v;
            } else {
#pragma unroll
                for (int k = SDF_MLP_JOINTS; k < INP / 2; ++k) o[k] = 0u;
            }
        }
    };
    bf16x8 b1[2][1], b2[2][8], b3[2][8], b4[1][8];
    load_b(w16 + SDF_MLP_W1, INP, n0, b1);
    load_b(w16 + SDF_MLP_W2, HID, n0, b2);
    load_b(w16 + SDF_MLP_W3, HID, n0, b3);
    if (wave < OUTP / 16) load_b(w16 + SDF_MLP_W4, HID, 16 * wave, b4);
    encode(blockIdx.x, t, 512);
    __syncthreads();
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int row0 = tile * ROWS;
        const int rows = min(ROWS, batch - row0);
        const int mt = (rows + 15) >> 4;   // 16-row tiles that hold states
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            const uint16_t* A = act[l & 1];
            uint16_t* O = act[(l & 1) ^ 1];
            const float* bias = master + (l == 0 ? SDF_MLP_B1 : l == 1 ? SDF_MLP_B2 : SDF_MLP_B3) + n0 + g4;
            float bv[2][4];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) bv[j][e] = bias[16 * j + e];
            constexpr int KS_MAX = HID / 32;
            const int ksn = l == 0 ? 1 : KS_MAX;
#pragma unroll
            for (int i = 0; i < MTI; ++i) {
                if (i >= mt) break;
                f32x4 acc[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                for (int ks = 0; ks < KS_MAX; ++ks) {
                    if (ks >= ksn) break;
                    const bf16x8 a = load8(A + (16 * i + r) * ACT_LD + ks * 32 + kq);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            l == 0 ? b1[j][0] : l == 1 ? b2[j][ks] : b3[j][ks], a, acc[j], 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    uint16_t v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float z = acc[j][e] + bv[j][e];
                        v[e] = cvt_bf((z > 0.0f || z != z) ? z : 0.0f);
                    }
                    *reinterpret_cast<uint2*>(O + (16 * i + r) * ACT_LD + n0 + 16 * j + g4) = pack4(v);
                }
            }
            __syncthreads();
        }
        const int next = tile + (int)gridDim.x;
        if (wave < OUTP / 16) {
            const int n = 16 * wave + g4;
            float bv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[e] = master[SDF_MLP_B4 + n + e];
#pragma unroll
            for (int i = 0; i < MTI; ++i) {
                if (i >= mt) break;
                f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < HID / 32; ++ks)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        b4[0][ks], load8(act[1] + (16 * i + r) * ACT_LD + ks * 32 + kq), acc, 0, 0, 0);
                const int m = 16 * i + r;
                if (n < SDF_MLP_OUT && m < rows) {   // SDF_MLP_OUT is a multiple of 4
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float z = acc[e] + bv[e];
                        y[(size_t)(row0 + m) * SDF_MLP_OUT + n + e] = z;
                        yout[m * SDF_MLP_OUT + n + e] = z;
                    }
                }
            }
        } else if (next < tiles) {
            encode(next, t - 64 * (OUTP / 16), 512 - 64 * (OUTP / 16));
        }
        __syncthreads();
        // yout is next written three barriers from here
        if (need && t < rows) {
            int flag = 0;
            for (int i = 0; i < SDF_MLP_OUT; ++i) {
                const float c = yout[t * SDF_MLP_OUT + i] * voxel - radii[i];
                const float thresh = margin + eps[i] * voxel;
                if (!(c >= thresh)) flag = 1;   // NaN predictions also fall back
            }
            need[row0 + t] = flag;
        }
    }
}

// The backward pass's preparation.  Work-groups below nloss: dY = bf16(2 (y -
// t) / (batch * 12)) on valid entries, 0 elsewhere, with t = min(target[idx[b]],
// clip) (clip <= 0: no clipping; NaN for an index outside [0, n_rows)), and
// partial sums of (y - t)^2 in a fixed order.  The others: W3, W2 (16 tiles of
// 64 x 64 each) and W4 (4 tiles of 32 x 64) transposed.
struct BwdPre {
    const uint16_t* w16;
    uint16_t *w2t, *w3t, *w4t;
};
constexpr int PRE_TILES = 16 + 16 + 4;

__global__ __launch_bounds__(256) void k_bwd_pre(BwdPre w, int nloss, const float* __restrict__ y32,
                                                 const float* __restrict__ target, int n_rows,
                                                 const int* __restrict__ idx, float clip, int batch, int P,
                                                 uint16_t* __restrict__ dy, float* __restrict__ part)
{
    __shared__ float red[256];
    __shared__ __attribute__((aligned(16))) uint16_t tile[64][72];
    if ((int)blockIdx.x >= nloss) {
        const int x = (int)blockIdx.x - nloss, t = threadIdx.x;
        const uint16_t* src = w.w16 + (x < 16 ? SDF_MLP_W3 : (x < 32 ? SDF_MLP_W2 : SDF_MLP_W4));
        uint16_t* dst = x < 16 ? w.w3t : (x < 32 ? w.w2t : w.w4t);
        const int rows = x < 32 ? 64 : 32, out = x < 32 ? HID : OUTP;
        const int m0 = x < 32 ? ((x & 15) >> 2) * 64 : 0, n0 = (x & 3) * 64;
        for (int i = t; i < rows * 8; i += 256)
            *reinterpret_cast<uint4*>(&tile[i >> 3][(i & 7) * 8]) =
                *reinterpret_cast<const uint4*>(src + (size_t)(m0 + (i >> 3)) * HID + n0 + (i & 7) * 8);
        __syncthreads();
        const int per = rows / 8;   // 16-byte pieces of an output row
        for (int i = t; i < 64 * per; i += 256) {
            const int n = i / per, k8 = (i % per) * 8;
            uint32_t v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = (uint32_t)tile[k8 + 2 * k][n] | ((uint32_t)tile[k8 + 2 * k + 1][n] << 16);
            *reinterpret_cast<uint4*>(dst + (size_t)(n0 + n) * out + m0 + k8) = make_uint4(v[0], v[1], v[2], v[3]);
        }
        return;
    }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const float scale = 2.0f / (float)(batch * SDF_MLP_OUT);
    float sq = 0.0f;
    if (i < P * OUTP) {
        const int b = i / OUTP, c = i % OUTP;
        float g = 0.0f;
        if (b < batch && c < SDF_MLP_OUT) {
            const int row = idx ? idx[b] : b;
            float t = __builtin_nanf("");   // an index outside target poisons its row
            if (row >= 0 && row < n_rows) t = target[(size_t)row * SDF_MLP_OUT + c];
            if (clip > 0.0f && t > clip) t = clip;
            const float d = y32[i] - t;
            sq = d * d;
            g = d * scale;
        }
        dy[i] = f2bf(g);
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// grad = sum over chunks s = 0 .. KS - 1 of the partial blocks, in that order
// (four parameters per thread); the last work-group adds up the loss.
static_assert(SDF_MLP_PARAMS % 4 == 0, "parameter blocks are read as float4");
constexpr int REDUCE_BLOCKS = (SDF_MLP_PARAMS / 4 + 255) / 256;

__global__ __launch_bounds__(256) void k_reduce_grad(const float* __restrict__ gpart, int KS,
                                                     float* __restrict__ grad, const float* __restrict__ part,
                                                     int nparts, int batch, float* __restrict__ loss)
{
    __shared__ float red[256];
    if (blockIdx.x < REDUCE_BLOCKS) {
        const int i = blockIdx.x * 256 + threadIdx.x;
        if (i >= SDF_MLP_PARAMS / 4) return;
        float4 v[DW_CHUNKS];
#pragma unroll
        for (int s = 0; s < DW_CHUNKS; ++s)
            v[s] = reinterpret_cast<const float4*>(gpart + (size_t)min(s, KS - 1) * SDF_MLP_PARAMS)[i];
        float g[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < DW_CHUNKS; ++s) {
            if (s < KS) {
                g[0] += v[s].x;
                g[1] += v[s].y;
                g[2] += v[s].z;
                g[3] += v[s].w;
            }
        }
        // the caller's grad need not be 16-byte aligned
#pragma unroll
        for (int k = 0; k < 4; ++k) grad[4 * i + k] = g[k];
        return;
    }
    float s = 0.0f;
    for (int i = threadIdx.x; i < nparts; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] / (float)(batch * SDF_MLP_OUT);
}

__global__ void k_pack(const float* __restrict__ master, uint16_t* __restrict__ w16, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w16[i] = f2bf(master[i]);
}

__global__ void k_adam(float* __restrict__ w, uint16_t* __restrict__ w16, float* __restrict__ m,
                       float* __restrict__ v, const float* __restrict__ g, int n, float lr, float b1,
                       float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    w16[i] = f2bf(wi);
}

__global__ __launch_bounds__(256) void k_fallback(const float* __restrict__ y,
                                                  const float* __restrict__ radii,
                                                  const float* __restrict__ eps, int batch,
                                                  float voxel, float margin, int* __restrict__ need,
                                                  int* __restrict__ count)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    int flag = 0;
    if (b < batch) {
        for (int i = 0; i < SDF_MLP_OUT; ++i) {
            const float c = y[b * SDF_MLP_OUT + i] * voxel - radii[i];
            const float thresh = margin + eps[i] * voxel;
            if (!(c >= thresh)) flag = 1;   // NaN predictions also fall back
        }
        need[b] = flag;
    }
    const unsigned long long bal = __ballot(flag);
    if ((threadIdx.x & 63) == 0 && bal) atomicAdd(count, (int)__popcll(bal));
}

// out[b][i] = need[b] ? exact[b * erow + i * ecol] : y[b][i]
__global__ void k_select(const float* __restrict__ y, const int* __restrict__ need,
                         const float* __restrict__ exact, int erow, int ecol, int batch,
                         float* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= batch * SDF_MLP_OUT) return;
    const int b = k / SDF_MLP_OUT, i = k % SDF_MLP_OUT;
    out[k] = need[b] ? exact[(size_t)b * erow + (size_t)i * ecol] : y[k];
}

__global__ void k_zero_int(int* p) { *p = 0; }

__global__ void k_zero_f32(float* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// eps[i] = max(0, max over rows b with target[b][i] < clip of
// pred[b][i] - target[b][i]) (clip <= 0: every row); a NaN prediction
// gives +inf.  Non-negative floats order like their bit patterns, so the
// maximum is an integer atomicMax on the bits and independent of order.
__global__ __launch_bounds__(256) void k_calibrate(const float* __restrict__ pred,
                                                   const float* __restrict__ target, int batch,
                                                   float clip, unsigned* __restrict__ eps)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= batch * SDF_MLP_OUT) return;
    const float t = target[i], p = pred[i];
    if (clip > 0.0f && !(t < clip)) return;
    float d = p - t;
    if (p != p) d = __builtin_huge_valf();
    if (d > 0.0f) atomicMax(eps + i % SDF_MLP_OUT, __float_as_uint(d));
}

}  // namespace

}  // namespace edtmi

using namespace edtmi;

extern "C" {

size_t sdf_mlp_workspace_bytes(int32_t batch)
{
    if (batch < 1) return 0;
    return ws_layout(padded_rows(batch)).total;
}

int sdf_mlp_pack(const float* master, uint16_t* w16, void* stream)
{
    if (!master || !w16) {
        set_error("sdf_mlp_pack: NULL pointer");
        return EDT_ERR_ARG;
    }
    hipLaunchKernelGGL(k_pack, dim3((SDF_MLP_PARAMS + 255) / 256), dim3(256), 0, as_stream(stream),
                       master, w16, (int)SDF_MLP_PARAMS);
    return check_launch("k_pack");
}

int sdf_mlp_forward(const uint16_t* w16, const float* master, const float* q, int32_t n_rows,
                    const int32_t* idx, int32_t batch, float* y, void* ws, size_t ws_bytes,
                    void* stream)
{
    if (!w16 || !master || !q || !ws || batch < 1 || n_rows < 1 || (!idx && n_rows < batch)) {
        set_error("sdf_mlp_forward: NULL pointer, batch < 1, or fewer rows than the batch");
        return EDT_ERR_ARG;
    }
    const int P = padded_rows(batch);
    const WsLayout L = ws_layout(P);
    if (ws_bytes < L.total) {
        set_error("sdf_mlp_forward: workspace %zu < %zu bytes", ws_bytes, L.total);
        return EDT_ERR_WORKSPACE;
    }
    char* w = static_cast<char*>(ws);
    auto u16 = [&](size_t at) { return reinterpret_cast<uint16_t*>(w + at); };
    FwdOut o{};
    o.x = u16(L.x);
    o.xt = u16(L.xt);
    const size_t h[3] = {L.h1, L.h2, L.h3}, ht[3] = {L.h1t, L.h2t, L.h3t};
    for (int l = 0; l < 3; ++l) {
        o.h[l] = u16(h[l]);
        o.ht[l] = u16(ht[l]);
    }
    o.y32 = reinterpret_cast<float*>(w + L.y);
    o.y = y;
    auto go = [&](auto kernel, int rows) {
        hipLaunchKernelGGL(kernel, dim3((P / rows + 7) / 8 * 8), dim3(512), 0, as_stream(stream), w16, master, q,
                           (int)n_rows, idx, (int)batch, P, o);
    };
    // more rows than a backward pass takes: 64 per work-group, or the weights are
    // read from the L2 for every 16, and without the transposed copies (12,288 rows 34
    // us, 65,536 164; 19 and 67 like this)
    if (P > TRAIN_ROWS) go(k_mlp_forward<4>, 16 * 4);
    else go(k_mlp_forward<TRAIN_MT>, 16 * TRAIN_MT);
    return check_launch("k_mlp_forward");
}

int sdf_mlp_backward(const uint16_t* w16, const float* target, int32_t n_rows, const int32_t* idx,
                     int32_t batch, float clip_vox, float* grad, float* loss, void* ws, size_t ws_bytes,
                     void* stream)
{
    if (!w16 || !target || !grad || !ws || batch < 1 || n_rows < 1 || (!idx && n_rows < batch)) {
        set_error("sdf_mlp_backward: NULL pointer, batch < 1, or fewer rows than the batch");
        return EDT_ERR_ARG;
    }
    const int P = padded_rows(batch);
    const WsLayout L = ws_layout(P);
    if (ws_bytes < L.total) {
        set_error("sdf_mlp_backward: workspace %zu < %zu bytes", ws_bytes, L.total);
        return EDT_ERR_WORKSPACE;
    }
    char* w = static_cast<char*>(ws);
    auto u16 = [&](size_t at) { return reinterpret_cast<uint16_t*>(w + at); };
    const float* y32 = reinterpret_cast<const float*>(w + L.y);
    float* part = reinterpret_cast<float*>(w + L.part);
    float* gpart = reinterpret_cast<float*>(w + L.gpart);
    const int KS = dw_chunks(P);
    const hipStream_t st = as_stream(stream);
    const int nblk = (P * OUTP + 255) / 256;
    static_assert(TRAIN_ROWS * OUTP / 256 == 1024, "one loss partial sum per work-group");
    if (P > TRAIN_ROWS) {
        set_error("sdf_mlp_backward: batch too large for the loss reduction");
        return EDT_ERR_UNSUPPORTED;
    }
    const BwdPre pre{w16, u16(L.w2t), u16(L.w3t), u16(L.w4t)};
    hipLaunchKernelGGL(k_bwd_pre, dim3(nblk + PRE_TILES), dim3(256), 0, st, pre, nblk, y32, target, (int)n_rows,
                       idx, clip_vox, (int)batch, P, u16(L.dy), part);
    int rc = check_launch("k_bwd_pre");
    if (rc) return rc;
    const BwdChain c{u16(L.dy), u16(L.w4t), u16(L.w3t), u16(L.w2t), {u16(L.h1t), u16(L.h2t), u16(L.h3t)},
                     u16(L.dyt), {u16(L.d1t), u16(L.d2t), u16(L.d3t)}};
    hipLaunchKernelGGL(k_bwd_chain, dim3((P / (16 * TRAIN_MT) + 7) / 8 * 8), dim3(512), 0, st, c, P);
    if ((rc = check_launch("k_bwd_chain"))) return rc;
    const DwArgs d{{u16(L.d1t), u16(L.d2t), u16(L.d3t), u16(L.dyt)},
                   {u16(L.xt), u16(L.h1t), u16(L.h2t), u16(L.h3t)}, gpart};
    hipLaunchKernelGGL(k_dw, dim3(8 * DW_TILES * ((KS + 7) / 8)), dim3(256), 0, st, d, P);
    if ((rc = check_launch("k_dw"))) return rc;
    hipLaunchKernelGGL(k_reduce_grad, dim3(REDUCE_BLOCKS + (loss ? 1 : 0)), dim3(256), 0, st, gpart, KS, grad, part,
                       nblk, (int)batch, loss);
    return check_launch("k_reduce_grad");
}

int sdf_mlp_adam(float* master, uint16_t* w16, float* m, float* v, const float* grad, int32_t step,
                 float lr, float beta1, float beta2, float eps, void* stream)
{
    if (!master || !w16 || !m || !v || !grad || step < 1) {
        set_error("sdf_mlp_adam: NULL pointer or step < 1");
        return EDT_ERR_ARG;
    }
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    hipLaunchKernelGGL(k_adam, dim3((SDF_MLP_PARAMS + 255) / 256), dim3(256), 0, as_stream(stream),
                       master, w16, m, v, grad, (int)SDF_MLP_PARAMS, lr, beta1, beta2, eps, c1, c2);
    return check_launch("k_adam");
}

int sdf_mlp_fallback(const float* y, const float* radii, const float* eps_vox, int32_t batch,
                     float voxel, float margin, int32_t* need, int32_t* count, void* stream)
{
    if (!y || !radii || !eps_vox || !need || !count || batch < 1 || !(voxel > 0.0f)) {
        set_error("sdf_mlp_fallback: bad argument");
        return EDT_ERR_ARG;
    }
    const hipStream_t st = as_stream(stream);
    hipLaunchKernelGGL(k_zero_int, dim3(1), dim3(1), 0, st, count);
    int rc = check_launch("k_zero_int");
    if (rc) return rc;
    hipLaunchKernelGGL(k_fallback, dim3((batch + 255) / 256), dim3(256), 0, st, y, radii, eps_vox,
                       (int)batch, voxel, margin, need, count);
    return check_launch("k_fallback");
}

int sdf_mlp_infer(const uint16_t* w16, const float* master, const float* q, int32_t batch, float* y,
                  const float* radii, const float* eps_vox, float voxel, float margin, int32_t* need,
                  void* stream)
{
    if (!w16 || !master || !q || !y || batch < 1) {
        set_error("sdf_mlp_infer: NULL pointer or batch < 1");
        return EDT_ERR_ARG;
    }
    if (need && (!radii || !eps_vox || !(voxel > 0.0f))) {
        set_error("sdf_mlp_infer: the fallback rule needs radii, eps_vox and a voxel size > 0");
        return EDT_ERR_ARG;
    }
    // one work-group per CU at most; tiles of 16 rows while that gives every
    // one at most two, else 64
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
        n_cu = 256;
    const bool small = batch <= 2 * 16 * n_cu;
    const int rows = small ? 16 : 64;
    const dim3 grid(std::min((batch + rows - 1) / rows, n_cu));
    if (small)
        hipLaunchKernelGGL(k_mlp_infer<1>, grid, dim3(512), 0, as_stream(stream), w16, master, q, (int)batch, y,
                           radii, eps_vox, voxel, margin, need);
    else
        hipLaunchKernelGGL(k_mlp_infer<4>, grid, dim3(512), 0, as_stream(stream), w16, master, q, (int)batch, y,
                           radii, eps_vox, voxel, margin, need);
    return check_launch("k_mlp_infer");
}

int sdf_mlp_select(const float* y, const int32_t* need, const float* exact, int32_t exact_row,
                   int32_t exact_col, int32_t batch, float* out, void* stream)
{
    if (!y || !need || !exact || !out || batch < 1 || exact_row < 0 || exact_col < 0) {
        set_error("sdf_mlp_select: NULL pointer, batch < 1 or negative stride");
        return EDT_ERR_ARG;
    }
    const int n = batch * SDF_MLP_OUT;
    hipLaunchKernelGGL(k_select, dim3((n + 255) / 256), dim3(256), 0, as_stream(stream), y, need, exact,
                       (int)exact_row, (int)exact_col, (int)batch, out);
    return check_launch("k_select");
}

int sdf_mlp_calibrate(const float* pred, const float* target, int32_t batch, float clip_vox,
                      float* eps_vox, void* stream)
{
    if (!pred || !target || !eps_vox || batch < 1) {
        set_error("sdf_mlp_calibrate: NULL pointer or batch < 1");
        return EDT_ERR_ARG;
    }
    const hipStream_t st = as_stream(stream);
    hipLaunchKernelGGL(k_zero_f32, dim3(1), dim3(64), 0, st, eps_vox, (int)SDF_MLP_OUT);
    int rc = check_launch("k_zero_f32");
    if (rc) return rc;
    const int n = batch * SDF_MLP_OUT;
    hipLaunchKernelGGL(k_calibrate, dim3((n + 255) / 256), dim3(256), 0, st, pred, target, (int)batch,
                       clip_vox, reinterpret_cast<unsigned*>(eps_vox));
    return check_launch("k_calibrate");
}

}  // extern "C"
