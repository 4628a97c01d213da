// MLP surrogate of the radiation force: BF16 MFMA forward and backward
// kernels, Adam, and the C ABI of include/lb_mlp.h.
//
// Matrix products use v_mfma_f32_16x16x32_bf16: per 64-lane wavefront,
// A (16 x 32) has lane l holding row l % 16, k = 8 (l / 16) .. + 7;
// B (32 x 16) has lane l holding column l % 16, the same k range;
// D (16 x 16) has lane l holding column l % 16, rows 4 (l / 16) .. + 3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../include/lb_mlp.h"
#include "../../include/lb_wave.h"

int lbw_fail_msg(int code, const char *msg);  // lb_wave.hip

namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kLayers = 5;
constexpr int kIn = 4;
constexpr int kDims[kLayers + 1] = {kIn, 256, 256, 256, 256, 1};
constexpr int kHidden = 256;

constexpr int param_offset_w(int l)
{
    int off = 0;
    for (int i = 0; i < l; ++i) off += kDims[i + 1] * kDims[i] + kDims[i + 1];
    return off;
}
constexpr int param_offset_b(int l) { return param_offset_w(l) + kDims[l + 1] * kDims[l]; }
constexpr int kParams = param_offset_w(kLayers);

__device__ inline float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
// FP32 -> BF16, round to nearest even (one hardware conversion on gfx950)
__device__ inline uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// two at once: a in the low half, b in the high half.  The pair is converted as
// one vector and split by the caller with shifts: reading a single element of a
// BF16 vector is lowered wrongly by this compiler (element 1 reads element 0).
__device__ inline uint32_t to_bf16x2(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

// Standard normal distribution in the tail, h = Phi(-|z|) = (1 - erf(|z| / sqrt 2)) / 2,
// from Hastings' rational-exponential form of erf (Abramowitz & Stegun 7.1.26,
// |error| <= 1.5e-7): for x >= 0, 1 - erf(x) ~ t (a1 + t (a2 + t (a3 + t (a4 + t a5))))
// exp(-x^2), t = 1 / (1 + p x).  Here x = |z| / sqrt 2, with 1/sqrt 2 folded into p and
// the factor 1/2 into the a_i.  In FP32 h is within 3e-7 of Phi(-|z|); e = exp(-z^2 / 2)
// is returned for the derivative.  About a dozen instructions against some 35 for the
// library erf, which evaluates both of its branches.
__device__ inline float normal_tail(float z, float &e)
{
    const float t = __builtin_amdgcn_rcpf(fmaf(0.23164188826636f, fabsf(z), 1.0f));
    float q = fmaf(t, 0.5307027145f, -0.7265760135f);
    q = fmaf(t, q, 0.7107068705f);
    q = fmaf(t, q, -0.142248368f);
    q = fmaf(t, q, 0.127414796f);
    e = __builtin_amdgcn_exp2f(z * (z * -0.72134752044448f));  // exp(-z^2 / 2)
    return (q * t) * e;
}

// max(z, 0) as one instruction (the compiler's fmaxf first quiets a possible
// signalling NaN with a second one; a NaN z still gives a NaN GELU below)
__device__ inline float relu(float z)
{
    float r;
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(z));
    return r;
}

// exact GELU g(z) = z Phi(z) = max(z, 0) - |z| Phi(-|z|), and its derivative
// g'(z) = Phi(z) + z phi(z)
__device__ inline float gelu(float z)
{
    float e;
    return fmaf(-fabsf(z), normal_tail(z, e), relu(z));
}
__device__ inline float gelu_d(float z)
{
    float e;
    const float h = normal_tail(z, e);
    return fmaf(z * 0.39894228040143268f, e, z >= 0.0f ? 1.0f - h : h);
}

// The BF16 mirrors of the 256 x 256 weights are kept in the order in which a wavefront loads them:
// the fragment of column tile n / 16 and K step k / 32 is 1 KiB, lane (n % 16) + 16 (k % 32 / 8)
// holding 8 consecutive k.  Row by row, a fragment load touched 64 bytes of each of 16 rows: the
// sweep below took 40 us for 4800 samples, now 27; infer_kernel 0.82 ms for 2^20, now 0.72.
__host__ __device__ constexpr int frag_index(int n, int k)
{
    return ((k / 32 * (kHidden / 16) + n / 16) * 64 + n % 16 + 16 * (k % 32 / 8)) * 8 + k % 8;
}
__device__ inline s16x8 weight_frag(const uint16_t *W, int step, int tile, int lane)
{
    return *reinterpret_cast<const s16x8 *>(W + ((step * (kHidden / 16) + tile) * 64 + lane) * 8);
}

// Operands of the weight gradients, rows (neurons or inputs) x samples, in the same order: fragment
// of rows 16 tile .. and samples 32 step .., `tiles` tiles of rows per step
__host__ __device__ constexpr int row_tiles(int rows) { return (rows + 15) / 16; }
__device__ inline int64_t sample_frag(int step, int tiles, int tile, int lane)
{
    return (((int64_t)step * tiles + tile) * 64 + lane) * 8;
}
__device__ inline int64_t sample_index(int m, int tiles, int r)
{
    return sample_frag(m / 32, tiles, r / 16, r % 16 + 16 * (m % 32 / 8)) + m % 8;
}

// ---------------------------------------------------------------------------
// Training.  One Adam step is three launches:
//   sweep_kernel   forward through all layers and back down to the error of
//                  every hidden layer, for 32 samples per block;
//   wgrad_kernel   the weight gradients dW_l = delta_l^T a_l of all layers;
//   finish_kernel  the sums of their parts, and Adam.
// Rows (samples) never mix before the weight gradients, so a block carries its
// samples through the whole network: activations and errors pass from layer to
// layer in LDS (BF16) and the pre-activations stay in registers (FP32), and
// only what the weight gradients read goes to memory: the activations and
// errors in the order of the MFMA fragments of those products (zero past the
// batch up to a multiple of 64 samples).  The weight gradients have K = batch: K is split into at most
// kMaxSplit chunks, each chunk's sum goes to its own slot, and finish_kernel
// adds the slots in chunk order (deterministic).  Bias gradients (column sums
// of the FP32 errors) and the loss are summed per 32 samples in the sweep and
// finished the same way.
// ---------------------------------------------------------------------------

constexpr int kTile = 64;      // weight gradients: 64 x 64 outputs per workgroup, 4 wavefronts of
                               // 32 x 32; the batch is padded to a multiple of it
constexpr int kStepsAhead = 5; // K steps of 32 whose fragments are loaded before use: 16 VGPRs a
                               // step, so that four blocks share a CU
constexpr int kMaxSplit = 16;  // K chunks of a weight-gradient product
constexpr int kMaxTrainBatch = 1 << 24;  // training batch limit (workspace about 8 KB per sample)

constexpr int kSweepRows = 32;
constexpr int kSweepWaves = 8;
constexpr int kActLd = kHidden + 8;  // LDS row of BF16 activations: 16-byte reads of 16 consecutive
                                     // rows spread over the banks

struct SweepArgs {
    const float *x;         // B x 4
    const float *target;    // B targets (kTrain)
    int B;
    float inv_b2;           // 2 / B
    const float *p;         // parameters
    const uint16_t *pb, *pbT;  // BF16 mirrors W and W^T
    uint16_t *act[kLayers];    // inputs of every layer (sample_index order), training only
    uint16_t *err[kLayers];    // errors of every layer, likewise
    float *bpart[kLayers];  // per 32 samples: column sums of the errors [block][N_l]
    double *lpart;          // per 32 samples: sum of squared errors
    float *y;               // B
};

// first parameter of hidden layer l (1 .. kLayers - 2)
__device__ inline int hidden_offset(int l)
{
    return param_offset_w(1) + (l - 1) * (param_offset_w(2) - param_offset_w(1));
}

// One hidden layer's weight fragments of this wavefront's 32 columns, 8 K steps x 2 column tiles,
// and where its sums start
struct LayerFrags {
    s16x8 b[8][2];
    float start[2];
    __device__ inline void load(const uint16_t *W, const float *bias, int w, int lane)
    {
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j) b[s][j] = weight_frag(W, s, 2 * w + j, lane);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            start[j] = bias ? bias[w * 32 + 16 * j + (lane & 15)] : 0.f;
    }
};

// What bounds the sweep: latency.  A block's layers follow one another, each a
// few hundred cycles of MFMA and GELU behind two barriers and the L2 latency of
// its weights (all of a layer's fragments are in flight together, loaded while
// the layer before is finished).  The layers are loops, not unrolled, and the
// pre-activations wait in LDS rather than in registers for that: 4800
// samples: 27 us (41 before the weights were loaded in fragment order).  32
// samples per block (RT = 2 row tiles) fill 150 CUs at that batch; the column
// sums below are those of 32 samples, so fewer would change the order of the
// sums.  One launch replaces nine (five products forward, four back, 7-16 us
// each).  The other modes are the forward pass of small batches, and the training forward alone.
enum SweepMode { kInfer, kForward, kTrain };  // kForward and kTrain leave the activations in memory
template <int RT, SweepMode MODE>
__global__ void __launch_bounds__(64 * kSweepWaves, 2) sweep_kernel(SweepArgs a)
{
    static_assert(MODE == kInfer || RT == kSweepRows / 16, "column sums are those of kSweepRows samples");
    constexpr int kRows = 16 * RT;
    constexpr bool train = MODE != kInfer, back = MODE == kTrain;
    __shared__ __attribute__((aligned(16))) uint16_t act[kRows][kActLd];
    // pre-activations, [layer][tile][thread], each thread's own
    __shared__ f32x4 z[back ? kLayers - 1 : 1][back ? 2 * RT : 1][back ? 64 * kSweepWaves : 1];
    __shared__ __attribute__((aligned(16))) uint16_t w_out[kHidden];
    __shared__ uint16_t d_out[kRows];
    __shared__ float t_out[kRows];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int kl = 8 * (lane >> 4);         // this lane's k offset within a 32-wide step
    const int col = w * 32 + (lane & 15);   // its column of column tile 0
    const int row = 4 * (lane >> 4);        // its first row of row tile 0
    const int m0 = blockIdx.x * kRows;
    f32x4 acc[RT][2];
    LayerFrags f;

    auto product = [&]() {  // acc = start + act . fragments
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = f32x4{f.start[j], f.start[j], f.start[j], f.start[j]};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            bf16x8 af[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i)
                af[i] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const s16x8 *>(&act[16 * i + (lane & 15)][32 * s + kl]));
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        af[i], __builtin_bit_cast(bf16x8, f.b[s][j]), acc[i][j], 0, 0, 0);
        }
    };
    // values v of this wavefront's tiles to LDS and to memory (zero for rows past the batch)
    auto publish = [&](const f32x4 (&v)[RT][2], uint16_t *out) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = 16 * i + row, c = col + 16 * j;
                const uint32_t lo = to_bf16x2(v[i][j][0], v[i][j][1]);
                const uint32_t hi = to_bf16x2(v[i][j][2], v[i][j][3]);
                act[r][c] = (uint16_t)lo;
                act[r + 1][c] = (uint16_t)(lo >> 16);
                act[r + 2][c] = (uint16_t)hi;
                act[r + 3][c] = (uint16_t)(hi >> 16);
                if (train)
                    *reinterpret_cast<uint2 *>(out + sample_index(m0 + r, row_tiles(kHidden), c)) =
                        make_uint2(lo, hi);
            }
    };
    auto activate = [&](int l) {
        f32x4 g[RT][2];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (back) z[l][2 * i + j][threadIdx.x] = acc[i][j];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    g[i][j][v] = m0 + 16 * i + row + v < a.B ? gelu(acc[i][j][v]) : 0.f;
            }
        publish(g, a.act[l + 1]);
    };

    // layer 0 (K = 4): lanes 0..15 carry k = 0..3 of their row (A) or column (B)
    {
        const uint16_t *W = a.pb + param_offset_w(0);
        bf16x8 bf[2], af[RT];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
            if (lane < 16) {
#pragma unroll
                for (int k = 0; k < kIn; ++k) b[k] = (short)W[(col + 16 * j) * kIn + k];
            }
            bf[j] = __builtin_bit_cast(bf16x8, b);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            s16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            const int m = m0 + 16 * i + lane;
            if (lane < 16 && m < a.B) {
#pragma unroll
                for (int k = 0; k < kIn; ++k) v[k] = (short)to_bf16(a.x[(int64_t)m * kIn + k]);
            }
            if (train && w == 0 && lane < 16) {
#pragma unroll
                for (int k = 0; k < kIn; ++k) a.act[0][sample_index(m, 1, k)] = (uint16_t)v[k];
            }
            af[i] = __builtin_bit_cast(bf16x8, v);
        }
        float b0[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) b0[j] = a.p[param_offset_b(0) + col + 16 * j];
        f.load(a.pb + hidden_offset(1), a.p + param_offset_b(1), w, lane);
        if (threadIdx.x < kHidden)
            w_out[threadIdx.x] = a.pb[param_offset_w(kLayers - 1) + threadIdx.x];
        if (back && threadIdx.x < kRows)
            t_out[threadIdx.x] = m0 + (int)threadIdx.x < a.B ? a.target[m0 + threadIdx.x] : 0.f;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    af[i], bf[j], f32x4{b0[j], b0[j], b0[j], b0[j]}, 0, 0, 0);
    }
    const float bias_out = a.p[param_offset_b(kLayers - 1)];
    activate(0);
    __syncthreads();
#pragma unroll 1
    for (int l = 1; l < kLayers - 1; ++l) {
        product();
        if (l + 1 < kLayers - 1)
            f.load(a.pb + hidden_offset(l + 1), a.p + hidden_offset(l + 1) + kHidden * kHidden, w, lane);
        else if (back)
            f.load(a.pbT + hidden_offset(l), nullptr, w, lane);  // the way back
        __syncthreads();  // every wavefront has read this layer's input
        activate(l);
        __syncthreads();
    }

    // output layer (256 -> 1): the first wavefront; the B fragment is nonzero only in column 0
    if (w == 0) {
        f32x4 o[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) o[i] = f32x4{bias_out, bias_out, bias_out, bias_out};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
            if ((lane & 15) == 0) b = *reinterpret_cast<const s16x8 *>(&w_out[32 * s + kl]);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const bf16x8 af = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const s16x8 *>(&act[16 * i + (lane & 15)][32 * s + kl]));
                o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, __builtin_bit_cast(bf16x8, b), o[i],
                                                               0, 0, 0);
            }
        }
        float csum = 0.f;
        double lsum = 0.0;
        if ((lane & 15) == 0) {
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                float d[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = m0 + 16 * i + row + v;
                    d[v] = 0.f;
                    if (m < a.B) {
                        a.y[m] = o[i][v];
                        if (back) {
                            const float e = o[i][v] - t_out[16 * i + row + v];
                            d[v] = e * a.inv_b2;
                            lsum += (double)e * (double)e;
                            csum = __builtin_fmaf(e, a.inv_b2, csum);
                        }
                    }
                }
                if (back) {
                    const uint32_t lo = to_bf16x2(d[0], d[1]), hi = to_bf16x2(d[2], d[3]);
                    const int r = 16 * i + row;
                    d_out[r] = (uint16_t)lo;
                    d_out[r + 1] = (uint16_t)(lo >> 16);
                    d_out[r + 2] = (uint16_t)hi;
                    d_out[r + 3] = (uint16_t)(hi >> 16);
                    *reinterpret_cast<uint2 *>(a.err[kLayers - 1] + sample_index(m0 + r, 1, 0)) =
                        make_uint2(lo, hi);
                }
            }
        }
        if (back) {
            csum += __shfl_xor(csum, 16);
            csum += __shfl_xor(csum, 32);
            lsum += __shfl_xor(lsum, 16);
            lsum += __shfl_xor(lsum, 32);
            if (lane == 0) {
                a.bpart[kLayers - 1][blockIdx.x] = csum;
                a.lpart[blockIdx.x] = lsum;
            }
        }
    }
    if constexpr (back) {
    __syncthreads();

    {
        // delta_4 W_4: K = 1, one 32-wide step whose other k are zero
        static_assert(RT == 2);
        bf16x8 af[2], bf[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            s16x8 v = {0, 0, 0, 0, 0, 0, 0, 0}, b = {0, 0, 0, 0, 0, 0, 0, 0};
            if (lane < 16) {
                v[0] = (short)d_out[16 * q + lane];
                b[0] = (short)w_out[col + 16 * q];
            }
            af[q] = __builtin_bit_cast(bf16x8, v);
            bf[q] = __builtin_bit_cast(bf16x8, b);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j],
                                                                    f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    // back: acc holds delta_{l+1} W_{l+1}; the error of layer l is that times gelu'(z_l)
#pragma unroll 1
    for (int l = kLayers - 2; l >= 0; --l) {
        f32x4 d[RT][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float csum = 0.f;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const f32x4 zl = z[l][2 * i + j][threadIdx.x];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float t = 0.f;
                    if (m0 + 16 * i + row + v < a.B) {
                        t = acc[i][j][v] * gelu_d(zl[v]);
                        asm("" : "+v"(t));  // the sum takes the rounded error: no fused operation
                        csum += t;
                    }
                    d[i][j][v] = t;
                }
            }
            csum += __shfl_xor(csum, 16);
            csum += __shfl_xor(csum, 32);
            if (lane < 16) a.bpart[l][(int64_t)blockIdx.x * kHidden + col + 16 * j] = csum;
        }
        publish(d, a.err[l]);
        if (l == 0) break;
        __syncthreads();
        product();
        if (l > 1) f.load(a.pbT + hidden_offset(l - 1), nullptr, w, lane);
        __syncthreads();
    }
    }
}

// One weight-gradient product C (M x N) = A (M x K) B (N x K)^T over the batch (K), in chunks.
struct WGrad {
    int M, N;
    int k_chunk;         // K range of chunk z: [z k_chunk, min(Kp, (z + 1) k_chunk))
    int tiles_m, tiles_n;
    int blk0;            // first block of this product
    const uint16_t *A;   // errors (sample_index order)
    const uint16_t *B;   // activations, likewise
    float *out;          // chunk z at out + z M N
};
struct WGradArgs {
    WGrad g[kLayers];
    int Kp;  // batch rounded up to 32
};

// fragment of row tile `tile` and K step `step`, zero past the last row
__device__ inline s16x8 load_frag(const uint16_t *base, int rows, int tile, int step, int lane)
{
    s16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if (tile * 16 + (lane & 15) < rows)
        v = *reinterpret_cast<const s16x8 *>(base + sample_frag(step, row_tiles(rows), tile, lane));
    return v;
}

// one 64 x 64 output tile of one K chunk
__device__ inline void wgrad_tile(const WGradArgs &a, const WGrad &g, int blk)
{
    const int m_blk = blk % g.tiles_m * kTile, n_blk = blk / g.tiles_m % g.tiles_n * kTile;
    const int kz = blk / (g.tiles_m * g.tiles_n);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k_beg = kz * g.k_chunk, k_end = min(a.Kp, k_beg + g.k_chunk);
    const int ta = m_blk / 16 + (w >> 1) * 2, tb = n_blk / 16 + (w & 1) * 2;  // first row tiles
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = k_beg; kb < k_end; kb += 32 * kStepsAhead) {
        s16x8 fa[kStepsAhead][2], fb[kStepsAhead][2];
#pragma unroll
        for (int s = 0; s < kStepsAhead; ++s) {
            const int k = kb + 32 * s;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[s][i] = s16x8{0, 0, 0, 0, 0, 0, 0, 0};
                fb[s][i] = s16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
            if (k < k_end) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    fa[s][i] = load_frag(g.A, g.M, ta + i, k / 32, lane);
                    fb[s][i] = load_frag(g.B, g.N, tb + i, k / 32, lane);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < kStepsAhead; ++s) {
            if (kb + 32 * s < k_end) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, fa[s][i]), __builtin_bit_cast(bf16x8, fb[s][j]),
                            acc[i][j], 0, 0, 0);
            }
        }
    }
    float *o = g.out + (int64_t)kz * g.M * g.N;
    const int mrow = m_blk + (w >> 1) * 32 + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = mrow + 16 * i + v, n = 16 * (tb + j) + (lane & 15);
                if (m < g.M && n < g.N) o[(int64_t)m * g.N + n] = acc[i][j][v];
            }
}

__global__ void __launch_bounds__(256) wgrad_kernel(WGradArgs a)
{
    int l = 0;
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if ((int)blockIdx.x >= a.g[q].blk0) l = q;
    wgrad_tile(a, a.g[l], blockIdx.x - a.g[l].blk0);
}

struct FinishArgs {
    float *p, *g, *m, *v;
    uint16_t *pb, *pbT;
    const float *wpart[kLayers];  // chunk sums of dW_l: [chunk][N_l][K_l]
    int wsplit[kLayers];
    const float *bpart[kLayers];  // sums of db_l over 32 samples: [block][N_l]
    int nblk;                     // blocks of 64 samples
    const double *losspart;
    double *loss;
    int B;
    int adam;
    float lr, b1, b2, eps, c1, c2;
};

constexpr int kBiasBlocks = (kLayers - 1) * (kHidden / 64) + 1;  // 64 biases each; the output's last
constexpr int kBiasStage = 64;  // 64-sample sums per bias staged in LDS at a time

// one parameter's Adam state, fetched before its gradient is summed
struct AdamState {
    float p, m, v;
    __device__ inline AdamState(const FinishArgs &f, int i)
        : p(f.adam ? f.p[i] : 0.f), m(f.adam ? f.m[i] : 0.f), v(f.adam ? f.v[i] : 0.f)
    {
    }
    // one step with gradient gi; returns the new parameter
    __device__ inline float step(const FinishArgs &f, int i, float gi) const
    {
        // the multiply-adds are written out, so that their rounding does not depend on the code
        // around them
        const float mi = __builtin_fmaf(gi, 1.f - f.b1, f.b1 * m);
        const float vi = __builtin_fmaf(f.b2, v, (1.f - f.b2) * gi * gi);
        f.m[i] = mi;
        f.v[i] = vi;
        const float pi = p - f.lr * (mi / f.c1) / (sqrtf(vi / f.c2) + f.eps);
        f.p[i] = pi;
        return pi;
    }
};

// the BF16 mirrors of weight (n, k) of a layer whose parameters start at `off`: W, for hidden
// layers in fragment order, and W^T
__device__ inline void mirror(uint16_t *pb, uint16_t *pbT, int off, int N, int K, int n, int k, float w)
{
    const uint16_t b = to_bf16(w);
    if (N == kHidden && K == kHidden) {
        pb[off + frag_index(n, k)] = b;
        pbT[off + frag_index(k, n)] = b;
    } else {
        pb[off + n * K + k] = b;
    }
}

// Gradients of 64 biases of layer l (the output layer has one) from the sums over 32 samples,
// added in pairs and then in block order; with the output layer, the loss.  The whole block
// fetches the sums, so that their latencies overlap; one wavefront adds.
__device__ inline void finish_biases(const FinishArgs &f, int blk, float (*sums)[64], double *loss)
{
    const bool out = blk == kBiasBlocks - 1;
    const int l = out ? kLayers - 1 : blk / (kHidden / 64);
    const int n0 = out ? 0 : blk % (kHidden / 64) * 64;
    const int N = out ? 1 : kHidden;
    const float *bp = f.bpart[0];
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if (l == q) bp = f.bpart[q];
    const int c = threadIdx.x & 63;
    int off = param_offset_b(0);
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if (l == q) off = param_offset_b(q);
    const int i = off + min(n0 + c, N - 1);
    const AdamState st(f, i);
    float gi = 0.f;
    double s = 0.0;
    for (int b0 = 0; b0 < f.nblk; b0 += kBiasStage) {
        const int nb = min(kBiasStage, f.nblk - b0);
        if (n0 + c < N) {
#pragma unroll 16
            for (int u = threadIdx.x / 64; u < nb; u += 4) {
                const int64_t o = (int64_t)(2 * (b0 + u)) * N + n0 + c;
                sums[u][c] = bp[o] + bp[o + N];
            }
        }
        if (out && threadIdx.x < nb)
            loss[threadIdx.x] = f.losspart[2 * (b0 + threadIdx.x)] + f.losspart[2 * (b0 + threadIdx.x) + 1];
        __syncthreads();
        if (threadIdx.x < 64 && n0 + c < N)
            for (int u = 0; u < nb; ++u) gi += sums[u][c];
        if (out && threadIdx.x == 0)
            for (int u = 0; u < nb; ++u) s += loss[u];
        __syncthreads();
    }
    if (out && threadIdx.x == 0) *f.loss = s / (double)f.B;
    if (threadIdx.x >= 64 || n0 + c >= N) return;
    f.g[i] = gi;
    if (f.adam) st.step(f, i, gi);
}

// gradient of every parameter from its partial sums (chunk or block order), the
// loss, and (adam != 0) one Adam step with the BF16 mirrors W and W^T refreshed.
// The first kBiasBlocks blocks take the biases, the rest the weights.
__global__ void __launch_bounds__(256) finish_kernel(FinishArgs f)
{
    __shared__ float sums[kBiasStage][64];
    __shared__ double loss[kBiasStage];
    if (blockIdx.x < kBiasBlocks) {
        finish_biases(f, blockIdx.x, sums, loss);
        return;
    }
    const int i = (blockIdx.x - kBiasBlocks) * blockDim.x + threadIdx.x;
    if (i >= kParams) return;
    int l = 0;
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if (i >= param_offset_w(q)) l = q;
    int K = kDims[0], N = kDims[1], S = f.wsplit[0], off = 0;
    const float *wp = f.wpart[0];
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if (l == q) {
            K = kDims[q];
            N = kDims[q + 1];
            S = f.wsplit[q];
            wp = f.wpart[q];
            off = param_offset_w(q);
        }
    const int local = i - off;
    if (local >= N * K) return;  // a bias
    // every partial is loaded before the first add (a runtime-length loop would wait
    // for each load in turn); the sums still run in chunk order
    const AdamState st(f, i);
    float gi = 0.f;
    float q[kMaxSplit];
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s) q[s] = s < S ? wp[(int64_t)s * N * K + local] : 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s)
        if (s < S) gi += q[s];
    f.g[i] = gi;
    if (!f.adam) return;
    mirror(f.pb, f.pbT, off, N, K, local / K, local % K, st.step(f, i, gi));
}

// BF16 mirrors W and W^T of the FP32 parameters (after they are set)
__global__ void mirror_kernel(const float *p, uint16_t *pb, uint16_t *pbT)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kParams) return;
    int K = kDims[0], N = kDims[1], off = 0;
#pragma unroll
    for (int q = 1; q < kLayers; ++q)
        if (i >= param_offset_w(q)) {
            K = kDims[q];
            N = kDims[q + 1];
            off = param_offset_w(q);
        }
    const int local = i - off;
    if (local < N * K) mirror(pb, pbT, off, N, K, local / K, local % K, p[i]);
}

__global__ void zero_f32_kernel(float *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

__global__ void activation_kernel(const float *z, int64_t n, int derivative, float *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = derivative ? gelu_d(z[i]) : gelu(z[i]);
}

// one MFMA tile with the network's fragment mapping (lane-layout check)
__global__ void __launch_bounds__(64) mfma_probe_kernel(const uint16_t *A, const uint16_t *B,
                                                        float *D)
{
    const int lane = threadIdx.x;
    const int kk = 8 * (lane >> 4);
    s16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        a[e] = (short)A[(lane & 15) * 32 + kk + e];
        b[e] = (short)B[(kk + e) * 16 + (lane & 15)];
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) D[(4 * (lane >> 4) + v) * 16 + (lane & 15)] = acc[v];
}

// Fused inference of large batches: one block carries kInferRows samples through all layers,
// their activations staying in LDS (BF16, rows padded by 8 elements so that
// the 16-byte fragment reads of 16 consecutive rows spread over the banks).
// Every layer runs on MFMA with the same operand roundings as the training
// forward: BF16 weights and activations, FP32 accumulation and bias, GELU in
// FP32 rounded to BF16.  The first layer's K = 4 is one 32-wide MFMA step with
// the other 28 k zero, and the last layer's single output is column 0 of a
// 16-column tile whose other columns have zero weights.  In the first four
// layers each of the kInferWaves wavefronts owns 256 / kInferWaves output
// columns for all kInferRows rows and its accumulators start at the bias; the
// weight fragments come from global memory (every block reads the same
// 128 KiB per layer, so they are L2 hits) one K step ahead of use.  The LDS
// tile (67.6 KB) allows two blocks per CU.
constexpr int kInferRows = 128;
constexpr int kInferWaves = 8;
constexpr int kInferThreads = 64 * kInferWaves;
// the 1D grid of ceil(B / kInferRows) blocks must hold fewer than 2^32 threads
constexpr int kMaxInferBatch = 1 << 30;
__global__ void __launch_bounds__(kInferThreads, kInferWaves / 2)
    infer_kernel(const float *__restrict__ x, int B, const float *__restrict__ p,
                 const uint16_t *__restrict__ pb, float *__restrict__ y)
{
    constexpr int RT = kInferRows / 16;        // row tiles
    constexpr int CW = kHidden / kInferWaves;  // columns per wavefront
    constexpr int JT = CW / 16;                // column tiles per wavefront
    constexpr int OT = RT / kInferWaves;       // output-layer row tiles per wavefront
    static_assert(JT >= 1 && OT >= 1, "wavefront count");
    __shared__ __attribute__((aligned(16))) uint16_t act[kInferRows][kActLd];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int kl = 8 * (lane >> 4);  // this lane's k offset within a 32-wide step
    const int64_t row0 = (int64_t)blockIdx.x * kInferRows;
    f32x4 acc[RT][JT];

    auto start = [&](int l) {
        const float *bias = p + param_offset_b(l);
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            const float bn = bias[w * CW + j * 16 + (lane & 15)];
#pragma unroll
            for (int i = 0; i < RT; ++i) acc[i][j] = f32x4{bn, bn, bn, bn};
        }
    };
    // GELU of the accumulators, rounded to BF16 in pairs, into this wavefront's columns
    auto finish = [&]() {
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            const int col = w * CW + j * 16 + (lane & 15);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int v = 0; v < 4; v += 2) {
                    const uint32_t g = to_bf16x2(gelu(acc[i][j][v]), gelu(acc[i][j][v + 1]));
                    const int r = i * 16 + 4 * (lane >> 4) + v;
                    act[r][col] = (uint16_t)g;
                    act[r + 1][col] = (uint16_t)(g >> 16);
                }
        }
    };

    // layer 0 (K = kIn): lanes 0..15 carry k = 0..3 of their row (A) or column (B)
    {
        const uint16_t *W = pb + param_offset_w(0);
        start(0);
        bf16x8 bfr[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
            if (lane < 16) {
                const int col = w * CW + j * 16 + lane;
#pragma unroll
                for (int k = 0; k < kIn; ++k) b[k] = (short)W[col * kIn + k];
            }
            bfr[j] = __builtin_bit_cast(bf16x8, b);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            s16x8 a = {0, 0, 0, 0, 0, 0, 0, 0};
            const int64_t r = row0 + i * 16 + lane;
            if (lane < 16 && r < B) {
#pragma unroll
                for (int k = 0; k < kIn; ++k) a[k] = (short)to_bf16(x[r * kIn + k]);
            }
            const bf16x8 af = __builtin_bit_cast(bf16x8, a);
#pragma unroll
            for (int j = 0; j < JT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfr[j], acc[i][j], 0, 0, 0);
        }
        finish();
        __syncthreads();
    }

    // hidden layers 1 .. kLayers-2 (256 x 256)
    for (int l = 1; l < kLayers - 1; ++l) {
        const uint16_t *W = pb + param_offset_w(l);
        start(l);
        s16x8 bnext[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) {
            bnext[j] = weight_frag(W, 0, w * JT + j, lane);
        }
        for (int k0 = 0; k0 < kHidden; k0 += 32) {
            bf16x8 bfr[JT];
#pragma unroll
            for (int j = 0; j < JT; ++j) bfr[j] = __builtin_bit_cast(bf16x8, bnext[j]);
            if (k0 + 32 < kHidden) {
#pragma unroll
                for (int j = 0; j < JT; ++j) {
                    bnext[j] = weight_frag(W, k0 / 32 + 1, w * JT + j, lane);
                }
            }
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const bf16x8 af = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const s16x8 *>(&act[i * 16 + (lane & 15)][k0 + kl]));
#pragma unroll
                for (int j = 0; j < JT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfr[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();  // every wavefront has read this layer's input
        finish();
        __syncthreads();
    }

    // output layer (256 -> 1): wavefront w takes row tiles OT w .. OT w + OT - 1; the B
    // fragment is nonzero only in column 0 (lanes 0, 16, 32, 48)
    {
        const uint16_t *W = pb + param_offset_w(kLayers - 1);
        const float bias = p[param_offset_b(kLayers - 1)];
        f32x4 o[OT];
#pragma unroll
        for (int ii = 0; ii < OT; ++ii) o[ii] = f32x4{bias, bias, bias, bias};
#pragma unroll
        for (int k0 = 0; k0 < kHidden; k0 += 32) {
            s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
            if ((lane & 15) == 0) b = *reinterpret_cast<const s16x8 *>(W + k0 + kl);
            const bf16x8 bf = __builtin_bit_cast(bf16x8, b);
#pragma unroll
            for (int ii = 0; ii < OT; ++ii) {
                const int rt = OT * w + ii;
                const bf16x8 af = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const s16x8 *>(&act[rt * 16 + (lane & 15)][k0 + kl]));
                o[ii] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, o[ii], 0, 0, 0);
            }
        }
        if ((lane & 15) == 0) {
#pragma unroll
            for (int ii = 0; ii < OT; ++ii)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int64_t r = row0 + (OT * w + ii) * 16 + 4 * (lane >> 4) + v;
                    if (r < B) y[r] = o[ii][v];
                }
        }
    }
}

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline int round_up(int v, int q) { return (v + q - 1) / q * q; }

struct Layout {
    size_t p, g, m, v, pb, pbT;      // parameters, gradients, Adam moments, BF16 mirrors W and W^T
    size_t act[kLayers];             // BF16 inputs of every layer (sample_index order)
    size_t err[kLayers];             // BF16 errors of every layer, likewise
    size_t y;                        // FP32 output (B)
    size_t wpart[kLayers];           // FP32 chunk sums of the weight gradients
    size_t bpart[kLayers];           // FP32 sums of the bias gradients over 32 samples
    size_t lpart;                    // FP64 sums of the squared errors over 32 samples
    size_t loss;                     // FP64
    size_t total;
};

Layout plan(int Bm)
{
    Layout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    const size_t Bp = (size_t)round_up(Bm, kTile);
    const size_t nblk = Bp / kSweepRows;
    L.p = take(4 * (size_t)kParams);
    L.g = take(4 * (size_t)kParams);
    L.m = take(4 * (size_t)kParams);
    L.v = take(4 * (size_t)kParams);
    L.pb = take(2 * (size_t)kParams);
    L.pbT = take(2 * (size_t)kParams);
    for (int l = 0; l < kLayers; ++l) {
        L.act[l] = take(2 * (size_t)(16 * row_tiles(kDims[l])) * Bp);
        L.err[l] = take(2 * (size_t)(16 * row_tiles(kDims[l + 1])) * Bp);
    }
    L.y = take(4 * (size_t)Bm);
    for (int l = 0; l < kLayers; ++l) {
        const size_t nk = (size_t)kDims[l + 1] * kDims[l];
        L.wpart[l] = take(4 * nk * kMaxSplit);
        L.bpart[l] = take(4 * (size_t)kDims[l + 1] * nblk);
    }
    L.lpart = take(8 * nblk);
    L.loss = take(8);
    L.total = off;
    return L;
}

}  // namespace mlp

using namespace mlp;

struct lb_mlp {
    int Bm = 0;
    char *ws = nullptr;
    hipStream_t stream = nullptr;
    Layout L;
    int64_t step = 0;
    template <typename T> T *at(size_t off) const { return reinterpret_cast<T *>(ws + off); }
};

namespace {

#define MLP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess) return lbw_fail_msg(LB_EDEVICE, hipGetErrorString(e_));   \
    } while (0)

// K split into chunks of whole 32-steps: at most `want` chunks, equal but the last
int split_chunks(int steps, int want, int *per_out = nullptr)
{
    want = std::max(1, std::min(want, steps));
    const int per = (steps + want - 1) / want;
    if (per_out) *per_out = per;
    return (steps + per - 1) / per;
}

// requested K chunks of a weight-gradient product: about 256 workgroups in all,
// each chunk at least 4 steps of 32, at most kMaxSplit chunks
int weight_split(int l, int B)
{
    const int tiles = ((kDims[l + 1] + kTile - 1) / kTile) * ((kDims[l] + kTile - 1) / kTile);
    const int steps = round_up(B, 32) / 32;
    const int want = std::min(kMaxSplit, std::max(1, 256 / tiles));
    return std::max(1, std::min(want, steps / 4));
}

SweepArgs sweep_args(const lb_mlp *h, const float *x, int B, float *y)
{
    const Layout &L = h->L;
    SweepArgs a;
    std::memset(&a, 0, sizeof a);
    a.x = x;
    a.B = B;
    a.p = h->at<float>(L.p);
    a.pb = h->at<uint16_t>(L.pb);
    a.pbT = h->at<uint16_t>(L.pbT);
    a.y = y;
    return a;
}

// Forward for B samples: 16 per block while that leaves no block waiting (256 CUs), else 32.
// Measured, us for 6 / 512 / 4096 / 8192 / 16384 samples: 16 per block 7.7 / 8.2 / 8.9 / 12.6 /
// 22.5, 32 per block 9.2 / 11.0 / 11.5 / 11.8 / 16.8.
void sweep_forward(const lb_mlp *h, const float *x, int B, float *y)
{
    const SweepArgs a = sweep_args(h, x, B, y);
    const dim3 threads(64 * kSweepWaves);
    if (B <= 16 * 256)
        hipLaunchKernelGGL((sweep_kernel<1, kInfer>), dim3((B + 15) / 16), threads, 0, h->stream, a);
    else
        hipLaunchKernelGGL((sweep_kernel<2, kInfer>), dim3((B + 31) / 32), threads, 0, h->stream, a);
}
// Batches up to this size run through the sweep, larger ones through infer_kernel, whose 128
// samples per block reuse each weight four times as often but take 25 us however few they are
// (24576 samples: 23.7 us in the sweep, 27.4 in infer_kernel; 32768: 28.7 and 27.6).
constexpr int kSweepInfer = 24576;

// training forward for B samples (activations to the workspace, outputs to y) and, with targets, back to
// the errors of every layer
void sweep_train(const lb_mlp *h, const float *x, int B, const float *t, float *y)
{
    const Layout &L = h->L;
    SweepArgs a = sweep_args(h, x, B, y);
    a.target = t;
    a.inv_b2 = 2.0f / (float)B;
    for (int l = 0; l < kLayers; ++l) {
        a.act[l] = h->at<uint16_t>(L.act[l]);
        a.err[l] = h->at<uint16_t>(L.err[l]);
        a.bpart[l] = h->at<float>(L.bpart[l]);
    }
    a.lpart = h->at<double>(L.lpart);
    const int blocks = round_up(B, kTile) / kSweepRows;  // the padding rows are written too
    const dim3 threads(64 * kSweepWaves);
    if (t)
        hipLaunchKernelGGL((sweep_kernel<2, kTrain>), dim3(blocks), threads, 0, h->stream, a);
    else
        hipLaunchKernelGGL((sweep_kernel<2, kForward>), dim3(blocks), threads, 0, h->stream, a);
}

// weight gradients (chunk sums) of every layer from what the sweep left
void wgrad(const lb_mlp *h, int B)
{
    const Layout &L = h->L;
    WGradArgs a;
    std::memset(&a, 0, sizeof a);
    a.Kp = round_up(B, 32);
    int blocks = 0;
    for (int l = 0; l < kLayers; ++l) {
        WGrad &g = a.g[l];
        g.M = kDims[l + 1];
        g.N = kDims[l];
        int per = 0;
        const int chunks = split_chunks(a.Kp / 32, weight_split(l, B), &per);
        g.k_chunk = 32 * per;
        g.tiles_m = (g.M + kTile - 1) / kTile;
        g.tiles_n = (g.N + kTile - 1) / kTile;
        g.blk0 = blocks;
        g.A = h->at<uint16_t>(L.err[l]);
        g.B = h->at<uint16_t>(L.act[l]);
        g.out = h->at<float>(L.wpart[l]);
        blocks += g.tiles_m * g.tiles_n * chunks;
    }
    hipLaunchKernelGGL(wgrad_kernel, dim3(blocks), dim3(256), 0, h->stream, a);
}

FinishArgs finish_args(const lb_mlp *h, int B)
{
    const Layout &L = h->L;
    FinishArgs f;
    std::memset(&f, 0, sizeof f);
    f.p = h->at<float>(L.p);
    f.g = h->at<float>(L.g);
    f.m = h->at<float>(L.m);
    f.v = h->at<float>(L.v);
    f.pb = h->at<uint16_t>(L.pb);
    f.pbT = h->at<uint16_t>(L.pbT);
    for (int l = 0; l < kLayers; ++l) {
        f.wpart[l] = h->at<float>(L.wpart[l]);
        f.wsplit[l] = split_chunks(round_up(B, 32) / 32, weight_split(l, B));
        f.bpart[l] = h->at<float>(L.bpart[l]);
    }
    f.nblk = round_up(B, kTile) / kTile;
    f.losspart = h->at<double>(L.lpart);
    f.loss = h->at<double>(L.loss);
    f.B = B;
    return f;
}

void finish(const lb_mlp *h, const FinishArgs &f)
{
    hipLaunchKernelGGL(finish_kernel, dim3(kBiasBlocks + (kParams + 255) / 256), dim3(256), 0,
                       h->stream, f);
}

int check_batch(const lb_mlp *h, int B)
{
    if (!h) return lbw_fail_msg(LB_EINVAL, "handle is NULL");
    if (B < 1 || B > h->Bm) return lbw_fail_msg(LB_EINVAL, "batch outside 1 .. max_batch");
    return LB_OK;
}

int check_adam(float lr, float beta1, float beta2, float eps)
{
    if (!(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
        return lbw_fail_msg(LB_EINVAL, "bad Adam hyper-parameters");
    return LB_OK;
}

// one Adam step (the caller has checked the arguments)
void adam_step(lb_mlp *h, const float *x, const float *t, int B, float lr, float beta1,
               float beta2, float eps)
{
    sweep_train(h, x, B, t, h->at<float>(h->L.y));
    wgrad(h, B);
    h->step++;
    FinishArgs f = finish_args(h, B);
    f.adam = 1;
    f.lr = lr;
    f.b1 = beta1;
    f.b2 = beta2;
    f.eps = eps;
    f.c1 = 1.f - std::pow(beta1, (float)h->step);
    f.c2 = 1.f - std::pow(beta2, (float)h->step);
    finish(h, f);
}

}  // namespace

extern "C" {

int32_t lb_mlp_num_params(void) { return kParams; }

size_t lb_mlp_workspace_bytes(int32_t max_batch)
{
    if (max_batch < 1 || max_batch > kMaxTrainBatch) return 0;
    return plan(max_batch).total;
}

int lb_mlp_create(int32_t max_batch, void *dev_workspace, size_t workspace_bytes, void *hip_stream,
                  lb_mlp **out)
{
    if (!out) return lbw_fail_msg(LB_EINVAL, "out is NULL");
    *out = nullptr;
    if (max_batch < 1 || max_batch > kMaxTrainBatch)
        return lbw_fail_msg(LB_EINVAL, "max_batch must be in 1 .. 2^24");
    Layout L = plan(max_batch);
    if (!dev_workspace || reinterpret_cast<uintptr_t>(dev_workspace) % kAlign)
        return lbw_fail_msg(LB_ENOMEM, "workspace must be 256-byte aligned device memory");
    if (workspace_bytes < L.total) return lbw_fail_msg(LB_ENOMEM, "workspace too small");
    lb_mlp *h = new lb_mlp();
    h->Bm = max_batch;
    h->ws = static_cast<char *>(dev_workspace);
    h->stream = static_cast<hipStream_t>(hip_stream);
    h->L = L;
    const int64_t nz = (int64_t)(L.pb - L.p) / 4;  // parameters, gradients, moments
    hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, h->stream,
                       h->at<float>(L.p), nz);
    hipLaunchKernelGGL(mirror_kernel, dim3((kParams + 255) / 256), dim3(256), 0, h->stream,
                       h->at<float>(L.p), h->at<uint16_t>(L.pb), h->at<uint16_t>(L.pbT));
    hipError_t e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) {
        delete h;
        return lbw_fail_msg(LB_EDEVICE, hipGetErrorString(e));
    }
    *out = h;
    return LB_OK;
}

int lb_mlp_destroy(lb_mlp *h)
{
    delete h;
    return LB_OK;
}

int lb_mlp_set_params(lb_mlp *h, const float *host_params)
{
    if (!h || !host_params) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    MLP_TRY(hipMemcpyAsync(h->at<float>(h->L.p), host_params, 4 * (size_t)kParams,
                           hipMemcpyHostToDevice, h->stream));
    for (size_t off : {h->L.m, h->L.v})
        hipLaunchKernelGGL(zero_f32_kernel, dim3((kParams + 255) / 256), dim3(256), 0, h->stream,
                           h->at<float>(off), (int64_t)kParams);
    hipLaunchKernelGGL(mirror_kernel, dim3((kParams + 255) / 256), dim3(256), 0, h->stream,
                       h->at<float>(h->L.p), h->at<uint16_t>(h->L.pb), h->at<uint16_t>(h->L.pbT));
    MLP_TRY(hipGetLastError());
    MLP_TRY(hipStreamSynchronize(h->stream));
    h->step = 0;
    return LB_OK;
}

int lb_mlp_get_params(lb_mlp *h, float *host_params)
{
    if (!h || !host_params) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    MLP_TRY(hipMemcpyAsync(host_params, h->at<float>(h->L.p), 4 * (size_t)kParams,
                           hipMemcpyDeviceToHost, h->stream));
    MLP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_mlp_forward(lb_mlp *h, const float *dev_x, int32_t B, float *dev_y)
{
    if (!h) return lbw_fail_msg(LB_EINVAL, "handle is NULL");
    if (B < 1) return lbw_fail_msg(LB_EINVAL, "batch must be >= 1");
    if (B > kMaxInferBatch) return lbw_fail_msg(LB_EINVAL, "batch above 2^30");
    if (!dev_x || !dev_y) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    if (B <= kSweepInfer) {
        sweep_forward(h, dev_x, B, dev_y);
        MLP_TRY(hipGetLastError());
        return LB_OK;
    }
    const unsigned blocks = (unsigned)(((int64_t)B + kInferRows - 1) / kInferRows);
    hipLaunchKernelGGL(infer_kernel, dim3(blocks), dim3(kInferThreads), 0, h->stream, dev_x, B,
                       h->at<float>(h->L.p), h->at<uint16_t>(h->L.pb), dev_y);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_mlp_forward_layered(lb_mlp *h, const float *dev_x, int32_t B, float *dev_y)
{
    int st = check_batch(h, B);
    if (st) return st;
    if (!dev_x || !dev_y) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    sweep_train(h, dev_x, B, nullptr, dev_y);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_mlp_grad(lb_mlp *h, const float *dev_x, const float *dev_t, int32_t B, float *host_grads,
                double *host_loss)
{
    int st = check_batch(h, B);
    if (st) return st;
    if (!dev_x || !dev_t || !host_grads) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    sweep_train(h, dev_x, B, dev_t, h->at<float>(h->L.y));
    wgrad(h, B);
    finish(h, finish_args(h, B));
    MLP_TRY(hipGetLastError());
    MLP_TRY(hipMemcpyAsync(host_grads, h->at<float>(h->L.g), 4 * (size_t)kParams,
                           hipMemcpyDeviceToHost, h->stream));
    if (host_loss)
        MLP_TRY(hipMemcpyAsync(host_loss, h->at<double>(h->L.loss), 8, hipMemcpyDeviceToHost,
                               h->stream));
    MLP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_mlp_train_step(lb_mlp *h, const float *dev_x, const float *dev_t, int32_t B, float lr,
                      float beta1, float beta2, float eps)
{
    int st = check_batch(h, B);
    if (st) return st;
    if (!dev_x || !dev_t) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    if ((st = check_adam(lr, beta1, beta2, eps))) return st;
    adam_step(h, dev_x, dev_t, B, lr, beta1, beta2, eps);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_mlp_train_steps(lb_mlp *h, const float *dev_x, const float *dev_t, int32_t B,
                       int32_t n_steps, const float *host_lr, float beta1, float beta2, float eps)
{
    int st = check_batch(h, B);
    if (st) return st;
    if (!dev_x || !dev_t || n_steps < 0 || (n_steps > 0 && !host_lr))
        return lbw_fail_msg(LB_EINVAL, "bad argument");
    for (int s = 0; s < n_steps; ++s)
        if ((st = check_adam(host_lr[s], beta1, beta2, eps))) return st;
    for (int s = 0; s < n_steps; ++s) adam_step(h, dev_x, dev_t, B, host_lr[s], beta1, beta2, eps);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_mlp_last_loss(lb_mlp *h, double *loss)
{
    if (!h || !loss) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    MLP_TRY(hipMemcpyAsync(loss, h->at<double>(h->L.loss), 8, hipMemcpyDeviceToHost, h->stream));
    MLP_TRY(hipStreamSynchronize(h->stream));
    return LB_OK;
}

int lb_mlp_mfma_probe(const uint16_t *dev_A, const uint16_t *dev_B, float *dev_D, void *hip_stream)
{
    if (!dev_A || !dev_B || !dev_D) return lbw_fail_msg(LB_EINVAL, "NULL argument");
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(hip_stream),
                       dev_A, dev_B, dev_D);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

int lb_mlp_activation(const float *dev_z, int64_t n, int32_t derivative, float *dev_out,
                      void *hip_stream)
{
    if (n < 0 || (n > 0 && (!dev_z || !dev_out)))
        return lbw_fail_msg(LB_EINVAL, "activation: bad arguments");
    // one thread per value in a 1D grid, whose thread count must fit 32 bits
    if (n > ((int64_t)1 << 31)) return lbw_fail_msg(LB_EINVAL, "activation: n above 2^31");
    if (n == 0) return LB_OK;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(activation_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(hip_stream), dev_z, n, derivative ? 1 : 0, dev_out);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

}  // extern "C"
