// surrogate.hip -- ensemble of small MLPs (4 -> H -> H -> 2, tanh) that maps
// the parameters of a channel run (capillary number, flow-rate ratio,
// viscosity ratio, width) to its droplet labels, trained on the GPU and
// queried with BF16 matrix-core inference.  Members whose predictions spread
// by more than a threshold send the query back to the lattice Boltzmann
// solver (the fallback mask).
//
// Training is full-batch Adam on the mean squared error, two launches per
// epoch (per CHUNK samples of a larger set):
//   k_fwd_bwd  one block per (16-sample tile, member): forward and backward,
//              both 128 x 128 products on FP32 matrix instructions; leaves
//              the activations and the back-propagated errors
//   k_grad     per 16x16 tile of W2, or per 64 of the other parameters: the
//              gradient, summed over 64-sample groups in order (so the result
//              does not depend on scheduling), then the Adam update in place
// Inference:
//   k_predict  one block per 16 queries, several members at a time: layer 1 on
//              VALU, layer 2 as 16x16x16 BF16 MFMA tiles with FP32
//              accumulation, layer 3 on VALU; ensemble mean, standard
//              deviation and the fallback flag.
// FP32 matrix instructions round every product-sum like a chain of FMAs in
// ascending k (checked bit for bit), so the sums have the order and the bits
// of the plain loops over k.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/lbm.h"

namespace {

constexpr int H = 128;                       // hidden width
constexpr int NIN = 4, NOUT = 2;
constexpr int QT = 16;                       // queries / samples per block
constexpr int FT = 512;                      // threads per block of the training kernels
constexpr int GROUP = 64;                    // samples whose gradient is summed before it joins the total
constexpr int CHUNK = 8192;                  // samples whose activations are held at once
constexpr int LH = H + 4;                    // row pitch of FP32 activations in LDS (rows 4 banks apart)
// parameter vector of one member
constexpr int O_W1 = 0;                      // [H][NIN]
constexpr int O_B1 = O_W1 + H * NIN;         // [H]
constexpr int O_W2 = O_B1 + H;               // [H][H], row i = output unit i
constexpr int O_B2 = O_W2 + H * H;           // [H]
constexpr int O_W3 = O_B2 + H;               // [NOUT][H]
constexpr int O_B3 = O_W3 + NOUT * H;        // [NOUT]
constexpr int P = O_B3 + NOUT;               // 17410 for H = 128

// FP32 -> BF16 bits, round to nearest even (NaN stays NaN)
__device__ __forceinline__ uint16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// counter-based uniform in [-1, 1): splitmix64 of (seed, member, index)
__device__ __forceinline__ float hash_uniform(uint64_t seed, uint64_t m, uint64_t i)
{
    uint64_t z = seed + 0x9E3779B97F4A7C15ull * (m * 0x100000001B3ull + i + 1);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (float)((double)(z >> 11) * (1.0 / 9007199254740992.0)) * 2.0f - 1.0f;
}

// weights uniform in +-1/sqrt(fan_in), biases zero; Adam moments zero
__global__ void k_init(float *__restrict__ params, float *__restrict__ am, float *__restrict__ av, int members,
                       uint64_t seed)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)members * P) return;
    const int m = (int)(t / P), p = (int)(t % P);
    float v = 0.0f;
    if (p < O_B1) v = hash_uniform(seed, m, p) * 0.5f;                      // fan-in 4
    else if (p >= O_W2 && p < O_B2) v = hash_uniform(seed, m, p) * 0.08838834764831845f;   // 1/sqrt(128)
    else if (p >= O_W3 && p < O_B3) v = hash_uniform(seed, m, p) * 0.08838834764831845f;
    params[t] = v;
    am[t] = 0.0f;
    av[t] = 0.0f;
}

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// What one chunk of samples leaves for the gradient: activations and errors
// [member][rows][H], output errors and loss terms [member][rows][NOUT].
struct Acts {
    float *h1, *h2, *z2, *z1, *dy, *lterm;
    int rows;                                // capacity per member
};

// Forward and backward pass of one 16-sample tile through one member.
// loss = sum over samples and outputs of (y - Y)^2 / (n * NOUT).  Row s of
// the chunk is sample base + s; rows past the last sample up to the tile's end
// carry zero errors.
//
// The work of a tile is three 128-deep products of 16 x 128 (0.5 MFLOP each):
// what bounds it is latency, so the tile is small (125 blocks for 385 samples
// and 5 members, where 64-sample tiles gave 35), every weight a wave needs is
// loaded before the layer that uses it, and the products run on matrix
// instructions, which read each activation from LDS once per 16 outputs
// (VALU loops read it once per output and held the whole of W2 in LDS: 102 us
// a launch for 385 samples, 5 members; now 11.5 us here and 7.8 us in k_grad,
// against 4.9 + 4.6 us for the separate gradient-sum and loss launches).
__global__ __launch_bounds__(FT) void k_fwd_bwd(const float *__restrict__ params, const float *__restrict__ w2t,
                                                 const float *__restrict__ X, const float *__restrict__ Y, int n,
                                                 int base, Acts act)
{
    const int m = blockIdx.y, s0 = blockIdx.x * QT;
    const float *w = params + (int64_t)m * P;
    const float *wt = w2t + (int64_t)m * H * H;
    const int64_t arow = (int64_t)m * act.rows + s0;
    __shared__ __align__(16) float s_h1[QT * LH], s_h2[QT * LH], s_z2[QT * LH], s_w3[NOUT * LH];
    __shared__ float s_x[QT * NIN], s_dy[QT * NOUT];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, r = lane % 16, q = lane / 16;
    const int ns = min(QT, n - base - s0);   // valid samples of this tile
    const int col = 16 * wave + r;           // this lane's output column

    // layer 2 weights in operand order: W2[col][4t + q]
    float wf[H / 4];
#pragma unroll
    for (int t = 0; t < H / 4; t++) wf[t] = wt[(4 * t + q) * H + col];
    if (tid < QT * NIN) s_x[tid] = tid / NIN < ns ? X[(int64_t)(base + s0) * NIN + tid] : 0.0f;
    if (tid < NOUT * H) s_w3[tid / H * LH + tid % H] = w[O_W3 + tid];
    __syncthreads();

    // layer 1: h1[s][i] = tanh(b1[i] + sum_c W1[i][c] x[s][c])
    const int i = tid % H, sb = tid / H;
    {
        const float b1 = w[O_B1 + i];
        float w1[NIN];
        for (int c = 0; c < NIN; c++) w1[c] = w[O_W1 + i * NIN + c];
        for (int s = sb; s < QT; s += FT / H) {
            float a = b1;
            for (int c = 0; c < NIN; c++) a = fmaf(w1[c], s_x[s * NIN + c], a);
            const float h = tanhf(a);
            s_h1[s * LH + i] = h;
            act.h1[(arow + s) * H + i] = h;
        }
    }
    __syncthreads();

    // layer 2: samples x 16 columns per wave, summed from the bias upwards in j
    {
        const float b2 = w[O_B2 + col];
        f32x4 acc = {b2, b2, b2, b2};
#pragma unroll
        for (int t = 0; t < H / 4; t++)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(s_h1[r * LH + 4 * t + q], wf[t], acc, 0, 0, 0);
        // the weights of the backward product, on their way while tanh runs:
        // W2[4t + q][col]
#pragma unroll
        for (int t = 0; t < H / 4; t++) wf[t] = w[O_W2 + (4 * t + q) * H + col];
        for (int e = 0; e < 4; e++) s_h2[(4 * q + e) * LH + col] = tanhf(acc[e]);
    }
    __syncthreads();

    // layer 3 and the loss: one thread per (sample, output)
    if (tid < QT * NOUT) {
        const int s = tid / NOUT, o = tid % NOUT;
        float y = w[O_B3 + o];
#pragma unroll 8
        for (int j = 0; j < H; j += 4) {
            const float4 a = *(const float4 *)(s_w3 + o * LH + j), b = *(const float4 *)(s_h2 + s * LH + j);
            y = fmaf(a.x, b.x, y);
            y = fmaf(a.y, b.y, y);
            y = fmaf(a.z, b.z, y);
            y = fmaf(a.w, b.w, y);
        }
        float d = 0.0f, lt = 0.0f;
        if (s < ns) {
            const float res = y - Y[(int64_t)(base + s0 + s) * NOUT + o];
            lt = res * res / (float)(n * NOUT);
            d = 2.0f * res / (float)(n * NOUT);
        }
        s_dy[tid] = d;
        act.dy[arow * NOUT + tid] = d;
        act.lterm[arow * NOUT + tid] = lt;
    }
    __syncthreads();
    // dz2[s][i] = (sum_o dy[s][o] W3[o][i]) (1 - h2^2)
    for (int s = sb; s < QT; s += FT / H) {
        float d = 0.0f;
        for (int o = 0; o < NOUT; o++) d = fmaf(s_dy[s * NOUT + o], s_w3[o * LH + i], d);
        const float h = s_h2[s * LH + i];
        const float z = d * (1.0f - h * h);
        s_z2[s * LH + i] = z;
        act.z2[(arow + s) * H + i] = z;
        act.h2[(arow + s) * H + i] = h;
    }
    __syncthreads();
    // dz1[s][j] = (sum_i dz2[s][i] W2[i][j]) (1 - h1^2)
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < H / 4; t++)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(s_z2[r * LH + 4 * t + q], wf[t], acc, 0, 0, 0);
    for (int e = 0; e < 4; e++) {
        const int s = 4 * q + e;
        const float h = s_h1[s * LH + col];
        act.z1[(arow + s) * H + col] = acc[e] * (1.0f - h * h);
    }
}

// Units of k_grad per member: the 16x16 tiles of W2, 64 of the other
// parameters each (b2, W3, W1 and b1, b3), the loss.
constexpr int G_TILES = (H / 16) * (H / 16);
constexpr int G_REST = H + NOUT * H + (NIN + 1) * H + NOUT;
constexpr int G_VECS = (G_REST + 63) / 64;
constexpr int G_UNITS = G_TILES + G_VECS + 1;

struct Adam {
    float lr, b1, b2, eps, c1, c2;
};

// The gradient of one unit over the rows [0, nr) of a chunk: wave v takes the
// 64-sample groups v, v + 8, ..., and the groups' sums are added in order.
// The total starts from 0, or from gsum after an earlier chunk; after the
// last chunk it is copied to gout and / or updates the parameters.
__global__ __launch_bounds__(FT) void k_grad(float *__restrict__ params, float *__restrict__ w2t,
                                              float *__restrict__ am, float *__restrict__ av,
                                              float *__restrict__ gsum, const float *__restrict__ X, int base, int nr,
                                              Acts act, int first, int last, int update, Adam ad,
                                              float *__restrict__ gout, float *__restrict__ loss)
{
    const int m = blockIdx.y, unit = blockIdx.x;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64, r = lane % 16, q = lane / 16;
    const int ng = (nr + GROUP - 1) / GROUP;
    const int64_t row0 = (int64_t)m * act.rows;
    constexpr int NW = FT / 64;
    __shared__ float s_part[NW * 256];
    const bool tile = unit < G_TILES, is_loss = unit == G_UNITS - 1;
    // the parameter this thread totals, and (other units) its two factors
    int p = -1;
    const float *pa = nullptr, *pb = nullptr;
    int sa = 0, sbs = 0;
    if (tile && tid < 256) {
        p = O_W2 + (16 * (unit / 8) + tid / 16) * H + 16 * (unit % 8) + tid % 16;
    } else if (!tile && !is_loss) {
        int e = (unit - G_TILES) * 64 + lane;
        if (e < H) {                                             // b2: sum of dz2
            p = O_B2 + e;
            pa = act.z2 + row0 * H + e;
            sa = H;
        } else if ((e -= H) < NOUT * H) {                        // W3: dy h2
            const int o = e / H;
            p = O_W3 + e;
            pa = act.h2 + row0 * H + e % H;
            sa = H;
            pb = act.dy + row0 * NOUT + o;
            sbs = NOUT;
        } else if ((e -= NOUT * H) < (NIN + 1) * H) {            // W1, b1: dz1 x, sum of dz1
            const int c = e / H, j = e % H;
            p = c < NIN ? O_W1 + j * NIN + c : O_B1 + j;
            pa = act.z1 + row0 * H + j;
            sa = H;
            if (c < NIN) {
                pb = X + (int64_t)base * NIN + c;
                sbs = NIN;
            }
        } else if ((e -= (NIN + 1) * H) < NOUT) {                // b3: sum of dy
            p = O_B3 + e;
            pa = act.dy + row0 * NOUT + e;
            sa = NOUT;
        }
    }
    const int64_t t = (int64_t)m * P + p;
    float total = 0.0f;
    if (!first) {
        if (is_loss) total = loss[m];
        else if (p >= 0) total = gsum[t];
    }
    for (int g0 = 0; g0 < ng; g0 += NW) {
        const int g = g0 + wave;
        if (g < ng) {
            const int s0 = g * GROUP, left = nr - s0;
            if (tile) {
                // rows beyond the last sample's tile add nothing
                const int steps = left >= GROUP ? GROUP / 4 : (left + QT - 1) / QT * (QT / 4);
                const float *za = act.z2 + (row0 + s0 + q) * H + 16 * (unit / 8) + r;
                const float *hb = act.h1 + (row0 + s0 + q) * H + 16 * (unit % 8) + r;
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                float a[GROUP / 4], b[GROUP / 4];
#pragma unroll
                for (int k = 0; k < GROUP / 4; k++) {
                    a[k] = za[4 * k * H];
                    b[k] = hb[4 * k * H];
                }
#pragma unroll
                for (int k = 0; k < GROUP / 4; k++) {
                    // (the buffers hold whole groups; what lies there is not used)
                    a[k] = k < steps ? a[k] : 0.0f;
                    b[k] = k < steps ? b[k] : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < GROUP / 4; k++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[k], acc, 0, 0, 0);
                for (int e = 0; e < 4; e++) s_part[wave * 256 + (4 * q + e) * 16 + r] = acc[e];
            } else if (is_loss) {
                const float *l = act.lterm + (row0 + s0) * NOUT;
                const int have = min(left, GROUP) * NOUT;
                float v = (lane < have ? l[lane] : 0.0f) + (lane + 64 < have ? l[lane + 64] : 0.0f);
                for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
                if (lane == 0) s_part[wave * 64] = v;
            } else if (p >= 0) {
                const int rows = min(left, GROUP);
                const float *qa = pa + (int64_t)s0 * sa, *qb = pb ? pb + (int64_t)s0 * sbs : nullptr;
                float a = 0.0f;
                int s = 0;
                // 16 rows' loads in flight at a time
                for (; s + 16 <= rows; s += 16) {
                    float f[16], h[16];
#pragma unroll
                    for (int k = 0; k < 16; k++) f[k] = qa[(s + k) * sa];
                    if (qb) {
#pragma unroll
                        for (int k = 0; k < 16; k++) h[k] = qb[(s + k) * sbs];
                    } else {
#pragma unroll
                        for (int k = 0; k < 16; k++) h[k] = 1.0f;
                    }
#pragma unroll
                    for (int k = 0; k < 16; k++) a = fmaf(f[k], h[k], a);
                }
                for (; s < rows; s++) a = fmaf(qa[s * sa], qb ? qb[s * sbs] : 1.0f, a);
                s_part[wave * 64 + lane] = a;
            }
        }
        __syncthreads();
        const int stride = tile ? 256 : 64, at = tile ? tid : lane;
        if (tid < 256)
            for (int v = 0; v < NW && g0 + v < ng; v++) total += s_part[v * stride + at];
        __syncthreads();
    }
    if (is_loss) {
        if (tid == 0) loss[m] = total;
        return;
    }
    if (p < 0 || (!tile && wave != 0)) return;
    if (!last) {
        gsum[t] = total;
        return;
    }
    if (gout) gout[t] = total;
    if (!update) return;
    const float mm = ad.b1 * am[t] + (1.0f - ad.b1) * total;
    const float vv = ad.b2 * av[t] + (1.0f - ad.b2) * total * total;
    am[t] = mm;
    av[t] = vv;
    const float nw = params[t] - ad.lr * (mm / ad.c1) / (sqrtf(vv / ad.c2) + ad.eps);
    params[t] = nw;
    if (tile) w2t[(int64_t)m * H * H + (p - O_W2) % H * H + (p - O_W2) / H] = nw;
}

// The copies of W2 below follow the weights on the context's stream: after
// surr_create and surr_set_params, and at the latest at the end of surr_train.
// Nothing on the host remembers whether they do, so a call that the caller
// captured reads the weights of its replay, not those of its capture.

// W2 of every member transposed, as the forward product of training reads it
// (k_grad updates it with the weights)
__global__ void k_w2_transpose(const float *__restrict__ params, int members, float *__restrict__ w2t)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)members * H * H) return;
    const int m = (int)(t / (H * H)), e = (int)(t % (H * H)), j = e / H, i = e % H;
    w2t[t] = params[(int64_t)m * P + O_W2 + i * H + j];
}

// W2 of every member as BF16 (round to nearest even) for inference, in the
// order the matrix instructions of k_predict read it: [column tile][pair of
// 16-wide k chunks][lane][chunk of the pair][4 values of k]
__global__ void k_w2_bf16(const float *__restrict__ params, int members, uint16_t *__restrict__ w2)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)members * H * H) return;
    const int m = (int)(t / (H * H)), e = (int)(t % (H * H));
    const int ct = e / (16 * H), kp = e / 512 % 4, lane = e / 8 % 64, c = e / 4 % 2, k = e % 4;
    const int i = 16 * ct + lane % 16, j = 32 * kp + 16 * c + 4 * (lane / 16) + k;
    w2[t] = to_bf16(params[(int64_t)m * P + O_W2 + i * H + j]);
}

// One block of 512 threads (8 waves) answers 16 queries, `mc` members at a
// time: wave v owns the columns 16v .. 16v + 15 of layer 2 of each of them.
//
// Two thirds of the time of a block is tanh, the rest latency, so the queries
// are spread thin (4096 queries are 256 blocks, one per CU; 64-query blocks
// left three CUs of four idle) and the members of a pass run side by side, not
// in turn: their layer-3 sums are 128-long dependent chains.  4096 queries and
// 5 members take 11.7 us a call, against 99 us with 64-query blocks, members
// in turn and 2-byte loads of W2.
constexpr int PT = 512;                      // threads per block
constexpr int LB = H + 8;                    // row pitch of BF16 activations in LDS
constexpr int MC_MAX = 5;                    // members per pass (69 KB of LDS: two blocks per CU)
constexpr size_t predict_lds(int mc) { return (size_t)mc * (QT * LH * 4 + QT * LB * 2 + NOUT * LH * 4); }

__global__ __launch_bounds__(PT) void k_predict(const float *__restrict__ params, const uint16_t *__restrict__ w2,
                                                int members, int mc, const float *__restrict__ X, int n,
                                                float *__restrict__ mean, float *__restrict__ sd,
                                                uint8_t *__restrict__ fallback, float thresh, float2 oscale,
                                                float2 oshift)
{
    extern __shared__ __align__(16) unsigned char s_dyn[];
    float *s_h2 = (float *)s_dyn;                                // [mc][QT][LH] layer-2 activations
    float *s_w3 = s_h2 + mc * QT * LH;                           // [mc][NOUT][LH]
    uint16_t *s_h1 = (uint16_t *)(s_w3 + mc * NOUT * LH);        // [mc][QT][LB] layer-1 activations, BF16
    __shared__ float s_x[QT * NIN], s_y[MC_MAX * QT * NOUT];
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int s0 = blockIdx.x * QT;
    const int ns = min(QT, n - s0);
    if (tid < QT * NIN) s_x[tid] = tid / NIN < ns ? X[(int64_t)s0 * NIN + tid] : 0.0f;
    float sum = 0.0f, sq = 0.0f;                                 // of query tid / 2, output tid % 2 (tid < 32)
    for (int m0 = 0; m0 < members; m0 += mc) {
        const int nm = min(mc, members - m0);
        __syncthreads();
        const int i = tid % H, sb = tid / H;
        for (int m = 0; m < nm; m++) {
            const float *w = params + (int64_t)(m0 + m) * P;
            const float b1 = w[O_B1 + i];
            float w1[NIN];
            for (int c = 0; c < NIN; c++) w1[c] = w[O_W1 + i * NIN + c];
            for (int s = sb; s < QT; s += PT / H) {
                float a = b1;
                if (s < ns)
                    for (int c = 0; c < NIN; c++) a = fmaf(w1[c], s_x[s * NIN + c], a);
                s_h1[(m * QT + s) * LB + i] = to_bf16(tanhf(a));
            }
            if (tid < NOUT * H) s_w3[(m * NOUT + tid / H) * LH + tid % H] = w[O_W3 + tid];
        }
        __syncthreads();
        // z2 = h1 W2^T.  16x16x16 operands: lane l holds row (A) / column (B)
        // l % 16 and k = 4 (l / 16) .. +3 of the 16-wide k chunk; the result
        // holds column l % 16 and rows 4 (l / 16) .. +3.
        const int r = lane % 16, q = lane / 16, col = 16 * wave + r;
        for (int m = 0; m < nm; m++) {
            const float b2 = params[(int64_t)(m0 + m) * P + O_B2 + col];
            const uint4 *wb = (const uint4 *)(w2 + (int64_t)(m0 + m) * H * H + wave * 16 * H) + lane;
            uint4 bw[4];
#pragma unroll
            for (int kp = 0; kp < 4; kp++) bw[kp] = wb[64 * kp];
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kp = 0; kp < 4; kp++) {
                const uint2 lo = make_uint2(bw[kp].x, bw[kp].y), hi = make_uint2(bw[kp].z, bw[kp].w);
                const uint16_t *pa = s_h1 + (m * QT + r) * LB + 32 * kp + 4 * q;
                const uint2 alo = *(const uint2 *)pa, ahi = *(const uint2 *)(pa + 16);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, alo),
                                                                __builtin_bit_cast(bf16x4, lo), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, ahi),
                                                                __builtin_bit_cast(bf16x4, hi), acc, 0, 0, 0);
            }
            for (int e = 0; e < 4; e++) s_h2[(m * QT + 4 * q + e) * LH + col] = tanhf(acc[e] + b2);
        }
        __syncthreads();
        if (tid < nm * QT * NOUT) {
            const int m = tid / (QT * NOUT), s = tid / NOUT % QT, o = tid % NOUT;
            float y = params[(int64_t)(m0 + m) * P + O_B3 + o];
            const float *w3 = s_w3 + (m * NOUT + o) * LH, *h2 = s_h2 + (m * QT + s) * LH;
#pragma unroll 4
            for (int j = 0; j < H; j += 4) {
                const float4 a = *(const float4 *)(w3 + j), b = *(const float4 *)(h2 + j);
                y = fmaf(a.x, b.x, y);
                y = fmaf(a.y, b.y, y);
                y = fmaf(a.z, b.z, y);
                y = fmaf(a.w, b.w, y);
            }
            // the caller's units (the statistics and the fallback test use them)
            y = o == 0 ? fmaf(y, oscale.x, oshift.x) : fmaf(y, oscale.y, oshift.y);
            s_y[tid] = y;
        }
        __syncthreads();
        if (tid < QT * NOUT)
            for (int m = 0; m < nm; m++) {
                const float y = s_y[m * QT * NOUT + tid];
                sum += y;
                sq += y * y;
            }
    }
    if (tid < 64) {                                              // the first wave, whole, for the exchange below
        const int s = tid / NOUT;
        const bool live = tid < QT * NOUT && s < ns;
        const float mu = sum / (float)members;
        const float var = fmaxf(sq / (float)members - mu * mu, 0.0f);
        const int off = sqrtf(var) > thresh * fabsf(mu) ? 1 : 0;
        const int any = off | __shfl_xor(off, 1, 64);
        if (live) {
            mean[(int64_t)s0 * NOUT + tid] = mu;
            sd[(int64_t)s0 * NOUT + tid] = sqrtf(var);
            if (tid % NOUT == 0) fallback[s0 + s] = any ? 1 : 0;
        }
    }
}

}  // namespace

struct surr_ctx {
    int members = 0, max_n = 0;
    char *ws = nullptr;
    hipStream_t stream = nullptr;
    float *params = nullptr, *am = nullptr, *av = nullptr, *gsum = nullptr, *w2t = nullptr, *loss = nullptr;
    Acts act{};
    uint16_t *w2 = nullptr;
    int64_t adam_t = 0;
    std::string err;
};

namespace {

thread_local std::string g_surr_error;

constexpr size_t SALIGN = 256;
size_t salign(size_t v) { return (v + SALIGN - 1) / SALIGN * SALIGN; }

struct SLayout {
    size_t params, am, av, gsum, w2t, act[4], out[2], loss, w2, total;
    int rows;
};

SLayout surr_layout(int members, int max_n)
{
    SLayout L{};
    L.rows = std::min((max_n + GROUP - 1) / GROUP * GROUP, CHUNK);
    size_t o = 0;
    auto take = [&](size_t b) { size_t at = o; o += salign(std::max<size_t>(b, 1)); return at; };
    L.params = take((size_t)members * P * 4);
    L.am = take((size_t)members * P * 4);
    L.av = take((size_t)members * P * 4);
    L.gsum = take((size_t)members * P * 4);
    L.w2t = take((size_t)members * H * H * 4);
    for (auto &a : L.act) a = take((size_t)members * L.rows * H * 4);
    for (auto &a : L.out) a = take((size_t)members * L.rows * NOUT * 4);
    L.loss = take((size_t)members * 4);
    L.w2 = take((size_t)members * H * H * 2);
    L.total = o;
    return L;
}

lbm_status sfail(surr_ctx *c, lbm_status st, const std::string &msg)
{
    if (c) c->err = msg;
    else g_surr_error = msg;
    return st;
}

#define SHIPCHECK(c, call)                                                                       \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return sfail(c, LBM_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_));     \
    } while (0)

bool args_ok(int members, int hidden, int max_n)
{
    return members >= 1 && members <= 64 && hidden == H && max_n >= 1 && max_n <= (1 << 22);
}

// the BF16 copy of W2, or both copies, from the parameters
lbm_status derive_bf16(surr_ctx *c)
{
    const int64_t ne = (int64_t)c->members * H * H;
    hipLaunchKernelGGL(k_w2_bf16, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, c->stream, c->params,
                       c->members, c->w2);
    SHIPCHECK(c, hipGetLastError());
    return LBM_OK;
}

lbm_status derive_w2(surr_ctx *c)
{
    const int64_t ne = (int64_t)c->members * H * H;
    hipLaunchKernelGGL(k_w2_transpose, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, c->stream, c->params,
                       c->members, c->w2t);
    return derive_bf16(c);
}

// forward + backward over n samples; gradients summed (and copied to gout if
// given), Adam step if update
lbm_status pass(surr_ctx *c, const float *X, const float *Y, int n, float lr, bool update, float *gout)
{
    Adam ad{lr, 0.9f, 0.999f, 1e-8f, 1.0f, 1.0f};
    if (update) {
        c->adam_t++;
        ad.c1 = 1.0f - std::pow(ad.b1, (float)c->adam_t);
        ad.c2 = 1.0f - std::pow(ad.b2, (float)c->adam_t);
    }
    for (int base = 0; base < n; base += c->act.rows) {
        const int nr = std::min(c->act.rows, n - base);
        hipLaunchKernelGGL(k_fwd_bwd, dim3((unsigned)((nr + QT - 1) / QT), (unsigned)c->members), dim3(FT), 0,
                           c->stream, c->params, c->w2t, X, Y, n, base, c->act);
        hipLaunchKernelGGL(k_grad, dim3(G_UNITS, (unsigned)c->members), dim3(FT), 0, c->stream, c->params, c->w2t,
                           c->am, c->av, c->gsum, X, base, nr, c->act, base == 0 ? 1 : 0,
                           base + nr >= n ? 1 : 0, update ? 1 : 0, ad, gout, c->loss);
    }
    SHIPCHECK(c, hipGetLastError());
    return LBM_OK;
}

}  // namespace

extern "C" {

size_t surr_workspace_bytes(int members, int hidden, int max_n)
{
    if (!args_ok(members, hidden, max_n)) return 0;
    return surr_layout(members, max_n).total;
}

int surr_param_count(int hidden) { return hidden == H ? P : 0; }

lbm_status surr_create(int members, int hidden, int max_n, uint64_t seed, void *dev_ws, size_t ws_bytes,
                       void *hip_stream, surr_ctx **out)
{
    if (!out) return sfail(nullptr, LBM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!args_ok(members, hidden, max_n))
        return sfail(nullptr, LBM_EINVAL, "members must be 1..64, hidden 128, max_n 1..4194304");
    const SLayout L = surr_layout(members, max_n);
    if (!dev_ws || ((uintptr_t)dev_ws) % SALIGN) return sfail(nullptr, LBM_EINVAL, "workspace NULL or misaligned");
    if (ws_bytes < L.total) return sfail(nullptr, LBM_ENOMEM, "workspace too small");
    surr_ctx *c = new surr_ctx();
    c->members = members;
    c->max_n = max_n;
    c->ws = (char *)dev_ws;
    c->stream = (hipStream_t)hip_stream;
    c->params = (float *)(c->ws + L.params);
    c->am = (float *)(c->ws + L.am);
    c->av = (float *)(c->ws + L.av);
    c->gsum = (float *)(c->ws + L.gsum);
    c->w2t = (float *)(c->ws + L.w2t);
    c->act = {(float *)(c->ws + L.act[0]), (float *)(c->ws + L.act[1]), (float *)(c->ws + L.act[2]),
              (float *)(c->ws + L.act[3]), (float *)(c->ws + L.out[0]), (float *)(c->ws + L.out[1]), L.rows};
    c->loss = (float *)(c->ws + L.loss);
    c->w2 = (uint16_t *)(c->ws + L.w2);
    const int64_t np = (int64_t)members * P;
    hipLaunchKernelGGL(k_init, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, c->stream, c->params, c->am, c->av,
                       members, seed);
    if (hipGetLastError() != hipSuccess || derive_w2(c) != LBM_OK || hipStreamSynchronize(c->stream) != hipSuccess) {
        delete c;
        return sfail(nullptr, LBM_EDEVICE, "initialisation failed");
    }
    *out = c;
    return LBM_OK;
}

lbm_status surr_train(surr_ctx *c, const float *X, const float *Y, int n, int epochs, float lr, float *loss_host)
{
    if (!c || !X || !Y || n < 1 || n > c->max_n || epochs < 0 || !(lr > 0.0f))
        return sfail(c, LBM_EINVAL, "bad arguments to surr_train");
    for (int e = 0; e < epochs; e++) {
        const lbm_status st = pass(c, X, Y, n, lr, true, nullptr);
        if (st != LBM_OK) return st;
    }
    // the BF16 copy once per call: stored at every update it made 50 epochs 1.3% slower
    const lbm_status st = epochs > 0 ? derive_bf16(c) : LBM_OK;
    if (st != LBM_OK) return st;
    if (loss_host) {
        SHIPCHECK(c, hipMemcpyAsync(loss_host, c->loss, (size_t)c->members * 4, hipMemcpyDeviceToHost, c->stream));
        SHIPCHECK(c, hipStreamSynchronize(c->stream));
    }
    return LBM_OK;
}

lbm_status surr_forward_backward(surr_ctx *c, const float *X, const float *Y, int n, float *grads, float *loss)
{
    if (!c || !X || !Y || !grads || n < 1 || n > c->max_n)
        return sfail(c, LBM_EINVAL, "bad arguments to surr_forward_backward");
    const lbm_status st = pass(c, X, Y, n, 0.0f, false, grads);
    if (st != LBM_OK) return st;
    if (loss) SHIPCHECK(c, hipMemcpyAsync(loss, c->loss, (size_t)c->members * 4, hipMemcpyDeviceToDevice, c->stream));
    return LBM_OK;
}

lbm_status surr_predict(surr_ctx *c, const float *X, int n, float *mean, float *sd, uint8_t *fallback, float thresh,
                        const float *out_scale, const float *out_shift)
{
    if (!c || !X || !mean || !sd || !fallback || n < 1 || !(thresh >= 0.0f))
        return sfail(c, LBM_EINVAL, "bad arguments to surr_predict");
    const float2 osc = out_scale ? make_float2(out_scale[0], out_scale[1]) : make_float2(1.0f, 1.0f);
    const float2 osh = out_shift ? make_float2(out_shift[0], out_shift[1]) : make_float2(0.0f, 0.0f);
    if (!std::isfinite(osc.x) || !std::isfinite(osc.y) || !std::isfinite(osh.x) || !std::isfinite(osh.y))
        return sfail(c, LBM_EINVAL, "non-finite output scale or shift");
    // as few passes over the members as the LDS allows, of equal size
    const int passes = (c->members + MC_MAX - 1) / MC_MAX, mc = (c->members + passes - 1) / passes;
    hipLaunchKernelGGL(k_predict, dim3((unsigned)((n + QT - 1) / QT)), dim3(PT), predict_lds(mc), c->stream, c->params,
                       c->w2, c->members, mc, X, n, mean, sd, fallback, thresh, osc, osh);
    SHIPCHECK(c, hipGetLastError());
    return LBM_OK;
}

lbm_status surr_get_params(surr_ctx *c, float *host, size_t bytes)
{
    if (!c || !host || bytes != (size_t)c->members * P * 4) return sfail(c, LBM_EINVAL, "bad arguments to surr_get_params");
    SHIPCHECK(c, hipMemcpyAsync(host, c->params, bytes, hipMemcpyDeviceToHost, c->stream));
    SHIPCHECK(c, hipStreamSynchronize(c->stream));
    return LBM_OK;
}

lbm_status surr_set_params(surr_ctx *c, const float *host, size_t bytes)
{
    if (!c || !host || bytes != (size_t)c->members * P * 4) return sfail(c, LBM_EINVAL, "bad arguments to surr_set_params");
    SHIPCHECK(c, hipMemcpyAsync(c->params, host, bytes, hipMemcpyHostToDevice, c->stream));
    const lbm_status st = derive_w2(c);
    if (st != LBM_OK) return st;
    SHIPCHECK(c, hipStreamSynchronize(c->stream));
    return LBM_OK;
}

void surr_destroy(surr_ctx *c) { delete c; }

const char *surr_last_error(const surr_ctx *c) { return c ? c->err.c_str() : g_surr_error.c_str(); }

}  // extern "C"
