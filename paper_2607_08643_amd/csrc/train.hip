// Codec training (Section III-C; eq. codec_loss, eq. codec_loss_terms) for
// one stage codec: the linear encoder z = E x, the sphere map u = z / ||z||,
// sign binarisation with the straight-through estimator, the symmetric
// decoder x_hat = W2 relu(W1 q + b1) + b2, and the loss
//   L = L_rec + lambda_c L_com + lambda_e L_ent
// over a mini-batch of chunks gathered from a category's stacked layers
// (Section III-G, category-batched codec optimisation), then Adam.
//
// Parameters are one fp32 vector theta = E [b][d] | W1 [h][b] | b1 [h] |
// W2 [d][h] | b2 [d]. Every reduction runs in a fixed order that depends on n
// and on d, b and h alone, so a step gives the same bits on every run:
//   1. train_bits_kernel: per chunk z, u and the bit probabilities
//      s_ij = sigma(2 tau u_ij / sqrt(b)); per block the sums of s and of the
//      per-chunk entropies;
//   2. train_back_kernel: s_bar_j (the batch's mean bit probability, summed by
//      every block from the bits kernel's partials), then per chunk the
//      decoder's forward and backward and the straight-through gradient into
//      u and z, and, tile by tile of chunks in LDS, the block's partial
//      gradient of every parameter;
//   3. train_sum_kernel: the blocks' gradients and loss partials;
//   4. train_adam_kernel: one Adam step.
// A mini-batch is small (65,536 chunks are 1.6 MB), so what bounds a step is
// the number of dependent launches and the serial chains inside them, not
// bytes or arithmetic.
#include <algorithm>

#include "bsq_internal.h"

namespace bsq {
namespace {

constexpr int TB = 256;        // threads per block in the per-chunk kernels
// Blocks of the bits and the back kernel at most; each walks the batch in
// steps of the whole grid. 1,024 blocks are four waves per SIMD. Every back
// block reads every bits block's partial sums (at most 64 KiB), and the sum
// kernel every back block's gradient, so more blocks cost more than they hide.
constexpr int64_t BITS_BLOCKS = 1024, BACK_BLOCKS = 768;

struct TrainArgs {
    const void *x;             // chunks [n_total][d], fp32 or bf16
    int x_bf16;
    const int64_t *idx;        // batch chunk indices [n], or null (chunks 0 .. n-1)
    int64_t n, n_total;
    int32_t *err;              // device error word (an index out of range), or null
    int d, b, h;
    const float *theta;
    float lambda_c, lambda_e, gamma, tau, cscale;
    float *s_part;             // [nbits][b] sums of s per block
    float *h_part;             // [nbits] sums of per-chunk entropies per block
    float *sbar;               // [b] (written by back block 0)
    float *l_part;             // [nback][2] sums of ||x_hat - x||^2 and ||u - q||^2 per block
    float *g_part;             // [nback][P]
    float *grad;               // [P]
    float *loss;               // [4]: L, L_rec, L_com, L_ent
    int64_t P, nbits, nback;
    int vec;                   // chunks 16-byte aligned: whole 16-byte loads
};

__device__ __forceinline__ float entropy2(float s) { return -(s * logf(s) + (1.0f - s) * logf(1.0f - s)); }

// z = E x (fmaf chain from +0, j in order), ||z||, u, and the code (bit m =
// z_m >= 0, the decision the oracle takes in the same chain)
template <int D, int B>
__device__ __forceinline__ void encode_chunk(const TrainArgs &a, const float *E, const float (&x)[D], float (&u)[B],
                                             float &nz, uint32_t &code)
{
    float z[B];
    float ss = 0.0f;
    code = 0;
#pragma unroll
    for (int m = 0; m < B; ++m) {
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) acc = __builtin_fmaf(E[m * D + j], x[j], acc);
        z[m] = acc;
        code |= (acc >= 0.0f ? 1u : 0u) << m;
        ss = __builtin_fmaf(acc, acc, ss);
    }
    nz = __builtin_sqrtf(ss);
    const float inv = (nz > 0.0f) ? 1.0f / nz : 0.0f;
#pragma unroll
    for (int m = 0; m < B; ++m) u[m] = z[m] * inv;
}

template <int D>
__device__ __forceinline__ void load_x_chunk(const TrainArgs &a, int64_t i, float (&x)[D])
{
    int64_t c = a.idx ? a.idx[i] : i;
    if (c < 0 || c >= a.n_total) {  // reported, and read as chunk 0
        if (a.err) atomicOr(a.err, int32_t(BSQ_DEVERR_BAD_SET));
        c = 0;
    }
    if (a.x_bf16) {
        const uint16_t *p = static_cast<const uint16_t *>(a.x) + c * D;
        if (a.vec) {
#pragma unroll
            for (int v = 0; v < D / 8; ++v) {
                const uint4 w = reinterpret_cast<const uint4 *>(p)[v];
                const uint32_t h[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[8 * v + 2 * e] = __uint_as_float(h[e] << 16);
                    x[8 * v + 2 * e + 1] = __uint_as_float(h[e] & 0xffff0000u);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < D; ++j) x[j] = bf16_to_f32(p[j]);
        }
    } else {
        const float *p = static_cast<const float *>(a.x) + c * D;
        if (a.vec) {
#pragma unroll
            for (int v = 0; v < D / 4; ++v) {
                const float4 w = reinterpret_cast<const float4 *>(p)[v];
                x[4 * v] = w.x;
                x[4 * v + 1] = w.y;
                x[4 * v + 2] = w.z;
                x[4 * v + 3] = w.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < D; ++j) x[j] = p[j];
        }
    }
}

// Block sums of N values per thread: a fixed tree over each wave's lanes, then
// the waves in order. Every thread gets every sum. `red` holds (TB / 64) N
// floats and is free again on return.
template <int N>
__device__ __forceinline__ void block_sums(float (&v)[N], float *red)
{
    const int t = threadIdx.x;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int m = 0; m < N; ++m) v[m] += __shfl_xor(v[m], o, 64);
    if ((t & 63) == 0) {
#pragma unroll
        for (int m = 0; m < N; ++m) red[(t >> 6) * N + m] = v[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < N; ++m) {
        float s = red[m];
        for (int w = 1; w < TB / 64; ++w) s += red[w * N + m];
        v[m] = s;
    }
    __syncthreads();
}

template <int D, int B>
__global__ __launch_bounds__(TB) void train_bits_kernel(const TrainArgs a)
{
    __shared__ float s_E[B * D];
    __shared__ float red[TB / 64 * (B + 1)];
    for (int e = threadIdx.x; e < B * D; e += TB) s_E[e] = a.theta[e];
    __syncthreads();
    float s[B + 1];  // the bit probabilities, then the entropy
#pragma unroll
    for (int m = 0; m <= B; ++m) s[m] = 0.0f;
    for (int64_t i = int64_t(blockIdx.x) * TB + threadIdx.x; i < a.n; i += a.nbits * TB) {
        float x[D], u[B], nz;
        uint32_t code;
        load_x_chunk<D>(a, i, x);
        encode_chunk<D, B>(a, s_E, x, u, nz, code);
        const float k = 2.0f * a.tau * a.cscale;
        float hsum = 0.0f;
#pragma unroll
        for (int m = 0; m < B; ++m) {
            const float p = 1.0f / (1.0f + expf(-k * u[m]));
            s[m] += p;
            hsum += entropy2(p);
        }
        s[B] += hsum;
    }
    block_sums<B + 1>(s, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int m = 0; m < B; ++m) a.s_part[int64_t(blockIdx.x) * B + m] = s[m];
        a.h_part[blockIdx.x] = s[B];
    }
}

// The two record fields whose product is parameter p's term (-1: the factor
// 1), from the packed layout of theta. A chunk's record is
//   [dx_hat (D) | a (h) | dpre (h) | q (B) | dz (B) | x (D)].
__device__ __forceinline__ void param_factors(int D, int B, int h, int p, int &o1, int &o2)
{
    const int oa = D, odp = D + h, oq = D + 2 * h, odz = D + 2 * h + B, ox = D + 2 * h + 2 * B;
    if (p < B * D) {                       // E[m][j]: dz_m x_j
        o1 = odz + p / D;
        o2 = ox + p % D;
        return;
    }
    p -= B * D;
    if (p < h * B) {                       // W1[k][j]: dpre_k q_j
        o1 = odp + p / B;
        o2 = oq + p % B;
        return;
    }
    p -= h * B;
    if (p < h) {                           // b1[k]: dpre_k
        o1 = odp + p;
        o2 = -1;
        return;
    }
    p -= h;
    if (p < D * h) {                       // W2[m][k]: dx_hat_m a_k
        o1 = p / h;
        o2 = oa + p % h;
        return;
    }
    p -= D * h;                            // b2[m]: dx_hat_m
    o1 = p;
    o2 = -1;
}

// Chunks per LDS tile of the back kernel, and the tile's row pitch in floats:
// a field's chunks are contiguous (each thread writes its own column), and
// four floats of padding put the 16-byte words of neighbouring fields in
// different banks for the parameter pass.
constexpr int back_pitch(int tc) { return tc + 4; }
// LDS floats: theta, the block's gradient, the tile
inline int64_t back_lds_floats(int64_t P, int64_t R, int tc) { return 2 * ((P + 3) & ~int64_t(3)) + R * back_pitch(tc); }
constexpr int64_t BACK_LDS_FLOATS = 15872;  // 62 KiB, beside the static 2 KiB
// the largest tile that fits: every (d, b, h) fits at 32 chunks
// (the largest, 16, 16, 64: 192 fields and 2,384 parameters, 45.6 KiB)
inline int back_tile(int64_t P, int64_t R)
{
    int tc = TB;
    while (tc > 32 && back_lds_floats(P, R, tc) > BACK_LDS_FLOATS) tc >>= 1;
    return tc;
}

// Per tile of TC chunks: the first TC threads compute one chunk's decoder
// forward and backward and the straight-through gradient into z, and leave its
// record in LDS (field-major); then every thread owns the parameters t, t +
// 256, ... and adds the tile's products of their two fields, chunks in order,
// 16-byte reads. At 65,536 chunks and d = b = h = 8 this kernel takes 11.6 us
// and the whole step with Adam 23 us. With the records written to memory and
// read back by a kernel of one thread per parameter and chunk group, the
// backward, parameter and sum kernels took 18.5 + 44 + 42 us of 145 us; a
// 128-chunk tile (twice the blocks) measured the same.
template <int D, int B, int TC>
__global__ __launch_bounds__(TB) void train_back_kernel(const TrainArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float s_mem[];
    __shared__ float red[TB / 64 * 2];
    __shared__ float s_bar[16], s_barp[TB];
    const int t = threadIdx.x, h = a.h, P = int(a.P), P4 = (P + 3) & ~3;
    constexpr int LD = back_pitch(TC);
    float *s_theta = s_mem, *s_acc = s_mem + P4, *rec = s_mem + 2 * P4;
    for (int e = t; e < P; e += TB) {
        s_theta[e] = a.theta[e];
        s_acc[e] = 0.0f;
    }
    {  // s_bar_j: TB / B threads per bit over the bits kernel's blocks, then in order
        constexpr int G = TB / B;
        const int m = t % B, g = t / B;
        float acc = 0.0f;
#pragma unroll 4
        for (int64_t k = g; k < a.nbits; k += G) acc += a.s_part[k * B + m];
        s_barp[t] = acc;
        __syncthreads();
        if (t < B) {
            float s = s_barp[t];
            for (int w = 1; w < G; ++w) s += s_barp[w * B + t];
            s_bar[t] = s / float(a.n);
            if (blockIdx.x == 0) a.sbar[t] = s_bar[t];
        }
        __syncthreads();
    }
    const float *E = s_theta, *W1 = E + B * D, *b1 = W1 + h * B, *W2 = b1 + h, *b2 = W2 + D * h;
    const float inv_n = 1.0f / float(a.n);
    const float k2 = 2.0f * a.tau * a.cscale;
    float loss[2] = {0.0f, 0.0f};  // sums of ||x_hat - x||^2 and ||u - q||^2
    const int64_t ntile = (a.n + TC - 1) / TC;
    for (int64_t tile = blockIdx.x; tile < ntile; tile += a.nback) {
        const int64_t i = tile * TC + t;
        const int live = int((a.n - tile * TC < TC) ? a.n - tile * TC : TC);
        if (t < TC && t < live) {
            float *r = rec + t;  // field f at r[f * LD]
            float x[D], u[B], nz;
            uint32_t code;
            load_x_chunk<D>(a, i, x);
            encode_chunk<D, B>(a, E, x, u, nz, code);
            float q[B];
#pragma unroll
            for (int m = 0; m < B; ++m) q[m] = ((code >> m) & 1u) ? a.cscale : -a.cscale;
            // decoder forward: pre_k = fmaf chain from b1_k over j (the decision
            // chain of the oracle), a = relu(pre), x_hat = W2 a + b2 (k in order)
            float dxh[D], du[B];
#pragma unroll
            for (int mm = 0; mm < D; ++mm) dxh[mm] = b2[mm];
            for (int k = 0; k < h; ++k) {
                float acc = b1[k];
#pragma unroll
                for (int j = 0; j < B; ++j) acc = __builtin_fmaf(W1[k * B + j], q[j], acc);
                acc = (acc > 0.0f) ? acc : 0.0f;
                r[(D + k) * LD] = acc;
#pragma unroll
                for (int mm = 0; mm < D; ++mm) dxh[mm] = __builtin_fmaf(W2[mm * h + k], acc, dxh[mm]);
            }
            float lrec = 0.0f, lcom = 0.0f;
#pragma unroll
            for (int mm = 0; mm < D; ++mm) {
                const float df = dxh[mm] - x[mm];
                lrec = __builtin_fmaf(df, df, lrec);
                dxh[mm] = 2.0f * df * inv_n;
            }
#pragma unroll
            for (int j = 0; j < B; ++j) du[j] = 0.0f;
            for (int k = 0; k < h; ++k) {
                float g = 0.0f;
#pragma unroll
                for (int mm = 0; mm < D; ++mm) g = __builtin_fmaf(W2[mm * h + k], dxh[mm], g);
                g = (r[(D + k) * LD] > 0.0f) ? g : 0.0f;
                r[(D + h + k) * LD] = g;  // dpre
#pragma unroll
                for (int j = 0; j < B; ++j) du[j] = __builtin_fmaf(W1[k * B + j], g, du[j]);
            }
            // commitment and entropy terms into u
            float udu = 0.0f;
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const float dq = u[j] - q[j];
                lcom = __builtin_fmaf(dq, dq, lcom);
                const float tt = k2 * u[j];
                const float s = 1.0f / (1.0f + expf(-tt));
                const float sd = s * (1.0f - s);
                const float dt = (-tt * sd - a.gamma * logf((1.0f - s_bar[j]) / s_bar[j]) * sd) * inv_n;
                du[j] += a.lambda_c * 2.0f * dq * inv_n + a.lambda_e * dt * k2;
                udu = __builtin_fmaf(u[j], du[j], udu);
            }
            const float inz = (nz > 0.0f) ? 1.0f / nz : 0.0f;
#pragma unroll
            for (int mm = 0; mm < D; ++mm) {
                r[mm * LD] = dxh[mm];
                r[(D + 2 * h + B + B + mm) * LD] = x[mm];
            }
#pragma unroll
            for (int j = 0; j < B; ++j) {
                r[(D + 2 * h + j) * LD] = q[j];
                r[(D + 2 * h + B + j) * LD] = (du[j] - u[j] * udu) * inz;
            }
            loss[0] += lrec;
            loss[1] += lcom;
        }
        if (t < TC && t >= live)  // the ragged last tile: empty chunks add nothing
            for (int f = 0; f < int(2 * (D + B + h)); ++f) rec[f * LD + t] = 0.0f;
        __syncthreads();
        for (int p = t; p < P; p += TB) {
            int o1, o2;
            param_factors(D, B, h, p, o1, o2);
            const float4 *f1 = reinterpret_cast<const float4 *>(rec + o1 * LD);
            float acc = 0.0f;
            if (o2 < 0) {
#pragma unroll 8
                for (int c = 0; c < TC / 4; ++c) {
                    const float4 v = f1[c];
                    acc = (((acc + v.x) + v.y) + v.z) + v.w;
                }
            } else {
                const float4 *f2 = reinterpret_cast<const float4 *>(rec + o2 * LD);
#pragma unroll 8
                for (int c = 0; c < TC / 4; ++c) {
                    const float4 v = f1[c], w = f2[c];
                    acc = __builtin_fmaf(v.x, w.x, acc);
                    acc = __builtin_fmaf(v.y, w.y, acc);
                    acc = __builtin_fmaf(v.z, w.z, acc);
                    acc = __builtin_fmaf(v.w, w.w, acc);
                }
            }
            s_acc[p] += acc;
        }
        __syncthreads();  // the tile's records are free again
    }
    for (int p = t; p < P; p += TB) a.g_part[int64_t(blockIdx.x) * P + p] = s_acc[p];
    block_sums<2>(loss, red);
    if (t == 0) {
        a.l_part[int64_t(blockIdx.x) * 2] = loss[0];
        a.l_part[int64_t(blockIdx.x) * 2 + 1] = loss[1];
    }
}

// Blocks 0 .. gridDim - 2: 16 parameters each, 16 threads per parameter over
// the back kernel's blocks (a thread's loads are independent), then those in
// order. The last block: the loss.
__global__ __launch_bounds__(TB) void train_sum_kernel(const TrainArgs a)
{
    __shared__ float s_red[TB];
    __shared__ float red[TB / 64 * 2];
    const int t = threadIdx.x;
    if (blockIdx.x + 1 < gridDim.x) {
        const int64_t p = int64_t(blockIdx.x) * 16 + (t & 15);
        const int g = t >> 4;
        float acc = 0.0f;
        if (p < a.P) {
#pragma unroll 8
            for (int64_t k = g; k < a.nback; k += 16) acc += a.g_part[k * a.P + p];
        }
        s_red[t] = acc;
        __syncthreads();
        if (t < 16 && p < a.P) {
            float s = s_red[t];
#pragma unroll
            for (int w = 1; w < 16; ++w) s += s_red[16 * w + t];
            a.grad[p] = s;
        }
        return;
    }
    // The entropy partials, up to 1,024, are added one after the other in fp32,
    // which keeps the reported loss what it was when every block had its own
    // partial. It is not the most exact order: L_ent is the small difference of
    // two entropies near b ln 2, and the chain's rounding shows in it (65,536
    // chunks, b = 8: up to 9e-5 of L_ent from its 64-bit value; 131,072 chunks,
    // b = 16: 1e-3, 5e-6 to 2e-5 of the loss; in a tree of the same partials
    // 3e-5 and less). The gradient does not depend on it.
    __shared__ float s_h[BITS_BLOCKS];
    float v[2] = {0.0f, 0.0f};  // reconstruction, commitment
    for (int64_t k = t; k < a.nback; k += TB) {
        v[0] += a.l_part[2 * k];
        v[1] += a.l_part[2 * k + 1];
    }
    for (int64_t k = t; k < a.nbits; k += TB) s_h[k] = a.h_part[k];
    block_sums<2>(v, red);  // (its barriers also cover s_h)
    if (t == 0) {
        float he = 0.0f;
#pragma unroll 16
        for (int k = 0; k < int(a.nbits); ++k) he += s_h[k];
        float bar_ent = 0.0f;
        for (int j = 0; j < a.b; ++j) bar_ent += entropy2(a.sbar[j]);
        const float inv_n = 1.0f / float(a.n);
        const float L_rec = v[0] * inv_n, L_com = v[1] * inv_n, L_ent = he * inv_n - a.gamma * bar_ent;
        a.loss[0] = L_rec + a.lambda_c * L_com + a.lambda_e * L_ent;
        a.loss[1] = L_rec;
        a.loss[2] = L_com;
        a.loss[3] = L_ent;
    }
}

struct AdamArgs {
    float *theta, *m, *v;
    const float *grad;
    int64_t P;
    float lr, beta1, beta2, eps, bc1, bc2;  // bc = 1 - beta^step
};

__global__ __launch_bounds__(TB) void train_adam_kernel(const AdamArgs a)
{
    const int64_t p = int64_t(blockIdx.x) * TB + threadIdx.x;
    if (p >= a.P) return;
    const float g = a.grad[p];
    const float m = a.beta1 * a.m[p] + (1.0f - a.beta1) * g;
    const float v = a.beta2 * a.v[p] + (1.0f - a.beta2) * g * g;
    a.m[p] = m;
    a.v[p] = v;
    a.theta[p] = a.theta[p] - a.lr * (m / a.bc1) / (__builtin_sqrtf(v / a.bc2) + a.eps);
}

template <int D, int B>
hipError_t launch_train_t(const TrainArgs &a, int tc, size_t lds, hipStream_t st)
{
    hipLaunchKernelGGL((train_bits_kernel<D, B>), dim3(unsigned(a.nbits)), dim3(TB), 0, st, a);
    const dim3 grid(unsigned(a.nback));
    switch (tc) {
    case 256: hipLaunchKernelGGL((train_back_kernel<D, B, 256>), grid, dim3(TB), lds, st, a); break;
    case 128: hipLaunchKernelGGL((train_back_kernel<D, B, 128>), grid, dim3(TB), lds, st, a); break;
    case 64: hipLaunchKernelGGL((train_back_kernel<D, B, 64>), grid, dim3(TB), lds, st, a); break;
    default: hipLaunchKernelGGL((train_back_kernel<D, B, 32>), grid, dim3(TB), lds, st, a); break;
    }
    hipLaunchKernelGGL(train_sum_kernel, dim3(unsigned((a.P + 15) / 16 + 1)), dim3(TB), 0, st, a);
    return hipGetLastError();
}

// Blocks of the two per-chunk kernels and the back kernel's tile for n chunks.
struct TrainPlan {
    int tc;
    int64_t nbits, nback;
};

TrainPlan train_plan(const bsq_config &cfg, int64_t n)
{
    TrainPlan p{};
    p.tc = back_tile(train_param_count(cfg), train_record_floats(cfg));
    p.nbits = std::min<int64_t>((n + TB - 1) / TB, BITS_BLOCKS);
    p.nback = std::min<int64_t>((n + p.tc - 1) / p.tc, BACK_BLOCKS);
    return p;
}

}  // namespace

int64_t train_param_count(const bsq_config &cfg)
{
    const int64_t d = cfg.d, b = cfg.b, h = cfg.hidden;
    return b * d + h * b + h + d * h + d;
}

int64_t train_record_floats(const bsq_config &cfg) { return 2 * cfg.d + 2 * int64_t(cfg.hidden) + 2 * cfg.b; }

// The stated size (what a caller allocates, and the least that is accepted)
// covers one record per chunk and a part sum per parameter of 512 groups. The
// kernels keep the records in LDS and use less than that for every n: where
// the back kernel has more than 512 blocks there are more than 512 x 32
// chunks, whose records outweigh the further part sums.
size_t train_ws_bytes(const bsq_config &cfg, int64_t n)
{
    const int64_t nblk = (n + TB - 1) / TB, P = train_param_count(cfg);
    const size_t stated = align256(size_t(nblk) * cfg.b * 4) + align256(size_t(nblk) * 4) + 256 + 256 +
                          align256(size_t(nblk) * 8) + align256(size_t(n) * train_record_floats(cfg) * 4) +
                          align256(size_t(512) * P * 4);
    const TrainPlan p = train_plan(cfg, n);
    const size_t used = align256(size_t(p.nbits) * cfg.b * 4) + align256(size_t(p.nbits) * 4) + 256 +
                        align256(size_t(p.nback) * 8) + align256(size_t(p.nback) * P * 4);
    return std::max(stated, used);
}

hipError_t launch_train_grad(const bsq_config &cfg, const bsq_train_hparams &hp, const void *x, int x_dtype,
                             int64_t n_total, const int64_t *idx, int64_t n, const float *theta, float *grad,
                             float *loss, int32_t *err, void *ws, hipStream_t st)
{
    TrainArgs a{};
    a.x = x;
    a.x_bf16 = (x_dtype == BSQ_BF16);
    a.idx = idx;
    a.n = n;
    a.n_total = n_total;
    a.err = err;
    a.d = cfg.d;
    a.b = cfg.b;
    a.h = cfg.hidden;
    a.theta = theta;
    a.lambda_c = hp.lambda_c;
    a.lambda_e = hp.lambda_e;
    a.gamma = hp.gamma;
    a.tau = hp.tau;
    a.cscale = float(1.0 / __builtin_sqrt(double(cfg.b)));
    const TrainPlan p = train_plan(cfg, n);
    a.nbits = p.nbits;
    a.nback = p.nback;
    a.P = train_param_count(cfg);
    a.vec = (reinterpret_cast<uintptr_t>(x) % 16 == 0);  // (a chunk is a multiple of 16 bytes)
    char *w = static_cast<char *>(ws);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = w + off;
        off += align256(bytes);
        return p;
    };
    a.s_part = reinterpret_cast<float *>(take(size_t(a.nbits) * cfg.b * 4));
    a.h_part = reinterpret_cast<float *>(take(size_t(a.nbits) * 4));
    a.sbar = reinterpret_cast<float *>(take(64));
    a.l_part = reinterpret_cast<float *>(take(size_t(a.nback) * 8));
    a.g_part = reinterpret_cast<float *>(take(size_t(a.nback) * a.P * 4));
    a.grad = grad;
    a.loss = loss;
    const size_t lds = size_t(back_lds_floats(a.P, train_record_floats(cfg), p.tc)) * 4;
    if (cfg.d == 8) return (cfg.b == 8) ? launch_train_t<8, 8>(a, p.tc, lds, st) : launch_train_t<8, 16>(a, p.tc, lds, st);
    return (cfg.b == 8) ? launch_train_t<16, 8>(a, p.tc, lds, st) : launch_train_t<16, 16>(a, p.tc, lds, st);
}

hipError_t launch_train_adam(const bsq_config &cfg, const bsq_train_hparams &hp, int step, float *theta,
                             const float *grad, float *m, float *v, hipStream_t st)
{
    AdamArgs a{};
    a.theta = theta;
    a.m = m;
    a.v = v;
    a.grad = grad;
    a.P = train_param_count(cfg);
    a.lr = hp.lr;
    a.beta1 = hp.beta1;
    a.beta2 = hp.beta2;
    a.eps = hp.eps;
    a.bc1 = float(1.0 - __builtin_pow(double(hp.beta1), double(step)));
    a.bc2 = float(1.0 - __builtin_pow(double(hp.beta2), double(step)));
    hipLaunchKernelGGL(train_adam_kernel, dim3(unsigned((a.P + TB - 1) / TB)), dim3(TB), 0, st, a);
    return hipGetLastError();
}

}  // namespace bsq
