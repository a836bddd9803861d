// Decode-once GEMM for many tokens: Y = X W_hat^T + (X A^T) B^T.
//
// gemm.hip decodes a block's weights again for every token tile, which the
// matrix cores wait for once there are several tiles. Here the weights are
// decoded once per call into bf16 in the workspace (in slabs of rows, which
// bound it), and a plain MFMA product reads them:
//
//   dense_operands  X -> Xe: X~ (protected columns zero), the gathered
//                   protected activations and T = X A^T in three bf16 parts;
//                   planes -> We: the decoded weights, the protected payload
//                   in bf16 and the rows of B, at the same positions of K;
//   dense_gemm      Y = Xe We^T.
//
// So the protected term and the adapter are further inputs of one product,
// with the values gemm.hip gives them: each weight the fp32 fmaf chain over
// fp16 gains and fp16 table entries rounded to bf16, T = hi + mid + lo exact
// to 2^-24, fp32 accumulation.
//
// Both operands are stored as units of 16 rows x 32 inputs in MFMA fragment
// order: 16 bytes per lane, lane l holding the 8 inputs of group l / 16 of
// row l % 16, so that a unit is one 1 KiB DMA to LDS and one conflict-free
// 16-byte LDS read per lane. Unit (row group, u) of KU units per row group.
// Group g of unit u holds inputs 32 u + 8 g .. + 8; after the 128-input steps
// come kp32 / 32 units of protected positions, two of the adapter (hi | mid,
// lo | 0), and a zero unit where KU would be odd.
#include <algorithm>
#include <atomic>

#include "gemm_common.h"

namespace bsq {
namespace {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

// Bytes of decoded weights per slab, which bound the workspace. Slabs of 128
// MiB (to stay in the last-level cache) left half the chip idle: 8192 x 8192
// at 2000 tokens took 362 us in two of them, 257 in one.
constexpr int64_t DENSE_SLAB_BYTES = int64_t(512) << 20;

// Decoded weights up to this size come from the last-level cache (256 MiB)
// when the product reads them.
constexpr int64_t DENSE_CACHED_BYTES = int64_t(224) << 20;

struct DenseArgs {
    const void *codes[BSQ_MAX_STAGES];
    const uint16_t *gains[BSQ_MAX_STAGES];
    const uint16_t *tabh[BSQ_MAX_STAGES];  // fp16 decoder tables [2^b][d]
    const int8_t *q8;
    const float *scale;
    const int32_t *idx;
    const uint32_t *bits;
    const uint16_t *X, *A, *B;
    float *T;        // X A^T [Mp][16] (read by the protected-row pass)
    float *Tp;       // its partial sums [nxseg][Mp][16]
    uint16_t *Xe;    // [Mp / 16][KU][64][8]
    uint16_t *We;    // [slab rows / 16][KU][64][8]
    void *Y;
    int64_t M, ldx, d_in, d_out, pitch, k, kp32, ldy;
    int64_t row0, rows;      // this slab
    int64_t ksteps, KU;      // 128-input steps, units per row group (even)
    int64_t Mp;              // tokens padded to whole blocks
    int mtiles, ntiles, nxseg;
    int ksplit;              // blocks per tile along K
    float *part;             // their fp32 tiles [ksplit][Mp][np] (ksplit > 1)
    int64_t np;
    int nf;                  // row groups of We per wave of the product
    int rank, pfmt, y_bf16, y_vec;
};

// ---------------------------------------------------------------------------
// Operands: one launch whose first workgroups write Xe and whose others write
// We, so that both run together (at 2000 tokens and 12288 x 4096 they took
// 16 and 23 us one after the other).
//
// Activations: a workgroup takes 16 tokens and 512 inputs (a wave one
// 128-input step: with the whole row in one workgroup, few compute units
// carried all of X and A), and one more per 16 tokens the gathered protected
// activations. A wave's loads are the units to store (masked) and, unmasked,
// the operand of T = X A^T on the matrix cores; dense_adapter adds the partial
// T in order of K.
// ---------------------------------------------------------------------------
constexpr int DO_WAVES = 4;

__device__ __forceinline__ void dense_tokens(const DenseArgs &a, int64_t tg, int seg, f32x4_t *s_t)
{
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t m = tg * 16 + r16;
    const bool live = m < a.M;
    const uint16_t *xr = a.X + (live ? m : a.M - 1) * a.ldx;
    u32x4_t *xe = reinterpret_cast<u32x4_t *>(a.Xe) + tg * a.KU * 64 + lane;
    const u32x4_t zero = u32x4_t{0u, 0u, 0u, 0u};
    if (seg == a.nxseg) {
        for (int64_t u = wave; u < a.kp32 / 32; u += DO_WAVES) {
            int32_t j[8];
            uint32_t v[4] = {0u, 0u, 0u, 0u};
            const int64_t p0 = 32 * u + 8 * g;
#pragma unroll
            for (int e = 0; e < 8; ++e) j[e] = a.idx[(p0 + e < a.k) ? p0 + e : a.k - 1];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in = live && p0 + e < a.k && j[e] >= 0 && j[e] < a.d_in;
                const uint32_t x = xr[in ? j[e] : 0];
                v[e >> 1] |= (in ? x : 0u) << (16 * (e & 1));
            }
            xe[(4 * a.ksteps + u) * 64] = u32x4_t{v[0], v[1], v[2], v[3]};
        }
        // zero unit where the used ones are odd in number
        const int64_t used = 4 * a.ksteps + a.kp32 / 32 + (a.rank > 0 ? 2 : 0);
        if (wave == 0 && used < a.KU) xe[used * 64] = zero;
        return;
    }
    const bool lora = a.rank > 0;
    const int64_t ks = int64_t(seg) * DO_WAVES + wave;
    f32x4_t acc = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    if (ks < a.ksteps) {
        // all loads in flight together (addresses clamped: a load under a
        // condition is waited for at once)
        u32x4_t xv[4], av[4];
        const int64_t c0 = ks * BK + 8 * g;
        const uint16_t *ar = a.A + int64_t(r16 < a.rank ? r16 : 0) * a.d_in;
        // rows of A are 16-byte aligned with its base (d_in is a multiple of 8)
        const bool avec = (reinterpret_cast<uintptr_t>(a.A) & 15) == 0;
        // bitmap word q covers unit q of the step (its words cover whole steps)
        uint32_t pm[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = (c0 + 32 * q < a.d_in) ? c0 + 32 * q : 0;
            pm[q] = (a.k > 0 && a.bits) ? a.bits[c >> 5] >> (8 * g) : 0u;
            xv[q] = *reinterpret_cast<const u32x4_t *>(xr + c);
            av[q] = zero;
            if (!lora) continue;
            if (avec) {
                av[q] = *reinterpret_cast<const u32x4_t *>(ar + c);
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) av[q][h] = uint32_t(ar[c + 2 * h]) | (uint32_t(ar[c + 2 * h + 1]) << 16);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = c0 + 32 * q < a.d_in;
            u32x4_t x = (live && in) ? xv[q] : zero;
            if (lora) {
                const u32x4_t w = (r16 < a.rank && in) ? av[q] : zero;
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, w),
                                                               acc, 0, 0, 0);
            }
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const uint32_t two = pm[q] >> (2 * h);
                x[h] &= ((two & 1u) ? 0u : 0xffffu) | ((two & 2u) ? 0u : 0xffff0000u);
            }
            xe[(4 * ks + q) * 64] = x;
        }
    }
    if (!lora) return;
    s_t[64 * wave + lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4_t sum = s_t[lane];
#pragma unroll
    for (int w = 1; w < DO_WAVES; ++w) sum += s_t[64 * w + lane];
    // partial T[16 tg + 4 g + r][r16] of this K segment
    float *tp = a.Tp + (int64_t(seg) * a.Mp + tg * 16) * BSQ_MAX_LORA_RANK;
#pragma unroll
    for (int r = 0; r < 4; ++r) tp[(4 * g + r) * BSQ_MAX_LORA_RANK + r16] = sum[r];
}

// The adapter's units of Xe: T summed over the K segments in order (zero past
// the rank), stored, and split exactly into three bf16 parts. A wave per 16
// tokens; lane (g, r16) holds T[r16][8 (g % 2) .. + 8].
__global__ __launch_bounds__(64) void dense_adapter(const DenseArgs a)
{
    const int lane = threadIdx.x, g = lane >> 4, r16 = lane & 15, q0 = 8 * (g & 1);
    const int64_t m = int64_t(blockIdx.x) * 16 + r16;
    const float *tp = a.Tp + m * BSQ_MAX_LORA_RANK + q0;
    f32x4_t t0 = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, t1 = t0;
#pragma unroll 4
    for (int s = 0; s < a.nxseg; ++s) {
        const f32x4_t *p = reinterpret_cast<const f32x4_t *>(tp + int64_t(s) * a.Mp * BSQ_MAX_LORA_RANK);
        t0 += p[0];
        t1 += p[1];
    }
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (q0 + e < a.rank) ? (e < 4 ? t0[e & 3] : t1[e & 3]) : 0.0f;
    if (g < 2) {
        float4 *tb = reinterpret_cast<float4 *>(a.T + m * BSQ_MAX_LORA_RANK + q0);
        tb[0] = make_float4(x[0], x[1], x[2], x[3]);
        tb[1] = make_float4(x[4], x[5], x[6], x[7]);
    }
    uint32_t hi[4], mid[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        hi[e] = pack_bf16x2(x[2 * e], x[2 * e + 1]);
        const float r0 = x[2 * e] - __uint_as_float(hi[e] << 16), r1 = x[2 * e + 1] - __uint_as_float(hi[e] & 0xffff0000u);
        mid[e] = pack_bf16x2(r0, r1);
        lo[e] = pack_bf16x2(r0 - __uint_as_float(mid[e] << 16), r1 - __uint_as_float(mid[e] & 0xffff0000u));
    }
    u32x4_t *xe = reinterpret_cast<u32x4_t *>(a.Xe) + (int64_t(blockIdx.x) * a.KU + 4 * a.ksteps + a.kp32 / 32) * 64 + lane;
    const uint32_t *p1 = (g < 2) ? hi : mid;
    xe[0] = u32x4_t{p1[0], p1[1], p1[2], p1[3]};
    xe[64] = (g < 2) ? u32x4_t{lo[0], lo[1], lo[2], lo[3]} : u32x4_t{0u, 0u, 0u, 0u};
}

// Weights: a workgroup decodes DW_STEPS 128-input steps of four row groups, a
// wave one group's; the last workgroup of the four groups writes their
// protected and adapter units. Bound by the write of 2 bytes per weight
// (d = 8) and by the table gathers from L2 (d = 16).
//
// Rows of a group: the nf groups that a wave of the product owns interleave
// their 16 nf rows in runs of four, so that a lane's accumulators are 4 nf
// consecutive outputs of a token.
constexpr int DW_STEPS = 4;

template <int D, int S>
__global__ __launch_bounds__(64 * DO_WAVES) __attribute__((amdgpu_waves_per_eu(S <= 2 ? 6 : 4))) void dense_operands(const DenseArgs a, int ntok)
{
    constexpr int TABU = (D == 8) ? S * 256 : 0;
    __shared__ u32x4_t s_mem[TABU > 64 * DO_WAVES ? TABU : 64 * DO_WAVES];
    if (int(blockIdx.x) < ntok) {
        const int per = a.nxseg + 1, tg = int(blockIdx.x) / per;
        dense_tokens(a, tg, int(blockIdx.x) - tg * per, reinterpret_cast<f32x4_t *>(s_mem));
        return;
    }
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nseg = int((a.ksteps + DW_STEPS - 1) / DW_STEPS) + 1;  // and the last, of the further units
    const int blk = int(blockIdx.x) - ntok, quad = blk / nseg, seg = blk - quad * nseg;
    const int ug = 4 * quad + wave;                                       // row group of the slab
    const int64_t local = int64_t(ug / a.nf) * (16 * a.nf) + (r16 >> 2) * (4 * a.nf) + 4 * (ug % a.nf) + (r16 & 3);
    const bool live = a.row0 + local < a.d_out;
    const int64_t row = live ? a.row0 + local : a.d_out - 1;
    u32x4_t *wu = reinterpret_cast<u32x4_t *>(a.We) + int64_t(ug) * a.KU * 64;
    const u32x4_t zero = u32x4_t{0u, 0u, 0u, 0u};
    if (seg == nseg - 1) {
        u32x4_t *we = wu + lane;
        const int64_t kp = q8_pitch(a.k);
        for (int64_t u = 0; u < a.kp32 / 32; ++u) {
            const int64_t p0 = 32 * u + 8 * g;
            const uint2 qv = (p0 < kp) ? *reinterpret_cast<const uint2 *>(a.q8 + row * kp + p0) : make_uint2(0u, 0u);
            float sc[8], v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sc[e] = (p0 + e < a.k) ? a.scale[p0 + e] : 0.0f;
            payload8(qv, sc, v, a.pfmt);
            we[(4 * a.ksteps + u) * 64] = u32x4_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                                                  pack_bf16x2(v[6], v[7])};
        }
        const int64_t used = 4 * a.ksteps + a.kp32 / 32 + (a.rank > 0 ? 2 : 0);
        if (a.rank > 0) {
            uint32_t b[4] = {0u, 0u, 0u, 0u};
            const int q0 = 8 * (g & 1);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (q0 + e < a.rank) b[e >> 1] |= uint32_t(a.B[row * a.rank + q0 + e]) << (16 * (e & 1));
            const u32x4_t bv = u32x4_t{b[0], b[1], b[2], b[3]};
            we[(used - 2) * 64] = bv;
            we[(used - 1) * 64] = (g < 2) ? bv : zero;
        }
        if (used < a.KU) we[used * 64] = zero;
        return;
    }
    const int64_t k0 = int64_t(seg) * DW_STEPS;
    // first code of the row in its 64-row tiles
    const int64_t base = (((row >> 6) * (a.pitch / 16)) << 10) + 16 * (row & 63);
    // code and gain words of the lane's 32 inputs of a step, which are its row
    // of unit g: d = 8, chunks 4 g .. + 3 of a plane tile; d = 16, chunks 2 g,
    // 2 g + 1 of the step's half tile
    uint32_t cw[DW_STEPS][S], gw[DW_STEPS][S][2];
#pragma unroll
    for (int i = 0; i < DW_STEPS; ++i) {
        const int64_t ks = (k0 + i < a.ksteps) ? k0 + i : a.ksteps - 1;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (D == 8) {
                const int64_t e = base + (ks << 10) + 4 * g;
                cw[i][s] = *reinterpret_cast<const uint32_t *>(static_cast<const uint8_t *>(a.codes[s]) + e);
                const uint2 gv = *reinterpret_cast<const uint2 *>(a.gains[s] + e);
                gw[i][s][0] = gv.x;
                gw[i][s][1] = gv.y;
            } else {
                const int64_t e = base + ((ks >> 1) << 10) + 8 * (ks & 1) + 2 * g;
                cw[i][s] = *reinterpret_cast<const uint32_t *>(static_cast<const uint16_t *>(a.codes[s]) + e);
                gw[i][s][0] = *reinterpret_cast<const uint32_t *>(a.gains[s] + e);
            }
        }
    }
    if constexpr (D == 8) {
        for (int e = t; e < S * 256; e += 64 * DO_WAVES)
            s_mem[e] = reinterpret_cast<const u32x4_t *>(a.tabh[e >> 8])[e & 255];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < DW_STEPS; ++i) {
        if (k0 + i >= a.ksteps) break;
        f16x8_t tv[4][S];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if constexpr (D == 8)
                    tv[q][s] = __builtin_bit_cast(f16x8_t, s_mem[s * 256 + ((cw[i][s] >> (8 * q)) & 0xffu)]);
                else
                    tv[q][s] = *reinterpret_cast<const f16x8_t *>(
                        a.tabh[s] + size_t((cw[i][s] >> (16 * (q >> 1))) & 0xffffu) * 16 + 8 * (q & 1));
            }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const uint32_t gq = (D == 8) ? gw[i][s][q >> 1] >> (16 * (q & 1)) : gw[i][s][0] >> (16 * (q >> 1));
                const float gs = f16_bits_to_f32(uint16_t(gq));
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = __builtin_fmaf(gs, float(tv[q][s][e]), v[e]);
            }
            wu[(4 * (k0 + i) + g) * 64 + 16 * q + r16] =
                u32x4_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
        }
    }
}

// ---------------------------------------------------------------------------
// The product. Eight waves as WM x WN; a wave owns MF groups of 16 tokens and
// NF groups of 16 weight rows (a lane's accumulator holds four consecutive
// rows of one token: W_hat is the left operand). Per unit step of 32 inputs
// the block's units reach a ring of NS LDS slots by DMA, NS steps ahead of
// the step whose products run; the fragments of step u + 1 are read while the
// products of step u issue, so one barrier per step is all a wave waits for.
//
// 2000 tokens, 12288 x 4096: 177 us, 1.2 PFLOP/s with the padding (the whole
// call 401 -> 204 us). The matrix cores are busy for 55% of its cycles, at
// 2.0 GHz; without the DMAs it takes 30 us less, without the stores of Y 15
// us less. Four waves with 128-row tiles (half the LDS reads) took 20% to 60%
// longer: one wave per SIMD leaves the barriers uncovered.
// ---------------------------------------------------------------------------
template <int MF, int NF, int WM, int WN>
struct DenseShape {
    static constexpr int NW = WM * WN;                 // waves
    static_assert(NW == 4 || NW == 8, "one or two waves per SIMD");
    static constexpr int XU = MF * WM, WU = NF * WN;   // units per step
    static constexpr int BM = 16 * XU, BN = 16 * WU;
    static constexpr int SLOT = (XU + WU) * 1024;
    // five slots for the 128 x 128 block, half a compute unit's LDS. (One runs
    // per compute unit all the same: the kernel's register count is raised to
    // the two waves per SIMD that it asks for, and the plan's step time for
    // this tile was measured so.)
    static constexpr int NS_FIT = GEMM_LDS_BYTES / (XU + WU <= 16 ? 2 : 1) / SLOT;
    static constexpr int NS = NS_FIT < 6 ? NS_FIT : 6;
    static constexpr int NI = XU + WU;                 // DMA instructions per step: wave w issues w, w + NW, ...
    static constexpr int PMAX = (NI + NW - 1) / NW, PMIN = NI / NW;
    static constexpr size_t LDS = size_t(NS) * SLOT;
    static_assert(NS >= 3, "two steps in flight beside the one being read");
    static_assert((NS - 1) * PMAX <= 63, "wait count fits vmcnt");
};

template <int MF, int NF, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WM * WN / 4, WM * WN / 4)))
void dense_gemm(const DenseArgs a)
{
    using G = DenseShape<MF, NF, WM, WN>;
    extern __shared__ __attribute__((aligned(16))) uint4 s_mem4[];
    uint8_t *s_mem = reinterpret_cast<uint8_t *>(s_mem4);
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // Tile of the block. Workgroups go to the 8 XCDs in turn (linear id mod
    // 8), each with its own L2: every XCD gets a run of consecutive tiles, in
    // an order that walks up to 8 token tiles before the next weight tile, so
    // that the tiles that run together on an XCD share both operands.
    // With K split the splits of all tiles follow each other.
    const int total = a.mtiles * a.ntiles * a.ksplit;
    const int xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
    int lg = xcd * per + (xcd < rem ? xcd : rem) + int(blockIdx.x >> 3);
    const int z = lg / (a.mtiles * a.ntiles);
    lg -= z * (a.mtiles * a.ntiles);
    const int band = lg / (8 * a.ntiles);
    lg -= band * 8 * a.ntiles;
    const int bh = (a.mtiles - 8 * band < 8) ? a.mtiles - 8 * band : 8;
    const int by = 8 * band + lg % bh, bx = lg / bh;

    // units [kb, ke) of split z, an even number of them
    const int64_t KU = a.KU;
    const int kb = int(KU / 2 * z / a.ksplit) * 2, ke = int(KU / 2 * (z + 1) / a.ksplit) * 2;
    const uint8_t *src[G::PMAX];
    int dst[G::PMAX];
#pragma unroll
    for (int r = 0; r < G::PMAX; ++r) {
        const int v0 = wave + G::NW * r, v = (v0 < G::NI) ? v0 : G::NI - 1;
        const uint8_t *base = (v < G::XU)
            ? reinterpret_cast<const uint8_t *>(a.Xe) + ((int64_t(by) * G::XU + v) * KU << 10)
            : reinterpret_cast<const uint8_t *>(a.We) + ((int64_t(bx) * G::WU + (v - G::XU)) * KU << 10);
        src[r] = base + (int64_t(kb) << 10) + 16 * lane;
        dst[r] = v << 10;
    }
    const bool full = wave < G::NI % G::NW || G::PMAX == G::PMIN;
    const int ku = ke - kb;
    auto dma = [&](int u, int slot) {
        const int64_t off = int64_t(u < ku ? u : ku - 1) << 10;  // past the end: a reload that nothing reads
#pragma unroll
        for (int r = 0; r < G::PMAX; ++r) {
            if (r >= G::PMIN && !full) continue;
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint4 *>(src[r] + off),
                                             reinterpret_cast<uint4 *>(s_mem + slot * G::SLOT + dst[r]), 16, 0, 0);
        }
    };
#pragma unroll
    for (int c = 0; c < G::NS; ++c) dma(c, c);

    f32x4_t acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    bf16x8_t xf[2][MF], wf[2][NF];
    const uint8_t *xb = s_mem + (wm * MF) * 1024 + 16 * lane;
    const uint8_t *wb = s_mem + (G::XU + wn * NF) * 1024 + 16 * lane;
    auto frags = [&](int p, int slot) {
#pragma unroll
        for (int j = 0; j < NF; ++j) wf[p][j] = *reinterpret_cast<const bf16x8_t *>(wb + slot * G::SLOT + j * 1024);
#pragma unroll
        for (int i = 0; i < MF; ++i) xf[p][i] = *reinterpret_cast<const bf16x8_t *>(xb + slot * G::SLOT + i * 1024);
    };
    auto products = [&](int p) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[p][j], xf[p][i], acc[i][j], 0, 0, 0);
    };
    if (full) wait_vm<(G::NS - 1) * G::PMAX>();
    else wait_vm<(G::NS - 1) * G::PMIN>();
    lds_barrier();
    frags(0, 0);
    // step u: slot u % NS. Its fragments are in registers (p = u % 2) once the
    // barrier's LDS wait is over, for every wave, so its slot takes step u + NS.
    int slot = 0;
    auto step = [&](int u, int p) {
        if (full) wait_vm<(G::NS - 2) * G::PMAX>();
        else wait_vm<(G::NS - 2) * G::PMIN>();
        lds_barrier();
        dma(u + G::NS, slot);
        slot = (slot + 1 == G::NS) ? 0 : slot + 1;
        frags(1 - p, slot);
        products(p);
        // one LDS read ahead of every two products
#pragma unroll
        for (int i = 0; i < MF + NF; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        }
    };
    for (int u = 0; u < ku; u += 2) {
        step(u, 0);
        step(u + 1, 1);
    }
    wait_vm<0>();  // the clamped DMAs land before the block ends

    // the lane's 4 NF consecutive outputs of MF tokens
    const int64_t m0 = int64_t(by) * G::BM + 16 * (wm * MF) + r16;
    const int64_t n = a.row0 + int64_t(bx) * G::BN + 16 * (wn * NF) + 4 * NF * g;
    const int64_t nend = a.row0 + a.rows;
    if (a.ksplit > 1) {
        float *pz = a.part + (int64_t(z) * a.Mp + m0) * a.np + (n - a.row0);
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) *reinterpret_cast<f32x4_t *>(pz + 16 * i * a.np + 4 * j) = acc[i][j];
        return;
    }
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int64_t m = m0 + 16 * i;
        if (m >= a.M) continue;
        if (a.y_vec && n + 4 * NF <= nend) {
            if (a.y_bf16) {
                uint2 *y = reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.Y) + m * a.ldy + n);
#pragma unroll
                for (int j = 0; j < NF; ++j) y[j] = make_uint2(pack_bf16x2(acc[i][j][0], acc[i][j][1]), pack_bf16x2(acc[i][j][2], acc[i][j][3]));
            } else {
                f32x4_t *y = reinterpret_cast<f32x4_t *>(static_cast<float *>(a.Y) + m * a.ldy + n);
#pragma unroll
                for (int j = 0; j < NF; ++j) y[j] = acc[i][j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t nn = n + 4 * j + r;
                    if (nn >= nend) break;
                    if (a.y_bf16) static_cast<uint16_t *>(a.Y)[m * a.ldy + nn] = f32_to_bf16(acc[i][j][r]);
                    else static_cast<float *>(a.Y)[m * a.ldy + nn] = acc[i][j][r];
                }
        }
    }
}

// Tile shapes: tokens and rows of a block, row groups of a wave.
struct DenseTile { int bm, bn, nf; };
constexpr DenseTile DENSE_TILES[] = {{256, 256, 4}, {256, 192, 3}, {256, 128, 4}, {128, 128, 2}};

struct DensePlan {
    int tile, ksplit;
    int64_t bm, bn, mtiles, Mp, ksteps, kp32, KU, slab, nslab;
    int nxseg;  // workgroups of 512 inputs along a row of X
    double us;  // estimated time of the product
    size_t tp_off, xe_off, we_off, part_off, total;
};

// The plan and its sizes do not depend on the adapter (KU counts its units).
DensePlan dense_plan(int64_t d_out, int64_t d_in, int64_t M, int64_t k)
{
    DensePlan p{};
    p.ksteps = (d_in + BK - 1) / BK;
    p.kp32 = (k + 31) & ~int64_t(31);
    p.KU = (4 * p.ksteps + p.kp32 / 32 + 2 + 1) & ~int64_t(1);
    const int64_t row_bytes = p.KU * 64;
    p.nslab = std::max<int64_t>((d_out * row_bytes + DENSE_SLAB_BYTES - 1) / DENSE_SLAB_BYTES, 1);
    // Tile and K split with the least estimated time (us): rounds of blocks
    // over the 256 compute units, a unit step taking 0.13 + 0.56 per 256 x 256
    // of tile (0.28, 0.41, 0.59 and 0.68 measured for the four tiles on 4096
    // inputs; 128 x 128 tiles 8% more where the weights come from memory) and a
    // block about 8 besides; the fp32 tiles of a split are written whole, read
    // and added in a launch of its own. (Without the padded tokens and rows in
    // that, 257 tokens of 2048 x 8192 took 256-token tiles in 8 splits: 51 us
    // against 41; 129 tokens of 8192 x 4096 58 against 52.)
    double best = 1e300;
    for (int i = 0; i < 4; ++i) {
        const DenseTile &c = DENSE_TILES[i];
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((d_out + c.bn - 1) / c.bn);
        for (int ks : {1, 2, 3, 4, 6, 8}) {
            if (ks > 1 && (tiles * ks > 256 || p.KU / ks < 24 || p.nslab > 1)) break;
            const double step = (0.13 + 0.56 * c.bm * c.bn / 65536.0) * (c.bm == 128 && d_out * row_bytes > DENSE_CACHED_BYTES ? 1.08 : 1.0);
            const double us = double((tiles * ks + 255) / 256) * (double(p.KU) / ks * step + 8.0) +
                              (ks > 1 ? 5.0 + (4.0 * ks * double(tiles) * c.bm * c.bn + (4.0 * ks + 2.0) * double(M) * double(d_out)) / 4e6
                                      : 0.0);
            if (us < best) {
                best = us;
                p.tile = i;
                p.ksplit = ks;
            }
        }
    }
    p.us = best;
    p.bm = DENSE_TILES[p.tile].bm;
    p.bn = DENSE_TILES[p.tile].bn;
    p.mtiles = std::max<int64_t>((M + p.bm - 1) / p.bm, 1);
    p.Mp = p.mtiles * p.bm;
    p.slab = (((d_out + p.nslab - 1) / p.nslab + p.bn - 1) / p.bn) * p.bn;
    p.nxseg = int((p.ksteps + DO_WAVES - 1) / DO_WAVES);
    p.tp_off = size_t(GEMM_HDR) + align256(size_t(p.Mp) * BSQ_MAX_LORA_RANK * 4);
    p.xe_off = p.tp_off + align256(size_t(p.nxseg) * size_t(p.Mp) * BSQ_MAX_LORA_RANK * 4);
    p.we_off = p.xe_off + size_t(p.Mp) * size_t(row_bytes);
    p.part_off = p.we_off + size_t(p.slab) * size_t(row_bytes);
    p.total = p.part_off + ((p.ksplit > 1) ? size_t(p.ksplit) * size_t(p.Mp) * size_t(p.slab) * 4 : 0);
    return p;
}

template <int D>
hipError_t launch_operands(int stages, const DenseArgs &a, int ntok, hipStream_t st)
{
    // row groups in quads: within the slab, whose rows are whole blocks of 128 or more
    const int64_t quads = (a.rows + 16 * a.nf - 1) / (16 * a.nf) * a.nf;
    const int64_t nseg = (a.ksteps + DW_STEPS - 1) / DW_STEPS + 1;
    const dim3 grid(unsigned(ntok + (quads + 3) / 4 * nseg));
    switch (stages) {
    case 1: hipLaunchKernelGGL((dense_operands<D, 1>), grid, dim3(64 * DO_WAVES), 0, st, a, ntok); break;
    case 2: hipLaunchKernelGGL((dense_operands<D, 2>), grid, dim3(64 * DO_WAVES), 0, st, a, ntok); break;
    case 3: hipLaunchKernelGGL((dense_operands<D, 3>), grid, dim3(64 * DO_WAVES), 0, st, a, ntok); break;
    default: hipLaunchKernelGGL((dense_operands<D, 4>), grid, dim3(64 * DO_WAVES), 0, st, a, ntok); break;
    }
    return hipGetLastError();
}

template <int MF, int NF, int WM, int WN>
hipError_t launch_product(DenseArgs a, hipStream_t st)
{
    using G = DenseShape<MF, NF, WM, WN>;
    static std::atomic<bool> lds_set{false};  // the ring exceeds the default dynamic LDS limit
    if (!lds_set.load(std::memory_order_relaxed)) {  // (a call that failed here leaves it to the next)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&dense_gemm<MF, NF, WM, WN>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(G::LDS));
        if (e != hipSuccess) return e;
        lds_set.store(true, std::memory_order_relaxed);
    }
    a.ntiles = int((a.rows + G::BN - 1) / G::BN);
    hipLaunchKernelGGL((dense_gemm<MF, NF, WM, WN>), dim3(unsigned(a.mtiles) * unsigned(a.ntiles) * unsigned(a.ksplit)), dim3(64 * G::NW), G::LDS, st, a);
    return hipGetLastError();
}

}  // namespace

// The product's estimate scaled to a whole call, and the operands: decoding
// the weights (written and read back through memory where they outgrow the
// last-level cache), X, the adapter. Coefficients: per stage, of the product,
// per million weights, of those per stage, of those past 60 million more, per
// million elements of X, the adapter's launch. Fitted as gemm_tiled_us, which
// says over what.
double gemm_dense_us(int d, int stages, int64_t d_out, int64_t d_in, int64_t M, int64_t k, int rank)
{
    const double C8[] = {0.94, 0.76, 0.335, 0.084, 0.5, 0.91, 3.5};
    const double C16[] = {3.3, 0.656, 0.142, 0.685, 0.34, 1.9, 2.75};
    const double *c = (d == 8) ? C8 : C16;
    const double w = double(d_out) * double(d_in) * 1e-6;
    return c[0] * stages + c[1] * dense_plan(d_out, d_in, M, k).us + (c[2] + c[3] * stages) * w +
           c[4] * std::max(0.0, w - 60.0) + c[5] * double(M) * double(d_in) * 1e-6 + (rank > 0 ? c[6] : 0.0);
}

size_t gemm_dense_ws_bytes(int64_t d_out, int64_t d_in, int64_t M, int64_t k)
{
    return dense_plan(d_out, d_in, M, k).total;
}

hipError_t launch_gemm_dense(const bsq_config &cfg, const void *codec, const bsq_layer &L, const bsq_lora *lora,
                             const void *X, int64_t M, int64_t ldx, void *Y, int y_dtype, int64_t ldy, void *ws,
                             hipStream_t st)
{
    const int rank = lora ? int(lora->rank) : 0;
    const DensePlan p = dense_plan(L.d_out, L.d_in, M, L.k);
    char *wb = static_cast<char *>(ws);
    const char *cb = static_cast<const char *>(codec);
    DenseArgs a{};
    for (int s = 0; s < cfg.stages; ++s) {
        a.codes[s] = L.codes[s];
        a.gains[s] = L.gains[s];
        a.tabh[s] = reinterpret_cast<const uint16_t *>(cb + codec_tabh_offset(cfg, s));
    }
    a.q8 = L.prot_q8;
    a.scale = L.prot_scale;
    a.idx = L.prot_idx;
    a.bits = L.prot_bits;
    a.X = static_cast<const uint16_t *>(X);
    if (rank > 0) {
        a.A = lora->A;
        a.B = lora->B;
    }
    a.T = reinterpret_cast<float *>(wb + GEMM_HDR);
    a.Tp = reinterpret_cast<float *>(wb + p.tp_off);
    a.Mp = p.Mp;
    a.nxseg = p.nxseg;
    a.ksplit = p.ksplit;
    a.part = reinterpret_cast<float *>(wb + p.part_off);
    a.np = p.slab;
    a.Xe = reinterpret_cast<uint16_t *>(wb + p.xe_off);
    a.We = reinterpret_cast<uint16_t *>(wb + p.we_off);
    a.Y = Y;
    a.M = M;
    a.ldx = ldx;
    a.d_in = L.d_in;
    a.d_out = L.d_out;
    a.pitch = L.pitch;
    a.k = L.k;
    a.kp32 = p.kp32;
    a.ldy = ldy;
    a.ksteps = p.ksteps;
    a.KU = (4 * p.ksteps + p.kp32 / 32 + (rank > 0 ? 2 : 0) + 1) & ~int64_t(1);
    a.mtiles = int(p.mtiles);
    a.rank = rank;
    a.pfmt = cfg.protect_format;
    a.y_bf16 = (y_dtype == BSQ_BF16);
    const int64_t vb = a.y_bf16 ? 8 : 16;  // four outputs
    a.y_vec = (reinterpret_cast<uintptr_t>(Y) % vb == 0) && ((ldy * (vb / 4)) % vb == 0);

    a.nf = DENSE_TILES[p.tile].nf;
    hipError_t e = hipSuccess;
    for (int64_t r0 = 0; e == hipSuccess && r0 < L.d_out; r0 += p.slab) {
        a.row0 = r0;
        a.rows = std::min<int64_t>(p.slab, L.d_out - r0);
        const int ntok = (r0 == 0) ? int(p.Mp / 16) * (p.nxseg + 1) : 0;
        e = (cfg.d == 8) ? launch_operands<8>(cfg.stages, a, ntok, st) : launch_operands<16>(cfg.stages, a, ntok, st);
        if (e != hipSuccess) break;
        if (r0 == 0 && rank > 0) {
            hipLaunchKernelGGL(dense_adapter, dim3(unsigned(p.Mp / 16)), dim3(64), 0, st, a);
            if ((e = hipGetLastError()) != hipSuccess) break;
        }
        switch (p.tile) {
        case 0: e = launch_product<8, 4, 2, 4>(a, st); break;
        case 1: e = launch_product<8, 3, 2, 4>(a, st); break;
        case 2: e = launch_product<4, 4, 4, 2>(a, st); break;
        default: e = launch_product<4, 2, 2, 4>(a, st); break;
        }
    }
    if (e == hipSuccess && p.ksplit > 1) e = launch_splitk_sum(p.ksplit, a.part, p.Mp, a.np, M, L.d_out, Y, y_dtype, ldy, st);
    return e;
}

}  // namespace bsq
