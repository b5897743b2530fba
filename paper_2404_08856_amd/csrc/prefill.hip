// Prefill: long runs of new rows of ONE sequence (the prompt) through the decoder, up to kPrefillRows rows per
// pass over the weights.  With hundreds of rows the projections are bound by the matrix cores, not by the
// weight stream, so everything here is organised around them:
//
//  * Operand layouts.  Weights: the packed 1 KiB blocks of common.h, unchanged (A operand).  Activations X[R, K]:
//    three bf16 terms per value as everywhere, but each term is a matrix-core operand of its own -- 16 rows fill
//    the 16 columns of the B operand -- and the three products go into the same accumulator: no column of a tile
//    is unused and no sum over term columns is needed.  Block (row tile rt of 16 rows, K-step s, term t) is the
//    1 KiB at index (rt * KS + s) * 3 + t, lane l = r + 16 g holding X[16 rt + r][32 s + 8 g .. + 7].
//  * prefill_gemm_kernel: tiled GEMM, both operands through LDS.  Bound by the matrix cores and the card's power: the 7B QKV projection of
//    2047 rows runs at 1.41 PFLOP/s counting all three terms (a large bf16 matrix product of the library: 1.43 to 1.68).
//  * prefill_attention_kernel: attention of 64 queries per workgroup over the cached keys (which by then include
//    the pass's own rows).
// Measured against passes of 64 rows through the batched verify kernels, whose attention takes 8 queries a launch:
// four 7B layers, 2047 rows 6.5 ms (was 41.1), 640 rows 2.3 (10.2); 12-layer draft, 1472 rows 1.50 ms (47.1).
#include <algorithm>

#include "gemm_core.h"
#include "launch.h"

namespace spd {

// element offset (bf16 units) of X[row][k] term t in the layout above
__device__ __forceinline__ size_t ppack_index(int row, int k, int KS, int t) {
    return (((size_t)(row >> 4) * KS + (k >> 5)) * kTerms + t) * 512 + packed_elem_index(row & 15, k & 31);
}

// four consecutive values (k % 4 == 0) of one row into the packed layout, 8 bytes per term
__device__ __forceinline__ void ppack_store4(uint16_t *X, int row, int k, int KS, const float (&y)[4]) {
    uint32_t lo[kTerms], hi[kTerms];
    split3_pair(y[0], y[1], lo);
    split3_pair(y[2], y[3], hi);
#pragma unroll
    for (int t = 0; t < kTerms; ++t) *reinterpret_cast<uint2 *>(X + ppack_index(row, k, KS, t)) = uint2{lo[t], hi[t]};
}

// 1 KiB from memory (16 bytes per lane) to LDS (lane-linear from `dst`, wave-uniform), without registers; counts on
// vmcnt.  As inline assembly because the compiler makes every LDS read wait for ALL outstanding LDS-direct loads it
// knows of (vmcnt(0)), which would undo the pipelining: the waits are written out in the loops below.  M0 carries the
// LDS address.  The compiler sets it anew wherever it uses it, so declaring it is all that is needed; its notice that it
// will not preserve a reserved register across the statement is turned off.  (Saved and put back around every load: 1 %
// of a short prompt; around a group of loads issued together: 2 %.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ unsigned lds_addr(const void *p) { return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void *)p; }
__device__ __forceinline__ void lds_dma16(const void *base_uniform, unsigned lane_offset, unsigned dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(lane_offset), "s"(base_uniform) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma16(const void *src, unsigned dst) {     // any address per lane
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// ---------------------------------------------------------------------------------
// input rows: h, packed (h * gain) and the rows' sums of squares, one part per kRowSteps K-steps
// ---------------------------------------------------------------------------------
// One workgroup per (row tile, kRowSteps K-steps): a wave writes whole blocks of the packed operand.  (A workgroup per row wrote 16 bytes of
// every line, and the 16 rows of a line ran on 8 XCDs: 640 rows of 4096 columns 27.8 us, 2047 55, now 12.2 and 25.5.)
constexpr int kRowSteps = 16;
__global__ __launch_bounds__(256) void prefill_rows_kernel(const uint16_t *__restrict__ E, const int32_t *__restrict__ tokens,
                                                           const float *__restrict__ embeds, int rows, int d, int vocab,
                                                           const float *__restrict__ gain, float *__restrict__ h,
                                                           uint4 *__restrict__ X, float *__restrict__ ssq, int ssq_ld) {
    const int KS = d / 32, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, w = threadIdx.x >> 6;
    const int row = blockIdx.x * 16 + r;
    const bool ok = row < rows;
    const uint16_t *src_tok = nullptr;
    if (tokens && ok) src_tok = E + (size_t)min(max(tokens[row], 0), vocab - 1) * d;      // never read outside the table
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kRowSteps / 4; ++i) {
        const int s = blockIdx.y * kRowSteps + 4 * i + w, k = 32 * s + 8 * g;
        if (s >= KS || !ok) continue;
        float v[8];
        if (tokens) {
            const uint4 p = *reinterpret_cast<const uint4 *>(src_tok + k);
            const uint32_t q[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[2 * e] = bf16_lo(q[e]); v[2 * e + 1] = bf16_hi(q[e]); }
        } else {
            const float *src = embeds + (size_t)row * d + k;
            const float4 a = *reinterpret_cast<const float4 *>(src), b = *reinterpret_cast<const float4 *>(src + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        }
        float *dst = h + (size_t)row * d + k;
        *reinterpret_cast<float4 *>(dst) = float4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<float4 *>(dst + 4) = float4{v[4], v[5], v[6], v[7]};
        ss += (v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]) + (v[4] * v[4] + v[5] * v[5] + v[6] * v[6] + v[7] * v[7]);
        const float4 ga = *reinterpret_cast<const float4 *>(gain + k), gb = *reinterpret_cast<const float4 *>(gain + k + 4);
        const float y[8] = {v[0] * ga.x, v[1] * ga.y, v[2] * ga.z, v[3] * ga.w, v[4] * gb.x, v[5] * gb.y, v[6] * gb.z, v[7] * gb.w};
        uint32_t t[4][kTerms];
#pragma unroll
        for (int e = 0; e < 4; ++e) split3_pair(y[2 * e], y[2 * e + 1], t[e]);
#pragma unroll
        for (int q = 0; q < kTerms; ++q) X[(((size_t)blockIdx.x * KS + s) * kTerms + q) * 64 + lane] = uint4{t[0][q], t[1][q], t[2][q], t[3][q]};
    }
    ss = xor_step<16>(ss, AddOp());
    ss = xor_step<32>(ss, AddOp());
    __shared__ float part[4][16];
    if (g == 0) part[w][r] = ss;
    __syncthreads();
    if (threadIdx.x < 16 && ok) ssq[(size_t)blockIdx.y * ssq_ld + row] = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
}

int prefill_row_parts(int d) { return (d / 32 + kRowSteps - 1) / kRowSteps; }

hipError_t launch_prefill_rows(const void *embed_bf16, const int32_t *tokens, const float *embeds, int rows, int d, int vocab,
                               const float *gain, float *h, void *X, float *ssq, int ssq_ld, hipStream_t stream) {
    if ((!tokens) == (!embeds) || rows < 1 || rows > ssq_ld) return hipErrorInvalidValue;
    hipLaunchKernelGGL(prefill_rows_kernel, dim3((rows + 15) / 16, prefill_row_parts(d)), dim3(256), 0, stream, (const uint16_t *)embed_bf16, tokens, embeds, rows, d, vocab,
                       gain, h, (uint4 *)X, ssq, ssq_ld);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// GEMM
// ---------------------------------------------------------------------------------
struct PrefillGemmKernelArgs {
    const uint4 *W;           // packed weights, n_tiles x KS blocks
    const uint4 *X;           // packed activations, n_rt x KS x 3 blocks
    int KS, n_tiles, n_rt, rows;
    int n_blk, r_blk;         // workgroups along the features / the rows
    float *Y;
    int ldy;
    const float *ssq_in;      // [ssq_parts][ssq_ld]: partial sums of squares of the rows, or NULL
    int ssq_ld, ssq_parts;
    float inv_d, eps;
    const float *gain_next;   // RESIDUAL: gain of the following norm
    uint16_t *Xnext;
    float *ssq_out;           // RESIDUAL: [part][ssq_ld], one part per NW tiles
    uint16_t *Xout;           // SWIGLU
    int KS_out;
    int J;                    // K slices
    bool fold;                // sums of 16 K-steps between the partial and the running sum (small shape)
    float *partials;          // J > 1: [tile][slice][TN * TR * 256] sums
    unsigned *arrive;         // J > 1: one counter per tile, zero between launches
};

// J > 1: the K range is cut into J slices, one workgroup each.
constexpr int kPgBuf = 3;     // LDS stages: one whose fragments are read, two on their way

// WN x WR waves; a wave owns NW weight tiles (16 features each) and NX row tiles (16 rows each).  One K-step of
// both operands (WN * NW + 3 * WR * NX blocks of 1 KiB) is one LDS stage, brought in by LDS-direct loads; all blocks are in
// operand order already, so the fragment reads are lane-linear and conflict-free.  A step multiplies fragments that are in
// registers; behind the products of each weight fragment go the read of the next step's one and one load of the stage three
// steps ahead (its buffer's fragments are in registers by then).  All loads of a stage at once held the wave up until the
// memory pipe had taken them (16 cycles each, 40 of them per step and CU), and the fragments' reads were a wait of their own: four 7B layers, 2047
// rows 6.94 -> 6.83 ms with the reads a step ahead, 7.14 -> 6.75 with the loads spread too; 640 rows 2.52 -> 2.41; the 12-layer draft, 1472
// rows 1.69 -> 1.67.  What is left is not the pipeline's depth (a fourth stage changes nothing) nor the barrier (without: -1.5 %) but the
// card's power: the matrix cores are busy 70 % of the cycles at 1.85 GHz, 60 % at 1.99 before; the loads into LDS alone cost 16 % and the reads 7 %.
// Accumulation: partial sums over 4 or 8 K-steps are added to a running sum, so no long chain rounds at the size of
// the result.  The second and third terms (2^-8 and 2^-16 of the first) have an accumulator of their own where the
// registers allow it (NW * NX <= 8); otherwise they go into the short partial sum ahead of the first term.
template <int WN, int WR, int NW, int NX, int EPI>
__global__ __launch_bounds__(WN *WR * 64, 2) void prefill_gemm_kernel(PrefillGemmKernelArgs a) {
    constexpr int WAVES = WN * WR, TN = WN * NW, TR = WR * NX, BLK = TN + kTerms * TR, PB = BLK / WAVES;
    static_assert(BLK % WAVES == 0, "equal loads per wave: the waits count them");
    constexpr bool OWN_REST = NW * NX <= 8;
    static_assert(NW % 2 == 0, "the SwiGLU epilogue takes tiles in pairs");
    __shared__ uint4 S[kPgBuf][BLK][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroup -> tile.  Workgroups go round robin over the 8 XCDs; each XCD takes a contiguous run of an order that
    // walks 8 row blocks for one feature block before the next, so that the ~32 workgroups an XCD runs together
    // share 8 row blocks and 4 feature blocks in its L2.
    int nb, rb, slice, tile;
    {
        const int tiles = a.n_blk * a.r_blk, total = tiles * a.J, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        const int base = total >> 3, extra = total & 7;
        const int lin = xcd * base + min(xcd, extra) + slot;
        slice = lin / tiles;                              // all tiles of one slice of K before the next
        tile = lin - slice * tiles;
        const int band = 8 * a.n_blk, b0 = tile / band, in = tile - b0 * band;
        const int rows_in = min(8, a.r_blk - 8 * b0);
        nb = in / rows_in;
        rb = 8 * b0 + in - nb * rows_in;
    }
    const int t0 = nb * TN, rt0 = rb * TR;
    const int k0 = (int)((long)a.KS * slice / a.J), KS = (int)((long)a.KS * (slice + 1) / a.J) - k0;    // K-steps k0 .. k0 + KS - 1

    const uint4 *src[PB];                                 // wave-uniform: block w + i * WAVES of stage 0
    int step[PB];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        const int b = w + i * WAVES;
        if (b < TN) {
            src[i] = a.W + (size_t)min(t0 + b, a.n_tiles - 1) * a.KS * 64 + (size_t)k0 * 64;      // beyond the matrix: a valid tile, result dropped
            step[i] = 64;
        } else {
            const int x = b - TN;
            src[i] = a.X + (((size_t)min(rt0 + x / kTerms, a.n_rt - 1) * a.KS + k0) * kTerms + x % kTerms) * 64;
            step[i] = 64 * kTerms;
        }
    }
    const unsigned lds0 = lds_addr(&S[0][0][0]);
    auto issue_one = [&](int s, int buf, int i) __attribute__((always_inline)) {
        const int ss = s < KS ? s : KS - 1;               // past the end: a harmless re-read
        lds_dma16(src[i] + (size_t)ss * step[i], 16u * lane, lds0 + (unsigned)((buf * BLK + w + i * WAVES) * 1024));
    };
    auto issue = [&](int s, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PB; ++i) issue_one(s, buf, i);
    };
    issue(0, 0);
    issue(1, 1);

    const int wn = w % WN, wr = w / WN;
    // 1 / rms of this lane's rows from the producer's partial sums: a lane group takes every fourth, fixed order.  The loads of 32 parts of
    // all rows go out together and read 16 neighbouring rows of a part.  Four 7B layers, a prompt of 64 rows: one part after the other, a
    // row's parts side by side 671 us, together 678, together and rows side by side 651; 128 rows 890 / 897 / 859, 2000 rows 6668 / - / 6275.
    float inv[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) inv[j] = 1.0f;
    if (a.ssq_in) {
        float ss[NX];
        int row[NX];
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            ss[j] = 0.f;
            row[j] = min((rt0 + wr * NX + j) * 16 + (lane & 15), a.rows - 1);
        }
        for (int p0 = lane >> 4; p0 < a.ssq_parts; p0 += 32) {
            float t[8][NX];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int j = 0; j < NX; ++j) t[u][j] = a.ssq_in[(size_t)min(p0 + 4 * u, a.ssq_parts - 1) * a.ssq_ld + row[j]];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int j = 0; j < NX; ++j) ss[j] += p0 + 4 * u < a.ssq_parts ? t[u][j] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            ss[j] = xor_step<16>(ss[j], AddOp());
            ss[j] = xor_step<32>(ss[j], AddOp());
            inv[j] = 1.0f / sqrtf(ss[j] * a.inv_d + a.eps);
        }
    }

    f32x4_t part[NW][NX], sum[NW][NX], rest[OWN_REST ? NW : 1][NX];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            part[i][j] = sum[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (OWN_REST) rest[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    // K-steps per partial sum; fold: partial sums go into sums of four before they reach the running sum
    const int chunk = a.fold || KS <= 64 ? 4 : 8;
    int left = chunk, quarter = a.fold ? 4 : 1 << 30;
    f32x4_t mid[OWN_REST ? NW : 1][NX];
    if (OWN_REST) {
#pragma unroll
        for (int i = 0; i < (OWN_REST ? NW : 0); ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j) mid[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    auto fold_partial = [&] __attribute__((always_inline)) {
        if (--left == 0) {
            left = chunk;
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    if (OWN_REST) mid[OWN_REST ? i : 0][j] += part[i][j];
                    else sum[i][j] += part[i][j];
                    part[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
            if (OWN_REST && --quarter == 0) {
                quarter = 4;
#pragma unroll
                for (int i = 0; i < NW; ++i)
#pragma unroll
                    for (int j = 0; j < NX; ++j) { sum[i][j] += mid[OWN_REST ? i : 0][j]; mid[OWN_REST ? i : 0][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
            }
        }
    };
    uint4 wf[NW], xa[kTerms][NX], xb[kTerms][NX];
    auto read_x = [&](uint4 (&x)[kTerms][NX], int q, int buf) __attribute__((always_inline)) {   // fragment q of the row tiles
        const int t = kTerms - 1 - q / NX, j = q % NX;
        x[t][j] = S[buf][TN + (wr * NX + j) * kTerms + t][lane];
    };
    // One K-step: its fragments are in wf and x, the next one's are read from buffer `next` (into wf and xn), stage `later` goes into `buf`
    auto multiply = [&](uint4 (&x)[kTerms][NX], uint4 (&xn)[kTerms][NX], int next, int later, int buf) __attribute__((always_inline)) {
        constexpr int XR = (kTerms * NX + NW - 1) / NW, LR = (PB + NW - 1) / NW;     // reads and loads per weight fragment
#pragma unroll
        for (int i = 0; i < NW; ++i) {
#pragma unroll
            for (int q = i * XR; q < (i + 1) * XR && q < kTerms * NX; ++q) read_x(xn, q, next);
#pragma unroll
            for (int t = kTerms - 1; t >= 0; --t)
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    if (OWN_REST && t > 0) rest[i][j] = mfma_bf16(wf[i], x[t][j], rest[i][j]);
                    else part[i][j] = mfma_bf16(wf[i], x[t][j], part[i][j]);
                }
            wf[i] = S[next][wn * NW + i][lane];
#pragma unroll
            for (int q = i * LR; q < (i + 1) * LR && q < PB; ++q) issue_one(later, buf, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        fold_partial();
    };
    // the older of the two stages on their way has landed for everyone, and nobody reads the one before it any more (lgkmcnt: not
    // a read of it is still under way when a wave passes the barrier, wherever the compiler put the products)
    auto arrive = [&] __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((kPgBuf - 2) * PB) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    int cur = 0, nxt = 1;
    auto advance = [&] __attribute__((always_inline)) {
        cur = nxt;
        nxt = nxt + 1 == kPgBuf ? 0 : nxt + 1;
    };
    arrive();
    issue(2, 2);
#pragma unroll
    for (int q = 0; q < kTerms * NX; ++q) read_x(xa, q, 0);
#pragma unroll
    for (int i = 0; i < NW; ++i) wf[i] = S[0][wn * NW + i][lane];
    int s = 0;
    for (; s + 1 < KS; s += 2) {
        arrive();
        multiply(xa, xb, nxt, s + kPgBuf, cur);
        advance();
        arrive();
        multiply(xb, xa, nxt, s + 1 + kPgBuf, cur);
        advance();
    }
    if (s < KS) {
        arrive();
        multiply(xa, xb, nxt, s + kPgBuf, cur);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no load to LDS may outlive the workgroup
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            if (OWN_REST) part[i][j] = mid[OWN_REST ? i : 0][j] + (part[i][j] + rest[i][j]);
            sum[i][j] += part[i][j];
        }

    if (a.J > 1) {
        // This slice's sums in whole lines (512 contiguous bytes per store), written through to memory; once they are acknowledged take a
        // ticket.  The last slice of the tile to arrive (nobody waits) adds all of them in slice order and goes on.
        constexpr size_t kTile = (size_t)TN * TR * 64;    // float4 quads of a tile
        unsigned long long *mine = reinterpret_cast<unsigned long long *>(a.partials) + ((size_t)tile * a.J + slice) * kTile * 2;
        auto at = [&](int i, int j, int half) { return (size_t)(((w * NW + i) * NX + j) * 2 + half) * 64 + lane; };
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                typedef __attribute__((ext_vector_type(2))) unsigned long long u64x2_t;
                const u64x2_t v = __builtin_bit_cast(u64x2_t, sum[i][j]);
                __hip_atomic_store(mine + at(i, j, 0), v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(mine + at(i, j, 1), v.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                                  // (nobody reads the stages any more either)
        int &is_last = *reinterpret_cast<int *>(&S[0][0][0]);
        if (threadIdx.x == 0) {
            const unsigned ticket = __hip_atomic_fetch_add(a.arrive + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = ticket == (unsigned)(a.J - 1);
            if (is_last) __hip_atomic_store(a.arrive + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        }
        __syncthreads();
        if (!is_last) return;
        // This slice's sums are still here: added in their place without the way back through memory (12-layer draft, 200 rows: 857 -> 831 us).
        float own[NW][NX][4];
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) { own[i][j][v] = sum[i][j][v]; sum[i][j][v] = 0.f; }
        for (int s = 0; s < a.J; ++s) {
            if (s == slice) {                             // workgroup-uniform
#pragma unroll
                for (int i = 0; i < NW; ++i)
#pragma unroll
                    for (int j = 0; j < NX; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) sum[i][j][v] += own[i][j][v];
                continue;
            }
            const unsigned long long *src = reinterpret_cast<const unsigned long long *>(a.partials) + ((size_t)tile * a.J + s) * kTile * 2;
            unsigned long long lo[NW][NX], hi[NW][NX];
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    lo[i][j] = __hip_atomic_load(src + at(i, j, 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    hi[i][j] = __hip_atomic_load(src + at(i, j, 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    sum[i][j][0] += __uint_as_float((unsigned)lo[i][j]); sum[i][j][1] += __uint_as_float((unsigned)(lo[i][j] >> 32));
                    sum[i][j][2] += __uint_as_float((unsigned)hi[i][j]); sum[i][j][3] += __uint_as_float((unsigned)(hi[i][j] >> 32));
                }
        }
    }

    // D[feature 4 g + v][row r] of tile (i, j): a lane holds 4 consecutive features of one row
    const int r = lane & 15, g = lane >> 4;
    float4 hold[NW][NX], gn[NW];
    if (EPI == EPI_RESIDUAL) {                            // all old values on their way together, before any store
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int t = min(t0 + wn * NW + i, a.n_tiles - 1), col = t * 16 + 4 * g;
            gn[i] = *reinterpret_cast<const float4 *>(a.gain_next + col);
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                const int row = min((rt0 + wr * NX + j) * 16 + r, a.rows - 1);
                hold[i][j] = *reinterpret_cast<const float4 *>(a.Y + (size_t)row * a.ldy + col);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int row = (rt0 + wr * NX + j) * 16 + r;
        const bool row_ok = row < a.rows;
        if (EPI == EPI_SWIGLU) {
            // rows 0..7 of a tile are gate features (g = 0, 1), rows 8..15 the matching up features (g = 2, 3): of a pair
            // of tiles the lower half-wave finishes the first, the upper half the second
#pragma unroll
            for (int i = 0; i < NW; i += 2) {
                const int t = t0 + wn * NW + i + (g >> 1);
                float y[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float p = sum[i][j][v] * inv[j], q = sum[i + 1][j][v] * inv[j];
                    const float got = lane_xor<32>(g < 2 ? q : p);
                    const float gate = g < 2 ? p : got, up = g < 2 ? got : q;
                    y[v] = gate / (1.0f + expf(-gate)) * up;
                }
                if (row_ok && t < a.n_tiles) ppack_store4(a.Xout, row, t * 8 + 4 * (g & 1), a.KS_out, y);
            }
        } else {
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int t = t0 + wn * NW + i, col = t * 16 + 4 * g;
                if (!(row_ok && t < a.n_tiles)) continue;
                float4 *dst = reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + col);
                if (EPI == EPI_STORE) {
                    *dst = float4{sum[i][j][0] * inv[j], sum[i][j][1] * inv[j], sum[i][j][2] * inv[j], sum[i][j][3] * inv[j]};
                } else {
                    float4 h = hold[i][j];
                    h.x += sum[i][j][0]; h.y += sum[i][j][1]; h.z += sum[i][j][2]; h.w += sum[i][j][3];
                    *dst = h;
                    const float y[4] = {h.x * gn[i].x, h.y * gn[i].y, h.z * gn[i].z, h.w * gn[i].w};
                    ppack_store4(a.Xnext, row, col, a.n_tiles / 2, y);
                    sq += (h.x * h.x + h.y * h.y) + (h.z * h.z + h.w * h.w);
                }
            }
            if (EPI == EPI_RESIDUAL) {
                sq = xor_step<16>(sq, AddOp());
                sq = xor_step<32>(sq, AddOp());
                const int p = nb * WN + wn;
                if (g == 0 && row_ok && p * NW < a.n_tiles) a.ssq_out[(size_t)p * a.ssq_ld + row] = sq;
            }
        }
    }
}

template <int WN, int WR, int NW, int NX>
static hipError_t launch_pg(PrefillGemmKernelArgs &k, int epilogue, hipStream_t stream) {
    k.n_blk = (k.n_tiles + WN * NW - 1) / (WN * NW);
    k.r_blk = (k.n_rt + WR * NX - 1) / (WR * NX);
    const dim3 grid(k.n_blk * k.r_blk * k.J), block(WN * WR * 64);
    switch (epilogue) {
        case EPI_STORE: hipLaunchKernelGGL((prefill_gemm_kernel<WN, WR, NW, NX, EPI_STORE>), grid, block, 0, stream, k); break;
        case EPI_RESIDUAL: hipLaunchKernelGGL((prefill_gemm_kernel<WN, WR, NW, NX, EPI_RESIDUAL>), grid, block, 0, stream, k); break;
        case EPI_SWIGLU: hipLaunchKernelGGL((prefill_gemm_kernel<WN, WR, NW, NX, EPI_SWIGLU>), grid, block, 0, stream, k); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Workgroup shape of a projection: large = 256 features x 128 rows, one 8-wave workgroup per CU; small = 128 x 64, two
// 4-wave workgroups per CU (a quarter of the work each, so a large workgroup stands for four small ones).  The large
// shape moves less through LDS per product; the small one wastes less of the last round and of ragged edges, and its sums are more exact (it has the
// registers to keep the second and third terms apart: K and V of a 7B layer, 2047 rows, 1.4 roundings of 10000 flipped against 2.2).  Large only where its rounds
// are at most half the small one's, though one of them costs 1.7 small ones: where the small shape is slower but more exact it stays (7B, small / large: gate|up, 896 rows 397 / 383 us,
// 1280 544 / 517, 1664 711 / 650, 2047 867 / 804; QKV, 1664 364 / 344).  640 rows, O: 80 large workgroups leave two thirds of the CUs idle (75 / 118).
static bool prefill_large(int n_tiles, int rows) {
    const int large = ((n_tiles + 15) / 16) * ((rows + 127) / 128), small = ((n_tiles + 7) / 8) * ((rows + 63) / 64);
    const int rounds_large = (large + 255) / 256, rounds_small = (small + 511) / 512;
    return rounds_large * 2 <= rounds_small;
}
// K slices of the small shape, so that a matrix with few tiles still fills the chip: the smallest estimate in us of rounds, each
// a start and an end (6) and the K-steps (0.65 on a CU shared by two workgroups, 0.45 on one of its own), and the exchange of the partial sums (a round
// trip, reading J of them, and 32 KiB per workgroup across the chip).  A fit to 1 to 8 slices of 12 matrices (K = 768 to 11008)
// at 14 row counts: on average 0.8 % slower than the fastest of them, at most 8 % (with an exchange of 6.7 us, whatever J, 5 % and 32 %).
// The 4-layer draft's QKV at 64 rows: 17.2 -> 14.1 us (8 -> 4 slices), its O at 256 rows 19.1 -> 15.0 (8 -> 5); gate|up of the 12-layer draft at 64 rows
// 15.6 -> 13.2 (1 -> 3); O of the 7B shape at 128 rows 31.3 -> 25.2 (8 -> 6).
static int prefill_slices(int tiles, int KS) {
    auto cost = [&](int J) {
        const int n = tiles * J, steps = (KS + J - 1) / J;
        return (float)((n + 511) / 512) * (6.f + (n <= 256 ? 0.45f : 0.65f) * steps) + (J > 1 ? 1.1f + 1.15f * J + 0.0088f * n : 0.f);
    };
    int best = 1;
    for (int J = 2; J <= kPrefillMaxSlices && tiles * J <= kPrefillMaxSplit && KS / J >= 4; ++J)
        if (cost(J) < cost(best)) best = J;
    return best;
}
size_t prefill_partial_bytes(int N, int max_rows) {
    const long tiles = (long)((N / 16 + 7) / 8) * ((max_rows + 63) / 64);
    return (size_t)std::min((long)kPrefillMaxSplit, tiles * kPrefillMaxSlices) * 32 * 1024;
}
int prefill_ssq_parts(int n_tiles, int rows) { return prefill_large(n_tiles, rows) ? (n_tiles + 7) / 8 : (n_tiles + 3) / 4; }

hipError_t launch_prefill_gemm(const PrefillGemmArgs &a, int epilogue, hipStream_t stream) {
    if (a.N % 16 != 0 || a.rows < 1 || a.rows > kPrefillRows) return hipErrorInvalidValue;
    if (epilogue == EPI_RESIDUAL && (a.N % 32 != 0 || !a.gain_next || !a.Xnext || !a.ssq_out)) return hipErrorInvalidValue;
    if (!a.partials || !a.arrive) return hipErrorInvalidValue;
    PrefillGemmKernelArgs k;
    k.W = (const uint4 *)a.W; k.X = (const uint4 *)a.X;
    k.KS = (a.K + 31) / 32; k.n_tiles = a.N / 16; k.n_rt = (a.rows + 15) / 16; k.rows = a.rows;
    k.Y = a.Y; k.ldy = a.ldy;
    k.ssq_in = a.ssq_in; k.ssq_ld = a.ssq_ld; k.ssq_parts = a.ssq_parts;
    k.inv_d = 1.0f / (float)a.K; k.eps = a.eps;
    k.gain_next = a.gain_next; k.Xnext = (uint16_t *)a.Xnext; k.ssq_out = a.ssq_out;
    k.Xout = (uint16_t *)a.Xout; k.KS_out = (a.N / 2 + 31) / 32;
    k.J = 1;
    k.fold = false;
    k.partials = a.partials; k.arrive = a.arrive;
    if (prefill_large(k.n_tiles, a.rows)) return launch_pg<2, 4, 8, 2>(k, epilogue, stream);
    const int tiles = ((k.n_tiles + 7) / 8) * ((a.rows + 63) / 64);
    k.J = prefill_slices(tiles, k.KS);
    // Slices that fill the chip's 512 places are as short as they can be.  Where the estimate leaves places empty, fewer and longer ones were
    // faster, and their running sums would be longer chains of additions: 7B QKV at 100 rows, two slices of 64 steps instead of five of 26,
    // 10 % more flipped roundings of K and V, and as many with sums in between (0.3 % of a short prompt's time).
    k.fold = k.J > 1 && tiles * k.J <= 384;
    return launch_pg<2, 2, 4, 2>(k, epilogue, stream);
}

// ---------------------------------------------------------------------------------
// RoPE on the new keys, append of K and V
// ---------------------------------------------------------------------------------
// KV length before the call, clamped so that `rows` more positions fit (only device-resident lengths can need it)
__device__ __forceinline__ int first_position(const PrefillAttnArgs &a, bool report) {
    int P0 = a.d_len ? *a.d_len : a.len;
    if (P0 < 0 || P0 + a.rows > a.max_positions) {
        if (report && a.d_error) *a.d_error = 1;
        P0 = max(0, min(P0, a.max_positions - a.rows));
    }
    return P0;
}

// one workgroup per (aligned unit of 32 positions, head)
template <int DH>
__global__ __launch_bounds__(256) void prefill_append_kernel(PrefillAttnArgs a) {
    constexpr int HALF = DH / 2;
    const int P0 = first_position(a, threadIdx.x == 0);
    const int hh = blockIdx.x, unit = P0 / 32 + blockIdx.y;
    const size_t HD = (size_t)a.H * DH;
    uint16_t *Kc = (uint16_t *)a.k_cache + (size_t)hh * a.max_positions * DH;
    uint16_t *Vt = (uint16_t *)a.v_cache + (size_t)hh * DH * a.v_stride + (size_t)unit * DH * 32;
    __shared__ uint16_t vs[DH][40];               // V transposed: [dim][position in the unit], rows of 80 bytes
    if (32 * unit >= P0 + a.rows) return;
    for (int idx = threadIdx.x; idx < 32 * (HALF / 4); idx += 256) {
        const int i = idx / (HALF / 4), j = 4 * (idx % (HALF / 4)), pos = 32 * unit + i, row = pos - P0;
        if (row < 0 || row >= a.rows) continue;
        const float *src = a.qkv + (size_t)row * 3 * HD + HD + (size_t)hh * DH + j;
        const float4 k1 = *reinterpret_cast<const float4 *>(src), k2 = *reinterpret_cast<const float4 *>(src + HALF);
        const float4 v1 = *reinterpret_cast<const float4 *>(src + HD), v2 = *reinterpret_cast<const float4 *>(src + HD + HALF);
        const float4 cs0 = *reinterpret_cast<const float4 *>(a.rope + ((size_t)pos * HALF + j) * 2);
        const float4 cs1 = *reinterpret_cast<const float4 *>(a.rope + ((size_t)pos * HALF + j) * 2 + 4);
        const float c[4] = {cs0.x, cs0.z, cs1.x, cs1.z}, s[4] = {cs0.y, cs0.w, cs1.y, cs1.w};
        const float ka[4] = {k1.x, k1.y, k1.z, k1.w}, kb[4] = {k2.x, k2.y, k2.z, k2.w};
        const float va[4] = {v1.x, v1.y, v1.z, v1.w}, vb[4] = {v2.x, v2.y, v2.z, v2.w};
        union { uint2 u; uint16_t h[4]; } o1, o2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o1.h[e] = f32_to_bf16_bits(ka[e] * c[e] - kb[e] * s[e]);
            o2.h[e] = f32_to_bf16_bits(kb[e] * c[e] + ka[e] * s[e]);
            vs[j + e][i] = f32_to_bf16_bits(va[e]);
            vs[j + e + HALF][i] = f32_to_bf16_bits(vb[e]);
        }
        *reinterpret_cast<uint2 *>(Kc + (size_t)pos * DH + j) = o1.u;
        *reinterpret_cast<uint2 *>(Kc + (size_t)pos * DH + j + HALF) = o2.u;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < DH * 4; idx += 256) {       // 8 positions of one dimension: 16 bytes
        const int dim = idx >> 2, p8 = 8 * (idx & 3), row = 32 * unit + p8 - P0;
        uint16_t *dst = Vt + (size_t)dim * 32 + p8;
        if (row >= 0 && row + 8 <= a.rows) {
            *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(&vs[dim][p8]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (row + e >= 0 && row + e < a.rows) dst[e] = vs[dim][p8 + e];
        }
    }
}

// ---------------------------------------------------------------------------------
// attention
// ---------------------------------------------------------------------------------
// One workgroup of 4 waves per (head, 64 queries), 16 queries per wave.  Units of 32 keys (K and V: DH / 16 KiB each)
// pass through LDS, already in operand order, two units ahead; every wave multiplies its queries with them:
//   S[key, query] = K q^T (A = 16 keys x 32 dims, B = q, three terms smallest first into one accumulator),
//   online softmax (a lane's column is one query), O[dim, query] += V^T p (B = p in three terms).
// The rows of the two score tiles of a unit stand for keys 8 (i / 4) + 4 ab + i % 4, so a lane ends up with the
// probabilities of 8 consecutive keys, which is its slot of the second product's B operand.
// Heavy query blocks (late positions) are launched first; the head index is fastest, so with a head count that is a
// multiple of 8 a head's workgroups share an XCD and its L2.
// Bound by the vector instructions of the softmax and the three-term split next to as many matrix-core cycles: no
// branches per key, packed conversions and register swaps instead of LDS for the maximum took the 7B shape at 2047
// rows from 133 to 114 us per layer, the 12-layer draft at 1472 rows from 58 to 34.  A second set of 4 waves on every other
// unit of the same 64 queries (merged at the end) was no faster where workgroups are few (31 us) and slower at 2047 rows (157): as many workgroups, twice the waves.
// (The form with two waves for the same queries has 32 queries and 4 waves: twice the workgroups, see prefill_split.)
// Heads of 64 take two units per step: a wave is alone on its SIMD for most of a launch (12 heads x 23 blocks of queries), and one unit's
// products run next to the other's softmax (1472 rows, 36.2 to 32.4 us).  Heads of 128 come with more workgroups: at 2047 rows three of them per CU
// (one unit per step, at most 168 registers) take 113 us, two 125 with two units and 131 with one.
constexpr int kPaBuf = 3;                        // steps in LDS: one in use, one there, one on its way
constexpr int prefill_step_units(int DH, bool SPLIT) { return SPLIT || DH == 64 ? 2 : 1; }

// bf16 pairs with an infinite or NaN value replaced by 0
__device__ __forceinline__ uint32_t finite_pair(uint32_t p) {
    if ((p & 0x7f80u) == 0x7f80u) p &= 0xffff0000u;
    if ((p & 0x7f800000u) == 0x7f800000u) p &= 0x0000ffffu;
    return p;
}

__device__ __forceinline__ uint32_t exponent_carry(uint32_t p) { return (p & 0x7f807f80u) + 0x00800080u; }
// A operand of ones where a bf16 value is +inf (or -inf) or NaN, zeros elsewhere (both signs count a NaN: inf - inf again)
__device__ __forceinline__ uint4 ones_where(const uint4 &q, bool negative) {
    auto half = [&](uint32_t h) {
        const bool nan = (h & 0x7fffu) > 0x7f80u;
        return nan || h == (negative ? 0xff80u : 0x7f80u) ? 0x3f80u : 0u;
    };
    auto pair = [&](uint32_t p) { return half(p & 0xffffu) | (half(p >> 16) << 16); };
    return uint4{pair(q.x), pair(q.y), pair(q.z), pair(q.w)};
}

constexpr float kLowest = -3.402823466e38f;      // start of the running maximum: below every score but -inf

// exp(x) for x <= 0 like exp_neg, but NaN stays NaN and very negative arguments (-inf too) give exactly 0
__device__ __forceinline__ float exp_score(float x) {
    x = __builtin_elementwise_maximum(x, -150.0f);
    const float c1 = 1.44269502162933349609375f, c2 = 1.925963033500011e-8f;   // log2(e) = c1 + c2
    const float t = x * c1;
    const float lo = __builtin_fmaf(x, c1, -t) + x * c2;
    const float p = __builtin_amdgcn_exp2f(t);
    return __builtin_fmaf(p, lo * 0.693147180559945f, p);
}

template <int DH, bool SPLIT>
__global__ __launch_bounds__(256, SPLIT && DH == 128 ? 1 : 2) void prefill_attention_kernel(PrefillAttnArgs a) {
    constexpr int HALF = DH / 2, NC = DH / 32, NDT = DH / 16, BLK = 2 * NC + NDT, PB = BLK / 4;
    constexpr int U = prefill_step_units(DH, SPLIT);
    constexpr int QW = SPLIT ? 2 : 4, QUERIES = 16 * QW;         // waves with queries of their own; queries of a workgroup
    __shared__ uint4 S[kPaBuf][U][BLK][64];
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hh = blockIdx.x, qt = gridDim.y - 1 - blockIdx.y;
    const int P0 = first_position(a, false);
    const size_t HD = (size_t)a.H * DH;
    const uint16_t *Kc = (const uint16_t *)a.k_cache + (size_t)hh * a.max_positions * DH;
    const uint16_t *Vt = (const uint16_t *)a.v_cache + (size_t)hh * DH * a.v_stride;
    const int k_end = P0 + a.rows - 1;                           // last valid position
    const int n_units = min(P0 + qt * QUERIES + QUERIES - 1, k_end) / 32 + 1;    // units any query of this workgroup sees

    // this wave's share of a unit: blocks w, w + 4, ...; 0 .. 2 NC - 1: K (tile ab, chunk c), then V (dim tile)
    const unsigned lds0 = lds_addr(&S[0][0][0][0]);
    auto issue = [&](int u, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < U; ++h) {
            const int uu = min(u + h, n_units - 1);              // past the end: a harmless re-read
#pragma unroll
            for (int i = 0; i < PB; ++i) {
                const int b = w + 4 * i;
                const uint16_t *src;
                if (i < NC / 2) {                                // b < 2 NC
                    const int key = min(32 * uu + 8 * (r >> 2) + 4 * (b / NC) + (r & 3), k_end);
                    src = Kc + (size_t)key * DH + 32 * (b % NC) + 8 * g;
                } else {
                    src = Vt + ((size_t)uu * DH + 16 * (b - 2 * NC) + r) * 32 + 8 * g;
                }
                lds_dma16(src, lds0 + (unsigned)(((buf * U + h) * BLK + b) * 1024));
            }
        }
    };
    const int qw = w % QW, kw = w / QW;                         // SPLIT: wave kw of the two with these queries takes unit kw of a step
    const int row = qt * QUERIES + qw * 16 + r;                 // this lane's query
    // q: RoPE, scale, three terms, as B operand blocks (chunk c: dims 32 c + 8 g .. + 7 of query r)
    uint4 q[NC][kTerms];
    {
        const float scale = 1.0f / sqrtf((float)DH);
        const int rr = min(row, a.rows - 1), pos = P0 + rr;
        const float *src = a.qkv + (size_t)rr * 3 * HD + (size_t)hh * DH + 8 * g;
#pragma unroll
        for (int c = 0; c < NC / 2; ++c) {
            union { uint4 v; uint32_t h[4]; } t1[kTerms], t2[kTerms];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                float y1[2], y2[2];
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const float x1 = src[32 * c + e + f], x2 = src[32 * c + HALF + e + f];
                    const float2 cs = *reinterpret_cast<const float2 *>(a.rope + ((size_t)pos * HALF + 32 * c + 8 * g + e + f) * 2);
                    y1[f] = (x1 * cs.x - x2 * cs.y) * scale;
                    y2[f] = (x2 * cs.x + x1 * cs.y) * scale;
                }
                uint32_t s1[kTerms], s2[kTerms];
                split3_pair(y1[0], y1[1], s1);
                split3_pair(y2[0], y2[1], s2);
#pragma unroll
                for (int t = 0; t < kTerms; ++t) { t1[t].h[e / 2] = s1[t]; t2[t].h[e / 2] = s2[t]; }
            }
#pragma unroll
            for (int t = 0; t < kTerms; ++t) { q[c][t] = t1[t].v; q[c + NC / 2][t] = t2[t].v; }
        }
    }
    issue(0, 0);
    issue(U, 1);

    const int q_pos = P0 + row, w_first = P0 + qt * QUERIES + qw * 16, w_last = min(w_first + 15, k_end);
    const bool wave_has_rows = w_first <= k_end;
    float m_run = kLowest, l_run = 0.f;
    f32x4_t acc[NDT];
#pragma unroll
    for (int i = 0; i < NDT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // scores of a unit: keys 32 u + 8 g + 4 ab + v of this lane's query
    auto scores = [&](const uint4 (*X)[64], f32x4_t (&sc)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int ab = 0; ab < 2; ++ab) {
            sc[ab] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            uint4 kf[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) kf[c] = X[ab * NC + c][lane];
#pragma unroll
            for (int t = kTerms - 1; t >= 0; --t)
#pragma unroll
                for (int c = 0; c < NC; ++c) sc[ab] = mfma_bf16(kf[c], q[c][t], sc[ab]);
        }
    };
    auto max_of = [&](const f32x4_t (&sc)[2]) __attribute__((always_inline)) {
        return max_over_rows(fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])), fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3]))));
    };
    union Terms { uint4 v; uint32_t h[4]; };
    // probabilities of a unit in three terms; their sum over this lane's keys
    auto probabilities = [&](const f32x4_t (&sc)[2], float m_new, Terms (&pb)[kTerms]) __attribute__((always_inline)) {
        float p[8], lsum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            p[e] = exp_score(sc[e >> 2][e & 3] - m_new);
            lsum += p[e];
        }
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            uint32_t t3[kTerms];
            split3_pair(p[e], p[e + 1], t3);
#pragma unroll
            for (int t = 0; t < kTerms; ++t) pb[t].h[e / 2] = t3[t];
        }
        return lsum;
    };
    // two units all of whose keys every query of the wave sees: the same steps in the same order, side by side
    auto two_units = [&](const uint4 (*X0)[64], const uint4 (*X1)[64]) __attribute__((always_inline)) {
        f32x4_t s0[2], s1[2];
        scores(X0, s0);
        scores(X1, s1);
        const float m0 = fmaxf(m_run, max_of(s0)), m1 = fmaxf(m0, max_of(s1));
        const float rescale0 = exp_score(m_run - m0), rescale1 = exp_score(m0 - m1);
        m_run = m1;
        Terms p0[kTerms], p1[kTerms];
        l_run = l_run * rescale0 + probabilities(s0, m0, p0);
        l_run = l_run * rescale1 + probabilities(s1, m1, p1);
#pragma unroll
        for (int i = 0; i < NDT; ++i) {
            const uint4 v0 = X0[2 * NC + i][lane], v1 = X1[2 * NC + i][lane];
            f32x4_t o0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, o1 = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = kTerms - 1; t >= 0; --t) {
                o0 = mfma_bf16(v0, p0[t].v, o0);
                o1 = mfma_bf16(v1, p1[t].v, o1);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][v] = __builtin_fmaf(__builtin_fmaf(acc[i][v], rescale0, o0[v]), rescale1, o1[v]);
        }
    };

    int buf = 0, nbuf = 2;
    for (int u = 0; u < n_units; u += U) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(U * PB) : "memory");   // as in the GEMM: this step's units are there, reads of the last step's are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(u + 2 * U, nbuf);
        const bool both = U == 2 && !SPLIT && 32 * u + 63 <= w_first && wave_has_rows;    // wave-uniform, like the conditions below
        if (both) two_units(S[buf][0], S[buf][U - 1]);
#pragma unroll
        for (int h = 0; h < U; ++h) {
            if (!both && wave_has_rows && (!SPLIT || h == kw) && 32 * (u + h) <= w_last) {
                const bool diagonal = 32 * (u + h) + 31 > w_first;         // some key is hidden from some query of the wave
                f32x4_t sc[2];
                scores(S[buf][h], sc);
                if (diagonal) {
#pragma unroll
                    for (int ab = 0; ab < 2; ++ab)
#pragma unroll
                        for (int v = 0; v < 4; ++v) sc[ab][v] = 32 * (u + h) + 8 * g + 4 * ab + v > q_pos ? -INFINITY : sc[ab][v];
                }
                const float m_new = fmaxf(m_run, max_of(sc));
                const float rescale = exp_score(m_run - m_new);      // (a first unit: 0)
                m_run = m_new;
                Terms pb[kTerms];
                l_run = l_run * rescale + probabilities(sc, m_new, pb);   // this lane's keys only: added up over the lane groups at the end
                uint4 vf[NDT];
#pragma unroll
                for (int i = 0; i < NDT; ++i) vf[i] = S[buf][h][2 * NC + i][lane];
                bool odd = false;                                    // wave-uniform: some V of a unit with hidden keys is not finite
                if (diagonal) {
                    uint32_t top = 0;                                // an exponent of all ones carries into its half's sign bit
#pragma unroll
                    for (int i = 0; i < NDT; ++i)
                        top |= exponent_carry(vf[i].x) | exponent_carry(vf[i].y) | exponent_carry(vf[i].z) | exponent_carry(vf[i].w);
                    odd = __any((top & 0x80008000u) != 0);
                    if (odd) {                                       // a hidden key's V must not leak through 0 * inf
#pragma unroll
                        for (int i = 0; i < NDT; ++i) {
                            vf[i].x = finite_pair(vf[i].x); vf[i].y = finite_pair(vf[i].y);
                            vf[i].z = finite_pair(vf[i].z); vf[i].w = finite_pair(vf[i].w);
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < NDT; ++i) {
                    f32x4_t o = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = kTerms - 1; t >= 0; --t) o = mfma_bf16(vf[i], pb[t].v, o);
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][v] = __builtin_fmaf(acc[i][v], rescale, o[v]);
                }
                if (odd) {                                           // rare: a V that is not finite reaches the queries that see its key
                    uint4 seen = {0, 0, 0, 0};                       // B operand: 1 where this lane's query sees the key
                    const int n_seen = q_pos + 1 - (32 * (u + h) + 8 * g); // of the lane's 8 keys
                    uint32_t *sw = reinterpret_cast<uint32_t *>(&seen);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sw[e] = (2 * e < n_seen ? 0x3f80u : 0u) | (2 * e + 1 < n_seen ? 0x3f800000u : 0u);
#pragma unroll
                    for (int i = 0; i < NDT; ++i) {
                        const uint4 raw = S[buf][h][2 * NC + i][lane];
                        const f32x4_t pos = mfma_bf16(ones_where(raw, false), seen, f32x4_t{0.f, 0.f, 0.f, 0.f});
                        const f32x4_t neg = mfma_bf16(ones_where(raw, true), seen, f32x4_t{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            if (pos[v] > 0.f) acc[i][v] += INFINITY;
                            if (neg[v] > 0.f) acc[i][v] -= INFINITY;
                        }
                    }
                }
            }
        }
        buf = buf + 1 == kPaBuf ? 0 : buf + 1;
        nbuf = nbuf + 1 == kPaBuf ? 0 : nbuf + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    l_run = xor_step<16>(l_run, AddOp());
    l_run = xor_step<32>(l_run, AddOp());
    if constexpr (SPLIT) {                                       // the two waves' results meet in LDS
        __syncthreads();                                         // (nobody reads the stages any more)
        float (*other)[64] = reinterpret_cast<float (*)[64]>(&S[0][0][0][0]) + qw * (4 * NDT + 2);
        if (kw == 1) {
#pragma unroll
            for (int i = 0; i < NDT; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) other[4 * i + v][lane] = acc[i][v];
            other[4 * NDT][lane] = m_run;
            other[4 * NDT + 1][lane] = l_run;
        }
        __syncthreads();
        if (kw == 1) return;
        const float m1 = other[4 * NDT][lane], m = fmaxf(m_run, m1), w0 = exp_score(m_run - m), w1 = exp_score(m1 - m);
        l_run = l_run * w0 + other[4 * NDT + 1][lane] * w1;
#pragma unroll
        for (int i = 0; i < NDT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][v] = __builtin_fmaf(acc[i][v], w0, other[4 * i + v][lane] * w1);
    }
    if (row < a.rows) {
#pragma unroll
        for (int i = 0; i < NDT; ++i) {
            const float y[4] = {acc[i][0] / l_run, acc[i][1] / l_run, acc[i][2] / l_run, acc[i][3] / l_run};
            ppack_store4((uint16_t *)a.xout, row, hh * DH + 16 * i + 4 * g, (int)(HD / 32), y);
        }
    }
}

// Where few workgroups of 64 queries make a launch, its time is that of the last block of queries, which sees all keys.  With 32 queries per workgroup and two
// waves for the same 16 (one takes every other unit, the two results are merged at the end) that block is spread over two CUs and its waves
// go through half as many units each.  Prompt of the 12-layer draft, 64 / 32 queries: 200 rows 726 / 715 us, 700 962 / 917, 1472 1518 / 1435 (attention 32.7 / 25.3 a
// layer), 2000 1866 / 1780; the 4-layer draft (heads of 128): 400 307 / 296, 1000 498 / 467, 2000 (256 workgroups) 809 / 762.  Heads of 128 take 96 KiB of
// LDS then, one workgroup per CU: four 7B layers, 256 rows (128 workgroups) 1104 / 1100, 512 (256) 1890 / 1896, 640 (320) 2190 / 2217.
static bool prefill_split(int heads, int rows, int dh) {
    const int blocks = (rows + 63) / 64, wgs = heads * blocks;
    return dh == 64 ? wgs <= 512 : wgs <= 128 || (wgs <= 256 && blocks >= 16);
}

hipError_t launch_prefill_attention(const PrefillAttnArgs &a, bool attend, hipStream_t stream) {
    if (a.rows < 1 || a.rows > a.max_positions || (a.v_stride % 32) != 0 || a.v_stride < a.max_positions) return hipErrorInvalidValue;
    if (a.dh != 128 && a.dh != 64) return hipErrorInvalidValue;
    const bool split = prefill_split(a.H, a.rows, a.dh);
    const int queries = split ? 32 : 64;
    const dim3 g1(a.H, (a.rows + 31) / 32 + 1), g2(a.H, (a.rows + queries - 1) / queries);
    if (a.dh == 128) hipLaunchKernelGGL(prefill_append_kernel<128>, g1, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(prefill_append_kernel<64>, g1, dim3(256), 0, stream, a);
    if (!attend) return hipGetLastError();
    if (a.dh == 128 && split) hipLaunchKernelGGL((prefill_attention_kernel<128, true>), g2, dim3(256), 0, stream, a);
    else if (a.dh == 128) hipLaunchKernelGGL((prefill_attention_kernel<128, false>), g2, dim3(256), 0, stream, a);
    else if (split) hipLaunchKernelGGL((prefill_attention_kernel<64, true>), g2, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((prefill_attention_kernel<64, false>), g2, dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace spd
