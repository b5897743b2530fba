// Prompt GEMM for models whose projections all contract over at least kWideK values (launch.h): activations as two f16 terms
// instead of three bf16 terms (prefill_core.h), weights converted on the way to the matrix cores.
#include <algorithm>

#include "gemm_core.h"
#include "launch.h"
#include "prefill_core.h"

namespace spd {

// ---------------------------------------------------------------------------------
// input rows: h, packed (h * gain) and the row's sum of squares (one part)
// ---------------------------------------------------------------------------------
// One workgroup per row tile, a wave takes whole blocks of 128 columns in operand order: lane r + 16 g holds 8 consecutive
// columns of row r, so every store of a term is one whole 1 KiB block (2047 rows of 4096 columns: 55 us with a workgroup per
// row and 8-byte pieces, 23 us like this).
__global__ __launch_bounds__(1024) void wide_rows_kernel(const uint16_t *__restrict__ E, const int32_t *__restrict__ tokens,
                                                            const float *__restrict__ embeds, int rows, int d, int vocab,
                                                            const float *__restrict__ gain, float *__restrict__ h,
                                                            uint16_t *__restrict__ X, float *__restrict__ xs, float *__restrict__ ssq, int ssq_ld) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, w = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int KS = d / 32, NB = (KS + 3) / 4, row = blockIdx.x * 16 + r;
    const bool row_ok = row < rows;
    const int rr = min(row, rows - 1);
    const uint16_t *src_tok = tokens ? E + (size_t)min(max(tokens[rr], 0), vocab - 1) * d : nullptr;      // never read outside the table
    const float *src_row = embeds ? embeds + (size_t)rr * d : nullptr;
    float ss = 0.f;
    for (int b = w; b < NB; b += waves) {
        float x[4][8], gn[4][8], top = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ks = 4 * b + u, k = min(ks, KS - 1) * 32 + 8 * g;
            if (src_tok) {
                const uint4 p = *reinterpret_cast<const uint4 *>(src_tok + k);
                const uint32_t q[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) { x[u][2 * e] = bf16_lo(q[e]); x[u][2 * e + 1] = bf16_hi(q[e]); }
            } else {
                const float4 p = *reinterpret_cast<const float4 *>(src_row + k), q = *reinterpret_cast<const float4 *>(src_row + k + 4);
                x[u][0] = p.x; x[u][1] = p.y; x[u][2] = p.z; x[u][3] = p.w; x[u][4] = q.x; x[u][5] = q.y; x[u][6] = q.z; x[u][7] = q.w;
            }
            const float4 ga = *reinterpret_cast<const float4 *>(gain + k), gb = *reinterpret_cast<const float4 *>(gain + k + 4);
            gn[u][0] = ga.x; gn[u][1] = ga.y; gn[u][2] = ga.z; gn[u][3] = ga.w; gn[u][4] = gb.x; gn[u][5] = gb.y; gn[u][6] = gb.z; gn[u][7] = gb.w;
            if (ks < KS && row_ok) {
                *reinterpret_cast<float4 *>(h + (size_t)row * d + k) = float4{x[u][0], x[u][1], x[u][2], x[u][3]};
                *reinterpret_cast<float4 *>(h + (size_t)row * d + k + 4) = float4{x[u][4], x[u][5], x[u][6], x[u][7]};
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (ks < KS) {
                    ss += x[u][e] * x[u][e];
                    top = fmaxf(top, fabsf(x[u][e] * gn[u][e]));
                }
            }
        }
        const float factor = block_factor(max_over_rows(top));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (4 * b + u >= KS) break;
            uint4 term[kWideTerms];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t t[kWideTerms];
                split2_products(x[u][2 * e], gn[u][2 * e], x[u][2 * e + 1], gn[u][2 * e + 1], factor, power_inverse(factor), t);
#pragma unroll
                for (int i = 0; i < kWideTerms; ++i) reinterpret_cast<uint32_t *>(&term[i])[e] = t[i];
            }
#pragma unroll
            for (int i = 0; i < kWideTerms; ++i)
                if (row_ok) reinterpret_cast<uint4 *>(X)[(((size_t)blockIdx.x * KS + 4 * b + u) * kWideTerms + i) * 64 + lane] = term[i];
        }
        if (g == 0 && row_ok) xs[pscale_index(row, b, NB)] = power_inverse(factor);
    }
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    __shared__ float part[16][16];
    if (g == 0) part[w][r] = ss;
    __syncthreads();
    if (threadIdx.x < 16 && row_ok) {
        float sum = 0.f;
        for (int i = 0; i < waves; ++i) sum += part[i][r];
        ssq[(size_t)row * ssq_ld] = sum;
    }
}

hipError_t launch_wide_rows(const void *embed_bf16, const int32_t *tokens, const float *embeds, int rows, int d, int vocab,
                            const float *gain, float *h, void *X, float *x_scale, float *ssq, int ssq_ld, hipStream_t stream) {
    if ((!tokens) == (!embeds) || rows < 1 || d % 32 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(wide_rows_kernel, dim3((rows + 15) / 16), dim3(64 * std::min(16, (d + 127) / 128)), 0, stream, (const uint16_t *)embed_bf16,
                       tokens, embeds, rows, d, vocab, gain, h, (uint16_t *)X, x_scale, ssq, ssq_ld);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// factors of the weights' rows
// ---------------------------------------------------------------------------------
// one workgroup per tile of 16 packed rows: the factor of a row from its largest finite magnitude
__global__ __launch_bounds__(256) void weight_factor_kernel(const uint4 *__restrict__ W, int KS, float *__restrict__ out) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t top = 0;                                     // bf16 magnitudes order like their bits
#pragma unroll 8
    for (int s = w; s < KS; s += 4) {
        const uint4 q = W[((size_t)blockIdx.x * KS + s) * 64 + lane];
        const uint32_t p[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = p[e] & 0x7fffu, hi = (p[e] >> 16) & 0x7fffu;
            if (lo < 0x7f80u) top = max(top, lo);
            if (hi < 0x7f80u) top = max(top, hi);
        }
    }
    top = max(top, (uint32_t)__shfl_xor((int)top, 16));
    top = max(top, (uint32_t)__shfl_xor((int)top, 32));
    __shared__ uint32_t part[4][16];
    if (lane < 16) part[w][lane] = top;
    __syncthreads();
    if (threadIdx.x < 16) {
        top = max(max(part[0][lane], part[1][lane]), max(part[2][lane], part[3][lane]));
        out[blockIdx.x * 16 + lane] = block_factor(bf16_bits_to_f32((uint16_t)top));
    }
}

hipError_t launch_weight_factors(const void *packed, int N, int K, float *out, hipStream_t stream) {
    hipLaunchKernelGGL(weight_factor_kernel, dim3(N / 16), dim3(256), 0, stream, (const uint4 *)packed, (K + 31) / 32, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// GEMM
// ---------------------------------------------------------------------------------
struct WideGemmKernelArgs {
    const uint4 *W;           // packed weights (bf16), n_tiles x KS blocks
    const float *w_factor;    // [16 n_tiles] factor of every weight row
    const uint4 *X;           // packed activations, n_rt x KS x 2 blocks
    const float *x_scale;     // [n_rt][ceil(KS / CH)][16] inverse factors of the activation blocks
    int KS, n_tiles, n_rt, rows;
    int n_blk, r_blk;         // workgroups along the features / the rows
    float *Y;
    int ldy;
    const float *ssq_in;      // [rows][ssq_ld], ssq_parts valid: partial sums of squares, or NULL
    int ssq_ld, ssq_parts;
    float inv_d, eps;
    const float *gain_next;   // RESIDUAL: gain of the following norm, or NULL: no Xout, no ssq_out
    float *ssq_out;           // RESIDUAL: [rows][ssq_ld], one part per NW tiles
    uint16_t *Xout;           // RESIDUAL: h * gain_next, SWIGLU: the activations
    float *xout_scale;
    int KS_out, NB_out;
    int J;                    // K slices
    float *partials;          // J > 1: [tile][slice][TN * TR * 256] sums
    unsigned *arrive;         // J > 1: one counter per tile, zero between launches
};

__device__ __forceinline__ f32x4_t mfma_f16(const uint4 &a, const uint4 &b, f32x4_t c) {
    typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}
// 8 bf16 weights of one row, times the row's factor, as f16: exact down to 2^-32 of the row's largest (8 significand bits, and
// f16 keeps them down to 2^-17), truncated to multiples of 2^-39 of it below
__device__ __forceinline__ uint32_t weights_to_f16(uint32_t p, float factor) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(bf16_lo(p) * factor, bf16_hi(p) * factor));
}

// a lane's part of a 1 KiB block at a wave-uniform address, which stays in scalar registers (the compiler would add it to the lane's offset)
__device__ __forceinline__ uint4 load_block(const uint4 *base, int lane) {
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
    auto *at = (const __attribute__((address_space(1))) u32x4_t *)(const u32x4_t *)base;
    asm("" : "+s"(at));
    const u32x4_t v = at[(unsigned)lane];
    return uint4{v.x, v.y, v.z, v.w};
}

// WN x WR waves; a wave owns NW weight tiles (16 features each) and NX row tiles (16 rows each).
//
// The weights come through registers (two K-steps ahead) and are converted once per workgroup on their way into LDS (four
// buffers of one K-step, written two steps ahead of their products; one barrier per K-step).  The activations' fragments are
// read straight from memory into registers, two K-steps ahead: WN waves read the same ones, which the L1 serves, and LDS is left
// to the weights, whose fragments WR waves read.  (Both operands through LDS, as three bf16 terms: LDS was busy 79 % of the
// time that the products take at their peak rate, in the small shape 125 %.)  The fragment of the tile after next is
// read while a tile is multiplied, and conversions and sums sit between the products.
// Accumulation: the products of CH K-steps, both terms, smaller term first, go into a partial sum, which is scaled by the
// activation block's inverse factor and added to the running sum.  Where registers allow it (NW * NX <= 8) the second term has
// an accumulator of its own, a partial sum takes 2 K-steps, and another sum, of 16 K-steps, sits between it and the running one.  Error of a product against 64 bits (K = 4096, in 2^-24 of the result, root mean square): 2.5, with three
// bf16 terms 3.0 (large shape) and 2.0 (small).
// Bound by the issue of its instructions (1570 cycles per K-step of the large shape for 1024 cycles of products: conversions, sums and waits
// do not all fit between them) and by the power limit (1.9 GHz with all CUs busy; loops of products alone reach 1.95 PFLOP/s).
// 7B shape, 2047 rows, three bf16 terms / this kernel: QKV 441 / 354 us, O 147 / 116, gate|up 923 / 690, down 384 / 306.
// Measured and dropped: weights converted ahead of time (109 against 116 us, for twice the memory or a pass over them per call), both operands
// through LDS with the conversion in place (126), conversion by dot products (119), loads four steps ahead (143), 128 x 128 tiles (150).
template <int WN, int WR, int NW, int NX, int CH, int AHEAD, int EPI>
__global__ __launch_bounds__(WN *WR * 64, 2) void wide_gemm_kernel(WideGemmKernelArgs a) {
    constexpr int WAVES = WN * WR, TN = WN * NW, TR = WR * NX, PA = TN / WAVES, WF = 4, PF = WF - 1, AD = AHEAD, BD = AHEAD;
    constexpr bool OWN_REST = NW * NX <= 8;
    constexpr int FL = OWN_REST ? 2 : CH;                 // K-steps per partial sum
    static_assert(TN % WAVES == 0 && PA < NW, "equal shares of the weight blocks, converted between the products");
    static_assert(NW % 4 == 0 && (CH == 2 || CH == 4), "ring positions are fixed at compile time");
    __shared__ uint4 S[4][TN][64];
    __shared__ float inv_s[TR * 16];
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
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
    const int t0 = nb * TN, rt0 = rb * TR, wn = w % WN, wr = w / WN;
    // K-steps k0 .. k0 + KS - 1: slices are whole groups of 4 K-steps, only the matrix's last group may be short
    const int groups = (a.KS + 3) / 4;
    const int k0 = 4 * (int)((long)groups * slice / a.J), KS = min(4 * (int)((long)groups * (slice + 1) / a.J), a.KS) - k0;

    const uint4 *asrc[PA], *bsrc[NX];                     // wave-uniform
    const float *ssrc[NX];
    float factor[PA];
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        const int t = min(t0 + w + i * WAVES, a.n_tiles - 1);         // beyond the matrix: a valid tile, result dropped
        asrc[i] = a.W + ((size_t)t * a.KS + k0) * 64;
        factor[i] = a.w_factor[t * 16 + r];
    }
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int rt = min(rt0 + wr * NX + j, a.n_rt - 1);
        bsrc[j] = a.X + ((size_t)rt * a.KS + k0) * kWideTerms * 64;
        ssrc[j] = a.x_scale + ((size_t)rt * ((a.KS + CH - 1) / CH) + k0 / CH) * 16;
    }
    uint4 ra[AD][PA], xf[BD][NX][kWideTerms], wf[WF];
    auto load_weights = [&](int slot, int s) __attribute__((always_inline)) {
        const int ss = min(s, KS - 1);                    // past the end: a harmless re-read
#pragma unroll
        for (int i = 0; i < PA; ++i) ra[slot][i] = load_block(asrc[i] + (size_t)ss * 64, lane);
    };
    auto load_rows = [&](int slot, int s) __attribute__((always_inline)) {
        const int ss = min(s, KS - 1);
#pragma unroll
        for (int j = 0; j < NX; ++j)
#pragma unroll
            for (int t = 0; t < kWideTerms; ++t) xf[slot][j][t] = load_block(bsrc[j] + (size_t)(ss * kWideTerms + t) * 64, lane);
    };
    // piece x of 4 PA: a quarter of a block is converted, with its last quarter the block goes into LDS
    auto put_weights = [&](uint4 (&from)[PA], int buf, int x) __attribute__((always_inline)) {
        const int i = x >> 2;
        uint32_t *q = reinterpret_cast<uint32_t *>(&from[i]);
        q[x & 3] = weights_to_f16(q[x & 3], factor[i]);
        if ((x & 3) == 3) S[buf][w + i * WAVES][lane] = from[i];
    };
    // The first two K-steps' weights; then what the loop finds under way when it starts, in the loop's own order (or the compiler, which
    // counts the outstanding loads of both ways into the loop, waits for too many in every round).
    uint4 first[2][PA];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        load_weights(s, s);
#pragma unroll
        for (int i = 0; i < PA; ++i) first[s][i] = ra[s][i];
    }
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        load_weights(s, 2 + s);
        load_rows(s, s);
    }

    // 1 / rms of the workgroup's rows, 4 threads per row, fixed order; read behind barriers
    if (a.ssq_in) {
        for (int i = threadIdx.x; i < TR * 64; i += WAVES * 64) {
            const int row = min(rt0 * 16 + i / 4, a.rows - 1), q = i & 3;
            float ss = 0.f;
            for (int p = q; p < a.ssq_parts; p += 4) ss += a.ssq_in[(size_t)row * a.ssq_ld + p];
            ss += __shfl_xor(ss, 1);
            ss += __shfl_xor(ss, 2);
            if (q == 0) inv_s[i / 4] = 1.0f / sqrtf(ss * a.inv_d + a.eps);
        }
    }

    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    f32x4_t part[NW][NX], rest[OWN_REST ? NW : 1][NX];
    float sum[NW][NX][4], mid[OWN_REST ? NW : 1][NX][4];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            part[i][j] = rest[OWN_REST ? i : 0][j] = zero;
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[i][j][v] = mid[OWN_REST ? i : 0][j][v] = 0.f;
        }
    float scale[NX];
    auto add_partial = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NX; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (OWN_REST) mid[OWN_REST ? i : 0][j][v] = __builtin_fmaf(part[i][j][v] + rest[OWN_REST ? i : 0][j][v], scale[j], mid[OWN_REST ? i : 0][j][v]);
                else sum[i][j][v] = __builtin_fmaf(part[i][j][v], scale[j], sum[i][j][v]);
            }
    };
    auto add_mid = [&] __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (OWN_REST ? NW : 0); ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) { sum[i][j][v] += mid[i][j][v]; mid[i][j][v] = 0.f; }
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int x = 0; x < 4 * PA; ++x) put_weights(first[s], s, x);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PF; ++i) wf[i] = S[0][wn * NW + i][lane];
    // K-steps s0 .. s0 + 3 (RAGGED: those of them below KS)
    auto group = [&](int s0, auto ragged_) __attribute__((always_inline)) {
        constexpr bool RAGGED = decltype(ragged_)::value;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = s0 + u;
            if (RAGGED && s >= KS) break;
            // A wave's LDS writes of step s + 1 (one step ago) are done, and with the barrier everyone's; everyone has read step
            // s - 1 and, long ago, step s - 2, whose buffer this step writes.  (Loads from memory need no wait here: at most these are under way.)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(AD * PA + BD * NX * kWideTerms + NX) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            if (u % CH == 0) {
#pragma unroll
                for (int j = 0; j < NX; ++j) scale[j] = ssrc[j][s / CH * 16 + r];
            }
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                wf[(i + PF) % WF] = i + PF < NW ? S[u][wn * NW + i + PF][lane] : S[(u + 1) & 3][wn * NW + i + PF - NW][lane];
#pragma unroll
                for (int t = kWideTerms - 1; t >= 0; --t)
#pragma unroll
                    for (int j = 0; j < NX; ++j) {
                        f32x4_t &acc = OWN_REST && t > 0 ? rest[OWN_REST ? i : 0][j] : part[i][j];
                        const bool first = u % FL == 0 && (OWN_REST || t == kWideTerms - 1);
                        acc = mfma_f16(wf[i % WF], xf[u % BD][j][t], first ? zero : acc);
                    }
                constexpr int PIECES = (4 * PA + NW - 2) / (NW - 1);              // all but the last tile's share of the conversions
#pragma unroll
                for (int x = i * PIECES; x < (i + 1) * PIECES && x < 4 * PA; ++x) put_weights(ra[u % AD], (u + 2) & 3, x);
                if (i == NW - 1) load_weights(u % AD, s + 2 + AD);
                if (u % FL == FL - 1 && i > 0) add_partial(i - 1);
                __builtin_amdgcn_sched_barrier(0);        // keep this order: conversions and sums between the products
            }
            load_rows(u % BD, s + BD);
            if (u % FL == FL - 1) add_partial(NW - 1);
        }
        if (RAGGED && KS % FL != 0)
#pragma unroll
            for (int i = 0; i < NW; ++i) add_partial(i);
    };
    int s0 = 0;
    for (; s0 + 4 <= KS; s0 += 4) {
        group(s0, std::false_type{});
        if (OWN_REST && (s0 & 12) == 12) add_mid();
    }
    if (s0 < KS) group(s0, std::true_type{});
    add_mid();

    __syncthreads();                                      // inv_s
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
                auto both = [&](int v) { return __float_as_uint(sum[i][j][v]) | (unsigned long long)__float_as_uint(sum[i][j][v + 1]) << 32; };
                __hip_atomic_store(mine + at(i, j, 0), both(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(mine + at(i, j, 1), both(2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __shared__ int is_last;
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned ticket = __hip_atomic_fetch_add(a.arrive + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = ticket == (unsigned)(a.J - 1);
            if (is_last) __hip_atomic_store(a.arrive + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        }
        __syncthreads();
        if (!is_last) return;
        // This slice's sums are still here: added in their place without the way back through memory (four 7B layers, 640 rows: 1960 -> 1944 us).
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
    float4 hold[NW][NX], gn[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {                        // all old values on their way together, before any store
        const int t = min(t0 + wn * NW + i, a.n_tiles - 1), col = t * 16 + 4 * g;
        const float4 f = *reinterpret_cast<const float4 *>(a.w_factor + col);
        const float back[4] = {power_inverse(f.x), power_inverse(f.y), power_inverse(f.z), power_inverse(f.w)};
        if (EPI == EPI_RESIDUAL) gn[i] = a.gain_next ? *reinterpret_cast<const float4 *>(a.gain_next + col) : float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int row = min((rt0 + wr * NX + j) * 16 + r, a.rows - 1);
            if (EPI == EPI_RESIDUAL) hold[i][j] = *reinterpret_cast<const float4 *>(a.Y + (size_t)row * a.ldy + col);
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[i][j][v] *= back[v];
        }
    }
    if (EPI == EPI_STORE) {
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int lrow = (wr * NX + j) * 16 + r, row = rt0 * 16 + lrow;
            const float inv = a.ssq_in ? inv_s[lrow] : 1.0f;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int t = t0 + wn * NW + i;
                if (row < a.rows && t < a.n_tiles)
                    *reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + t * 16 + 4 * g) = float4{sum[i][j][0] * inv, sum[i][j][1] * inv, sum[i][j][2] * inv, sum[i][j][3] * inv};
            }
        }
        return;
    }
    // The next projection's operand, kept as two factors: RESIDUAL h and the gain of the next norm; SWIGLU (NW / 2 tiles) silu(gate) and
    // up: rows 0..7 of a tile are gate features (g = 0, 1), rows 8..15 the matching up features (g = 2, 3): of a pair of tiles
    // the lower half-wave finishes the first, the upper half the second.  `top`: the largest magnitude among this wave's columns of a row.
    constexpr int NY = EPI == EPI_SWIGLU ? NW / 2 : NW;
    float top[NX], ya[NY][NX][4], yb[NY][NX][4];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int lrow = (wr * NX + j) * 16 + r, row = rt0 * 16 + lrow;
        const bool row_ok = row < a.rows;
        top[j] = 0.f;
        if (EPI == EPI_SWIGLU) {
            const float inv = a.ssq_in ? inv_s[lrow] : 1.0f;
#pragma unroll
            for (int i = 0; i < NW; i += 2) {
                const bool in = t0 + wn * NW + i + (g >> 1) < a.n_tiles;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float p = sum[i][j][v] * inv, q = sum[i + 1][j][v] * inv;
                    const float got = __shfl_xor(g < 2 ? q : p, 32);
                    const float gate = g < 2 ? p : got, up = g < 2 ? got : q;
                    ya[i / 2][j][v] = gate / (1.0f + expf(-gate));
                    yb[i / 2][j][v] = up;
                    if (in) top[j] = fmaxf(top[j], fabsf(ya[i / 2][j][v] * up));
                }
            }
        } else {
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int t = t0 + wn * NW + i;
                if (!(row_ok && t < a.n_tiles)) continue;
                float4 h = hold[i][j];
                h.x += sum[i][j][0]; h.y += sum[i][j][1]; h.z += sum[i][j][2]; h.w += sum[i][j][3];
                *reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + t * 16 + 4 * g) = h;
                sq += (h.x * h.x + h.y * h.y) + (h.z * h.z + h.w * h.w);
                const float hv[4] = {h.x, h.y, h.z, h.w}, gv[4] = {gn[i].x, gn[i].y, gn[i].z, gn[i].w};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    ya[i][j][v] = hv[v];
                    yb[i][j][v] = gv[v];
                    top[j] = fmaxf(top[j], fabsf(hv[v] * gv[v]));
                }
            }
            if (a.gain_next) {
                sq += __shfl_xor(sq, 16);
                sq += __shfl_xor(sq, 32);
                const int p = nb * WN + wn;
                if (g == 0 && row_ok && p * NW < a.n_tiles) a.ssq_out[(size_t)row * a.ssq_ld + p] = sq;
            }
        }
        top[j] = max_over_rows(top[j]);
    }
    if (EPI == EPI_RESIDUAL && !a.gain_next) return;
    // A block of the operand is what the workgroup produces of a row -- 128 columns, 64 from the small shape's SwiGLU -- or, where
    // it produces 256, what one wave does.
    constexpr bool BY_WAVE = EPI == EPI_RESIDUAL && NW * 16 == 128;
    if (!BY_WAVE) {
        __shared__ float top_s[WN][TR * 16];
#pragma unroll
        for (int j = 0; j < NX; ++j)
            if (g == 0) top_s[wn][(wr * NX + j) * 16 + r] = top[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NX; ++j)
#pragma unroll
            for (int x = 0; x < WN; ++x) top[j] = fmaxf(top[j], top_s[x][(wr * NX + j) * 16 + r]);
    }
    const int block = BY_WAVE ? nb * WN + wn : nb;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int row = (rt0 + wr * NX + j) * 16 + r;
        if (row >= a.rows) continue;
        const float f = block_factor(top[j]);
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            const int t = t0 + wn * NW + (EPI == EPI_SWIGLU ? 2 * i + (g >> 1) : i);
            if (t >= a.n_tiles) continue;
            ppack_store4<kWideTerms>(a.Xout, row, EPI == EPI_SWIGLU ? t * 8 + 4 * (g & 1) : t * 16 + 4 * g, a.KS_out, ya[i][j], yb[i][j], f);
        }
        if (g == 0 && (BY_WAVE || wn == 0) && block < a.NB_out) a.xout_scale[pscale_index(row, block, a.NB_out)] = power_inverse(f);
    }
}

template <int WN, int WR, int NW, int NX, int CH, int AHEAD>
static hipError_t launch_wide(WideGemmKernelArgs &k, int epilogue, hipStream_t stream) {
    k.n_blk = (k.n_tiles + WN * NW - 1) / (WN * NW);
    k.r_blk = (k.n_rt + WR * NX - 1) / (WR * NX);
    const dim3 grid(k.n_blk * k.r_blk * k.J), block(WN * WR * 64);
    switch (epilogue) {
        case EPI_STORE: hipLaunchKernelGGL((wide_gemm_kernel<WN, WR, NW, NX, CH, AHEAD, EPI_STORE>), grid, block, 0, stream, k); break;
        case EPI_RESIDUAL: hipLaunchKernelGGL((wide_gemm_kernel<WN, WR, NW, NX, CH, AHEAD, EPI_RESIDUAL>), grid, block, 0, stream, k); break;
        case EPI_SWIGLU: hipLaunchKernelGGL((wide_gemm_kernel<WN, WR, NW, NX, CH, AHEAD, EPI_SWIGLU>), grid, block, 0, stream, k); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Workgroup shapes: large = 256 features x 128 rows, one 8-wave workgroup per CU; small = 128 x 64, two 4-wave workgroups per CU.
// The large one moves half as much per product; the small one wastes less of the last round and of ragged edges.
static int wide_tiles(bool large, int n_tiles, int rows) {
    return large ? ((n_tiles + 15) / 16) * ((rows + 127) / 128) : ((n_tiles + 7) / 8) * ((rows + 63) / 64);
}
// Shape and number of K slices (so that a matrix with few tiles still fills the chip): the smallest estimate in us of rounds of
// workgroups, each a start and an end and a time per K-step, and, for slices, the exchange of their sums: a few round trips and
// 32 KiB (small) or 128 KiB (large) per workgroup through memory.  The constants are a fit to both shapes and 1 to 8 slices of 12 matrices
// (K = 768 to 11008) at 14 row counts from 33 to 2047: what it chooses is on average 1.2 % and at most 17 % slower than the fastest of them.
// E.g. the 7B down projection, 640 rows: large 1 / 3 / 4 slices 248 / 123 / 183 us, small 1 / 3 174 / 142; gate|up of the 12-layer draft,
// 1472 rows: large 29.8, small 32.6, 640 rows: large 26.9, small 20.0.
static float wide_cost(bool large, int slices, int tiles, int groups) {
    const int n = tiles * slices, steps = 4 * ((groups + slices - 1) / slices);
    const float rounds = large ? (float)((n + 255) / 256) * (11.4f + 0.855f * steps) : (float)((n + 511) / 512) * (5.1f + (n <= 256 ? 0.37f : 0.57f) * steps);
    return rounds + (slices > 1 ? 1.7f + 0.67f * slices + 0.0084f * (large ? 4 * n : n) : 0.f);
}
WidePlan wide_plan(int N, int K, int rows) {
    const int groups = ((K + 31) / 32 + 3) / 4;
    WidePlan best{false, 1};
    float least = 0.f;
    for (const bool large : {false, true}) {
        const int tiles = wide_tiles(large, N / 16, rows);
        for (int J = 1; J <= std::min(kPrefillMaxSlices, groups); ++J) {
            if (J > 1 && tiles * J * (large ? 4 : 1) > kPrefillMaxSplit) break;
            const float c = wide_cost(large, J, tiles, groups);
            if ((!large && J == 1) || c < least) { least = c; best = WidePlan{large, J}; }
        }
    }
    return best;
}
size_t wide_partial_bytes(int N, int K, int max_rows) {
    size_t worst = 0;
    for (int rows = 64;; rows += 64) {                    // (a plan depends on ceil(rows / 64) alone)
        const WidePlan p = wide_plan(N, K, rows);
        if (p.slices > 1) worst = std::max(worst, (size_t)wide_tiles(p.large, N / 16, rows) * p.slices * (p.large ? 128 : 32) * 1024);
        if (rows >= max_rows) return worst;
    }
}
int wide_ssq_parts(int N, int K, int rows) { return wide_plan(N, K, rows).large ? (N / 16 + 7) / 8 : (N / 16 + 3) / 4; }
int wide_out_chunk(int N, int K, int rows, int epilogue) { return epilogue == EPI_SWIGLU && !wide_plan(N, K, rows).large ? 2 : 4; }

static hipError_t launch_wide_gemm_as(const WideGemmArgs &a, int epilogue, WidePlan plan, hipStream_t stream) {
    if (a.N % 16 != 0 || a.rows < 1 || a.rows > kPrefillRows || (a.chunk != 2 && a.chunk != 4)) return hipErrorInvalidValue;
    if (epilogue == EPI_RESIDUAL && a.gain_next && a.N % 32 != 0) return hipErrorInvalidValue;
    WideGemmKernelArgs k;
    k.W = (const uint4 *)a.W; k.w_factor = a.w_factor; k.X = (const uint4 *)a.X; k.x_scale = a.x_scale;
    k.KS = (a.K + 31) / 32; k.n_tiles = a.N / 16; k.n_rt = (a.rows + 15) / 16; k.rows = a.rows;
    k.Y = a.Y; k.ldy = a.ldy;
    k.ssq_in = a.ssq_in; k.ssq_ld = a.ssq_ld; k.ssq_parts = a.ssq_parts;
    k.inv_d = 1.0f / (float)a.K; k.eps = a.eps;
    k.gain_next = a.gain_next; k.ssq_out = a.ssq_out;
    k.Xout = (uint16_t *)a.Xout; k.xout_scale = a.xout_scale;
    k.KS_out = ((epilogue == EPI_SWIGLU ? a.N / 2 : a.N) + 31) / 32;
    const int out_chunk = epilogue == EPI_SWIGLU && !plan.large ? 2 : 4;
    k.NB_out = (k.KS_out + out_chunk - 1) / out_chunk;
    k.J = a.partials && a.arrive ? plan.slices : 1;
    if (k.J > 1 && wide_tiles(plan.large, k.n_tiles, a.rows) * k.J * (plan.large ? 4 : 1) > kPrefillMaxSplit) return hipErrorInvalidValue;   // beyond the scratch
    k.partials = a.partials; k.arrive = a.arrive;
    if (plan.large) return a.chunk == 4 ? launch_wide<2, 4, 8, 2, 4, 2>(k, epilogue, stream) : launch_wide<2, 4, 8, 2, 2, 2>(k, epilogue, stream);
    return a.chunk == 4 ? launch_wide<2, 2, 4, 2, 4, 2>(k, epilogue, stream) : launch_wide<2, 2, 4, 2, 2, 2>(k, epilogue, stream);
}
hipError_t launch_wide_gemm(const WideGemmArgs &a, int epilogue, hipStream_t stream) {
    return launch_wide_gemm_as(a, epilogue, wide_plan(a.N, a.K, a.rows), stream);
}

}  // namespace spd
