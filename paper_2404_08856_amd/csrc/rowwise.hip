// Row-wise kernels of the decoder forward: the input rows (embedding gather or caller's
// embedding rows) with the first RMSNorm's operand, and buffer clearing.
#include <algorithm>

#include "launch.h"

namespace spd {

// One workgroup per input row.  Writes the float32 residual row h, the packed three-term bf16
// operand of (h * gain) for the first QKV projection, and sum(h^2) of the row
// (the RMSNorm scale itself is applied inside that projection).
constexpr int kInputThreads = 1024;       // d = 4096: one load per thread (256 threads: 5.4 us a launch of 5 rows, now 4.9; 40 rows 7.3, now 6.1)
__global__ __launch_bounds__(kInputThreads) void input_rows_kernel(const uint16_t *__restrict__ E,
                                                         const int32_t *__restrict__ tokens, int M, int token_stride,
                                                         const float *__restrict__ embeds, int d, int vocab,
                                                         const float *__restrict__ gain, float *__restrict__ h,
                                                         uint16_t *__restrict__ xpack, float *__restrict__ ssq) {
    const int row = blockIdx.x;
    const int KS = d / 32;
    const uint16_t *src_tok = nullptr;
    if (tokens) {
        // row = seq * M + i; the ids of one sequence are token_stride apart from the next one's
        int tok = tokens[(size_t)(row / M) * token_stride + row % M];
        tok = min(max(tok, 0), vocab - 1);                            // never read outside the table
        src_tok = E + (size_t)tok * d;
    }
    const float *src_row = embeds ? embeds + (size_t)row * d : nullptr;
    float *dst = h + (size_t)row * d;
    float ss = 0.f;
    for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {       // d % 32 == 0
        float4 v;
        if (src_tok) {
            uint2 p = *reinterpret_cast<const uint2 *>(src_tok + k);
            v = float4{bf16_lo(p.x), bf16_hi(p.x), bf16_lo(p.y), bf16_hi(p.y)};
        } else {
            v = *reinterpret_cast<const float4 *>(src_row + k);
        }
        *reinterpret_cast<float4 *>(dst + k) = v;
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        float4 g = *reinterpret_cast<const float4 *>(gain + k);
        float y[4] = {v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w};
        union { uint2 v; uint16_t h[4]; } term[kTerms];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint16_t t3[kTerms];
            split3(y[e], t3);
#pragma unroll
            for (int t = 0; t < kTerms; ++t) term[t].h[e] = t3[t];
        }
        // 4 consecutive k stay inside one 8-element lane slot
#pragma unroll
        for (int t = 0; t < kTerms; ++t) *reinterpret_cast<uint2 *>(xpack + xpack_index(row, k, KS, t)) = term[t].v;
    }
    ss = wave_sum(ss);
    __shared__ float part[kInputThreads / kWave];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const int waves = blockDim.x / kWave, lane = threadIdx.x;
    ss = row_sum(lane < waves ? part[lane] : 0.f);                    // at most 16 of them
    if (lane == 0) ssq[(size_t)row * (d / 16)] = ss;                  // part 0 of [rows][d / 16]
}

hipError_t launch_input_rows(const void *embed_bf16, const int32_t *tokens, int M, int token_stride,
                             const float *embeds, int rows, int d, int vocab, const float *gain, float *h,
                             void *xpack, float *ssq, hipStream_t stream) {
    if ((!tokens) == (!embeds) || M < 1 || token_stride < M) return hipErrorInvalidValue;
    hipLaunchKernelGGL(input_rows_kernel, dim3(rows), dim3(std::min(kInputThreads, (d / 4 + kWave - 1) / kWave * kWave)), 0, stream, (const uint16_t *)embed_bf16,
                       tokens, M, token_stride, embeds, d, vocab, gain, h, (uint16_t *)xpack, ssq);
    return hipGetLastError();
}

// ---- KV lengths kept on the device ---------------------------------------------------------
__global__ void lens_add_kernel(int32_t *lens, int n, int delta) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) lens[i] += delta;
}

hipError_t launch_lens_add(int32_t *lens, int n, int delta, hipStream_t stream) {
    hipLaunchKernelGGL(lens_add_kernel, dim3((n + 63) / 64), dim3(64), 0, stream, lens, n, delta);
    return hipGetLastError();
}

// End of a speculative-decoding block, one thread per sequence: emit d_1 .. d_k and y, make y the
// first token of the next verify call, hand the draft its next two inputs and roll both KV
// lengths back by the gamma - k rejected positions.
__global__ void block_commit_kernel(CommitArgs a) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= a.n_seqs) return;
    const int G = a.gamma;
    const int k = min(max(a.n_accepted[s], 0), G);
    const int y = a.next_token[s];
    int32_t *vt = a.verify_tokens + (size_t)s * (G + 1);
    if (a.out_tokens) {
        int n = a.n_out[s];
        for (int j = 0; j <= k; ++j)
            if (n + j < a.out_capacity) a.out_tokens[(size_t)s * a.out_capacity + n + j] = (j < k) ? vt[1 + j] : y;
        a.n_out[s] = min(n + k + 1, a.out_capacity);
    }
    a.draft_in[2 * s + 0] = vt[k];             // token before y: d_k, or t when nothing was accepted
    a.draft_in[2 * s + 1] = y;
    vt[0] = y;
    a.target_lens[s] -= G - k;
    a.draft_lens[s] -= G - k;
}

hipError_t launch_block_commit(const CommitArgs &a, hipStream_t stream) {
    if (a.n_seqs < 1 || a.gamma < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(block_commit_kernel, dim3((a.n_seqs + 63) / 64), dim3(64), 0, stream, a);
    return hipGetLastError();
}

// ---- KV cache read-out (inspection: tests, the benchmark's CPU baseline) -------------------
// K[pos][head][d] and V[pos][head][d] of one (layer, sequence) as float32, from the cache's own layouts:
// K bf16 [head][pos][dh], V bf16 [head][v_stride / 32][dh][32].
// One workgroup per (aligned unit of 32 positions, head): K rows 8 values per thread, the unit's V tile transposed
// through LDS, so that every access is whole lines (element by element through the transposed cache: 47 us for 2047
// positions of the 7B shape).
__global__ __launch_bounds__(256) void kv_export_kernel(const uint16_t *__restrict__ Kc, const uint16_t *__restrict__ Vt, int H, int dh, int max_positions,
                                                        int pos0, int n, float *__restrict__ k_out, float *__restrict__ v_out) {
    __shared__ uint16_t tile[128][34];                      // [dim][position in the unit], 17 words a row: no bank conflicts
    const int h = blockIdx.x, unit = pos0 / 32 + blockIdx.y, d8 = dh / 8;
    const size_t ld = (size_t)H * dh;
    const uint16_t *vt = Vt + ((size_t)h * ((max_positions + 31) / 32) + unit) * dh * 32;
    for (int i = threadIdx.x; i < dh * 4; i += 256) {       // 8 positions of one dimension
        const uint4 q = reinterpret_cast<const uint4 *>(vt)[i];
        uint32_t *dst = reinterpret_cast<uint32_t *>(&tile[i >> 2][8 * (i & 3)]);
        dst[0] = q.x; dst[1] = q.y; dst[2] = q.z; dst[3] = q.w;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * d8; i += 256) {      // 8 dimensions of one position
        const int p = i / d8, d = 8 * (i % d8), pos = 32 * unit + p;
        if (pos < pos0 || pos >= pos0 + n) continue;
        const size_t o = (size_t)(pos - pos0) * ld + (size_t)h * dh + d;
        const uint4 k = *reinterpret_cast<const uint4 *>(Kc + ((size_t)h * max_positions + pos) * dh + d);
        float4 a = {bf16_lo(k.x), bf16_hi(k.x), bf16_lo(k.y), bf16_hi(k.y)}, b = {bf16_lo(k.z), bf16_hi(k.z), bf16_lo(k.w), bf16_hi(k.w)};
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = bf16_bits_to_f32(tile[d + e][p]);
        if ((((uintptr_t)k_out | (uintptr_t)v_out) & 15) == 0) {
            *reinterpret_cast<float4 *>(k_out + o) = a;
            *reinterpret_cast<float4 *>(k_out + o + 4) = b;
            *reinterpret_cast<float4 *>(v_out + o) = float4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<float4 *>(v_out + o + 4) = float4{v[4], v[5], v[6], v[7]};
        } else {                                            // outputs aligned to single floats only
            const float k8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) { k_out[o + e] = k8[e]; v_out[o + e] = v[e]; }
        }
    }
}

hipError_t launch_kv_export(const void *k_cache, const void *v_cache, int H, int dh, int max_positions, int pos0, int n,
                            float *k_out, float *v_out, hipStream_t stream) {
    if (n < 1 || pos0 < 0 || pos0 + n > max_positions || (dh != 64 && dh != 128)) return hipErrorInvalidValue;
    const int units = (pos0 + n - 1) / 32 - pos0 / 32 + 1;
    hipLaunchKernelGGL(kv_export_kernel, dim3(H, units), dim3(256), 0, stream, (const uint16_t *)k_cache, (const uint16_t *)v_cache, H, dh,
                       max_positions, pos0, n, k_out, v_out);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(uint4 *p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = uint4{0, 0, 0, 0};
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t stream) {
    size_t n16 = bytes / 16;                                           // callers pass multiples of 16
    if (n16 == 0) return hipSuccess;
    unsigned grid = (unsigned)((n16 + 255) / 256);
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, stream, (uint4 *)p, n16);
    return hipGetLastError();
}

}  // namespace spd
