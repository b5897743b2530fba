// Stand-alone attention kernel: RoPE + KV-cache append + causal attention (see attention_core.h).
#include "attention_core.h"

namespace spd {

constexpr int kXcds = 8;

// The share of a prefetching workgroup (index `id` >= `own` of `all`): of the tiles of its XCD, over all matrices, every n-th
// for the n prefetching workgroups on that XCD; read and dropped.
template <int THREADS>
__device__ __forceinline__ void prefetch_tiles(const WeightPrefetch &pf, int id, int own, int all) {
    const int xcd = id % kXcds, first = own + (xcd - own % kXcds + kXcds) % kXcds;
    const int n = (all - first + kXcds - 1) / kXcds;
    int at = (id - first) / kXcds;                          // position in the run of this XCD's tiles
    for (int k = 0; k < pf.n; ++k) {
        const int mine = (pf.m[k].tiles - xcd + kXcds - 1) / kXcds;
        for (; at < mine; at += n) {
            const uint4 *src = reinterpret_cast<const uint4 *>((const char *)pf.m[k].w + (size_t)(xcd + kXcds * at) * pf.m[k].tile_bytes);
            const int quads = pf.m[k].tile_bytes / 16;
            for (int o = threadIdx.x; o < quads; o += 4 * THREADS) {
                uint4 v[4];                                 // four loads under way (beyond the tile: its last quad again)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = src[min(o + i * THREADS, quads - 1)];
#pragma unroll
                for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(v[i].x), "v"(v[i].y), "v"(v[i].z), "v"(v[i].w));
            }
        }
        at -= mine;
    }
}

// grid: heads, slices x runs of keys, sequences (and planes of prefetching workgroups behind them)
template <int DH, int DS, int AW, int QG, int KSP, bool K_ONCE, bool CACHED = false>
__global__ __launch_bounds__(AW * 64) void attention_kernel(AttnArgs a, WeightPrefetch pf) {
    if ((int)blockIdx.z >= a.n_seqs) {
        const int id = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        prefetch_tiles<AW * 64>(pf, id, gridDim.x * gridDim.y * a.n_seqs, gridDim.x * gridDim.y * gridDim.z);
        return;
    }
    // head index fastest: consecutive workgroups go to consecutive XCDs, so with a head count that is
    // a multiple of 8 all slices of one head share an XCD and its L2 holds that head's K once
    attention_core<DH, DS, AW, kUnitsPerIter, QG, KSP, K_ONCE, CACHED, false>(a, blockIdx.x, KSP == 1 ? blockIdx.y : blockIdx.y % DS, KSP == 1 ? 0 : blockIdx.y / DS, blockIdx.z,
                                                                       PlainRows<false>{a.qkv}, PackedOut{(uint16_t *)a.xout, a.H * DH / 32}, [] {});
}

constexpr int kAttnRuns = 4;
// at most 64 (sequence, head) pairs; a run's result is [8][dh] sums and 16 statistics
size_t attention_partial_bytes(int dh) { return (size_t)64 * kAttnRuns * (8 * dh + 16) * sizeof(float); }

hipError_t launch_attention(const AttnArgs &a, int longest, const WeightPrefetch &pf, hipStream_t stream) {
    if (a.M < 1 || a.M > kMaxRows || (a.v_stride % 32) != 0 || a.v_stride < a.max_positions) return hipErrorInvalidValue;
    if (a.Mq < 1 || a.Mq > 8 || a.m0 < 0 || a.m0 + a.Mq > a.M || a.M > a.max_positions) return hipErrorInvalidValue;
    // A prompt's last row: 16 output dimensions per workgroup, whatever the number of heads (one layer of a whole prompt)
    if (a.row_cached) {
        if (a.M != 1) return hipErrorInvalidValue;
        if (a.dh == 128) hipLaunchKernelGGL((attention_kernel<128, 8, kAttnWaves, 1, 1, false, true>), dim3(a.H, 8, a.n_seqs), dim3(kAttnWaves * 64), 0, stream, a, WeightPrefetch{});
        else if (a.dh == 64) hipLaunchKernelGGL((attention_kernel<64, 4, kAttnWaves, 1, 1, false, true>), dim3(a.H, 4, a.n_seqs), dim3(kAttnWaves * 64), 0, stream, a, WeightPrefetch{});
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // Workgroups per head (slices of the head dimension).  One sequence: 16 output dimensions per
    // workgroup is fastest at the 7B shape (15.4 us per layer against 16.2 with 32 and 18.8 with 64).
    // More (sequence, head) pairs: every slice re-reads K, so slices beyond one workgroup per CU only
    // cost (8 sequences, context 2048: 73 us per layer unsliced, 76 with 2, 108 with 4, 160 with 8 slices;
    // context 640, 5 queries, 32 heads: 3 sequences 17.8 us with 2 slices against 24.2 with 4, 5 sequences
    // 22.3 unsliced against 28.9 with 2): the largest count that keeps pairs * slices within the 256 CUs.
    // a.slices (a tuning knob for tests and sweeps) overrides; 64-wide heads have at most 4 slices.
    int slices = a.slices;
    const int pairs = a.n_seqs * a.H;
    if (slices != 1 && slices != 2 && slices != 4 && slices != 8) slices = pairs > 128 ? 1 : (pairs > 64 ? 2 : (pairs > 32 ? 4 : 8));
    if (slices == 1 && a.Mq > kGroupRows) slices = 2;   // two query groups and a whole head do not fit the registers
    // up to 5 queries per sequence: one query group; 6..8: two groups share the cached keys' registers
    // Prefetching workgroups: whole (head, slice) planes of the grid, at least kPrefetchWgs together, where attention leaves at
    // least half of the CUs idle.  12-layer draft, one sequence (48 workgroups): attention 5.9 -> 6.2 us, the projections
    // behind it 18.3 -> 16.0 per layer.  Whole draft step without / with, one sequence, 12 layers: 66 cached positions 287 / 253 us,
    // 1000 350 / 316, 2000 412 / 377; two sequences 2000 415 / 387; 4 layers, one sequence 66 125 / 113, 2000 191 / 178.  4-layer draft, 8 sequences (256 workgroups): attention
    // 18.7 -> 23.0, projections 25.1 -> 20.6: nothing gained, so not there.  From the O projection's idle CUs instead: O itself
    // 1 to 3 us slower, no gain.
    constexpr int kPrefetchWgs = 192;
#define SPD_ATTN(DH_, DS_, AW_)                                                                                              \
    do {                                                                                                                     \
        const int plane = a.H * DS_;                                                                                         \
        const int planes = pf.n > 0 && plane * a.n_seqs <= 128 ? (kPrefetchWgs + plane - 1) / plane : 0;                     \
        const dim3 grid(a.H, DS_, a.n_seqs + planes);                                                                        \
        if (a.Mq <= kGroupRows)                                                                                              \
            hipLaunchKernelGGL((attention_kernel<DH_, DS_, AW_, 1, 1, false>), grid, dim3(AW_ * 64), 0, stream, a, pf);                \
        else                                                                                                                 \
            hipLaunchKernelGGL((attention_kernel<DH_, DS_, 8, 2, 1, false>), grid, dim3(8 * 64), 0, stream, a, pf);                    \
    } while (0)
    // Where 4 slices of a head would all score all keys of a long cache, its keys are cut into 4 runs instead, if they pay for the
    // exchange of the runs' results (about 4 us, more with more queries).  Per layer, runs / slices, 64 pairs: 4-layer
    // draft, one query, 512 positions 35.7 / 35.6 us, 1000 38.5 / 40.5, 2000 44.1 / 49.4; five queries, 1000 70.8 / 71.1,
    // 2000 77.1 / 80.2.  With lengths on the device only their lower bound is known: an upper bound, which grows by gamma + 1 a
    // block whatever is accepted, would put short caches through the runs (a whole draft step of that batch at 40 positions
    // 152.6 us against 142.8, at 256 156.8 / 149.4).  Two runs instead of two slices (65 to 128 pairs) gain 1 us at 1500 positions and lose 3 below 1000.
    if (a.slices == 0 && a.partials && a.arrive && pairs > 32 && pairs <= 64 && a.Mq <= kGroupRows && a.m0 == 0 && longest >= 512 + 96 * a.Mq) {
        const dim3 grid(a.H, kAttnRuns, a.n_seqs);
        if (a.dh == 128) hipLaunchKernelGGL((attention_kernel<128, 1, 8, 1, kAttnRuns, true>), grid, dim3(8 * 64), 0, stream, a, WeightPrefetch{});
        else if (a.dh == 64) hipLaunchKernelGGL((attention_kernel<64, 1, kAttnWaves, 1, kAttnRuns, true>), grid, dim3(kAttnWaves * 64), 0, stream, a, WeightPrefetch{});
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // Keys by non-temporal loads where nearly every CU holds one workgroup of a long cache.  Whole step of eight 7B layers,
    // non-temporal / plain, one query: 256 pairs, 300 positions 834 / 826 us, 700 891 / 894, 1900 1094 / 1105; 224 pairs, 300
    // 827 / 819, 1900 1069 / 1068; 160 pairs, 700 822 / 801, 1900 997 / 970; 384 pairs, 1900 1451 / 1434; five queries, 256
    // pairs, 700 1226 / 1238, 1900 1427 / 1444.  (Values so everywhere: 256 pairs, 1900 1105 against 1132.  The runs of keys above
    // too: the 4-layer draft, 8 sequences at 1472, 977 / 986 a case of five steps; two 7B sequences at 1900 go the other way, 804 / 796.)
    if (a.dh == 128 && slices == 1 && a.Mq <= kGroupRows && pairs > 224 && pairs <= 256 && longest >= 600) {
        hipLaunchKernelGGL((attention_kernel<128, 1, 8, 1, 1, true>), dim3(a.H, 1, a.n_seqs), dim3(8 * 64), 0, stream, a, WeightPrefetch{});
    } else if (a.dh == 128 && slices == 1) {
        SPD_ATTN(128, 1, 8);
    } else if (a.dh == 128 && slices == 2) {
        SPD_ATTN(128, 2, kAttnWaves);
    } else if (a.dh == 128 && slices == 4) {
        SPD_ATTN(128, 4, kAttnWaves);
    } else if (a.dh == 128) {
        SPD_ATTN(128, 8, kAttnWaves);
    } else if (a.dh == 64 && slices >= 4) {
        SPD_ATTN(64, 4, kAttnWaves);
    } else if (a.dh == 64 && slices == 2) {
        SPD_ATTN(64, 2, kAttnWaves);
    } else if (a.dh == 64) {
        SPD_ATTN(64, 1, kAttnWaves);
    } else {
        return hipErrorInvalidValue;
    }
#undef SPD_ATTN
    return hipGetLastError();
}

}  // namespace spd
