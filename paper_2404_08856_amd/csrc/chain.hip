// All layers of a small decoder, up to 5 rows, in one launch.
//
// One projection or attention of a small model lasts as long as a launch: 63 launches of 3.3 to 6 us made a step of the 12-layer
// draft.  Here every (layer, stage, one or two tiles) is a workgroup of one grid, in the order of the data: QKV, attention, O, gate|up, down of
// layer 0, then of layer 1, and so on.  A workgroup brings its weights (or cached keys and values) into registers, waits for the
// vector it works on, and leaves its columns to the next stage.  Its place in the
// order is the count of workgroups that started before it, so it only ever waits for ones that have started: the first unfinished one in the
// order runs and waits for nobody, whatever else the GPU runs, and the launch ends.  (By blockIdx two such launches side by side could each hold the
// places on one XCD that the other's first unfinished workgroup needs: XCDs start workgroups in order, but each in its own.)  Later stages' workgroups that
// are resident already have their weights by the time their turn comes.
// (Waits are bounded all the same, as in the fused QKV + attention kernel.)
//
// Between two stages a value travels with its proof of arrival: 8-byte words, stored and loaded whole at device scope, that hold the
// value and the number of the layer pass (a float32 and the number, or the three bf16 terms and 16 bits of it).
// A consumer loads the words until the number fits.  That is one trip through memory per stage, where data behind a counter takes three (stores
// acknowledged, counter, data).  Words of one line come from one workgroup: parts of a line from several are merged one after the other (a line of
// sums of squares, a word from each tile, cost 1.2 us a stage, so the consumers work out 1 / rms themselves).
//
// A word's buffer is used again by the next layer.  Nobody can be late: whoever writes a stage's words of layer l + 1 has waited for words that
// depend on every workgroup of the following stage of layer l, each of which had read all its words before it wrote.  The number of a pass
// counts layers over all launches with the same count of rows, each count has buffers of its own, and every pass writes all
// words of three terms: one holds this pass's number or the one before, so 16 bits are plenty.  The number comes
// from device memory, where each launch leaves it for the next, so that a captured launch can be replayed.
//
// Bound by the stages' latency, about 2.3 us each (12-layer draft, 66 positions, from the last word written to the last word written: QKV 1.9, attention
// 2.6, O 2.0, gate|up 2.3, down 3.0), and by the count of starts at the beginning of a launch.  Whole draft step, one by one / in one launch, 12-layer draft:
// 1 sequence, 66 cached positions 240 / 171 us, 640 272 / 196, 2000 366 / 222; 3 sequences, 200 279 / 232; 5 sequences, 66 282 / 259, 300 294 / 267, 640 310 / 273, 2000
// 362 / 309; 4-layer draft: 1 sequence, 66 108 / 85, 2000 172 / 112; 4 sequences, 66 120 / 111, 300 126 / 121, 1472 166 / 142.  (With the place by blockIdx, which is not
// safe, 155 at 66 positions; with the count taken and not used 163: 8 us are the count, the rest is how a stage's workgroups spread over the CUs.)
//
// The workgroups that wait hold the registers and the LDS of nearly all CUs, so work on another stream gets its turn between two launches, where it ran beside the short kernels
// before.  40 steps of the 12-layer draft on one stream, on another (kernel by kernel / in one launch): 10 verify calls of four 7B layers, done after 4.2 / 9.5 ms (alone 4.0),
// the draft after 12.5 / 7.4; 40 accept steps 0.44 / 2.35 ms (alone 0.39), the draft 9.3 / 6.4; a second draft, both 11.2 / 7.6.
#include <algorithm>

#include "attention_core.h"
#include "gemm_core.h"

namespace spd {

typedef unsigned long long u64;

constexpr int kChainWaves = 8, kChainThreads = kChainWaves * 64;
constexpr int kChainTiles = 2;   // tiles per workgroup of QKV and gate|up

struct ChainKernelArgs {
    ChainArgs c;
    int KSd, KShd, KSf, n_qkv, n_att, n_gu, per_layer;     // K-steps; workgroups per stage (O and down: d / 16) and layer
    u64 *H1, *H2, *Q, *A, *Fw;                              // words of this count of rows: h before QKV and before gate|up (float32), q | k | v
                                                            // (float32), attention's result and the activations (terms)
    u64 *turn;                                              // number of the last pass of the launch before << 32 | workgroups of this launch that have started
    const uint16_t *E;                                      // input rows: of the embedding table, by token, or
    const int32_t *tokens;
    const float *embeds;                                    // as they are
    int M, token_stride, vocab;
};

// Columns k and k + 1 of input row `row`
__device__ __forceinline__ float2 input_pair(const ChainKernelArgs &a, int row, int k) {
    if (a.embeds) return *reinterpret_cast<const float2 *>(a.embeds + (size_t)row * a.c.d + k);
    const int token = min(max(a.tokens[(size_t)(row / a.M) * a.token_stride + row % a.M], 0), a.vocab - 1);     // never read outside the table
    const uint32_t two = *reinterpret_cast<const uint32_t *>(a.E + (size_t)token * a.c.d + k);
    return float2{bf16_lo(two), bf16_hi(two)};
}

__device__ __forceinline__ u64 load_word(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_word(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Two words next to each other per address (16-byte aligned), all of them on their way together; each word is whole, the pair need not be.  As
// inline assembly for the scope.  With two 8-byte loads per pair a step of the 12-layer draft took 159 us instead of 156.5, with 5 rows 249 instead of 231
// (places by blockIdx).
typedef __attribute__((ext_vector_type(2))) u64 u64x2_t;
__device__ __forceinline__ void load_words(const u64 *const (&at)[1], u64 (&v)[2]) {
    u64x2_t a;
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(a) : "v"(at[0]) : "memory");
    v[0] = a.x; v[1] = a.y;
}
__device__ __forceinline__ void load_words(const u64 *const (&at)[2], u64 (&v)[4]) {
    u64x2_t a, b;
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(a), "=&v"(b) : "v"(at[0]), "v"(at[1]) : "memory");
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void load_words(const u64 *const (&at)[4], u64 (&v)[8]) {
    u64x2_t a, b, c, d;
    asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\tglobal_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\t"
                 "s_waitcnt vmcnt(0)" : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d) : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]) : "memory");
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y; v[4] = c.x; v[5] = c.y; v[6] = d.x; v[7] = d.y;
}
__device__ __forceinline__ u64 float_word(float x, unsigned pass) { return (u64)pass << 32 | __float_as_uint(x); }
__device__ __forceinline__ float word_float(u64 w) { return __uint_as_float((unsigned)w); }
__device__ __forceinline__ bool float_there(u64 w, unsigned pass) { return (unsigned)(w >> 32) == pass; }
__device__ __forceinline__ u64 terms_word(float x, unsigned pass) {
    uint16_t t[kTerms];
    split3(x, t);
    return (u64)(pass << 16 | t[2]) << 32 | (unsigned)t[1] << 16 | t[0];
}
__device__ __forceinline__ bool terms_there(u64 w, unsigned pass) { return (unsigned)(w >> 48) == (pass & 0xffffu); }

// polls of one wait; after `limit` of them (or once another wait has given up) it is over, whatever has arrived
struct Patience {
    unsigned limit, n = 0;
    int *abort_flag;
    __device__ __forceinline__ Patience(const ChainArgs &c) : limit(c.spin_limit), abort_flag(c.abort_flag) {}
    __device__ __forceinline__ bool over() {
        if (++n > limit) {                                  // never in a healthy run: let everything drain
            __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        return (n & 1023) == 0 && __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
};

// q, k and v from words
struct WordRows {
    const u64 *q;
    unsigned pass;
    const ChainArgs &c;
    __device__ __forceinline__ void load(int row, size_t col, size_t half, size_t hd, bool, float (&x)[6]) const {
        const u64 *p = q + (size_t)row * 3 * hd + col;
        u64 w[6];
        Patience patience(c);
        while (true) {
            bool there = true;
#pragma unroll
            for (int i = 0; i < 6; ++i) w[i] = load_word(p + (i >> 1) * hd + (i & 1) * half);
#pragma unroll
            for (int i = 0; i < 6; ++i) there = there && float_there(w[i], pass);
            if (there || patience.over()) break;
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) x[i] = word_float(w[i]);
    }
};
struct WordsOut {
    u64 *x;
    int K;
    unsigned pass;
    __device__ __forceinline__ void store(int row, int k, float y) const { store_word(x + (size_t)row * K + k, terms_word(y, pass)); }
};

enum ChainStage { CH_QKV = 0, CH_ATT, CH_O, CH_GU, CH_DOWN };

// The row of pair p of values, `per` pairs a row
__device__ __forceinline__ int row_of(int p, int per) { return (p >= per) + (p >= 2 * per) + (p >= 3 * per) + (p >= 4 * per); }

// Pairs of input values base, base + kChainThreads, ... (P of them, all loads of a look under way together): waits for their words and puts
// three terms of each value into LDS in operand order.
template <int P>
struct Pairs {
    const u64 *at[P];
    int slot[P];                                            // of xs, in 16-bit units
    bool mine[P], padding[P];
    // pairs beyond the last one look at the last one's words; columns beyond K (which is even) are zero
    __device__ __forceinline__ Pairs(const u64 *in, int K, int per, int n_pairs, int base, int R) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int p = base + i * kChainThreads, q = min(p, n_pairs - 1), row = row_of(q, per), k = 2 * (q - row * per);
            mine[i] = p < n_pairs;
            padding[i] = k >= K;
            at[i] = in + (size_t)row * K + (padding[i] ? 0 : k);
            slot[i] = ((k >> 3) * R + row) * (kTerms * 8) + (k & 7);
        }
    }
    template <class There>
    __device__ __forceinline__ void wait(const ChainArgs &c, There there, u64 (&v)[2 * P]) const {
        Patience patience(c);
        while (true) {
            bool all = true;
            load_words(at, v);
#pragma unroll
            for (int i = 0; i < 2 * P; ++i) all &= there(v[i]);
            if (all || patience.over()) break;
        }
    }
    __device__ __forceinline__ void put(int i, unsigned t0, unsigned t1, unsigned t2, uint16_t *xs) const {
        if (!mine[i]) return;
        unsigned *dst = reinterpret_cast<unsigned *>(xs + slot[i]);
        dst[0] = t0; dst[4] = t1; dst[8] = t2;
    }
    // words of three terms
    __device__ __forceinline__ void take_terms(const ChainArgs &c, unsigned pass, uint16_t *xs) const {
        u64 v[2 * P];
        wait(c, [&](u64 w) { return terms_there(w, pass); }, v);
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const unsigned a0 = (unsigned)v[2 * i], a1 = (unsigned)(v[2 * i] >> 32), b0 = (unsigned)v[2 * i + 1], b1 = (unsigned)(v[2 * i + 1] >> 32);
            const unsigned keep = padding[i] ? 0u : ~0u;
            put(i, ((a0 & 0xffffu) | b0 << 16) & keep, (a0 >> 16 | (b0 & 0xffff0000u)) & keep, ((a1 & 0xffffu) | b1 << 16) & keep, xs);
        }
    }
    // float words of h
    __device__ __forceinline__ void take_floats(const ChainArgs &c, unsigned pass, float2 (&h)[P]) const {
        u64 v[2 * P];
        wait(c, [&](u64 w) { return float_there(w, pass); }, v);
#pragma unroll
        for (int i = 0; i < P; ++i) h[i] = float2{word_float(v[2 * i]), word_float(v[2 * i + 1])};
    }
    // the terms of h * gain, and the sum of squares of each run of 64 pairs, which is of one row (per is a multiple of 64)
    __device__ __forceinline__ void put_norm(const float2 (&h)[P], const float2 (&gain)[P], int base, uint16_t *xs, float *squares) const {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const float h0 = h[i].x, h1 = h[i].y;
            uint32_t t[kTerms];
            split3_pair(h0 * gain[i].x, h1 * gain[i].y, t);
            put(i, t[0], t[1], t[2], xs);
            const float sq = wave_sum(h0 * h0 + h1 * h1);
            if ((threadIdx.x & 63) == 0 && mine[i]) squares[(base + i * kChainThreads) >> 6] = sq;
        }
    }
};

// A launch argument as a value: a choice between two of them is otherwise made between their addresses, which puts all of them in scratch memory
template <class T>
__device__ __forceinline__ T *arg(T *p) {
    asm("" : "+s"(p));
    return p;
}

// NT tiles of a projection; K split over the waves, NB K-steps each at most
template <int NB, int NT, class Gate>
__device__ __forceinline__ void chain_project(const ChainKernelArgs &a, const int stage, const int l, const int id, const unsigned pass, Gate gate,
                                              uint16_t *xs, float (*red)[kChainWaves][kGroupRows][16], float *squares) {
    const ChainArgs &c = a.c;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr bool NORM = NT > 1;                           // QKV, gate|up
    const int n_d = c.d / 16, R = c.rows;
    const int KS = NORM ? a.KSd : stage == CH_O ? a.KShd : a.KSf;
    const int K = NORM ? c.d : stage == CH_O ? c.HD : c.F;
    const int n_tiles = stage == CH_QKV ? 3 * c.HD / 16 : stage == CH_GU ? c.F / 8 : n_d;
    const char *w_qkv = arg(c.wqkv), *w_o = arg(c.wo), *w_gu = arg(c.wgu), *w_down = arg(c.wdown);
    const char *Wb = stage == CH_QKV ? w_qkv : stage == CH_O ? w_o : stage == CH_GU ? w_gu : w_down;
    const uint4 *W = reinterpret_cast<const uint4 *>(Wb + (size_t)l * c.layer_stride) + lane;
    const int s0 = KS * w / kChainWaves, ns = KS * (w + 1) / kChainWaves - s0;
    uint4 wv[NT][NB];
#pragma unroll
    for (int t = 0; t < NT; ++t)                            // (beyond the wave's share or the matrix: some block, dropped below)
#pragma unroll
        for (int u = 0; u < NB; ++u) wv[t][u] = load_stream(W + ((size_t)min(id * NT + t, n_tiles - 1) * KS + min(s0 + u, KS - 1)) * 64);
    // epilogue element of this thread: two waves a tile, column en, row em
    const int en = lane & 15, em = (w & 1) * 4 + (lane >> 4), et = w >> 1, tile = id * NT + et;
    const bool e_in = et < NT && em < R && tile < n_tiles;
    const int col = tile * 16 + en;
    const size_t norm_stride = c.layer_stride / sizeof(float);
    const float *attn_norm = arg(c.attn_norm), *mlp_norm = arg(c.mlp_norm), *gain = (stage == CH_QKV ? attn_norm : mlp_norm) + l * norm_stride;
    const bool to_head = stage == CH_DOWN && l + 1 == c.n_layers;
    float gain_at = 0.f;
    if (to_head && e_in) gain_at = c.final_norm[col];
    u64 *h1 = arg(a.H1), *h2 = arg(a.H2), *att = arg(a.A), *act = arg(a.Fw);
    const u64 *in = stage == CH_QKV ? h1 : stage == CH_O ? att : stage == CH_GU ? h2 : act;
    const int per = KS * 16, n_pairs = R * per;
    auto take = [&](auto pairs_, int base) __attribute__((always_inline)) {
        constexpr int P = decltype(pairs_)::value;
        const Pairs<P> pairs(in, K, per, n_pairs, base + (int)threadIdx.x, R);
        if constexpr (NORM) {
            float2 g[P];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int q = min(base + (int)threadIdx.x + i * kChainThreads, n_pairs - 1);
                g[i] = *reinterpret_cast<const float2 *>(gain + 2 * (q - row_of(q, per) * per));
            }
            float2 h[P];
            if (stage == CH_QKV && l == 0) {                // the input rows themselves
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const int q = min(base + (int)threadIdx.x + i * kChainThreads, n_pairs - 1), row = row_of(q, per);
                    h[i] = input_pair(a, row, 2 * (q - row * per));
                }
            } else {
                if (base == 0) gate();
                pairs.take_floats(c, pass, h);
            }
            pairs.put_norm(h, g, base + (int)threadIdx.x, xs, squares);
        } else {
            if (base == 0) gate();
            pairs.take_terms(c, pass, xs);
        }
    };
    if (n_pairs <= kChainThreads) take(std::integral_constant<int, 1>{}, 0);
    else if (n_pairs <= 2 * kChainThreads) take(std::integral_constant<int, 2>{}, 0);
    else
        for (int base = 0; base < n_pairs; base += 4 * kChainThreads) take(std::integral_constant<int, 4>{}, base);
    // the residual: one word per epilogue thread, left two stages ago
    float residual = 0.f;
    if (!NORM && e_in && stage == CH_O && l == 0) {
        const float2 two = input_pair(a, em, col & ~1);
        residual = col & 1 ? two.y : two.x;
    } else if (!NORM && e_in) {
        const u64 *p = (stage == CH_O ? h1 : h2) + (size_t)em * c.d + col;
        Patience patience(c);
        u64 v;
        do v = load_word(p); while (!float_there(v, pass) && !patience.over());
        residual = word_float(v);
    }
    if (threadIdx.x < 8) reinterpret_cast<unsigned *>(xs)[KS * 4 * R * kTerms * 4 + (threadIdx.x & 3)] = 0u;      // a fragment of zeros
    __syncthreads();

    const int r = lane & 15, g = lane >> 4, rc = r % kGroupRows, rt = r / kGroupRows;
    const bool used = r < 15 && rc < R;
    const uint4 *xf = reinterpret_cast<const uint4 *>(xs);
    const int zero = KS * 4 * R * kTerms, mine = (g * R + rc) * kTerms + rt;
    uint4 b[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) b[u] = xf[used && u < ns ? (s0 + u) * 4 * R * kTerms + mine : zero];
    f32x4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16(wv[t][u], b[u], acc[t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float4 x = {sum_terms(acc[t][0]), sum_terms(acc[t][1]), sum_terms(acc[t][2]), sum_terms(acc[t][3])};
        if (r < kGroupRows) *reinterpret_cast<float4 *>(&red[t][w][r][4 * g]) = x;
    }
    const int er = min(em, R - 1);
    float inv = 1.0f;
    if (NORM && et < NT) {                                  // 1 / rms of row em, its runs in order
        const int n_runs = per / 64;
        float sq[8], ss = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) sq[i] = squares[er * n_runs + min(i, n_runs - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i) ss += i < n_runs ? sq[i] : 0.f;
        inv = 1.0f / sqrtf(ss * c.inv_d + c.eps);
    }
    __syncthreads();
    if (et >= NT) return;                                   // two waves finish a tile

    if (stage == CH_GU) {                                   // rows 0..7 of a tile are gate features, rows 8..15 the matching up features
        float gate_v = 0.f, up_v = 0.f;
#pragma unroll
        for (int ww = 0; ww < kChainWaves; ++ww) { gate_v += red[et][ww][er][en & 7]; up_v += red[et][ww][er][8 + (en & 7)]; }
        gate_v *= inv;
        up_v *= inv;
        if (e_in && en < 8) store_word(act + (size_t)em * c.F + tile * 8 + en, terms_word(gate_v / (1.0f + expf(-gate_v)) * up_v, pass));
        return;
    }
    float sum = 0.f;
#pragma unroll
    for (int ww = 0; ww < kChainWaves; ++ww) sum += red[et][ww][er][en];
    if (stage == CH_QKV) {
        if (e_in) store_word(a.Q + (size_t)em * 3 * c.HD + col, float_word(sum * inv, pass));
        return;
    }
    const float h = residual + sum;
    if (to_head) {                                          // what the LM head's projection reads
        const float sq = row_sum(e_in ? h * h : 0.f);
        if (!e_in) return;
        uint16_t t3[kTerms];
        split3(h * gain_at, t3);
#pragma unroll
        for (int q = 0; q < kTerms; ++q) c.x_final[xpack_index(em, col, a.KSd, q)] = t3[q];
        if (en == 0) c.ssq_final[(size_t)em * n_d + tile] = sq;
    } else if (e_in) {
        store_word((stage == CH_O ? h2 : h1) + (size_t)em * c.d + col, float_word(h, stage == CH_O ? pass : pass + 1));
    }
}

// LONG: the cached keys of a head are cut into kChainRuns runs (merged by the last workgroup to arrive) instead of its dimensions into slices of 16, all
// of which score all keys.
constexpr int kChainRuns = 4;
constexpr int chain_slices(int DH, bool LONG) { return LONG ? (DH == 128 ? 2 : 1) : DH / 16; }
template <int DH, bool LONG>
__global__ __launch_bounds__(kChainThreads, 4) void chain_kernel(ChainKernelArgs a, AttnArgs at) {
    constexpr int DS = chain_slices(DH, LONG), KSP = LONG ? kChainRuns : 1, UPI = LONG && DH == 128 ? 1 : kUnitsPerIter;
    const ChainArgs &c = a.c;
    extern __shared__ __align__(16) uint16_t xs[];                        // activations as operand fragments: [K-step][lane group][row][term][8]
    __shared__ __align__(16) float red[kChainTiles][kChainWaves][kGroupRows][16];
    __shared__ float squares[kGroupRows * 8];               // d <= 1024: at most 8 runs a row
    // This workgroup's place in the order, and the number of the pass with it.  Who starts last leaves the number for the next launch: all others have theirs.
    __shared__ u64 turn_s;
    if (threadIdx.x == 0) {
        const u64 t = __hip_atomic_fetch_add(a.turn, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((unsigned)t == gridDim.x - 1) __hip_atomic_store(a.turn, (u64)((unsigned)(t >> 32) + (unsigned)c.n_layers) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        turn_s = t;
    }
    __syncthreads();
    const int turn = __builtin_amdgcn_readfirstlane((int)(unsigned)turn_s);
    const int l = turn / a.per_layer;
    int id = turn - l * a.per_layer, stage = CH_QKV;
    const int n_d = c.d / 16;
    if (id >= a.n_qkv) { id -= a.n_qkv; stage = CH_ATT;
        if (id >= a.n_att) { id -= a.n_att; stage = CH_O;
            if (id >= n_d) { id -= n_d; stage = CH_GU;
                if (id >= a.n_gu) { id -= a.n_gu; stage = CH_DOWN; } } } }
    const unsigned pass = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(turn_s >> 32)) + 1 + (unsigned)l;     // (the words start at zero, which is no pass's number)

    // Workgroups that are here early look at one word now and then, until the stage before the one they wait for has its input
    auto gate_on = [&](const u64 *word, bool is_float, unsigned p) __attribute__((always_inline)) {
        if (threadIdx.x == 0) {
            Patience patience(c);
            while (true) {
                const u64 v = load_word(word);
                if (is_float ? float_there(v, p) : terms_there(v, p)) break;
                if (patience.over()) break;
                __builtin_amdgcn_s_sleep(4);
            }
        }
        __syncthreads();
    };
    if (stage == CH_ATT) {
        const int H = at.H, hh = id % H, ds = (id / H) % DS, ks = (id / (H * DS)) % KSP, seq = id / (H * DS * KSP);
        attention_core<DH, DS, kChainWaves, UPI, 1, KSP, false, false, true>(at, hh, ds, ks, seq, WordRows{a.Q, pass, c}, WordsOut{a.A, c.HD, pass},
                                                                              [&] { if (l > 0) gate_on(a.H1, true, pass); }, (size_t)l * c.kv_stride);
        return;
    }
    auto gate = [&] __attribute__((always_inline)) {
        const u64 *q = arg(a.Q), *att = arg(a.A), *h2 = arg(a.H2), *act = arg(a.Fw);
        gate_on(stage == CH_QKV ? act : stage == CH_O ? q : stage == CH_GU ? att : h2, stage == CH_O || stage == CH_DOWN, stage == CH_QKV ? pass - 1 : pass);
    };
    if (stage == CH_QKV || stage == CH_GU) {
        if (a.KSd <= 3 * kChainWaves) chain_project<3, kChainTiles>(a, stage, l, id, pass, gate, xs, red, squares);
        else chain_project<4, kChainTiles>(a, stage, l, id, pass, gate, xs, red, squares);
    } else {
        const int KS = stage == CH_O ? a.KShd : a.KSf;
        if (KS <= 4 * kChainWaves) chain_project<4, 1>(a, stage, l, id, pass, gate, xs, red, squares);
        else if (KS <= 8 * kChainWaves) chain_project<8, 1>(a, stage, l, id, pass, gate, xs, red, squares);
        else chain_project<12, 1>(a, stage, l, id, pass, gate, xs, red, squares);
    }
}

// From how many cached positions of the longest sequence on its keys are cut into runs.  Up to 256 every wave of a slice has one unit of keys at most.  A call's layers and
// LM head, slices / runs: 12-layer draft, 1 sequence, 300 positions 181 / 184 us, 500 190 / 186, 1000 236 / 192; 2 sequences, 300 202 / 207, 500 209 / 208; 2 rows of one, 400 204 / 208,
// 500 208 / 207; 3 rows of one, 300 235 / 238, 400 243 / 240; 4 sequences, 300 246 / 243; 5 rows, 200 245 / 240 (1 sequence) and 256 / 259 (5), 300 260 / 240 and 272 / 257.  Heads of
// 128 gain earlier (4-layer draft): 1 sequence, 300 84.8 / 85.0, 2 98.0 / 96.4, 3 108.5 / 98.8, 4 118.2 / 111.2; 3 rows of one, 300 106.3 / 95.3 (kernel by kernel 104.2).
static int chain_runs_from(int n_seqs, int rows, int dh) {
    if (rows >= (dh == 128 ? 3 : 5)) return 257;
    return 256 + 256 / (dh == 64 && rows == 2 ? n_seqs : rows);
}
// Fragments of the longest input in LDS.  Two workgroups fit a CU up to 52 KiB (kChainLdsTwo: next to 19 KiB of static LDS, heads of 64, or 27, heads of 128; 31 or 39
// with runs of keys), one beyond.  One is enough for the 4-layer draft at 4 rows (66 KiB, 66 positions: 101 us a call against 111 one by one), not at 5 (82 KiB: 121 / 112).
constexpr size_t kChainLds = 72 * 1024, kChainLdsTwo = 52 * 1024;
static size_t words_per_row(int d, int HD, int F) { return (size_t)2 * d + 4 * (size_t)HD + F; }
static size_t chain_lds(int KS, int rows) { return (size_t)KS * rows * 4 * kTerms * 16 + 16; }       // and a fragment of zeros

bool chain_shape_ok(int d, int HD, int F) { return d % 128 == 0 && d <= 1024 && HD <= 3072 && F <= 3072; }
// results and counters of the runs of up to 5 sequences (a slice's result: [8][dims] sums and 16 statistics)
static size_t run_bytes(int HD) { return (size_t)kGroupRows * kChainRuns * (8 * HD + 16 * (HD / 32)) * sizeof(float); }
size_t chain_bytes(int d, int HD, int F) {
    return 256 + (size_t)kGroupRows * (HD / 32) * sizeof(unsigned) + 256 + run_bytes(HD) + words_per_row(d, HD, F) * sizeof(u64) * (kGroupRows * (kGroupRows + 1) / 2);     // counters; words for 1 .. 5 rows
}

static int chain_steps(int d, int HD, int F) { return std::max({d, HD, F + 31}) / 32; }
int chain_rows(int d, int HD, int F) {
    int rows = chain_shape_ok(d, HD, F) ? kGroupRows : 0;
    while (rows > 0 && chain_lds(chain_steps(d, HD, F), rows) > kChainLds) --rows;
    return rows;
}
// The fifth row: where QKV, gate|up and O still see all their inputs in one look (4 pairs a thread, 4096 values); each further look is a trip more.  5 rows, 66 positions, 4 layers, one
// launch / one by one: d = 768, 12 heads of 64, ffn 2304 77 / 89 us (1 sequence) and 84 / 96 (5); d = 896, 14 heads, ffn 2048 103 / 85 and 106 / 92; d = 1024, 16 heads 105 / 86 and
// 108 / 93; d = 768, 18 heads 91 / 85; d = 512, 24 heads 90 / 87.
// Attention cuts each head into workgroups of 16 dimensions that all score all keys (one by one it takes fewer where there are many pairs of sequence and head): worth it
// while they leave places free.  One launch / one by one, 4 layers, 66 and 640 positions: d = 512, ffn 2048, heads of 128: 16, 3 sequences (384 workgroups) 0.93 and 0.91, 4 (512) 1.02
// and 1.11, 5 (640) 1.21 and 1.17; 24, 3 sequences (576) 1.12 and 1.06; d = 256, 24 heads of 64, ffn 1024: 4 sequences (384) 0.89 and 0.84, 5 (480) 1.03 and 0.94;
// one workgroup per CU: 4-layer draft, 4 sequences (256) 0.92 and 0.89, d = 512, 24 heads of 128, 2 sequences of 2 rows (384) 0.99 and 0.95, at 300 positions 1.05.
// Over a long cache the runs of keys make up for the one and, with heads of 64, for some of the other: 1000 and 2000 positions, 5 rows of one sequence, d = 1024, 16 heads of 64 0.93 and
// 0.82, d = 512, 16 heads of 128 0.87 and 0.75; 24 heads of 64, 5 sequences (480), d = 768 0.88 and 0.87; 16 heads of 128, 4 sequences (512) 1.07 and 1.10.
bool chain_pays(int d, int HD, int F, int dh, int n_seqs, int M, int longest) {
    const int rows = n_seqs * M, groups = n_seqs * (HD / 16);
    const bool long_cache = longest >= 1000;
    if (rows > chain_rows(d, HD, F) || (rows == kGroupRows && rows * std::max(d, HD) > 8 * kChainThreads && !long_cache)) return false;
    if (long_cache && dh == 64) return groups <= 512;
    return groups <= (chain_lds(chain_steps(d, HD, F), rows) <= kChainLdsTwo ? 384 : 256);
}
bool chain_supported(int d, int HD, int F, int dh) {
    for (const void *f : {dh == 128 ? (const void *)chain_kernel<128, false> : (const void *)chain_kernel<64, false>,
                          dh == 128 ? (const void *)chain_kernel<128, true> : (const void *)chain_kernel<64, true>})
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kChainLds) != hipSuccess) return false;
    return chain_rows(d, HD, F) > 0;
}

hipError_t launch_chain(const ChainArgs &c, const AttnArgs &given, int longest, const void *embed_bf16, const int32_t *tokens, int token_stride, const float *embeds, int vocab, hipStream_t stream) {
    AttnArgs t = given;
    if (c.rows < 1 || c.rows > chain_rows(c.d, c.HD, c.F) || t.M < 1 || t.M * t.n_seqs != c.rows || t.m0 != 0 || t.Mq != t.M) return hipErrorInvalidValue;
    if ((t.dh != 64 && t.dh != 128) || t.H * t.dh != c.HD || (t.v_stride % 32) != 0 || t.v_stride < t.max_positions || t.M > t.max_positions) return hipErrorInvalidValue;
    if ((!tokens) == (!embeds) || token_stride < t.M || c.n_layers < 1 || c.d % 32 || c.HD % 32 || c.F % 8 || c.layer_stride % 256) return hipErrorInvalidValue;
    const bool runs = longest >= chain_runs_from(t.n_seqs, c.rows, t.dh);
    ChainKernelArgs k;
    k.c = c;
    k.KSd = c.d / 32; k.KShd = c.HD / 32; k.KSf = (c.F + 31) / 32;
    k.n_qkv = (3 * c.HD / 16 + kChainTiles - 1) / kChainTiles; k.n_att = t.n_seqs * t.H * chain_slices(t.dh, runs) * (runs ? kChainRuns : 1); k.n_gu = (c.F / 8 + kChainTiles - 1) / kChainTiles;
    k.per_layer = k.n_qkv + k.n_att + k.n_gu + 2 * (c.d / 16);
    t.arrive = (unsigned *)((char *)c.words + 256);
    t.partials = (float *)((char *)c.words + 512 + (size_t)kGroupRows * (c.HD / 32) * sizeof(unsigned) / 256 * 256);
    u64 *p = (u64 *)((char *)t.partials + run_bytes(c.HD)) + words_per_row(c.d, c.HD, c.F) * (c.rows * (c.rows - 1) / 2);
    auto take = [&](size_t per_row) { u64 *q = p; p += per_row * c.rows; return q; };
    k.H1 = take(c.d); k.H2 = take(c.d); k.Q = take(3 * c.HD); k.A = take(c.HD); k.Fw = take(c.F);
    k.turn = (u64 *)c.words + (c.rows - 1);
    k.E = (const uint16_t *)embed_bf16; k.tokens = tokens; k.embeds = embeds; k.M = t.M; k.token_stride = token_stride; k.vocab = vocab;
    const size_t lds = chain_lds(std::max({k.KSd, k.KShd, k.KSf}), c.rows);
    const dim3 grid((unsigned)k.per_layer * c.n_layers), block(kChainThreads);
    if (t.dh == 128 && runs) hipLaunchKernelGGL((chain_kernel<128, true>), grid, block, lds, stream, k, t);
    else if (t.dh == 128) hipLaunchKernelGGL((chain_kernel<128, false>), grid, block, lds, stream, k, t);
    else if (runs) hipLaunchKernelGGL((chain_kernel<64, true>), grid, block, lds, stream, k, t);
    else hipLaunchKernelGGL((chain_kernel<64, false>), grid, block, lds, stream, k, t);
    return hipGetLastError();
}

}  // namespace spd
