// Speculative sampling on the device: softmax statistics of logit rows, the accept
// test u * D(d) < T(d), the residual max(0, T - D) and the fixed-point inverse-CDF
// sampler that draws the replacement / bonus token (and the draft's own samples).
//
// Fixed-point sampler: w(x) = floor(r(x) * 2^32) as 64-bit integers, S = sum w (integer,
// so independent of the reduction tree), threshold = floor(k_u * S / 2^24) with
// k_u = u * 2^24, result = first x whose inclusive running sum exceeds the threshold.
// Every decision after the float32 probabilities is integer arithmetic, which is what
// makes the result reproducible bit for bit by any other implementation.
#include <atomic>

#include "launch.h"

namespace spd {

constexpr int kSampThreads = 1024;

struct RowStats { float mx; float sum; int argmax; int pad; };

// Numerator of the softmax: exp((l - max) / temp) through the hardware exponential (relative
// error about |argument| * 6e-8).  Statistics, accept test, residual and the draft's D row all
// use this one function, so the probabilities of a row are consistent with its sum.
__device__ __forceinline__ float softmax_num(float l, float mx, float inv_temp) { return __expf((l - mx) * inv_temp); }

__device__ __forceinline__ unsigned long long join_u64(unsigned lo, unsigned hi) { return ((unsigned long long)hi << 32) | lo; }
// Sum over the wave, on every lane, and inclusive prefix sum over the lanes, without a trip through LDS (integers: any order)
template <int N = 32>
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
    v += join_u64(lane_xor<N>((unsigned)v), lane_xor<N>((unsigned)(v >> 32)));
    if constexpr (N > 1) v = wave_sum_u64<N / 2>(v);
    return v;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_from_below(unsigned long long v) {    // 0 where no lane is below, and outside ROWS
    return join_u64((unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROWS, 0xf, false),
                    (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ unsigned long long wave_scan_u64(unsigned long long v) {
    v += dpp_from_below<0x111, 0xf>(v);                       // 1, 2, 4, 8 lanes below in the row of 16
    v += dpp_from_below<0x112, 0xf>(v);
    v += dpp_from_below<0x114, 0xf>(v);
    v += dpp_from_below<0x118, 0xf>(v);
    v += dpp_from_below<0x142, 0xa>(v);                       // last lane of rows 0 and 2 to rows 1 and 3
    v += dpp_from_below<0x143, 0xc>(v);                       // last lane of row 1 to rows 2 and 3
    return v;
}

// Exclusive prefix sum of one value per thread over the whole workgroup (1024 threads);
// *total receives the workgroup sum.  `tmp` = 17 x u64 of shared memory.
__device__ unsigned long long block_exclusive_scan(unsigned long long v, unsigned long long *tmp,
                                                   unsigned long long *total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long incl = wave_scan_u64(v);
    __syncthreads();                      // tmp may still be in use by a previous call
    if (lane == 63) tmp[w] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long run = 0;
        for (int i = 0; i < kSampThreads / 64; ++i) { unsigned long long t = tmp[i]; tmp[i] = run; run += t; }
        tmp[16] = run;
    }
    __syncthreads();
    *total = tmp[16];
    return tmp[w] + incl - v;
}

// floor(r * 2^32) for r >= 0: the scale is exact (a power of two).  Below 1 -- every probability except an
// exact 1 -- the result fits 32 bits and one truncating conversion instruction gives it; the general
// float -> 64-bit conversion (a long instruction sequence) is only needed for r >= 1.
__device__ __forceinline__ unsigned long long fixed_weight(float r) {
    const float scaled = r * 4294967296.0f;
    if (__builtin_expect(r >= 1.0f, 0)) return (unsigned long long)scaled;
    return (unsigned long long)__float2uint_rz(scaled);
}

__device__ __forceinline__ unsigned long long threshold_of(float u, unsigned long long S) {
    unsigned long long k_u = (unsigned long long)(u * 16777216.0f);   // u is a multiple of 2^-24
    unsigned long long hi = __umul64hi(k_u, S), lo = k_u * S;
    return (hi << 40) | (lo >> 24);                           // floor(k_u * S / 2^24), 128-bit product
}

// Draw from the distribution proportional to r(x), x in [0, V).  Returns -1 if every
// weight truncates to zero.  All threads of the workgroup must call it; all get the result.
template <class F>
__device__ int sample_inverse_cdf(F r, int V, float u, unsigned long long *tmp, int *result) {
    const int C = (V + kSampThreads - 1) / kSampThreads;
    const int x0 = min(V, (int)threadIdx.x * C), x1 = min(V, x0 + C);
    unsigned long long part = 0;
    for (int x = x0; x < x1; ++x) part += fixed_weight(r(x));
    unsigned long long S;
    unsigned long long excl = block_exclusive_scan(part, tmp, &S);
    if (threadIdx.x == 0) *result = -1;
    __syncthreads();
    if (S != 0) {
        unsigned long long thr = threshold_of(u, S);
        if (excl <= thr && thr < excl + part) {               // exactly one thread
            unsigned long long run = excl;
            for (int x = x0; x < x1; ++x) {
                run += fixed_weight(r(x));
                if (run > thr) { *result = x; break; }
            }
        }
    }
    __syncthreads();
    return *result;
}

// ---------------------------------------------------------------------------------
// softmax statistics of logit rows: max, argmax (lowest index), sum exp((l - max) / temp)
// ---------------------------------------------------------------------------------
// maximum and its lowest index over the lanes N, N / 2, ... 1 away
template <int N>
__device__ __forceinline__ void argmax_over(float &mx, int &arg) {
    const float om = lane_xor<N>(mx);
    const int oa = lane_xor<N>(arg);
    if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
    if constexpr (N > 1) argmax_over<N / 2>(mx, arg);
}
__device__ void row_stats(const float *__restrict__ row, int V, float inv_temp, RowStats *out_shared) {
    // out_shared: one RowStats in shared memory, valid after the call for all threads
    __shared__ float s_mx[kSampThreads / 64];
    __shared__ int s_arg[kSampThreads / 64];
    __shared__ float s_sum[kSampThreads / 64];
    float mx = -INFINITY;
    int arg = 0x7fffffff;
    for (int x = threadIdx.x; x < V; x += blockDim.x) {
        float v = row[x];
        if (v > mx) { mx = v; arg = x; }                       // strided: first hit is the lowest index
    }
    argmax_over<32>(mx, arg);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane == 0) { s_mx[w] = mx; s_arg[w] = arg; }
    __syncthreads();
    mx = s_mx[0]; arg = s_arg[0];
    for (int i = 1; i < nw; ++i)
        if (s_mx[i] > mx || (s_mx[i] == mx && s_arg[i] < arg)) { mx = s_mx[i]; arg = s_arg[i]; }
    float sum = 0.f;
    for (int x = threadIdx.x; x < V; x += blockDim.x) sum += softmax_num(row[x], mx, inv_temp);
    sum = wave_sum(sum);
    if (lane == 0) s_sum[w] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int i = 0; i < nw; ++i) t += s_sum[i];
        out_shared->mx = mx; out_shared->sum = t; out_shared->argmax = arg; out_shared->pad = 0;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------
// Register-staged fast path: rows of up to 32768 entries are read exactly once, with coalesced 16-byte loads that are all in flight together:
// thread t holds float4 number i * 1024 + t of the row, i < kRowVec.  The generic code above
// (any vocabulary size) walks the row with dependent loads and is several times slower.
// ---------------------------------------------------------------------------------
constexpr int kRowVec = 8;

// How a row is read: entry by entry from memory, or once into registers, with or without the alignment.  Rows of no
// alignment take the registers from 12288 entries on (accept step, one sequence, 32003 entries: 45.3 us from memory, 17 in
// registers; 9001 entries 16.3 / 18.4).
enum RowKind { ROW_MEMORY, ROW_ALIGNED, ROW_QUADS };
__host__ __device__ __forceinline__ RowKind row_kind(const void *row0, const void *row1, int V) {
    if (V > kRowVec * kSampThreads * 4) return ROW_MEMORY;
    if ((V & 3) == 0 && (((uintptr_t)row0 | (uintptr_t)row1) & 15) == 0) return ROW_ALIGNED;
    return V >= 12288 ? ROW_QUADS : ROW_MEMORY;
}

// Quad q of a row (entries 4 q .. 4 q + 3), `fill` beyond its end.  ALIGNED: the row is 16-byte aligned and a multiple of 4
// long.  Otherwise it starts at any multiple of 4 bytes and may end with a part of a quad: 16-byte accesses of that
// alignment, entry by entry at the end (which costs 1 us for one sequence and 4 for 64, so the two are kept apart).
struct __attribute__((packed, aligned(4))) Quad { float x, y, z, w; };
template <bool ALIGNED>
__device__ __forceinline__ float4 load_quad(const float *__restrict__ row, int q, int V, float fill) {
    if (ALIGNED) return 4 * q < V ? reinterpret_cast<const float4 *>(row)[q] : float4{fill, fill, fill, fill};
    const int left = V - 4 * q;
    if (left >= 4) {
        const Quad v = *reinterpret_cast<const Quad *>(row + 4 * q);
        return float4{v.x, v.y, v.z, v.w};
    }
    float4 v = {fill, fill, fill, fill};
    if (left > 0) v.x = row[4 * q];
    if (left > 1) v.y = row[4 * q + 1];
    if (left > 2) v.z = row[4 * q + 2];
    return v;
}
// entries beyond the row read as `fill`
template <bool ALIGNED>
__device__ __forceinline__ void load_row(const float *__restrict__ row, int V, float fill, float4 (&v)[kRowVec]) {
#pragma unroll
    for (int i = 0; i < kRowVec; ++i) v[i] = load_quad<ALIGNED>(row, i * kSampThreads + (int)threadIdx.x, V, fill);
}

// quad (group of 4 entries) of the row that register slot i of this thread holds.  WAVE_MAJOR: every wave owns a contiguous
// run of 64 * NV quads, so that the order of the entries is wave, slot, lane (what the inverse-CDF search wants);
// otherwise slot, thread.  Both are one contiguous KiB per wave and load.
template <int NV, bool WAVE_MAJOR>
__device__ __forceinline__ int quad_of(int i) {
    return WAVE_MAJOR ? (int)(threadIdx.x >> 6) * (64 * NV) + 64 * i + (int)(threadIdx.x & 63) : i * kSampThreads + (int)threadIdx.x;
}

// softmax statistics from a row held in registers (same definition as row_stats; the argmax only where it is used)
// KEEP: above temperature 0 the numerators exp((l - max) / temp) take the place of the row's entries.
// Every thread gets the result.  Two calls may follow each other without a barrier between them: a wave writes a call's partials behind a
// barrier that the others reach after reading the same partials of the call before.
template <bool WAVE_MAJOR, bool KEEP, class Row>
__device__ RowStats row_stats_regs(Row &v, bool greedy, float inv_temp) {
    __shared__ float s_mx[kSampThreads / 64];
    __shared__ int s_arg[kSampThreads / 64];
    __shared__ float s_sum[kSampThreads / 64];
    static_assert(kSampThreads / 64 == 16, "the cross-wave steps below combine 16 partials in 16 lanes");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float mx = -INFINITY;
    int arg = 0x7fffffff;
    if (greedy) {
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) {                   // ascending x within the thread
            const int x0 = 4 * quad_of<kRowVec, WAVE_MAJOR>(i);
            const float e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (e[j] > mx) { mx = e[j]; arg = x0 + j; }
        }
        argmax_over<32>(mx, arg);
        if (lane == 0) { s_mx[w] = mx; s_arg[w] = arg; }
        __syncthreads();
        mx = s_mx[lane & 15]; arg = s_arg[lane & 15];         // 16 wave results, combined by every 16-lane group
        argmax_over<8>(mx, arg);
    } else {
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) mx = fmaxf(mx, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
        mx = wave_max(mx);
        if (lane == 0) s_mx[w] = mx;
        __syncthreads();
        mx = row_max(s_mx[lane & 15]);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < kRowVec; ++i) {                       // padding is -inf: exp gives 0
        const float4 e = {softmax_num(v[i].x, mx, inv_temp), softmax_num(v[i].y, mx, inv_temp),
                          softmax_num(v[i].z, mx, inv_temp), softmax_num(v[i].w, mx, inv_temp)};
        sum += e.x;
        sum += e.y;
        sum += e.z;
        sum += e.w;
        if constexpr (KEEP)
            if (!greedy) v[i] = e;
    }
    sum = wave_sum(sum);
    if (lane == 0) s_sum[w] = sum;
    __syncthreads();
    const float t = row_sum(s_sum[lane & 15]);                // fixed tree over the 16 wave sums
    return RowStats{mx, t, arg, 0};
}

// Inverse-CDF draw (same definition as sample_inverse_cdf) over a row, or one slice of it, whose values r >= 0 sit in
// registers in wave-major order (entries outside the slice are 0): a wave's total needs one reduction, whatever the
// number of slots; the slots are only looked at by the one wave the threshold falls into.
template <int NV>
struct SliceSampler {
    unsigned long long part[NV];        // fixed-point sum of each slot's 4 entries
    unsigned long long before;          // total of the waves before this one (valid after total())

    __device__ __forceinline__ void weigh(const float4 (&r)[NV]) {
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) top = fmaxf(top, fmaxf(fmaxf(r[i].x, r[i].y), fmaxf(r[i].z, r[i].w)));
        if (__any(top >= 1.0f)) {       // weights of 2^32 and more: the general conversion
#pragma unroll
            for (int i = 0; i < NV; ++i) part[i] = fixed_weight(r[i].x) + fixed_weight(r[i].y) + fixed_weight(r[i].z) + fixed_weight(r[i].w);
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i)
                part[i] = (unsigned long long)__float2uint_rz(r[i].x * 4294967296.0f) + __float2uint_rz(r[i].y * 4294967296.0f) +
                          __float2uint_rz(r[i].z * 4294967296.0f) + __float2uint_rz(r[i].w * 4294967296.0f);
        }
    }
    // total of the slice; all threads of the workgroup call it and get it.  tmp: 17 u64 of shared memory
    __device__ __forceinline__ unsigned long long total(unsigned long long *tmp) {
        unsigned long long v = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) v += part[i];
        v = wave_sum_u64(v);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        __syncthreads();                // tmp may still be in use by a previous call
        if (lane == 0) tmp[w] = v;
        __syncthreads();
        unsigned long long all = 0;
        before = 0;
#pragma unroll
        for (int i = 0; i < kSampThreads / 64; ++i) {
            const unsigned long long t = tmp[i];
            before = i == w ? all : before;
            all += t;
        }
        mine = v;
        return all;
    }
    // the entry (4 * quad + j, quad relative to the slice) whose running sum first exceeds thr < total(); written by
    // one thread to *result: the caller synchronises
    __device__ __forceinline__ void find(const float4 (&r)[NV], unsigned long long thr, int first_quad, int *result) const {
        if (!(before <= thr && thr < before + mine)) return;  // wave-uniform
        unsigned long long run = before, slot[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) slot[i] = wave_sum_u64(part[i]);        // side by side
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const unsigned long long t = slot[i];
            if (run <= thr && thr < run + t) {                // exactly one slot
                const unsigned long long incl = wave_scan_u64(part[i]);
                unsigned long long c = run + incl - part[i];
                if (c <= thr && thr < run + incl) {           // exactly one lane
                    const int x0 = 4 * (first_quad + quad_of<NV, true>(i));
                    const float e[4] = {r[i].x, r[i].y, r[i].z, r[i].w};
                    int found = -1;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        c += fixed_weight(e[j]);
                        if (found < 0 && c > thr) found = x0 + j;
                    }
                    *result = found;
                }
            }
            run += t;
        }
    }

  private:
    unsigned long long mine;            // this wave's total
};

// MIXED: rows are read from memory unless they are aligned themselves (only one side's are).  From 8000 entries on: 64
// sequences, whole step, all from memory / MIXED, target or draft rows not aligned: 12000 entries 31.1 / 23.2 and 29.4 / 26.7
// us, 8000 24.9 / 22.2 and 24.7 / 23.8; 4000 at temperature 0 15.4 / 16.7 and 15.5 / 17.2.
template <RowKind KIND, bool MIXED>
__global__ __launch_bounds__(kSampThreads) void accept_stats_kernel(AcceptArgs a) {
    // one workgroup per logits row: target rows first, then draft rows
    const int n_t = a.n_seqs * (a.gamma + 1);
    const int r = blockIdx.x;
    const bool is_t = r < n_t;
    if (a.flags & (is_t ? 1u : 2u)) {                         // probabilities: no statistics (but the slices' ticket starts at 0)
        if (threadIdx.x == 0) reinterpret_cast<RowStats *>(a.stats)[r].pad = 0;
        return;
    }
    const float *row = is_t ? a.target + (size_t)r * a.vocab : a.draft + (size_t)(r - n_t) * a.vocab;
    const float inv_temp = a.temperature > 0.f ? 1.0f / a.temperature : 1.0f;
    __shared__ RowStats st;
    if (KIND != ROW_MEMORY || (MIXED && ((uintptr_t)row & 15) == 0)) {
        float4 v[kRowVec];
        load_row<KIND != ROW_QUADS>(row, a.vocab, -INFINITY, v);
        const RowStats got = row_stats_regs<false, false>(v, !(a.temperature > 0.f), inv_temp);
        if (threadIdx.x == 0) reinterpret_cast<RowStats *>(a.stats)[r] = got;
    } else {
        row_stats(row, a.vocab, inv_temp, &st);
        if (threadIdx.x == 0) reinterpret_cast<RowStats *>(a.stats)[r] = st;
    }
}

// probability of token x in a row given its statistics (or the row itself if it holds probabilities)
struct RowProb {
    const float *row;
    RowStats st;
    float inv_temp;
    float inv_sum;      // 1 / st.sum (one exact division per row, one multiply per entry)
    int mode;           // 0 probabilities, 1 softmax of logits, 2 greedy one-hot
    __device__ __forceinline__ float operator()(int x) const { return of(row[x], x); }
    // probability of token x whose row entry is `value`
    __device__ __forceinline__ float of(float value, int x) const {
        if (mode == 0) return value;
        if (mode == 2) return x == st.argmax ? 1.0f : 0.0f;
        return softmax_num(value, st.mx, inv_temp) * inv_sum;
    }
};

constexpr int kMaxGamma = 63;

// Statistics of a sequence's rows and its accept tests.  Everything that does not depend on anything else is loaded
// first, then the drafted tokens' entries: two dependent round trips in all, and later readers find the statistics in LDS.
struct SeqRows {
    RowStats t[kMaxGamma + 1], d[kMaxGamma];
    int acc[kMaxGamma + 1];
};
struct SeqView {
    const AcceptArgs &a;
    SeqRows &rows;
    int seq, t_mode, d_mode;
    float inv_temp;
    __device__ __forceinline__ SeqView(const AcceptArgs &a_, SeqRows &rows_, int seq_) : a(a_), rows(rows_), seq(seq_) {
        inv_temp = a.temperature > 0.f ? 1.0f / a.temperature : 1.0f;
        t_mode = (a.flags & 1u) ? 0 : (a.temperature > 0.f ? 1 : 2);
        d_mode = (a.flags & 2u) ? 0 : (a.temperature > 0.f ? 1 : 2);
    }
    __device__ __forceinline__ RowStats *stats_t(int j) const { return reinterpret_cast<RowStats *>(a.stats) + seq * (a.gamma + 1) + j; }
    __device__ __forceinline__ RowStats *stats_d(int j) const {
        return reinterpret_cast<RowStats *>(a.stats) + a.n_seqs * (a.gamma + 1) + seq * a.gamma + j;
    }
    __device__ __forceinline__ const float *t_ptr(int j) const { return a.target + ((size_t)seq * (a.gamma + 1) + j) * a.vocab; }
    __device__ __forceinline__ const float *d_ptr(int j) const { return a.draft + ((size_t)seq * a.gamma + j) * a.vocab; }
    __device__ __forceinline__ RowProb prob(const float *row, const RowStats &st, int mode) const {
        RowProb p;
        p.row = row; p.st = st; p.inv_temp = inv_temp; p.mode = mode; p.inv_sum = 1.0f / st.sum;
        return p;
    }
    __device__ __forceinline__ RowProb t_row(int j) const { return prob(t_ptr(j), rows.t[j], t_mode); }
    __device__ __forceinline__ RowProb d_row(int j) const { return prob(d_ptr(j), rows.d[j], d_mode); }
    // accept tests: u_j * D_j(d_j) < T_j(d_j), one float32 multiply and one compare; number of leading accepts.
    // All threads of the workgroup call it.
    __device__ __forceinline__ int accepted(bool write_prob) const {
        const int G = a.gamma, j = threadIdx.x;
        if (j <= G) {
            RowStats st = {0.f, 1.f, 0, 0}, sd = {0.f, 1.f, 0, 0};
            if (t_mode != 0) st = *stats_t(j);
            if (j < G) {
                int d = a.draft_tokens[(size_t)seq * a.token_stride + j];
                if (d_mode != 0) sd = *stats_d(j);
                const float u = a.u[seq * (G + 1) + j];
                d = min(max(d, 0), a.vocab - 1);                                    // never index outside the row
                const float Tx = prob(t_ptr(j), st, t_mode)(d), Dx = prob(d_ptr(j), sd, d_mode)(d);
                rows.acc[j] = (__fmul_rn(u, Dx) < Tx) ? 1 : 0;
                if (write_prob && a.accept_prob)
                    a.accept_prob[seq * G + j] = (Dx == 0.f) ? (Tx > 0.f ? 1.0f : 0.0f) : fminf(1.0f, Tx / Dx);
                rows.d[j] = sd;
            }
            rows.t[j] = st;
        }
        __syncthreads();
        int k = 0;
        while (k < G && rows.acc[k]) ++k;
        return k;
    }
};

// The general draw, out of line: where it is a rare fallback its registers are nobody else's business.
__device__ __noinline__ int sample_row_slowly(RowProb T, int V, float u, unsigned long long *tmp, int *result) {
    return sample_inverse_cdf(T, V, u, tmp, result);
}

// Any vocabulary size: one workgroup per sequence walks the rows from memory.
__global__ __launch_bounds__(kSampThreads) void accept_decide_kernel(AcceptArgs a) {
    const int seq = blockIdx.x, G = a.gamma, V = a.vocab;
    __shared__ SeqRows rows;
    __shared__ unsigned long long tmp[17];
    __shared__ int result;
    const SeqView q(a, rows, seq);
    const float u_last = a.u[seq * (G + 1) + G];
    const int k = q.accepted(true);
    const RowProb T = q.t_row(k);
    int y = -1;
    if (k < G) {
        const RowProb D = q.d_row(k);
        y = sample_inverse_cdf([&](int x) { return fmaxf(0.0f, __fsub_rn(T(x), D(x))); }, V, u_last, tmp, &result);
    }
    if (y < 0) y = sample_inverse_cdf(T, V, u_last, tmp, &result);    // bonus row, or the residual mass truncates to zero
    if (threadIdx.x == 0) {
        a.n_accepted[seq] = k;
        a.next_token[seq] = y < 0 ? 0 : y;
    }
}

// Rows that fit the registers (see row_kind): NS workgroups per sequence, each with a slice of the row to
// draw from, read once.  Every slice adds up its fixed-point weights, publishes the total and takes a ticket; the last
// one to arrive finds the slice the threshold falls into, reads that slice again and searches it.  The totals are
// integers: the result does not depend on the number of slices.
// Totals and ticket live in the words of the row statistics nobody else uses at a temperature above 0 (argmax and
// padding): the ticket in the padding of the first target row, which the statistics kernel clears, slice total i
// behind row i + 1 of the 2 gamma rows that follow -- so NS <= 2 gamma.
// Bound by a chain of dependent round trips (statistics and tokens, drafted entries, rows, total, ticket, totals, the hit
// slice), no longer by one CU's vector instructions.
constexpr int kSlices = 4;
template <int NS, bool ALIGNED>
__global__ __launch_bounds__(kSampThreads, 4) void accept_decide_slices_kernel(AcceptArgs a) {
    constexpr int NV = kRowVec / NS;
    const int seq = blockIdx.x / NS, slice = blockIdx.x % NS, G = a.gamma, V = a.vocab;
    __shared__ SeqRows rows;
    __shared__ unsigned long long tmp[17];
    __shared__ int result;
    __shared__ int is_last;
    const SeqView q(a, rows, seq);
    const float u_last = a.u[seq * (G + 1) + G];
    const int n4 = (V + 3) >> 2, per = (n4 + NS - 1) / NS;    // quads of the row (the last one may be a part), of a slice
    float4 t[NV], d[NV];
    // (entries beyond the row: probability 0 in every mode; quads beyond the slice are cleared below)
    auto load = [&](const float *row, int mode, int sl, float4 (&v)[NV]) __attribute__((always_inline)) {
        const int q0 = sl * per, q1 = min(n4, q0 + per);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int qi = q0 + quad_of<NV, true>(i);
            v[i] = load_quad<ALIGNED>(row, qi < q1 ? qi : n4, V, ALIGNED || mode == 0 ? 0.f : -INFINITY);
        }
    };
    const int k = q.accepted(slice == 0);
    load(q.t_ptr(k), q.t_mode, slice, t);
    if (k < G) load(q.d_ptr(k), q.d_mode, slice, d);
    const RowProb T = q.t_row(k), D = k < G ? q.d_row(k) : T;
    // the values of the distribution to draw from: residual max(0, T - D), or the bonus row
    float4 r[NV];
    auto values = [&](int sl) __attribute__((always_inline)) {
        const int q0 = sl * per, q1 = min(n4, q0 + per);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int qi = q0 + quad_of<NV, true>(i), x0 = 4 * qi;
            r[i] = float4{T.of(t[i].x, x0), T.of(t[i].y, x0 + 1), T.of(t[i].z, x0 + 2), T.of(t[i].w, x0 + 3)};
            if (k < G) {
                r[i].x = fmaxf(0.0f, __fsub_rn(r[i].x, D.of(d[i].x, x0)));
                r[i].y = fmaxf(0.0f, __fsub_rn(r[i].y, D.of(d[i].y, x0 + 1)));
                r[i].z = fmaxf(0.0f, __fsub_rn(r[i].z, D.of(d[i].z, x0 + 2)));
                r[i].w = fmaxf(0.0f, __fsub_rn(r[i].w, D.of(d[i].w, x0 + 3)));
            }
            if (qi >= q1) r[i] = float4{0.f, 0.f, 0.f, 0.f};
        }
    };
    SliceSampler<NV> s;
    unsigned long long S = 0, off = 0, thr = 0;
    int hit = slice;
    for (int pass = 0;; ++pass) {                             // pass 1: the last workgroup, on the slice that was hit
        values(hit);
        s.weigh(r);
        const unsigned long long mine = s.total(tmp);
        if (pass > 0) break;
        if (NS == 1) {
            S = mine;
            thr = threshold_of(u_last, S);
            break;
        }
        // total of slice i: 8 bytes at `argmax` of row i + 1 (the target rows, then the draft rows)
        auto slot = [&](int i) { return reinterpret_cast<unsigned long long *>(&(i < G ? q.stats_t(i + 1) : q.stats_d(i - G))->argmax); };
        if (threadIdx.x == 0) {
            __hip_atomic_store(slot(slice), mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const unsigned ticket = __hip_atomic_fetch_add(reinterpret_cast<unsigned *>(&q.stats_t(0)->pad), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = ticket == NS - 1;
        }
        __syncthreads();
        if (!is_last) return;
        unsigned long long tot[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) tot[i] = __hip_atomic_load(slot(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < NS; ++i) S += tot[i];
        if (S == 0) break;
        thr = threshold_of(u_last, S);
        unsigned long long run = 0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (run <= thr && thr < run + tot[i]) { hit = i; off = run; }
            run += tot[i];
        }
        if (hit == slice) break;
        load(T.row, q.t_mode, hit, t);
        if (k < G) load(D.row, q.d_mode, hit, d);
    }
    int y = -1;
    if (S != 0) {
        if (threadIdx.x == 0) result = -1;
        __syncthreads();
        s.find(r, thr - off, hit * per, &result);
        __syncthreads();
        y = result;
    } else if (k < G) {
        y = sample_row_slowly(T, V, u_last, tmp, &result);    // residual mass truncates to zero: rare
    }
    if (threadIdx.x == 0) {
        a.n_accepted[seq] = k;
        a.next_token[seq] = y < 0 ? 0 : y;
    }
}

// The whole accept step in one launch: a workgroup per (sequence, position j) holds both rows of its position in registers,
// takes their statistics, runs its accept test and, if that rejects (or j is the bonus position), draws the token that the
// sequence goes on with should j be its first reject.  Every position leaves its answer in the words of target row j's
// statistics; then it looks at all answers of its sequence, and whoever finds them complete writes the result (the last one
// to arrive does for certain, since its own answer is acknowledged before it looks; two may, with the same values) and takes the
// answers away again.  Nobody waits, nothing needs clearing before the launch, and no row is read twice.
// An answer is the token (or kAccepted) under a mark, and its complement under another.  The marks hold the number of the call, so what calls that overlapped
// on one workspace may have left (one can take half of the other's answers away) is nobody's answer later.  Only a captured call keeps its number from replay to replay.
// Bound by one CU's vector instructions (about 64 cycles per entry and wave: 3 us) and its loads (256 KiB, 4 us).  32000 entries, draft
// length 4, graph replays, one launch / statistics and slices: draft as probabilities, 1 sequence 10.3 / 14.0 us, 32 12.8 / 15.9, 51 17.0 / 19.3; draft as logits, 51
// 19.7 / 23.6; greedy, 51 22.2 / 25.2; 1000 entries as logits, 51 13.0 / 16.2.  With a second round of workgroups: 52 sequences (260 positions) probabilities 21.1 / 21.1, logits
// 23.7 / 23.8, greedy 27.3 / 25.5, 1000 entries 19.7 / 16.3, greedy 22.9 / 18.2; 64 (320) 22.6 / 22.2, 28.0 / 26.8, 32.2 / 28.5, 20.6 / 18.0, 24.6 / 20.7.
constexpr unsigned kAnswerMark = 0xffc5a11cu, kAnswerMark2 = 0x9e3779b9u, kAccepted = 0x80000000u;    // marks of call 0, which there is not
template <bool ALIGNED>
__global__ __launch_bounds__(kSampThreads) void accept_positions_kernel(AcceptArgs a, unsigned long long call) {
    const int G = a.gamma, V = a.vocab, seq = blockIdx.x / (G + 1), j = blockIdx.x - seq * (G + 1);
    __shared__ SeqRows rows;            // (only for the view below)
    __shared__ unsigned long long tmp[17];
    __shared__ int result;
    if (threadIdx.x == 0) result = -1;                        // (barriers before it is written again)
    const SeqView q(a, rows, seq);
    const bool greedy = !(a.temperature > 0.f), bonus = j == G;
    float4 t[kRowVec], d[kRowVec];
    auto load = [&](const float *row, int mode, float4 (&v)[kRowVec]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) v[i] = load_quad<ALIGNED>(row, quad_of<kRowVec, true>(i), V, mode == 0 ? 0.f : -INFINITY);
    };
    const float *t_row = q.t_ptr(j), *d_row = bonus ? t_row : q.d_ptr(j);
    const int token = bonus ? 0 : min(max(a.draft_tokens[(size_t)seq * a.token_stride + j], 0), V - 1);     // never index outside the row
    const float u_j = a.u[seq * (G + 1) + j], u_last = a.u[seq * (G + 1) + G];
    load(t_row, q.t_mode, t);
    if (!bonus) load(d_row, q.d_mode, d);
    const float t_at = t_row[token], d_at = d_row[token];
    // probabilities in place of the entries; what the drafted token's entry becomes
    auto probabilities = [&](const float *row, int mode, float at, RowStats &stats, float4 (&v)[kRowVec]) __attribute__((always_inline)) {
        if (mode == 0) return at;
        stats = row_stats_regs<true, true>(v, greedy, q.inv_temp);
        const RowProb p = q.prob(row, stats, mode);
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) {
            const int x0 = 4 * quad_of<kRowVec, true>(i);
            if (mode == 1) v[i] = float4{v[i].x * p.inv_sum, v[i].y * p.inv_sum, v[i].z * p.inv_sum, v[i].w * p.inv_sum};
            else v[i] = float4{p.of(v[i].x, x0), p.of(v[i].y, x0 + 1), p.of(v[i].z, x0 + 2), p.of(v[i].w, x0 + 3)};
            if (x0 >= V) v[i] = float4{0.f, 0.f, 0.f, 0.f};
        }
        return p.of(at, token);
    };
    RowStats st = {0.f, 1.f, 0, 0}, sd = st;
    const float Tx = probabilities(t_row, q.t_mode, t_at, st, t);
    unsigned answer = kAccepted;
    bool accepted = false;
    if (!bonus) {
        const float Dx = probabilities(d_row, q.d_mode, d_at, sd, d);
        accepted = __fmul_rn(u_j, Dx) < Tx;                   // one float32 multiply and one compare
        if (threadIdx.x == 0 && a.accept_prob) a.accept_prob[seq * G + j] = (Dx == 0.f) ? (Tx > 0.f ? 1.0f : 0.0f) : fminf(1.0f, Tx / Dx);
#pragma unroll
        for (int i = 0; i < kRowVec; ++i)                     // residual max(0, T - D), in the target's place
            t[i] = float4{fmaxf(0.0f, __fsub_rn(t[i].x, d[i].x)), fmaxf(0.0f, __fsub_rn(t[i].y, d[i].y)),
                          fmaxf(0.0f, __fsub_rn(t[i].z, d[i].z)), fmaxf(0.0f, __fsub_rn(t[i].w, d[i].w))};
    }
    if (!accepted) {                                          // workgroup-uniform
        SliceSampler<kRowVec> s;
        s.weigh(t);
        const unsigned long long S = s.total(tmp);
        int y = -1;
        if (S != 0) {
            s.find(t, threshold_of(u_last, S), 0, &result);
            __syncthreads();
            y = result;
        } else if (!bonus) {
            y = sample_row_slowly(q.prob(t_row, st, q.t_mode), V, u_last, tmp, &result);   // residual mass truncates to zero: rare
        }
        answer = (unsigned)max(y, 0);
    }
    if (threadIdx.x >= kWave) return;
    unsigned long long *slot = reinterpret_cast<unsigned long long *>(q.stats_t(min((int)threadIdx.x, G)));
    const unsigned mark = kAnswerMark + (unsigned)call, mark2 = kAnswerMark2 + (unsigned)(call >> 32);
    auto marked = [](unsigned m, unsigned v) { return (unsigned long long)m << 32 | v; };
    if ((int)threadIdx.x == j) {
        __hip_atomic_store(slot, marked(mark, answer), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(slot + 1, marked(mark2, ~answer), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // acknowledged before any answer is looked at
    const unsigned long long w0 = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long w1 = __hip_atomic_load(slot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned got = (unsigned)w0;
    if (!__all(w0 == marked(mark, got) && w1 == marked(mark2, ~got))) return;
    const unsigned long long stops = __ballot(got != kAccepted);   // positions G and beyond stop always
    const int k = min(__ffsll((long long)stops) - 1, G);
    if ((int)threadIdx.x == k) {
        a.n_accepted[seq] = k;
        a.next_token[seq] = (int)got;
    }
    if ((int)threadIdx.x <= G) __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

size_t accept_workspace_bytes(int n_seqs, int gamma) {
    return (size_t)n_seqs * (2 * gamma + 1) * sizeof(RowStats);
}

hipError_t launch_accept(const AcceptArgs &a, hipStream_t stream) {
    if (a.gamma < 1 || a.gamma > 63) return hipErrorInvalidValue;
    const RowKind kind = row_kind(a.target, a.draft, a.vocab);
    const bool need_stats = ((a.flags & 3u) != 3u);
    // one round of workgroups, one per CU (a second one saves nothing and costs up to 6 us: see above); answers are 8-byte words
    if (kind != ROW_MEMORY && ((uintptr_t)a.stats & 7) == 0 && (long)a.n_seqs * (a.gamma + 1) <= 256) {
        static std::atomic<unsigned long long> calls{0};          // numbers calls of all threads and devices
        const unsigned long long call = calls.fetch_add(1, std::memory_order_relaxed) + 1;
        const dim3 grid(a.n_seqs * (a.gamma + 1)), block(kSampThreads);
        if (kind == ROW_ALIGNED) hipLaunchKernelGGL(accept_positions_kernel<true>, grid, block, 0, stream, a, call);
        else hipLaunchKernelGGL(accept_positions_kernel<false>, grid, block, 0, stream, a, call);
        return hipGetLastError();
    }
    if (need_stats) {
        int n_rows = a.n_seqs * (2 * a.gamma + 1);
        const dim3 grid(n_rows), block(kSampThreads);
        const bool one_aligned = a.vocab >= 8000 && (row_kind(a.target, a.target, a.vocab) == ROW_ALIGNED || row_kind(a.draft, a.draft, a.vocab) == ROW_ALIGNED);
        if (kind == ROW_ALIGNED) hipLaunchKernelGGL((accept_stats_kernel<ROW_ALIGNED, false>), grid, block, 0, stream, a);
        else if (kind == ROW_QUADS) hipLaunchKernelGGL((accept_stats_kernel<ROW_QUADS, false>), grid, block, 0, stream, a);
        else if (one_aligned) hipLaunchKernelGGL((accept_stats_kernel<ROW_MEMORY, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((accept_stats_kernel<ROW_MEMORY, false>), grid, block, 0, stream, a);
    }
    // Four slices per sequence where there are words for their totals (2 gamma of them, none without statistics or where
    // the statistics' argmax is in use; 8-byte words: a workspace aligned to single floats only keeps one slice) and where
    // they run in one round of one workgroup per CU.  Whole step, 32000 entries, 1 / 2 / 4 / 8 slices, the same inputs again
    // and again: one sequence, draft length 4, 14.8 / 14 / 13.9 / 14.5 us, 8 sequences 17.4 / 18.8 / 15.5 / 15.8, 32 19.0 /
    // 19.9 / 16.8 / 21.8; inputs that are not in any cache: 17.0 / 16 / 16.1 / 18.0, 22.0 / 22.0 / 18.9 / 19.5, 23.2 / 23.4 /
    // 20.1 / 23.1.  At 1000 entries the same order (8 sequences 16.0 / 17.7 / 14.8 / 15.0).  Two slices never paid: 96
    // sequences 26.9 / 28.4, draft length 1, 8 sequences 17.2 / 18.7.
    const bool sliced = need_stats && a.temperature > 0.f && ((uintptr_t)a.stats & 7) == 0 && 2 * a.gamma >= kSlices && (long)a.n_seqs * kSlices <= 256;
    const int ns = sliced ? kSlices : 1;
    const dim3 grid(a.n_seqs * ns), block(kSampThreads);
    if (kind == ROW_MEMORY) hipLaunchKernelGGL(accept_decide_kernel, dim3(a.n_seqs), block, 0, stream, a);
    else if (sliced && kind == ROW_ALIGNED) hipLaunchKernelGGL((accept_decide_slices_kernel<kSlices, true>), grid, block, 0, stream, a);
    else if (sliced) hipLaunchKernelGGL((accept_decide_slices_kernel<kSlices, false>), grid, block, 0, stream, a);
    else if (kind == ROW_ALIGNED) hipLaunchKernelGGL((accept_decide_slices_kernel<1, true>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((accept_decide_slices_kernel<1, false>), grid, block, 0, stream, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// draft step tail: D row = softmax(logits / temp) written out, one token drawn from it
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kSampThreads) void softmax_sample_kernel(const float *__restrict__ logits,
                                                                       size_t row_stride, int V,
                                                                       float temperature,
                                                                       const float *__restrict__ u, int u_stride,
                                                                       float *__restrict__ probs_out, size_t probs_stride,
                                                                       int32_t *__restrict__ token_out, int token_stride) {
    const int seq = blockIdx.x;
    const float *row = logits + (size_t)seq * row_stride;
    float *out = probs_out + (size_t)seq * probs_stride;
    const float u_seq = u[(size_t)seq * u_stride];
    __shared__ RowStats st;
    __shared__ unsigned long long tmp[17];
    __shared__ int result;
    const float inv_temp = temperature > 0.f ? 1.0f / temperature : 1.0f;
    RowProb p;
    p.row = row; p.inv_temp = inv_temp; p.mode = temperature > 0.f ? 1 : 2;
    int y;
    if (row_kind(row, out, V) == ROW_ALIGNED) {
        float4 v[kRowVec];
        if (threadIdx.x == 0) result = -1;                    // (several barriers before it is written again)
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) v[i] = load_quad<true>(row, quad_of<kRowVec, true>(i), V, -INFINITY);
        p.st = row_stats_regs<true, true>(v, p.mode == 2, inv_temp);
        p.inv_sum = 1.0f / p.st.sum;
#pragma unroll
        for (int i = 0; i < kRowVec; ++i) {
            const int q = quad_of<kRowVec, true>(i);
            const int x0 = 4 * q;
            if (p.mode == 1) v[i] = float4{v[i].x * p.inv_sum, v[i].y * p.inv_sum, v[i].z * p.inv_sum, v[i].w * p.inv_sum};
            else v[i] = float4{p.of(v[i].x, x0), p.of(v[i].y, x0 + 1), p.of(v[i].z, x0 + 2), p.of(v[i].w, x0 + 3)};
            if (4 * q < V) reinterpret_cast<float4 *>(out)[q] = v[i];
        }
        SliceSampler<kRowVec> s;
        s.weigh(v);
        const unsigned long long S = s.total(tmp);
        if (S != 0) s.find(v, threshold_of(u_seq, S), 0, &result);
        __syncthreads();
        y = result;
    } else {
        row_stats(row, V, inv_temp, &st);
        p.st = st; p.inv_sum = 1.0f / st.sum;
        for (int x = threadIdx.x; x < V; x += blockDim.x) out[x] = p(x);
        y = sample_inverse_cdf(p, V, u_seq, tmp, &result);
    }
    if (threadIdx.x == 0) token_out[(size_t)seq * token_stride] = y < 0 ? 0 : y;
}

hipError_t launch_softmax_sample(const float *logits, size_t row_stride, int n_seqs, int vocab,
                                 float temperature, const float *u, int u_stride, float *probs_out,
                                 size_t probs_stride, int32_t *token_out, int token_stride, hipStream_t stream) {
    hipLaunchKernelGGL(softmax_sample_kernel, dim3(n_seqs), dim3(kSampThreads), 0, stream, logits,
                       row_stride, vocab, temperature, u, u_stride, probs_out, probs_stride, token_out, token_stride);
    return hipGetLastError();
}

}  // namespace spd
