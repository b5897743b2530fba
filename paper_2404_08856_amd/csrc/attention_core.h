// RoPE + KV-cache append + causal attention of up to 8 new queries per sequence and launch over
// the cached prefix (image rows + text + already accepted tokens), on the matrix cores.  The
// queries form groups of 5 (three bf16 terms each fill 15 of the 16 operand columns); 6..8
// queries are two groups multiplied with the same cached keys.  Longer runs of new rows (the
// prefill) take several launches: a later one sees the earlier ones' rows in the cache like any
// other prefix position.
//
// One workgroup (12 waves) per (sequence, head, slice of 16 or more output dimensions).  The cached keys are cut
// into units of 32; every wave owns a contiguous run of units and walks it 2 units (64 keys)
// at a time.  All loads of an iteration -- the K rows and the V columns of the wave's keys --
// are issued before anything is computed, so for contexts up to 768 keys the whole kernel pays
// a single round trip.  Every workgroup of a head scores all keys and produces its own slice of the
// output dimensions; nothing is merged across workgroups.  K is therefore read by all slices of a
// head; they are launched so that they share an XCD, whose L2 then serves the repeats (HBM sees
// K once), and V, the other half of the bytes, is read exactly once.  Over a long cache the keys of
// a head may be cut into KSP runs instead: a workgroup then scores one run for all output
// dimensions, and the last of the KSP to arrive merges their results through memory.
//
//   scores  S[key, m] = sum_d K[key, d] q[m, d]     v_mfma_f32_16x16x32_bf16, A = 16 keys x 32 dims
//           of the bf16 cache as stored, B = q as three bf16 terms (columns m, m + 5, m + 10 of
//           query m), so S is exact up to float32 rounding of q.
//   softmax per wave with running max / sum ("online"), wavefront shuffles for the
//           reductions across the 4 lane groups.
//   output  O[d, m] = sum_key V[key, d] p[m, key]   A = 16 dims x 32 keys of the TRANSPOSED V
//           cache (keys contiguous), B = p as three bf16 terms.
// The rows of the two score tiles of a unit are assigned to keys so that each lane ends up
// with the probabilities of 8 consecutive keys, which is exactly the B-operand slot of the
// second product: no data moves between lanes.
//
// The M new keys/values (this call's own rows, causal among themselves) are handled from
// LDS with plain float32 arithmetic as one more partial; the partials (one per wave + this one)
// are merged in a fixed order.  K (after RoPE) and V are rounded to bf16 -- the cache precision -- before
// they are used, appended to the cache, and the result is written as three bf16 terms in
// B-operand order for the O projection.
#pragma once
#include "launch.h"

namespace spd {

constexpr int kAttnWaves = 12;
constexpr int kUnitsPerIter = 2;      // units of 32 keys per wave per iteration

template <bool DEV>
__device__ __forceinline__ float ldf(const float *p) {
    if (DEV) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}

// Where the new rows come from: q, k and v of row `row` at head columns j and j + half (hd: columns of q, of k, of v).  DEV: written by other
// workgroups of the same kernel, read with device-scope loads.
template <bool DEV>
struct PlainRows {
    const float *qkv;
    __device__ __forceinline__ void load(int row, size_t col, size_t half, size_t hd, bool kv, float (&x)[6]) const {
        const float *p = qkv + (size_t)row * 3 * hd + col;
        x[0] = ldf<DEV>(p); x[1] = ldf<DEV>(p + half);
        x[2] = kv ? ldf<DEV>(p + hd) : 0.f; x[3] = kv ? ldf<DEV>(p + hd + half) : 0.f;
        x[4] = kv ? ldf<DEV>(p + 2 * hd) : 0.f; x[5] = kv ? ldf<DEV>(p + 2 * hd + half) : 0.f;
    }
};
// Where the results go: value k of row `row` as three bf16 terms in B-operand order (KS K-steps)
struct PackedOut {
    uint16_t *x;
    int KS;
    __device__ __forceinline__ void store(int row, int k, float y) const {
        uint16_t t3[kTerms];
        split3(y, t3);
#pragma unroll
        for (int t = 0; t < kTerms; ++t) x[xpack_index(row, k, KS, t)] = t3[t];
    }
};

__device__ __forceinline__ f32x4_t mfma16(const uint4 &a, const uint4 &b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// Cached values, which this launch reads exactly once (and keys where K_ONCE says so): non-temporal loads.
__device__ __forceinline__ uint4 load_once(const uint4 *p) {
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    return uint4{v.x, v.y, v.z, v.w};
}

// x rounded to the nearest bf16 (ties to even), as a float
__device__ __forceinline__ float rne_bf16(float x) { return bf16_bits_to_f32(f32_to_bf16_bits(x)); }

__device__ __forceinline__ uint32_t pack2(uint16_t lo, uint16_t hi) { return (uint32_t)lo | ((uint32_t)hi << 16); }

// One (sequence, head, slice of the head dimension).  Must be called by all AW waves of the
// workgroup.
// `rows_ready()` is called by every thread after the loads of the cached keys have been issued and
// before the new rows are read: the place to wait for their producer.
// QG: query groups of 5 handled by one launch (1: up to 5 new rows per sequence, 2: up to 8; the
// cached keys are then multiplied with both groups from the same registers).
// KSP > 1: the cached keys are cut into KSP contiguous runs of units, one workgroup (index ks) each.  Every one leaves its
// unnormalised result in a.partials and takes a ticket; the last of the KSP to arrive (nobody waits) combines them in
// order.  The new rows belong to run 0.  COUNTS_ON: the counters are never cleared (KSP is a power of two, and all rounds are whole).
// cache_offset: bytes from a.k_cache and a.v_cache to the layer at hand.
// K_ONCE: non-temporal loads of the keys as well (only with DS == 1: several slices of a head share its K in L2).
// CACHED: one row whose key and value are the last ones in the cache already (the length counts them): nothing is appended,
// a score that is NaN (an infinite key on a dimension where the query is zero) leaves NaN as in the prompt's other rows, and what lies behind the end of the cache counts as zero (a weight of zero alone would not do: rolled back values may not be finite.
// For every form of the kernel: 4 registers more, 12-layer draft of 2 sequences, a case of four steps, 1057 -> 1087 us).
template <int DH, int DS, int AW, int UPI, int QG, int KSP, bool K_ONCE, bool CACHED, bool COUNTS_ON, class Rows, class Out, class ReadyFn>
__device__ __forceinline__ void attention_core(const AttnArgs &a, const int hh, const int ds, const int ks, const int seq, const Rows &rows, const Out &out_rows, ReadyFn rows_ready,
                                               const size_t cache_offset = 0) {
    constexpr int HALF = DH / 2;
    constexpr int NC = DH / 32;                   // 32-dim chunks of a key row
    constexpr int DW = DH / DS;                   // output dims of this workgroup
    constexpr int NDT = DW / 16;                  // 16-dim tiles of this workgroup
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int M = a.Mq, H = a.H;                  // queries of this launch
    int P0 = a.d_lens ? a.d_lens[seq] : a.lens.len[seq];
    const int fewest = CACHED ? 1 : 0, new_rows = CACHED ? 0 : a.M;
    if (P0 < fewest || P0 + new_rows > a.max_positions) {   // only possible with device-resident lengths
        if (a.d_error && threadIdx.x == 0) *a.d_error = 1;
        P0 = max(fewest, min(P0, a.max_positions - new_rows));
    }
    const int P = P0 + a.m0;                      // cached positions before this launch's rows
    const int row_base = seq * a.M + a.m0;        // first row of this launch in qkv / xout
    const int dim0 = ds * DW;
    const size_t pair = (size_t)seq * H + hh;
    const size_t HD = (size_t)H * DH;
    const int VS = a.v_stride;                    // positions per row of the transposed V cache
    uint16_t *Kc = (uint16_t *)((char *)a.k_cache + cache_offset) + pair * a.max_positions * DH;        // [pos][DH]
    uint16_t *Vt = (uint16_t *)((char *)a.v_cache + cache_offset) + pair * (size_t)DH * VS;             // [VS / 32][DH][32]: see launch.h

    __shared__ float qf[8][DH + 4];               // rows 4 banks apart: 8 rows are read side by side below
    __shared__ float kf[8][DH + 4];
    __shared__ float vf[8][DH];
    __shared__ uint16_t qb[QG][NC][64][8];        // q as matrix-core B operand (three bf16 terms), per query group
    __shared__ float pn[8][8];
    __shared__ float part_m[AW + 1][8];
    __shared__ float part_l[AW + 1][8];
    __shared__ float part_w[AW + 1][8];           // weights of the partials in the merge
    __shared__ float top_m[8];                    // maxima over the partials
    __shared__ float part_o[AW][8][DW];

    // ---- key units of this wave; first iteration's loads go out before anything else --------
    const int n_units = (P + 31) / 32;
    const int run0 = (n_units * ks) / KSP, run_n = (n_units * (ks + 1)) / KSP - run0;      // this workgroup's run of units
    const int u_begin = run0 + (run_n * w) / AW, u_end = run0 + (run_n * (w + 1)) / AW;

    uint4 kreg[UPI][2][NC], vreg[UPI][NDT];
    auto issue_loads = [&](int u0) {
#pragma unroll
        for (int s = 0; s < UPI; ++s) {
            const int unit = u0 + s;
            if (unit < u_end) {                                        // wave-uniform
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) {
                    int key = 32 * unit + 8 * (r >> 2) + 4 * ab + (r & 3);
                    key = min(key, P - 1);                             // stay inside the valid rows
                    const uint16_t *row = Kc + (size_t)key * DH + g * 8;
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const uint4 *src = reinterpret_cast<const uint4 *>(row + c * 32);
                        kreg[s][ab][c] = K_ONCE ? load_once(src) : *src;
                    }
                }
#pragma unroll
                for (int i = 0; i < NDT; ++i)
                    vreg[s][i] = load_once(reinterpret_cast<const uint4 *>(Vt + ((size_t)unit * DH + dim0 + 16 * i + r) * 32 + 8 * g));
            }
        }
    };
    issue_loads(u_begin);
    rows_ready();

    const bool own = !CACHED && (KSP == 1 || ks == 0);      // the new rows belong to run 0
    // ---- RoPE on q, k of the new rows; bf16 rounding of new k, v; cache append ------------
    {
        const float scale = 1.0f / sqrtf((float)DH);
        for (int idx = tid; idx < (QG == 1 ? 8 : 10) * HALF; idx += AW * 64) {      // rows 8, 9: zero columns of group 1
            const int i = idx / HALF, j = idx % HALF;
            float qa = 0.f, qc = 0.f;
            if (i < M) {
                const int pos = CACHED ? P - 1 : P + i;
                const float c = a.rope[((size_t)pos * HALF + j) * 2 + 0];
                const float s = a.rope[((size_t)pos * HALF + j) * 2 + 1];
                float x[6];
                rows.load(row_base + i, (size_t)hh * DH + j, HALF, HD, own, x);
                const float q1 = x[0], q2 = x[1], k1 = x[2], k2 = x[3], v1 = x[4], v2 = x[5];
                qa = (q1 * c - q2 * s) * scale;
                qc = (q2 * c + q1 * s) * scale;
                const uint16_t kb1 = f32_to_bf16_bits(k1 * c - k2 * s);
                const uint16_t kb2 = f32_to_bf16_bits(k2 * c + k1 * s);
                const uint16_t vb1 = f32_to_bf16_bits(v1), vb2 = f32_to_bf16_bits(v2);
                kf[i][j] = bf16_bits_to_f32(kb1);
                kf[i][j + HALF] = bf16_bits_to_f32(kb2);
                vf[i][j] = bf16_bits_to_f32(vb1);
                vf[i][j + HALF] = bf16_bits_to_f32(vb2);
                if (ds == 0 && own) {                                  // one workgroup of the head appends
                    Kc[(size_t)pos * DH + j] = kb1;
                    Kc[(size_t)pos * DH + j + HALF] = kb2;
                    Vt[((size_t)(pos >> 5) * DH + j) * 32 + (pos & 31)] = vb1;
                    Vt[((size_t)(pos >> 5) * DH + j + HALF) * 32 + (pos & 31)] = vb2;
                }
            } else if (i < 8) {
                kf[i][j] = 0.f; kf[i][j + HALF] = 0.f;
                vf[i][j] = 0.f; vf[i][j + HALF] = 0.f;
            }
            if (i < 8) {
                qf[i][j] = qa;
                qf[i][j + HALF] = qc;
            }
            // B operand: column c + 5 t of group i / 5 holds bf16 term t of q_i, c = i % 5 (rows beyond M carry zeros)
            if (i < kGroupRows * QG) {
                uint16_t t1[kTerms], t2[kTerms];
                split3(qa, t1);
                split3(qc, t2);
                const int d1 = j, d2 = j + HALF, qg = i / kGroupRows, c5 = i % kGroupRows;
#pragma unroll
                for (int t = 0; t < kTerms; ++t) {
                    qb[qg][d1 >> 5][c5 + kGroupRows * t + 16 * ((d1 & 31) >> 3)][d1 & 7] = t1[t];
                    qb[qg][d2 >> 5][c5 + kGroupRows * t + 16 * ((d2 & 31) >> 3)][d2 & 7] = t2[t];
                }
            }
        }
        for (int idx = tid; idx < QG * DH; idx += AW * 64) {          // column 15 (unused): keep it finite
            const int qg = idx / DH, dd = idx % DH;
            qb[qg][dd >> 5][15 + 16 * ((dd & 31) >> 3)][dd & 7] = 0;
        }
    }
    __syncthreads();

    // ---- cached keys on the matrix cores ----------------------------------------------------
    float m_run[QG], l_run[QG];                   // of query 5 qg + r % 5 (replicated over lane groups and terms)
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) { m_run[qg] = -INFINITY; l_run[qg] = 0.f; }
    const float sel0 = r < 5 ? 1.f : 0.f, sel1 = (r >= 5 && r < 10) ? 1.f : 0.f, sel2 = (r >= 10 && r < 15) ? 1.f : 0.f;
    f32x4_t acc_o[QG][NDT];
    uint4 qreg[QG][NC];
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) {
#pragma unroll
        for (int i = 0; i < NDT; ++i) acc_o[qg][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) qreg[qg][c] = *reinterpret_cast<const uint4 *>(&qb[qg][c][lane][0]);
    }

    for (int u0 = u_begin; u0 < u_end; u0 += UPI) {
        if (u0 != u_begin) issue_loads(u0);
        // one online-softmax step per unit of 32 keys: its K registers die after the scores, its V
        // registers after the second product, so the units' temporaries never coexist
#pragma unroll
        for (int s = 0; s < UPI; ++s) {
            const int unit = u0 + s;
            if (unit >= u_end) break;                                  // wave-uniform
#pragma unroll
            for (int qg = 0; qg < QG; ++qg) {
                float sv[2][4];
                float mx = -INFINITY;
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) {
                    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc = mfma16(kreg[s][ab][c], qreg[qg][c], acc);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        float x = acc[v];                              // summed over the three term columns of this lane's query
                        x = sum_terms_all(x, r);
                        const int key = 32 * unit + 8 * g + 4 * ab + v;    // D row 4g + v of tile ab
                        x = key < P ? x : -INFINITY;
                        sv[ab][v] = x;
                        mx = fmaxf(mx, x);
                    }
                }
                mx = max_over_rows(mx);
                const float m_new = fmaxf(m_run[qg], mx);              // finite: a unit has >= 1 valid key
                const float rescale = (m_run[qg] == -INFINITY) ? 0.f : expf(m_run[qg] - m_new);   // NaN at inf - inf
                float lsum = 0.f;
                uint32_t hv[8];
#pragma unroll
                for (int ab = 0; ab < 2; ++ab)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float p = sv[ab][v] == -INFINITY ? 0.f : exp_neg<CACHED>(sv[ab][v] - m_new);   // masked keys: 0
                        lsum += p;
                        // this lane's column carries term r / 5 of query r % 5: p, p - t0 or p - t0 - t1
                        const float r1 = p - rne_bf16(p);
                        const float r2 = r1 - rne_bf16(r1);
                        hv[4 * ab + v] = f32_to_bf16_bits(sel0 * p + sel1 * r1 + sel2 * r2);
                    }
                const uint4 pb = uint4{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16), hv[4] | (hv[5] << 16), hv[6] | (hv[7] << 16)};
                lsum = xor_step<16>(lsum, AddOp());
                lsum = xor_step<32>(lsum, AddOp());
                l_run[qg] = l_run[qg] * rescale + lsum;
                m_run[qg] = m_new;
                if constexpr (CACHED) {
                    uint32_t keep[4];                                  // of this lane's 8 positions those inside the cache
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int key = 32 * unit + 8 * g + 2 * e;
                        keep[e] = (key < P ? 0xffffu : 0u) | (key + 1 < P ? 0xffff0000u : 0u);
                    }
#pragma unroll
                    for (int i = 0; i < NDT; ++i) {
                        vreg[s][i].x &= keep[0]; vreg[s][i].y &= keep[1]; vreg[s][i].z &= keep[2]; vreg[s][i].w &= keep[3];
                    }
                }
#pragma unroll
                for (int i = 0; i < NDT; ++i) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc_o[qg][i][v] *= rescale;
                    acc_o[qg][i] = mfma16(vreg[s][i], pb, acc_o[qg][i]);
                }
            }
        }
    }
    // partial of this wave: O[dim 16 i + 4 g + v][column r]; the three term columns summed
#pragma unroll
    for (int qg = 0; qg < QG; ++qg) {
        const int m = qg * kGroupRows + r;            // query of this lane's column (rows beyond 7 do not exist)
#pragma unroll
        for (int i = 0; i < NDT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = sum_terms(acc_o[qg][i][v]);
                if (r < kGroupRows && m < 8) part_o[w][m][16 * i + 4 * g + v] = x;
            }
        if (lane < kGroupRows && m < 8) { part_m[w][m] = m_run[qg]; part_l[w][m] = l_run[qg]; }
    }

    // ---- the M new keys (causal among the new rows), float32 from LDS -----------------------
    // Two queries per wave on the first four waves: lane = quarter of the dimensions, key j, query.  (One lane per (query,
    // key) on one wave walked the dimensions in a chain of conflicting reads while every other wave waited.)
    if (!own) {
        if (tid < 8) { part_m[AW][tid] = -INFINITY; part_l[AW][tid] = 0.f; }
    } else if (w < 4) {
        const int part = lane & 3, j = (lane >> 2) & 7, m = 2 * w + (lane >> 5);
        float s = 0.f;
        if (m < M && j <= m) {
#pragma unroll
            for (int e = 0; e < DH / 4; e += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(&qf[m][part * (DH / 4) + e]);
                const float4 y = *reinterpret_cast<const float4 *>(&kf[j][part * (DH / 4) + e]);
                s += (x.x * y.x + x.y * y.y) + (x.z * y.z + x.w * y.w);
            }
        }
        s += lane_xor<1>(s);
        s += lane_xor<2>(s);
        if (m >= M || j > m) s = -INFINITY;
        float mx = s;
        mx = xor_reduce<16, 4>(mx, MaxOp());
        const float p = (mx == -INFINITY) ? 0.f : expf(s - mx);        // rows m >= M: nothing visible
        float l = p;
        l = xor_step<4>(l, AddOp());
        l = xor_step<8>(l, AddOp());
        l = xor_step<16>(l, AddOp());
        if (part == 0) {
            pn[m][j] = p;
            if (j == 0) { part_m[AW][m] = mx; part_l[AW][m] = l; }
        }
    }
    __syncthreads();

    // ---- merge the AW + 1 partials in index order, write the B operand of the O projection ----
    // The weights once per (partial, query), not once per output: exponentials in every thread were 1 us of a launch with 8
    // queries per sequence and 256 pairs.  (expf here and in the rescaling above, not exp_neg, whose lower bound would turn NaN
    // into a small weight: a score that overflowed to +inf has to leave NaN, as inf - inf does, and not plausible values)
    if (tid < (AW + 1) * 8) {
        const int p = tid >> 3, m = tid & 7;
        float mstar = -INFINITY;
#pragma unroll
        for (int i = 0; i <= AW; ++i) mstar = fmaxf(mstar, part_m[i][m]);
        const float pm = part_m[p][m];
        part_w[p][m] = (pm == -INFINITY) ? 0.f : expf(pm - mstar);
        if (p == 0) top_m[m] = mstar;
    }
    __syncthreads();
    constexpr int kPart = 8 * DW + 16;            // floats of a partial result: [8][DW] sums, 8 maxima, 8 denominators
    const size_t group = pair * DS + ds;
    float *mine = KSP > 1 ? a.partials + (group * KSP + ks) * kPart : nullptr;
    for (int idx = tid; idx < M * DW; idx += AW * 64) {
        const int m = idx / DW, dd = idx % DW;
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int p = 0; p < AW; ++p) {
            const float wg = part_w[p][m];
            den += wg * part_l[p][m];
            num += wg * part_o[p][m][dd];
        }
        if (own) {
            float o = 0.f;
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) o += pn[m][jj] * vf[jj][dim0 + dd];
            const float wg = part_w[AW][m];
            den += wg * part_l[AW][m];
            num += wg * o;
        }
        if constexpr (KSP > 1) {                                       // (a run without units: maximum -inf, sums 0)
            float *out = mine + m * DW + dd;
            __hip_atomic_store(out, num, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (dd == 0) {
                __hip_atomic_store(mine + 8 * DW + m, top_m[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(mine + 8 * DW + 8 + m, den, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            continue;
        }
        out_rows.store(row_base + m, hh * DH + dim0 + dd, num / den);
    }
    if (KSP > 1) {
        __shared__ int is_last;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // the partial result is acknowledged by memory
        __syncthreads();
        if (tid == 0) {
            const unsigned ticket = __hip_atomic_fetch_add(a.arrive + group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = (COUNTS_ON ? ticket % (unsigned)KSP : ticket) == (unsigned)(KSP - 1);
            if (is_last && !COUNTS_ON) __hip_atomic_store(a.arrive + group, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
        }
        __syncthreads();
        if (!is_last) return;
        const float *all = a.partials + group * KSP * kPart;
        for (int idx = tid; idx < M * DW; idx += AW * 64) {
            const int m = idx / DW, dd = idx % DW;
            float pm[KSP], pl[KSP], po[KSP];
#pragma unroll
            for (int p = 0; p < KSP; ++p) {
                pm[p] = ldf<true>(all + (size_t)p * kPart + 8 * DW + m);
                pl[p] = ldf<true>(all + (size_t)p * kPart + 8 * DW + 8 + m);
                po[p] = ldf<true>(all + (size_t)p * kPart + idx);
            }
            float mstar = pm[0];                                       // run 0 holds the query itself
#pragma unroll
            for (int p = 1; p < KSP; ++p) mstar = fmaxf(mstar, pm[p]);
            float num = 0.f, den = 0.f;
#pragma unroll
            for (int p = 0; p < KSP; ++p) {
                const float wg = pm[p] == -INFINITY ? 0.f : expf(pm[p] - mstar);
                den += wg * pl[p];
                num += wg * po[p];
            }
            out_rows.store(row_base + m, hh * DH + dim0 + dd, num / den);
        }
    }
}

}  // namespace spd
