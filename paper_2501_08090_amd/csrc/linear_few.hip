// Projections of a few rows (up to 16, narrow ones up to 32).  There the weight stream is everything, and what the tiled kernel of linear.hip
// spends around it is launches: K-slices that a kernel of their own has to add up, the norm before, the rotary embedding
// behind.  Here a workgroup owns 16 or 32 output columns over the WHOLE of K: its 8 waves take an eighth of K each, add
// their accumulators through LDS, and the result is final.  So the residual stream is complete when the kernel ends, the
// next projection can take the RMS norm in its own operand load (gain on the way in, the row's 1/rms, which it learns from
// the same loads, on the way out), and the QKV projection can rotate and write the cache itself.
//
// The waves share nothing until the end: each loads its weights and its activations (fp32, from L2) straight into operand
// registers (v_mfma_f32_16x16x32_bf16, weights as A, 16 activation rows as B, two bf16 terms each), 8 k-steps of 32 ahead;
// no LDS and no barrier in the loop.  Every workgroup reads all rows of its input, which is what ends the range: at 16 rows
// the activations of a 4096-wide input are as many bytes per workgroup (256 KiB) as the weights of its 32 columns.  Where
// that is depends on the widths: see "which rows take this path" below.
//
// Measured per layer at the 8B widths and one row, against the tiled kernels with the norms and the rotary embedding as
// launches of their own: QKV 12.2 us (11.4 + 4.8 + 4.7), O 7.4 (8.2; 4.5 TB/s with the launch), gate/up with its norm 38.8
// (37.7 + 4.8), down 20.6 (19.6; 5.7 TB/s); four layers and the head 575 -> 522 us, 664 -> 623 at 11 rows.  A single
// projection of 4096 x 4096 with its K-slices summed 27 -> 7.7 us.
// Rings of 12 or 16 k-steps were slower (8.4 .. 9.0 against 7.7 us at 4096 x 4096), as bytes in flight are not what is short.
#include "chiron_internal.h"
#include "device_util.h"
#include "kv_layout.h"

namespace chiron {

constexpr int kFewWaves = 8;
constexpr int kFewRing = 8;  // k-steps of 32 in flight per wave with one row tile

// CT: 16-column tiles per workgroup.
// FEW_ROWS: A is fp32 rows.
// FEW_PACKED: A holds the two bf16 terms, [k/8][M rows][8], hi terms first (lda = distance to the lo terms in 16-byte
//   units): no conversion, and a wave's loads are contiguous pieces of 16*M bytes instead of 32 bytes of each row.
// FEW_SWIGLU: fp32 rows times a fused gate/up matrix; the result is the two terms of silu(gate) * up as FEW_PACKED reads them
//   (ldy = distance to the lo terms in 16-byte units).
// The other modes take rmsnorm(A) * gain of fp32 rows A:
// FEW_NORM: a plain projection of it.  FEW_SWIGLU_NORM: FEW_SWIGLU of it.
// FEW_QKV: the fused QKV projection of a decode step, which ends in the rotary embedding and the append to the cache.
enum FewMode { FEW_ROWS, FEW_PACKED, FEW_SWIGLU, FEW_NORM, FEW_SWIGLU_NORM, FEW_QKV };
// RT: 16-row tiles; two of them (17 .. 32 rows) leave registers for half the k-steps in flight.
template <int CT, int MODE, int RT = 1>
__global__ __launch_bounds__(64 * kFewWaves) void linear_few_kernel(const uint16_t* __restrict__ Wp, size_t tstride, int N, int K, int Kpad,
                                                                   const float* __restrict__ A, int64_t lda, int M,
                                                                   const uint16_t* __restrict__ gain, float eps,
                                                                   float* __restrict__ Y, int ldy, int add, RopeOut ro) {
    constexpr bool QKV = MODE == FEW_QKV, NORM = MODE >= FEW_NORM, SWIGLU = MODE == FEW_SWIGLU || MODE == FEW_SWIGLU_NORM;
    constexpr int D = RT == 1 ? kFewRing : kFewRing / 2;  // k-steps in flight per wave (CT KiB of weights each)
    constexpr int WS = 72;      // float4 units between the 16x16 tiles in LDS, 18 between a tile's row groups: no two
    constexpr int QS = 18;      // threads of the final sum that read at once share a bank
    __shared__ float4 s_acc[RT][kFewWaves * CT * WS];
    __shared__ float s_ss[RT][kFewWaves][16];
    static_assert(CT == 2 || (!QKV && !SWIGLU), "a rotary pair, and gate and up of a column, sit in one 32-column tile");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = lane & 15, kq = lane >> 4;
    const int ct0 = blockIdx.x * CT;  // first 16-column tile

    // this thread's output: row om, column oc of the workgroup's columns.  What the epilogue needs for it (the old value of
    // the residual stream, or a chain of dependent loads for the rotation and the slot) is fetched first and is there long
    // before the weights are.
    // With two row tiles: rows om and om + 16.
    const int om = tid / (16 * CT), oc = tid % (16 * CT);
    float cs[RT], sn[RT];
    int block[RT], slot[RT];
    const int half = QKV ? ro.pool.d / 2 : 1;
    const int hd = QKV ? (int)blockIdx.x / (ro.pool.d / 32) : 0;                          // head
    const int j = QKV ? ((int)blockIdx.x % (ro.pool.d / 32)) * 16 + (oc & 15) : 0;        // first dim of this thread's pair
    const int n_out = ct0 * 16 + oc;
    float y_old[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int m = om + 16 * r;
        cs[r] = sn[r] = y_old[r] = 0.f;
        block[r] = slot[r] = 0;
        if (QKV && m < M) {
            const int req = m / ro.q_len;
            const int ps = ro.seq_lens[req] + m % ro.q_len;
            cs[r] = ro.cos_t[(size_t)m * half + j];
            sn[r] = ro.sin_t[(size_t)m * half + j];
            block[r] = ro.bt[(size_t)req * ro.max_blocks + ps / kBlockSize];
            slot[r] = ps % kBlockSize;
        }
        if (!QKV && !SWIGLU && add && m < M && n_out < N && tid < 256 * CT) y_old[r] = Y[(size_t)m * ldy + n_out];
    }

    const int S = Kpad / (32 * kFewWaves);  // k-steps of this wave (the packed weights are zero past K)
    const int st0 = wave * S;
    // A wave walks its eighth of K from a start that differs between workgroups: with K a power of two the weight streams of
    // all workgroups would stay in step on the same memory channels (8192 x 8192, 256 workgroups: 24.1 against 21.3 us).
    const int rot = (int)(blockIdx.x / 8 * 3) % S;
    auto k_step = [&](int step) {
        const int sr = step + rot;
        return st0 + (sr >= S ? sr - S : sr);
    };
    const uint16_t* wp = Wp + (size_t)(ct0 / 2) * tstride + (size_t)((ct0 & 1) * 128) + kq * 256 + row * 8;
    const float* arow[RT];   // fp32 rows
    const uint4* apack[RT];  // packed terms
    floatx4 acc[RT][CT];
    float ss[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        arow[r] = A + (size_t)min(row + 16 * r, M - 1) * lda;
        apack[r] = reinterpret_cast<const uint4*>(A) + kq * M + min(row + 16 * r, M - 1);
#pragma unroll
        for (int t = 0; t < CT; ++t) acc[r][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        ss[r] = 0.f;
    }
    uint4 w[D][CT], g[NORM ? D : 1];
    float4 a[D][RT][2];                           // fp32 rows
    uint4 p[MODE == FEW_PACKED ? D : 1][RT][2];   // packed terms: hi, lo

    auto load = [&](int step, int s) {
        const int st = k_step(min(step, S - 1));
        const uint16_t* wk = wp + (size_t)st * 1024;
#pragma unroll
        for (int t = 0; t < CT; ++t) w[s][t] = load_stream_16(wk + t * 128);
        if (MODE == FEW_PACKED) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                p[s][r][0] = apack[r][(size_t)st * (4 * M)];
                p[s][r][1] = apack[r][(size_t)st * (4 * M) + lda];
            }
            return;
        }
        const int k = min(st * 32 + kq * 8, K - 8);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            a[s][r][0] = *reinterpret_cast<const float4*>(arow[r] + k);
            a[s][r][1] = *reinterpret_cast<const float4*>(arow[r] + k + 4);
        }
        if (NORM) g[s] = *reinterpret_cast<const uint4*>(gain + k);
    };
    auto compute = [&](int step, int s) {
        const int k0 = k_step(step) * 32;
        uint4 hi[RT], lo[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if (MODE == FEW_PACKED) {
                hi[r] = p[s][r][0];
                lo[r] = p[s][r][1];
                if (k0 + 32 > K && k0 + kq * 8 >= K) hi[r] = lo[r] = make_uint4(0, 0, 0, 0);  // the padding of K may hold any bits
                continue;
            }
            const float4 &a0 = a[s][r][0], &a1 = a[s][r][1];
            float v[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            if (k0 + 32 > K) {  // uniform: a step that reaches past K
                const bool ok = k0 + kq * 8 < K;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = ok ? v[e] : 0.f;
            }
            if (NORM) {
                const uint32_t gw[4] = {g[s].x, g[s].y, g[s].z, g[s].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    ss[r] = fmaf(v[e], v[e], ss[r]);
                    v[e] *= (e & 1) ? bf16_hi(gw[e / 2]) : bf16_lo(gw[e / 2]);
                }
            }
            split2(v[0], v[1], hi[r].x, lo[r].x);
            split2(v[2], v[3], hi[r].y, lo[r].y);
            split2(v[4], v[5], hi[r].z, lo[r].z);
            split2(v[6], v[7], hi[r].w, lo[r].w);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8*>(&w[s][t]), *reinterpret_cast<bf16x8*>(&hi[r]), acc[r][t], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8*>(&w[s][t]), *reinterpret_cast<bf16x8*>(&lo[r]), acc[r][t], 0, 0, 0);
    };

    if (S >= D) {
        // whole rings: a slot is reloaded as soon as it has been multiplied.  Loads are unconditional (past the wave's
        // last k-step they repeat it), so the number in flight is the same on every path and no wait drains the queue.
#pragma unroll
        for (int s = 0; s < D; ++s) {
            load(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        int step = 0;
        for (; step + D < S; step += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                compute(step + s, s);
                load(step + D + s, s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (step + s < S) compute(step + s, s);  // uniform
    } else {
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (s < S) load(s, s);
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (s < S) compute(s, s);
    }

    // D[i][j]: lane holds column j = lane % 16 (an activation row) and rows i = 4 * (lane / 16) + r (output columns)
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int t = 0; t < CT; ++t)
            s_acc[r][(wave * CT + t) * WS + row + kq * QS] = make_float4(acc[r][t][0], acc[r][t][1], acc[r][t][2], acc[r][t][3]);
        if (NORM) {
            ss[r] += __shfl_xor(ss[r], 16);
            ss[r] += __shfl_xor(ss[r], 32);
            if (lane < 16) s_ss[r][wave][lane] = ss[r];
        }
    }
    __syncthreads();
    if (CT == 1 && tid >= 256) return;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int m = om + 16 * r;
        const bool live = m < M;
        const float* sp = reinterpret_cast<const float*>(s_acc[r]) + (size_t)((oc / 16) * WS + om + ((oc & 15) / 4) * QS) * 4 + (oc & 3);
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < kFewWaves; ++k) v += sp[k * CT * WS * 4];
        if (NORM) {
            float tot = 0.f;
#pragma unroll
            for (int k = 0; k < kFewWaves; ++k) tot += s_ss[r][k][om];
            v *= 1.0f / sqrtf(tot / (float)K + eps);
        }
        if (QKV) {
            const float other = __shfl_xor(v, 16);  // the other half of the rotary pair (dims j and j + d/2)
            if (!live) return;
            const int hi = oc / 16, e = j + hi * half;
            // (one rounding less than two products and a sum; written out, as the compiler contracts it in some forms of this loop only)
            if (hd < ro.n_q + ro.pool.n_kv) v = fmaf(v, cs[r], hi ? other * sn[r] : -(other * sn[r]));
            if (hd < ro.n_q) {
                ro.q_out[(size_t)m * ro.n_q * 2 * half + (size_t)hd * 2 * half + e] = v;
            } else {
                const int kv = hd - ro.n_q;  // K heads, then V heads
                const bool is_v = kv >= ro.pool.n_kv;
                uint16_t* tile = ro.pool.base + tile_base(ro.pool, ro.layer, block[r], is_v ? kv - ro.pool.n_kv : kv);
                tile[is_v ? 32 * half + v_off(slot[r], e) : k_off(slot[r], e)] = f32_to_bf16_rne(v);
            }
        } else if (SWIGLU) {
            // column oc of the tile is gate (oc / 4 even) or up of column 4 * (oc / 8) + oc % 4 of its 16 (gate_up_packed_row in linear.hip)
            const float up = __shfl_xor(v, 4);
            const float act = v / (1.0f + __expf(-v)) * up;  // (in the lanes of gate columns)
            const float next = __shfl_xor(act, 1);
            if (!live || (oc & 5) != 0 || n_out >= N) continue;  // a lane of an even gate column writes its own and the next one
            uint32_t hi, lo;
            split2(act, next, hi, lo);
            const int col = (int)blockIdx.x * 16 + oc / 8 * 4 + (oc & 3);
            uint32_t* dst = reinterpret_cast<uint32_t*>(Y) + ((size_t)(col / 8) * M + m) * 4 + (col & 7) / 2;
            dst[0] = hi;
            dst[(size_t)ldy * 4] = lo;
        } else {
            if (live && n_out < N) Y[(size_t)m * ldy + n_out] = y_old[r] + v;
        }
    }
}

// ---- which rows take this path -------------------------------------------------------------------------------
bool linear_few_rows(int M) {
    const Tuning& t = tuning();
    if (M > 16 && t.linear_big_min_m > 0 && M >= t.linear_big_min_m) return false;  // as from there on the tiled two-term form is asked for
    return M <= 32 && !t.linear_mt && !t.linear_nf && !t.linear_ksplit && !t.linear_ks && !t.linear_big_all;
}

// 16-column tiles per workgroup.  Two (half as many loads of the same activations) where that takes a round of the chip less: 8192
// outputs of 28672 inputs 68 against 75 us at one row, 72 against 89 us at 8; 5120 outputs of 8192 inputs 16.1 against 21.1 and
// 19.3 against 25.6; 4096 outputs of 14336 inputs 25 against 20.  Two rounds of them against three of one (9216 columns) are
// as fast at 8 rows and faster above.
static int few_col_tiles(const Linear& L, int M) {
    const int tiles = (L.N + 15) / 16;
    return tiles > kNumCU && (tiles <= 2 * kNumCU || tiles > 3 * kNumCU || M > 8) ? 2 : 1;
}

// Time of the kernel above at M rows, in microseconds: a launch's start and end, and the longest of
//   the weight stream at 7.2 TB/s;
//   what one CU takes in, weights and activations of its workgroups: 50 GB/s (fp32 rows; 45 with the rotation behind them,
//     70 for packed terms), and 27 (one column tile) or 31 GB/s of weights for workgroups that share a CU while others idle; of two
//     column tiles in one round 42 GB/s of weights and then 95 of packed terms or 57 of fp32 rows (5120 outputs of 14336 inputs:
//     packed 26.8 us at one row, 36.5 at 16);
//   what all CUs together take in: 12 TB/s, of fp32 rows less the longer K is (10.4 at 28672), and a sixth less with two
//     column tiles if K is no multiple of 256 (16384 x 5808 and 14000 x 5008 at 16 rows: 10.0 and 9.4, 16384 x 6144: 11.5).
// The rates are fitted to single projections of 256 .. 16384 columns, K = 1024 .. 32768, and to the layers of 15 decoders of
// 256 .. 16384 hidden columns, at 1 .. 16 rows; it is within 10 % of most of them (8B widths at 16 rows: 61 against 60 us for
// QKV, O and down; 5120 wide with 40 KV heads: 119 against 126).
static double few_us(const Linear& L, int M, FewMode mode, int ct) {
    const int wgs = (L.N + 16 * ct - 1) / (16 * ct), rounds = (wgs + kNumCU - 1) / kNumCU;
    const double w = 32e-6 * ct * L.K, a = 4e-6 * M * L.K;  // MB of weights and activations per workgroup
    const double cu = mode >= FEW_NORM ? 0.045 : (mode == FEW_PACKED ? 0.070 : 0.050);  // MB/us
    const double chip = mode == FEW_PACKED ? 12.0 : (12.2 - L.K / 16000.0) * (ct == 2 && L.K % 256 ? 0.84 : 1.0);
    double t = wgs * w / 7.2;
    const auto at_least = [&](double v) { t = v > t ? v : t; };
    at_least(rounds * (w + a) / cu);
    at_least((rounds > 1 ? rounds * kNumCU : wgs) * (w + a) / chip);
    if (rounds > 1) at_least(rounds * w / (ct == 1 ? 0.027 : 0.031));
    else if (ct == 2 && mode <= FEW_PACKED) at_least(w / 0.042 + a / (mode == FEW_PACKED ? 0.095 : 0.057));
    return 4.0 + t;
}
// the tiled kernel's, whose K-slices fill the chip evenly; it hardly depends on the rows there
static double tiled_us(const Linear& L) { return 3.5 + 2e-6 * L.N * L.K / 6.6; }

// Products that the tiled kernel does not slice, with or without the norm in the operand load: gate/up and the head.  There a
// workgroup walks the whole of K in one chain of chunks (5.8 ns per k), which with fewer than a column tile per wave and CU nothing
// hides.  Up to one round of 32 columns a workgroup the few-row kernel is faster at any K (28.6 -> 10.6 us for 2816 columns
// of K = 4096 at one row, 29.9 -> 15.3 for 8192 at 16; 5.9 -> 3.1 for 512 of K = 256), in two rounds from K = 2048, and if the second
// one is more than half full only up to 8 rows (16384 columns: 17.6 -> 14.7 at 8 rows; at K = 1024 11.2 against 11.4; inside a step
// at K = 3072 and 13 rows 1 us a layer lost, at K = 2048 with 11264 columns 3 gained); beyond that the weight stream decides.
// Whole steps of two layers, 1024 wide: 92 -> 81 us at 4 rows, 102 -> 94 at 16.
static double unsliced_us(const Linear& L) {
    const double chain = 3.3 + 0.0058 * L.K;
    return chain > tiled_us(L) ? chain : tiled_us(L);
}
// From 17 rows on the activations weigh twice as much and the estimate decides, in the same range of widths (32 rows: gate/up of a
// block of 4096 x 4096 27 -> 15 us; 11264 columns of K = 2048 15 against 18).
constexpr double kNormUs = 4.5;  // an RMSNorm of its own
static bool gate_up_few(const Linear& L, int M, bool norm, double* us) {
    *us = few_us(L, M, norm ? FEW_SWIGLU_NORM : FEW_SWIGLU, 2);
    return L.N <= 64 * kNumCU && *us <= unsliced_us(L) + (norm ? kNormUs : 0.0);
}
bool norm_few_pays(const Linear& L, int M, bool norm) {
    double us;
    if (M > 16) return linear_few_rows(M) && gate_up_few(L, M, norm, &us);
    return linear_few_rows(M) && (L.N <= 32 * kNumCU || (L.N <= 64 * kNumCU && L.K >= 2048 && (M <= 8 || L.N <= 48 * kNumCU)));
}

// A whole layer: what the few-row QKV, O and down projections take longer than the tiled ones must stay below the two norms and
// the rotation that become part of them (13.6 us up to 4096 columns, 20 at 8192, 25 at 16384, less what the norm costs where it
// goes).  A QKV of two rounds over a K that is no whole number of rings per wave (8 k-steps of 32, 8 waves) takes some 1.5 us per 1024 of
// K longer than estimated, as the last ring is loaded in full, again in either round.  Measured end to end, us per layer gained by this path:
//   8B widths 9 / 6 / 1 / -4 at 1 / 8 / 12 / 16 rows, 70B widths 6 / 6 / 5 / 2 / 0 at 1 / 9 / 10 / 11 / 12, 12288 wide 6 / -12 / -23 / -51 at 1 / 8 / 12 / 16;
//   hidden columns, QKV columns: 4096, 12288 6 / 5 / 2 / -4 at 1 / 8 / 11 / 16; 2048, 10240 5 / 4 / 1 at 1 / 4 / 8;
//   two rounds and part of a ring: 5120, 15360 5 / 3 / 0 / -4 at 1 / 4 / 5 / 8; 5120, 12288 2 / 0 / -6 and 4608, 13824 2 / 0 / -6 at 1 / 4 / 8;
//   7168, 10240 5 / 4 / 3 / -1 at 1 / 4 / 7 / 8; 3584, 10240 5 / 4 / 1 / -1 and 3072, 10240 5 / 4 / 0 / -4 at 1 / 4 / 8 / 10; 2560, 10240 1 / 0 / -2 / -6
//   at 1 / 4 / 6 / 8; three rounds: 6144, 18432 10 / 6 / 2 / -4 at 1 / 8 / 10 / 11.
// On one set of weights, whole steps by this rule are within 1 % of the better path.
// From 17 rows on the few-row kernel must take gate/up too (the tiled one has the norm for 16 rows), and 1 us must be left: gained
// at 17 / 24 / 32 rows 9 / 8 / 7 us a layer at 256 hidden columns, 6 / 4 / 2 at 1024; it would be -1 / -5 / -11 at 2048 and
// -11 / -19 / -25 at the 8B widths.
bool step_few_rows(const Linear& qkv, const Linear& o, const Linear& gu, const Linear& down, int M) {
    if (!linear_few_rows(M) || (M > 16 && qkv.N > 32 * kNumCU)) return false;
    const double saved = 5.9 + 1.3 / 1024 * qkv.K;
    double pays = tiled_us(qkv) + tiled_us(o) + tiled_us(down) + (saved > 13.0 ? saved : 13.0);
    const int ct_o = few_col_tiles(o, M), ct_down = few_col_tiles(down, M);
    if (qkv.N <= 32 * kNumCU) {
        if (norm_few_pays(gu, M)) {
            const double gu_saved = unsliced_us(gu) - few_us(gu, M, FEW_SWIGLU_NORM, 2);
            if (M > 16) pays += gu_saved - 1.0;
            else if (gu_saved > 0.0) pays += gu_saved;
        } else if (M > 16) {
            return false;
        }
    } else if (qkv.N <= 64 * kNumCU && qkv.Kpad % (32 * kFewWaves * kFewRing) != 0) {
        pays -= 0.0015 * qkv.K;
    }
    return few_us(qkv, M, FEW_QKV, 2) + few_us(o, M, FEW_ROWS, ct_o) + few_us(down, M, FEW_PACKED, ct_down) <= pays;
}

// A projection by itself: against the tiled kernel, the sum of its slices (5 us), and no less than 25.5 us, which a call with slices takes
// however fast its kernels are (18 where the few-row kernel has two row tiles; 18 .. 24 measured).  That is their scratch memory: its
// allocation waits until the stream has nothing left to do, so a call behind other work takes as long as one on an idle stream,
// and in a captured graph the memory nodes take it (10 rows of 357 x 4256: 10.4 us behind other work, 10.7 in a graph, against 20
// and 22 with slices; 17 rows of 128 x 6912 18.7 and 18.9 against 24 and 22; 20 rows: 1024 x 1024 6.7, 2048 x 8192 9.0; 32 rows of
// 1024 x 16384 12).  Behind a gate/up, whose block allocates for both, there is no such floor (2048 x 5632 at 20 rows would take 39 us with it
// against 31).  A long K without a workgroup for every CU is a serial chain that nothing hides
// (2048 x 28672, one row: 33 against 29 us).  4096 x 14336: 24 against 28 us at 8 rows, 33 against 30 at 16; 10240 x 28672 (320
// workgroups): 112 against 98 at one row.  Very wide outputs have enough column tiles for the tiled kernel unsliced.
bool linear_few_pays(const Linear& L, int M, SliceCost slices) {
    if (!linear_few_rows(M) || L.N > 16384 || (L.K > 16384 && L.N < 4096)) return false;
    const double tiled = 5.0 + tiled_us(L);
    const double call = M <= 16 ? 25.5 : slices == SLICES_ALONE ? 18.0 : 0.0;
    return few_us(L, M, FEW_ROWS, few_col_tiles(L, M)) <= (tiled > call ? tiled : call);
}

// the same for the down projection of a feed-forward block, whose scratch memory is there anyway; from 17 rows on with what the
// few-row kernel saves at gate/up (4096 x 4096: 45 -> 30 us at 20 rows, 47 -> 35 at 32; 2048 x 5632 would go from 31 to 33 and from 32 to 38)
bool ffn_few_pays(const Linear& gu, const Linear& down, int M) {
    if (!linear_few_rows(M) || down.N > 16384) return false;
    double us, pays = 5.0 + tiled_us(down);
    if (M > 16 && gate_up_few(gu, M, false, &us)) pays += unsliced_us(gu) - us;
    return few_us(down, M, FEW_PACKED, few_col_tiles(down, M)) <= pays;
}

int32_t launch_linear_few(const Linear& L, const float* A, int64_t lda, int M, int packed, float* y, int ldy, int add, hipStream_t st) {
    if (M == 0) return CHIRON_OK;
    if (M > 32) return fail(CHIRON_ERR_INVALID_ARG, "linear: %d rows on the few-row path", M);
    if (L.K % 16 != 0 || L.K < 16) return fail(CHIRON_ERR_SHAPE, "linear: K=%d must be a positive multiple of 16", L.K);
    if ((!packed && lda % 4 != 0) || ((uintptr_t)A & 15)) return fail(CHIRON_ERR_INVALID_ARG, "linear: input rows must be 16-byte aligned");
    const int ct = few_col_tiles(L, M);
    const dim3 grid((L.N + 16 * ct - 1) / (16 * ct)), block(64 * kFewWaves);
#define CHIRON_FEW(CT_, MODE_) \
    launch(M > 16 ? linear_few_kernel<CT_, MODE_, 2> : linear_few_kernel<CT_, MODE_, 1>, grid, block, st, L.w, L.tstride, L.N, L.K, L.Kpad, A, lda, M, \
           (const uint16_t*)nullptr, 0.f, y, ldy, add, RopeOut())
    if (ct == 1 && packed) CHIRON_FEW(1, FEW_PACKED);
    else if (ct == 1) CHIRON_FEW(1, FEW_ROWS);
    else if (packed) CHIRON_FEW(2, FEW_PACKED);
    else CHIRON_FEW(2, FEW_ROWS);
#undef CHIRON_FEW
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// A fused gate/up matrix (ldy: the padded K of its consumer), with the norm in its operand load or without, or a plain projection with it
int32_t launch_norm_few(const Linear& L, const float* h, int lda, int M, const NormIn* norm, int swiglu, float* y, int ldy, hipStream_t st) {
    if (M == 0) return CHIRON_OK;
    if (M > (swiglu ? 32 : 16)) return fail(CHIRON_ERR_INVALID_ARG, "linear: %d rows on the few-row path", M);
    if (L.K % 16 != 0 || L.K < 16) return fail(CHIRON_ERR_SHAPE, "linear: K=%d must be a positive multiple of 16", L.K);
    if (lda % 4 != 0 || ((uintptr_t)h & 15)) return fail(CHIRON_ERR_INVALID_ARG, "linear: input rows must be 16-byte aligned");
    if (swiglu && (L.N % 32 != 0 || ldy % 8 != 0 || ((uintptr_t)y & 15))) return fail(CHIRON_ERR_INVALID_ARG, "linear: SwiGLU needs whole gate/up tiles and 16-byte aligned output");
    if (!swiglu && !norm) return fail(CHIRON_ERR_INVALID_ARG, "linear: no norm");
    const int ct = swiglu ? 2 : few_col_tiles(L, M);
    const NormIn nm = norm ? *norm : NormIn();
    const dim3 grid((L.N + 16 * ct - 1) / (16 * ct)), block(64 * kFewWaves);
#define CHIRON_FEW(CT_, MODE_, RT_, LDY_) \
    launch(linear_few_kernel<CT_, MODE_, RT_>, grid, block, st, L.w, L.tstride, L.N, L.K, L.Kpad, h, (int64_t)lda, M, nm.gain, nm.eps, y, LDY_, 0, RopeOut())
    if (swiglu && norm && M > 16) CHIRON_FEW(2, FEW_SWIGLU_NORM, 2, M * (ldy / 8));
    else if (swiglu && norm) CHIRON_FEW(2, FEW_SWIGLU_NORM, 1, M * (ldy / 8));
    else if (swiglu && M > 16) CHIRON_FEW(2, FEW_SWIGLU, 2, M * (ldy / 8));
    else if (swiglu) CHIRON_FEW(2, FEW_SWIGLU, 1, M * (ldy / 8));
    else if (ct == 1) CHIRON_FEW(1, FEW_NORM, 1, ldy);
    else CHIRON_FEW(2, FEW_NORM, 1, ldy);
#undef CHIRON_FEW
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

int32_t launch_qkv_few(const Linear& L, const float* h, int lda, int M, const NormIn& norm, const RopeOut& ro, hipStream_t st) {
    if (M == 0) return CHIRON_OK;
    if (M > 32) return fail(CHIRON_ERR_INVALID_ARG, "linear: %d rows on the few-row path", M);
    if (L.N != (ro.n_q + 2 * ro.pool.n_kv) * ro.pool.d || ro.pool.d % 32 != 0)
        return fail(CHIRON_ERR_SHAPE, "linear: %d columns are not the heads of a fused QKV projection", L.N);
    launch(M > 16 ? linear_few_kernel<2, FEW_QKV, 2> : linear_few_kernel<2, FEW_QKV, 1>, dim3(L.N / 32), dim3(64 * kFewWaves), st, L.w, L.tstride, L.N, L.K, L.Kpad, h, (int64_t)lda, M, norm.gain,
           norm.eps, (float*)nullptr, 0, 0, ro);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

}  // namespace chiron
