// Projections of the decode step: y[M,N] (+)= A[M,K] * W^T with bf16 weights streamed from HBM
// straight into matrix-core operand registers, and fp32 activations staged through LDS as two
// bf16 terms (hi + lo).  gfx950, wave64, v_mfma_f32_32x32x16_bf16.
//
// Work split: a workgroup of NW = 4 (or 8) waves owns NW*NF tiles of 32 output columns (one wave = NF tiles),
// one M-tile of 32*MT rows and one slice of K.  Weights are read exactly once per M-tile; the
// activation chunk of the current K-slice is shared by the waves through LDS.  With more than
// one K-slice each slice stores its partial product in a workspace [slice][M][N]; the kernel that
// consumes the projection (residual add + RMSNorm, or RoPE) sums the slices while it reads them,
// in a fixed order, so results are reproducible run to run.
//
// PRO_PACKED (large batches, see linear_big.hip): the activations arrive already split into their two bf16
// terms in tile order and are copied global -> LDS directly, without staging registers or conversion work.
//
// The gate/up projection of the feed-forward block ends in SwiGLU: its weights are packed so that every 32-column
// tile holds 16 gate columns and the 16 up columns of the same indices (gate_up_packed_row below), which puts
// gate[m][j] and up[m][j] into the two halves of one wave, and the epilogue writes silu(gate) * up, either as fp32
// rows or already split into bf16 terms in the tile order that PRO_PACKED reads.  The down projection then is a plain
// projection over half the bytes, and nothing evaluates exp() more than once per element.
#include <climits>
#include <cstdlib>

#include "chiron_internal.h"
#include "device_util.h"

namespace chiron {

// ---- weight repacking -------------------------------------------------------------------------------
// Packed row of gate (kind 0) or up (kind 1) column j in the fused gate/up matrix.  Row i of a 32-row tile lands in
// accumulator register r of the lanes of half h with i = 8*(r/4) + 4*h + r%4: the gate column 16*tile + r goes to
// half 0, register r, the up column of the same index to half 1, register r.
__host__ __device__ inline int gate_up_packed_row(int j, int kind) {
    return 32 * (j / 16) + 8 * ((j % 16) / 4) + 4 * kind + j % 4;
}

// interleave: 0 = rows go to row_offset + r; 1 / 2 = r is a gate / up column of a fused gate/up matrix; 64 or more = head dimension of a
// fused QKV matrix
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint16_t* __restrict__ src, int rows, int K, size_t tstride,
                                                        uint16_t* __restrict__ dst, int row_offset, int interleave) {
    int kgroups = K / 8;
    int64_t total = (int64_t)rows * kgroups;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        int r = (int)(t / kgroups), kg = (int)(t % kgroups);
        int n = r + row_offset;
        if (interleave >= 64) n = n / interleave * interleave + qkv_packed_dim(n % interleave, interleave);
        else if (interleave) n = gate_up_packed_row(r, interleave - 1);
        uint4 v = *reinterpret_cast<const uint4*>(src + (size_t)r * K + (size_t)kg * 8);
        *reinterpret_cast<uint4*>(dst + (size_t)(n / 32) * tstride + (size_t)kg * 256 + (size_t)(n % 32) * 8) = v;
    }
}

int32_t launch_pack_rows(const uint16_t* src, int rows, int K, size_t tstride, uint16_t* dst_packed, int row_offset,
                         hipStream_t st, int interleave) {
    if (rows == 0) return CHIRON_OK;
    if ((interleave == 1 || interleave == 2) && rows % 16 != 0) return fail(CHIRON_ERR_SHAPE, "gate/up packing: %d columns are not a multiple of 16", rows);
    if (interleave >= 64 && (rows % interleave || row_offset % interleave)) return fail(CHIRON_ERR_SHAPE, "QKV packing: %d rows are not whole heads", rows);
    int64_t total = (int64_t)rows * (K / 8);
    int blocks = (int)((total + 255) / 256 < 8192 ? (total + 255) / 256 : 8192);
    launch(pack_rows_kernel, dim3(blocks), dim3(256), st, src, rows, K, tstride, dst_packed, row_offset, interleave);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

// Byte of a 64-byte line at which a kernel's loop over the chunks of K starts (-1: wherever it falls).  With the same instructions in it a
// loop takes up to 6 % longer at some places than at others.  us a launch on the same weights, every place in turn (K = 4096):
//   96 x 256     gate/up of 160 rows (8B widths)   94.1 at 28 and 60, 95.3 .. 96.5 at 12, 24, 44 and 56, 98.9 .. 100.4 elsewhere
//   64 x 512     gate/up of 200 rows               112.0 at 28, 112.3 .. 113.2 at 24, 56 and 60, 113.8 .. 117.4 elsewhere
//   128 x 512    gate/up of 500 rows               199.4 .. 200.9 at 8 .. 20 and 40 .. 52, 202 .. 209 elsewhere
//   64 x 256, eight waves, 150 rows of 20000 columns    70.8 at 16 and 48, 71.3 at 20 and 52, up to 73.2 elsewhere
//   96 x 128, gate/up of 80 rows, 65.1 at 20 and 66.2 at 60; 128 x 512 of two-term input 0.3 to 1.3 % of a block of 400 rows (8192 -> 28672 -> 8192)
//   less at 12 than at 24.  The other kernels showed no difference beyond the runs' own.
constexpr int loop_byte(int mt, int nf, int ks, int pro, int nw) {
    if (pro == PRO_PACKED) return mt == 4 && nf == 4 ? 12 : -1;
    if (nw == 8) return mt == 4 ? 20 : 16;
    if (mt == 3) return nf == 2 ? 28 : (ks == 8 ? 20 : -1);
    return mt == 2 && nf == 4 ? 28 : -1;
}
// What follows starts there as long as the compiler puts nothing in between: a test reads the places out of the built library.
template <int BYTE>
__device__ __forceinline__ void place_loop() {
    if constexpr (BYTE >= 0) asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"n"(BYTE / 4));
}

// ---- the kernel ------------------------------------------------------------------------------------------
// Pipeline per workgroup: weights sit in a ring of KS*NF register fragments per wave; as soon as the MFMAs of
// k-step s have been issued, slot s is reloaded with the same k-step of the NEXT chunk, so about one chunk of
// weight loads (KS*NF KiB per wave) is always in flight.  Activations are double-buffered in LDS: while chunk c
// is consumed, chunk c+1 is written to the other buffer and chunk c+2 is on its way from L2 into registers;
// one barrier per chunk.
// WNT: weight loads carry the non-temporal hint (every weight is read once: a single M-tile).  With several M-tiles
// the same weights are read once per M-tile through the L2, and the hint makes those re-reads slower (measured on the
// 8B gate/up shape at 2048 rows: the weight stream alone 268 us with the hint, 194 us without).
// NORM: the input is rmsnorm(A) * gain.  A workgroup of an unsliced projection reads whole rows anyway: the gain is applied
// while a chunk is staged, the sum of squares is taken from the same values, and the row's 1/rms multiplies the accumulators.
// The workgroup's columns, K-slice and M-tile are bx, by, bz.
template <int MT, int NF, int KS, int PRO, bool WNT = true, bool NORM = false, int NW = 4>
__device__ __forceinline__ void linear_tile(const uint16_t* __restrict__ Wp, size_t tstride, int Npad, int Nreal, int K, int Kpad,
                                            const float* __restrict__ A, int lda, int M, float* __restrict__ Y, int ldy, int chunks_per_split,
                                            int mode, size_t part_stride, int bx, int by, int bz, const uint16_t* __restrict__ gain, float eps) {
    constexpr int MROWS = 32 * MT;
    constexpr int RS = MROWS + 1;      // LDS row stride in 16-byte units (+1 breaks the power-of-two stride)
    constexpr int KG = 2 * KS;         // 8-wide k-groups per chunk
    constexpr int KC = 16 * KS;        // k per chunk
    // (with NORM there are at most 16 rows: the upper half of the tile is not staged where that saves whole passes, and the
    // columns of the product that it would give are never stored)
    constexpr int T = 64 * NW;  // threads
    constexpr int SROWS = NORM && MT == 1 && 16 * KG % T == 0 ? 16 : MROWS;
    constexpr int TASKS = SROWS * KG;  // 8-float staging tasks per chunk
    static_assert(TASKS % T == 0, "staging assumes whole passes of the workgroup");
    constexpr int TPT = TASKS / T;
    // activation loads and staging spread over the k-steps of a chunk (see below; measured on one device against the
    // bunched form: gate/up at 64 rows 50.3 against 53.6 us, at 192 rows 101 against 109 us).  The widest tile keeps
    // them bunched: it has no registers left for the first chunk's separate staging set.
    constexpr bool SPREAD = PRO != PRO_PACKED && MT * NF <= 8 && TPT <= KS;
    static_assert(!NORM || SPREAD, "the norm is built into the spread staging only");

    __shared__ uint4 lds_hi[2][KG * RS];
    __shared__ uint4 lds_lo[2][KG * RS];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = bz * MROWS;
    const int tile0 = (bx * NW + wave) * NF;  // first 32-column tile of this wave
    const int chunks_total = (K + KC - 1) / KC;
    const int c_begin = by * chunks_per_split;
    int c_end = c_begin + chunks_per_split;
    if (c_end > chunks_total) c_end = chunks_total;

    floatx16 acc[NF][MT];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][t][r] = 0.f;

    uint4 w[KS][NF];
    float4 areg[TPT][2];  // fp32 staging registers (unused with PRO_PACKED, whose input goes straight into LDS)
    // PRO_PACKED: A points at the hi terms in 32-row x 8-k tile order, the lo terms follow them
    const int mtiles_all = (M + 31) / 32;
    const float4* Ahi = reinterpret_cast<const float4*>(A);
    const float4* Alo = Ahi + (size_t)mtiles_all * 32 * (Kpad / 8);

    // The loop body holds no divergent branch: every load is unconditional on a clamped address (the packed
    // weights are zero-padded in K to a whole chunk, out-of-range activation rows/columns are zeroed by a
    // select), so the compiler can count outstanding loads exactly and never drains the queue.
    const int kgroups = Kpad / 8;
    const uint16_t* wp[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        int tile = min(tile0 + f, Npad / 32 - 1);  // a wave past the last tile recomputes it; its stores are masked
        wp[f] = Wp + (size_t)tile * tstride + (lane >> 5) * 256 + (lane & 31) * 8;
    }
    auto load_w = [&](int c, int s) {
        size_t off = (size_t)(c * KC + s * 16) * 32;
#pragma unroll
        // non-temporal: a step reads every weight once, and what the weights do not displace stays cached for the
        // activations and the K/V pages (same-device A/B on the whole step: -7 % at 1 request, -1.5 % at 64..2048)
        for (int f = 0; f < NF; ++f)
            w[s][f] = WNT ? load_stream_16(wp[f] + off) : *reinterpret_cast<const uint4*>(wp[f] + off);
    };
    // staging task i of a chunk: 8 consecutive k of one row, thread tid + T*i.  A thread's tasks share their k, so the
    // gains of a chunk are one load, with the last task: by then the previous chunk's gains have been used.
    uint4 g0 = make_uint4(0, 0, 0, 0), greg = g0;  // gains of the first chunk and of the one being staged
    float ss[TPT];                                 // this thread's part of its rows' sums of squares
#pragma unroll
    for (int i = 0; i < TPT; ++i) ss[i] = 0.f;
    auto load_task = [&](int c, int i, float4 (&ar)[2], uint4& gr) {
        int task = tid + i * T;
        int kg = task % KG, m = task / KG;
        int k = c * KC + kg * 8;
        const float* p = A + (size_t)min(m0 + m, M - 1) * lda + min(k, K - 8);
        ar[0] = *reinterpret_cast<const float4*>(p);
        ar[1] = *reinterpret_cast<const float4*>(p + 4);
        if (NORM && i == TPT - 1) gr = *reinterpret_cast<const uint4*>(gain + min(k, K - 8));
    };
    auto stage_task = [&](int c, int i, int buf, const float4 (&ar)[2], const uint4& gr) {
        int task = tid + i * T;
        int kg = task % KG, m = task / KG;
        const bool ok = (m0 + m < M) && (c * KC + kg * 8 < K);
        float v[8] = {ar[0].x, ar[0].y, ar[0].z, ar[0].w, ar[1].x, ar[1].y, ar[1].z, ar[1].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ok ? v[e] : 0.f;
        if (NORM) {
            const uint32_t gw[4] = {gr.x, gr.y, gr.z, gr.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ss[i] = fmaf(v[e], v[e], ss[i]);
                v[e] *= (e & 1) ? bf16_hi(gw[e / 2]) : bf16_lo(gw[e / 2]);
            }
        }
        uint4 hi, lo;
        split2(v[0], v[1], hi.x, lo.x);
        split2(v[2], v[3], hi.y, lo.y);
        split2(v[4], v[5], hi.z, lo.z);
        split2(v[6], v[7], hi.w, lo.w);
        lds_hi[buf][kg * RS + m] = hi;
        lds_lo[buf][kg * RS + m] = lo;
    };
    auto load_a = [&](int c) {
#pragma unroll
        for (int i = 0; i < TPT; ++i) load_task(c, i, areg[i], greg);
    };
    auto stage_a = [&](int c, int buf) {
#pragma unroll
        for (int i = 0; i < TPT; ++i) stage_task(c, i, buf, areg[i], greg);
    };
    // PRO_PACKED: chunk c of the pre-split activations goes HBM/L2 -> LDS directly (16 bytes per lane, a wave
    // fills 64 consecutive rows of one k-group), no registers and no LDS store instructions in between
    constexpr int JOBS = KG * (MROWS / 64) * 2;  // (k-group, 64-row half, hi|lo) per chunk, dealt to the waves
    static_assert(PRO != PRO_PACKED || (MROWS % 64 == 0 && JOBS % NW == 0), "packed input needs 64-row halves");
    constexpr int WJOBS = PRO == PRO_PACKED ? JOBS / NW : 1;
    // per job: this lane's source at chunk 0 (it advances by one chunk of k-groups per chunk) and the wave-uniform
    // LDS byte address of the job's destination in either buffer
    const float4* dma_src[WJOBS];
    uint32_t dma_dst[WJOBS];  // in buffer 0; buffer 1 lies KG*RS pieces further in both arrays
    if (PRO == PRO_PACKED) {
#pragma unroll
        for (int j = 0; j < WJOBS; ++j) {
            const int job = wave + NW * j;
            const int lo = job & 1, half = (job >> 1) % (MROWS / 64), kg = (job >> 1) / (MROWS / 64);
            const int m = half * 64 + lane;
            const size_t idx = ((size_t)min(bz * MT + m / 32, mtiles_all - 1) * kgroups + kg) * 32 + (m & 31);
            dma_src[j] = (lo ? Alo : Ahi) + idx;
            dma_dst[j] = __builtin_amdgcn_readfirstlane(lds_address((lo ? lds_lo[0] : lds_hi[0]) + kg * RS + half * 64));
        }
    }
    auto dma_a = [&](int c, int buf) {
#pragma unroll
        for (int j = 0; j < WJOBS; ++j)
            global_to_lds_16(dma_src[j] + (size_t)c * (KG * 32), dma_dst[j] + (uint32_t)buf * (uint32_t)(KG * RS * sizeof(uint4)));
    };
    // LDS fragments of one k-step: hi and lo terms of the MT row tiles
    struct Frags {
        bf16x8 h[MT], l[MT];
    };
    auto read_frags = [&](int buf, int s, Frags& fr) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            int idx = (s * 2 + (lane >> 5)) * RS + t * 32 + (lane & 31);
            uint4 h = lds_hi[buf][idx], l = lds_lo[buf][idx];
            fr.h[t] = *reinterpret_cast<bf16x8*>(&h);
            fr.l[t] = *reinterpret_cast<bf16x8*>(&l);
        }
    };
    auto mma_frags = [&](int s, const Frags& fr) {
        // hi terms of every accumulator first, then the lo terms: consecutive MFMAs never chain on one accumulator
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[f][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&w[s][f]), fr.h[t], acc[f][t], 0, 0, 0);
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int t = 0; t < MT; ++t)
                acc[f][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&w[s][f]), fr.l[t], acc[f][t], 0, 0, 0);
    };
    // Up to 96 rows a workgroup has one wave per SIMD and few MFMAs per k-step, so the chain "fragments arrive from
    // LDS -> MFMAs -> reload the weight slot" paces the weight stream.  There the fragments of k-step s+1 are read while
    // the MFMAs of k-step s run (two register sets); only a chunk's first k-step waits for LDS.  (Measured on the 8B
    // gate/up shape at 64 rows with the LDS reads taken out: 5.5 of 55 us.)  The 128-row tiles have enough MFMAs per
    // k-step to cover the reads and no registers to spare.
    constexpr bool PIPE = MT < 4;
    Frags fr[PIPE ? 2 : 1];
    auto mma_step = [&](int buf, int s) {
        if constexpr (PIPE) {
            if (s == 0) read_frags(buf, 0, fr[0]);
            if (s + 1 < KS) read_frags(buf, s + 1, fr[(s + 1) & 1]);
            mma_frags(s, fr[s & 1]);
        } else {
            read_frags(buf, s, fr[0]);
            mma_frags(s, fr[0]);
        }
    };

    // Order of memory operations (kept in place by the scheduling fences): per iteration the KS weight reloads
    // come first, the activation loads last, in the prologue likewise, so at every use the number of younger
    // loads in flight is the same on the loop's entry edge and on its back edge.
    if (PRO == PRO_PACKED) {
        if (c_begin < c_end) {  // uniform over the workgroup
            const int c_last = c_end - 1;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                load_w(c_begin, s);
                __builtin_amdgcn_sched_barrier(0);  // same issue order as in the loop: k-step 0 is the oldest
            }
            dma_a(c_begin, 0);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();
            int buf = 0, c = c_begin;
            if (c < c_last) {
                place_loop<loop_byte(MT, NF, KS, PRO, NW)>();
                do {
                    // start the copy of chunk c+1 into the idle buffer (last read before the barrier that ended the
                    // previous round), multiply chunk c out of the other one while refilling the weight ring
                    dma_a(c + 1, buf ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        mma_step(buf, s);
                        load_w(c + 1, s);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // the KS*NF weight loads just issued are younger than the activation copy: let them fly
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KS * NF) : "memory");
                    lds_barrier();
                    buf ^= 1;
                } while (++c < c_last);
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) mma_step(buf, s);
        }
    } else if (SPREAD) {
        // Activation traffic spread over the chunk: the loads of a task's next-but-one chunk are issued, and the task's
        // next chunk is converted and written to LDS, right after one particular k-step's weight reload instead of all
        // together before the barrier.  A burst of activation loads keeps the CU's address unit busy (1 KiB per load
        // instruction at 64 bytes per cycle, four waves at once) exactly when the next chunk's weight reloads want to
        // go out, and in a latency-bound weight stream every delayed request is lost time.
        if (c_begin < c_end) {  // uniform over the workgroup
            const int c_last = c_end - 1;
            // first chunk through a register set of its own, issued before everything else; the ring and the second
            // chunk's tasks follow in the loop's order, so that the wait counts of entry and back edge agree.  (Two
            // chunks or more and a single chunk are separate paths: in one path the compiler moves the second chunk's
            // loads, which only the loop uses, behind the barrier and out of that order.)
            float4 a0[TPT][2];
#pragma unroll
            for (int i = 0; i < TPT; ++i) load_task(c_begin, i, a0[i], g0);
            __builtin_amdgcn_sched_barrier(0);
            if (c_begin < c_last) {
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    load_w(c_begin, s);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < TPT; ++i)
                        if (i * KS / TPT == s) {
                            load_task(c_begin + 1, i, areg[i], greg);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                }
#pragma unroll
                for (int i = 0; i < TPT; ++i) stage_task(c_begin, i, 0, a0[i], g0);
                lds_barrier();
                int buf = 0, c = c_begin;
                place_loop<loop_byte(MT, NF, KS, PRO, NW)>();
                do {
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        mma_step(buf, s);
                        load_w(c + 1, s);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < TPT; ++i)
                            if (i * KS / TPT == s) {
                                stage_task(c + 1, i, buf ^ 1, areg[i], greg);
                                __builtin_amdgcn_sched_barrier(0);
                                load_task(min(c + 2, c_last), i, areg[i], greg);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                    lds_barrier();
                    buf ^= 1;
                } while (++c < c_last);
#pragma unroll
                for (int s = 0; s < KS; ++s) mma_step(buf, s);
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s) load_w(c_begin, s);
#pragma unroll
                for (int i = 0; i < TPT; ++i) stage_task(c_begin, i, 0, a0[i], g0);
                lds_barrier();
#pragma unroll
                for (int s = 0; s < KS; ++s) mma_step(0, s);
            }
        }
    } else
    if (c_begin < c_end) {   // uniform over the workgroup
        const int c_last = c_end - 1;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            load_w(c_begin, s);
            __builtin_amdgcn_sched_barrier(0);  // same issue order as in the loop: k-step 0 is the oldest
        }
        load_a(c_begin);
        stage_a(c_begin, 0);
        load_a(min(c_begin + 1, c_last));
        lds_barrier();
        int buf = 0;
        for (int c = c_begin; c < c_last; ++c) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                mma_step(buf, s);
                load_w(c + 1, s);  // slot s is free again: fetch the same k-step of the next chunk
                __builtin_amdgcn_sched_barrier(0);
            }
            stage_a(c + 1, buf ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            load_a(min(c + 2, c_last));
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
            buf ^= 1;
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) mma_step(buf, s);
    }

    if constexpr (NORM) {
        __shared__ float s_inv[MROWS];
        // the KG threads that staged a row sit side by side in one wave
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            float s = ss[i];
#pragma unroll
            for (int o = 1; o < KG; o <<= 1) s += __shfl_xor(s, o);
            if (tid % KG == 0) s_inv[(tid + i * T) / KG] = 1.0f / sqrtf(s / (float)K + eps);
        }
        lds_barrier();
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const float inv = s_inv[t * 32 + (lane & 31)];
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[f][t][r] *= inv;
        }
    }

    // D[i][j]: lane holds column j = lane%32 (an activation row m) and rows i = 8*(r/4) + 4*(lane/32) + r%4
    // (output columns n) for r = 0..15.
    if (mode >= EPI_SWIGLU) {
        // Fused gate/up: in tile T the lanes of half 0 hold gate[m][16T + r], those of half 1 up[m][16T + r].  The halves
        // swap eight values each, after which half h owns the columns 16T + 8h .. + 7 of row m.
        const int half = lane >> 5;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int tile = tile0 + f;
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float mine_g = acc[f][t][e], mine_u = acc[f][t][8 + e];  // half 0: gate e, (gate 8+e); half 1: (up e), up 8+e
                    const float got = __shfl_xor(half ? mine_g : mine_u, 32);       // half 0 receives up e, half 1 gate 8+e
                    const float g = half ? got : mine_g, u = half ? mine_u : got;
                    v[e] = g / (1.0f + __expf(-g)) * u;
                }
                const int m = m0 + t * 32 + (lane & 31);
                if (m >= M || tile >= Npad / 32) continue;
                if (mode == EPI_SWIGLU) {
                    float* dst = Y + (size_t)m * ldy + tile * 16 + half * 8;
                    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
                } else {
                    // the two bf16 terms in 32-row x 8-k tile order (ldy = k-groups of the consumer, part_stride = distance
                    // from the hi to the lo terms in 16-byte units), or with the M rows of a k-group side by side
                    uint4 hi, lo;
                    split2(v[0], v[1], hi.x, lo.x);
                    split2(v[2], v[3], hi.y, lo.y);
                    split2(v[4], v[5], hi.z, lo.z);
                    split2(v[6], v[7], hi.w, lo.w);
                    uint4* dst = reinterpret_cast<uint4*>(Y) + (mode == EPI_SWIGLU_FEW ? (size_t)(2 * tile + half) * M + m
                                     : ((size_t)(m / 32) * ldy + (size_t)(2 * tile + half)) * 32 + (m & 31));
                    dst[0] = hi;
                    dst[part_stride] = lo;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        int nb = (tile0 + f) * 32 + (lane >> 5) * 4;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            int m = m0 + t * 32 + (lane & 31);
            if (m >= M) continue;
            // EPI_STORE: y = acc;  EPI_ADD: y += acc (this workgroup is the only writer);  EPI_SLICES: slice `by` of the workspace
            float* yrow = Y + (mode == EPI_SLICES ? (size_t)by * part_stride : (size_t)0) + (size_t)m * ldy;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int n = nb + q * 8;
                if (n + 3 < Nreal && (ldy & 3) == 0) {
                    float4 v = make_float4(acc[f][t][q * 4], acc[f][t][q * 4 + 1], acc[f][t][q * 4 + 2], acc[f][t][q * 4 + 3]);
                    float4* dst = reinterpret_cast<float4*>(yrow + n);
                    if (mode == EPI_ADD) {
                        float4 o = *dst;
                        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
                    }
                    *dst = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < Nreal) {
                            float v = acc[f][t][q * 4 + e];
                            yrow[n + e] = mode == EPI_ADD ? yrow[n + e] + v : v;
                        }
                }
            }
        }
    }
}

// Workgroups are dealt to the 8 XCDs round-robin.  The 1-D grid (of a multiple of 8) is re-read so that consecutive logical ids
// sit on ONE XCD, and the M-tile index varies fastest: the workgroups that stream the same weight tiles for
// different rows then share that XCD's L2 instead of each pulling the tile from HBM.
__device__ __forceinline__ int logical_block(unsigned block, int total, int remap) {
    const int per_xcd = (total + 7) / 8;
    return remap ? (block % 8) * per_xcd + block / 8 : block;
}

template <int MT, int NF, int KS, int PRO, bool WNT = true, bool NORM = false, int NW = 4>
__global__ __launch_bounds__(64 * NW, (NW == 8 || (MT * NF <= 8 && !(MT == 4 && PRO != PRO_NONE)) ? 2 : 1)) void linear_kernel(const uint16_t* __restrict__ Wp, size_t tstride, int Npad, int Nreal, int K, int Kpad,
                                                     const float* __restrict__ A, int lda, int M,
                                                     float* __restrict__ Y, int ldy, int chunks_per_split,
                                                     int mode, size_t part_stride, int gx, int gy, int gz, int remap,
                                                     const uint16_t* __restrict__ gain, float eps) {
    const int total = gx * gy * gz;
    const int logical = logical_block(blockIdx.x, total, remap);
    if (logical >= total) return;  // uniform over the workgroup
    const int bz = logical % gz, bx = (logical / gz) % gx, by = logical / (gz * gx);
    linear_tile<MT, NF, KS, PRO, WNT, NORM, NW>(Wp, tstride, Npad, Nreal, K, Kpad, A, lda, M, Y, ldy, chunks_per_split, mode, part_stride, bx, by, bz,
                                                gain, eps);
}

// 128 rows x 512 columns by eight waves, K whole.  The tiles of whole rounds of the chip as they are (`whole` of them, a multiple of
// 256), those of a last round that would be at most half full as two of 128 x 256, which then fill it: 2048 rows of 28672
// columns at K = 4096 are 3.5 rounds.  Whole feed-forward blocks, us: 640 rows of 4096 -> 14336 -> 4096 455 -> 438, 1280 rows
// 795 -> 763, 1500 rows of 2048 -> 11008 -> 2048 415 -> 395, 2048 rows of the first 1158 -> 1147 (there the card's power is short: the
// clock falls as more of its matrix cores work).
__global__ __launch_bounds__(512, 2) void linear_wide_kernel(const uint16_t* __restrict__ Wp, size_t tstride, int Npad, int Nreal, int K, int Kpad,
                                                             const float* __restrict__ A, int lda, int M, float* __restrict__ Y, int ldy, int mode,
                                                             size_t part_stride, int gx, int gz, int whole, int remap) {
    const int chunks = (K + 63) / 64;
    if ((int)blockIdx.x < whole) {
        const int logical = logical_block(blockIdx.x, whole, remap);
        linear_tile<4, 2, 4, PRO_NONE, false, false, 8>(Wp, tstride, Npad, Nreal, K, Kpad, A, lda, M, Y, ldy, chunks, mode, part_stride, logical / gz, 0,
                                                        logical % gz, nullptr, 0.f);
    } else {
        const int rest = gx * gz - whole, logical = logical_block(blockIdx.x - whole, 2 * rest, remap);
        if (logical >= 2 * rest) return;  // uniform over the workgroup
        const int tile = whole + logical % rest;
        linear_tile<4, 1, 4, PRO_NONE, false, false, 8>(Wp, tstride, Npad, Nreal, K, Kpad, A, lda, M, Y, ldy, chunks, mode, part_stride,
                                                        2 * (tile / gz) + logical / rest, 0, tile % gz, nullptr, 0.f);
    }
}

// sum of K-slices: y (+)= sum_s part[s]  (used by the single-kernel entry points; inside the decode step the
// consumers of a projection do this sum themselves)
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ part, int ks, size_t stride,
                                                              int64_t n, float* __restrict__ y, int accumulate) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        float v = accumulate ? y[i] : 0.f;
        for (int s = 0; s < ks; ++s) v += part[(size_t)s * stride + i];
        y[i] = v;
    }
}

// the same, 16 bytes a thread and four slices' loads in flight (100 x 8192 from 8 slices 12.8 -> 9.5 us, bounded by memory)
__global__ __launch_bounds__(256) void reduce_partials_vec_kernel(const float4* __restrict__ part, int ks, size_t stride4,
                                                                  int64_t n4, float4* __restrict__ y, int accumulate) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) {
        float4 v = accumulate ? y[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        auto add = [&](const float4& t) { v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; };
        int s = 0;
        for (; s + 4 <= ks; s += 4) {
            float4 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = part[(size_t)(s + u) * stride4 + i];
#pragma unroll
            for (int u = 0; u < 4; ++u) add(t[u]);
        }
        for (; s < ks; ++s) add(part[(size_t)s * stride4 + i]);
        y[i] = v;
    }
}

int32_t launch_reduce_partials(const float* part, int ks, int64_t n, float* y, int accumulate, hipStream_t st) {
    if (n % 4 == 0 && (((uintptr_t)part | (uintptr_t)y) & 15) == 0) {
        const int64_t n4 = n / 4;
        const int blocks = (int)((n4 + 255) / 256 < 8192 ? (n4 + 255) / 256 : 8192);
        launch(reduce_partials_vec_kernel, dim3(blocks), dim3(256), st, reinterpret_cast<const float4*>(part), ks, (size_t)n4, n4,
               reinterpret_cast<float4*>(y), accumulate);
        CHIRON_HIP(hipGetLastError());
        return CHIRON_OK;
    }
    int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    launch(reduce_partials_kernel, dim3(blocks), dim3(256), st, part, ks, (size_t)n, n, y, accumulate);
    CHIRON_HIP(hipGetLastError());
    return CHIRON_OK;
}

Tuning& tuning() {
    static Tuning t;
    return t;
}

template <int MT, int NF, int PRO, int KS = 4, bool WNT = true, bool NORM = false, int NW = 4>
static void launch_cfg(int nblocks, hipStream_t st, const Linear& L, const float* A, int lda, int M, float* y, int ldy,
                       int cps, int mode, size_t part_stride, int gx, int gy, int gz, const NormIn& norm = NormIn()) {
    launch(linear_kernel<MT, NF, KS, PRO, WNT, NORM, NW>, dim3(nblocks), dim3(64 * NW), st, L.w, L.tstride, L.Npad, L.N, L.K, L.Kpad, A, lda, M, y, ldy, cps, mode,
                                                           part_stride, gx, gy, gz, tuning().linear_xcd_remap, norm.gain, norm.eps);
}

constexpr int kMaxSplit = 16;
int linear_max_split() { return kMaxSplit; }

// Rows from which the down projection is faster on the tiled two-term form of its input (128-row tiles, copied straight
// into LDS) than on fp32 rows (64- and 96-row tiles, split on the way into LDS); the gate/up epilogue writes whichever
// is asked for.  Measured inside the step, gate/up + down per layer: at K = 14336 (N = 4096) fp32 rows win up to 320
// rows (160 rows: 138 against 155 us), the two are level at 384..512, the tiled form wins from 768 (533 against 556 us);
// at K = 28672 (N = 8192) fp32 rows win at 96 rows (92 against 100 us), the tiled form at 128 (102 against 108 us).
static int big_min_rows_default(const Linear& L) { return L.K >= 16384 ? 97 : 513; }

int linear_big_min_rows(const Linear& L) {
    const int v = tuning().linear_big_min_m;
    return v == 0 ? big_min_rows_default(L) : (v < 0 ? INT32_MAX : v);
}

// ---- what a launch shape costs ------------------------------------------------------------------------------------
// A CU's time per k of the K range, in ns, by tile: with up to one workgroup per CU (what an almost empty grid takes, and how much
// more a full one does), and with several, per workgroup.  Measured with every tile forced in turn on fused gate/up matrices of
// 688 .. 14336 columns, K = 512 .. 4096, 40 .. 2048 rows, and checked on others (2048, 28672 and 64128 columns, K up to 8192; K sliced,
// 512 .. 8192 columns, K = 512 .. 14336, 20 .. 2048 rows): the median is within 5 % of the measured time, nine in ten within 18 %.
struct TileCost {
    int mt, nf;
    double one, fill, many;
};
static constexpr TileCost kTileCost[] = {{1, 1, 6.5, 1.2, 6.7},    {1, 2, 9.9, 1.8, 11.3},   {2, 1, 8.8, 2.5, 9.5},   {2, 2, 13.4, 2.9, 15.4}, {2, 4, 22.5, 6.0, 27.4},
                                         {3, 1, 12.3, 2.8, 15.0},  {3, 2, 20.0, 3.9, 21.5},  {4, 1, 19.2, 2.6, 17.5}, {4, 2, 25.2, 4.8, 26.5}, {4, 4, 37.3, 11.8, 48.7}};
// A launch, its slowest CU or the weights at 6.4 TB/s, the result at 4.5 TB/s; K-slices (of M x N fp32) are written and read again by
// whoever adds them: 0.4 us per MB, and 4 us for a launch of its own.
// (128 x 512 tiles: a last round that is at most half full is taken as tiles of 256 columns, see linear_wide_kernel)
static bool halved_last_round(int64_t wgs) { return wgs > kNumCU && wgs % kNumCU != 0 && wgs % kNumCU <= kNumCU / 2; }
static double shape_us(const Linear& L, int M, const TileCost& t, int64_t tiles, int ksplit, int64_t k_per_slice, SliceCost slices) {
    const int64_t wgs = tiles * ksplit;
    double per_k = wgs <= kNumCU ? t.one + t.fill * wgs / kNumCU : t.many * ((wgs + kNumCU - 1) / kNumCU);
    if (t.mt * t.nf == 16 && ksplit == 1 && halved_last_round(wgs)) per_k = t.many * (wgs / kNumCU) + 28.0;
    const double run = 1e-3 * k_per_slice * per_k, stream = 2e-6 * L.N * L.K / 6.4;
    const double us = 4.0 + (run > stream ? run : stream);
    if (ksplit == 1) return us + 4e-6 * M * L.N / 4.5;
    return us + 0.4e-6 * 4.0 * ksplit * M * L.N + (slices == SLICES_STEP ? 1.0 : 4.0);
}
// A call with slices takes this long however fast its kernels are, so a sliced shape is no better than that against an unsliced one.
// A projection by itself: it allocates the slices, and the allocation waits until the stream has nothing left to do (18 .. 26 us a call
// behind other work as well as alone); in a captured graph its memory nodes take as long (22 .. 24 us a call, where one launch
// takes what its kernel does: 8 .. 17 us for 20 to 30 rows of 100 .. 400 columns at K = 2000 .. 4000).  The second half of a block:
// what the host needs for it.
static double sliced_call_us(SliceCost slices) { return slices == SLICES_ALONE ? 26.0 : slices == SLICES_BLOCK ? 15.0 : 0.0; }

// Puts the shape with the least estimate in the place of the one given (tile, slices and chunks of kc per slice) if it is 5 % below
// that one's; `most` slices at most.  Sliced shapes are compared among each other by their kernels, also where the call
// takes longer than those (182 rows of 4254 x 3056: 39 us with the shape of the rules, 35 with the best; 128 rows of 2048 x 2048
// from a graph 26 and 22).
static void by_estimate(const Linear& L, int M, int kc, int most, SliceCost slices, int& mt, int& nf, int& ksplit, int& cps) {
    struct Candidate {
        double us;
        int mt, nf, ksplit, cps;
    };
    const auto tiles = [&](const TileCost& t) { return (int64_t)((L.Npad / 32 + 4 * t.nf - 1) / (4 * t.nf)) * ((M + 32 * t.mt - 1) / (32 * t.mt)); };
    Candidate best[2] = {{1e30, 0, 0, 0, 0}, {1e30, 0, 0, 0, 0}};  // unsliced, sliced
    const int given = ksplit > 1;
    double floor_us = sliced_call_us(slices);
    for (const TileCost& t : kTileCost)
        if (t.mt == mt && t.nf == nf) best[given] = Candidate{0.95 * shape_us(L, M, t, tiles(t), ksplit, (int64_t)cps * kc, slices), mt, nf, ksplit, cps};
    const int chunks = (L.K + 63) / 64;
    int per_slice[kMaxSplit + 1] = {0};  // chunks, for each number of slices (0: not to be tried)
    for (int want = 1; want <= most && want <= kMaxSplit && (want == 1 || want <= chunks / 2); ++want) {
        const int c = (chunks + want - 1) / want;
        if ((chunks + c - 1) / c != want || (most > 1 && c > 16 && c > cps)) continue;  // an empty slice; too long a one
        per_slice[want] = c;
    }
    bool stays = true;
    for (const TileCost& t : kTileCost) {
        const int64_t n = tiles(t);
        for (int want = 1; want <= kMaxSplit; ++want) {
            if (!per_slice[want]) continue;
            const double us = shape_us(L, M, t, n, want, (int64_t)per_slice[want] * 64, slices);
            Candidate& b = best[want > 1];
            if (us >= b.us) continue;
            b = Candidate{us, t.mt, t.nf, want, per_slice[want]};
            if ((want > 1) == given) stays = false;
        }
    }
    if (given && stays) floor_us *= 0.95;
    const double sliced = best[1].us > floor_us ? best[1].us : floor_us;
    const Candidate& b = best[given ? sliced <= best[0].us : sliced < best[0].us];
    mt = b.mt;
    nf = b.nf;
    ksplit = b.ksplit;
    cps = b.cps;
}

int64_t& linear_shape_searches() {
    static thread_local int64_t n = 0;
    return n;
}

LinearShape linear_shape(const Linear& L, int M, bool sliceable, int prologue, int max_split, SliceCost slices, bool swept) {
    const Tuning& tn = tuning();
    // Tile shape.  Up to 64 rows the kernel is HBM-bound: 32- or 64-row tiles; one column tile per wave when K can
    // be sliced (twice the workgroups along N, so half the K-slices for the consumer to add up) or when that is
    // what it takes to give every CU a workgroup, else two.  With many rows it is matrix-core bound and the
    // 128-row x 4-tile wave shape wins (fewer LDS reads and staging per MFMA, at one wave per SIMD): always from
    // 384 rows, and earlier when 128-row tiles pad the rows no further than 64-row tiles do, from 96 rows for a
    // very wide output (the LM head), at K >= 8192 past one such tile, or from 224 rows if K is sliced (70B-wide gate/up at
    // 200 rows 594 us with 64-row tiles, 345 with 128-row ones), and below 384 rows only if that gives three quarters of the
    // CUs a workgroup (32000 columns at K = 8192, 256 rows: 126 workgroups 328 us, 252 of 64 rows 200).  97..128 rows of a very
    // wide output take one 128-row tile also where two of 64 x 512 would need more than a round of the chip (80000 columns
    // at K = 4096, 97 rows: 200 against 232 us; 65536 columns, where they just fit, 190 against 131).  Measured on the 8B and
    // 70B shapes.
    const int tiles_n = L.Npad / 32;
    const int pad64 = (M + 63) / 64 * 64, pad128 = (M + 127) / 128 * 128;
    const int thr128 = tiles_n >= 2048 ? 96 : (L.K >= 8192 ? (sliceable ? 224 : 129) : 384);
    // (outputs narrower than 256 column tiles keep the 64-row shape at any row count: measured 8-12 % faster)
    const int cols512 = (tiles_n + 15) / 16;
    const bool fills128 = sliceable || cols512 * (pad128 / 128) >= kNumCU * 3 / 4 || (M > 96 && pad128 == 128 && cols512 * 2 > kNumCU);
    const bool big = tiles_n >= 256 && (M >= 384 || (pad128 == pad64 && M >= thr128 && fills128));
    // 65..96 rows take one 96-row tile: with 64-row tiles the second M-tile would stream every weight again for a
    // handful of rows (a step of 17 % in the whole decode step's latency between batch 64 and 65).  Likewise above
    // 128 rows wherever 96-row tiles pad the rows no further than 64-row tiles do (129..192, 257..288, 321..384:
    // a third fewer passes over the weights; measured 10-20 % on the gate/up and O projections).
    const int pad96 = (M + 95) / 96 * 96;
    int mt = tn.linear_mt ? tn.linear_mt : (big ? 4 : (M > 64 && pad96 <= pad64 ? 3 : (M > 32 ? 2 : 1)));
    int tiles = L.Npad / 32;
    int gz = (M + 32 * mt - 1) / (32 * mt);
    // Column tiles per wave.  A projection that cannot slice K takes the smallest count that fits the grid into one
    // round of the chip (224 workgroups for a 57344-wide gate/up with two tiles: 190 against 260 us at 65 rows; 251 for
    // the LM head with four: 169 against 192 us at 64 rows), two if none does.  A sliced one takes one tile up to 64
    // rows and two above, and more where the K-slices that fill the grid still hold twelve chunks or more (hidden
    // size 8192: QKV 34 against 39 us at 64 rows with two tiles, 50 against 56 us at 128 rows with four): wider
    // workgroups re-read the activations less often, but short slices are mostly ramp.
    int nf;
    if (tn.linear_nf) nf = tn.linear_nf;
    else if (big && tiles >= 256) nf = 4;
    else if (tiles < 64) nf = 1;
    else if (!sliceable) {
        const int max_nf = mt == 3 ? 2 : 4;
        nf = 1;
        while (nf < max_nf && ((tiles + 4 * nf - 1) / (4 * nf)) * gz > kNumCU) nf *= 2;
        if (((tiles + 4 * nf - 1) / (4 * nf)) * gz > kNumCU) nf = 2;
    } else {
        nf = M <= 64 ? 1 : 2;
        const int max_nf = mt == 3 ? 2 : 4;
        const int chunks64 = (L.K + 63) / 64;
        for (int c = max_nf; c > nf; c /= 2) {
            const int g = ((tiles + 4 * c - 1) / (4 * c)) * gz;
            const int ks = g >= kNumCU ? 1 : (kNumCU / g < max_split ? kNumCU / g : max_split);
            if (chunks64 / ks >= 12 && g * ks >= kNumCU * 3 / 4) {  // (and the sliced grid still covers the chip)
                nf = c;
                break;
            }
        }
    }
    if (prologue == PRO_PACKED) {  // only the large-batch shapes are built for pre-split input
        mt = 4;
        // four column tiles per wave unless K-slicing cannot make up for the smaller grid (one 128-row tile of a
        // 4096-wide output: 8 workgroup columns x 16 slices = half the chip; 58 against 45 us)
        const int gx4 = (tiles + 15) / 16, gz4 = (M + 127) / 128;
        const bool fills = !sliceable || (int64_t)gx4 * gz4 * max_split >= 200;
        nf = tn.linear_nf ? (tn.linear_nf == 4 ? 4 : 2) : (tiles >= 128 && fills ? 4 : 2);
    }
    if (nf == 4 && mt == 1) mt = 2;
    if (nf == 4 && mt == 3) mt = 4;  // four column tiles per wave are built for 64- and 128-row tiles only
    gz = (M + 32 * mt - 1) / (32 * mt);  // mt may have changed above
    int gx = (tiles + 4 * nf - 1) / (4 * nf);
    // an unsliced projection whose 64-row tiles give a few workgroups more than two per CU takes 96-row tiles if those
    // fit (gate/up at 289..320 rows: 560 workgroups 190 us, 448 workgroups 167 us)
    if (!tn.linear_mt && !sliceable && mt == 2 && prologue == PRO_NONE && nf <= 2 && gx * gz > 2 * kNumCU && gx * gz <= 3 * kNumCU &&
        gx * ((M + 95) / 96) <= 2 * kNumCU) {
        mt = 3;
        gz = (M + 95) / 96;
    }
    // A projection that cannot slice K (no workspace) runs one workgroup per CU; a ring of 8 k-steps then keeps twice
    // the weight bytes in flight per wave, which measured 9 % faster on the gate/up shape at 64 rows.
    const auto ring8 = [&] { return (mt == 2 || (mt == 3 && nf == 1)) && nf <= 2 && prologue != PRO_PACKED &&
                     (tn.linear_ks == 8 || (tn.linear_ks == 0 && nf == 1 && !sliceable && prologue == PRO_NONE)); };
    // Up to 32 rows a wave has two MFMAs per k-step and its weight stream is bound by the bytes it keeps in flight over
    // the load latency: the unsliced one-tile-per-wave shape takes a ring of 16 k-steps (16 KiB per wave; measured on the
    // 8B gate/up shape: 37.3 against 40.0 us at one row, 39.8 against 41.4 us at 32 rows; no gain at 64 rows)
    const auto ring16 = [&] { return mt == 1 && nf == 1 && prologue == PRO_NONE && L.Kpad % 256 == 0 &&
                                     (tn.linear_ks == 16 || (tn.linear_ks == 0 && !sliceable)); };
    bool ks8 = ring8(), ks16 = ring16();
    const int KC = ks16 ? 256 : (ks8 ? 128 : 64);
    int chunks = (L.K + KC - 1) / KC;
    int ksplit = tn.linear_ksplit ? tn.linear_ksplit : (tn.linear_target_blocks + gx * gz - 1) / (gx * gz);
    // never a few workgroups more than one per CU: the CUs that get a second one take twice as long (264 workgroups
    // of the one-per-CU shape took 141 us where 240 take 100; the QKV projection at 64 rows 20.7 us with 288
    // workgroups, 16.2 us with 240)
    // (except that two slices on two workgroups per CU beat one slice on fewer workgroups than CUs, for the shapes
    // that fit two on a CU: 384 workgroups 65 us, 192 workgroups 73 us; but 192 with two slices 40 us, 288 with
    // three 46 us)
    const bool one_per_cu = mt * nf > 8 || (mt == 4 && prologue != PRO_NONE);
    if (!tn.linear_ksplit && gx * gz * ksplit > kNumCU && gx * gz <= kNumCU) {
        const int fl = kNumCU / (gx * gz);
        if (one_per_cu || fl >= 2) ksplit = fl;
    }
    if (ksplit > chunks / 2) ksplit = chunks / 2;
    if (ksplit > max_split) ksplit = max_split;
    if (!sliceable) ksplit = 1;
    if (ksplit < 1) ksplit = 1;
    int cps = (chunks + ksplit - 1) / ksplit;
    ksplit = (chunks + cps - 1) / cps;  // no empty slices
    // The rules above come from sweeps at the 8B and 70B widths.  Elsewhere they can leave most of the chip idle (128-row tiles of 512
    // columns from 384 rows on: 48 workgroups for a gate/up of 4096 columns) or double the rounds of the grid, and a short K is
    // sliced into ramps.  So any other shape whose estimate is 5 % below theirs takes their place.  Slices stay at most 1024 long
    // (or as long as theirs): longer sums would round a little more.
    //   gate/up, us: 4096 columns, K = 4096, 384 rows 162 -> 63; 5632, K = 2048, 512 rows 85 -> 56; 1376, K = 4096, 160 rows 55 -> 33;
    //   512 shapes of the sweep 0.88 of the time on average, none over 1.01.
    //   sliced, with the sum of the slices: 8192 x 512, 512 rows 36 -> 14; 6144 x 4096, 384 rows 58 -> 53; 2048 x 2048, 100 rows
    //   16 -> 12; 462 shapes 0.88, none over 1.04.  (Up to 32 rows their choice is within 3 % of the best everywhere.)
    // At the widths of the sweeps and up to 256 rows it replaces, inside a step, us a launch by the rules -> now:
    //   8B QKV at 65 .. 96 rows 20.6 -> 18.9 (96-row tiles of 256 columns in 10 slices -> of 128 in 5) and O 17.0 -> 15.6, with less for
    //   the rotation (6.1 -> 4.8) and the norms (12.9 -> 11.7 a layer) to add up; O at 129 .. 192 rows 20.0 -> 17.5 (8 slices of 96-row
    //   tiles -> 5 of 64-row ones); 70B QKV at 129 .. 192 rows 72.8 -> 64.9 (3 slices -> 4), down at 129 .. 152 rows 173.6 -> 175.6 and at
    //   193 .. 223 187.4 -> 187.5 (4 -> 8); the head of 128256 columns at 96 rows 238 -> 226, at K = 8192 473 -> 444.
    //   Error of a product against 64 bits, in 1e-6 of it: 8B QKV 2.456 -> 2.461 (slices of 448 and 832 inputs), O 2.451 -> 2.454 and
    //   2.463 -> 2.468, 70B QKV 2.498 -> 2.488, down 2.573 -> 2.513.
    if (!swept && prologue == PRO_NONE && M > 32 && !tn.linear_mt && !tn.linear_nf && !tn.linear_ksplit && !tn.linear_ks && tn.linear_target_blocks == kNumCU) {
        // A pure function of these sizes, 1 .. 3 us of the host's time: a thread keeps its last 32 answers, which are looked through one by
        // one (some 20 ns).  A step of many layers asks for five products again and again, so all five have to stay, whatever their widths.
        struct Answer {
            int N, K, M, most, slices, mt, nf, ksplit, cps;
        };
        static thread_local Answer answers[32];
        static thread_local unsigned next = 0;
        const int most = sliceable ? max_split : 1;
        const Answer* known = nullptr;
        for (const Answer& e : answers)
            if (e.N == L.N && e.K == L.K && e.M == M && e.most == most && e.slices == slices) {
                known = &e;
                break;
            }
        if (!known) {
            Answer& e = answers[next++ % 32];
            e = Answer{L.N, L.K, M, most, slices, mt, nf, ksplit, cps};
            by_estimate(L, M, KC, most, slices, e.mt, e.nf, e.ksplit, e.cps);
            ++linear_shape_searches();
            known = &e;
        }
        const Answer& a = *known;
        mt = a.mt;
        nf = a.nf;
        ksplit = a.ksplit;
        cps = a.cps;
        gx = (tiles + 4 * nf - 1) / (4 * nf);
        gz = (M + 32 * mt - 1) / (32 * mt);
        ks8 = ring8();
        ks16 = ring16();
        if (!sliceable) cps = (L.K + (ks16 ? 256 : (ks8 ? 128 : 64)) - 1) / (ks16 ? 256 : (ks8 ? 128 : 64));
    }
    // Eight waves instead of four over the same columns where that pays: two waves per SIMD, of which one multiplies while
    // the other converts activations or waits.  Measured (whole calls, one device):
    //   128 rows x 512 columns: the 8B-wide feed-forward block of 2048 rows 1160 -> 1144 us, two layers and the head at 500
    //     requests 3114 -> 3088 us (and no accumulator spills);
    //   64 x 256 with several M-tiles: four layers of 128 rows 1110 -> 1096 us; 200 rows of 5632 gate/up columns at K = 2048
    //     33.6 -> 30.4; with one M-tile 64 rows get 0.3 % slower, the workgroup then being short of bytes in flight and not of
    //     issue slots.
    // One 128 x 256 tile for two of 64 x 512 (97..128 rows, K sliced) was tried: level within a step, but 3..10 % slower as a
    // projection by itself (128 rows, 8192 x 28672: 144 against 130 us), so wide outputs keep 64-row tiles there.
    // 64 x 512 shows no difference, pre-split input 1 % less.
    int nw = 4;
    if (prologue == PRO_NONE) {
        if (mt == 4 && nf == 4) {
            nw = 8;
            nf = 2;
        } else if (mt == 2 && nf == 2 && gz > 1 && !ks8) {
            nw = 8;
            nf = 1;
        }
    }
    return LinearShape{mt, nf, nw, ks16 ? 16 : (ks8 ? 8 : 4), gx, gz, ksplit, cps};
}

int linear_slices(const Linear& L, int M, int prologue, int max_split, SliceCost slices) {
    return M > 0 ? linear_shape(L, M, true, prologue, max_split, slices).ksplit : 1;
}

int32_t launch_linear(const Linear& L, const float* A, int lda, int M, float* y, int ldy, int epilogue, int prologue,
                      float* part, int max_split, int* ksplit_out, uint16_t* asplit, hipStream_t st, const NormIn* norm, SliceCost slices) {
    if (ksplit_out) *ksplit_out = 1;
    if (M == 0) return CHIRON_OK;
    if (norm && (max_split > 1 || prologue != PRO_NONE || M > 16 || !linear_few_rows(M)))
        return fail(CHIRON_ERR_INVALID_ARG, "linear: a norm in the operand load needs an unsliced launch of few rows");
    if (epilogue != EPI_STORE && epilogue != EPI_ADD && epilogue != EPI_SWIGLU && epilogue != EPI_SWIGLU_PACKED && epilogue != EPI_SWIGLU_FEW)
        return fail(CHIRON_ERR_INVALID_ARG, "linear: unknown epilogue %d", epilogue);
    if (epilogue >= EPI_SWIGLU) {
        // gate and up of one column must meet in one workgroup with the whole sum over K
        if (max_split > 1) return fail(CHIRON_ERR_INVALID_ARG, "linear: the SwiGLU epilogue cannot slice K");
        if (L.N % 32 != 0) return fail(CHIRON_ERR_SHAPE, "linear: a fused gate/up matrix has a multiple of 32 rows (got %d)", L.N);
        if (ldy % (epilogue == EPI_SWIGLU ? 4 : 8) != 0 || ((uintptr_t)y & 15))
            return fail(CHIRON_ERR_INVALID_ARG, "linear: SwiGLU output rows must be 16-byte aligned");
    }
    if (asplit && prologue != PRO_PACKED && M >= linear_big_min_rows(L) && tuning().linear_big_all)
        return launch_linear_big(L, A, lda, M, y, ldy, epilogue, part, max_split, ksplit_out, asplit, st);
    if (L.K % 16 != 0 || L.K < 16) return fail(CHIRON_ERR_SHAPE, "linear: K=%d must be a positive multiple of 16", L.K);
    if (prologue != PRO_PACKED && (lda % 4 != 0 || ((uintptr_t)A & 15)))
        return fail(CHIRON_ERR_INVALID_ARG, "linear: input rows must be 16-byte aligned");
    const LinearShape shape = linear_shape(L, M, max_split > 1, prologue, max_split, slices);
    const int mt = shape.mt, nf = shape.nf, nw = shape.nw, gx = shape.gx, gz = shape.gz, ksplit = shape.ksplit, cps = shape.cps;
    const bool ks8 = shape.ks == 8, ks16 = shape.ks == 16;
    if (ksplit > 1 && !part) return fail(CHIRON_ERR_INVALID_ARG, "linear: no workspace for %d K-slices", ksplit);
    int mode = ksplit > 1 ? EPI_SLICES : epilogue;
    float* dst = ksplit > 1 ? part : y;
    int ldd = ksplit > 1 ? L.N : ldy;
    size_t part_stride = (size_t)M * L.N;
    if (epilogue == EPI_SWIGLU_PACKED) {  // ldy: the consumer's padded K
        ldd = ldy / 8;
        part_stride = linear_big_split_elems(M, ldy) / 8;
    } else if (epilogue == EPI_SWIGLU_FEW) {
        part_stride = (size_t)M * (ldy / 8);
    }
    int nblocks = (gx * ksplit * gz + 7) / 8 * 8;
#define CHIRON_LAUNCH(MT_, NF_) launch_cfg<MT_, NF_, PRO_NONE>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz)
    if (norm) {  // at most 16 rows, unsliced: one of these three
        if (ks16) launch_cfg<1, 1, PRO_NONE, 16, true, true>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz, *norm);
        else if (mt == 1 && nf == 2) launch_cfg<1, 2, PRO_NONE, 4, true, true>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz, *norm);
        else if (mt == 2 && nf == 4) launch_cfg<1, 4, PRO_NONE, 4, true, true>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz, *norm);
        else return fail(CHIRON_ERR_INVALID_ARG, "linear: no shape with the norm for %d rows of %d columns", M, L.N);
    } else if (ks16) {
        launch_cfg<1, 1, PRO_NONE, 16>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (ks8 && mt == 3) {
        launch_cfg<3, 1, PRO_NONE, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (ks8) {
        if (nf == 1) launch_cfg<2, 1, PRO_NONE, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else launch_cfg<2, 2, PRO_NONE, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (prologue == PRO_PACKED) {
        // several M-tiles re-read the weights through the L2: no streaming hint then
        if (nf == 4 && gz > 1) launch_cfg<4, 4, PRO_PACKED, 4, false>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else if (nf == 4) launch_cfg<4, 4, PRO_PACKED>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else if (gz > 1) launch_cfg<4, 2, PRO_PACKED, 4, false>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else launch_cfg<4, 2, PRO_PACKED>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (nw == 8) {
        const int tiles = gx * gz;
        if (mt == 4 && nf == 2 && gz > 1 && ksplit == 1 && halved_last_round(tiles)) {
            const int whole = tiles / kNumCU * kNumCU, blocks = whole + (2 * (tiles - whole) + 7) / 8 * 8;
            launch(linear_wide_kernel, dim3(blocks), dim3(512), st, L.w, L.tstride, L.Npad, L.N, L.K, L.Kpad, A, lda, M, dst, ldd, mode, part_stride, gx, gz,
                   whole, tuning().linear_xcd_remap);
        } else if (mt == 4 && nf == 2 && gz > 1) launch_cfg<4, 2, PRO_NONE, 4, false, false, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else if (mt == 4 && nf == 2) launch_cfg<4, 2, PRO_NONE, 4, true, false, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
        else launch_cfg<2, 1, PRO_NONE, 4, true, false, 8>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (nf == 4) {
        launch_cfg<2, 4, PRO_NONE>(nblocks, st, L, A, lda, M, dst, ldd, cps, mode, part_stride, gx, ksplit, gz);
    } else if (mt == 1 && nf == 1) CHIRON_LAUNCH(1, 1);
    else if (mt == 1) CHIRON_LAUNCH(1, 2);
    else if (mt == 2 && nf == 1) CHIRON_LAUNCH(2, 1);
    else if (mt == 2) CHIRON_LAUNCH(2, 2);
    else if (mt == 3 && nf == 1) CHIRON_LAUNCH(3, 1);
    else if (mt == 3) CHIRON_LAUNCH(3, 2);
    else if (nf == 1) CHIRON_LAUNCH(4, 1);
    else CHIRON_LAUNCH(4, 2);
#undef CHIRON_LAUNCH
    CHIRON_HIP(hipGetLastError());
    if (ksplit_out) *ksplit_out = ksplit;
    return CHIRON_OK;
}

}  // namespace chiron
