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
template <int MT, int NF, int KS, int PRO, bool WNT = true, bool NORM = false, int NW = 4>
__global__ __launch_bounds__(64 * NW, (NW == 8 || (MT * NF <= 8 && !(MT == 4 && PRO != PRO_NONE)) ? 2 : 1)) void linear_kernel(const uint16_t* __restrict__ Wp, size_t tstride, int Npad, int Nreal, int K, int Kpad,
                                                     const float* __restrict__ A, int lda, int M,
                                                     float* __restrict__ Y, int ldy, int chunks_per_split,
                                                     int mode, size_t part_stride, int gx, int gy, int gz, int remap,
                                                     const uint16_t* __restrict__ gain, float eps) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Workgroups are dealt to the 8 XCDs round-robin.  The 1-D grid is re-read so that consecutive logical ids
    // sit on ONE XCD, and the M-tile index varies fastest: the workgroups that stream the same weight tiles for
    // different rows then share that XCD's L2 instead of each pulling the tile from HBM.
    const int total = gx * gy * gz;
    const int per_xcd = (total + 7) / 8;
    const int logical = remap ? (blockIdx.x % 8) * per_xcd + blockIdx.x / 8 : blockIdx.x;
    if (logical >= total) return;  // grid is padded to a multiple of 8 (uniform over the workgroup)
    const int bz = logical % gz, bx = (logical / gz) % gx, by = logical / (gz * gx);
#include "linear_tile.inc"
}

// 128 rows x 512 columns by eight waves, K whole.  The tiles of whole rounds of the chip as they are (`whole` of them, a multiple of
// 256), those of a last round that would be at most half full as two of 128 x 256, which then fill it: 2048 rows of 28672
// columns at K = 4096 are 3.5 rounds.  Whole feed-forward blocks, us: 640 rows of 4096 -> 14336 -> 4096 455 -> 438, 1280 rows
// 795 -> 763, 1500 rows of 2048 -> 11008 -> 2048 415 -> 395, 2048 rows of the first 1158 -> 1147 (there the card's power is short: the
// clock falls as more of its matrix cores work).
__global__ __launch_bounds__(512, 2) void linear_wide_kernel(const uint16_t* __restrict__ Wp, size_t tstride, int Npad, int Nreal, int K, int Kpad,
                                                             const float* __restrict__ A, int lda, int M, float* __restrict__ Y, int ldy, int mode,
                                                             size_t part_stride, int gx, int gz, int whole, int remap) {
    constexpr int MT = 4, KS = 4, PRO = PRO_NONE, NW = 8, by = 0;
    constexpr bool WNT = false, NORM = false;
    constexpr const uint16_t* gain = nullptr;
    constexpr float eps = 0.f;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunks_per_split = (K + 63) / 64;
    if ((int)blockIdx.x < whole) {
        constexpr int NF = 2;
        const int tile = remap ? (int)(blockIdx.x % 8) * (whole / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
        const int bx = tile / gz, bz = tile % gz;
#include "linear_tile.inc"
    } else {
        constexpr int NF = 1;
        const int rest = gx * gz - whole, block = (int)blockIdx.x - whole, per_xcd = (2 * rest + 7) / 8;
        const int half = remap ? block % 8 * per_xcd + block / 8 : block;
        if (half >= 2 * rest) return;  // grid is padded to a multiple of 8 (uniform over the workgroup)
        const int tile = whole + half % rest;
        const int bx = 2 * (tile / gz) + half / rest, bz = tile % gz;
#include "linear_tile.inc"
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
