// The attention work list: its layout in memory and the workgroup that builds it from seq_lens on the device.
// Device code shared by the kernel that begins a decode step and the single attention entry point.
#pragma once

#include "chiron_internal.h"
#include "device_util.h"

namespace chiron {

// plan buffer layout (int32): [0] n_items, [1] chunk_pages, [2..3] unused,
// [4, 4+max_batch) first item of pass v, [.., +max_batch) number of items of pass v.
// A pass v = request * ng + token group (AttnShape).
// Then, 32-byte aligned, one record of 8 ints per item: {pass, first page, attended length, the ids of the item's
// first four pages (past its end: its last page), 0}: everything a wave needs before its first tile load, in one
// scalar load instead of a chain of four dependent ones (the block table does not differ between layers).
// After the records, kTicketQueues ticket counters kTicketStride ints apart, all 0 between attention launches.
__host__ __device__ inline int64_t plan_rec_offset(int max_batch) { return (4 + 2 * (int64_t)max_batch + 7) / 8 * 8; }
constexpr int kTicketQueues = 8, kTicketStride = 64;
__host__ __device__ inline int64_t plan_ticket_offset(int max_batch, int cap_items) {
    return (plan_rec_offset(max_batch) + 8 * (int64_t)cap_items + kTicketStride - 1) / kTicketStride * kTicketStride;
}

constexpr int kPlanThreads = 1024;  // threads of the workgroup that runs attn_plan_block
constexpr int kPlanCached = 2048;   // passes whose page counts and offsets are kept in LDS

struct PlanArgs {
    int32_t* plan;
    const int32_t* seq_lens;
    const int32_t* bt;
    AttnShape sh;
    int max_batch, cap_items, batch, n_kv, slots, target_waves, force_cp, item_limit, max_blocks;
};

// positions attended by pass v (its last token's view)
__device__ __forceinline__ int pass_len(const int32_t* __restrict__ seq_lens, const AttnShape& sh, int v) {
    const int i = v / sh.ng, g = v - i * sh.ng;
    return seq_lens[i] + sh.bias0 + g * sh.tg + min(sh.tg, sh.q_len - g * sh.tg);
}

// One workgroup of kPlanThreads threads.  It is a chain of workgroup-wide sums and of dependent loads, so it keeps the
// page counts in LDS, sums through wave shuffles (one barrier per sum), and deals the records out item by item (an
// item's request is found by bisection), not request by request: one long request is no serial loop of one thread.
// Measured on the attention entry point: 664 -> 646 us at 32 requests of 28k tokens, where the serial loop took 28 us.
__device__ __forceinline__ void attn_plan_block(const PlanArgs& a) {
    __shared__ int s_np[kPlanCached], s_off[kPlanCached];
    __shared__ int s_sum[2][kPlanThreads / 64];
    const AttnShape sh = a.sh;
    const int batch = a.batch * sh.ng;  // passes
    const int max_batch = a.max_batch, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int32_t* plan = a.plan;
    int32_t* seq_item0 = plan + 4;
    int32_t* seq_nch = plan + 4 + max_batch;
    if (tid < kTicketQueues) plan[plan_ticket_offset(max_batch, a.cap_items) + tid * kTicketStride] = 0;
    for (int v = tid; v < min(batch, kPlanCached); v += kPlanThreads) s_np[v] = (pass_len(a.seq_lens, sh, v) + kBlockSize - 1) / kBlockSize;
    __syncthreads();
    auto pages_of = [&](int v) { return v < kPlanCached ? s_np[v] : (pass_len(a.seq_lens, sh, v) + kBlockSize - 1) / kBlockSize; };
    const int per = (batch + kPlanThreads - 1) / kPlanThreads;  // requests per thread, contiguous
    const int i0 = min(batch, tid * per), i1 = min(batch, i0 + per);

    // workgroup-wide sum, every thread gets the total; two buffers in turn, so that one barrier per sum is enough
    int turn = 0;
    auto block_sum = [&](int v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) s_sum[turn][wave] = v;
        __syncthreads();
        int t = 0;
#pragma unroll
        for (int k = 0; k < kPlanThreads / 64; ++k) t += s_sum[turn][k];
        turn ^= 1;
        return t;
    };
    auto count_items = [&](int cp) {
        int n = 0;
        for (int i = i0; i < i1; ++i) n += (pages_of(i) + cp - 1) / cp;
        return block_sum(n);
    };
    const int total = count_items(1);

    // Pages per item.  A wave takes items w, w + slots, ...: if the list is only a little longer than the number of
    // wave slots, a few waves run a second item alone, at latency-bound speed, after everyone else has finished.
    // So: when one round can hold everything, take the smallest item size that fits one round (all items stream
    // concurrently); otherwise make the items small enough for at least four rounds, where a ragged last round
    // costs little, but not so small that the per-item partial result weighs against the bytes the item reads.
    int cp;
    if ((int64_t)count_items(64) * a.n_kv <= a.slots) {
        int lo = 2, hi = 64;
        while (lo < hi) {  // uniform over the workgroup: every thread sees the same counts
            const int mid = (lo + hi) / 2;
            if ((int64_t)count_items(mid) * a.n_kv <= a.slots) hi = mid;
            else lo = mid + 1;
        }
        cp = lo;
    } else {
        cp = 64;
        while (cp > 8 && (int64_t)(total / cp) * a.n_kv < a.target_waves) cp >>= 1;
    }
    while (cp < (1 << 24) && total / cp + batch > a.item_limit) cp <<= 1;  // the host has checked that batch < item_limit
    if (a.force_cp > 0 && total / a.force_cp + batch <= a.item_limit) cp = a.force_cp;

    // exclusive scan of items per request
    int items = 0;
    for (int i = i0; i < i1; ++i) items += (pages_of(i) + cp - 1) / cp;
    int scan = items;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(scan, o);
        if (lane >= o) scan += v;
    }
    if (lane == 63) s_sum[turn][wave] = scan;
    __syncthreads();
    int off = scan - items, n_items = 0;
#pragma unroll
    for (int k = 0; k < kPlanThreads / 64; ++k) {
        if (k < wave) off += s_sum[turn][k];
        n_items += s_sum[turn][k];
    }
    for (int i = i0; i < i1; ++i) {
        const int nch = (pages_of(i) + cp - 1) / cp;
        if (i < kPlanCached) s_off[i] = off;
        seq_item0[i] = off;
        seq_nch[i] = nch;
        off += nch;
    }
    if (tid == 0) {
        plan[0] = n_items;
        plan[1] = cp;
    }
    __syncthreads();  // (also orders the offsets past kPlanCached, which this workgroup reads back from global memory)

    int4* recs = reinterpret_cast<int4*>(plan + plan_rec_offset(max_batch));
    for (int it = tid; it < n_items; it += kPlanThreads) {
        int lo = 0, hi = batch - 1;  // the last pass whose first item is not past `it`
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            const int first = mid < kPlanCached ? s_off[mid] : seq_item0[mid];
            if (first <= it) lo = mid;
            else hi = mid - 1;
        }
        const int pg0 = (it - (lo < kPlanCached ? s_off[lo] : seq_item0[lo])) * cp;
        const int last = min(pg0 + cp, pages_of(lo)) - 1;
        const int32_t* btrow = a.bt + (size_t)(lo / sh.ng) * a.max_blocks;
        const int b0 = btrow[pg0], b1 = btrow[min(pg0 + 1, last)], b2 = btrow[min(pg0 + 2, last)], b3 = btrow[min(pg0 + 3, last)];
        recs[2 * it] = make_int4(lo, pg0, pass_len(a.seq_lens, sh, lo), b0);
        recs[2 * it + 1] = make_int4(b1, b2, b3, 0);
    }
}

}  // namespace chiron
