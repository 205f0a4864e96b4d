// The attention work list: its layout in memory and the workgroup that builds it from seq_lens on the device.
// Device code shared by the kernel that begins a decode step and the single attention entry point.
#pragma once

#include "chiron_internal.h"
#include "device_util.h"

namespace chiron {

// plan buffer layout (int32): [0] n_items, [1] chunk_pages, [2] number of long passes (more than kMergeLong items), [3] unused,
// [4, 4+max_batch) first partial result of pass v, [.., +max_batch) number of partial results of pass v (one per item, in
// page order), [.., +max_batch) and [.., +max_batch) scratch of the workgroup that builds the list: items placed before v's first and
// place of v's last piece if that is no whole item, of passes from kPlanCached on only (those before are in LDS, their words
// hold anything), [.., +max_batch) the long passes in any order.  A pass v = request * ng + token group (AttnShape).
// Then, 32-byte aligned, one record of 8 ints per item, in the order in which items are taken: {pass, first
// page, attended length, the ids of the item's first four pages (past its end: its last page), partial result}: everything a
// wave needs before its first tile load, in one scalar load instead of a chain of four dependent ones (the block table does
// not differ between layers).
// After the records, kTicketQueues ticket counters kTicketStride ints apart, all 0 between attention launches.
__host__ __device__ inline int64_t plan_rec_offset(int max_batch) { return (4 + 5 * (int64_t)max_batch + 7) / 8 * 8; }
constexpr int kTicketQueues = 8, kTicketStride = 64;
__host__ __device__ inline int64_t plan_ticket_offset(int max_batch, int cap_items) {
    return (plan_rec_offset(max_batch) + 8 * (int64_t)cap_items + kTicketStride - 1) / kTicketStride * kTicketStride;
}

constexpr int kPlanThreads = 1024;  // threads of the workgroup that runs attn_plan_block
constexpr int kPlanMaxRound = 4096; // largest item, in pages, of a list that one round of the grid holds
constexpr int kMergeLong = 16;      // a pass of more items is long for the merge
constexpr int kPlanCached = 2048;   // passes whose lengths and places are kept in LDS

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
// page counts in LDS, takes one barrier per sum, and deals the records out item by item (an
// item's request is found by bisection), not request by request: one long request is no serial loop of one thread.
// Measured on the attention entry point: 664 -> 646 us at 32 requests of 28k tokens, where the serial loop took 28 us.
// Sums go through the lanes' registers, what the workgroup reads back stays in LDS, and up to 64 passes all item sizes are counted at
// once: the kernel that begins a step 8.1 -> 4.9 us (toy decoder), 10.0 -> 6.5 (64 requests); attention of 8 requests 25.9 -> 22.6.
__device__ __forceinline__ void attn_plan_block(const PlanArgs& a) {
    __shared__ int s_len[kPlanCached], s_item0[kPlanCached], s_whole[kPlanCached], s_last[kPlanCached];
    __shared__ int s_sum[2][kPlanThreads / 64], s_scan[4][kPlanThreads / 64], s_count[64], s_long;
    const AttnShape sh = a.sh;
    const int batch = a.batch * sh.ng;  // passes
    const int max_batch = a.max_batch, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int32_t* plan = a.plan;
    int32_t* seq_item0 = plan + 4;
    int32_t* seq_nch = plan + 4 + max_batch;
    int32_t* seq_whole = plan + 4 + 2 * max_batch;
    int32_t* seq_last = plan + 4 + 3 * max_batch;
    int32_t* long_passes = plan + 4 + 4 * max_batch;
    if (tid == 0) s_long = 0;
    if (tid < kTicketQueues) plan[plan_ticket_offset(max_batch, a.cap_items) + tid * kTicketStride] = 0;
    for (int v = tid; v < min(batch, kPlanCached); v += kPlanThreads) s_len[v] = pass_len(a.seq_lens, sh, v);
    lds_barrier();
    auto len_of = [&](int v) { return v < kPlanCached ? s_len[v] : pass_len(a.seq_lens, sh, v); };
    auto pages_of = [&](int v) { return (len_of(v) + kBlockSize - 1) / kBlockSize; };
    const int per = (batch + kPlanThreads - 1) / kPlanThreads;  // requests per thread, contiguous
    const int i0 = min(batch, tid * per), i1 = min(batch, i0 + per);

    // workgroup-wide sum, every thread gets the total; two buffers in turn, so that one barrier per sum is enough
    int turn = 0;
    auto block_sum = [&](int v) {
        v = wave_total(v);
        if (lane == 0) s_sum[turn][wave] = v;
        lds_barrier();
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
    // Up to 64 passes: the counts of all item sizes up to 64 pages at once, four sizes a wave, instead of one sum over the workgroup
    // after the other (each a barrier and a trip through LDS, some 0.2 us; a search takes up to nine).
    const bool at_once = batch <= 64;
    if (at_once) {
        const int np = lane < batch ? pages_of(lane) : 0;
#pragma unroll
        for (int i = 0; i < 64 / (kPlanThreads / 64); ++i) {
            const int c = 1 + wave + i * (kPlanThreads / 64), n = wave_total((np + c - 1) / c);
            if (lane == 0) s_count[c - 1] = n;
        }
        lds_barrier();
    }
    const int total = at_once ? s_count[0] : count_items(1);

    // Pages per item.  Starting an item costs a wave a load latency or two, and an item that is left when the others have
    // run out streams alone, at a fraction of the rate (about 15 GB/s a wave).  So: when one round of the grid can hold
    // everything, take the smallest item size for which it does (all items stream concurrently, nothing is drawn), whatever
    // that size is as long as it leaves no more than a quarter of the round empty (32 requests of 24k .. 32k tokens: 227
    // pages 571 us, 32 pages in seven rounds 648 us; 96 requests of 2k tokens 187 against 214 us).  Otherwise items of
    // 64 pages (with 128 / 250 requests of both classes 193 / 382 us, with 16 pages 206 / 392), fewer pages only while
    // that does not fill one round.
    int cp = 0;
    bool drawn = true;  // whether waves draw further items after their first
    const auto fits = [&](int c) { return (int64_t)count_items(c) * a.n_kv <= a.slots; };  // uniform: every thread sees the same counts
    // the largest item that leaves no more than a quarter of the round's page slots empty
    const int full = (int)min((int64_t)kPlanMaxRound, (int64_t)total * a.n_kv * 4 / ((int64_t)a.slots * 3));
    const bool small = at_once ? (int64_t)s_count[63] * a.n_kv <= a.slots : fits(64);
    if (small && at_once) {
        const uint64_t fit = __ballot(lane > 0 && (int64_t)s_count[lane] * a.n_kv <= a.slots);  // counts fall with the size
        cp = __builtin_ctzll(fit) + 1;
        drawn = false;
    } else if (small || (full > 64 && fits(full))) {
        int lo = small ? 2 : (int)max((int64_t)65, (int64_t)total * a.n_kv / a.slots), hi = small ? 64 : full;
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (fits(mid)) hi = mid;
            else lo = mid + 1;
        }
        cp = lo;
        drawn = false;
    } else {
        cp = 64;
        while (cp > 8 && (int64_t)(total / cp) * a.n_kv < a.target_waves) cp >>= 1;
    }
    const int cp_rule = cp;
    while (cp < (1 << 24) && total / cp + batch > a.item_limit) cp <<= 1;  // the host has checked that batch < item_limit
    if (a.force_cp > 0 && total / a.force_cp + batch <= a.item_limit) cp = a.force_cp;
    drawn = drawn || cp != cp_rule;

    // The items in the order in which waves draw them: whole ones (cp pages) first, then the requests' last pieces of at
    // least half that, then the rest, so that what is drawn last is short (512 / 300 / 250 requests of both classes:
    // 744 -> 727, 464 -> 442, 379 -> 358 us).  In a single round nothing is drawn, and request order, which mixes long and
    // short items on a CU, is 2 us faster at 64 requests.
    // Exclusive scans over the requests of the numbers of items and, if drawn, of whole items, long and short last pieces.
    auto last_piece = [&](int np) { return np % cp; };
    int cnt[4] = {0, 0, 0, 0}, off[4], total4[4] = {0, 0, 0, 0};
    for (int i = i0; i < i1; ++i) {
        const int np = pages_of(i), r = last_piece(np);
        cnt[0] += (np + cp - 1) / cp;
        if (!drawn) continue;
        cnt[1] += np / cp;
        cnt[2] += r > 0 && 2 * r >= cp;
        cnt[3] += r > 0 && 2 * r < cp;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (c > 0 && !drawn) break;
        const int scan = wave_scan(cnt[c]);
        if (lane == 63) s_scan[c][wave] = scan;
        off[c] = scan - cnt[c];
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < kPlanThreads / 64; ++k) {
            if (c > 0 && !drawn) break;
            if (k < wave) off[c] += s_scan[c][k];
            total4[c] += s_scan[c][k];
        }
    const int n_whole = drawn ? total4[1] : total4[0];  // items placed by bisection: whole ones, or all in request order
    int4* recs = reinterpret_cast<int4*>(plan + plan_rec_offset(max_batch));
    auto put = [&](int it, int v, int ch, int partial) {  // the record of chunk ch of pass v
        const int pg0 = ch * cp, last = min(pg0 + cp, pages_of(v)) - 1;
        const int32_t* btrow = a.bt + (size_t)(v / sh.ng) * a.max_blocks;
        const int b0 = btrow[pg0], b1 = btrow[min(pg0 + 1, last)], b2 = btrow[min(pg0 + 2, last)], b3 = btrow[min(pg0 + 3, last)];
        recs[2 * it] = make_int4(v, pg0, len_of(v), b0);
        recs[2 * it + 1] = make_int4(b1, b2, b3, partial);
    };
    off[2] += n_whole;
    off[3] += n_whole + total4[2];
    for (int i = i0; i < i1; ++i) {
        const int np = pages_of(i), nch = (np + cp - 1) / cp, r = last_piece(np), before = drawn ? off[1] : off[0];
        if (i < kPlanCached) {
            s_whole[i] = before;
            s_item0[i] = off[0];
        } else seq_whole[i] = before;
        seq_item0[i] = off[0];
        seq_nch[i] = nch;
        if (nch > kMergeLong) long_passes[atomicAdd(&s_long, 1)] = i;
        if (drawn) {
            const int place = r == 0 ? -1 : (2 * r >= cp ? off[2]++ : off[3]++);
            if (i < kPlanCached) s_last[i] = place;
            else seq_last[i] = place;
        }
        off[0] += nch;
        if (drawn) off[1] += np / cp;
    }
    if (tid == 0) {
        plan[0] = total4[0];
        plan[1] = cp;
    }
    if (batch > kPlanCached) __syncthreads();  // this workgroup reads back from global memory what does not fit in LDS
    else lds_barrier();
    auto item0_of = [&](int v) { return v < kPlanCached ? s_item0[v] : seq_item0[v]; };
    if (tid == 0) plan[2] = s_long;
    for (int u = tid; u < n_whole + (drawn ? batch : 0); u += kPlanThreads) {
        if (u >= n_whole) {  // a last piece
            const int v = u - n_whole, place = v < kPlanCached ? s_last[v] : seq_last[v];
            if (place >= 0) put(place, v, pages_of(v) / cp, item0_of(v) + pages_of(v) / cp);
            continue;
        }
        const int it = u;
        int lo = 0, hi = batch - 1;  // the last pass with no more than `it` of these items before it
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            const int before = mid < kPlanCached ? s_whole[mid] : seq_whole[mid];
            if (before <= it) lo = mid;
            else hi = mid - 1;
        }
        const int ch = it - (lo < kPlanCached ? s_whole[lo] : seq_whole[lo]);
        put(it, lo, ch, drawn ? item0_of(lo) + ch : it);
    }
}

}  // namespace chiron
