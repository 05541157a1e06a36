// The work list of the attention (see attn_bf16.hip): built once per forward pass by one workgroup, next to whatever else the pass starts with.
#pragma once
#include "common.h"

namespace specv {

constexpr int ATT_CP_MAX = 256;              // longest chunk (pages per workgroup): a wavefront's page ids sit in one register
constexpr int KV_ERR_BOUND = 8;              // error bit: more work items than the launch was sized for
constexpr int ATT_WAVES = 4;

// One work item: pages [page0, page_end) of batch entry b (sequence seq, cached length ctx, `total` keys visible to the
// last row; b = -1: unused slot of the list).  32 bytes, read with two 16-byte loads.
struct AttnItem { int32_t b, seq, page0, page_end, ctx, total, chunk, pad; };

// What the attention takes the new rows' queries, keys and values from: the K-split slices of the QKV projection (row m = b T + i, columns
// q heads | k heads | v heads of 128) and cos, sin of every row's 64 angles.
struct QkvSlices { const float* part; int splits; int64_t split_stride; int ld; const float2* rope; };

struct AttnPlanArgs { int budget, min_pages, alone_pages, forced, max_items; AttnItem* items; int2* entry_items; };

constexpr int PLAN_KEPT = 1024;              // batch entries whose page counts are kept in LDS

// The whole workgroup (a multiple of 64 threads, at most 1024).  pages(b) = pages holding the keys batch entry b may see
// (0 for a dropped entry).  Chunk length L: the smallest multiple of 4 in [min_pages, 256] with sum_b ceil(pages(b) / L)
// <= budget (256 if none; `forced` > 0 fixes L instead); entry b then has n = ceil(pages / L) items of
// ceil(pages / n) pages rounded up to a multiple of 4 (the 4 wavefronts take every 4th page).  While chunks of up to alone_pages (0 if the list is cut for several rounds) make at most
// half that many items, no CU gets two of them: each costs the sums of its queries and a share of the merge, and a CU with two takes
// as long as one chunk of twice the length (8B shape, us a step or eight layers of it: 7 sequences of 1k-8k 4 102 -> 4 042, two of 7k-8k 1 041 -> 1 017, four of
// 500-4 000 with 8-bit matrices and cache 737 -> 705; chunks beyond 120 pages gain nothing or lose, 23 sequences of 500-4 000 1 560 -> 1 575).  Items are listed in batch
// order; entry_items[b] = (first item, number of items).  Slots of the list beyond the last item get b = -1.  More
// items than max_items (contexts beyond the bound the launch was sized for) set KV_ERR_BOUND and are dropped.
// A chain of dependent steps on one workgroup: 7.7, 11 and 23 us at 5, 64 and 256 entries as a launch of its own that read the bookkeeping
// again for every candidate length; now 6-9 us beside the embedding and the rotary table.
__device__ inline void attn_plan(int B, int T, const KvView& kv, const AttnPlanArgs& a)
{
    __shared__ int s_pages[PLAN_KEPT], s_cnt[1024], s_wave[16], s_len, s_carry;
    const int threads = blockDim.x, waves = threads >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    auto pages_of = [&](int b, int& seq, int& ctx, int& total) {
        seq = kv.entry_seq[b];
        ctx = total = 0;
        if (seq >= 0) {
            ctx = kv.ctx_len[seq];
            total = ctx + T;
            const int cap = kv.n_held[seq] * SPEC_PAGE_SIZE;
            if (total > cap) total = cap;
        }
        return (total + SPEC_PAGE_SIZE - 1) / SPEC_PAGE_SIZE;
    };
    auto div_up = [](int p, int len, float r) {                          // ceil(p / len); r = 1 / len, page counts are below 2^24
        const int n = p + len - 1;
        int q = (int)((float)n * r);
        const int rest = n - q * len;
        return rest < 0 ? q - 1 : (rest >= len ? q + 1 : q);
    };
    int seq, ctx, total;
    for (int b = threadIdx.x; b < B && b < PLAN_KEPT; b += threads) s_pages[b] = pages_of(b, seq, ctx, total);
    __syncthreads();
    {
        // candidate `lane`: chunks of 4 (lane + 1) pages; a wavefront counts them over every `waves`-th entry
        const int len = 4 * (lane + 1);
        const float r = 1.0f / (float)len;
        int cnt = 0;
        for (int b = wave; b < B; b += waves) cnt += div_up(b < PLAN_KEPT ? s_pages[b] : pages_of(b, seq, ctx, total), len, r);
        s_cnt[threadIdx.x] = cnt;
        __syncthreads();
        if (wave == 0) {
            cnt = 0;
            for (int w = 0; w < waves; ++w) cnt += s_cnt[w * 64 + lane];
            const unsigned long long fits = __builtin_amdgcn_ballot_w64(len >= a.min_pages && cnt <= a.budget);
            const unsigned long long alone = __builtin_amdgcn_ballot_w64(len >= a.min_pages && len <= a.alone_pages && 2 * cnt <= a.budget);
            const unsigned long long take = alone ? alone : fits;
            if (lane == 0) {
                s_len = a.forced > 0 ? a.forced : (take ? 4 * (__builtin_ctzll(take) + 1) : ATT_CP_MAX);
                s_carry = 0;
            }
        }
        __syncthreads();
    }
    const int L = s_len;
    for (int base = 0; base < B; base += threads) {
        const int b = base + threadIdx.x;
        const int p = b < B ? pages_of(b, seq, ctx, total) : 0, n = (p + L - 1) / L;
        // exclusive scan of n over the workgroup
        int upto = n;
        for (int off = 1; off < 64; off <<= 1) {
            const int add = __shfl_up(upto, off);
            if (lane >= off) upto += add;
        }
        if (lane == 63) s_wave[wave] = upto;
        __syncthreads();
        int first = s_carry + upto - n, group_total = 0;
        for (int w = 0; w < waves; ++w) {
            if (w < wave) first += s_wave[w];
            group_total += s_wave[w];
        }
        __syncthreads();
        if (b < B) {
            const int len = n > 0 ? ((p + n - 1) / n + ATT_WAVES - 1) / ATT_WAVES * ATT_WAVES : 0;
            int wrote = 0;
            for (int c = 0; c < n; ++c) {
                const int it = first + c;
                if (it >= a.max_items) break;
                AttnItem x;
                x.b = b; x.seq = seq; x.page0 = c * len; x.page_end = (c + 1) * len < p ? (c + 1) * len : p;
                x.ctx = ctx; x.total = total; x.chunk = c; x.pad = 0;
                a.items[it] = x;
                ++wrote;
            }
            a.entry_items[b] = make_int2(first < a.max_items ? first : 0, wrote);
            if (wrote < n) atomicOr(kv.error, KV_ERR_BOUND);
        }
        if (threadIdx.x == 0) s_carry += group_total;
        __syncthreads();
    }
    const int n_items = s_carry < a.max_items ? s_carry : a.max_items;
    for (int it = n_items + threadIdx.x; it < a.max_items; it += threads) {
        AttnItem x;
        x.b = -1; x.seq = -1; x.page0 = 0; x.page_end = 0; x.ctx = 0; x.total = 0; x.chunk = 0; x.pad = 0;
        a.items[it] = x;
    }
}

}  // namespace specv
