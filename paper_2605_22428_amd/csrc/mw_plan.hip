// Send-side plan kernels: destination bitmaps, (bitmap, token) ordering, multicast
// groups, descriptor table and byte accounting.
//
// Paper hooks: the bitmap is Section 4.1's metadata encoding (bit r <-> rank r, ranks
// from zero, a preconfigured id -> rank table); groups are discovered per batch because
// the space of destination sets cannot be provisioned in advance (Section 2.3.2,
// C(64,8) sets at EP=64/top-8); the accounting is Section 1's "one copy however many
// destinations" against one copy per destination.
//
// No host synchronisation, launches on the caller's stream only:
//   k_plan_order  batches of up to 8192 tokens whose bitmaps have a 64-bit key (one word, or at most
//                 eight ids a token): every workgroup holds all keys and finishes a few tokens, nothing is
//                 exchanged between workgroups.  Above 2048 tokens k_plan_keys makes and sorts the keys first.
//   k_rank        otherwise (several words, more than eight ids): a workgroup owns 256 tokens and a
//                 slice of all tokens.  It builds the bitmaps of both from the top-k ids (one lane per
//                 token; the slice goes to LDS), then every lane counts, over the slice, the tokens whose
//                 (bitmap, index) is smaller than its own, and how many carry an equal bitmap before /
//                 at-or-after it.  Slices are spread over the whole chip and combined with one 64-bit
//                 integer atomic add per lane (a sum, so the result does not depend on arrival order).
//                 The workgroups of slice 0 also write the bitmaps out and turn 64 tokens'
//                 bitmaps into per-rank counts with wavefront ballots and popcounts.
//   k_groups      behind k_rank and the sorted chunks: workgroup b owns packed rows [256 b, 256 b + 256): it
//                 finds their tokens from the counts (predecessor count = packed row), writes perm, ranks
//                 the group starts (tokens with no equal bitmap before them) and writes their
//                 descriptors; a group's row count is the number of equal bitmaps.  Writing is
//                 spread over many workgroups because one CU retires only about one cache line
//                 of scattered stores per cycle.
// The count and histogram buffers are zero between plans: the k_groups workgroup that is the
// last to have read them clears them, so there is no clearing launch and no host-side state
// (a captured mw_plan can be replayed).
// Batches above 8192 tokens with keys take k_chunk_sort + k_merge_rank (sorted chunks, ranks by
// binary search: T log T instead of T^2) in k_rank's place; batches of at most 256 tokens can take
// k_plan_pack, which plans and packs in one launch.
#include "mw_internal.h"
#include "mw_plan_dev.h"

namespace {

constexpr int kBlock = 256;
template <int W>
__global__ __launch_bounds__(kBlock) void k_rank(const int32_t *__restrict__ topk, int T, int K,
                                                 const int32_t *__restrict__ eslot, int E, int slice,
                                                 uint64_t *__restrict__ mask_out,
                                                 unsigned long long *__restrict__ cnt,
                                                 uint32_t *__restrict__ pstate)
{
    extern __shared__ uint64_t smask[];
    mw_rank_body<W, false>(topk, T, K, eslot, E, slice, mask_out, cnt, pstate, blockIdx.x, blockIdx.y, kBlock, smask);
}

// For very large batches the walk below (every workgroup over every token's counters) is
// itself T^2 / 256 loads.  This kernel turns the counters into arrays indexed by packed row
// first -- perm, the row's counters and a "group starts here" byte -- so that k_groups<true>
// only sums the start bytes in front of its rows.
__global__ __launch_bounds__(kBlock) void k_rows_from_counters(int T, const unsigned long long *__restrict__ cnt,
                                                               const uint32_t *__restrict__ pstate,
                                                               int32_t *__restrict__ perm,
                                                               unsigned long long *__restrict__ row_cnt,
                                                               unsigned char *__restrict__ row_start)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= T) return;
    const uint32_t N = min(pstate[kPsKept], (uint32_t)T), n_empty = (uint32_t)T - N;
    const unsigned long long c = cnt[t];
    if ((c >> 42) == 0) return;                               // empty bitmap
    const uint32_t p = (uint32_t)(c & kField) - n_empty;
    if (p >= N) return;
    perm[p] = t;
    row_cnt[p] = c;
    row_start[p] = ((c >> 21) & kField) == 0 ? 1 : 0;
}

template <bool kByRow>
__global__ __launch_bounds__(kBlock) void k_groups(const uint64_t *__restrict__ mask, int T, uint64_t row_bytes,
                                                   unsigned long long *__restrict__ cnt,
                                                   uint32_t *__restrict__ pstate,
                                                   int32_t *__restrict__ perm, mw_group_desc *__restrict__ desc,
                                                   mw_send_stats *__restrict__ stats,
                                                   const unsigned long long *__restrict__ row_cnt,
                                                   const unsigned char *__restrict__ row_start)
{
    __shared__ int32_t tok[kBlock];
    __shared__ unsigned long long tokc[kBlock];     // the token's counters, so they are not fetched again
    __shared__ uint32_t scratch[17];
    const int tid = threadIdx.x;
    const uint32_t N = min(pstate[kPsKept], (uint32_t)T), n_empty = (uint32_t)T - N;
    const uint32_t i0 = blockIdx.x * kBlock;

    // every workgroup walks all tokens' counters (coalesced): which of them land in its rows,
    // how many groups start before its first row, how many groups there are.  Sixteen counters
    // per lane are requested before the first is looked at: one memory round trip per 4096 tokens.
    uint32_t starts_before = 0, starts_total = 0;
    if constexpr (kByRow) {
        // rows in front of this workgroup's, sixteen start bytes per load (i0 is a multiple of 256);
        // the first workgroup also counts all groups for the statistics
        const u32x4 *sb = (const u32x4 *)row_start;
        auto ones = [](u32x4 v) { return (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)); };
        for (uint32_t q = tid; q < i0 / 16; q += kBlock) starts_before += ones(sb[q]);
        if (blockIdx.x == 0) {
            for (uint32_t r = tid; r < N; r += kBlock) starts_total += row_start[r];
        }
        if (i0 + tid < N) { tok[tid] = perm[i0 + tid]; tokc[tid] = row_cnt[i0 + tid]; }
    } else
    for (int t0 = 0; t0 < T; t0 += 16 * kBlock) {
        unsigned long long cc[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int t = t0 + u * kBlock + tid;
            cc[u] = t < T ? cnt[t] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const unsigned long long c = cc[u];
            if ((c >> 42) == 0) continue;                         // empty bitmap (or past the end)
            const uint32_t p = (uint32_t)(c & kField) - n_empty;  // packed row of the token
            const uint32_t st = ((c >> 21) & kField) == 0 ? 1u : 0u;
            starts_total += st;
            starts_before += (st && p < i0) ? 1u : 0u;
            if (p - i0 < (uint32_t)kBlock && p < N) { tok[p - i0] = t0 + u * kBlock + tid; tokc[p - i0] = c; }
        }
    }
    uint32_t g_base, G;
    mw_block_exscan(starts_before, scratch, &g_base);
    mw_block_exscan(starts_total, scratch, &G);                // ends with a barrier: tok[] is complete

    const uint32_t i = i0 + tid;
    uint32_t st = 0;
    int32_t t = 0;
    unsigned long long c = 0;
    if (i < N) {
        t = tok[tid];
        if ((uint32_t)t >= (uint32_t)T) t = 0;      // (only counters corrupted by overlapping plans leave a row unclaimed)
        perm[i] = t;
        c = tokc[tid];
        st = ((c >> 21) & kField) == 0 ? 1u : 0u;
    }
    uint32_t local_total;
    const uint32_t g = g_base + mw_block_exscan(st, scratch, &local_total);
    if (st) {
        const uint64_t *m = mask + (size_t)t * MW_MASK_WORDS;
        mw_group_desc d;
        uint32_t nd = 0;
#pragma unroll
        for (int w = 0; w < MW_MASK_WORDS; ++w) { d.mask[w] = m[w]; nd += (uint32_t)__popcll(m[w]); }
        d.row_offset = i;
        d.row_count = (uint32_t)((c >> 42) & kField);          // equal bitmaps, this token included
        d.n_dest = nd;
        d.reserved0 = 0;
        if (g < (uint32_t)T) desc[g] = d;                      // (always, unless the counters were corrupted)
    }

    if (blockIdx.x == 0) {
        uint32_t dests = 0;
        for (int r = tid; r < MW_MAX_RANKS; r += kBlock) {
            const uint32_t h = pstate[r];
            stats->rows_per_dest[r] = h;
            dests += h;
        }
        uint32_t D;
        mw_block_exscan(dests, scratch, &D);
        if (tid == 0) {
            stats->n_rows = N;
            stats->n_groups = G;
            stats->multicast_bytes = (uint64_t)N * row_bytes;
            stats->unicast_bytes = (uint64_t)D * row_bytes;
            stats->error_flags = pstate[kPsFlags];
            stats->reserved0 = 0;
        }
    }

    // Leave the counters and the plan state zero for the next plan.  Nobody may clear them
    // while a workgroup still reads them: every workgroup reports when it has read all it
    // needs (its loads have returned: their values were used above), and the one that reports
    // last does the clearing (publication rules in mw_internal.h: the reports order every
    // workgroup's reads before the last one's stores).  The zeros are ordinary stores, read by
    // the next plan's kernels only.  With row-indexed arrays this kernel does not read the
    // counters at all, and every workgroup clears its own slice.
    __shared__ uint32_t i_am_last;
    mw_publish_barrier();
    if (tid == 0) i_am_last = mw_report(&pstate[kPsDone]) == gridDim.x - 1u ? 1u : 0u;
    if constexpr (kByRow) {
        if (i0 + tid < (uint32_t)T) cnt[i0 + tid] = 0;
    }
    __syncthreads();
    if (!i_am_last) return;
    if constexpr (!kByRow) {
        for (int z = tid; z < T; z += kBlock) cnt[z] = 0;
    }
    for (int r = tid; r < MW_PLAN_STATE_WORDS; r += kBlock) pstate[r] = 0;
}

// ---- the plan of a batch whose bitmaps have a 64-bit order-preserving key, at most 8192 tokens -------
// (bitmaps of one word, or of up to eight ranks anywhere: top_k <= 8.)  Every workgroup holds the keys of ALL
// tokens, a few a lane in registers, and finishes n_own of them by itself:
//   packed row   the number of tokens with (key, index) below: one 64-bit compare per 64 tokens, whose
//                result mask is counted by scalar instructions, or searches in sorted chunks of keys;
//   group index  the number of DISTINCT keys below: one token of every key is made its representative, and
//                the same compares or searches count the representatives.
// So no workgroup waits for another, nothing is summed up in global memory, nothing has to be cleared and
// one launch does it all; what it costs is that the keys are made once per workgroup.  Up to kKeysFrom
// tokens each workgroup makes them from the ids; beyond, a first launch makes them once and sorts them in chunks
// (k_plan_keys) and the workgroups only load them: 8 instead of 4 top_k bytes a token, no look-ups.
// Bound by latency and, from 4096 tokens on, by the instructions that all workgroups repeat (a dependent instruction 3.4
// ns, a block barrier with its LDS traffic about 0.1 us): of 15 us for 8192 tokens 3.4 are the first launch, 2 load and
// clear, 5 find the representatives and count ranks, 2 write the chunks, 2 search them.
// Before, with per-slice counts joined by global atomics and a second launch that inverted them (mw_plan
// alone, us): 1000 tokens 15.0 -> 5.4, 2048 15.8 -> 8.7, 4096 19.2 -> 10.8, 8192 33.9 -> 15.1 (256 ranks 37.3 -> 16.0).
//
// The key of a multi-word bitmap: its rank positions, highest first, a byte each; the highest as it
// is, the others plus one (they are at most 254, since a higher one precedes them), zero for "no further
// rank".  Comparing keys is comparing the bitmaps as numbers, and different bitmaps have different
// keys.  The key of a one-word bitmap is the word.
constexpr int kOrderBlock = 1024, kOrderMaxTokens = kPlanOrderMax, kOwnMax = 32;
constexpr int kOrderChunks = 64, kFilterBits = 32;       // (sorted) chunks of 8192 tokens; bits of each of the hash table's bitmaps for one slot

template <bool kBytes> struct mw_order_key {
    // a value no kept token's key has: marks free slots of the hash table.  (One word: 0 is the empty
    // bitmap.  Bytes: the third byte from the top is at most 254.)
    static constexpr uint64_t kNone = kBytes ? ~0ull : 0ull;
};

// Key of one token from its ranks plus one (0: no rank).
template <bool kBytes>
__device__ __forceinline__ uint64_t order_key_of(uint32_t (&v)[8])
{
    static_assert(kBytes, "one-word bitmaps are their own keys");
#define MW_CE(i, j) do { const uint32_t hi_ = max(v[i], v[j]), lo_ = min(v[i], v[j]); v[i] = hi_; v[j] = lo_; } while (0)
    MW_CE(0, 1); MW_CE(2, 3); MW_CE(4, 5); MW_CE(6, 7);          // odd-even merge sort of eight, descending
    MW_CE(0, 2); MW_CE(1, 3); MW_CE(4, 6); MW_CE(5, 7);
    MW_CE(1, 2); MW_CE(5, 6);
    MW_CE(0, 4); MW_CE(1, 5); MW_CE(2, 6); MW_CE(3, 7);
    MW_CE(2, 4); MW_CE(3, 5);
    MW_CE(1, 2); MW_CE(3, 4); MW_CE(5, 6);
#undef MW_CE
    uint64_t key = 0;
    int n = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool take = v[j] != 0 && (j == 0 || v[j] != v[j - 1]);       // a rank named twice counts once
        const uint32_t byte = n == 0 ? v[j] - 1u : v[j];
        key |= take ? (uint64_t)byte << (56 - 8 * n) : 0ull;
        n += take ? 1 : 0;
    }
    return n ? key : mw_order_key<true>::kNone;
}

// The bitmap a key stands for.
template <bool kBytes>
__device__ __forceinline__ void mask_of_key(uint64_t key, uint64_t (&m)[MW_MASK_WORDS])
{
#pragma unroll
    for (int q = 0; q < MW_MASK_WORDS; ++q) m[q] = 0;
    if (key == mw_order_key<kBytes>::kNone) return;
    if constexpr (!kBytes) {
        m[0] = key;
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t b = (uint32_t)(key >> (56 - 8 * j)) & 0xffu;
            if (j > 0 && b == 0) continue;
            const uint32_t r = j > 0 ? b - 1u : b;
#pragma unroll
            for (int q = 0; q < MW_MASK_WORDS; ++q) m[q] |= (r >> 6) == (uint32_t)q ? 1ull << (r & 63u) : 0ull;
        }
    }
}

// The first eight ids of kN tokens t, t + stride, ... of one lane, all requested together (past the last token
// the last one is read again: T > 0).
template <int kN>
__device__ __forceinline__ void load_ids(const int32_t *__restrict__ topk, int T, int K, int j0, int t, int stride, int32_t (&e)[kN][8])
{
    const bool wide = (K & 3) == 0 && ((uintptr_t)topk & 15u) == 0;        // id lists of whole 16-byte units
#pragma unroll
    for (int n = 0; n < kN; ++n) {
        const int32_t *row = topk + (size_t)min(t + n * stride, T - 1) * K + j0;
#pragma unroll
        for (int k = 0; k < 8; ++k) e[n][k] = -1;
        if (wide) {
            const u32x4 q = *(const u32x4 *)row;
            e[n][0] = (int32_t)q.x; e[n][1] = (int32_t)q.y; e[n][2] = (int32_t)q.z; e[n][3] = (int32_t)q.w;
            if (j0 + 4 < K) {
                const u32x4 p = *((const u32x4 *)row + 1);
                e[n][4] = (int32_t)p.x; e[n][5] = (int32_t)p.y; e[n][6] = (int32_t)p.z; e[n][7] = (int32_t)p.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) if (j0 + k < K) e[n][k] = row[k];
        }
    }
}

// Their keys.  `tab`: LDS table of rank + 1 per expert (0: none), entry E for ids outside [0, E); null: the rank
// table in memory.
template <bool kBytes, int kN>
__device__ __forceinline__ void keys_of_ids(int32_t (&e)[kN][8], const int32_t *__restrict__ topk, int T, int K,
                                            const int32_t *__restrict__ eslot, int E, const uint16_t *tab, int t, int stride,
                                            uint64_t (&key)[kN], bool &bad)
{
#pragma unroll
    for (int n = 0; n < kN; ++n) key[n] = 0;
    for (int j0 = 0; j0 < K; j0 += 8) {                                     // (one turn where keys are bytes)
        if (j0 > 0) load_ids<kN>(topk, T, K, j0, t, stride, e);
#pragma unroll
        for (int n = 0; n < kN; ++n) {
            uint32_t v[8], out = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t x = min((uint32_t)e[n][k], (uint32_t)E);
                if (tab) v[k] = tab[x];
                else { const int32_t q = x < (uint32_t)E ? eslot[x] : -1; v[k] = q < 0 ? 0u : (uint32_t)(q >> 16) + 1u; }
                out |= (x == (uint32_t)E && e[n][k] != -1) ? 1u : 0u;
            }
            bad |= out != 0 && t + n * stride < T;
            if constexpr (kBytes) {
                key[n] = order_key_of<true>(v);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) key[n] |= v[k] ? 1ull << ((v[k] - 1u) & 63u) : 0ull;
            }
        }
    }
#pragma unroll
    for (int n = 0; n < kN; ++n) if (t + n * stride >= T) key[n] = mw_order_key<kBytes>::kNone;
}

// LDS table of rank + 1 per expert: needs (E + 1) halfwords; entry E is 0.
__device__ __forceinline__ void fill_rank_table(uint16_t *tab, const int32_t *__restrict__ eslot, int E)
{
    for (int e = threadIdx.x; e <= E; e += (int)blockDim.x) {
        const int32_t q = e < E ? eslot[e] : -1;
        tab[e] = q < 0 ? (uint16_t)0 : (uint16_t)((q >> 16) + 1);
    }
}
constexpr int kTableExperts = 4095;        // experts of the LDS table (8 KiB); more: look-ups in memory

// First launch of the two-launch form: the keys of kChunkTokens tokens in (key, token) order, one below its value where a key
// is a bitmap (tokens without a destination then have ~0 in both kinds and come last), idx[i] the token of place i
// inside the chunk.  A chunk is ordered by counting: four lanes a token, each comparing it with 32 keys that all lanes read at
// once.  bad[wg]: one of the workgroup's ids was outside [0, E).
constexpr int kChunkTokens = 128, kKeysBlock = 4 * kChunkTokens;
template <bool kBytes>
__global__ __launch_bounds__(kKeysBlock) void k_plan_keys(const int32_t *__restrict__ topk, int T, int K,
                                                          const int32_t *__restrict__ eslot, int E,
                                                          uint64_t *__restrict__ keys, uint8_t *__restrict__ idx,
                                                          uint32_t *__restrict__ bad_out)
{
    extern __shared__ uint64_t keys_lds[];
    uint16_t *tab = E <= kTableExperts ? (uint16_t *)keys_lds : nullptr;
    __shared__ __align__(16) uint64_t val[kChunkTokens];
    __shared__ uint32_t below[4][kChunkTokens];
    __shared__ uint32_t any_bad;
    if (threadIdx.x == 0) any_bad = 0;
    const int i = threadIdx.x & (kChunkTokens - 1);
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kChunkTokens);
    const int t = blockIdx.x * kChunkTokens + i;
    int32_t e[1][8];
    if (part == 0) load_ids<1>(topk, T, K, 0, t, 0, e);
    if (tab) fill_rank_table(tab, eslot, E);
    mw_lds_barrier();
    uint64_t v = 0;
    if (part == 0) {
        uint64_t key[1];
        bool bad = false;
        keys_of_ids<kBytes, 1>(e, topk, T, K, eslot, E, tab, t, 0, key, bad);
        v = kBytes ? key[0] : key[0] - 1u;
        val[i] = v;
        if (bad) any_bad = 1;
    }
    mw_lds_barrier();
    if (part != 0) v = val[i];
    {
        const ulonglong2 *q = (const ulonglong2 *)(val + part * 32);
        const int half = __builtin_amdgcn_readfirstlane(i >> 6);             // the wave's tokens are one half of the chunk
        uint32_t n = 0;
        if ((part >> 1) < half) {                                            // keys of earlier tokens: equal ones count
#pragma unroll
            for (int u = 0; u < 16; ++u) { const ulonglong2 x = q[u]; n += (x.x <= v ? 1u : 0u) + (x.y <= v ? 1u : 0u); }
        } else if ((part >> 1) > half) {
#pragma unroll
            for (int u = 0; u < 16; ++u) { const ulonglong2 x = q[u]; n += (x.x < v ? 1u : 0u) + (x.y < v ? 1u : 0u); }
        } else {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const ulonglong2 x = q[u];
                const int j = part * 32 + 2 * u;
                n += (x.x < v || (x.x == v && j < i) ? 1u : 0u) + (x.y < v || (x.y == v && j + 1 < i) ? 1u : 0u);
            }
        }
        below[part][i] = n;
    }
    mw_lds_barrier();
    if (part == 0 && t < T) {
        const uint32_t at = blockIdx.x * kChunkTokens + below[0][i] + below[1][i] + below[2][i] + below[3][i];
        keys[at] = v;
        idx[at] = (uint8_t)i;
    }
    if (threadIdx.x == 0) bad_out[blockIdx.x] = any_bad;
}

// kU: tokens a lane holds (T <= kU blockDim.x).
// kFew: so few keys are possible that nearly every wave has one like a token's (the rule is where it is launched): equals are counted
// without asking whether there are any.
// kSorted: keys, idx and bad[n_bad] come from k_plan_keys, and what counts the keys below a token's is a binary search in every
// chunk, a lane a chunk: 64 chunks of 8192 tokens cost a wave eight LDS reads a lane, however the keys are spread.  A wave holds
// whole chunks, so a running count of the representatives inside a chunk turns the same searches into the group index.
// (With the keys counted into 4096 buckets and a token compared with its bucket, 8192 tokens of 256 ranks with skewed ids
// spent 7 us in the buckets' atomics, 2 in their scan and 6 in the compares of 24; the searches take 2.)
// pstate: only its flag word is looked at (mw_plan_static reports bad table entries there).
template <bool kBytes, int kU, bool kSorted, bool kFew>
__global__ __launch_bounds__(kOrderBlock) void k_plan_order(
    const int32_t *__restrict__ topk, int T, int K, const int32_t *__restrict__ eslot, int E, int R, int n_own, int slots_log,
    const uint64_t *__restrict__ keys, const uint8_t *__restrict__ idx, const uint32_t *__restrict__ bad_in, int n_bad,
    const uint32_t *__restrict__ pstate,
    uint64_t row_bytes, uint64_t *__restrict__ mask_out, int32_t *__restrict__ perm, mw_group_desc *__restrict__ desc,
    mw_send_stats *__restrict__ stats)
{
    constexpr uint64_t kNone = mw_order_key<kBytes>::kNone;
    extern __shared__ __align__(16) uint64_t order_lds[];
    const uint32_t n_slots = 1u << slots_log;
    // [1 << slots_log] hash table of keys, (sorted) two bitmaps of kFilterBits bits a slot in front of it
    const uint32_t filter_words = kSorted ? n_slots * kFilterBits / 32 : 0;
    uint32_t *taken = (uint32_t *)order_lds, *shared = taken + filter_words;
    unsigned long long *slot = (unsigned long long *)(shared + filter_words);
    uint64_t *own = (uint64_t *)(slot + n_slots);                     // [kOwnMax]          keys of this workgroup's tokens
    uint2 *part = (uint2 *)(own + kOwnMax);                           // [16][kOwnMax]      the waves' counts for them
    uint32_t *wave_n = (uint32_t *)(part + 16 * kOwnMax);             // [16][4]            kept, distinct, destinations, bad
    uint32_t *wave_r = wave_n + 64;                                   // [16][4]            tokens that name rank r
    uint32_t *in_chunk = wave_r + 64;                                 // [kOrderChunks]     (sorted) a chunk's kept tokens
    uint16_t *tab = kSorted || E > kTableExperts ? nullptr : (uint16_t *)(wave_r + 64);
    const int tid = threadIdx.x, bs = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_wave = bs >> 6;
    // This workgroup's tokens: t0 .. t0 + n_own - 1, or (sorted) those in these places of the chunks.
    const int wg = blockIdx.x, n_wg = gridDim.x, t0 = wg * n_own;
    // token or place of the lane's key j (sorted: chunk wave + 16 (j / 2), its first or second half)
    auto at_of = [&](int j) __attribute__((always_inline)) {
        return kSorted ? (wave + 16 * (j >> 1)) * kChunkTokens + (j & 1) * 64 + lane : tid + j * bs;
    };

    uint64_t key[kU];
    int32_t e[kSorted ? 1 : kU][8];
    bool bad = false;
    uint32_t own_idx = 0;
    if constexpr (kSorted) {
#pragma unroll
        for (int j = 0; j < kU; ++j) key[j] = keys[min(at_of(j), T - 1)];
        if (tid < n_own && t0 + tid < T) own_idx = idx[t0 + tid];
        bad = wg == 0 && tid < n_bad && bad_in[tid] != 0;
    } else if (T > 0) {
        load_ids<kU>(topk, T, K, 0, tid, bs, e);
    }
    if (tab) fill_rank_table(tab, eslot, E);
    // keys that have a bit each: bitmaps of R ranks below 32 << slots_log, and keys of at most two ranks
    const bool few_ranks = !kBytes && R <= 5 + slots_log, own_bit = kSorted && (few_ranks || K <= 2);
    if (!own_bit) for (uint32_t s = tid; s < n_slots / 2; s += bs) ((ulonglong2 *)slot)[s] = make_ulonglong2(kNone, kNone);
    for (uint32_t w = tid; w < filter_words / (own_bit ? 4 : 2); w += bs) ((uint4 *)taken)[w] = make_uint4(0, 0, 0, 0);
    mw_lds_barrier();
    if constexpr (!kSorted) {
        if (T > 0) {
            keys_of_ids<kBytes, kU>(e, topk, T, K, eslot, E, tab, tid, bs, key, bad);
        } else {                                                      // an empty batch has no ids to read
#pragma unroll
            for (int j = 0; j < kU; ++j) key[j] = kNone;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kU; ++j) key[j] = at_of(j) >= T ? kNone : kBytes ? key[j] : key[j] + 1u;
    }
#pragma unroll
    for (int j = 0; j < kU; ++j) {
        const int o = at_of(j) - t0;
        if (o >= 0 && o < n_own) own[o] = key[j];
    }

    // ---- one representative per distinct key.
    // Sorted: equal keys of a wave are neighbours, and the first of them stands for all.  Most keys are nobody else's, and a
    // bit tells: 32 a token, and who finds his taken marks it as shared.  Only tokens of shared bits go on to a hash table, whose
    // slots belong to the token that fills them: a wave seldom has one, and the table is nearly empty.  (All tokens in a
    // table of two slots a token: every wave waits for the longest probe chain, 6 to 9 us of a plan of 8192.)  The table has a slot for
    // every token, so a chain ends whatever the keys are.  Bitmaps of few ranks and keys of one or two have a bit each: who finds
    // it free is the representative (72 ranks, two ids: 2600 possible keys for 4414 tokens, 16.2 us through the table).
    // Not sorted: all tokens go to the table, of four slots a token; a wave whose tokens all have one key sends one lane
    // (thousands of compare-and-swaps on one address would queue).
    uint64_t kept[kU], rep[kU];                                       // wave masks
    if constexpr (kSorted) {
        uint32_t hash[kU], word[kU], bit[kU], old[kU];
        bool first[kU], sent[kU];                                     // sent: the table decides
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const uint32_t lo = (uint32_t)key[j], hi = (uint32_t)(key[j] >> 32);
            // (the lane before: wave_shr:1; lane 0 gets kNone)
            const uint32_t plo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)kNone, (int)lo, 0x138, 0xf, 0xf, false);
            const uint32_t phi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(kNone >> 32), (int)hi, 0x138, 0xf, 0xf, false);
            kept[j] = __ballot(key[j] != kNone);
            first[j] = key[j] != kNone && ((lo ^ plo) | (hi ^ phi)) != 0;
            hash[j] = mw_key_hash(lo, hi);
            uint32_t own_at = kBytes ? hi >> 16 : lo;                            // (two ranks: two bytes, or two positions)
            if (!kBytes && own_bit && !few_ranks) {                              // (uniform)
                const int h = 63 - __clzll((long long)(key[j] | 1ull));
                const uint64_t rest = key[j] & ~(1ull << h);
                own_at = (uint32_t)(h * 64 + (rest ? 63 - __clzll((long long)rest) : h));
            }
            word[j] = own_bit ? own_at >> 5 : hash[j] >> (32 - slots_log);       // (kFilterBits == 32: a word a slot)
            bit[j] = 1u << ((own_bit ? own_at : hash[j] >> 12) & 31u);
            old[j] = 0;
            if (first[j]) old[j] = atomicOr(&taken[word[j]], bit[j]);
        }
        if (own_bit) {
#pragma unroll
            for (int j = 0; j < kU; ++j) rep[j] = __ballot(first[j] && !(old[j] & bit[j]));
        } else {
#pragma unroll
            for (int j = 0; j < kU; ++j) if (old[j] & bit[j]) atomicOr(&shared[word[j]], bit[j]);
            mw_lds_barrier();
            bool any = false;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                sent[j] = first[j] && (shared[word[j]] & bit[j]) != 0;
                any |= sent[j];
            }
            if (__any(any)) {
                bool going[kU];
#pragma unroll
                for (int j = 0; j < kU; ++j) {
                    hash[j] = (hash[j] ^ hash[j] >> 15) * 0x2C1B3C6Du;
                    word[j] = hash[j] >> (32 - slots_log);
                    going[j] = sent[j];
                }
                while (true) {
                    bool more = false;
                    unsigned long long held[kU];
#pragma unroll
                    for (int j = 0; j < kU; ++j)
                        if (going[j]) held[j] = atomicCAS(&slot[word[j]], (unsigned long long)kNone, (unsigned long long)key[j]);
#pragma unroll
                    for (int j = 0; j < kU; ++j) {
                        if (!going[j]) continue;
                        if (held[j] == kNone) sent[j] = false;        // the slot is this token's
                        going[j] = held[j] != kNone && held[j] != key[j];
                        word[j] = (word[j] + (hash[j] << 1 | 1u)) & (n_slots - 1u);          // (odd: visits every slot)
                        more |= going[j];
                    }
                    if (!__any(more)) break;
                }
            }
#pragma unroll
            for (int j = 0; j < kU; ++j) rep[j] = __ballot(first[j] && !sent[j]);
        }
    } else {
        uint64_t hit[kU];                                             // what the token's slot held: kNone for a representative
        uint32_t at[kU], stride[kU];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const bool k = key[j] != kNone;
            kept[j] = __ballot(k);
            const int first = kept[j] ? (int)__builtin_ctzll(kept[j]) : 0;
            const uint64_t fk = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key[j], first) |
                                (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(key[j] >> 32), first) << 32;
            const bool same = __ballot(key[j] == fk) == kept[j];      // (uniform) the wave's kept tokens have one key
            const uint32_t h = mw_key_hash((uint32_t)key[j], (uint32_t)(key[j] >> 32));
            at[j] = h >> (32 - slots_log);
            stride[j] = (h >> 3) | 1u;                                // odd: visits every slot
            hit[j] = key[j];
            if (k && (!same || lane == first))
                hit[j] = atomicCAS(&slot[at[j]], (unsigned long long)kNone, (unsigned long long)key[j]);
        }
        while (true) {                                                // a lane's probes go out together
            bool more = false;
#pragma unroll
            for (int j = 0; j < kU; ++j) more |= hit[j] != kNone && hit[j] != key[j];
            if (!__any(more)) break;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                if (hit[j] != kNone && hit[j] != key[j]) {            // taken by another key
                    at[j] = (at[j] + stride[j]) & (n_slots - 1u);
                    hit[j] = atomicCAS(&slot[at[j]], (unsigned long long)kNone, (unsigned long long)key[j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) rep[j] = __ballot(hit[j] == kNone) & kept[j];   // (a lane without a key: hit == key == kNone)
    }

    // ---- totals (workgroup 0) and rows per destination (rank r: workgroup r modulo the grid)
    if (lane == 0) {
        uint32_t n = 0, g = 0;
#pragma unroll
        for (int j = 0; j < kU; ++j) { n += (uint32_t)__popcll(kept[j]); g += (uint32_t)__popcll(rep[j]); }
        wave_n[wave * 4] = n;
        wave_n[wave * 4 + 1] = g;
    }
    if (wg == 0) {
        uint32_t d = 0;
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            if constexpr (!kBytes) {
                d += (uint32_t)__popcll(key[j]);
            } else if (key[j] != kNone) {
                uint64_t x = key[j] & 0x00ffffffffffffffull;          // its non-zero bytes, and the first rank
                x |= x >> 4; x |= x >> 2; x |= x >> 1;
                d += 1u + (uint32_t)__popcll(x & 0x0001010101010101ull);
            }
        }
        d = mw_wave_sum(d);
        const uint64_t any_bad = __ballot(bad);
        if (lane == 0) { wave_n[wave * 4 + 2] = d; wave_n[wave * 4 + 3] = any_bad ? 1u : 0u; }
    }
    for (int q = 0, r = wg; q < 4 && r < R; ++q, r += n_wg) {         // (the grid has at least R / 4 workgroups)
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            bool names;
            if constexpr (!kBytes) {
                names = (key[j] >> r) & 1ull;
            } else {
                // a byte of the key is this rank's: a zero byte after the exclusive or (the last rank is never a lower byte)
                const uint32_t b = 0x01010101u * (uint32_t)(r + 1);
                const uint32_t lo = (uint32_t)key[j] ^ b, hi = (uint32_t)(key[j] >> 32) ^ ((b & 0xffffffu) | (uint32_t)r << 24);
                names = r < 255 ? ((((lo - 0x01010101u) & ~lo) | ((hi - 0x01010101u) & ~hi)) & 0x80808080u) != 0 : hi >> 24 == 0;
            }
            n += (uint32_t)__popcll(__ballot(names) & kept[j]);
        }
        if (lane == 0) wave_r[wave * 4 + q] = n;
    }
    mw_lds_barrier();

    if constexpr (kSorted) {
        // ---- the chunks in the hash table's place, an entry apart so that a place is in another bank in every chunk
        constexpr int kStride = kChunkTokens + 1, kRepStride = kChunkTokens + 4, kChunks = 8 * kU;      // (16 waves of kU / 2)
        uint64_t *chunk = order_lds;                                  // [kChunks][kStride]
        uint8_t *reps = (uint8_t *)(chunk + kChunks * kStride);       // [kChunks][kRepStride] representatives in front of a place
        static_assert(kChunkTokens == 1 << 7 && kStride * 8 + kRepStride <= kChunkTokens * (8 + kFilterBits / 4), "room of the table and its bitmaps");
#pragma unroll
        for (int j = 0; j < kU; j += 2) {
            const int c = wave + 16 * (j >> 1);
            const uint64_t lower = (1ull << lane) - 1ull;
            const uint32_t first = (uint32_t)__popcll(rep[j]);
            chunk[c * kStride + lane] = key[j];
            chunk[c * kStride + 64 + lane] = key[j + 1];
            reps[c * kRepStride + lane] = (uint8_t)__popcll(rep[j] & lower);
            reps[c * kRepStride + 64 + lane] = (uint8_t)(first + (uint32_t)__popcll(rep[j + 1] & lower));
            if (lane == 0) {
                reps[c * kRepStride + kChunkTokens] = (uint8_t)(first + (uint32_t)__popcll(rep[j + 1]));
                in_chunk[c] = (uint32_t)__popcll(kept[j]) + (uint32_t)__popcll(kept[j + 1]);
            }
        }
        mw_lds_barrier();
        // ---- a wave per own token (two side by side beyond 4096 tokens), a lane per chunk
        constexpr int kN = (kU + 3) / 4;
        const bool mine = lane < kChunks;
        const uint32_t n = mine ? in_chunk[lane] : 0u;
        const uint64_t *c = chunk + (mine ? lane : 0) * kStride;
        uint64_t k[kN];
        uint32_t lb[kN], ub[kN], place[kN];
        int own_c[kN];
        bool more = false;
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            const int o = wave + 16 * q;
            k[q] = o < n_own && t0 + o < T ? own[o] : kNone;
            own_c[q] = (t0 + o) / kChunkTokens;
            place[q] = (uint32_t)(t0 + o) % kChunkTokens;
            lb[q] = 0;                                                // keys below k
        }
#pragma unroll
        for (int b = 7; b >= 0; --b)
#pragma unroll
            for (int q = 0; q < kN; ++q) { const uint32_t at_ = lb[q] + (1u << b); if (at_ <= n && c[at_ - 1] < k[q]) lb[q] = at_; }
        // tokens of the same key: the own one, seldom others
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            const uint32_t look = lane == own_c[q] ? place[q] + 1u : lb[q];
            more |= look < n && c[look] == k[q];
            ub[q] = lb[q];
        }
        if (__any(more)) {
#pragma unroll
            for (int b = 7; b >= 0; --b)
#pragma unroll
                for (int q = 0; q < kN; ++q) { const uint32_t at_ = ub[q] + (1u << b); if (at_ <= n && c[at_ - 1] <= k[q]) ub[q] = at_; }
        } else {
#pragma unroll
            for (int q = 0; q < kN; ++q) if (lane == own_c[q]) ub[q] = place[q] + 1u;
        }
#pragma unroll
        for (int q = 0; q < kN; ++q) {
            if (k[q] == kNone) continue;                              // (the whole wave)
            const uint32_t distinct = mine ? reps[lane * kRepStride + lb[q]] : 0u;
            const uint32_t before = lane < own_c[q] ? ub[q] - lb[q] : lane == own_c[q] ? place[q] - lb[q] : 0u;
            const uint32_t s0 = mw_wave_sum(lb[q] | distinct << 16), s1 = mw_wave_sum(before | (ub[q] - lb[q] - before) << 16);
            if (lane == 0) part[wave + 16 * q] = make_uint2(s0, s1);
        }
    } else
    // ---- counts for the workgroup's own tokens
    if (t0 < T) {
        const uint64_t mine = lane < kOwnMax ? own[lane] : kNone;     // (entries past n_own are not used)
        uint32_t c0 = 0, c1 = 0;                                      // lane o: (below, distinct below), (equal before, equal at or after)
#pragma unroll
        for (int j = 0; j < kU; ++j) if (key[j] == kNone) key[j] = ~0ull;      // below no token; equals are masked by `kept`
        const int n = min(n_own, T - t0);
        for (int o = 0; o < n; ++o) {
            const uint64_t k = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, o) |
                               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), o) << 32;
            uint32_t below = 0, distinct = 0, before = 0, after = 0;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint64_t lt = __ballot(key[j] < k);
                below += (uint32_t)__popcll(lt);
                distinct += (uint32_t)__popcll(lt & rep[j]);
                const uint64_t eq = __ballot(key[j] == k) & kept[j];
                const int first = j * bs + wave * 64;
                if constexpr (kFew) {
                    uint64_t m = first + 64 <= t0 ? ~0ull : 0ull;     // the wave's tokens that come before: all or none of them ...
                    if (first < t0 + n && first + 64 > t0) {          // ... but in the wave around the own ones (a branch: 7.9 -> 9.1 us without)
                        const int ahead = t0 + o - first;
                        m = ahead <= 0 ? 0ull : ahead >= 64 ? ~0ull : (1ull << ahead) - 1ull;
                    }
                    before += (uint32_t)__popcll(eq & m);
                    after += (uint32_t)__popcll(eq);
                } else if (eq) {
                    const int ahead = t0 + o - first;
                    const uint64_t m = ahead <= 0 ? 0ull : ahead >= 64 ? ~0ull : (1ull << ahead) - 1ull;
                    before += (uint32_t)__popcll(eq & m);
                    after += (uint32_t)__popcll(eq & ~m);
                }
            }
            if (kFew) after -= before;
            if (lane == o) { c0 = below | distinct << 16; c1 = before | after << 16; }
        }
        if (lane < n) part[wave * kOwnMax + lane] = make_uint2(c0, c1);
    }
    mw_lds_barrier();
    if (tid < n_own && t0 + tid < T) {
        const int t = kSorted ? (t0 + tid) / kChunkTokens * kChunkTokens + (int)own_idx : t0 + tid;
        uint32_t c0 = 0, c1 = 0;
        for (int w = 0; w < (kSorted ? 1 : n_wave); ++w) { const uint2 c = part[w * kOwnMax + tid]; c0 += c.x; c1 += c.y; }     // (halves stay below 2^16)
        uint64_t m[MW_MASK_WORDS];
        const uint64_t k = own[tid];
        mask_of_key<kBytes>(k, m);
        uint64_t *mo = mask_out + (size_t)t * MW_MASK_WORDS;
#pragma unroll
        for (int q = 0; q < MW_MASK_WORDS; ++q) mo[q] = m[q];
        if (k != kNone) {
            const uint32_t below = c0 & 0xffffu, distinct = c0 >> 16, before = c1 & 0xffffu, after = c1 >> 16;
            const uint32_t row = below + before;
            perm[row] = t;
            if (before == 0) {
                mw_group_desc d;
                uint32_t nd = 0;
#pragma unroll
                for (int q = 0; q < MW_MASK_WORDS; ++q) { d.mask[q] = m[q]; nd += (uint32_t)__popcll(m[q]); }
                d.row_offset = row; d.row_count = after; d.n_dest = nd; d.reserved0 = 0;
                desc[distinct] = d;
            }
        }
    }
    if (tid < 4 && wg + tid * n_wg < R) {
        uint32_t n = 0;
        for (int w = 0; w < n_wave; ++w) n += wave_r[w * 4 + tid];
        stats->rows_per_dest[wg + tid * n_wg] = n;
    }
    if (wg == 0) {
        for (int r = R + tid; r < MW_MAX_RANKS; r += bs) stats->rows_per_dest[r] = 0;
        if (tid == 0) {
            uint32_t n = 0, g = 0, d = 0, b = 0;
            for (int w = 0; w < n_wave; ++w) {
                n += wave_n[w * 4]; g += wave_n[w * 4 + 1]; d += wave_n[w * 4 + 2]; b |= wave_n[w * 4 + 3];
            }
            stats->n_rows = n;
            stats->n_groups = g;
            stats->multicast_bytes = (uint64_t)n * row_bytes;
            stats->unicast_bytes = (uint64_t)d * row_bytes;
            stats->error_flags = pstate[kPsFlags] | (b ? MW_FLAG_BAD_EXPERT : 0u);
            stats->reserved0 = 0;
        }
    }
}

__global__ __launch_bounds__(256) void k_plan_allgather(int R, uint64_t shard_bytes, mw_group_desc *desc,
                                                        mw_send_stats *stats)
{
    mw_plan_allgather_body(R, shard_bytes, desc, stats);
}

// Descriptor pair of a fragment split into a direct and a relayed segment (Section 5.2),
// in units of 16 bytes.
__global__ __launch_bounds__(256) void k_plan_allgather_split(int R, uint64_t shard_bytes, uint64_t direct_bytes,
                                                              mw_group_desc *desc, mw_send_stats *stats)
{
    const int tid = threadIdx.x;
    const uint32_t units = (uint32_t)(shard_bytes / 16), d_units = (uint32_t)(direct_bytes / 16);
    if (tid < MW_MAX_RANKS) stats->rows_per_dest[tid] = (tid < R) ? units : 0u;
    if (tid < 2) {
        mw_group_desc d;
#pragma unroll
        for (int w = 0; w < MW_MASK_WORDS; ++w) {
            const int lo = w * 64;
            d.mask[w] = (R >= lo + 64) ? ~0ull : (R > lo ? ((1ull << (R - lo)) - 1ull) : 0ull);
        }
        d.row_offset = tid == 0 ? 0u : d_units;
        d.row_count = tid == 0 ? d_units : units - d_units;
        d.n_dest = (uint32_t)R; d.reserved0 = 0;
        desc[tid] = d;
    }
    if (tid == 0) {
        stats->n_rows = units; stats->n_groups = 2;
        stats->multicast_bytes = direct_bytes * (uint64_t)R + (shard_bytes - direct_bytes);
        stats->unicast_bytes = shard_bytes * (uint64_t)R;
        stats->error_flags = 0; stats->reserved0 = 0;
    }
}

// Plan and pack of a decode-sized batch (at most kFusedMax tokens) in one launch.  The results
// are those of mw_plan and the packer; what changes is the latency: dependent launches become one
// without any global scratch.  Workgroup 0 makes the plan.  Workgroup 1 + b moves token b's row
// and does not wait for it: the row is requested first, and beside it the workgroup builds all
// bitmaps itself, one token per lane, and counts those in front of its own, which is the packed
// row.  (A workgroup per packed row has to rank all tokens before it knows what to load.)
// Measured (us, 14336-byte rows, workgroup per packed row / this): 16 tokens 8.0 / 4.2, 64 of 64 ranks 10.0 / 4.3,
// 128 11.5 / 5.4, 256 14.7 / 8.3, 64 of 256 ranks 17.9 / 6.1; the plan alone is most of it.
constexpr int kFusedMax = MW_FUSED_MAX_TOKENS;

// kKeyed (bitmaps of more than one word, top_k <= 8): the plan's all-pairs walk compares short keys.
template <int W, bool kKeyed>
__global__ __launch_bounds__(kSmallPlanLanes) void k_plan_pack(
    const int32_t *__restrict__ topk, int T, int K, const int32_t *__restrict__ eslot, int E,
    const u32x4 *__restrict__ x, const u32x4 *__restrict__ scales, int xc, int sc, int ns, uint64_t row_bytes,
    uint64_t *__restrict__ mask_out, int32_t *__restrict__ perm, mw_group_desc *__restrict__ desc,
    mw_send_stats *__restrict__ stats, u32x4 *__restrict__ packed, int32_t *__restrict__ row_src_token,
    int32_t *__restrict__ row_topk)
{
    constexpr int kPlanWords = mw_small_plan_words<W, kKeyed>();
    __shared__ uint64_t lds[kPlanWords];
    if (blockIdx.x == 0) {
        mw_small_plan<W, kKeyed>(topk, T, K, eslot, E, row_bytes, mask_out, perm, desc, stats, lds);
        return;
    }
    const int b = (int)blockIdx.x - 1, t = threadIdx.x, n = xc + sc;
    int32_t *tab = (int32_t *)lds;                                      // [kSmallTab]
    uint64_t *own = (uint64_t *)(tab + kSmallTab);                      // [MW_MASK_WORDS] token b's bitmap
    uint32_t *before = (uint32_t *)(own + MW_MASK_WORDS);               // [kSmallPlanLanes / 64]
    static_assert(kSmallTab / 2 + MW_MASK_WORDS + kSmallPlanLanes / 128 <= kPlanWords, "LDS of a mover");
    auto chunk = [&](int ch) {
        return ch < xc ? mw_ld16(x + (size_t)b * xc + ch) : mw_ld16(scales + (size_t)b * sc + (ch - xc));
    };
    u32x4 v0 = {0u, 0u, 0u, 0u};
    if (t < n) v0 = chunk(t);
    uint64_t m[MW_MASK_WORDS];
    bool bad = false;
    small_token_mask(topk, T, K, eslot, E, tab, m, bad);
    if (t == b)
#pragma unroll
        for (int w = 0; w < MW_MASK_WORDS; ++w) own[w] = m[w];
    mw_lds_barrier();
    uint64_t mine[W], any = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) { mine[w] = own[w]; any |= mine[w]; }
    if (any == 0) return;                                               // (the whole workgroup) no destination
    // kept tokens with (bitmap, token) < (mine, b); lanes from T on hold an empty bitmap and are not kept
    uint64_t mine_any = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) mine_any |= m[w];
    const bool less = mine_any != 0 && (mask_less<W>(m, mine) || (t < b && !mask_less<W>(mine, m)));
    const uint32_t c = (uint32_t)__popcll(__ballot(less));
    if ((t & 63) == 0) before[t >> 6] = c;
    mw_lds_barrier();
    uint32_t i = 0;
#pragma unroll
    for (int w = 0; w < kFusedMax / 64; ++w) i += before[w];            // (tokens live in the first waves)
    if (t < n) mw_st16(packed + (size_t)i * ns + t, v0);
    for (int ch = t + kSmallPlanLanes; ch < n; ch += kSmallPlanLanes) mw_st16(packed + (size_t)i * ns + ch, chunk(ch));
    if (t == 0) row_src_token[i] = b;
    for (int j = t; j < K; j += kSmallPlanLanes) row_topk[(size_t)i * K + j] = topk[(size_t)b * K + j];
}

// ---- ordering of large batches: sorted chunks, then ranks by binary search ------------------
// The all-pairs walk of k_rank costs T^2 compares: 84 us at 16 k tokens, 220 us at 32 k, 700 us
// at 64 k (one-word bitmaps; 120 / 335 / 1085 us with short keys).  This path: 48 / 68 / 97 us
// (53 / 74 / 107 us).  For batches beyond k_plan_order's whose bitmaps have a 64-bit order-preserving key (one word, or
// short keys) the same counters are produced in T log T work:
//   k_chunk_sort   one workgroup per chunk of 1024 tokens: bitmaps, keys, a bitonic sort of
//                  (key, second word) pairs in LDS; the sorted chunk goes to the workspace.
//   k_merge_rank   workgroup (c, part), one lane per sorted element of chunk c: the chunks of its
//                  part are staged through LDS in turn and searched for the element's key.  A
//                  chunk of lower index contributes its keys <= mine (ties there come before me),
//                  one of higher index its keys < mine, my own chunk my sorted position.  The
//                  parts' sums meet in one 64-bit atomic add per element, as in k_rank.
// k_groups then runs unchanged on the counters.
// Second word of a sort element: (bit-0 flag << 31) | index inside the chunk for kept tokens;
// tokens without a destination and the padding of the last chunk carry the largest key and a
// second word above every kept token's, so they sort behind all kept tokens of the chunk.
constexpr int kChunk = 1024;
constexpr uint32_t kSecEmpty = 0x40000000u, kSecPad = 0x7fffffffu;

template <int W>
__global__ __launch_bounds__(kChunk) void k_chunk_sort(const int32_t *__restrict__ topk, int T, int K,
                                                       const int32_t *__restrict__ eslot, int E,
                                                       uint64_t *__restrict__ mask_out, uint32_t *__restrict__ pstate,
                                                       uint64_t *__restrict__ sort_key, uint32_t *__restrict__ sort_sec,
                                                       uint32_t *__restrict__ chunk_kept)
{
    __shared__ uint64_t sk[kChunk];
    __shared__ uint32_t ss[kChunk];
    __shared__ uint32_t hist[MW_MAX_RANKS];
    __shared__ uint32_t scratch[17];
    const int tid = threadIdx.x;
    const int t = blockIdx.x * kChunk + tid;
    if (tid < MW_MAX_RANKS) hist[tid] = 0;
    bool bad = false;
    uint64_t m[MW_MASK_WORDS] = {0, 0, 0, 0};
    if (t < T) {
        token_mask(topk + (size_t)t * K, K, eslot, E, m, bad);
        uint64_t *o = mask_out + (size_t)t * MW_MASK_WORDS;
#pragma unroll
        for (int q = 0; q < MW_MASK_WORDS; ++q) o[q] = m[q];
        if (bad) atomicOr(&pstate[kPsFlags], MW_FLAG_BAD_EXPERT);
    }
    const bool any = (m[0] | m[1] | m[2] | m[3]) != 0;
    uint64_t key = ~0ull;
    uint32_t sec = t < T ? (kSecEmpty | (uint32_t)tid) : kSecPad;
    if (any) {
        if constexpr (W == 1) { key = m[0]; sec = (uint32_t)tid; }
        else { const mw_short_key k = short_key(m); key = k.key; sec = (k.flag << 31) | (uint32_t)tid; }
    }
    uint32_t kept;
    mw_block_exscan(any ? 1u : 0u, scratch, &kept);        // (its barriers also publish the cleared histogram)
    if (tid == 0) {
        chunk_kept[blockIdx.x] = kept;
        if (kept) atomicAdd(&pstate[kPsKept], kept);
    }
    // rows per destination: one LDS atomic per set bit (at most top_k per token), then one
    // global atomic per rank and chunk
#pragma unroll
    for (int q = 0; q < W; ++q) {
        uint64_t left = m[q];
        while (left) {
            const int b = __ffsll((unsigned long long)left) - 1;
            left &= left - 1;
            atomicAdd(&hist[q * 64 + b], 1u);
        }
    }

    // Bitonic network with one element per lane.  Partners closer than 64 are in the same
    // wavefront and are exchanged in registers; the ten steps with partners 64 or more apart go
    // through LDS.  Position e keeps the smaller of the pair iff it is the lower position of an
    // ascending block or the upper position of a descending one.
    const int e = tid;
    for (int k = 2; k <= kChunk; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            uint64_t pk;
            uint32_t ps;
            if (j >= 64) {
                sk[e] = key; ss[e] = sec;
                mw_lds_barrier();
                pk = sk[e ^ j]; ps = ss[e ^ j];
                mw_lds_barrier();
            } else {
                pk = __shfl_xor(key, j, 64);
                ps = __shfl_xor(sec, j, 64);
            }
            const bool mine_after = key > pk || (key == pk && sec > ps);
            const bool keep_smaller = ((e & j) == 0) == ((e & k) == 0);
            if (mine_after == keep_smaller) { key = pk; sec = ps; }
        }
    }
    sort_key[(size_t)blockIdx.x * kChunk + tid] = key;
    sort_sec[(size_t)blockIdx.x * kChunk + tid] = sec;
    mw_lds_barrier();                                       // every lane's histogram atomics are done
    if (tid < MW_MAX_RANKS && hist[tid]) atomicAdd(&pstate[tid], hist[tid]);
}

template <int W>
__global__ __launch_bounds__(kChunk) void k_merge_rank(int T, int n_chunks, const uint32_t *__restrict__ pstate,
                                                       const uint64_t *__restrict__ sort_key,
                                                       const uint32_t *__restrict__ sort_sec,
                                                       const uint32_t *__restrict__ chunk_kept,
                                                       unsigned long long *__restrict__ cnt)
{
    __shared__ uint64_t sk[kChunk];
    __shared__ uint32_t ss[kChunk];
    __shared__ uint32_t kept_of[64];                       // 65536 tokens / 1024
    const int tid = threadIdx.x, c = blockIdx.x;
    const int per = (n_chunks + (int)gridDim.y - 1) / (int)gridDim.y;
    const int c_first = blockIdx.y * per, c_end = min(n_chunks, c_first + per);
    if (c_first >= c_end) return;
    if (tid < n_chunks) kept_of[tid] = chunk_kept[tid];
    const uint64_t key = sort_key[(size_t)c * kChunk + tid];
    const uint32_t sec = sort_sec[(size_t)c * kChunk + tid];
    const uint32_t flag = sec >> 31;
    const uint32_t n_empty = blockIdx.y == 0 ? (uint32_t)T - min(pstate[kPsKept], (uint32_t)T) : 0u;
    uint64_t nk = sort_key[(size_t)c_first * kChunk + tid];  // the part's first chunk, staged below
    uint32_t ns = sort_sec[(size_t)c_first * kChunk + tid];
    uint32_t c_lt = 0, c_eqb = 0, c_eqa = 0;
    // entries of the staged chunk that are below / not above my (key, flag)
    auto below = [&](uint32_t idx) -> bool {
        const uint64_t q = sk[idx];
        if constexpr (W == 1) return q < key;
        else return q < key || (q == key && (ss[idx] >> 31) < flag);
    };
    auto not_above = [&](uint32_t idx) -> bool {
        const uint64_t q = sk[idx];
        if constexpr (W == 1) return q <= key;
        else return q < key || (q == key && (ss[idx] >> 31) <= flag);
    };
    for (int c2 = c_first; c2 < c_end; ++c2) {
        mw_lds_barrier();                                   // the previous chunk has been searched
        sk[tid] = nk; ss[tid] = ns;
        mw_lds_barrier();
        if (c2 + 1 < c_end) {                               // next chunk in flight during the search
            nk = sort_key[(size_t)(c2 + 1) * kChunk + tid];
            ns = sort_sec[(size_t)(c2 + 1) * kChunk + tid];
        }
        const uint32_t n = kept_of[c2];
        uint32_t lb = 0, ub = 0;
#pragma unroll
        for (uint32_t st = kChunk; st >= 1; st >>= 1) {
            if (lb + st <= n && below(lb + st - 1)) lb += st;
            if (ub + st <= n && not_above(ub + st - 1)) ub += st;
        }
        c_lt += lb;
        if (c2 < c) c_eqb += ub - lb;
        else if (c2 > c) c_eqa += ub - lb;
        else { c_eqb += (uint32_t)tid - lb; c_eqa += ub - (uint32_t)tid; }
    }
    if ((uint32_t)tid < kept_of[c]) {
        const int t = c * kChunk + (int)(sec & 0x3fffffffu);
        const unsigned long long add = (unsigned long long)(c_lt + c_eqb + n_empty) |
                                       ((unsigned long long)c_eqb << 21) | ((unsigned long long)c_eqa << 42);
        if (add) atomicAdd(&cnt[t], add);
    }
}

}  // namespace

int32_t mw_launch_plan_allgather_split(mw_ctx *ctx, int64_t shard_bytes, int64_t direct_bytes, mw_group_desc *desc,
                                       mw_send_stats *stats, hipStream_t s)
{
    hipLaunchKernelGGL(k_plan_allgather_split, dim3(1), dim3(256), 0, s, ctx->cfg.n_ranks, (uint64_t)shard_bytes,
                       (uint64_t)direct_bytes, desc, stats);
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

// Tokens from which the keys get a launch of their own, in sorted chunks (mw_plan alone, us: 64 ranks uniform / 256 ranks
// skewed / 8 ranks).  1025 tokens 7.4 / 9.6 / 7.3 in one launch, 2048 8.5 / 10.5 / 8.2; sorted, 2049 10.1 / 11.8 / 9.9, 4096
// 10.8 / 11.9 / 10.4, 6000 12.9 / 15.1 / 12.7, 8192 15.1 / 16.1 / 14.1.  (One launch that compared a token with a bucket of keys instead
// of with all: 1025 8.1 / 10.3 / 7.7, 2048 8.8 / 11.4 / 7.9; keys not sorted, buckets behind them: 4096 12.8 / 14.6 / 10.8, 6000 18.7 /
// 22.4 / 13.5, 8192 21.8 / 28.0 / 14.6.)
constexpr int kKeysFrom = 2049;

template <bool kBytes>
static void launch_plan_order(mw_ctx *ctx, const int32_t *topk, int32_t T, uint64_t *mask, int32_t *perm, mw_group_desc *desc,
                              mw_send_stats *stats, hipStream_t s)
{
    const int K = ctx->cfg.top_k, E = ctx->cfg.n_experts, R = ctx->cfg.n_ranks;
    const bool sorted = T >= kKeysFrom;
    const int bs = T <= 256 ? 256 : T <= 512 ? 512 : kOrderBlock;
    // About a workgroup per CU, and enough of them that each counts at most four ranks.  (Half as many: the plan alone 2 us
    // slower at 8192 tokens.)
    int n_own = (T + 255) / 256;
    if (n_own < 1) n_own = 1;
    int n_wg = (T + n_own - 1) / n_own;
    if (n_wg < (R + 3) / 4) n_wg = (R + 3) / 4;
    // four slots a token: half the slots taken means probe chains of up to ten, and every wave waits for the longest.  Sorted:
    // one for each of the lanes' tokens
    int slots_log = 6;
    while ((1 << slots_log) < 4 * T) ++slots_log;
    if (sorted) slots_log = T <= 4 * kOrderBlock ? 12 : 13;
    const size_t tab = E <= kTableExperts ? ((size_t)E + 4) / 4 * 8 : 0;
    const size_t lds = ((size_t)(sorted ? 8 + kFilterBits / 4 : 8) << slots_log) + 8 * kOwnMax + 8 * 16 * kOwnMax + 4 * 128 + (sorted ? 4 * kOrderChunks : tab);
    const int n_key_wg = (T + kChunkTokens - 1) / kChunkTokens;
    if (sorted) {
        mw_timed tm(ctx, MW_KERNEL_PLAN_RANK, s);
        hipLaunchKernelGGL(k_plan_keys<kBytes>, dim3(n_key_wg), dim3(kKeysBlock), tab, s, topk, T, K, ctx->d_eslot, E,
                           ctx->d_plan_keys, ctx->d_plan_idx, ctx->d_plan_bad);
    }
    mw_timed tm(ctx, sorted ? MW_KERNEL_PLAN_GROUPS : MW_KERNEL_PLAN_RANK, s);
    // Destination sets that K ids can name among R ranks: up to 256 of them a wave nearly always has a key like a token's.  2048
    // tokens, us asking whether there are equals / not asking: 8 ranks, one to eight ids 8.9 / 7.8, 8.8 / 7.9, 8.0 / 7.8,
    // 8.2 / 7.9 (8 to 255 sets), 24 ranks, one and two ids 8.9 / 7.9, 8.1 / 8.2 (300 sets), 12 ranks, four ids 7.5 / 7.8, 256 ranks,
    // one and eight ids 9.8 / 9.5, 10.4 / 10.6.
    int64_t sets = 1, of_size = 1;
    for (int j = 1; j <= K && j <= R && sets <= 257; ++j) { of_size = of_size * (R - j + 1) / j; sets += of_size; }
    const bool few = sets <= 257;                                     // (the empty set among them)
#define MW_ORDER(U_, SORTED_, FEW_)                                                                                     \
    hipLaunchKernelGGL((k_plan_order<kBytes, U_, SORTED_, FEW_>), dim3(n_wg), dim3(bs), lds, s, topk, T, K, ctx->d_eslot, E, R,  \
                       n_own, slots_log, ctx->d_plan_keys, ctx->d_plan_idx, ctx->d_plan_bad, n_key_wg, ctx->d_plan_state,     \
                       (uint64_t)ctx->row_bytes, mask, perm, desc, stats)
    static_assert(kKeysFrom == 2 * kOrderBlock + 1, "tokens a lane of each form");
    if (T <= kOrderBlock) MW_ORDER(1, false, false);
    else if (!sorted && few) MW_ORDER(2, false, true);
    else if (!sorted) MW_ORDER(2, false, false);
    else if (T <= 4 * kOrderBlock) MW_ORDER(4, true, false);
    else if (T <= 6 * kOrderBlock) MW_ORDER(6, true, false);
    else MW_ORDER(8, true, false);
#undef MW_ORDER
}

int32_t mw_launch_plan(mw_ctx *ctx, const int32_t *topk, int32_t T, uint64_t *mask, int32_t *perm,
                       mw_group_desc *desc, mw_send_stats *stats, hipStream_t s)
{
    const int K = ctx->cfg.top_k, E = ctx->cfg.n_experts;
    // both start out zero: mw_ctx_create cleared them, every plan's last kernel clears them again
    unsigned long long *cnt = (unsigned long long *)ctx->d_plan_cnt;
    uint32_t *pstate = ctx->d_plan_state;
    const int tb = (T + kBlock - 1) / kBlock;
    const bool has_key = ctx->mask_words == 1 || K <= 8;
    if (has_key && T <= kOrderMaxTokens) {
        if (ctx->mask_words == 1) launch_plan_order<false>(ctx, topk, T, mask, perm, desc, stats, s);
        else launch_plan_order<true>(ctx, topk, T, mask, perm, desc, stats, s);
        // (the other kernel's event pair, where a caller has set one, brackets nothing)
        if (T < kKeysFrom) { mw_timed tm(ctx, MW_KERNEL_PLAN_GROUPS, s); }
        MW_HIP_CHECK(hipGetLastError());
        return MW_OK;
    }
    if (T > kOrderMaxTokens && has_key && ctx->d_sort_key) {
        const int nc = (T + kChunk - 1) / kChunk;
        // split every chunk's walk over the other chunks into parts so that the grid fills the chip
        int parts = (2 * ctx->n_cu + nc - 1) / nc;
        if (parts > nc) parts = nc;
        if (parts < 1) parts = 1;
        mw_timed tm(ctx, MW_KERNEL_PLAN_RANK, s);
        if (ctx->mask_words == 1) {
            hipLaunchKernelGGL(k_chunk_sort<1>, dim3(nc), dim3(kChunk), 0, s, topk, T, K, ctx->d_eslot, E, mask,
                               pstate, ctx->d_sort_key, ctx->d_sort_sec, ctx->d_chunk_kept);
            hipLaunchKernelGGL(k_merge_rank<1>, dim3(nc, parts), dim3(kChunk), 0, s, T, nc, pstate,
                               ctx->d_sort_key, ctx->d_sort_sec, ctx->d_chunk_kept, cnt);
        } else {
            hipLaunchKernelGGL(k_chunk_sort<4>, dim3(nc), dim3(kChunk), 0, s, topk, T, K, ctx->d_eslot, E, mask,
                               pstate, ctx->d_sort_key, ctx->d_sort_sec, ctx->d_chunk_kept);
            hipLaunchKernelGGL(k_merge_rank<4>, dim3(nc, parts), dim3(kChunk), 0, s, T, nc, pstate,
                               ctx->d_sort_key, ctx->d_sort_sec, ctx->d_chunk_kept, cnt);
        }
    } else if (T > 0) {
        if (ctx->mask_words == 1) return MW_ERR_UNSUPPORTED;       // (k_rank has no one-word form: every such batch has a key)
        // Bitmaps of more than one word and more than eight ids: no 64-bit key.  Split the predecessor walk into
        // slices so that about 4 workgroups land on every CU; a slice's bitmaps must fit in LDS.
        int ns = (4 * ctx->n_cu + tb - 1) / tb;
        if (ns < 1) ns = 1;
        int slice = (T + ns - 1) / ns;
        if (slice < 64) slice = 64;
        if (slice > 1024) slice = 1024;
        ns = (T + slice - 1) / slice;
        const dim3 grid(tb, ns), block(kBlock);
        const int W = ctx->mask_words;
        const size_t lds = (size_t)slice * W * sizeof(uint64_t);
        mw_timed tm(ctx, MW_KERNEL_PLAN_RANK, s);
#define MW_RANK(W_)                                                                                         \
    hipLaunchKernelGGL(k_rank<W_>, grid, block, lds, s, topk, T, K, ctx->d_eslot, E, slice, mask, cnt, pstate)
        if (W == 2) MW_RANK(2);
        else if (W == 3) MW_RANK(3);
        else MW_RANK(4);
#undef MW_RANK
    }
    {
        mw_timed tm(ctx, MW_KERNEL_PLAN_GROUPS, s);
        if (T >= kPlanRowsFrom && ctx->d_row_cnt) {
            hipLaunchKernelGGL(k_rows_from_counters, dim3(tb), dim3(kBlock), 0, s, T, cnt, pstate, perm,
                               (unsigned long long *)ctx->d_row_cnt, ctx->d_row_start);
            hipLaunchKernelGGL(k_groups<true>, dim3(tb), dim3(kBlock), 0, s, mask, T, (uint64_t)ctx->row_bytes, cnt,
                               pstate, perm, desc, stats, (const unsigned long long *)ctx->d_row_cnt, ctx->d_row_start);
        } else {
            hipLaunchKernelGGL(k_groups<false>, dim3(tb > 0 ? tb : 1), dim3(kBlock), 0, s, mask, T,
                               (uint64_t)ctx->row_bytes, cnt, pstate, perm, desc, stats, nullptr, nullptr);
        }
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}


int32_t mw_launch_plan_pack(mw_ctx *ctx, const int32_t *topk, int32_t T, const void *x, const float *scales,
                            uint64_t *mask, int32_t *perm, mw_group_desc *desc, mw_send_stats *stats, void *packed,
                            int32_t *row_src_token, int32_t *row_topk, hipStream_t s)
{
    const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
    const dim3 grid(1 + T), block(kSmallPlanLanes);
    const int K = ctx->cfg.top_k, E = ctx->cfg.n_experts;
    const uint64_t rb = (uint64_t)ctx->row_bytes;
    mw_timed tm(ctx, MW_KERNEL_PLAN_PACK, s);
#define MW_FUSED(W, KEYED)                                                                                        \
    hipLaunchKernelGGL((k_plan_pack<W, KEYED>), grid, block, 0, s, topk, T, K, ctx->d_eslot, E, (const u32x4 *)x, \
                       (const u32x4 *)scales, xc, sc, (int)(ctx->row_stride / 16), rb, mask, perm, desc, stats,       \
                       (u32x4 *)packed, row_src_token,                                                           \
                       row_topk)
    const bool keyed = K <= 8;              // at most eight bits per bitmap: short keys
    switch (ctx->mask_words) {
    case 1: MW_FUSED(1, false); break;
    case 2: if (keyed) MW_FUSED(2, true); else MW_FUSED(2, false); break;
    case 3: if (keyed) MW_FUSED(3, true); else MW_FUSED(3, false); break;
    default: if (keyed) MW_FUSED(4, true); else MW_FUSED(4, false); break;
    }
#undef MW_FUSED
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_plan_allgather(mw_ctx *ctx, int64_t shard_bytes, mw_group_desc *desc,
                                 mw_send_stats *stats, hipStream_t s)
{
    hipLaunchKernelGGL(k_plan_allgather, dim3(1), dim3(256), 0, s, ctx->cfg.n_ranks, (uint64_t)shard_bytes,
                       desc, stats);
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}
