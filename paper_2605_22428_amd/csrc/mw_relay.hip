// Relay step: one node's part of the recursive MultiWrite execution model.
//
// Paper hooks: Section 4.3.3 -- a node holding a MultiWrite for a destination set M
// partitions M by next hop and starts one child MultiWrite per subset, a subset of one
// destination being an ordinary write; Section 4.1, "Local forwarding table" -- the next
// hop of every destination comes from the node's unicast forwarding table and the number
// of distinct next hops is the number of copies; Section 4.1, "Replication and
// forwarding" -- each copy carries updated metadata naming only the destinations served
// through its hop, so nothing is delivered twice; Section 3.2 -- the same-index device of
// the remote server replicates a token to the targets inside that server.
//
// Two launches on the caller's stream:
//   k_relay_index  workgroup (h, c) builds chunk c of child h's descriptor table: a group is kept
//                  if its bitmap intersects the hop's rank set; kept groups are ranked with
//                  block scans (group index, first row), so the child is in parent order
//                  whatever the timing.  What the chunks before it keep a workgroup counts for itself.
//                  The (group, hop) -> first child row table feeds the
//                  copy.  Further workgroups map rows to groups and do the byte accounting.
//   k_relay_copy   small workgroups (a single wave for cache-line-sized rows), each moving
//                  consecutive 16-byte chunks of one input row: read once, stored once per next hop that keeps the row's group
//                  (lane h of every wave holds hop h's position; a ballot lists the hops).  Bound by HBM
//                  bandwidth: rows * row_bytes read, rows * copies * row_bytes written.
#include "mw_internal.h"

namespace {

constexpr int kBlock = 512;                  // lanes of an index workgroup in a launch of its own
constexpr uint32_t kNoChild = 0xffffffffu;
constexpr uint32_t kLongGroup = 32;          // rows; longer groups are filled by their whole wave
constexpr uint32_t kMaxChunks = 16;          // workgroups per hop

// Entries from one group's (packet's) child positions to the next one's: a power of two from 16, so that
// a group's positions are one or two cache lines.
__host__ __device__ __forceinline__ uint32_t relay_pos_stride(int n_hops) { return n_hops <= 16 ? 16u : n_hops <= 32 ? 32u : 64u; }
// Words behind the relay flags in the workspace: what the accounting workgroups of one index add up (zero between
// indexes; the workgroup that reports last writes the statistics and clears them).
struct mw_relay_acc { uint32_t flags, groups, done, reserved0; unsigned long long rows, dest_rows; };

// Everything the index of one relay step needs (one kernel argument).
struct mw_relay_index_args {
    const mw_recv_peer *in; const mw_relay_child *children; int n_hops, n_ranks;
    uint32_t max_tokens, cap; uint64_t row_bytes; const uint64_t *hop_bits;
    int32_t *group_of_row; uint32_t *child_pos; uint32_t *relay_flags; mw_relay_stats *stats;
    uint32_t keep_metadata;     // 1: children carry the parent's bitmaps (Section 4.1: the update may be omitted)
    uint32_t chunks;            // workgroups per hop
};

// The bitmap of ranks below n_ranks, word w.
__device__ __forceinline__ uint64_t valid_rank_word(int n_ranks, int w)
{
    const int lo = w * 64;
    return (n_ranks >= lo + 64) ? ~0ull : (n_ranks > lo ? ((1ull << (n_ranks - lo)) - 1ull) : 0ull);
}

// Sum of one value per lane over the workgroup; scratch of 17 words.
__device__ __forceinline__ uint32_t relay_block_sum(uint32_t v, uint32_t *scratch)
{
    uint32_t total;
    mw_block_exscan(v, scratch, &total);
    return total;
}

// Chunk c of `chunks` of next hop h's child descriptor table, by one workgroup.  Of a descriptor the
// ranking needs the NW bitmap words that can name a rank (ranks < 64 NW; the hop's rank set and the valid
// ranks have nothing above them), the row range, and the end of the range in front (a descriptor is valid
// if its row range is not empty, lies inside the buffer and starts at or after the end of the previous
// descriptor's).  A workgroup first counts what the hop keeps of all groups before its chunk -- four of them a lane
// in flight, nothing to scan -- and then places its own, a group a lane, with one scan of the kept groups
// and one of their rows.  Bound by latency: one workgroup a hop, walking all groups three a lane and step, took
// 3.5 us a step plus the scans (4096 groups, 15 hops: the index 14.7 us, now 7 us).
template <int NW>
__device__ __forceinline__ uint32_t relay_index_hop(
    const mw_recv_peer &src, const uint32_t G, const uint32_t n_rows, mw_group_desc *__restrict__ cdesc, const int h,
    const uint32_t c, const uint32_t chunks, const int n_ranks, const uint32_t cap, const uint64_t *__restrict__ hop_bits,
    uint32_t *__restrict__ child_pos, const uint32_t pos_stride, mw_relay_stats *__restrict__ stats,
    const uint32_t keep_metadata, uint32_t *scratch, uint32_t *fit)
{
    const uint32_t bs = blockDim.x, tid = threadIdx.x;
    const uint32_t per = ((G + chunks - 1) / chunks + bs - 1) / bs * bs;
    const uint32_t g_first = min(G, c * per), g_end = min(G, g_first + per);
    if (g_first >= G && c + 1 < chunks) return 0;                            // (the last chunk reports the totals)
    uint32_t err = 0;
    uint64_t hb[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) hb[w] = hop_bits[(size_t)h * MW_MASK_WORDS + w];
    uint64_t m[NW];
    uint2 oc, po;
    auto load = [&](uint32_t g, uint64_t (&mm)[NW], uint2 &o, uint2 &p) __attribute__((always_inline)) {
        const mw_group_desc *d = src.desc + g;
#pragma unroll
        for (int w = 0; w < NW; ++w) mm[w] = d->mask[w];
        o = *(const uint2 *)&d->row_offset;          // (row_offset, row_count)
        p = *(const uint2 *)&src.desc[g > 0 ? g - 1u : 0u].row_offset;
        if (g == 0) p = make_uint2(0u, 0u);
    };
    auto valid = [&](uint2 o, uint2 p) __attribute__((always_inline)) {
        return o.y >= 1 && (uint64_t)o.x + o.y <= n_rows && o.x >= (uint64_t)p.x + p.y;
    };
    auto kept = [&](const uint64_t (&mm)[NW]) __attribute__((always_inline)) {
        uint64_t any = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) any |= mm[w] & hb[w];
        return any != 0;
    };
    const bool work = g_first < g_end;
    if (work) load(min(g_first + tid, g_end - 1u), m, oc, po);               // in flight beside the counting
    uint32_t carry_g = 0, carry_r = 0;
    constexpr int kFly = NW == 1 ? 4 : NW == 2 ? 3 : 1;                      // (within the 64 registers of the riding form)
    for (uint32_t g0 = 0; g0 < g_first; g0 += (uint32_t)kFly * bs) {
        uint64_t mm[kFly][NW];
        uint2 o[kFly], p[kFly];
#pragma unroll
        for (int k = 0; k < kFly; ++k)
            if (g0 + (uint32_t)k * bs < g_first) load(min(g0 + (uint32_t)k * bs + tid, g_first - 1u), mm[k], o[k], p[k]);
#pragma unroll
        for (int k = 0; k < kFly; ++k) {
            if (g0 + (uint32_t)k * bs + tid < g_first && kept(mm[k]) && valid(o[k], p[k])) { ++carry_g; carry_r += o[k].y; }
        }
    }
    if (g_first > 0) { carry_g = relay_block_sum(carry_g, scratch); carry_r = relay_block_sum(carry_r, scratch); }
    const uint32_t before_r = carry_r;
    if (tid == 0) { fit[0] = carry_g; fit[1] = carry_r; }
    for (uint32_t g0 = g_first; g0 < g_end; g0 += bs) {
        const uint32_t g = g0 + tid;
        if (g0 > g_first) load(min(g, g_end - 1u), m, oc, po);
        const uint32_t cnt = oc.y;
        const bool keep = g < g_end && valid(oc, po) && kept(m);
        uint32_t tot_g, tot_r;
        const uint32_t cg = carry_g + mw_block_exscan(keep ? 1u : 0u, scratch, &tot_g);
        const uint32_t cr = carry_r + mw_block_exscan(keep ? cnt : 0u, scratch, &tot_r);
        uint32_t pos = kNoChild, fit_g = 0, fit_r = 0;
        if (keep) {
            if ((uint64_t)cr + cnt <= cap) {
                mw_group_desc d;
                uint32_t n = 0;
#pragma unroll
                for (int w = 0; w < MW_MASK_WORDS; ++w) d.mask[w] = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    d.mask[w] = m[w] & (keep_metadata ? valid_rank_word(n_ranks, w) : hb[w]);   // (keep: every destination the parent named)
                    n += (uint32_t)__popcll(d.mask[w]);
                }
                d.row_offset = cr; d.row_count = cnt; d.n_dest = n; d.reserved0 = 0;
                cdesc[cg] = d;
                pos = cr;
                fit_g = cg + 1u; fit_r = cr + cnt;
            } else {
                err |= MW_FLAG_OUT_CAPACITY;
            }
        }
        if (g < g_end) child_pos[(size_t)g * pos_stride + h] = pos;
        carry_g += tot_g; carry_r += tot_r;
        // kept groups that fit are a prefix of the kept groups: the largest (index + 1, end row) pair describes
        // the child where its capacity ends inside this chunk
        if (carry_r > cap) {
            fit_g = mw_wave_max(fit_g);
            fit_r = mw_wave_max(fit_r);
            if ((tid & 63) == 0 && fit_g) { atomicMax(&fit[0], fit_g); atomicMax(&fit[1], fit_r); }
        } else if (tid == 0) {
            fit[0] = carry_g; fit[1] = carry_r;      // everything so far fits
        }
    }
    mw_lds_barrier();
    // the capacity ends in exactly one chunk, or nowhere: then the last chunk has the totals
    if (tid == 0) {
        if (before_r <= cap && carry_r > cap) {
            stats->groups_per_hop[h] = fit[0];
            stats->rows_per_hop[h] = fit[1];
        } else if (c + 1 == chunks && carry_r <= cap) {
            stats->groups_per_hop[h] = carry_g;
            stats->rows_per_hop[h] = carry_r;
        }
    }
    return err;
}

// What the accounting workgroups of one index found, added up in the workspace; the one that reports last
// writes the statistics (publication rules in mw_internal.h) and leaves the sums zero.  `groups`, `rows` and
// `dests`: this lane's.  Rows times destinations need 64 bits: a descriptor is checked against the one in front of it
// only, so in a damaged table any number of valid ranges may cover the same rows (a sound one stays below 2^25).  A lane
// takes at most 1024 groups of 2^24, so its 20 low bits and the rest are summed over at most 1024 lanes in 32 bits each.
__device__ __forceinline__ void relay_account_finish(uint32_t groups, uint32_t rows, unsigned long long dests, uint32_t chunks,
                                                     uint64_t row_bytes, mw_relay_acc *acc, mw_relay_stats *__restrict__ stats,
                                                     uint32_t *scratch)
{
    groups = relay_block_sum(groups, scratch);
    rows = relay_block_sum(rows, scratch);
    const uint32_t dests_lo = relay_block_sum((uint32_t)dests & 0xfffffu, scratch);
    const uint32_t dests_hi = relay_block_sum((uint32_t)(dests >> 20), scratch);
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&acc->groups, groups, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&acc->rows, (unsigned long long)rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&acc->dest_rows, dests_lo + ((unsigned long long)dests_hi << 20), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    mw_publish_barrier();
    if (threadIdx.x != 0 || mw_report(&acc->done) != chunks - 1u) return;
    stats->n_groups_in = __hip_atomic_load(&acc->groups, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    stats->n_rows_in = (uint32_t)__hip_atomic_load(&acc->rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    stats->unicast_bytes = (uint64_t)__hip_atomic_load(&acc->dest_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * row_bytes;
    stats->reserved0 = 0;
    __hip_atomic_store(&acc->groups, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&acc->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&acc->rows, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&acc->dest_rows, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup `wg` of the relay index, of (n_hops + 1) chunks: wg / chunks < n_hops builds a chunk of that child's
// descriptor table, the last `chunks` map rows to groups and do the accounting.  Any workgroup size that is a multiple of 64.
__device__ __forceinline__ void relay_index_body(const mw_relay_index_args &a, const uint32_t wg)
{
    const uint32_t bs = blockDim.x, tid = threadIdx.x, lane = tid & 63u;
    __shared__ uint32_t scratch[17];
    __shared__ uint32_t fit[2];                  // groups, rows of the child that fit its capacity
    const uint32_t chunks = a.chunks, h = wg / chunks, c = wg - h * chunks;
    const mw_recv_peer src = a.in[0];
    const uint32_t G = min(src.n_desc, a.max_tokens), n_rows = min(src.n_rows, a.max_tokens);
    const uint32_t pos_stride = relay_pos_stride(a.n_hops);
    uint32_t err = (src.n_desc > a.max_tokens || src.n_rows > a.max_tokens) ? MW_FLAG_BAD_DESC : 0u;

    if (h < (uint32_t)a.n_hops) {
        mw_group_desc *cdesc = a.children[h].desc;
#define MW_HOP(NW_)                                                                                                      \
    relay_index_hop<NW_>(src, G, n_rows, cdesc, (int)h, c, chunks, a.n_ranks, a.cap, a.hop_bits, a.child_pos, pos_stride, a.stats, \
                         a.keep_metadata, scratch, fit)
        if (a.n_ranks <= 64) err |= MW_HOP(1);
        else if (a.n_ranks <= 128) err |= MW_HOP(2);
        else err |= MW_HOP(MW_MASK_WORDS);
#undef MW_HOP
    } else {
        // ---- rows -> groups, accounting, a group a lane.  A group's lane writes the group's index over its
        // rows; groups longer than kLongGroup rows are filled by their wave.  Rows of no valid group keep whatever
        // the array held: the copy kernel checks every entry against the descriptors.
        const uint32_t per = ((G + chunks - 1) / chunks + bs - 1) / bs * bs;
        const uint32_t g_first = min(G, c * per), g_end = min(G, g_first + per);
        uint32_t groups = 0, rows = 0;
        unsigned long long dests = 0;
        for (uint32_t g0 = g_first; g0 < g_end; g0 += bs) {
            const uint32_t g = g0 + tid, gl = min(g, g_end - 1u);
            const mw_group_desc *d = src.desc + gl;
            uint64_t m[MW_MASK_WORDS];
#pragma unroll
            for (int w = 0; w < MW_MASK_WORDS; ++w) m[w] = d->mask[w];
            const uint2 oc = *(const uint2 *)&d->row_offset;
            uint2 po = *(const uint2 *)&src.desc[gl > 0 ? gl - 1u : 0u].row_offset;
            if (gl == 0) po = make_uint2(0u, 0u);
            const uint32_t off = oc.x, cnt = oc.y;
            const bool valid = g < g_end && cnt >= 1 && (uint64_t)off + cnt <= n_rows && off >= (uint64_t)po.x + po.y;
            if (g < g_end && !valid) err |= MW_FLAG_BAD_DESC;
            if (valid) {
                uint32_t nd = 0;
#pragma unroll
                for (int w = 0; w < MW_MASK_WORDS; ++w) {
                    const uint64_t ok = valid_rank_word(a.n_ranks, w);
                    if (m[w] & ~ok) err |= MW_FLAG_BAD_RANK;
                    nd += (uint32_t)__popcll(m[w] & ok);
                }
                ++groups; rows += cnt; dests += (unsigned long long)cnt * nd;
                if (cnt <= kLongGroup) for (uint32_t r = 0; r < cnt; ++r) a.group_of_row[off + r] = (int32_t)g;
            }
            uint64_t longs = __ballot(valid && cnt > kLongGroup);
            while (longs) {
                const int l = (int)__builtin_ctzll(longs);
                longs &= longs - 1;
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)off, l), lc = (uint32_t)__builtin_amdgcn_readlane((int)cnt, l);
                const int32_t lg = __builtin_amdgcn_readlane((int)g, l);
                for (uint32_t r = lane; r < lc; r += 64u) a.group_of_row[lo + r] = lg;
            }
        }
        if (c == 0) for (uint32_t q = (uint32_t)a.n_hops + tid; q < MW_MAX_HOPS; q += bs) { a.stats->groups_per_hop[q] = 0; a.stats->rows_per_hop[q] = 0; }
        relay_account_finish(groups, rows, dests, chunks, a.row_bytes, (mw_relay_acc *)a.relay_flags, a.stats, scratch);
    }
    if (err) atomicOr(a.relay_flags, err);
}

__global__ __launch_bounds__(kBlock) void k_relay_index(const mw_relay_index_args a)
{
    relay_index_body(a, blockIdx.x);
}

// blockIdx.x selects a segment of blockDim.x chunks of a row; rows i_first, i_first + i_stride, ...  kPart: the rows by mw_st16_part
// (mw_relay_rows_part).
template <bool kPart>
__device__ __forceinline__ void relay_copy_body(
    const mw_recv_peer *__restrict__ in, const mw_relay_child *__restrict__ children, int n_hops, int K, int n_chunks,
    int ns, uint32_t max_tokens, uint64_t row_bytes, const int32_t *__restrict__ group_of_row,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats,
    const uint32_t i_first, const uint32_t i_stride)
{
    const mw_recv_peer src = in[0];
    const uint32_t n_rows = min(src.n_rows, max_tokens), n_desc = min(src.n_desc, max_tokens);
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    for (uint32_t i = i_first; i < n_rows; i += i_stride) {
        // the payload's address depends on the row alone: requested first, the group lookups
        // (two dependent round trips) are in flight beside it
        u32x4 v = {0u, 0u, 0u, 0u};
        if (c < n_chunks) v = mw_ld16((const u32x4 *)src.rows + (size_t)i * ns + c);     // ns: chunks from row to row
        const int32_t st = src.row_src_token[i];
        const int32_t g = group_of_row[i];
        if (g < 0 || (uint32_t)g >= n_desc) continue;        // (stale or never written)
        const uint32_t off = i - src.desc[g].row_offset;
        if (off >= src.desc[g].row_count) continue;          // behind its group's end: in no valid group
        const uint32_t p = (lane < n_hops) ? child_pos[(size_t)g * relay_pos_stride(n_hops) + lane] : kNoChild;
        int32_t tk = 0;
        if ((int)threadIdx.x < K && blockIdx.x == 0) tk = src.row_topk[(size_t)i * K + threadIdx.x];
        uint64_t hops = __ballot(p != kNoChild);              // the same in every wave
        while (hops) {
            const int h = __ffsll((unsigned long long)hops) - 1;
            hops &= hops - 1;
            const uint32_t dst = (uint32_t)__shfl((int)p, h, 64) + off;
            const mw_relay_child ch = children[h];
            if (c < n_chunks) mw_st16_as<kPart>((u32x4 *)ch.rows + (size_t)dst * ns + c, v);
            if (blockIdx.x == 0) {
                if (threadIdx.x == 0) ch.row_src_token[dst] = st;
                if ((int)threadIdx.x < K) ch.row_topk[(size_t)dst * K + threadIdx.x] = tk;
            }
        }
    }
    if (blockIdx.x == 0 && i_first == 0 && threadIdx.x == 0) {
        unsigned long long rows_out = 0;
        for (int h = 0; h < n_hops; ++h) rows_out += stats->rows_per_hop[h];
        stats->forward_bytes = rows_out * row_bytes;
        stats->error_flags = __hip_atomic_load(relay_flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(relay_flags, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next relay
    }
}

template <bool kPart>
__global__ __launch_bounds__(1024) void k_relay_copy(
    const mw_recv_peer *__restrict__ in, const mw_relay_child *__restrict__ children, int n_hops, int K, int n_chunks,
    int ns, uint32_t max_tokens, uint64_t row_bytes, const int32_t *__restrict__ group_of_row,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats)
{
    relay_copy_body<kPart>(in, children, n_hops, K, n_chunks, ns, max_tokens, row_bytes, group_of_row, child_pos, relay_flags,
                    stats, blockIdx.y, gridDim.y);
}

// A stream of relay steps on one stream (Section 4.3.3; the relay module of Section 5.1 handles
// one buffer after the other): the copy of this step's buffer and, in the first
// rows of the grid, the index of the NEXT step's buffer, written to another context's
// workspace.  The index is a chain of memory round trips that moves almost nothing; as a launch
// of its own it costs about 15 us in front of every copy.  Held to 64 registers so that the copy
// keeps every wave slot.
template <bool kPart>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_relay_copy_index_next(
    const uint32_t first_copy_row, const uint32_t unused0,     // (the copy's arguments first: in registers when a wave starts)
    const mw_recv_peer *__restrict__ in, const mw_relay_child *__restrict__ children, int n_hops, int K, int n_chunks,
    int ns, uint32_t max_tokens, uint64_t row_bytes, const int32_t *__restrict__ group_of_row,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats,
    const mw_relay_index_args next)
{
    if (blockIdx.y >= first_copy_row) {          // the copy's branch first: nothing to fetch in front of it
        relay_copy_body<kPart>(in, children, n_hops, K, n_chunks, ns, max_tokens, row_bytes, group_of_row, child_pos,
                        relay_flags, stats, blockIdx.y - first_copy_row, gridDim.y - first_copy_row);
        return;
    }
    const uint32_t w = blockIdx.y * gridDim.x + blockIdx.x;
    if (w < ((uint32_t)next.n_hops + 1u) * next.chunks) relay_index_body(next, w);
}

// Several buffers in one launch (mw_relay_batch): the copies of n_copy buffers, `rows_per_copy`
// grid rows each, behind the index rows of n_index further buffers.  A copy workgroup finds its
// buffer by one division and reads that buffer's arguments from the kernel arguments.
struct mw_relay_copy_args {
    const mw_recv_peer *in; const mw_relay_child *children; const int32_t *group_of_row; const uint32_t *child_pos;
    uint32_t *relay_flags; mw_relay_stats *stats; int n_hops; int reserved0;
};
struct mw_relay_batch_args {
    mw_relay_copy_args copy[MW_RELAY_BATCH_MAX];
    mw_relay_index_args index[MW_RELAY_BATCH_MAX];
    uint32_t index_first_row[MW_RELAY_BATCH_MAX + 1];      // grid rows [first[k], first[k + 1]) index buffer k
};

template <bool kPart>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_relay_batch(
    const uint32_t first_copy_row, const uint32_t rows_per_copy, int K, int n_chunks, int ns, uint32_t max_tokens,
    uint64_t row_bytes, const mw_relay_batch_args b)
{
    if (blockIdx.y >= first_copy_row) {
        const uint32_t y = blockIdx.y - first_copy_row, j = y / rows_per_copy;
        const mw_relay_copy_args &c = b.copy[j];
        relay_copy_body<kPart>(c.in, c.children, c.n_hops, K, n_chunks, ns, max_tokens, row_bytes, c.group_of_row, c.child_pos,
                        c.relay_flags, c.stats, y - j * rows_per_copy, rows_per_copy);
        return;
    }
    int k = 0;
#pragma unroll
    for (int q = 1; q < MW_RELAY_BATCH_MAX; ++q) k += (blockIdx.y >= b.index_first_row[q]) ? 1 : 0;
    const mw_relay_index_args &a = b.index[k];
    const uint32_t w = (blockIdx.y - b.index_first_row[k]) * gridDim.x + blockIdx.x;
    if (w < ((uint32_t)a.n_hops + 1u) * a.chunks) relay_index_body(a, w);
}

// ---- the same step for packets (Section 4.1, "Replication and forwarding": the relay parses the
// bitmap in front of the payload, makes one copy per distinct egress port and updates the
// in-packet metadata of each copy).  Every packet is its own group, so there is no row -> group
// map: workgroup h ranks the packets that hop h keeps (child position = exclusive count), the
// extra workgroup does the accounting, and the copy kernel reads a packet once and stores it
// once per hop with the first 32 bytes -- the bitmap -- replaced by its restriction to that hop.
// Everything the index of one relay step of packets needs (one kernel argument).
struct mw_relay_packets_index_args {
    const mw_recv_packets *in; int n_hops, n_ranks; uint32_t K, max_tokens, cap; uint64_t packet_bytes;
    const uint64_t *hop_bits; uint32_t *child_pos; uint32_t *relay_flags; mw_relay_stats *stats;
    uint32_t chunks;            // workgroups per hop
};

// Positions of the packets of chunk c that next hop h keeps: what the hop keeps of the chunks before is counted
// first, several headers a lane in flight, then a packet a lane (as relay_index_hop).  Of a header: the NW
// bitmap words that can name a rank and the id count.  Four headers of four words took the riding form to 64 vector
// registers and scratch, which its movers paid for: 4096 packets of 14464 bytes over 15 hops 59.1 us a step, with
// one 56.2 (38 registers).
template <int NW>
__device__ __forceinline__ uint32_t relay_packets_index_hop(
    const char *__restrict__ packets, const uint64_t packet_bytes, const uint32_t n_rows, const uint32_t K, const int h,
    const uint32_t c, const uint32_t chunks, const uint32_t cap, const uint64_t *__restrict__ hop_bits,
    uint32_t *__restrict__ child_pos, const uint32_t pos_stride, mw_relay_stats *__restrict__ stats, uint32_t *scratch)
{
    const uint32_t tid = threadIdx.x, bs = blockDim.x;
    const uint32_t per = ((n_rows + chunks - 1) / chunks + bs - 1) / bs * bs;
    const uint32_t first = min(n_rows, c * per), end = min(n_rows, first + per);
    if (first >= n_rows && c + 1 < chunks) return 0;
    uint32_t err = 0;
    uint64_t hb[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) hb[w] = hop_bits[(size_t)h * MW_MASK_WORDS + w];
    auto load = [&](uint32_t i, uint64_t (&m)[NW], uint32_t &nid) __attribute__((always_inline)) {
        const char *hd = packets + (size_t)i * packet_bytes;
#pragma unroll
        for (int w = 0; w < NW; ++w) m[w] = *(const uint64_t *)(hd + 8 * w);
        nid = *(const uint32_t *)(hd + 36);
    };
    auto kept = [&](const uint64_t (&m)[NW], uint32_t nid) __attribute__((always_inline)) {
        uint64_t any = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) any |= m[w] & hb[w];
        return any != 0 && nid == K;
    };
    uint64_t m[NW];
    uint32_t nid = 0;
    if (first < end) load(min(first + tid, end - 1u), m, nid);
    uint32_t carry = 0;
    constexpr int kFly = NW == 1 ? 4 : NW == 2 ? 3 : 1;
    for (uint32_t i0 = 0; i0 < first; i0 += (uint32_t)kFly * bs) {
        uint64_t mm[kFly][NW];
        uint32_t nn[kFly];
#pragma unroll
        for (int k = 0; k < kFly; ++k)
            if (i0 + (uint32_t)k * bs < first) load(min(i0 + (uint32_t)k * bs + tid, first - 1u), mm[k], nn[k]);
#pragma unroll
        for (int k = 0; k < kFly; ++k)
            if (i0 + (uint32_t)k * bs + tid < first && kept(mm[k], nn[k])) ++carry;
    }
    if (first > 0) carry = relay_block_sum(carry, scratch);
    for (uint32_t i0 = first; i0 < end; i0 += bs) {
        const uint32_t i = i0 + tid;
        if (i0 > first) load(min(i, end - 1u), m, nid);
        const bool keep = i < end && kept(m, nid);
        uint32_t tot;
        const uint32_t pos = carry + mw_block_exscan(keep ? 1u : 0u, scratch, &tot);
        const bool fits = keep && pos < cap;
        if (keep && !fits) err |= MW_FLAG_OUT_CAPACITY;
        if (i < end) child_pos[(size_t)i * pos_stride + h] = fits ? pos : kNoChild;
        carry += tot;
    }
    if (tid == 0 && c + 1 == chunks) {
        const uint32_t fit = min(carry, cap);      // the packets that fit are a prefix of the kept ones
        stats->groups_per_hop[h] = fit; stats->rows_per_hop[h] = fit;
    }
    return err;
}

// Workgroup `wg` of the packets' relay index, of (n_hops + 1) chunks: positions of a chunk for a hop, then the
// accounting's chunks.  Any workgroup size that is a multiple of 64.
__device__ __forceinline__ void relay_packets_index_body(const mw_relay_packets_index_args &a, const uint32_t wg)
{
    __shared__ uint32_t scratch[17];
    const uint32_t tid = threadIdx.x, bs = blockDim.x;
    const uint32_t chunks = a.chunks, h = wg / chunks, c = wg - h * chunks;
    const mw_recv_packets src = a.in[0];
    const char *packets = (const char *)src.packets;
    const uint32_t n_rows = min(src.n_rows, a.max_tokens);
    uint32_t err = src.n_rows > a.max_tokens ? MW_FLAG_BAD_DESC : 0u;

    if (h < (uint32_t)a.n_hops) {
#define MW_HOP(NW_)                                                                                                      \
    relay_packets_index_hop<NW_>(packets, a.packet_bytes, n_rows, a.K, (int)h, c, chunks, a.cap, a.hop_bits, a.child_pos,   \
                                 relay_pos_stride(a.n_hops), a.stats, scratch)
        if (a.n_ranks <= 64) err |= MW_HOP(1);
        else if (a.n_ranks <= 128) err |= MW_HOP(2);
        else err |= MW_HOP(MW_MASK_WORDS);
#undef MW_HOP
    } else {
        const uint32_t per = ((n_rows + chunks - 1) / chunks + bs - 1) / bs * bs;
        const uint32_t first = min(n_rows, c * per), end = min(n_rows, first + per);
        uint32_t taken = 0, dests = 0;
        for (uint32_t i0 = first; i0 < end; i0 += bs) {
            const char *hd = packets + (size_t)min(i0 + tid, end - 1u) * a.packet_bytes;
            uint64_t m[MW_MASK_WORDS];
#pragma unroll
            for (int w = 0; w < MW_MASK_WORDS; ++w) m[w] = *(const uint64_t *)(hd + 8 * w);
            const uint32_t nid = *(const uint32_t *)(hd + 36);
            if (i0 + tid >= end) continue;
            if (nid != a.K) { err |= MW_FLAG_BAD_DESC; continue; }
#pragma unroll
            for (int w = 0; w < MW_MASK_WORDS; ++w) {
                const uint64_t ok = valid_rank_word(a.n_ranks, w);
                if (m[w] & ~ok) err |= MW_FLAG_BAD_RANK;
                dests += (uint32_t)__popcll(m[w] & ok);
            }
            ++taken;
        }
        if (c == 0) for (uint32_t q = (uint32_t)a.n_hops + tid; q < MW_MAX_HOPS; q += bs) { a.stats->groups_per_hop[q] = 0; a.stats->rows_per_hop[q] = 0; }
        relay_account_finish(taken, taken, dests, chunks, a.packet_bytes, (mw_relay_acc *)a.relay_flags, a.stats, scratch);
    }
    if (err) atomicOr(a.relay_flags, err);
}

__global__ __launch_bounds__(kBlock) void k_relay_packets_index(const mw_relay_packets_index_args a)
{
    relay_packets_index_body(a, blockIdx.x);
}

// blockIdx.x selects a segment of blockDim.x chunks of a packet; packets i_first, i_first + i_stride, ...
template <bool kPart>
__device__ __forceinline__ void relay_packets_copy_body(
    const mw_recv_packets *__restrict__ in, void *const *__restrict__ children, int n_hops, int n_chunks,
    uint32_t max_tokens, uint64_t packet_bytes, const uint64_t *__restrict__ hop_bits,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats,
    const uint32_t keep_metadata, const uint32_t i_first, const uint32_t i_stride)
{
    const mw_recv_packets src = in[0];
    const uint32_t n_rows = min(src.n_rows, max_tokens);
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    for (uint32_t i = i_first; i < n_rows; i += i_stride) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (c < n_chunks) v = mw_ld16((const u32x4 *)src.packets + (size_t)i * n_chunks + c);
        const uint32_t p = (lane < n_hops) ? child_pos[(size_t)i * relay_pos_stride(n_hops) + lane] : kNoChild;
        uint64_t hops = __ballot(p != kNoChild);              // the same in every wave
        while (hops) {
            const int h = __ffsll((unsigned long long)hops) - 1;
            hops &= hops - 1;
            const uint32_t dst = (uint32_t)__shfl((int)p, h, 64);
            u32x4 o = v;
            if (c < 2 && !keep_metadata) {                    // chunks 0 and 1 are the bitmap: restricted to the hop's ranks
                const uint64_t b0 = hop_bits[(size_t)h * MW_MASK_WORDS + 2 * c];
                const uint64_t b1 = hop_bits[(size_t)h * MW_MASK_WORDS + 2 * c + 1];
                o.x &= (uint32_t)b0; o.y &= (uint32_t)(b0 >> 32); o.z &= (uint32_t)b1; o.w &= (uint32_t)(b1 >> 32);
            }
            if (c < n_chunks) mw_st16_as<kPart>((u32x4 *)children[h] + (size_t)dst * n_chunks + c, o);
        }
    }
    if (blockIdx.x == 0 && i_first == 0 && threadIdx.x == 0) {
        unsigned long long rows_out = 0;
        for (int h = 0; h < n_hops; ++h) rows_out += stats->rows_per_hop[h];
        stats->forward_bytes = rows_out * packet_bytes;
        stats->error_flags = __hip_atomic_load(relay_flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(relay_flags, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next relay
    }
}

template <bool kPart>
__global__ __launch_bounds__(1024) void k_relay_packets_copy(
    const mw_recv_packets *__restrict__ in, void *const *__restrict__ children, int n_hops, int n_chunks,
    uint32_t max_tokens, uint64_t packet_bytes, const uint64_t *__restrict__ hop_bits,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats,
    const uint32_t keep_metadata)
{
    relay_packets_copy_body<kPart>(in, children, n_hops, n_chunks, max_tokens, packet_bytes, hop_bits, child_pos, relay_flags,
                            stats, keep_metadata, blockIdx.y, gridDim.y);
}

// The packets' form of k_relay_copy_index_next: this buffer's copy with the next buffer's index
// (another context's workspace) in the first rows of the grid.  Held to 64 scalar
// registers as well: with the 69 the index's branch would take, the copy's step is 6 % longer
// (56.9 -> 60.4 us; forcing the count up with nothing else changed shows the same), the four
// values over the limit live in lanes of a vector register instead.
template <bool kPart>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8), amdgpu_num_sgpr(64))) void k_relay_packets_copy_index_next(
    const uint32_t first_copy_row, const uint32_t unused0,
    const mw_recv_packets *__restrict__ in, void *const *__restrict__ children, int n_hops, int n_chunks,
    uint32_t max_tokens, uint64_t packet_bytes, const uint64_t *__restrict__ hop_bits,
    const uint32_t *__restrict__ child_pos, uint32_t *relay_flags, mw_relay_stats *__restrict__ stats,
    const uint32_t keep_metadata, const mw_relay_packets_index_args next)
{
    if (blockIdx.y >= first_copy_row) {
        relay_packets_copy_body<kPart>(in, children, n_hops, n_chunks, max_tokens, packet_bytes, hop_bits, child_pos,
                                relay_flags, stats, keep_metadata, blockIdx.y - first_copy_row,
                                gridDim.y - first_copy_row);
        return;
    }
    const uint32_t w = blockIdx.y * gridDim.x + blockIdx.x;
    if (w < ((uint32_t)next.n_hops + 1u) * next.chunks) relay_packets_index_body(next, w);
}

}  // namespace

// Workgroup shape of a copy that carries a riding index, for long rows that would otherwise move
// as single waves: wide enough for the index, whose workgroups take a group a lane.  The copy hardly minds:
// 14336-byte rows, 15 next hops, per step of a stream: 64 lanes 60.5 us, 128: 55.9, 192: 57.1, 320: 55.9 (the copy alone 53).
// An even number of unequal segments would hand the short segment to the same XCDs every row.
static mw_row_shape relay_stream_shape(int n_chunks)
{
    int nseg = (n_chunks + 383) / 384;
    if (nseg > 1 && nseg % 2 == 0) ++nseg;
    return mw_row_shape{((n_chunks + nseg - 1) / nseg + 63) / 64 * 64, nseg};
}

// Index workgroups of `bs` lanes per hop: one per `bs` groups the buffer may hold, at most kMaxChunks.
static uint32_t relay_chunks(const mw_ctx *ctx, int bs)
{
    const uint32_t n = ((uint32_t)ctx->cfg.max_tokens + (uint32_t)bs - 1u) / (uint32_t)bs;
    return n < 1 ? 1u : n < kMaxChunks ? n : kMaxChunks;
}
// Grid rows of `nseg` workgroups that a riding index takes.
static uint32_t relay_index_rows(const mw_ctx *next, uint32_t chunks, int nseg)
{
    return (((uint32_t)next->n_hops + 1u) * chunks + (uint32_t)nseg - 1u) / (uint32_t)nseg;
}

// Whether the next buffer's index rides in a copy of `ctx` with `bs`-lane workgroups or gets a launch of its own
// in front.  A riding workgroup takes about 1.6 us for four groups a lane of those it counts (the last
// chunk's: all in front of it) and for every group a lane it places, and narrow workgroups have few lanes; the copy takes at
// least its rows once in and, say, twice out at 6 TB/s; a launch of its own about 10 us.  (16384 rows of 2048 bytes, 128 lanes: riding 64.5 us a step,
// apart 48.8; 4096 rows of 14336 bytes, 320 lanes: 55.9 and 60.5.)
static double relay_rider_us(const mw_ctx *next, int bs, uint32_t chunks)
{
    const double groups = (double)next->cfg.max_tokens;
    return 1.6 * ((chunks > 1 ? groups / (4.0 * bs) : 0.0) + groups / ((double)chunks * bs));
}
static double relay_copy_us(const mw_ctx *ctx, int64_t row_bytes) { return 3.0 * (double)ctx->cfg.max_tokens * (double)row_bytes / 6e6; }
static bool relay_index_rides(const mw_ctx *ctx, const mw_ctx *next, int bs, int64_t row_bytes)
{
    return relay_rider_us(next, bs, relay_chunks(next, bs)) < relay_copy_us(ctx, row_bytes) + 10.0;
}

// Chunks a hop of an index that rides beside copies of `copy_us`: as few as they hide, since every chunk of every hop reads
// the descriptors in front of it again (a rider takes about 5 us before its first group).  4096 rows of 14336 bytes, us a
// buffer with 1, 3, 13 chunks: 15 hops 55.0, 55.1, 55.4, 39 hops of 256 ranks 54.3, 54.5, 56.1, two buffers a
// launch 54.2, 55.5, 58.0; 8192 rows of 4096 bytes, two buffers a launch, with 1, 3, 16 chunks 36.3, 31.2, 39.5.
static uint32_t relay_riding_chunks(const mw_ctx *next, int bs, double copy_us)
{
    const uint32_t most = relay_chunks(next, bs);
    uint32_t n = 1;
    while (n < most && 5.0 + relay_rider_us(next, bs, n) >= copy_us) ++n;
    return n;
}

static mw_relay_index_args relay_index_args(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children,
                                            int64_t cap, mw_relay_stats *stats, int bs)
{
    mw_relay_index_args a;
    a.in = in; a.children = children; a.n_hops = ctx->n_hops; a.n_ranks = ctx->cfg.n_ranks;
    a.max_tokens = (uint32_t)ctx->cfg.max_tokens; a.cap = (uint32_t)cap; a.row_bytes = (uint64_t)ctx->row_bytes;
    a.hop_bits = ctx->d_hop_bits; a.group_of_row = ctx->d_group_of_row; a.child_pos = ctx->d_child_pos;
    a.relay_flags = ctx->d_relay_flags; a.stats = stats;
    a.keep_metadata = (ctx->options & MW_OPT_RELAY_KEEP_METADATA) ? 1u : 0u;
    a.chunks = relay_chunks(ctx, bs);
    return a;
}

int32_t mw_launch_relay_index(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children, int64_t cap,
                              mw_relay_stats *stats, hipStream_t s)
{
    {
        mw_timed tm(ctx, MW_KERNEL_RELAY_INDEX, s);
        const mw_relay_index_args a = relay_index_args(ctx, in, children, cap, stats, kBlock);
        hipLaunchKernelGGL(k_relay_index, dim3(((uint32_t)ctx->n_hops + 1u) * a.chunks), dim3(kBlock), 0, s, a);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

// `next` != nullptr: the index of the next step's buffer rides in the same launch.
int32_t mw_launch_relay_copy(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children,
                             mw_relay_stats *stats, mw_ctx *next, const mw_recv_peer *next_in,
                             const mw_relay_child *next_children, int64_t next_cap, mw_relay_stats *next_stats,
                             hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    const int n_chunks = (int)(ctx->row_bytes / 16);
    mw_row_shape shape = mw_row_shape_of(n_chunks);
    if (next) {
        const mw_row_shape wide = shape.bs == 64 && n_chunks % 16 == 0 ? relay_stream_shape(n_chunks) : shape;
        if (relay_index_rides(ctx, next, wide.bs, ctx->row_bytes)) {
            shape = wide;
        } else {
            const int32_t rc = mw_launch_relay_index(next, next_in, next_children, next_cap, next_stats, s);
            if (rc != MW_OK) return rc;
            next = nullptr;
        }
    }
    uint32_t gy = (uint32_t)c.max_tokens < kRowGridMax ? (uint32_t)c.max_tokens : kRowGridMax;
    if (gy < 1) gy = 1;
    const bool part = mw_relay_rows_part(ctx->row_stride, c.max_tokens, false, next != nullptr);
    {
        mw_timed tm(ctx, MW_KERNEL_RELAY_COPY, s);
        if (!next) {
            hipLaunchKernelGGL(part ? k_relay_copy<true> : k_relay_copy<false>, dim3(shape.nseg, gy), dim3(shape.bs), 0, s, in, children, ctx->n_hops,
                               c.top_k, n_chunks, (int)(ctx->row_stride / 16), (uint32_t)c.max_tokens,
                               (uint64_t)ctx->row_bytes, ctx->d_group_of_row, ctx->d_child_pos, ctx->d_relay_flags, stats);
        } else {
            mw_relay_index_args a = relay_index_args(next, next_in, next_children, next_cap, next_stats, shape.bs);
            a.chunks = relay_riding_chunks(next, shape.bs, relay_copy_us(ctx, ctx->row_bytes));
            const uint32_t riders = relay_index_rows(next, a.chunks, shape.nseg);
            hipLaunchKernelGGL(part ? k_relay_copy_index_next<true> : k_relay_copy_index_next<false>, dim3(shape.nseg, gy + riders), dim3(shape.bs), 0, s,
                               riders, 0u, in, children, ctx->n_hops, c.top_k, n_chunks, (int)(ctx->row_stride / 16), (uint32_t)c.max_tokens, (uint64_t)ctx->row_bytes,
                               ctx->d_group_of_row, ctx->d_child_pos, ctx->d_relay_flags, stats, a);
        }
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_relay_batch(const mw_relay_job *copy, int32_t n_copy, const mw_relay_job *index, int32_t n_index,
                              hipStream_t s)
{
    mw_ctx *ctx = copy[0].ctx;
    const mw_config &c = ctx->cfg;
    const int n_chunks = (int)(ctx->row_bytes / 16);
    mw_row_shape shape = mw_row_shape_of(n_chunks);
    // long rows of whole cache lines: a few large workgroups per row beside a riding index (see mw_launch_relay_copy)
    if (n_index > 0 && shape.bs == 64 && n_chunks % 16 == 0) shape = relay_stream_shape(n_chunks);
    uint32_t gy = (uint32_t)c.max_tokens < 8192u ? (uint32_t)c.max_tokens : 8192u;      // per buffer; more rows by striding
    if (gy < 1) gy = 1;
    mw_relay_batch_args b = {};
    for (int j = 0; j < n_copy; ++j) {
        mw_ctx *x = copy[j].ctx;
        b.copy[j] = mw_relay_copy_args{copy[j].in_dev, copy[j].children_dev, x->d_group_of_row, x->d_child_pos,
                                       x->d_relay_flags, copy[j].stats_dev, x->n_hops, 0};
    }
    uint32_t first = 0;
    for (int k = 0; k < MW_RELAY_BATCH_MAX; ++k) {
        b.index_first_row[k] = first;
        if (k < n_index) {
            b.index[k] = relay_index_args(index[k].ctx, index[k].in_dev, index[k].children_dev,
                                          index[k].child_capacity_rows, index[k].stats_dev, shape.bs);
            b.index[k].chunks = relay_riding_chunks(index[k].ctx, shape.bs, n_copy * relay_copy_us(ctx, ctx->row_bytes));
            first += relay_index_rows(index[k].ctx, b.index[k].chunks, shape.nseg);
        }
    }
    b.index_first_row[MW_RELAY_BATCH_MAX] = first;
    const bool part = mw_relay_rows_part(ctx->row_stride, c.max_tokens, false, n_index > 0);
    {
        mw_timed tm(ctx, MW_KERNEL_RELAY_COPY, s);
        hipLaunchKernelGGL(part ? k_relay_batch<true> : k_relay_batch<false>, dim3(shape.nseg, first + gy * (uint32_t)n_copy), dim3(shape.bs), 0, s, first, gy,
                           c.top_k, n_chunks, (int)(ctx->row_stride / 16), (uint32_t)c.max_tokens,
                           (uint64_t)ctx->row_bytes, b);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_relay(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children, int64_t cap,
                        mw_relay_stats *stats, hipStream_t s)
{
    const int32_t rc = mw_launch_relay_index(ctx, in, children, cap, stats, s);
    if (rc != MW_OK) return rc;
    return mw_launch_relay_copy(ctx, in, children, stats, nullptr, nullptr, nullptr, 0, nullptr, s);
}

static mw_relay_packets_index_args relay_packets_index_args(mw_ctx *ctx, const mw_recv_packets *in, int64_t cap,
                                                            mw_relay_stats *stats, int bs)
{
    mw_relay_packets_index_args a;
    a.in = in; a.n_hops = ctx->n_hops; a.n_ranks = ctx->cfg.n_ranks; a.K = (uint32_t)ctx->cfg.top_k;
    a.max_tokens = (uint32_t)ctx->cfg.max_tokens; a.cap = (uint32_t)cap;
    a.packet_bytes = (uint64_t)(mw_packet_header_bytes_of(ctx->cfg.top_k) + ctx->row_bytes);
    a.hop_bits = ctx->d_hop_bits; a.child_pos = ctx->d_child_pos; a.relay_flags = ctx->d_relay_flags; a.stats = stats;
    a.chunks = relay_chunks(ctx, bs);
    return a;
}

int32_t mw_launch_relay_packets_index(mw_ctx *ctx, const mw_recv_packets *in, int64_t cap, mw_relay_stats *stats,
                                      hipStream_t s)
{
    {
        mw_timed tm(ctx, MW_KERNEL_RELAY_INDEX, s);
        mw_relay_packets_index_args a = relay_packets_index_args(ctx, in, cap, stats, kBlock);
        // No more workgroups than CUs (4096 packets of 14464 bytes, 256 ranks, 39 hops: mw_relay_packets with 8 chunks a hop, 320
        // workgroups, 70.0 us, with 6 64.9, with 4 65.5, with one 70.8).
        while (a.chunks > 1 && ((uint32_t)ctx->n_hops + 1u) * a.chunks > (uint32_t)ctx->n_cu) --a.chunks;
        hipLaunchKernelGGL(k_relay_packets_index, dim3(((uint32_t)ctx->n_hops + 1u) * a.chunks), dim3(kBlock), 0, s, a);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

// `next` != nullptr: the index of the next step's packets rides in the same launch.
int32_t mw_launch_relay_packets_copy(mw_ctx *ctx, const mw_recv_packets *in, void *const *children,
                                     mw_relay_stats *stats, mw_ctx *next, const mw_recv_packets *next_in,
                                     int64_t next_cap, mw_relay_stats *next_stats, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    const uint64_t pb = (uint64_t)(mw_packet_header_bytes_of(c.top_k) + ctx->row_bytes);
    const int n_chunks = (int)(pb / 16);
    const uint32_t keep = (ctx->options & MW_OPT_RELAY_KEEP_METADATA) ? 1u : 0u;
    mw_row_shape shape = mw_row_shape_of(n_chunks);
    if (next) {
        // long packets: a few larger workgroups per packet instead of single waves, for the
        // riding index's sake (see relay_stream_shape); pieces stay whole cache lines
        const mw_row_shape wide = shape.bs == 64 ? relay_stream_shape(n_chunks) : shape;
        if (relay_index_rides(ctx, next, wide.bs, (int64_t)pb)) {
            shape = wide;
        } else {
            const int32_t rc = mw_launch_relay_packets_index(next, next_in, next_cap, next_stats, s);
            if (rc != MW_OK) return rc;
            next = nullptr;
        }
    }
    uint32_t gy = (uint32_t)c.max_tokens < kRowGridMax ? (uint32_t)c.max_tokens : kRowGridMax;
    if (gy < 1) gy = 1;
    const bool part = mw_relay_rows_part((int64_t)pb, c.max_tokens, true, next != nullptr);
    {
        mw_timed tm(ctx, MW_KERNEL_RELAY_COPY, s);
        if (!next) {
            hipLaunchKernelGGL(part ? k_relay_packets_copy<true> : k_relay_packets_copy<false>, dim3(shape.nseg, gy), dim3(shape.bs), 0, s, in, children, ctx->n_hops,
                               n_chunks, (uint32_t)c.max_tokens, pb, ctx->d_hop_bits, ctx->d_child_pos,
                               ctx->d_relay_flags, stats, keep);
        } else {
            mw_relay_packets_index_args a = relay_packets_index_args(next, next_in, next_cap, next_stats, shape.bs);
            // A chunk reads the header, a cache line, of every packet in front of it: thirteen chunks are seven times
            // the headers, which the copy pays for.  So as few chunks as the copy hides.  (us a step with 1, 3, 13 chunks: 4096
            // packets of 14464 bytes, 15 hops 56.2, 56.8, 60.1; 256 ranks, 39 hops 55.9, 58.0, 65.0; 4224 bytes,
            // 23 hops 31.5, 31.3, 34.5.)
            const double copy_us = relay_copy_us(ctx, (int64_t)pb);
            for (uint32_t n = 1; n < a.chunks; ++n)
                if (relay_rider_us(next, shape.bs, n) < copy_us + 10.0) a.chunks = n;
            const uint32_t riders = relay_index_rows(next, a.chunks, shape.nseg);
            hipLaunchKernelGGL(part ? k_relay_packets_copy_index_next<true> : k_relay_packets_copy_index_next<false>, dim3(shape.nseg, gy + riders),
                               dim3(shape.bs), 0, s, riders, 0u, in, children, ctx->n_hops, n_chunks, (uint32_t)c.max_tokens, pb,
                               ctx->d_hop_bits, ctx->d_child_pos, ctx->d_relay_flags, stats, keep, a);
        }
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_relay_packets(mw_ctx *ctx, const mw_recv_packets *in, void *const *children, int64_t cap,
                                mw_relay_stats *stats, hipStream_t s)
{
    const int32_t rc = mw_launch_relay_packets_index(ctx, in, cap, stats, s);
    if (rc != MW_OK) return rc;
    return mw_launch_relay_packets_copy(ctx, in, children, stats, nullptr, nullptr, 0, nullptr, s);
}
