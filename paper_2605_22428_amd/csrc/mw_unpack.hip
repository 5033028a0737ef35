// Receive side: index builder and expander.
//
// Paper hooks: Section 4.1 workflow steps 3-4 -- the receiver parses the carried
// metadata and, if it is one of the destinations, delivers the payload to the target
// memory; Section 5.1 -- the receive module does reception, reassembly and delivery of
// the final buffers; Section 6.4 "Memory usage" -- one pre-allocated receive region per
// peer.  The bitmap of a row's group is the authority on whether this rank is addressed;
// which local experts get the row follows from the row's top-k ids and the rank table.
//
// Two launches on the caller's stream (a batch of a few hundred rows: one, k_unpack_small):
//   k_recv_index  one workgroup per peer (a few where a peer has many experts here).  Marks
//                 addressed rows from the descriptor bitmaps, then for every local expert
//                 builds an LDS bitmap over the peer's source-token indices.  A prefix of popcounts over that bitmap
//                 is the stable rank of a row among the peer's rows for that expert,
//                 whatever order the rows were packed in -- no sort, no order-dependent
//                 atomics (LDS atomic ORs only set bits).  Emits per-(expert, peer)
//                 counts and one record per received row: source address, source token,
//                 peer and (expert slot, rank) pairs.
//                 Who turns the counts into output bases: up to 512 of them in mw_unpack and mw_unpack_packets,
//                 where the payload is not too long for it (mw_counts_by_expander), the expander behind, k_expand_counts.  Its
//                 waves add up what is in front of their places, and one wave of the launch writes bases, offsets and statistics.
//                 Else -- more counts, long payloads, mw_unpack_index, an index that rides -- the workgroup that
//                 reports its counts last (device-scope counter) scans them.  No third launch, no grid-wide barrier either way.
//   k_expand, k_expand_counts
//                 small workgroups (a single wave for long cache-line-sized rows, one
//                 workgroup per row up to 10 KiB), each moving consecutive 16-byte chunks of
//                 one received row (rows beyond 32768 by striding): a chunk is read once with
//                 a streaming load and stored to each of the row's experts' slots.  Measured
//                 on MI355X, many small waves with a single load in flight each track the
//                 plain-copy ceiling, while fewer waves with deep per-lane unrolling fall
//                 10-30 % short, and a persistent grid loses ~5 % to the hardware dispatcher.
//                 This kernel moves ~all receive-side bytes and is bound by HBM bandwidth.
// Further entry points share these bodies: k_recv_index<true> reads per-row headers (packets),
// k_expand_index_next runs the expander with the next batch's index in the same launch, and
// k_combine is the expander's mirror image for the way back.
#include <cmath>

#include "mw_internal.h"
#include "mw_plan_dev.h"
#include "mw_pack_dev.h"

namespace {

constexpr int kIndexBlock = 1024;

__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr uint32_t kWaveCounts = 8;       // counts a lane of mw_finish_counts_wave
// k_expand_counts has the same wave write the bases, unconditionally, and its own lanes hold at most eight counts
static_assert(kCountsMax <= 64 * kWaveCounts && kCountsMax <= 64 * 8, "more counts than the expander can add up");

// One workgroup: exclusive scan of the (expert, peer) counts in output order, expert
// offsets, totals and flags.  `scratch` is LDS scan scratch of 17 words.  Every device-scope
// read that does not depend on another is issued before the first scan.
__device__ __forceinline__ void mw_finish_counts(const uint32_t *cnt, const uint32_t *addr_cnt, uint32_t *flags,
                                                 const uint32_t *row_base, uint32_t L, uint32_t P, int64_t out_cap,
                                                 uint32_t *base, int64_t *expert_offsets, mw_recv_stats *stats,
                                                 uint32_t *scratch)
{
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    const uint32_t n_lp = L * P;
    uint32_t m = 0;
    for (uint32_t q = tid; q < P; q += nthr) m += ld_agent(&addr_cnt[q]);
    const uint32_t err = (tid == 0) ? ld_agent(&flags[1]) : 0u;
    const uint32_t row_base_total = (tid == 0) ? ld_agent(&row_base[P]) : 0u;
    uint32_t v_next = (tid < n_lp) ? ld_agent(&cnt[tid]) : 0u;
    uint32_t carry = 0;
    for (uint32_t f0 = 0; f0 < n_lp; f0 += nthr) {          // (expert, peer) order = output order
        const uint32_t f = f0 + tid, v = v_next;
        v_next = (f + nthr < n_lp) ? ld_agent(&cnt[f + nthr]) : 0u;
        uint32_t tot;
        const uint32_t ex = mw_block_exscan(v, scratch, &tot);
        if (f < n_lp) {
            base[f] = carry + ex;
            if (f % P == 0) expert_offsets[f / P] = (int64_t)(carry + ex);
        }
        carry += tot;
    }
    uint32_t m_tot;
    mw_block_exscan(m, scratch, &m_tot);
    if (tid == 0) {
        const uint32_t Q = carry;
        expert_offsets[L] = Q;
        stats->n_recv_rows = m_tot;
        stats->n_out_rows = Q;
        stats->error_flags = err | (((int64_t)Q > out_cap) ? MW_FLAG_OUT_CAPACITY : 0u);
        stats->n_rows_seen = row_base_total;
        st_agent(&flags[1], 0u);           // ready for the next unpack
        st_agent(&flags[2], 0u);
    }
}

// The same by one wave, without a barrier, for at most 64 kWaveCounts counts, all requested together.  (The workgroup's two
// scans and their barriers: 1.5 us after the last report, this 1.0.)
__device__ __forceinline__ void mw_finish_counts_wave(const uint32_t *cnt, const uint32_t *addr_cnt, uint32_t *flags,
                                                      const uint32_t *row_base, uint32_t L, uint32_t P, int64_t out_cap,
                                                      uint32_t *base, int64_t *expert_offsets, mw_recv_stats *stats)
{
    const uint32_t lane = threadIdx.x & 63u, n_lp = L * P;
    uint32_t v[kWaveCounts], w[4];                   // (P <= 256)
#pragma unroll
    for (uint32_t j = 0; j < kWaveCounts; ++j) v[j] = lane + 64u * j < n_lp ? ld_agent(&cnt[lane + 64u * j]) : 0u;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) w[j] = lane + 64u * j < P ? ld_agent(&addr_cnt[lane + 64u * j]) : 0u;
    const uint32_t err = ld_agent(&flags[1]), seen = ld_agent(&row_base[P]);
    const float per = 1.0f / (float)P;               // (f + 1/2) / P is at least 1/512 away from a whole number: f below 2^9 is exact
    uint32_t Q = 0;
#pragma unroll
    for (uint32_t j = 0; j < kWaveCounts; ++j) {
        const uint32_t f = lane + 64u * j;
        if (64u * j >= n_lp) break;
        const uint32_t inc = mw_wave_incl_scan(v[j]), at = Q + inc - v[j], l = (uint32_t)(((float)f + 0.5f) * per);
        if (f < n_lp) {
            base[f] = at;
            if (l * P == f) expert_offsets[l] = (int64_t)at;
        }
        Q += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    const uint32_t m = mw_wave_sum(w[0] + w[1] + w[2] + w[3]);
    if (lane == 0) {
        expert_offsets[L] = Q;
        stats->n_recv_rows = m;
        stats->n_out_rows = Q;
        stats->error_flags = err | (((int64_t)Q > out_cap) ? MW_FLAG_OUT_CAPACITY : 0u);
        stats->n_rows_seen = seen;
        st_agent(&flags[1], 0u);           // ready for the next unpack
        st_agent(&flags[2], 0u);
    }
}

// kPackets: the peers' regions hold packets (mw_recv_packets): every row is its own group and
// carries its bitmap, source token and expert ids in a header in front of it; `row_bytes` is
// then the distance between packets and `header_bytes` the payload's offset inside one.
// Everything the index of one batch needs (one kernel argument; the fused launch below carries
// it beside the expander's arguments).
struct mw_index_args {
    const void *peers; int P; const int32_t *eslot;
    int E, K, Kd, my_rank, L, Lc;
    uint32_t max_tokens, wpl, cap_rows; uint64_t row_bytes; uint32_t header_bytes; int64_t out_cap;
    uint32_t *cnt, *row_base, *addr_cnt; mw_row_rec *recs; mw_hit *hits; uint32_t *base;
    int64_t *expert_offsets; mw_recv_stats *stats; uint32_t *flags;
    uint32_t dedup;     // 1: of the rows of one peer that carry the same source token only one is taken
    uint32_t parts;     // workgroups per peer: part j takes the expert chunks j, j + parts, ... of Lc experts each
    uint32_t row_parts; // ... times this many: all of them mark every row, each ranks and writes its share of the rows
    uint32_t tab_words; // LDS words of the table of local slots (0: the rank table in memory is looked up)
};

constexpr uint32_t kLaneWords = 24;       // words of an expert that one lane walks
constexpr uint32_t kNotLocal = 0xffu;     // table entry of an expert that lives elsewhere; local slots are below 255

// What the index may assume: at most eight ids a token, at most 64 local experts and the table in LDS; the
// same with any number of ids; nothing.
constexpr int kFormFew = 0, kFormMany = 1, kFormAny = 2;

// LDS words of an index workgroup that handles Lc experts at a time.
static inline size_t mw_index_lds_words(uint32_t wpl, uint32_t Lc, uint32_t tab_words, bool dedup)
{
    const size_t n = (size_t)Lc * wpl;
    return wpl + tab_words + n + (n + 1) / 2 + 64 + (dedup ? wpl : 0);
}

// The work of workgroup (part, row_part) of peer p; any workgroup size that is a multiple of 64.
// A workgroup looks at all rows of its peer and at the experts of its chunks: it sets the bit
// (expert, source token) of every row, scans the popcounts, and a row's rank is a lookup.  Chunks are
// independent of one another (a row's hit k belongs to the workgroup that has the hit's expert, the row's
// record to the one that has hit 0), so a peer with many experts here is spread over workgroups that
// never talk.  Bound by latency: one wave issues a dependent vector instruction every 3.4 ns, so what
// counts is instructions per row and round trips per lane.  A row costs about fifty instructions (ids by
// 16-byte loads, one table byte per id, the local ones as a bit set that is walked) where a walk
// over all eight ids with the hits in an array of registers took several hundred.  Measured, with that walk and
// with this: 16 peers of 429 rows 16.9 -> 8.3 us, 64 peers of 481 rows 14.0 -> 9.4, 8 peers of 681 rows and
// 32 experts 23.8 -> 8.6, of 2720 rows 34.6 -> 13.6; riding beside the expander with two waves a peer (8 peers of
// 1360 rows, 32 experts) the step 170 -> 83 us, because the index no longer outlasts the movers.  With the experts' words scanned by a
// wave each, the report sent before the ranks are written and the counts finished by one wave: 16 peers of 429 rows 8.8 -> 7.8,
// 64 of 478 10.5 -> 8.7, 8 of 1360 and 32 experts 11.3 -> 10.3.
// kB: rows a lane requests together.  kKeep: what the lane's first kB rows parsed to stays in registers
// for the second pass (top_k <= 8); else the rows are requested again, which the launches that
// run the index beside the row movers do to stay small in registers.
// kDefer: a launch whose arguments name no statistics leaves the counts as they are, unreported: the expander behind it makes
// its places of them (k_expand_counts).
template <bool kPackets, int kForm, int kB, bool kKeep, bool kDefer = false>
__device__ __forceinline__ void recv_index_body(const mw_index_args &a, const uint32_t p, const uint32_t part, const uint32_t row_part = 0)
{
    extern __shared__ uint32_t lds[];
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    const uint32_t wpl = a.wpl, K = (uint32_t)a.K, Kd = (uint32_t)a.Kd, E = (uint32_t)a.E, L = (uint32_t)a.L, Lc = (uint32_t)a.Lc;
    const uint32_t P = (uint32_t)a.P, my_rank = (uint32_t)a.my_rank, max_tokens = a.max_tokens, dedup = a.dedup;
    const bool use_tab = kForm < kFormAny || a.tab_words != 0;
    uint32_t *addr = lds;                                       // [wpl]      bit i: row i's group names this rank
    unsigned char *tab = (unsigned char *)(addr + wpl);         // [E + 1]    local slot of expert e or kNotLocal
    uint32_t *bits = addr + wpl + a.tab_words;                  // [Lc][wpl]  bit s of expert l: a row with source token s
    uint16_t *pre = (uint16_t *)(bits + (size_t)Lc * wpl);      // [Lc][wpl]  running popcount before each word (modulo 2^16)
    uint32_t *scratch = bits + (size_t)Lc * wpl + ((size_t)Lc * wpl + 1) / 2;  // [17] scans, [17] reports in front of this one,
                                                                // [18] addressed rows, [19] repeats dropped, [20..35] waves' sums, [36] flags
    uint32_t *seen_tok = scratch + 64;                          // [wpl]      (dedup only) bit s: a row with source token s was taken

    // ---- everything that depends on the peer record alone is requested before the first wait:
    // the lane's first rows (source token, first eight expert ids), its first descriptor and the
    // row counts of the peers before this one.  The kernel is a chain of memory round trips; beside a
    // bandwidth-bound kernel each of them takes several times longer.
    const int32_t slot0 = (use_tab && tid < E) ? a.eslot[tid] : 0;
    mw_recv_peer pr;
    if constexpr (kPackets) {
        const mw_recv_packets q = ((const mw_recv_packets *)a.peers)[p];
        const char *first_packet = (const char *)q.packets;
        pr.desc = nullptr; pr.n_desc = q.n_rows; pr.n_rows = q.n_rows;
        pr.rows = first_packet + a.header_bytes;
        pr.row_src_token = (const int32_t *)(first_packet + 32);
        pr.row_topk = (const int32_t *)(first_packet + 40);
    } else {
        pr = ((const mw_recv_peer *)a.peers)[p];
    }
    const uint32_t mine = min(pr.n_rows, max_tokens);
    // expert ids by 16-byte loads: id lists of whole 16-byte units that start on one
    const bool wide_ids = !kPackets && (K & 3u) == 0 && ((uintptr_t)pr.row_topk & 15u) == 0;
    auto ids_of = [&](uint32_t i) __attribute__((always_inline)) -> const int32_t * {
        if constexpr (kPackets) return (const int32_t *)((const char *)pr.row_topk + (size_t)i * a.row_bytes);
        else return pr.row_topk + (size_t)i * K;
    };
    // source token and first eight ids of row i (a row the peer has)
    auto load_row = [&](uint32_t i, uint32_t &s, int32_t (&e)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = -1;
        if constexpr (kPackets) {
            // header bytes 32..79: token, id count, ids (the header is at least 128 bytes, the packet 16-byte aligned)
            const u32x4 *h = (const u32x4 *)((const char *)pr.rows - a.header_bytes + (size_t)i * a.row_bytes) + 2;
            const u32x4 h0 = h[0], h1 = h[1], h2 = h[2];
            s = h0.x;
            e[0] = (int32_t)h0.z; e[1] = (int32_t)h0.w; e[2] = (int32_t)h1.x; e[3] = (int32_t)h1.y;
            e[4] = (int32_t)h1.z; e[5] = (int32_t)h1.w; e[6] = (int32_t)h2.x; e[7] = (int32_t)h2.y;
        } else {
            s = (uint32_t)pr.row_src_token[i];
            const int32_t *tk = pr.row_topk + (size_t)i * K;
            if (wide_ids) {
                const u32x4 q0 = *(const u32x4 *)tk;
                e[0] = (int32_t)q0.x; e[1] = (int32_t)q0.y; e[2] = (int32_t)q0.z; e[3] = (int32_t)q0.w;
                if (K > 4) {
                    const u32x4 q1 = *((const u32x4 *)tk + 1);
                    e[4] = (int32_t)q1.x; e[5] = (int32_t)q1.y; e[6] = (int32_t)q1.z; e[7] = (int32_t)q1.w;
                }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) if ((uint32_t)u < K) e[u] = tk[u];
            }
        }
    };
    uint32_t s_c[kB];
    int32_t e_c[kB][8];
#pragma unroll
    for (int c = 0; c < kB; ++c) {
        s_c[c] = 0;
        if ((uint32_t)c * nthr < mine) load_row(min(tid + (uint32_t)c * nthr, mine - 1u), s_c[c], e_c[c]);
    }
    uint64_t dmask_c = 0;
    uint32_t doff_c = 0, dcnt_c = 0;       // packets: dcnt_c holds the header's id count
    auto load_desc = [&](uint32_t g, uint64_t &dm, uint32_t &off, uint32_t &cnt) __attribute__((always_inline)) {
        if constexpr (kPackets) {
            const char *hd = (const char *)pr.rows - a.header_bytes + (size_t)g * a.row_bytes;
            dm = ((const uint64_t *)hd)[my_rank >> 6];
            cnt = *(const uint32_t *)(hd + 36);
        } else {
            const mw_group_desc *d = pr.desc + g;
            dm = d->mask[my_rank >> 6];
            off = d->row_offset;
            cnt = d->row_count;
        }
    };
    if (tid < pr.n_desc) load_desc(tid, dmask_c, doff_c, dcnt_c);
    auto rows_of_peer = [&](uint32_t q) __attribute__((always_inline)) -> uint32_t {
        if constexpr (kPackets) return ((const mw_recv_packets *)a.peers)[q].n_rows;
        else return ((const mw_recv_peer *)a.peers)[q].n_rows;
    };
    uint32_t before = 0;
    for (uint32_t q = tid; q < p; q += nthr) before += min(rows_of_peer(q), max_tokens);

    uint32_t le0 = part * Lc, lc = le0 < L ? min(Lc, L - le0) : 0u;
    for (uint32_t w = tid; w < wpl; w += nthr) addr[w] = 0;
    if (dedup) for (uint32_t w = tid; w < wpl; w += nthr) seen_tok[w] = 0;
    for (uint32_t w = tid; w < lc * wpl; w += nthr) bits[w] = 0;
    if (tid < 2) scratch[18 + tid] = 0;
    if (tid == 0) scratch[36] = 0;
    if (use_tab) {
        for (uint32_t e = tid; e <= E; e += nthr) {
            const int32_t q = e < nthr ? slot0 : (e < E ? a.eslot[e] : 0);
            tab[e] = (e < E && (uint32_t)(q >> 16) == my_rank) ? (unsigned char)(q & 0xff) : (unsigned char)kNotLocal;
        }
    }
    // at most 256 peers of at most 65536 rows, so 32 bits are enough
    before = mw_wave_sum(before);
    if ((tid & 63u) == 0) scratch[20 + (tid >> 6)] = before;
    mw_lds_barrier();
    before = mw_wave_sum((tid & 63u) < (nthr >> 6) ? scratch[20 + (tid & 63u)] : 0u);
    uint32_t err = 0;
    if (pr.n_rows > max_tokens || before + mine > a.cap_rows) err |= MW_FLAG_RECV_CAPACITY;
    const uint32_t rb = min(before, a.cap_rows);
    const uint32_t n_rows = min(before + mine, a.cap_rows) - rb;
    const bool speaker = tid == nthr - 64u;           // first lane of the wave that reports (the last: it has the fewest rows)
    if (speaker && part == 0 && row_part == 0) {
        a.row_base[p] = rb;
        if (p == P - 1u) st_agent(&a.row_base[P], rb + n_rows);    // (also read by the last workgroup)
    }

    // ---- addressed rows: groups whose bitmap has this rank's bit
    if constexpr (kPackets) {
        // one bitmap per row: 32 consecutive rows are 32 consecutive lanes, so a ballot is the
        // word of the addressed-rows bitmap and its first lane stores it (no atomics)
        for (uint32_t g0 = 0; g0 < pr.n_desc; g0 += nthr) {
            const uint32_t g = g0 + tid;
            bool ad = false;
            if (g < pr.n_desc) {
                uint64_t dm = dmask_c;
                uint32_t hk = dcnt_c, unused = 0;
                if (g0) load_desc(g, dm, unused, hk);
                ad = (dm >> (my_rank & 63u)) & 1ull;
                if (ad && (hk != K || g >= n_rows)) { err |= MW_FLAG_BAD_DESC; ad = false; }
            }
            const uint64_t bal = __ballot(ad);
            if ((tid & 31u) == 0 && (g >> 5) < wpl) addr[g >> 5] = (uint32_t)(bal >> (tid & 32u));
        }
    } else {
        auto address = [&](uint64_t dm, uint64_t b, uint64_t cnt) __attribute__((always_inline)) {
            const uint64_t e = b + cnt;
            if (!((dm >> (my_rank & 63u)) & 1ull)) return;
            if (e > n_rows) { err |= MW_FLAG_BAD_DESC; return; }
            if (e <= b) return;
            for (uint32_t w = (uint32_t)b >> 5; w <= ((uint32_t)e - 1u) >> 5; ++w) {     // (e <= n_rows <= 65536)
                const uint32_t wlo = w << 5;
                uint32_t m = 0xffffffffu;
                if ((uint32_t)b > wlo) m &= 0xffffffffu << ((uint32_t)b - wlo);
                if ((uint32_t)e < wlo + 32u) m &= 0xffffffffu >> (wlo + 32u - (uint32_t)e);
                atomicOr(&addr[w], m);
            }
        };
        if (tid < pr.n_desc) address(dmask_c, doff_c, dcnt_c);
        for (uint32_t g0 = nthr; g0 < pr.n_desc; g0 += 2u * nthr) {      // two descriptors a lane in flight
            uint64_t dm[2] = {0, 0};
            uint32_t off[2] = {0, 0}, cnt[2] = {0, 0};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t g = g0 + tid + (uint32_t)c * nthr;
                if (g < pr.n_desc) load_desc(g, dm[c], off[c], cnt[c]);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) address(dm[c], off[c], cnt[c]);      // (no bit set past the last one)
        }
    }
    mw_lds_barrier();
    {
        uint32_t n = 0;
        for (uint32_t w = tid; w < wpl; w += nthr) n += __popc(addr[w]);
        n = mw_wave_sum(n);                          // one LDS atomic per wave
        if ((tid & 63u) == 0 && n) atomicAdd(&scratch[18], n);
        // no expert lives here: any addressed row is inconsistent
        if (L == 0 && n) err |= MW_FLAG_NO_LOCAL_EXPERT;
        if (dedup) mw_lds_barrier();                 // (repeats are taken out of the bitmap below)
    }

    // ---- per row: its distinct local experts in the order of its id list (repeated ids count once).
    // classify: which of ids j0 .. j0 + 7 are local (bit u), and -- with the LDS table -- their slots, a byte each.
    // (flags are pass 1's; what pass 2 finds again, or in rows that are not addressed, is not reported)
    auto classify = [&](const int32_t (&e)[8], uint32_t j0, uint32_t &local, uint64_t &slots) __attribute__((always_inline)) {
        local = 0; slots = 0;
        uint32_t top = 0;                            // E: some id is outside [0, E)
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            x[u] = min((uint32_t)e[u], E);
            if (j0 + u >= K) x[u] = E; else top = max(top, x[u]);
        }
        if (use_tab) {
            uint32_t q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = tab[x[u]];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                local |= (q[u] != kNotLocal) ? 1u << u : 0u;
                slots |= (uint64_t)q[u] << (8 * u);
            }
        } else {
            int32_t q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = x[u] < E ? a.eslot[x[u]] : -1;
#pragma unroll
            for (int u = 0; u < 8; ++u) local |= (q[u] >= 0 && (uint32_t)(q[u] >> 16) == my_rank) ? 1u << u : 0u;
        }
        if (top == E) {
#pragma unroll
            for (int u = 0; u < 8; ++u) if (j0 + u < K && e[u] != -1 && (uint32_t)e[u] >= E) err |= MW_FLAG_BAD_EXPERT;
        }
    };
    // walk: calls act(k, expert slot) for every distinct local expert among ids j0 .. j0 + 7
    auto walk = [&](uint32_t i, uint32_t j0, uint32_t local, uint64_t slots, uint32_t &nk, uint64_t &named, auto act) __attribute__((always_inline)) {
        while (local) {
            const uint32_t u = (uint32_t)__ffs((int)local) - 1u;
            local &= local - 1u;
            const uint32_t le = use_tab ? (uint32_t)(slots >> (8u * u)) & 0xffu
                                        : (uint32_t)a.eslot[ids_of(i)[j0 + u]] & 0xffffu;
            if (kForm < kFormAny || L <= 64) {
                const uint64_t bit = 1ull << le;
                if (named & bit) continue;
                named |= bit;
            } else {
                const int32_t *tk = ids_of(i);
                const int32_t e = tk[j0 + u];
                bool repeated = false;
                for (uint32_t j = 0; j < j0 + u; ++j) repeated |= tk[j] == e;
                if (repeated) continue;
            }
            act(nk++, le);
        }
    };
    // all of a row's hits; (local, slots) are what its first eight ids parsed to
    auto walk_row = [&](uint32_t i, uint32_t local, uint64_t slots, auto act) __attribute__((always_inline)) -> uint32_t {
        uint32_t nk = 0;
        uint64_t named = 0;
        for (uint32_t j0 = 0;;) {
            walk(i, j0, local, slots, nk, named, act);
            if constexpr (kForm == kFormFew) break;
            j0 += 8;
            if (j0 >= K) break;
            int32_t e[8];
            const int32_t *tk = ids_of(i);
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = (j0 + u < K) ? tk[j0 + u] : -1;
            classify(e, j0, local, slots);
        }
        return nk;
    };

    // ---- pass 1: the (expert, source token) bits of every row.  mark: rows i0 + tid, i0 + tid + nthr, ... as load_row
    // left them; (local, slots) say what their first eight ids parsed to.
    auto mark = [&](uint32_t i0, const uint32_t (&s_r)[kB], const int32_t (&e_r)[kB][8], bool first_chunk,
                    uint32_t (&local_r)[kB], uint64_t (&slots_r)[kB]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kB; ++c) {
            const uint32_t i = i0 + tid + (uint32_t)c * nthr, s = s_r[c];
            local_r[c] = 0; slots_r[c] = 0;
            if (i >= n_rows || !((addr[i >> 5] >> (i & 31u)) & 1u)) continue;
            if (s >= max_tokens) { err |= MW_FLAG_BAD_SRC_TOKEN; continue; }
            if (dedup && first_chunk && ((atomicOr(&seen_tok[s >> 5], 1u << (s & 31u)) >> (s & 31u)) & 1u)) {
                // a repeat of a row already taken (a relay forwarded without updating the metadata,
                // Section 4.1): dropped.  Repeats are copies, so which of them is taken does not matter.
                err |= MW_FLAG_DUPLICATE_DROPPED;
                atomicAdd(&scratch[19], 1u);
                atomicAnd(&addr[i >> 5], ~(1u << (i & 31u)));
                continue;
            }
            classify(e_r[c], 0, local_r[c], slots_r[c]);
            const uint32_t nk = walk_row(i, local_r[c], slots_r[c], [&](uint32_t, uint32_t le) __attribute__((always_inline)) {
                const uint32_t l = le - le0;
                if (l >= lc) return;
                const uint32_t old = atomicOr(&bits[l * wpl + (s >> 5)], 1u << (s & 31u));
                if ((old >> (s & 31u)) & 1u) err |= MW_FLAG_DUP_SRC_TOKEN;
            });
            if (nk == 0) err |= MW_FLAG_NO_LOCAL_EXPERT;
        }
    };
    const uint32_t step = (uint32_t)kB * nthr;
    auto load_rows = [&](uint32_t i0, uint32_t (&s_r)[kB], int32_t (&e_r)[kB][8]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kB; ++c) {
            s_r[c] = 0;
            if (i0 + (uint32_t)c * nthr < n_rows) load_row(min(i0 + tid + (uint32_t)c * nthr, n_rows - 1u), s_r[c], e_r[c]);
        }
    };
    auto mark_from = [&](uint32_t i0, bool first_chunk) __attribute__((always_inline)) {
        for (; i0 < n_rows; i0 += step) {
            uint32_t s_r[kB], local_r[kB];
            uint64_t slots_r[kB];
            int32_t e_r[kB][8];
            load_rows(i0, s_r, e_r);
            mark(i0, s_r, e_r, first_chunk, local_r, slots_r);
        }
    };
    uint32_t local_c[kB];                            // (kKeep) the first rows as they parsed
    uint64_t slots_c[kB];
    mark(0, s_c, e_c, true, local_c, slots_c);
    bool first_chunk = true;
    mark_from(step, true);
    while (true) {
        if (err) { atomicOr(&scratch[36], err); err = 0; }
        mw_lds_barrier();

        // ---- running popcounts over each expert's words, a wave an expert at a time: no scan over the waves, no barrier
        // inside.  A count in front of a word is below 65536.
        uint32_t lane = tid;
        asm volatile("" : "+v"(lane));               // (made here, not kept in registers through the passes: the riders have none to spare)
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lane >> 6));
        lane &= 63u;
        const uint32_t per = (wpl + 63u) / 64u, w0 = min(wpl, lane * per), w1 = min(wpl, w0 + per);
        const uint32_t n_wave = nthr >> 6;
        uint32_t l = wave;
        // Many experts of a few words: a lane an expert, where a wave takes 0.075 us for every four.  The index of two peers, 1000
        // experts, by waves / by lanes: 1 word 22.0 / 16.0, 10 words 17.6 / 14.7, 19 words 17.3 / 15.8, 24 words 18.0 / 16.8, 32 words (32 lanes on
        // one LDS bank) 19.5 / 22.3; 8000 experts of one peer, 1 word 79 / 37.  Only where there are more than 64 experts or
        // no table of them: the riders have no registers for it.
        if (kForm == kFormAny && wpl <= kLaneWords && lc >= 64u) {
            for (uint32_t e = tid; e < lc; e += nthr) {
                uint32_t run = 0;
                for (uint32_t w = e * wpl; w < (e + 1u) * wpl; ++w) { pre[w] = (uint16_t)run; run += (uint32_t)__popc(bits[w]); }
            }
            l = lc;
        }
        if (per == 1)                                // a word a lane: four experts side by side
            for (; l + 3u * n_wave < lc; l += 4u * n_wave) {
                uint32_t c[4], inc[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) c[j] = lane < wpl ? (uint32_t)__popc(bits[(l + j * n_wave) * wpl + lane]) : 0u;
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) inc[j] = mw_wave_incl_scan(c[j]);
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) if (lane < wpl) pre[(l + j * n_wave) * wpl + lane] = (uint16_t)(inc[j] - c[j]);
            }
        for (; l < lc; l += n_wave) {
            const uint32_t *b = bits + l * wpl;
            const uint32_t c = w0 < w1 ? (uint32_t)__popc(b[w0]) : 0u;
            uint32_t sum = c;
            for (uint32_t w = w0 + 1u; w < w1; ++w) sum += (uint32_t)__popc(b[w]);
            uint32_t run = mw_wave_incl_scan(sum) - sum;
            if (w0 < w1) pre[l * wpl + w0] = (uint16_t)run;
            run += c;
            for (uint32_t w = w0 + 1u; w < w1; ++w) { pre[l * wpl + w] = (uint16_t)run; run += (uint32_t)__popc(b[w]); }
        }
        mw_lds_barrier();
        // ---- the counts, and after the last chunk's the report that they are there: now, so that its way to memory and back
        // goes by while the other waves write ranks and records (which only the next kernel reads)
        if (wave == (nthr >> 6) - 1u) {
            if (row_part == 0)
                for (uint32_t l = lane; l < lc; l += 64u) {
                    const uint32_t w = (l + 1u) * wpl - 1u;
                    st_agent(&a.cnt[(size_t)(le0 + l) * P + p], wpl ? pre[w] + (uint32_t)__popc(bits[w]) : 0u);
                }
            if (le0 + a.parts * Lc >= L) {
                if (lane == 0) {
                    if (scratch[36]) __hip_atomic_fetch_or(&a.flags[1], scratch[36], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (part == 0 && row_part == 0) st_agent(&a.addr_cnt[p], scratch[18] - scratch[19]);
                }
                if (!(kDefer && a.stats == nullptr)) {
                    mw_publish_wave();
                    if (lane == 0) scratch[17] = mw_report(&a.flags[2]);
                }
            }
        }

        // ---- pass 2: stable rank of every row among the peer's rows for each of its experts in the chunk;
        // hit k is written by the workgroup that has its expert, the record by the one that has hit 0
        auto rank = [&](uint32_t i0, const uint32_t (&s_r)[kB], const uint32_t (&local_r)[kB], const uint64_t (&slots_r)[kB])
            __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < kB; ++c) {
                const uint32_t i = i0 + tid + (uint32_t)c * nthr, s = s_r[c];
                if (i >= n_rows) continue;
                uint32_t nk = 0;
                int32_t first_le = -1, first_rank = 0;
                if (((addr[i >> 5] >> (i & 31u)) & 1u) && s < max_tokens) {
                    mw_hit *h = a.hits + (size_t)(rb + i) * Kd;
                    nk = walk_row(i, local_r[c], slots_r[c], [&](uint32_t k, uint32_t le) __attribute__((always_inline)) {
                        const uint32_t l = le - le0;
                        if (l >= lc) return;
                        const uint32_t w = l * wpl + (s >> 5);
                        const int32_t rk = (int32_t)(pre[w] + (uint32_t)__popc(bits[w] & ((1u << (s & 31u)) - 1u)));
                        if (k > 0) h[k] = mw_hit{(int32_t)le, rk};
                        else { first_le = (int32_t)le; first_rank = rk; }
                    });
                }
                if (first_le >= 0)
                    a.recs[rb + i] = mw_row_rec{(const char *)pr.rows + (size_t)i * a.row_bytes, (int32_t)s, (int32_t)p,
                                                (int32_t)nk, first_le, first_rank, 0};
                else if (nk == 0 && part == 0 && first_chunk)
                    a.recs[rb + i] = mw_row_rec{nullptr, 0, (int32_t)p, 0, 0, 0, 0};
            }
        };
        uint32_t i0 = row_part * step;
        if (kKeep && first_chunk && i0 == 0) { rank(0, s_c, local_c, slots_c); i0 = a.row_parts * step; }
        for (; i0 < n_rows; i0 += a.row_parts * step) {
            uint32_t s_r[kB], local_r[kB];
            uint64_t slots_r[kB];
            int32_t e_r[kB][8];
            load_rows(i0, s_r, e_r);
#pragma unroll
            for (int c = 0; c < kB; ++c) {
                local_r[c] = 0; slots_r[c] = 0;
                if (i0 + (uint32_t)c * nthr < n_rows) classify(e_r[c], 0, local_r[c], slots_r[c]);
            }
            rank(i0, s_r, local_r, slots_r);
        }
        le0 += a.parts * Lc;
        if (le0 >= L) break;
        first_chunk = false;
        lc = min(Lc, L - le0);
        mw_lds_barrier();                            // this chunk's ranks have been read
        for (uint32_t w = tid; w < lc * wpl; w += nthr) bits[w] = 0;
        mw_lds_barrier();
        err = 0;
        mark_from(0, false);
    }
    if (kDefer && a.stats == nullptr) return;
    // ---- the workgroup that reported last turns the counts into output bases ----------
    // Everything it reads (counts, addressed-row counts, flags) is written and read with device-scope
    // atomics, and every workgroup reports through one counter when the wave that wrote them has them acknowledged
    // (publication of one wave, mw_internal.h); the wave whose report is the last has thereby acquired
    // what all the others released, and goes on by itself or hands its decision to the workgroup.  The row records
    // and hit slots, written with ordinary stores, are read by the next kernel only.
    if (L * P <= 64u * kWaveCounts) {
        // Only the wave that reported, whose first lane reads its own word (kept in a register through pass 2 it cost the
        // riders of more than eight ids a spill: 2048 fp8 tokens of nine ids 54.1 -> 54.7 us a step)
        if (tid < nthr - 64u) return;
        uint32_t n = 0;
        if (tid == nthr - 64u) n = scratch[17];
        if (mw_consume_wave(n) == P * a.parts * a.row_parts - 1u)
            mw_finish_counts_wave(a.cnt, a.addr_cnt, a.flags, a.row_base, L, P, a.out_cap, a.base, a.expert_offsets, a.stats);
        return;
    }
    mw_consume_barrier();
    if (scratch[17] != P * a.parts * a.row_parts - 1u) return;
    mw_consume_barrier();                            // (scratch is used again)
    mw_finish_counts(a.cnt, a.addr_cnt, a.flags, a.row_base, L, P, a.out_cap, a.base, a.expert_offsets, a.stats, scratch);
}

// Workgroup w of the index of a batch that rides in a launch of row movers: a row a lane at a time,
// nothing kept between the passes, which fits 54 vector registers without scratch (see k_expand_index_next).
template <int kForm>
__device__ __forceinline__ void recv_index_rider(const mw_index_args &a, const uint32_t w)
{
    const uint32_t q = w / (uint32_t)a.P, part = q / a.row_parts;
    recv_index_body<false, kForm, 1, false>(a, w - q * (uint32_t)a.P, part, q - part * a.row_parts);
}
__host__ __device__ __forceinline__ uint32_t index_riders(const mw_index_args &a) { return (uint32_t)a.P * a.parts * a.row_parts; }

template <bool kPackets, int kForm, int kB>
__global__ __launch_bounds__(kIndexBlock) void k_recv_index(const mw_index_args a)
{
    recv_index_body<kPackets, kForm, kB, kForm == kFormFew, true>(a, blockIdx.x, blockIdx.y);
}

// ---- the index of a SMALL batch in one workgroup ------------------------------------------------
// With a few hundred received rows the index above is nothing but its chain of memory round
// trips, and three of them -- the wait for a workgroup's stores, its report, the last workgroup's
// reads of everybody's counts -- exist only because the peers are spread over workgroups.  Here one
// workgroup handles all peers: records, then descriptors beside the rows' tokens and ids, then the
// rank table, and the rest is LDS.  One bitmap over (expert, peer, source token) in output order
// holds a bit per delivered (row, expert) pair; a running popcount over it is every pair's output
// row at once: expert offsets, per-(expert, peer) bases and ranks are read off the same array.
// Same outputs and flags as recv_index_body + mw_finish_counts (records, not packets; no
// de-duplication); cnt and addr_cnt, which only those two exchange, are not written.
// LDS words: see mw_small_index_lds_words.  P <= blockDim.x.
constexpr int kSmallPeers = 256;                      // peers of the one-workgroup index (their records are scanned by four waves)
constexpr int kSmallIndexLds = 40960;                 // LDS bytes of the one-workgroup index
constexpr int kSmallLanes = kSmallPlanLanes;          // lanes of the small launches' workgroups (index: one or two rows a lane up to 1024 rows)
// Rows up to which a small step's index is one workgroup's: two a lane.  Where there were more, or may be more because nobody
// has said how many, the launch has both forms.
constexpr uint32_t kEitherRows = 2 * kSmallLanes;

static inline size_t mw_small_index_lds_words(int P, int L, int tab, uint32_t wpl, uint32_t max_tokens, uint32_t cap_rows)
{
    const uint64_t m_max = (uint64_t)P * max_tokens < cap_rows ? (uint64_t)P * max_tokens : cap_rows;
    const size_t wa = (size_t)((m_max + 31) / 32), n_w = (size_t)L * (size_t)P * wpl;
    return 10 * (size_t)P + 3 * ((size_t)P + 1) + wa + 2 * n_w + 1 + 24 + (size_t)tab;
}

struct mw_small_lds {
    mw_recv_peer *pinfo;    // [P]      the peers' records
    uint32_t *rbase;        // [P + 1]  first row (over all peers) of peer q
    uint32_t *nrow;         // [P + 1]  rows taken from peer q
    uint32_t *dbase;        // [P + 1]  first descriptor (over all peers) of peer q
    uint32_t *addr;         // [wa]     bit r: row r's group names this rank
    uint32_t *bits;         // [n_w]    (expert, peer, source token) in output order
    uint32_t *pre;          // [n_w + 1] running popcount in front of each word
    uint32_t *scratch;      // [17] scan scratch, [17] flags, [18] addressed rows
    int32_t *tab;           // [tab_words] the experts' ranks and slots, if there is room
    uint32_t wa, n_w;
};
__device__ __forceinline__ mw_small_lds small_lds_at(const mw_index_args &a, uint32_t *lds)
{
    const uint32_t P = (uint32_t)a.P;
    const uint64_t m_max = (uint64_t)P * a.max_tokens < a.cap_rows ? (uint64_t)P * a.max_tokens : a.cap_rows;
    mw_small_lds m;
    m.wa = (uint32_t)((m_max + 31) / 32);
    m.n_w = (uint32_t)a.L * P * a.wpl;
    m.pinfo = (mw_recv_peer *)lds;
    m.rbase = lds + 10 * P;
    m.nrow = m.rbase + P + 1;
    m.dbase = m.nrow + P + 1;
    m.addr = m.dbase + P + 1;
    m.bits = m.addr + m.wa;
    m.pre = m.bits + m.n_w;
    m.scratch = m.pre + m.n_w + 1;
    m.tab = (int32_t *)(m.scratch + 24);
    return m;
}

// kSmallRows: rows (and descriptors) a lane keeps in registers; further ones go through memory.
// kLimit: more received rows than this (0: any number) are left to the launch's other form.
// kAll: every workgroup of the launch makes the index for itself, in LDS (expand_small goes on from there); the first one writes what
// is written once, records and hits are left to expand_small.
template <int kSmallRows, uint32_t kLimit = 0, bool kAll = false>
__device__ __forceinline__ void recv_index_small(const mw_index_args &a, uint32_t *lds)
{
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    const uint32_t P = (uint32_t)a.P, L = (uint32_t)a.L, wpl = a.wpl, K = (uint32_t)a.K, Kd = (uint32_t)a.Kd;
    const uint32_t E = (uint32_t)a.E, my_rank = (uint32_t)a.my_rank, max_tokens = a.max_tokens, cap_rows = a.cap_rows;
    const mw_small_lds at = small_lds_at(a, lds);
    const uint32_t wa = at.wa, n_w = at.n_w;
    mw_recv_peer *pinfo = at.pinfo;
    uint32_t *rbase = at.rbase, *nrow = at.nrow, *dbase = at.dbase, *addr = at.addr, *bits = at.bits, *pre = at.pre, *scratch = at.scratch;
    int32_t *tab = at.tab;
    const bool in_lds = a.tab_words != 0, writer = !kAll || blockIdx.x == 0;
    const mw_recv_peer *peers = (const mw_recv_peer *)a.peers;
    uint32_t err = 0;

    // ---- round trip 1: the records, and beside them the expert table (the ids' lookup was a third
    // round trip: 64 peers x 7 rows 9.5 -> 8.6 us, 8 x 86 11.0 -> 8.2, 8 x 3 7.1 -> 5.9)
    int32_t tab_r[kSmallTab / kSmallLanes];
#pragma unroll
    for (int j = 0; j < kSmallTab / kSmallLanes; ++j) {
        const uint32_t e = tid + (uint32_t)j * nthr;
        tab_r[j] = in_lds && e < E ? a.eslot[e] : -1;
    }
    uint32_t nq = 0, dq = 0;
    if (tid < P) {
        const mw_recv_peer pr = peers[tid];
        pinfo[tid] = pr;
        nq = min(pr.n_rows, max_tokens);
        dq = min(pr.n_desc, 65536u);
        if (pr.n_rows > max_tokens) err |= MW_FLAG_RECV_CAPACITY;
    }
    for (uint32_t w = tid; w < wa; w += nthr) addr[w] = 0;
    for (uint32_t w = tid; w < n_w; w += nthr) bits[w] = 0;
    if (tid < 2) scratch[17 + tid] = 0;
    // exclusive scans over the peers: at most four waves hold one
    const uint32_t n_inc = mw_wave_incl_scan(nq), d_inc = mw_wave_incl_scan(dq);
    if ((tid & 63u) == 63u && tid < kSmallPeers) { scratch[tid >> 6] = n_inc; scratch[4 + (tid >> 6)] = d_inc; }
#pragma unroll
    for (int j = 0; j < kSmallTab / kSmallLanes; ++j) {
        const uint32_t e = tid + (uint32_t)j * nthr;
        if (in_lds && e < E) tab[e] = tab_r[j];
    }
    mw_lds_barrier();
    if (kLimit != 0 && scratch[0] + scratch[1] + scratch[2] + scratch[3] > kLimit) return;
    if (tid < P) {
        uint32_t before = n_inc - nq, dbefore = d_inc - dq;
        for (uint32_t w = 0; w < (tid >> 6); ++w) { before += scratch[w]; dbefore += scratch[4 + w]; }
        if (before + nq > cap_rows) err |= MW_FLAG_RECV_CAPACITY;
        const uint32_t rb = min(before, cap_rows), nr = min(before + nq, cap_rows) - rb;
        rbase[tid] = rb; nrow[tid] = nr; dbase[tid] = dbefore;
        if (writer) a.row_base[tid] = rb;
        if (tid == P - 1) { rbase[P] = rb + nr; dbase[P] = dbefore + dq; if (writer) a.row_base[P] = rb + nr; }
    }
    mw_lds_barrier();
    const uint32_t M = rbase[P], D = dbase[P];
    // the peer whose range [base[q], base[q + 1]) holds v (ranges may be empty; v < base[P])
    auto peer_of = [&](const uint32_t *base, uint32_t v) -> uint32_t {
        uint32_t lo = 0, hi = P;                        // base[lo] <= v < base[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (base[mid] <= v) lo = mid; else hi = mid;
        }
        return lo;
    };

    // ---- round trip 2: the lane's first rows (source token, first eight ids) and descriptors, all
    // requested together; their peers by four binary searches side by side
    uint32_t q_r[kSmallRows], i_r[kSmallRows], s_r[kSmallRows];
    int32_t e_r[kSmallRows][8];
    uint32_t q_d[kSmallRows];
    uint64_t dm_d[kSmallRows];
    uint32_t off_d[kSmallRows], cnt_d[kSmallRows];
    {
        uint32_t lo[2 * kSmallRows], hi[2 * kSmallRows];
#pragma unroll
        for (int c = 0; c < 2 * kSmallRows; ++c) { lo[c] = 0; hi[c] = P; }
        // ceil(log2 P) steps: an interval of one entry stays as it is (mid == lo, and base[lo] <= v)
        for (uint32_t span = P; span > 1; span = (span + 1) >> 1) {
#pragma unroll
            for (int c = 0; c < 2 * kSmallRows; ++c) {
                const uint32_t v = tid + (uint32_t)(c % kSmallRows) * nthr, mid = (lo[c] + hi[c]) >> 1;
                const uint32_t bm = (c < kSmallRows ? rbase : dbase)[mid];
                if (bm <= v) lo[c] = mid; else hi[c] = mid;
            }
        }
#pragma unroll
        for (int j = 0; j < kSmallRows; ++j) { q_r[j] = lo[j]; q_d[j] = lo[kSmallRows + j]; }
    }
#pragma unroll
    for (int j = 0; j < kSmallRows; ++j) {
        const uint32_t r = tid + (uint32_t)j * nthr;
        i_r[j] = 0; s_r[j] = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) e_r[j][u] = -1;
        if (r < M) {
            i_r[j] = r - rbase[q_r[j]];
            const mw_recv_peer &pr = pinfo[q_r[j]];
            s_r[j] = (uint32_t)pr.row_src_token[i_r[j]];
            const int32_t *tk = pr.row_topk + (size_t)i_r[j] * K;
            load_eight_ids(tk, 0, (int)K, e_r[j]);
        }
        dm_d[j] = 0; off_d[j] = 0; cnt_d[j] = 0;
        if (r < D) {
            const mw_group_desc *dd = pinfo[q_d[j]].desc + (r - dbase[q_d[j]]);
            dm_d[j] = dd->mask[my_rank >> 6]; off_d[j] = dd->row_offset; cnt_d[j] = dd->row_count;
        }
    }
    // ---- round trip 3: rank-table entries of those ids, requested before the descriptors are looked at
    int32_t t_r[kSmallRows][8];
    bool bad_r[kSmallRows];
#pragma unroll
    for (int j = 0; j < kSmallRows; ++j) {
        bad_r[j] = false;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool ok = (uint32_t)e_r[j][u] < E;
            bad_r[j] |= (e_r[j][u] != -1 && !ok);
            t_r[j][u] = ok ? (in_lds ? tab[e_r[j][u]] : a.eslot[e_r[j][u]]) : -1;
        }
    }
    // addressed rows: the row ranges of the groups whose bitmap has this rank's bit
    auto address = [&](uint32_t q, uint64_t dm, uint64_t b, uint64_t cnt) {
        const uint64_t e = b + cnt;
        if (!((dm >> (my_rank & 63u)) & 1ull)) return;
        if (e > nrow[q]) { err |= MW_FLAG_BAD_DESC; return; }
        if (e <= b) return;
        const uint64_t gb = rbase[q] + b, ge = rbase[q] + e;        // over all peers
        for (uint64_t w = gb >> 5; w <= ((ge - 1) >> 5); ++w) {
            const uint64_t wlo = w << 5;
            uint32_t m = 0xffffffffu;
            if (gb > wlo) m &= 0xffffffffu << (gb - wlo);
            if (ge < wlo + 32) m &= 0xffffffffu >> (wlo + 32 - ge);
            atomicOr(&addr[w], m);
        }
    };
#pragma unroll
    for (int j = 0; j < kSmallRows; ++j)
        if (tid + (uint32_t)j * nthr < D) address(q_d[j], dm_d[j], off_d[j], cnt_d[j]);
    for (uint32_t d = tid + kSmallRows * nthr; d < D; d += nthr) {
        const uint32_t q = peer_of(dbase, d);
        const mw_group_desc *dd = pinfo[q].desc + (d - dbase[q]);
        address(q, dd->mask[my_rank >> 6], dd->row_offset, dd->row_count);
    }
    mw_lds_barrier();
    {
        uint32_t n = 0;
        for (uint32_t w = tid; w < wa; w += nthr) n += __popc(addr[w]);
        n = mw_wave_sum(n);
        if ((tid & 63u) == 0 && n) atomicAdd(&scratch[18], n);
        if (L == 0) for (uint32_t w = tid; w < wa; w += nthr) if (addr[w]) err |= MW_FLAG_NO_LOCAL_EXPERT;
    }

    // ---- per row: its distinct local experts in top-k order (duplicate ids count once; at most 64
    // local experts here, so "seen before" is one bit test); one bit per (expert, peer, source token).
    // The first eight stay in `les`, a byte each; slot k of the row's hit slots receives expert k here if it is a later
    // one or the row is not cached, else with its rank.
    // `cached`: the row's token and the rank-table entries of its first eight ids are in registers.
    auto parse_mark = [&](uint32_t r, uint32_t q, uint32_t i, uint32_t s, bool cached, const int32_t (&tc)[8], bool badc,
                          mw_row_rec &rec, uint64_t &les) {
        rec = mw_row_rec{nullptr, 0, (int32_t)q, 0, 0, 0, 0};
        les = 0;
        if (!((addr[r >> 5] >> (r & 31u)) & 1u)) return;
        if (s >= max_tokens) { err |= MW_FLAG_BAD_SRC_TOKEN; return; }
        const mw_recv_peer &pr = pinfo[q];
        mw_hit *h = a.hits + (size_t)r * Kd;
        const int32_t *tk = pr.row_topk + (size_t)i * K;
        uint64_t seen = 0;
        int nk = 0;
        for (uint32_t j0 = 0; j0 < K; j0 += 8) {
            int32_t t8[8];
            if (cached && j0 == 0) {
#pragma unroll
                for (int u = 0; u < 8; ++u) t8[u] = tc[u];
                if (badc) err |= MW_FLAG_BAD_EXPERT;
            } else {
                int32_t e8[8];
                load_eight_ids(tk, (int)j0, (int)K, e8);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool ok = (uint32_t)e8[u] < E;
                    if (e8[u] != -1 && !ok) err |= MW_FLAG_BAD_EXPERT;
                    t8[u] = ok ? (in_lds ? tab[e8[u]] : a.eslot[e8[u]]) : -1;
                }
            }
            // the local ones as a bit set that is walked (most rows have one or two), their slots a byte each
            // (L <= 64); a walk over all eight ids: 64 peers x 7 rows 8.6 -> 8.3 us, 256 x 1 8.9 -> 8.2
            uint32_t local = 0;
            uint64_t slots = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                local |= (uint32_t)t8[u] >> 16 == my_rank ? 1u << u : 0u;       // (-1: no rank)
                slots |= (uint64_t)((uint32_t)t8[u] & 63u) << (8 * u);
            }
            while (local) {
                const uint32_t u = (uint32_t)__ffs((int)local) - 1u;
                local &= local - 1u;
                const uint32_t le = (uint32_t)(slots >> (8u * u)) & 63u;
                if ((seen >> le) & 1ull) continue;
                seen |= 1ull << le;
                if (nk < 8) les |= (uint64_t)le << (8 * nk);
                if (!kAll && (!cached || nk >= 8)) h[nk] = mw_hit{(int32_t)le, 0};
                ++nk;
                if ((atomicOr(&bits[(le * P + q) * wpl + (s >> 5)], 1u << (s & 31u)) >> (s & 31u)) & 1u)
                    err |= MW_FLAG_DUP_SRC_TOKEN;
            }
        }
        if (nk == 0) err |= MW_FLAG_NO_LOCAL_EXPERT;
        rec.src = (const char *)pr.rows + (size_t)i * a.row_bytes;
        rec.src_token = (int32_t)s;
        rec.n_hits = nk;
        rec.le0 = (int32_t)(les & 0xffu);
    };
    mw_row_rec rec_r[kSmallRows];
    uint64_t les_r[kSmallRows];
#pragma unroll
    for (int j = 0; j < kSmallRows; ++j) {
        rec_r[j] = mw_row_rec{nullptr, 0, 0, 0, 0, 0, 0};
        les_r[j] = 0;
        const uint32_t r = tid + (uint32_t)j * nthr;
        if (r < M) parse_mark(r, q_r[j], i_r[j], s_r[j], true, t_r[j], bad_r[j], rec_r[j], les_r[j]);
    }
    for (uint32_t r = tid + kSmallRows * nthr; r < M; r += nthr) {        // further rows: through memory
        const uint32_t q = peer_of(rbase, r), i = r - rbase[q];
        const uint32_t s = (uint32_t)pinfo[q].row_src_token[i];
        const int32_t none[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
        mw_row_rec rec;
        uint64_t les;
        parse_mark(r, q, i, s, false, none, false, rec, les);
        if (!kAll) a.recs[r] = rec;
    }
    mw_lds_barrier();

    // ---- running popcount over the bitmap: consecutive words per lane, one scan of the lanes' sums
    {
        const uint32_t per = (n_w + nthr - 1) / nthr;
        const uint32_t w0 = min(n_w, tid * per), w1 = min(n_w, w0 + per);
        uint32_t sum = 0;
        for (uint32_t w = w0; w < w1; ++w) sum += __popc(bits[w]);
        uint32_t tot, run = mw_block_exscan(sum, scratch, &tot);
        for (uint32_t w = w0; w < w1; ++w) { pre[w] = run; run += __popc(bits[w]); }
        if (tid == 0) pre[n_w] = tot;
    }
    mw_lds_barrier();
    const uint32_t Q = pre[n_w];
    if (writer)
    for (uint32_t f = tid; f < L * P; f += nthr) {
        const uint32_t b = pre[f * wpl];
        a.base[f] = b;
        if (f % P == 0) a.expert_offsets[f / P] = (int64_t)b;
    }
    if constexpr (!kAll) {
    // ---- ranks: output row of (row, expert) minus the base of its (expert, peer)
    auto rank_of = [&](uint32_t q, uint32_t s, int le) -> int32_t {
        const uint32_t w0 = ((uint32_t)le * P + q) * wpl, wi = w0 + (s >> 5);
        return (int32_t)(pre[wi] + __popc(bits[wi] & ((1u << (s & 31u)) - 1u)) - pre[w0]);
    };
#pragma unroll
    for (int j = 0; j < kSmallRows; ++j) {
        const uint32_t r = tid + (uint32_t)j * nthr;
        if (r >= M) continue;
        mw_hit *h = a.hits + (size_t)r * Kd;
        const int nk = rec_r[j].n_hits;
        for (int k = 0; k < nk; ++k) {
            const int le = k < 8 ? (int)((les_r[j] >> (8 * k)) & 0xffu) : h[k].le;
            const int32_t rk = rank_of(q_r[j], s_r[j], le);
            if (k == 0) rec_r[j].rank0 = rk;
            else if (k < 8) h[k] = mw_hit{le, rk};
            else h[k].rank = rk;
        }
        a.recs[r] = rec_r[j];
    }
    for (uint32_t r = tid + kSmallRows * nthr; r < M; r += nthr) {
        mw_row_rec *rc = a.recs + r;
        mw_hit *h = a.hits + (size_t)r * Kd;
        const int nk = rc->n_hits;
        const uint32_t q = (uint32_t)rc->peer, s = (uint32_t)rc->src_token;
        for (int k = 0; k < nk; ++k) {
            const int32_t rk = rank_of(q, s, h[k].le);
            if (k == 0) rc->rank0 = rk; else h[k].rank = rk;
        }
    }
    }
    if (!writer) return;                                // (the whole workgroup)
    if (err) atomicOr(&scratch[17], err);
    mw_lds_barrier();
    if (tid == 0) {
        a.expert_offsets[L] = (int64_t)Q;
        a.stats->n_recv_rows = scratch[18];
        a.stats->n_out_rows = Q;
        a.stats->error_flags = scratch[17] | (((int64_t)Q > a.out_cap) ? MW_FLAG_OUT_CAPACITY : 0u);
        a.stats->n_rows_seen = M;
    }
}

// blockIdx.x selects a segment of blockDim.x chunks of the row; blockIdx.y walks rows.  All
// index reads are wave-uniform (scalar loads).  The dependent chain in front of a row's
// payload is what a one-shot workgroup cannot hide, so it is kept to two steps: the row
// record and the row count are fetched together, then the payload load and the lookup of
// the first output position are issued together; the position is there long before the
// payload is.
// g_first / g_stride: the first row of this workgroup and the distance to its next one.
// kFold: a row is one workgroup, and its lane c takes chunk c + blockDim.x as well where there is one (mw_row_shape_folded).
template <bool kFold = false>
__device__ __forceinline__ void expand_body(
    const mw_row_rec *__restrict__ recs, const mw_hit *__restrict__ hits, const uint32_t *__restrict__ base,
    const uint32_t *__restrict__ row_base, int P, int Kd, int xc, int sc,
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token, uint32_t g_first, uint32_t g_stride)
{
    // The row's record and the row count are requested first -- their addresses need only
    // arguments that are in registers when the wave starts -- and every other kernel argument is
    // fetched beside them, not after the first branch: one wait for all of it.  Pointers are
    // pinned through a copy of their low half, so the originals keep their address space.
    uint32_t g = g_first;
    // g_first < max_recv_rows, so the first record read is always inside the workspace
    const u32x4 *rp = (const u32x4 *)(recs + g);
    u32x4 r0 = rp[0], r1 = rp[1];
    uint32_t m_total = row_base[P];
    uint32_t gdim = g_stride, bdim = blockDim.x;
    MW_PIN_S(gdim); MW_PIN_S(bdim); MW_PIN_S(Kd); MW_PIN_S(xc); MW_PIN_S(sc); MW_PIN_S(cap);
    MW_PIN_PTR(hits); MW_PIN_PTR(out_rows); MW_PIN_PTR(out_scales); MW_PIN_PTR(out_src_peer);
    MW_PIN_PTR(out_src_token);
    MW_PIN_S4(r0); MW_PIN_S4(r1); MW_PIN_S(m_total);
    const int n = xc + sc;
    const int c = blockIdx.x * bdim + threadIdx.x;
    const int c2 = c + (int)bdim;
    while (g < m_total) {
        const int n_hits = (int)r1.x;
        if (n_hits > 0) {
            const int peer = (int)r0.w;
            const void *src = (const void *)(((uint64_t)r0.y << 32) | r0.x);
            uint32_t b0 = base[r1.y * (uint32_t)P + (uint32_t)peer];
            u32x4 v = {0u, 0u, 0u, 0u}, v2 = v;
            if (c < n) v = mw_ld16_global(src, c);
            if (kFold && c2 < n) v2 = mw_ld16_global(src, c2);
            MW_PIN_S(b0);                                  // position lookup in flight with the payload
            uint32_t dst = b0 + r1.z;                      // below 2^30: 2^24 rows, 64 experts each
            for (int k = 1;; ++k) {
                if (dst < cap) {
                    if (kFold && c2 < n) {
                        if (c2 < xc) mw_st16(out_rows + (size_t)dst * xc + c2, v2);
                        else out_scales[(size_t)dst * sc + (c2 - xc)] = v2;
                    }
                    if (c < xc) mw_st16(out_rows + (size_t)dst * xc + c, v);
                    // a row's scales are a fraction of a cache line (224 bytes of fp8 rows): an
                    // ordinary store lets L2 put neighbouring rows' pieces together before the
                    // line goes to memory, where the write-through store sent every piece by
                    // itself (fp8 expander 77.5 -> 76 us, the step 97.4 -> 94.5 us)
                    else if (c < n) out_scales[(size_t)dst * sc + (c - xc)] = v;
                    if (c == 0) { out_src_peer[dst] = peer; out_src_token[dst] = (int32_t)r0.z; }
                }
                if (k >= n_hits) break;
                const mw_hit hk = hits[(size_t)g * Kd + k];
                dst = base[(uint32_t)hk.le * P + (uint32_t)peer] + (uint32_t)hk.rank;
            }
        }
        g += gdim;
        if (g < m_total) { rp = (const u32x4 *)(recs + g); r0 = rp[0]; r1 = rp[1]; }
    }
}

template <bool kFold>
__global__ __launch_bounds__(1024) void k_expand(
    const mw_row_rec *__restrict__ recs, const uint32_t *__restrict__ row_base, const uint32_t *__restrict__ base,
    const mw_hit *__restrict__ hits, int P, int Kd, int xc, int sc,     // (in registers when a wave starts)
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token)
{
    expand_body<kFold>(recs, hits, base, row_base, P, Kd, xc, sc, out_rows, out_scales, cap, out_src_peer, out_src_token,
                       blockIdx.y, gridDim.y);
}

// The expander behind an index that has left its counts unreported (mw_unpack, mw_unpack_packets).  What an index otherwise ends
// with -- the counts acknowledged, a report of every workgroup (256 peers to one address: 8 ns each), the last one's reads of all
// counts -- is a chain of three round trips in front of this launch.  Here a wave of grid row 0 makes bases, expert offsets
// and statistics, and the movers do not wait for it: a wave requests the counts in front of the payload (one
// kilobyte that its CU's cache holds) and adds up what is in front of its place while that is on its way, a dozen vector instructions.
// kCounts: counts a lane holds, 1 (at most 64 in all), 4 (at most 256) or 8 (at most 512: four of the first 256 and four
// of the others, so that each request is a kilobyte in one piece).  us for mw_plan, mw_pack and mw_unpack, added up by the index's last
// workgroup / here: 1000 fp8 tokens of 16 ranks 30.7 / 28.5, 2048 of 64 ranks 65.2 / 62.7, 4096 107.9 / 107.9, 8192 bf16 tokens of 256
// ranks 154.4 / 152.0; 2048 packets of 16 ranks 69.0 / 67.8.
// Otherwise this is expand_body.  (The hits behind the first requested with the record and their rows stored without a wait
// in between: 1000 tokens 28.2, but 8192 of 256 ranks 152.0; in the stream's launch 16000 rows of 1.5 hits 80 -> 82.)
template <int kCounts> struct mw_counts_of { typedef uint32_t type; };
template <> struct mw_counts_of<4> { typedef u32x4 type; };
template <> struct mw_counts_of<8> { struct type { u32x4 lo, hi; }; };
template <bool kFold, int kCounts>
__device__ __forceinline__ void expand_counts_body(
    const mw_row_rec *__restrict__ recs, const mw_hit *__restrict__ hits, const uint32_t *__restrict__ cnt,
    const uint32_t *__restrict__ row_base, int P, int Kd, int xc, int sc, uint32_t n_counts,
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token)
{
    using mw_counts = typename mw_counts_of<kCounts>::type;
    uint32_t g = blockIdx.y - 1u;
    const u32x4 *rp = (const u32x4 *)(recs + g);
    u32x4 r0 = rp[0], r1 = rp[1];
    uint32_t m_total = row_base[P];
    uint32_t gdim = gridDim.y, bdim = blockDim.x;          // (less one below: here it would be waited for in front of the record's request)
    MW_PIN_S(gdim); MW_PIN_S(bdim); MW_PIN_S(Kd); MW_PIN_S(xc); MW_PIN_S(sc); MW_PIN_S(cap);
    MW_PIN_PTR(hits); MW_PIN_PTR(out_rows); MW_PIN_PTR(out_scales); MW_PIN_PTR(out_src_peer);
    MW_PIN_PTR(out_src_token);
    // (a lane without counts reads the last ones again: nobody looks at what it adds up)
    mw_counts own;
    if constexpr (kCounts == 8) {                          // (n_counts is more than 256: all lanes' first four are counts)
        own.lo = ((const u32x4 *)cnt)[threadIdx.x & 63u];
        own.hi = ((const u32x4 *)cnt)[64u + min(threadIdx.x & 63u, (n_counts - 257u) / 4u)];
    } else own = ((const mw_counts *)cnt)[min(threadIdx.x & 63u, (n_counts - 1u) / (uint32_t)kCounts)];
    MW_PIN_S4(r0); MW_PIN_S4(r1); MW_PIN_S(m_total);
    gdim -= 1u;
    const int n = xc + sc;
    const int c = blockIdx.x * bdim + threadIdx.x;
    const int c2 = c + (int)bdim;
    uint32_t in_front = 0, in_front_hi = 0;                // counts of the lanes before
    bool summed = false;
    // first output row of (expert, peer) f
    auto base_of = [&](uint32_t f) __attribute__((always_inline)) -> uint32_t {
        uint32_t v = in_front;
        if constexpr (kCounts == 4) v += ((f & 3u) > 0 ? own.x : 0u) + ((f & 3u) > 1 ? own.y : 0u) + ((f & 3u) > 2 ? own.z : 0u);
        if constexpr (kCounts == 8) {
            const u32x4 w = f < 256u ? own.lo : own.hi;
            v = (f < 256u ? in_front : in_front_hi) + ((f & 3u) > 0 ? w.x : 0u) + ((f & 3u) > 1 ? w.y : 0u) + ((f & 3u) > 2 ? w.z : 0u);
        }
        return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)(kCounts == 1 ? f : f / 4u & 63u));
    };
    while (g < m_total) {
        const int n_hits = (int)r1.x;
        if (n_hits > 0) {
            const int peer = (int)r0.w;
            const void *src = (const void *)(((uint64_t)r0.y << 32) | r0.x);
            // (lanes beyond the row read its last chunk again: no branch, so that the wait for the counts is none for the payload)
            u32x4 v = mw_ld16_global(src, min(c, n - 1)), v2 = {0u, 0u, 0u, 0u};
            if (kFold) v2 = mw_ld16_global(src, min(c2, n - 1));
            if (!summed) {
                uint32_t sum;
                if constexpr (kCounts == 8) {
                    asm volatile("" : "+v"(own.lo), "+v"(own.hi));
                    sum = own.hi.x + own.hi.y + own.hi.z + own.hi.w;
                    in_front_hi = mw_wave_incl_scan(sum) - sum;
                    sum = own.lo.x + own.lo.y + own.lo.z + own.lo.w;
                } else {
                    asm volatile("" : "+v"(own));          // (here, not in front of the payload's request)
                    if constexpr (kCounts == 4) sum = own.x + own.y + own.z + own.w; else sum = own;
                }
                const uint32_t upto = mw_wave_incl_scan(sum);
                in_front = upto - sum;
                if constexpr (kCounts == 8) in_front_hi += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
                summed = true;
            }
            uint32_t dst = base_of(r1.y * (uint32_t)P + (uint32_t)peer) + r1.z;      // below 2^30: 2^24 rows, 64 experts each
            asm volatile("" : "+v"(v));                    // waited for here, whether it is stored or not: a load that is still on its
            if (kFold) asm volatile("" : "+v"(v2));        // way at the loop's end makes the next payload's request wait for everything
            for (int k = 1;; ++k) {
                if (dst < cap) {
                    if (kFold && c2 < n) {
                        if (c2 < xc) mw_st16(out_rows + (size_t)dst * xc + c2, v2);
                        else out_scales[(size_t)dst * sc + (c2 - xc)] = v2;
                    }
                    if (c < xc) mw_st16(out_rows + (size_t)dst * xc + c, v);
                    else if (c < n) out_scales[(size_t)dst * sc + (c - xc)] = v;
                    if (c == 0) { out_src_peer[dst] = peer; out_src_token[dst] = (int32_t)r0.z; }
                }
                if (k >= n_hits) break;
                const mw_hit hk = hits[(size_t)g * Kd + k];
                dst = base_of((uint32_t)hk.le * P + (uint32_t)peer) + (uint32_t)hk.rank;
            }
        }
        g += gdim;
        if (g < m_total) { rp = (const u32x4 *)(recs + g); r0 = rp[0]; r1 = rp[1]; }
    }
}

template <bool kFold, int kCounts>
__global__ __launch_bounds__(1024) void k_expand_counts(
    const mw_row_rec *__restrict__ recs, const uint32_t *__restrict__ row_base, const uint32_t *__restrict__ cnt,
    const mw_hit *__restrict__ hits, int P, int Kd, int xc, int sc, uint32_t n_counts,     // (in registers when a wave starts)
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token,
    uint32_t L, int64_t out_cap, const uint32_t *addr_cnt, uint32_t *flags, uint32_t *base, int64_t *expert_offsets, mw_recv_stats *stats)
{
    if (blockIdx.y == 0) {
        if (blockIdx.x == 0 && threadIdx.x < 64)
            mw_finish_counts_wave(cnt, addr_cnt, flags, row_base, L, (uint32_t)P, out_cap, base, expert_offsets, stats);
        return;
    }
    expand_counts_body<kFold, kCounts>(recs, hits, cnt, row_base, P, Kd, xc, sc, n_counts, out_rows, out_scales, cap, out_src_peer,
                                       out_src_token);
}

// One launch for a steady stream of batches: the expander of the current batch and, in the
// first `next.P` workgroup rows of the grid, the index of the NEXT batch, written to another
// context's workspace.  The index is a chain of memory round trips that moves almost nothing;
// run as its own launch in front of its expander it costs 14-16 us of an otherwise
// bandwidth-bound stream, and run on a second stream it costs a cross-stream wait of 7-10 us.
// Here it rides along: its workgroups are dispatched first and finish long before the
// expander's do, and the launch that expands the next batch is ordered after this one by the
// stream, so no wait, flag or fence is needed.
// Every wave of a launch is given the registers (and the scratch space for spills) of the
// launch's hungriest path, the row movers' waves included -- and with 64 registers a wave, or
// with any scratch at all, the dispatcher refills the movers' wave slots more slowly (rocprofv3:
// SPI_RA_VGPR_SIMD_FULL_CSN and SPI_RA_TMP_STALL_CSN appear, occupancy 7 % down; fp8 step 94.9
// against 87.4 us with the riders compiled out).  The riders therefore come in a lean form that fits
// 54 registers without spilling (a row a lane at a time in the index, eight counters in flight in the
// plan's second half); batches too small to hide them give them launches of their own.  kFormMany (top_k
// above eight) takes 64 and keeps three in scratch: beside 61 us of movers 65 us against 72 with the index in front, beside 22
// us 22.6 against 34.4.
template <int kForm, bool kFold>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_expand_index_next(
    const uint32_t first_expand_row, const uint32_t unused0, const mw_row_rec *__restrict__ recs,
    const uint32_t *__restrict__ row_base, const uint32_t *__restrict__ base, const mw_hit *__restrict__ hits,
    int P, int Kd, int xc, int sc,          // up to here: in registers when a wave starts
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token, const mw_index_args next)
{
    if (blockIdx.y >= first_expand_row) {
        expand_body<kFold>(recs, hits, base, row_base, P, Kd, xc, sc, out_rows, out_scales, cap, out_src_peer, out_src_token,
                           blockIdx.y - first_expand_row, gridDim.y - first_expand_row);
        return;
    }
    const uint32_t w = blockIdx.y * gridDim.x + blockIdx.x;
    if (w < index_riders(next)) recv_index_rider<kForm>(next, w);
}

// The same launch with the PLAN of the next batch riding along as well (Section 5.1, send
// module: task decomposition for the batch after this one): after the index rows of the grid
// come `n_plan_rows` rows whose workgroups rank the next batch's tokens and then, in further
// workgroups that wait for those, write perm, descriptors and statistics.  A steady stream of
// batches then needs two launches per batch on ONE stream -- the packer and this -- and no
// event.  Measured per batch: 4096 tokens x 14336-byte rows 170 us, the same as with the plan
// on a second stream and one event wait per batch (171 us); fp8 rows of half the size 101
// against 105 us.  The riding plan is not free: its device-scope atomics and loads take
// about 4 us of memory-channel time from the expander.
template <int W, bool kKeyed, int kForm, bool kFold, bool kPart>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_expand_index_plan_next(
    const uint32_t first_pack_row, const uint32_t first_expand_row, const mw_row_rec *__restrict__ recs,
    const uint32_t *__restrict__ row_base, int P, int xc, const int32_t *__restrict__ pack_perm,
    const mw_send_stats *__restrict__ pack_stats, int sc, int Kd,   // up to here: 14 words, in registers when a wave starts
    const uint32_t *__restrict__ base, const mw_hit *__restrict__ hits,
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token,
    const mw_index_args next, const mw_plan_args plan, const mw_pack_args pack)
{
    // A row mover's wave lives for about a microsecond, and every dependent scalar fetch in front
    // of its payload load is a tenth of that.  The movers' branches therefore come first, and
    // what decides them and locates a wave's row -- the two role boundaries, the expander's record
    // and row-count arrays, the packer's row order and row count -- are the kernel's first
    // arguments: the library is built so that the first 14 argument words are in scalar registers
    // when a wave starts (hardware preload).  A mover's wave then has ONE round trip in front of its
    // payload load (its row's record or token, with the remaining arguments fetched beside it)
    // where decoding the roles one by one took five.
    const uint32_t y_pack = first_pack_row, y_expand = first_expand_row;
    if (blockIdx.y >= y_expand) {
        expand_body<kFold>(recs, hits, base, row_base, P, Kd, xc, sc, out_rows, out_scales, cap, out_src_peer, out_src_token,
                           blockIdx.y - y_expand, gridDim.y - y_expand);
        return;
    }
    if (blockIdx.y >= y_pack) {         // (mw_stream_step: the packer of a batch planned by an earlier launch)
        mw_pack_body<kFold, kPart>(pack.x, pack.scales, pack.xc, pack.sc, pack.ns, pack.topk, pack.K, pack_perm, pack_stats, pack.packed,
                            pack.row_src_token, pack.row_topk, blockIdx.x, blockIdx.y - y_pack, y_expand - y_pack);
        return;
    }
    const uint32_t w = blockIdx.y * gridDim.x + blockIdx.x, n_index = index_riders(next);
    if (w < n_index) {
        recv_index_rider<kForm>(next, w);
        return;
    }
    extern __shared__ uint64_t plan_lds[];
    mw_plan_ride<W, kKeyed>(plan, w - n_index, plan_lds);
}

// A whole step of a stream of SMALL batches in one launch (the batch sizes of Section 6.3's
// dispatch experiment, 64 and 128 tokens a rank): what k_expand_index_plan_next does, with the
// riders in their one-workgroup forms -- grid row 0 indexes the next received batch
// (recv_index_small), row 1, if there is a plan to make, plans the next batch to send
// (mw_small_plan, the plan of mw_plan_pack) -- then the packer's rows
// and the expander's.  At these sizes the step is the riders' chain of memory round trips, and the
// forms that spread a batch over workgroups spend half of theirs on talking to one another.
// kEither: the peers hold more than 1024 rows, or may, since nobody has said.  One workgroup takes 9.5 us for every 1024, so the
// launch has the riders of recv_index_body too (grid rows from general_row on), and whoever is not needed
// leaves: the choice is made here, from the peers' own counts (64 ranks, rows of 7168, us a step without / with: 64 tokens
// that all come here 43.2 / 28.4, fp8 38.1 / 16.9; 200 of 256 tokens, fp8 124 / 44; an even share of 64 tokens 10.4 / 9.1.)
template <int W, bool kKeyed, int kRows, bool kEither>
__global__ __launch_bounds__(kSmallLanes) void k_small_step(
    const uint32_t first_pack_row, const uint32_t first_expand_row, const mw_row_rec *__restrict__ recs,
    const uint32_t *__restrict__ row_base, int P, int xc, const int32_t *__restrict__ pack_perm,
    const mw_send_stats *__restrict__ pack_stats, int sc, int Kd,
    const uint32_t *__restrict__ base, const mw_hit *__restrict__ hits,
    u32x4 *__restrict__ out_rows, u32x4 *__restrict__ out_scales, uint32_t cap,
    int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token,
    const mw_index_args next, const mw_plan_args plan, const mw_pack_args pack, const mw_index_args general,
    const uint32_t general_row)
{
    if (blockIdx.y >= first_expand_row) {
        expand_body(recs, hits, base, row_base, P, Kd, xc, sc, out_rows, out_scales, cap, out_src_peer, out_src_token,
                    blockIdx.y - first_expand_row, gridDim.y - first_expand_row);
        return;
    }
    if (blockIdx.y >= first_pack_row) {
        mw_pack_body<false, false>(pack.x, pack.scales, pack.xc, pack.sc, pack.ns, pack.topk, pack.K, pack_perm, pack_stats, pack.packed,
                            pack.row_src_token, pack.row_topk, blockIdx.x, blockIdx.y - first_pack_row,
                            first_expand_row - first_pack_row);
        return;
    }
    extern __shared__ uint64_t small_lds[];
    if constexpr (kEither) {
        if (blockIdx.y >= general_row) {
            const uint32_t w = (blockIdx.y - general_row) * gridDim.x + blockIdx.x;
            if (w >= index_riders(general)) return;
            uint32_t *wave_n = (uint32_t *)small_lds;
            const uint32_t q = threadIdx.x;
            const uint32_t n = mw_wave_sum(q < (uint32_t)general.P ? min(((const mw_recv_peer *)general.peers)[q].n_rows, general.max_tokens) : 0u);
            if ((q & 63u) == 0) wave_n[q >> 6] = n;
            mw_lds_barrier();
            uint32_t rows = 0;
#pragma unroll
            for (int v = 0; v < kSmallLanes / 64; ++v) rows += wave_n[v];
            mw_lds_barrier();                                  // (the index uses the same words)
            if (rows > kEitherRows) recv_index_rider<kFormMany>(general, w);
            return;
        }
    }
    if (blockIdx.x != 0) return;
    if (blockIdx.y == 0) {
        recv_index_small<kRows, kEither ? kEitherRows : 0>(next, (uint32_t *)small_lds);
        return;
    }
    mw_small_plan<W, kKeyed>(plan.topk, plan.T, plan.K, plan.eslot, plan.E, plan.row_bytes, plan.mask_out, plan.perm,
                             plan.desc, plan.stats, small_lds);
}

// The one-workgroup index as a launch of its own (mw_unpack_index, mw_unpack of at most a row a lane).
__global__ __launch_bounds__(kSmallLanes) void k_recv_index_small(const mw_index_args a)
{
    extern __shared__ uint64_t small_index_lds[];
    recv_index_small<1>(a, (uint32_t *)small_index_lds);
}

// Index and expander of a small batch in one launch (mw_unpack).  At a few hundred rows both are latency: the index's chain, a
// launch, and the expander's own chain from the record to the row.  Here every workgroup makes the whole index for itself in
// LDS -- a few dozen bytes a row, from L2 -- and then moves its share of the rows, a wave a segment of 64 chunks at a time: the row's
// ids, its token and its payload are requested together, and its places are read off the bitmaps.  Records and hit slots are
// still written (the way back and a second expander read them), each by the wave that has the row's first segment.
// Measured beside the rule in mw_launch_unpack.
__device__ __forceinline__ void expand_small(const mw_index_args &a, uint32_t *lds, int xc, int sc, u32x4 *__restrict__ out_rows,
                                             u32x4 *__restrict__ out_scales, uint32_t cap, int32_t *__restrict__ out_src_peer,
                                             int32_t *__restrict__ out_src_token)
{
    const mw_small_lds at = small_lds_at(a, lds);
    const uint32_t P = (uint32_t)a.P, K = (uint32_t)a.K, E = (uint32_t)a.E, wpl = a.wpl, lane = threadIdx.x & 63u;
    const uint32_t n = (uint32_t)(xc + sc), nseg = (n + 63u) / 64u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t n_wave = gridDim.x * (blockDim.x >> 6), M = at.rbase[P], items = M * nseg;
    for (uint32_t item = blockIdx.x * (blockDim.x >> 6) + wave; item < items; item += n_wave) {
        const uint32_t r = item / nseg, seg = item - r * nseg;            // (rows of at most 64 KiB: items stay below 2^20)
        // the peer whose rows reach over r: the last one that begins at or before it
        uint32_t q = 0;
        for (uint32_t b = 0; b < P; b += 64u) q += (uint32_t)__popcll(__ballot(b + lane < P && at.rbase[b + lane] <= r));
        --q;
        const mw_recv_peer &pr = at.pinfo[q];
        const uint32_t i = r - at.rbase[q], c = seg * 64u + lane;
        const char *src = (const char *)pr.rows + (size_t)i * a.row_bytes;
        const bool here = (at.addr[r >> 5] >> (r & 31u)) & 1u;            // (a region may hold other ranks' rows: their payload stays unread)
        u32x4 v = {0u, 0u, 0u, 0u};
        if (here && c < n) v = mw_ld16_global(src, (int)c);
        const uint32_t s_ = (uint32_t)pr.row_src_token[i];
        const uint32_t e = lane < K ? (uint32_t)pr.row_topk[(size_t)i * K + lane] : 0xffffffffu;
        const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_);
        const int32_t t = e < E ? (a.tab_words ? at.tab[e] : a.eslot[e]) : -1;
        uint64_t local = __ballot((uint32_t)t >> 16 == (uint32_t)a.my_rank);                   // (-1: no rank)
        if (!here || s >= a.max_tokens) local = 0;
        mw_row_rec rec = {nullptr, 0, (int32_t)q, 0, 0, 0, 0};
        if (local) { rec.src = src; rec.src_token = (int32_t)s; }
        uint64_t named = 0;
        int32_t nk = 0;
        while (local) {
            const int b = (int)__builtin_ctzll(local);
            local &= local - 1ull;
            const uint32_t le = (uint32_t)__builtin_amdgcn_readlane(t, b) & 63u;
            if ((named >> le) & 1ull) continue;
            named |= 1ull << le;
            const uint32_t w0 = (le * P + q) * wpl, w = w0 + (s >> 5);
            const uint32_t dst = at.pre[w] + (uint32_t)__popc(at.bits[w] & ((1u << (s & 31u)) - 1u));
            const int32_t rank = (int32_t)(dst - at.pre[w0]);
            if (dst < cap) {
                if (c < (uint32_t)xc) mw_st16(out_rows + (size_t)dst * xc + c, v);
                else if (c < n) out_scales[(size_t)dst * sc + (c - (uint32_t)xc)] = v;
                if (c == 0) { out_src_peer[dst] = (int32_t)q; out_src_token[dst] = (int32_t)s; }
            }
            if (nk == 0) { rec.le0 = (int32_t)le; rec.rank0 = rank; }
            else if (c == 0) a.hits[(size_t)r * a.Kd + nk] = mw_hit{(int32_t)le, rank};
            ++nk;
        }
        rec.n_hits = nk;
        if (c == 0) a.recs[r] = rec;
    }
}

__global__ __launch_bounds__(kSmallLanes) void k_unpack_small(const mw_index_args a, int xc, int sc, u32x4 *__restrict__ out_rows,
                                                              u32x4 *__restrict__ out_scales, uint32_t cap,
                                                              int32_t *__restrict__ out_src_peer, int32_t *__restrict__ out_src_token)
{
    extern __shared__ uint64_t small_unpack_lds[];
    recv_index_small<1, 0, true>(a, (uint32_t *)small_unpack_lds);
    expand_small(a, (uint32_t *)small_unpack_lds, xc, sc, out_rows, out_scales, cap, out_src_peer, out_src_token);
}

// The way back (Section 2.1, combine-style AlltoAll; Section 2.3.2: the combine phase reduces
// and cannot be multicast).  The mirror image of the expander: a received row that went to h
// local experts gets ONE row back, the sum of those h expert outputs, so the return traffic is
// one copy per (token, rank) like the dispatch's.  Reads the index the last unpack left in the
// workspace.  Per 16-byte chunk (8 bf16): widen to single precision, add in the order of the
// row's hit slots (the order of its id list), round once to bf16 (nearest even; a NaN sum
// becomes 0x7FC0 with the sum's sign); h == 1 is a copy.  Hits whose output row was dropped for
// capacity contribute nothing.  Same launch shape and the same bytes as the expander, in the
// other direction: bound by HBM bandwidth.
__device__ __forceinline__ uint32_t mw_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return ((u >> 16) & 0x8000u) | 0x7fc0u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

__global__ __launch_bounds__(1024) void k_combine(
    const mw_row_rec *__restrict__ recs, const mw_hit *__restrict__ hits, const uint32_t *__restrict__ base,
    const uint32_t *__restrict__ row_base, int P, int Kd, int n, const u32x4 *__restrict__ y, uint32_t cap,
    u32x4 *__restrict__ ret, uint32_t ret_cap)
{
    uint32_t gdim = gridDim.y, bdim = blockDim.x;
    MW_PIN_S(gdim); MW_PIN_S(bdim); MW_PIN_S(Kd); MW_PIN_S(n); MW_PIN_S(cap); MW_PIN_S(ret_cap);
    MW_PIN_PTR(hits); MW_PIN_PTR(y); MW_PIN_PTR(ret);
    const int c = blockIdx.x * bdim + threadIdx.x;
    uint32_t g = blockIdx.y;
    const u32x4 *rp = (const u32x4 *)(recs + g);
    u32x4 r0 = rp[0], r1 = rp[1];
    uint32_t m_total = row_base[P];
    MW_PIN_S4(r0); MW_PIN_S4(r1); MW_PIN_S(m_total);
    while (g < m_total) {
        const int n_hits = (int)r1.x;
        if (n_hits > 0 && g < ret_cap) {
            const uint32_t peer = r0.w;
            uint32_t pos = base[r1.y * (uint32_t)P + peer] + r1.z;
            if (n_hits == 1) {
                if (pos < cap && c < n) mw_st16(ret + (size_t)g * n + c, mw_ld16(y + (size_t)pos * n + c));
            } else {
                // Three rows at a time: their hit slots are requested together, then their places, and every row
                // before any is added.  One after the other (slot, place, row, sum) a row with two hits held its wave for
                // two chains of three round trips: 22000 rows of 14336 bytes, 1.5 hits each, 130 -> 125 us.
                float acc[8];
                bool any = false;
                auto add = [&](uint32_t at, const u32x4 &v) __attribute__((always_inline)) {
                    if (at >= cap) return;
                    const float f[8] = {__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                                        __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u),
                                        __uint_as_float(v.z << 16), __uint_as_float(v.z & 0xffff0000u),
                                        __uint_as_float(v.w << 16), __uint_as_float(v.w & 0xffff0000u)};
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[j] = any ? acc[j] + f[j] : f[j];
                    any = true;
                };
                const mw_hit *h = hits + (size_t)g * Kd;
                for (int k = 1; k < n_hits; k += 2) {
                    const bool two = k + 1 < n_hits;
                    const mw_hit ha = h[k], hb = h[two ? k + 1 : k];
                    u32x4 v0 = {0u, 0u, 0u, 0u}, va = v0, vb = v0;
                    if (k == 1 && pos < cap && c < n) v0 = mw_ld16(y + (size_t)pos * n + c);
                    const uint32_t pa = base[(uint32_t)ha.le * P + peer] + (uint32_t)ha.rank;
                    const uint32_t pb = two ? base[(uint32_t)hb.le * P + peer] + (uint32_t)hb.rank : 0xffffffffu;
                    if (pa < cap && c < n) va = mw_ld16(y + (size_t)pa * n + c);
                    if (pb < cap && c < n) vb = mw_ld16(y + (size_t)pb * n + c);
                    if (k == 1) add(pos, v0);
                    add(pa, va);
                    add(pb, vb);
                }
                if (any && c < n) {
                    u32x4 o;
                    o.x = mw_bf16_rne(acc[0]) | (mw_bf16_rne(acc[1]) << 16);
                    o.y = mw_bf16_rne(acc[2]) | (mw_bf16_rne(acc[3]) << 16);
                    o.z = mw_bf16_rne(acc[4]) | (mw_bf16_rne(acc[5]) << 16);
                    o.w = mw_bf16_rne(acc[6]) | (mw_bf16_rne(acc[7]) << 16);
                    mw_st16(ret + (size_t)g * n + c, o);
                }
            }
        }
        g += gdim;
        if (g < m_total) { rp = (const u32x4 *)(recs + g); r0 = rp[0]; r1 = rp[1]; }
    }
}

}  // namespace

// The part of a peer's tokens that has an expert here, if ids are drawn evenly, and the experts such a token
// has here on average.
static double addressed_share(const mw_ctx *ctx, double *copies)
{
    const mw_config &c = ctx->cfg;
    const double share = c.n_experts > 0 ? (double)ctx->n_local / c.n_experts : 0.0;
    double none = 1.0;
    for (int k = 0; k < c.top_k; ++k) none *= 1.0 - share;
    *copies = none < 1.0 ? c.top_k * share / (1.0 - none) : 1.0;
    return 1.0 - none;
}

// Rows the peers' buffers will hold: as many as the context saw last, if the caller has asked for the
// statistics, else what full batches of evenly drawn ids would send.  For launch shapes only.
static int64_t expected_rows(const mw_ctx *ctx, int32_t P)
{
    if (ctx->recv_rows_hint > 0) return ctx->recv_rows_hint;
    double copies;
    const double rows = (double)P * ctx->cfg.max_tokens * addressed_share(ctx, &copies);
    return rows < (double)ctx->cfg.max_recv_rows ? (int64_t)rows : ctx->cfg.max_recv_rows;
}

// Index arguments of `ctx` for a launch whose workgroups may use `lds_words` words of LDS each: the
// addressed-rows bitmap, the table of local slots if there is room for it, and one and a half words per
// 32 source tokens for every expert of a chunk.  The chunks go to `parts` workgroups a peer, at most
// max_parts (further chunks by further passes), at least min_parts where the experts allow it.
// Returns false if max_tokens is beyond what the call takes (accept_words: the limit it states,
// three arrays of a bit per token).
static bool make_index_args(mw_ctx *ctx, const void *peers, bool packets, int32_t P, int64_t cap,
                            int64_t *expert_offsets, mw_recv_stats *stats, uint32_t accept_words, uint32_t lds_words,
                            uint32_t min_parts, uint32_t max_parts, mw_index_args *a, size_t *lds_bytes)
{
    const mw_config &c = ctx->cfg;
    const uint32_t L = (uint32_t)ctx->n_local;
    const uint32_t wpl = ((uint32_t)c.max_tokens + 31u) / 32u;
    const uint32_t dedup = (ctx->options & MW_OPT_RECV_DEDUP) ? 1u : 0u;
    if (accept_words < 3 * wpl + 64 + (dedup ? wpl : 0)) return false;
    uint32_t tab_words = ((uint32_t)c.n_experts + 4u) / 4u;             // a byte per expert and one for ids outside the range
    if (L > kNotLocal || tab_words > lds_words / 4 || mw_index_lds_words(wpl, 1, tab_words, dedup) > lds_words) tab_words = 0;
    uint32_t Lc = L > 0 ? L : 1;
    if (dedup) min_parts = max_parts = 1;            // one workgroup decides which of the repeats is taken
    if (L >= 2 * min_parts) Lc = (L + min_parts - 1) / min_parts;
    if (wpl > 0) {
        const size_t fixed = mw_index_lds_words(wpl, 0, tab_words, dedup);
        const size_t fit = lds_words > fixed ? 2 * (lds_words - fixed) / (3 * (size_t)wpl) : 0;
        if (fit < 1) return false;
        if (Lc > fit) Lc = (uint32_t)fit;
        while (Lc > 1 && mw_index_lds_words(wpl, Lc, tab_words, dedup) > lds_words) --Lc;
    }
    const uint32_t n_chunks = L > 0 ? (L + Lc - 1) / Lc : 1;
    *lds_bytes = mw_index_lds_words(wpl, Lc, tab_words, dedup) * sizeof(uint32_t);
    const uint32_t hb = packets ? (uint32_t)mw_packet_header_bytes_of(c.top_k) : 0u;
    *a = mw_index_args{peers, P, ctx->d_eslot, c.n_experts, c.top_k, ctx->hit_slots, c.my_rank, (int)L, (int)Lc,
                       (uint32_t)c.max_tokens, wpl, (uint32_t)c.max_recv_rows,
                       (uint64_t)(packets ? hb + ctx->row_bytes : ctx->row_stride), hb, cap,
                       ctx->d_cnt, ctx->d_row_base, ctx->d_addr_cnt, ctx->d_recs, ctx->d_hits, ctx->d_base,
                       expert_offsets, stats, ctx->d_flags, dedup, n_chunks < max_parts ? n_chunks : max_parts, 1u, tab_words};
    return true;
}

// Id lists of at most eight, at most 64 local experts and a table of their slots in LDS: a row's ids are
// one request and its distinct experts a 64-bit set, all in registers.  Anything beyond takes
// the general forms, a row a lane at a time.
static int index_form(const mw_index_args &a)
{
    return a.L > 64 || a.tab_words == 0 ? kFormAny : a.K > 8 ? kFormMany : kFormFew;
}

// LDS words a workgroup of `bs` lanes may reserve in a launch whose row movers should keep every wave
// slot: its share of a CU's 160 KiB when 2048 lanes are resident.
static uint32_t rider_lds_words(int bs) { return (uint32_t)bs * 20u; }
constexpr uint32_t kRiderAcceptWords = 1280, kIndexAcceptWords = 12288;   // limits on max_tokens the entry points state
constexpr uint32_t kMaxIndexParts = 16;
// What the row movers of a launch will take, in microseconds: `pack_tokens` rows packed and the received rows
// read once and written once per local expert, at 5.6 TB/s.
static double movers_us(const mw_ctx *ctx, int32_t P, int32_t pack_tokens)
{
    double copies;
    addressed_share(ctx, &copies);
    return ((double)expected_rows(ctx, P) * (1.0 + copies) + 2.0 * pack_tokens) * (double)ctx->row_bytes / 5.6e6;
}

// Workgroups over which the rows of a peer are spread, and what a rider then takes.
static int64_t rows_a_lane(const mw_ctx *next, int32_t P, int bs)
{
    const int64_t rows = (expected_rows(next, P) + P - 1) / P;
    return (rows + bs - 1) / bs;
}
static uint32_t index_row_parts(const mw_ctx *next, int32_t P, int bs)
{
    const int64_t per_lane = rows_a_lane(next, P, bs);
    return per_lane >= 8 ? 4u : per_lane >= 4 ? 2u : 1u;
}
static double rider_us(const mw_ctx *next, int32_t P, int bs, uint32_t row_parts)
{
    const double row_us = 1.4 * (double)((next->cfg.top_k + 7) / 8);
    return 6.0 + row_us * (double)rows_a_lane(next, P, bs) * (1.0 + 1.0 / row_parts);
}

// Row movers beside riders: folded where the narrower riders stay well below the movers (2048 fp8 tokens of 264 chunks, us a step not
// folded / folded: 16 ranks, 860 rows a peer, 39.3 / 36.4; 8 ranks, 1344 rows a peer and 32 experts, 37.2 / 38.6), and where they
// have room and time for the table of experts: of four waves up to ten experts a lane (100 ranks, 160 rows a peer, 2400 experts
// 44.5 / 41.4, 2560 44.7 / 42.5, 3200 44.9 / 44.7, 4800 48.4 / 52.8, and 5600, for whose table a rider has no LDS, 51.5 / 70.7), of eight
// waves as long as there is LDS (528 chunks, 256 ranks, 130 rows a peer, 4800 experts 55.7 / 50.3, 10000 56.1 / 51.6).  Sixteen waves
// are not narrower than rows in two workgroups.
static mw_row_shape rider_row_shape(const mw_ctx *ctx, const mw_ctx *next, int32_t P, int32_t next_P, int32_t pack_tokens, int chunks)
{
    const mw_row_shape s = mw_row_shape_folded(chunks);
    if (mw_is_folded(s, chunks) && s.bs < 1024 && next->cfg.n_experts > (s.bs < 512 ? 10 * s.bs : 20 * s.bs - 4)) return mw_row_shape_of(chunks);
    if (mw_is_folded(s, chunks) && rider_us(next, next_P, s.bs, index_row_parts(next, next_P, s.bs)) > 0.7 * movers_us(ctx, P, pack_tokens))
        return mw_row_shape_of(chunks);
    return s;
}

// Whether the next batch's index rides beside movers of `mover_us` in workgroups of `bs` lanes, and over how many
// workgroups its rows are then spread.  A rider takes about 1.4 us for every row and eight ids a lane of each pass; a launch of its own
// about 12 us.  Measured (us for expander and index; rows of a peer / lanes): 42 rows a lane, expander 80 us: 85.6 riding
// (110 with the rows not spread), 17 rows a lane, expander 11 us: 44 riding, 23.6 apart.
static bool index_rides(const mw_ctx *next, double mover_us, int bs, mw_index_args *a)
{
    if (index_form(*a) == kFormAny) return false;                   // (spills 25 of the riders' 64 registers)
    a->row_parts = a->dedup ? 1u : index_row_parts(next, a->P, bs);
    return rider_us(next, a->P, bs, a->row_parts) < mover_us + 12.0;
}

// Whether the next batch's plan rides beside movers of `mover_us` in workgroups of `bs` lanes.  It ranks tokens all-pairs over
// workgroups that talk through memory; the finishing ones walk every token's counters, T * T / bs of them, which
// is what grows beyond a thousand tokens.  Beside movers that are shorter it takes 48 us for 1000 tokens in wide workgroups, 6
// more with keys of several words, 56 in workgroups of two waves, and there 64 (4096 tokens), 72 (6144), 90 (8192).  A launch of its
// own takes 8 (up to 2048 tokens), 11 (4096), 16 us (8192), 18 with more than eight ids and bitmaps of several words.  Measured,
// us a step riding / apart, rows of 7168 from 16 and from 64 peers:
//   bf16, 256 ranks   1024 tokens 56 / 18, 59 / 23   4096 65 / 41, 68 / 65   6144 72 / 57, 91 / 94   8192 89 / 72, 130 / 121
//   fp8, 256 ranks    1024 tokens 53 / 15, 54 / 18   4096 57 / 33, 57 / 47   6144 58 / 45, 61 / 66   8192 59 / 56, 82 / 85
//   bf16, 64 ranks    1024 tokens 56 / 23, 63 / 47   4096 68 / 65, 161 / 169 6144 90 / 95, 252 / 254 8192 121 / 123, 347 / 345
//   fp8, 64 ranks     1024 tokens 47 / 18, 49 / 31   4096 50 / 47, 94 / 104  6144 57 / 66, 146 / 155 8192 78 / 85, 201 / 209
// Beside movers of any length it still takes memory time from them, beyond 7168 tokens in two-wave workgroups with keys of
// several words more than a launch of its own (130 / 121 above).
// The 13 and 21 below are what a launch took before its keys were sorted.  They make the plan ride at three of these points where
// it is no longer ahead: 68 for 65 us twice (4096 bf16 tokens, 256 ranks and 64 peers, 64 ranks and 16) and 347 for 345.
// A context whose wait limit the caller has set keeps its plans riding.
static bool plan_rides(const mw_ctx *next, double mover_us, int32_t T, bool keyed, int bs)
{
    if (T == 0 || next->ride_wait_limit != kRideWaitDefault) return true;
    if (keyed && bs < 256 && T > 7168) return false;
    const double t = T / 8192.0;
    const double rider_us = 13.0 + 35.0 * (T < 1024 ? T : 1024) / 1024.0 + (bs < 256 ? 8.0 : keyed ? 6.0 : 0.0) +
                            32.0 * t * t * 128.0 / bs;
    const double apart_us = !keyed && next->mask_words > 1 ? 18.0 : T <= 2048 ? 8.0 : T <= 4096 ? 13.0 : 21.0;
    return rider_us < mover_us + apart_us;
}

// the index of `P` peers' regions on `ctx` fits the one-workgroup form
static bool small_index_fits(const mw_ctx *ctx, int32_t P)
{
    if (ctx->options & MW_OPT_RECV_DEDUP) return false;
    if (P > kSmallPeers || ctx->n_local > 64) return false;
    if ((int64_t)P * ctx->cfg.max_tokens > 16384) return false;
    const uint32_t wpl = ((uint32_t)ctx->cfg.max_tokens + 31u) / 32u;
    return mw_small_index_lds_words(P, ctx->n_local, 0, wpl, (uint32_t)ctx->cfg.max_tokens,
                                    (uint32_t)ctx->cfg.max_recv_rows) * 4 <= kSmallIndexLds;
}

// LDS bytes of the one-workgroup index; a->tab_words: with the expert table where it has room
static size_t small_index_lds(const mw_ctx *ctx, int32_t P, mw_index_args *a)
{
    const uint32_t wpl = ((uint32_t)ctx->cfg.max_tokens + 31u) / 32u;
    const size_t words = mw_small_index_lds_words(P, ctx->n_local, 0, wpl, (uint32_t)ctx->cfg.max_tokens,
                                                  (uint32_t)ctx->cfg.max_recv_rows);
    const int E = ctx->cfg.n_experts;
    a->tab_words = E <= kSmallTab && 4 * (words + (size_t)E) <= kSmallIndexLds ? (uint32_t)E : 0;
    return 4 * (words + a->tab_words) + 16;
}

// Rows that a small step's index has to reckon with: as many as the context saw last time, if the caller has asked
// for the statistics, else all there can be.  The one-workgroup index keeps one or two of them a lane in registers (448 rows: with
// two 8.3 us, with one 7.6); more go through memory.
static int64_t small_index_rows(const mw_ctx *ctx, int32_t P)
{
    return ctx->recv_rows_hint > 0 ? ctx->recv_rows_hint : (int64_t)P * ctx->cfg.max_tokens;
}

// defer: the caller's expander can make its places of the counts (k_expand_counts).  *deferred: it has to (the one-workgroup index
// has them in LDS and finishes by itself).
static int32_t launch_unpack_index(mw_ctx *ctx, const void *peers, bool packets, int32_t P, int64_t cap, int64_t *expert_offsets,
                                   mw_recv_stats *stats, bool defer, bool *deferred, hipStream_t s)
{
    *deferred = false;
    mw_index_args a;
    size_t lds_index;
    // A few peers with many experts each: up to four workgroups a peer (8 peers of 2720 rows, 32 experts:
    // 14.5 us with four, 16.1 with one, 14.5 with eight; no difference where a peer has fewer rows than lanes).
    uint32_t min_parts = 1;
    while (min_parts < 4 && (uint32_t)P * min_parts < 32) min_parts *= 2;
    if (!make_index_args(ctx, peers, packets, P, cap, expert_offsets, stats, kIndexAcceptWords, 16384, min_parts,
                         kMaxIndexParts, &a, &lds_index))
        return MW_ERR_UNSUPPORTED;
    // A lane per row as long as a workgroup has that many (a peer seldom sends more than a fraction of its
    // tokens to one rank): fewer lanes have shorter barriers and scans, more of them fewer rows each.  The rows of one
    // peer spread about their mean, and the peer with one row more than lanes is the one all wait for: three roots more than
    // the mean (64 peers of 478 +- 21 rows: 10.0 us with 512 lanes, 8.7 with 1024).  With
    // more rows than lanes three a lane are requested together (8 peers of 2720 rows: 13.6 us, one at a time
    // 14.5), with fewer one (16 peers of 429 rows: 8.3 us, with room for three 8.7).
    const int64_t rows_of_peer = (expected_rows(ctx, P) + P - 1) / P;
    const double most = (double)rows_of_peer + 3.0 * std::sqrt((double)rows_of_peer);
    const int ib = most <= 256.0 ? 256 : most <= 512.0 ? 512 : kIndexBlock;
    {
        mw_timed tm(ctx, MW_KERNEL_RECV_INDEX, s);
        const int64_t expected = ctx->recv_rows_hint > 0 ? ctx->recv_rows_hint : (int64_t)P * ctx->cfg.max_tokens;
        if (!packets && expected <= kSmallLanes && small_index_fits(ctx, P)) {
            // a row a lane at most: one workgroup for all peers, nothing to exchange between workgroups
            // (9.6 against 10.9 us at 443 rows; with two rows a lane the workgroup-per-peer form is ahead)
            const size_t lds = small_index_lds(ctx, P, &a);
            hipLaunchKernelGGL(k_recv_index_small, dim3(1), dim3(kSmallLanes), lds, s, a);
        } else
        {
            if (defer) { a.stats = nullptr; *deferred = true; }
#define MW_INDEX(GENERAL_, ROWS_)                                                                                              \
    do {                                                                                                                       \
        if (packets) hipLaunchKernelGGL((k_recv_index<true, GENERAL_, ROWS_>), dim3(P, a.parts), dim3(ib), lds_index, s, a);   \
        else hipLaunchKernelGGL((k_recv_index<false, GENERAL_, ROWS_>), dim3(P, a.parts), dim3(ib), lds_index, s, a);          \
    } while (0)
            if (index_form(a) == kFormAny) MW_INDEX(kFormAny, 1);
            else if (index_form(a) == kFormMany) MW_INDEX(kFormMany, 1);
            else if (rows_of_peer <= ib) MW_INDEX(kFormFew, 1);
            else MW_INDEX(kFormFew, 3);
#undef MW_INDEX
        }
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_unpack_index(mw_ctx *ctx, const void *peers, bool packets, int32_t P, int64_t cap, int64_t *expert_offsets,
                               mw_recv_stats *stats, hipStream_t s)
{
    bool deferred;
    return launch_unpack_index(ctx, peers, packets, P, cap, expert_offsets, stats, false, &deferred, s);
}

// Grid rows of the expander and of the combine: about as many as the peers will hold, not the capacity -- workgroups are
// dispatched at a finite rate, empty ones included (16 ranks, 1000 tokens, capacity 16000 rows, 6750 there: mw_plan,
// mw_pack and mw_unpack 34.3 us for the capacity, 32.0 for the rows).  More rows than that are reached by striding.
// Where nobody has said how many there are, at least what fills every CU's wave slots, and no second filling of a few
// workgroups: a rank that the routing favours gets many times its share.  (256 ranks, one
// expert each, 64 tokens, all 16384 of them here, us for a grid of the expected 129 rows / one filling / two / the capacity:
// mw_unpack of 14336-byte rows 150 / 86 / 86 / 81, of 4096-byte 116 / 33 / 33 / 33, of 1024-byte 67 / 18 / 19 / 21; 32000 fp8
// rows where 1089 grid rows were expected, 1.06 fillings, 107 / - / 90 / 92.)  What is left: 114688 rows where 4036 were
// expected stride 27 times, 620 us against 569 for 32768 grid rows, the combine 605 against 511; evenly spread batches are
// several times faster than with the capacity (64 ranks, 512 tokens: 134 us and 27).
// The filling is that of folded rows for every caller, also where the launch does not fold them (the combine, small steps, riders
// that refuse): a few more grid rows than the launch's own shape would give.  Neither is ahead everywhere (us for the filling of
// folded / unfolded rows, 12800 rows that nobody had announced: combine of 264 chunks 19.8 / 21.9, of 528 36.7 / 37.9; steps of 256 tokens
// of 264 chunks 18.3 / 17.5, of 64 tokens 9.4 / 9.4, of 1025 chunks 16.9 / 17.3).
static uint32_t expand_grid_rows(const mw_ctx *ctx, int32_t P)
{
    int64_t rows = expected_rows(ctx, P);
    rows += rows / 64 + 64;
    if (ctx->recv_rows_hint == 0) {
        const mw_row_shape shape = mw_row_shape_folded((int)(ctx->row_bytes / 16));
        const int64_t filling = (int64_t)ctx->n_cu * 2048 / ((int64_t)shape.bs * shape.nseg);
        if (rows < filling) rows = filling;
        else if (rows < 2 * filling) rows = 2 * filling;
        const int64_t most = (int64_t)P * ctx->cfg.max_tokens;
        if (rows > most) rows = most;
    }
    if (rows > ctx->cfg.max_recv_rows) rows = ctx->cfg.max_recv_rows;
    if (rows < 1) rows = 1;
    return (uint32_t)(rows < kRowGridMax ? rows : kRowGridMax);
}

int32_t mw_launch_unpack_expand(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                int32_t *out_src_peer, int32_t *out_src_token, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    if (c.max_recv_rows > 0) {
        const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
        const mw_row_shape shape = mw_row_shape_folded(xc + sc);
        const uint32_t gy = expand_grid_rows(ctx, P);
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        hipLaunchKernelGGL(mw_is_folded(shape, xc + sc) ? k_expand<true> : k_expand<false>, dim3(shape.nseg, gy), dim3(shape.bs), 0, s,
                           ctx->d_recs, ctx->d_row_base, ctx->d_base, ctx->d_hits, P, ctx->hit_slots, xc, sc, (u32x4 *)out_rows,
                           (u32x4 *)out_scales, (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL), out_src_peer, out_src_token);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

// Index and expander of one batch in two launches.
int32_t mw_launch_unpack_two(mw_ctx *ctx, const void *peers, bool packets, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                             int32_t *out_src_peer, int32_t *out_src_token, int64_t *expert_offsets, mw_recv_stats *stats, hipStream_t s)
{
    const uint32_t n_counts = (uint32_t)ctx->n_local * (uint32_t)P;
    const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
    const mw_row_shape shape = mw_row_shape_folded(xc + sc);
    const bool fold = mw_is_folded(shape, xc + sc);
    double hits;
    addressed_share(ctx, &hits);
    const bool defer = ctx->cfg.max_recv_rows > 0 &&
                       mw_counts_by_expander(ctx->n_local, P, packets, fold, hits, expected_rows(ctx, P) * ctx->row_bytes);
    bool deferred;
    const int32_t rc = launch_unpack_index(ctx, peers, packets, P, cap, expert_offsets, stats, defer, &deferred, s);
    if (rc != MW_OK) return rc;
    if (!deferred) return mw_launch_unpack_expand(ctx, P, out_rows, out_scales, cap, out_src_peer, out_src_token, s);
    const uint32_t gy = expand_grid_rows(ctx, P) + 1;
    {
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        hipLaunchKernelGGL((n_counts <= 64    ? fold ? k_expand_counts<true, 1> : k_expand_counts<false, 1>
                            : n_counts <= 256 ? fold ? k_expand_counts<true, 4> : k_expand_counts<false, 4>
                                              : fold ? k_expand_counts<true, 8> : k_expand_counts<false, 8>),
                           dim3(shape.nseg, gy), dim3(shape.bs), 0, s, ctx->d_recs, ctx->d_row_base, ctx->d_cnt, ctx->d_hits, P,
                           ctx->hit_slots, xc, sc, n_counts, (u32x4 *)out_rows, (u32x4 *)out_scales,
                           (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL), out_src_peer, out_src_token, (uint32_t)ctx->n_local, cap,
                           ctx->d_addr_cnt, ctx->d_flags, ctx->d_base, expert_offsets, stats);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_unpack(mw_ctx *ctx, const mw_recv_peer *peers, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                         int32_t *out_src_peer, int32_t *out_src_token, int64_t *expert_offsets, mw_recv_stats *stats, hipStream_t s)
{
    // Index and expander in one launch as long as a row is at most a lane's and the payload is short (us in two launches / in
    // one: 244 rows of 512 bytes 9.6 / 6.7, 355 of 14336 12.9 / 10.6, 506 of 14336 12.4 / 11.7 but 14.0 / 14.2 for a call among
    // idle ones, 244 of 65536 12.5 / 16.1; 812 rows of 2048 12.9 / 11.7, 646 of 14336 15.4 / 16.2, 1007 of 14336 15.5 / 21.0).
    // More rows than expected are moved all the same.  A caller who has set events for the index wants its own duration:
    // two launches then.
    constexpr int64_t kSmallUnpackBytes = 6 << 20;
    const int64_t expected = ctx->recv_rows_hint > 0 ? ctx->recv_rows_hint : (int64_t)P * ctx->cfg.max_tokens;
    mw_index_args a;
    size_t lds_index;
    const bool timed = ctx->ev_start[MW_KERNEL_RECV_INDEX] || ctx->ev_stop[MW_KERNEL_RECV_INDEX];
    if (expected <= kSmallLanes && small_index_fits(ctx, P) && expected * ctx->row_bytes <= kSmallUnpackBytes && !timed &&
        ctx->row_bytes <= 65536 && ctx->cfg.max_recv_rows > 0 &&
        make_index_args(ctx, peers, false, P, cap, expert_offsets, stats, kIndexAcceptWords, 16384, 1, kMaxIndexParts, &a, &lds_index)) {
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
        // (64 rows more than the last batch had: the next one may be larger, and a wave then strides)
        const int64_t rows = ctx->recv_rows_hint > 0 ? expected + 64 : expected;
        const int64_t waves = rows * ((xc + sc + 63) / 64), wgs = (waves + kSmallLanes / 64 - 1) / (kSmallLanes / 64);
        const int grid = wgs < 1 ? 1 : wgs < ctx->n_cu ? (int)wgs : ctx->n_cu;
        const size_t lds = small_index_lds(ctx, P, &a);
        hipLaunchKernelGGL(k_unpack_small, dim3(grid), dim3(kSmallLanes), lds, s, a, xc, sc, (u32x4 *)out_rows, (u32x4 *)out_scales,
                           (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL), out_src_peer, out_src_token);
        MW_HIP_CHECK(hipGetLastError());
        return MW_OK;
    }
    return mw_launch_unpack_two(ctx, peers, false, P, out_rows, out_scales, cap, out_src_peer, out_src_token, expert_offsets, stats, s);
}

// The riders of k_small_step beside its one-workgroup index (false: they are not needed).  *fits: both forms can be had.
static bool small_step_riders(mw_ctx *next, const void *peers, int32_t P, int64_t cap, int64_t *expert_offsets,
                              mw_recv_stats *stats, mw_index_args *general, size_t *lds, bool *fits)
{
    *fits = true;
    if (small_index_rows(next, P) <= (int64_t)kEitherRows) return false;
    const uint32_t words = kSmallIndexLds / 4;
    *fits = make_index_args(next, peers, false, P, cap, expert_offsets, stats, words, words, 1, kMaxIndexParts, general, lds) &&
            index_form(*general) != kFormAny;
    if (!*fits) return false;
    const int per_lane = (next->cfg.max_tokens + kSmallLanes - 1) / kSmallLanes;
    general->row_parts = per_lane >= 8 ? 4u : per_lane >= 4 ? 2u : 1u;
    return true;
}

// Whether a step is small enough for k_small_step -- this batch's rows (received and to pack) under
// 24 MiB, so that the riders and not the movers are the step; the next batch's index in one
// workgroup's LDS and at most MW_FUSED_MAX_TOKENS tokens to plan -- and, if so, its launch.
// with_plan: the launch plans next_T tokens (possibly none); pk: rows to pack, or null.
static bool small_step_fits(const mw_ctx *ctx, mw_ctx *next, int32_t next_P, int32_t next_T, const mw_pack_call *pk,
                            uint32_t gy)
{
    const int64_t rows = (int64_t)gy + (pk ? pk->n_tokens : 0);
    if (rows * ctx->row_bytes > (24LL << 20)) return false;
    if (next_T > MW_FUSED_MAX_TOKENS) return false;
    if (!small_index_fits(next, next_P)) return false;
    mw_index_args general;
    size_t lds;
    bool fits;
    small_step_riders(next, nullptr, next_P, 0, nullptr, nullptr, &general, &lds, &fits);
    return fits;
}

static int32_t launch_small_step(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                 int32_t *out_src_peer, int32_t *out_src_token, mw_ctx *next, const mw_index_args &a,
                                 bool with_plan, const int32_t *next_topk, int32_t next_T, uint64_t *next_mask,
                                 int32_t *next_perm, mw_group_desc *next_desc, mw_send_stats *next_send_stats,
                                 const mw_pack_call *pk, uint32_t gy, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
    const int nseg = (xc + sc + kSmallLanes - 1) / kSmallLanes;
    const int K = next->cfg.top_k, W = next->mask_words;
    const bool keyed = W > 1 && K <= 8;
    mw_plan_args pl = {};
    pl.topk = next_topk; pl.T = next_T; pl.K = K; pl.E = next->cfg.n_experts; pl.eslot = next->d_eslot;
    pl.mask_out = next_mask; pl.perm = next_perm; pl.desc = next_desc; pl.stats = next_send_stats;
    pl.row_bytes = (uint64_t)next->row_bytes;
    mw_pack_args pa = {};
    uint32_t n_pack_rows = 0;
    if (pk && pk->n_tokens > 0) {
        pa.x = (const u32x4 *)pk->x; pa.scales = (const u32x4 *)pk->scales; pa.xc = xc; pa.sc = sc;
        pa.ns = (int)(ctx->row_stride / 16);
        pa.topk = pk->topk; pa.K = c.top_k; pa.perm = pk->perm; pa.stats = pk->stats;
        pa.packed = (u32x4 *)pk->packed; pa.row_src_token = pk->row_src_token; pa.row_topk = pk->row_topk;
        n_pack_rows = (uint32_t)pk->n_tokens;
    }
    mw_index_args ai = a;
    const size_t lds_index = small_index_lds(next, a.P, &ai);
    const size_t lds_plan = 8 * (size_t)(keyed    ? mw_small_plan_words<4, true>()
                                         : W == 1 ? mw_small_plan_words<1, false>()
                                         : W == 2 ? mw_small_plan_words<2, false>()
                                         : W == 3 ? mw_small_plan_words<3, false>()
                                                  : mw_small_plan_words<4, false>());
    size_t lds = with_plan && lds_plan > lds_index ? lds_plan : lds_index;
    const uint32_t general_row = with_plan ? 2u : 1u;
    mw_index_args general = {};
    size_t lds_general = 0;
    bool fits;
    const bool either = small_step_riders(next, a.peers, a.P, a.out_cap, a.expert_offsets, a.stats, &general, &lds_general, &fits);
    if (either && lds < lds_general) lds = lds_general;
    const uint32_t riders = general_row + (either ? (index_riders(general) + (uint32_t)nseg - 1) / (uint32_t)nseg : 0u);
    const dim3 grid(nseg, riders + n_pack_rows + gy), block(kSmallLanes);
    const uint32_t cap32 = (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL);
    {
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        const bool one_row = small_index_rows(next, a.P) <= kSmallLanes;
#define MW_SMALL_(W_, KEYED_, ROWS_, EITHER_)                                                                          \
    hipLaunchKernelGGL((k_small_step<W_, KEYED_, ROWS_, EITHER_>), grid, block, lds, s, riders, riders + n_pack_rows, ctx->d_recs, \
                       ctx->d_row_base, P, xc, pa.perm, pa.stats, sc, ctx->hit_slots, ctx->d_base, ctx->d_hits,         \
                       (u32x4 *)out_rows, (u32x4 *)out_scales, cap32, out_src_peer, out_src_token, ai, pl, pa, general, general_row)
#define MW_SMALL(W_, KEYED_)                                                                                           \
    do {                                                                                                               \
        if (either) MW_SMALL_(W_, KEYED_, 2, true);                                                                    \
        else if (one_row) MW_SMALL_(W_, KEYED_, 1, false);                                                             \
        else MW_SMALL_(W_, KEYED_, 2, false);                                                                          \
    } while (0)
        if (keyed) MW_SMALL(4, true);
        else if (W == 1) MW_SMALL(1, false);
        else if (W == 2) MW_SMALL(2, false);
        else if (W == 3) MW_SMALL(3, false);
        else MW_SMALL(4, false);
#undef MW_SMALL
#undef MW_SMALL_
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_unpack_expand_index_next(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                           int32_t *out_src_peer, int32_t *out_src_token, mw_ctx *next,
                                           const mw_recv_peer *next_peers, int32_t next_P, int64_t next_cap,
                                           int64_t *next_expert_offsets, mw_recv_stats *next_stats, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    if (c.max_recv_rows < 1) return MW_ERR_UNSUPPORTED;       // nothing to ride on
    const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
    mw_row_shape shape = rider_row_shape(ctx, next, P, next_P, 0, xc + sc);
    // Rows of whole cache lines: two-wave workgroups here.  The expander runs as fast with them
    // as with single waves (138.8 against 139.4 us at 30590 rows of 14336 bytes), and the riding
    // index gets two waves per peer: with one it outlasts the expander (142 against 139 us).
    if (shape.bs == 64 && (xc + sc) % 16 == 0) { shape.bs = 128; shape.nseg = (xc + sc) / 128 + ((xc + sc) % 128 ? 1 : 0); }
    // Every workgroup of the launch reserves the index's LDS, the expander's included: no more than
    // leaves a CU a full set of the expander's waves.
    mw_index_args a;
    size_t lds_index;
    if (!make_index_args(next, next_peers, false, next_P, next_cap, next_expert_offsets, next_stats, kRiderAcceptWords,
                         rider_lds_words(shape.bs), 1, kMaxIndexParts, &a, &lds_index))
        return MW_ERR_UNSUPPORTED;
    const uint32_t gy = expand_grid_rows(ctx, P);
    if (small_step_fits(ctx, next, next_P, 0, nullptr, gy))
        return launch_small_step(ctx, P, out_rows, out_scales, cap, out_src_peer, out_src_token, next, a, false, nullptr,
                                 0, nullptr, nullptr, nullptr, nullptr, nullptr, gy, s);
    if (!index_rides(next, movers_us(ctx, P, 0), shape.bs, &a)) {      // a launch of its own in front
        const int32_t rc = mw_launch_unpack_index(next, next_peers, false, next_P, next_cap, next_expert_offsets, next_stats, s);
        if (rc != MW_OK) return rc;
        return mw_launch_unpack_expand(ctx, P, out_rows, out_scales, cap, out_src_peer, out_src_token, s);
    }
    const uint32_t index_rows = ((uint32_t)next_P * a.parts * a.row_parts + (uint32_t)shape.nseg - 1) / (uint32_t)shape.nseg;
    {
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        const uint32_t cap32 = (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(shape.nseg, gy + index_rows), dim3(shape.bs), lds_index, s, index_rows, 0u,
                               ctx->d_recs, ctx->d_row_base, ctx->d_base, ctx->d_hits, P, ctx->hit_slots, xc, sc,
                               (u32x4 *)out_rows, (u32x4 *)out_scales, cap32, out_src_peer, out_src_token, a);
        };
        const bool fold = mw_is_folded(shape, xc + sc);
        if (index_form(a) == kFormMany) launch(fold ? k_expand_index_next<kFormMany, true> : k_expand_index_next<kFormMany, false>);
        else launch(fold ? k_expand_index_next<kFormFew, true> : k_expand_index_next<kFormFew, false>);
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_unpack_expand_index_plan_next(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                                int32_t *out_src_peer, int32_t *out_src_token, mw_ctx *next,
                                                const mw_recv_peer *next_peers, int32_t next_P, int64_t next_cap,
                                                int64_t *next_expert_offsets, mw_recv_stats *next_stats,
                                                const int32_t *next_topk, int32_t next_T, uint64_t *next_mask,
                                                int32_t *next_perm, mw_group_desc *next_desc,
                                                mw_send_stats *next_send_stats, const mw_pack_call *pk, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    if (c.max_recv_rows < 1) return MW_ERR_UNSUPPORTED;       // nothing to ride on
    if (next_T > MW_RIDE_MAX_TOKENS) return MW_ERR_UNSUPPORTED;
    const int xc = (int)(ctx->x_row_bytes / 16), sc = (int)(ctx->s_row_bytes / 16);
    mw_row_shape shape = rider_row_shape(ctx, next, P, next_P, pk ? pk->n_tokens : 0, xc + sc);
    if (shape.bs == 64 && (xc + sc) % 16 == 0) { shape.bs = 128; shape.nseg = (xc + sc) / 128 + ((xc + sc) % 128 ? 1 : 0); }
    mw_index_args a;
    size_t lds_index;
    if (!make_index_args(next, next_peers, false, next_P, next_cap, next_expert_offsets, next_stats, kRiderAcceptWords,
                         rider_lds_words(shape.bs), 1, kMaxIndexParts, &a, &lds_index))
        return MW_ERR_UNSUPPORTED;
    const uint32_t gy = expand_grid_rows(ctx, P);
    if (small_step_fits(ctx, next, next_P, next_T, pk, gy))
        return launch_small_step(ctx, P, out_rows, out_scales, cap, out_src_peer, out_src_token, next, a, true, next_topk,
                                 next_T, next_mask, next_perm, next_desc, next_send_stats, pk, gy, s);

    const int K = next->cfg.top_k, W = next->mask_words;
    const bool keyed = W > 1 && K <= 8;
    const double mover_us = movers_us(ctx, P, pk ? pk->n_tokens : 0);
    if (!index_rides(next, mover_us, shape.bs, &a)) {                // a launch of its own in front
        const int32_t rc = mw_launch_unpack_index(next, next_peers, false, next_P, next_cap, next_expert_offsets, next_stats, s);
        if (rc != MW_OK) return rc;
        a.parts = 0;
    }
    const bool with_plan = plan_rides(next, mover_us, next_T, keyed, shape.bs);
    if (!with_plan) {
        const int32_t rc = mw_launch_plan(next, next_topk, next_T, next_mask, next_perm, next_desc, next_send_stats, s);
        if (rc != MW_OK) return rc;
    }

    // the riding plan: workgroups of the launch's size
    mw_plan_args pl;
    pl.topk = next_topk; pl.T = next_T; pl.K = K; pl.E = next->cfg.n_experts; pl.eslot = next->d_eslot;
    pl.mask_out = next_mask; pl.cnt = (unsigned long long *)next->d_plan_cnt; pl.pstate = next->d_plan_state;
    pl.perm = next_perm; pl.desc = next_desc; pl.stats = next_send_stats; pl.row_bytes = (uint64_t)next->row_bytes;
    // Slices as long as LDS allows: every (token, slice) pair costs one device-scope atomic and
    // every rank workgroup one more on a single counter, and those -- unlike the ranking itself --
    // take memory-channel time from the expander (slices of 128 tokens: +22 us per launch at
    // 4096 tokens; of 1024: +4 us).  Workgroups of two or more waves leave room for 8 KiB each.
    const size_t key_bytes = keyed ? sizeof(mw_short_key) : (size_t)W * sizeof(uint64_t);
    const size_t lds_budget = shape.bs >= 128 ? 8192 : 5120;
    pl.slice = (int)(lds_budget / key_bytes) / 128 * 128;
    if (pl.slice > (next_T + 127) / 128 * 128) pl.slice = (next_T + 127) / 128 * 128;
    if (pl.slice < 128) pl.slice = 128;
    pl.tb = next_T > 0 ? (next_T + shape.bs - 1) / shape.bs : 1;
    pl.ns = next_T > 0 ? (next_T + pl.slice - 1) / pl.slice : 1;
    pl.n_rank = (uint32_t)pl.tb * (uint32_t)pl.ns;
    pl.finish_rows = mw_plan_finish_rows(shape.bs);
    pl.n_finish = next_T > 0 ? ((uint32_t)next_T + pl.finish_rows - 1) / pl.finish_rows : 1u;
    pl.wait_limit = next->ride_wait_limit;
    if (!with_plan) pl.n_rank = pl.n_finish = 0;
    const uint32_t rider_rows = ((uint32_t)next_P * a.parts * a.row_parts + pl.n_rank + pl.n_finish + (uint32_t)shape.nseg - 1) /
                                (uint32_t)shape.nseg;
    size_t lds_plan = (size_t)pl.slice * key_bytes;
    if (lds_plan < mw_plan_finish_lds(shape.bs)) lds_plan = mw_plan_finish_lds(shape.bs);
    size_t lds = 0;                                              // of the riders there are
    if (a.parts > 0) lds = lds_index;
    if (with_plan && lds < lds_plan) lds = lds_plan;
    {
        mw_timed tm(ctx, MW_KERNEL_EXPAND, s);
        // the packer of this context's own rows, if asked for: same row shape as the expander
        mw_pack_args pa = {};
        uint32_t n_pack_rows = 0;
        if (pk && pk->n_tokens > 0) {
            pa.x = (const u32x4 *)pk->x; pa.scales = (const u32x4 *)pk->scales; pa.xc = xc; pa.sc = sc;
            pa.ns = (int)(ctx->row_stride / 16);
            pa.topk = pk->topk; pa.K = c.top_k; pa.perm = pk->perm; pa.stats = pk->stats;
            pa.packed = (u32x4 *)pk->packed; pa.row_src_token = pk->row_src_token; pa.row_topk = pk->row_topk;
            n_pack_rows = (uint32_t)pk->n_tokens < 16384u ? (uint32_t)pk->n_tokens : 16384u;   // more by striding
        }
        // a grid has at most 65535 rows: the expander takes what the riders leave (more by striding)
        const uint32_t riders = rider_rows + n_pack_rows;                         // <= 16384 + 8192 + 16384
        const uint32_t gy_fit = gy < 65535u - riders ? gy : 65535u - riders;
        const dim3 grid(shape.nseg, gy_fit + riders), block(shape.bs);
        const uint32_t cap32 = (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL);
        const bool fold = mw_is_folded(shape, xc + sc), part = n_pack_rows > 0 && mw_step_rows_part(ctx->row_stride);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, lds, s, rider_rows, rider_rows + n_pack_rows, ctx->d_recs,
                               ctx->d_row_base, P, xc, pa.perm, pa.stats, sc, ctx->hit_slots, ctx->d_base, ctx->d_hits,
                               (u32x4 *)out_rows, (u32x4 *)out_scales, cap32, out_src_peer, out_src_token, a, pl, pa);
        };
#define MW_RIDE_(W_, KEYED_, FORM_)                                                                                  \
    launch(fold   ? k_expand_index_plan_next<W_, KEYED_, FORM_, true, false>                                         \
           : part ? k_expand_index_plan_next<W_, KEYED_, FORM_, false, true>                                         \
                  : k_expand_index_plan_next<W_, KEYED_, FORM_, false, false>)
#define MW_RIDE(W_, KEYED_)                                                                                          \
    do {                                                                                                             \
        if (index_form(a) == kFormMany) MW_RIDE_(W_, false, kFormMany);                            /* (not keyed) */ \
        else MW_RIDE_(W_, KEYED_, kFormFew);                                                                         \
    } while (0)
        if (keyed) MW_RIDE(4, true);
        else if (W == 1) MW_RIDE(1, false);
        else if (W == 2) MW_RIDE(2, false);
        else if (W == 3) MW_RIDE(3, false);
        else MW_RIDE(4, false);
#undef MW_RIDE
#undef MW_RIDE_
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}

int32_t mw_launch_combine(mw_ctx *ctx, int32_t P, const void *y, int64_t cap, void *ret, int64_t ret_cap, hipStream_t s)
{
    const mw_config &c = ctx->cfg;
    if (c.max_recv_rows > 0 && ret_cap > 0) {
        const int n = (int)(ctx->x_row_bytes / 16);
        const mw_row_shape shape = mw_row_shape_of(n);
        const uint32_t gy = expand_grid_rows(ctx, P);
        mw_timed tm(ctx, MW_KERNEL_COMBINE, s);
        hipLaunchKernelGGL(k_combine, dim3(shape.nseg, gy), dim3(shape.bs), 0, s, ctx->d_recs, ctx->d_hits, ctx->d_base,
                           ctx->d_row_base, P, ctx->hit_slots, n, (const u32x4 *)y,
                           (uint32_t)(cap < 0x7fffffffLL ? cap : 0x7fffffffLL), (u32x4 *)ret,
                           (uint32_t)(ret_cap < 0x7fffffffLL ? ret_cap : 0x7fffffffLL));
    }
    MW_HIP_CHECK(hipGetLastError());
    return MW_OK;
}
