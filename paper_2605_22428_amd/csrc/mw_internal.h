// Internal declarations shared by the HIP sources of the MultiWrite library.
// Not installed; the public C ABI is include/mw.h.
#ifndef MW_INTERNAL_H_
#define MW_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mw.h"

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define MW_PLAN_STATE_WORDS 264   // 256 histogram bins + kept tokens + flags + two counts of workgroups done (+ padding)

// (local expert slot, rank among the peer's rows for that expert); le < 0 = unused slot
struct mw_hit { int32_t le; int32_t rank; };

// One received row as the expander needs it, in one 32-byte record: where it lies, its
// source token and peer, how many local experts it goes to and the first of them.  Further
// (expert slot, rank) pairs are in the row's hit slots 1 .. n_hits - 1.
struct mw_row_rec {
    const void *src;
    int32_t src_token;
    int32_t peer;
    int32_t n_hits;     // 0: nothing to deliver
    int32_t le0;        // first local expert slot
    int32_t rank0;      // rank among the peer's rows for that expert
    int32_t reserved0;
};

// Launch shape of the row movers: one 16-byte chunk per lane, grid x = segment of `bs` chunks
// of a row, grid y = row, so workgroups are dispatched in address order along a row and then
// row by row.  Measured on MI355X (expander, 30590 received rows, GB/s of HBM traffic):
//
//   row bytes              2048  4096  7168  8192  10240  12288  14336  16384  24576
//   single-wave segments   4413  4753  4848  4872   5879   6470   6485   6350   6427
//   one workgroup per row  5824  6194  6158  6332   5976   6225   6073   6225   6448
//
// Rows of up to 10 KiB are moved by one workgroup each (a wave per KiB).  Longer rows that are
// whole 128-byte cache lines (bf16 rows of 14336 bytes) are cut into single-wave workgroups:
// whole-row workgroups of 14 waves leave an eighth of a CU's wave slots empty, and several
// chunks per lane, or all rows' first segments first, are slower still.  Rows that are not whole
// cache lines (fp8 rows of 7392 bytes start and end inside lines) are never cut into single
// waves, so the lines two pieces share are touched from one CU: cut, such rows were 40 % slower.
constexpr uint32_t kRowGridMax = 32768;       // grid y; further rows by striding
struct mw_row_shape { int bs; int nseg; };
static inline mw_row_shape mw_row_shape_of(int chunks)
{
    if (chunks < 1) return mw_row_shape{64, 1};
    if (chunks % 8 == 0 && chunks > 640) return mw_row_shape{64, (chunks + 63) / 64};
    int b = (chunks + 63) / 64 * 64;
    if (b > 1024) b = 1024;
    return mw_row_shape{b, (chunks + b - 1) / b};
}

// The same for movers whose first lanes can take a second chunk (expander, packer).  A row whose last wave would have at most
// sixteen chunks gives them to its first lanes where four, eight or sixteen waves are left: a CU's 32 wave slots then hold a
// third more rows, and no slot is left over.  An fp8 row's scales are a thirty-second of it and make just such a wave: 264
// chunks (4096 codes) in five waves are six rows a CU, in four eight.  Measured, us, before / after: 6600 rows of 264 chunks
// expanded 13.6 / 13.0, a stream step of 2048 such tokens of 16 ranks 39.3 / 36.4; of 528 chunks 43.5 / 42.8 and 57.6 / 52.7; of
// 1025 chunks (two workgroups before) 77.4 / 52.6 and 189.4 / 128.0.  Elsewhere it only costs.  Ten waves, three rows a CU instead
// of two: 644 chunks expanded 28.2 / 28.9, a step of 655 chunks 87.2 / 88.9.  Where the CU holds hardly more rows: 330 chunks
// 29.4 / 29.4, 396 chunks 33.4 / 33.5 and 49.0 / 49.2, 462 chunks (four rows a CU either way) 76.0 / 76.3 and 90.0 / 94.8.  Short
// rows: 132 chunks (three waves) 25.2 / 24.6, but 6700 rows of 1.4 hits 10.8 / 11.2.
static inline mw_row_shape mw_row_shape_folded(int chunks)
{
    mw_row_shape s = mw_row_shape_of(chunks);
    const int rest = chunks % 64, waves = chunks / 64;
    if (s.bs > 64 && (waves == 4 || waves == 8 || waves == 16) && rest >= 1 && rest <= 16) s = mw_row_shape{waves * 64, 1};
    return s;
}
static inline bool mw_is_folded(const mw_row_shape &s, int chunks) { return (int64_t)s.bs * s.nseg < chunks; }

// Rows that are no whole number of cache lines apart are stored streaming only (mw_st16_part) or written through (mw_st16), by launch.
// Whether a packer's launch of up to n_rows rows stores them streaming only.  Short rows of a batch of 2 to 18 MiB are written through: what the L2 has
// put together is written at the launch's end, and with rows under 2560 bytes there is little to put together.  us of k_pack, written
// through / not: 8192 rows of 272 bytes 6.0 / 6.2; 4096 of 656 4.4 / 4.3, 1056 4.5 / 4.9, 1584 4.8 / 5.1, 2112 4.8 / 5.1, 2448 5.6 / 5.9, 3168 6.6 / 6.6; 8192 of
// 1056 6.1 / 6.9, 2112 7.9 / 8.2, 2448 9.5 / 9.3; 16384 of 656 9.6 / 10.7, 1200 12.6 / 12.2, 2112 15.4 / 14.5, 5280 39.1 / 31.3; 1024 of 1200
// 3.2 / 2.8, 5280 4.1 / 4.0; 50000 of 656 20.3 / 19.3, 1584 37.3 / 34.1, 7392 152.6 / 129.0.
static inline bool mw_rows_part(int64_t stride_bytes, int64_t n_rows)
{
    const int64_t bytes = stride_bytes * n_rows;
    return stride_bytes % 128 != 0 && (stride_bytes >= 2560 || bytes < 2 << 20 || bytes > 18 << 20);
}
// The same beside the expander's rows in a step's launch.  us, two steps of 8192 tokens over 8 ranks: rows of 272 bytes 76.3 / 77.6, 656 77.2 /
// 78.1, 1040 83.8 / 83.2, 2448 87.3 / 85.1, 7392 152.3 / 140.9.
static inline bool mw_step_rows_part(int64_t stride_bytes) { return stride_bytes % 128 != 0 && stride_bytes >= 1024; }
// The same for a relay's copies of up to n_rows rows or packets; `rides`: beside the index of the next buffer.  A copy scatters over
// several buffers.  Pieces that begin on 64 bytes are written through as well as whole lines: 15 hops, us, written through / not,
// relays of 8000 rows of 5824 bytes 67.5 / 70.4, of 14400 158.1 / 169.5, two of a stream 112.5 / 119.0 and 291.0 / 317.6, packets of 6464
// bytes 73.0 / 80.3; only short ones of packets (3136 bytes 43.4 / 41.4) and beside an index (3008 bytes 80.9 / 79.0) are not.  Other
// rows: relays of 4096 rows of 1056 bytes 15.8 / 15.1, of 272 bytes 12.2 / 12.4, of 1024 rows of 1584 bytes 9.6 / 10.0; packets of 400 bytes 15.4 /
// 12.7.
static inline bool mw_relay_rows_part(int64_t stride_bytes, int64_t n_rows, bool packets, bool rides)
{
    if (stride_bytes % 64 == 0) return stride_bytes % 128 != 0 && (packets || rides) && stride_bytes < 4096;
    return packets || stride_bytes * n_rows >= 2 << 20;
}

// Whether the expander of mw_unpack and mw_unpack_packets makes its places of the index's counts (k_expand_counts) or the index does.
// What adding them up costs in every wave grows with the payload, what the index saves does not (it grows with the peers: a report
// each), so there is a most of expected bytes.  Up to 256 counts are one a lane or four, one request of at most a kilobyte; up to 512
// eight, two requests.  A wave of a folded row has two payload chunks a lane that wait for the counts.  us for mw_plan, mw_pack and
// mw_unpack, added up by the index's last workgroup / by every wave:
//   384 counts, rows of 7424 bytes, 55 MB 40.1 / 38.5, 111 MB 64.3 / 63.4, 167 MB 86.8 / 87.1, 222 MB 108.3 / 109.7; of 4224 bytes (folded),
//     54 MB 46.9 / 44.7, 109 MB 72.9 / 71.6; of 2048 bytes, 123 MB 81.3 / 79.6.  512 counts of 128 ranks 32.5 / 30.0.
//   Folded rows of 4224 bytes, 256 ranks, 169 MB 86.7 / 84.0, 237 MB 111.3 / 110.0, 277 MB 125.0 / 125.2, 473 MB 227.4 / 231.1; 128 ranks, 203 MB
//     97.4 / 96.4, 250 MB 115.6 / 115.7, 277 MB 125.5 / 126.7; 64 ranks, 169 MB 84.8 / 83.8, 203 MB 97.0 / 96.9, 237 MB 111.2 / 111.6, 277 MB
//     126.6 / 127.5.  Of 8448 bytes, 256 ranks, 237 MB 107.7 / 105.6, 338 MB 144.2 / 144.8, 541 MB 215.2 / 225.4; 64 ranks, 203 MB 93.9 / 94.3.
//     Packets of 4352 bytes, 256 ranks, 203 MB 100.2 / 100.0, 237 MB 113.9 / 114.3, 250 MB 117.3 / 118.9; 64 ranks, 132 MB 74.4 / 73.9, 169 MB
//     86.4 / 86.5, 203 MB 99.5 / 100.2; 128 ranks, 169 MB 87.6 / 86.8, 203 MB 99.4 / 99.5.
//   The same of a rank with many experts, 1.2 hits a row and more, whose waves wait for their stores: 16 experts of 16 ranks, 226 MB 135.7 /
//     134.2, 441 MB 286.9 / 284.7; 20 of 12, 360 MB 249.5 / 248.1; 32 of 8, 313 MB 249.0 / 247.2; of 8448 bytes, 220 MB 119.8 / 120.0.
//   Other rows, 256 counts, 8192 bytes, 513 MB 228.5 / 227.8, 1002 MB 474.2 / 477.0; 14336 bytes, 705 MB 266.5 / 263.2, 897 MB 371.7 /
//     372.2; 128 counts, 8192 bytes, 522 MB 221.4 / 220.8, 764 MB 352.1 / 353.0, 1019 MB 472.5 / 474.9.
// A rank without experts has no counts that a lane could request.
constexpr int64_t kCountsMax = 512;
static inline bool mw_counts_by_expander(int64_t n_local, int64_t n_peers, bool packets, bool folded, double hits_a_row, int64_t expected_bytes)
{
    const int64_t n_counts = n_local * n_peers;
    const int64_t most_mib = n_counts > 256      ? 128
                             : !folded           ? 720
                             : hits_a_row >= 1.2 ? 448
                                                 : 160 + n_peers / 2 - (packets ? 56 : 0);
    return n_counts >= 1 && n_counts <= kCountsMax && expected_bytes <= most_mib << 20;
}

// Hash of a plan key (a bitmap of up to 64 ranks, or up to eight ranks a byte each) from its halves; its upper bits name a slot, bits
// 12 to 16 a bit.  Each half is multiplied before they meet: a rotated upper half xor'ed in folds three of 64 ranks onto 5000 values,
// so that most of 8192 tokens shared theirs with another key (mw_plan 71.9 us, with this 19.2; four ranks 23.2 / 16.7).
#ifdef __HIPCC__
__host__ __device__
#endif
static inline uint32_t mw_key_hash(uint32_t lo, uint32_t hi) { return (lo ^ hi * 0x9E3779B1u) * 0x85EBCA6Bu; }

// Tokens up to which k_plan_order makes the plan (beyond: sorted chunks), and from which k_groups works on
// row-indexed arrays; the workspace has the arrays of either only where a batch can need them.
constexpr int kPlanOrderMax = 8192, kPlanRowsFrom = 24576;
constexpr uint32_t kRideWaitDefault = 1u << 21;      // polls a riding plan's second half waits for its first

// Host-side context.  Every d_* pointer is a slice of the caller's workspace.
struct mw_ctx {
    mw_config cfg;
    int32_t n_local;        // L: experts hosted by my_rank
    int32_t hit_slots;      // Kd = max(1, min(K, L)): local experts one row can name
    int32_t mask_words;     // ceil(R / 64): bitmap words that can be non-zero
    int64_t x_row_bytes;    // payload part of a row
    int64_t s_row_bytes;    // scale part of a row (fp8) or 0
    int64_t row_bytes;
    int64_t row_stride;     // bytes from one row to the next in packed / received row arrays (>= row_bytes)
    int device;
    int n_cu;
    // workspace slices
    int32_t *d_eslot;       // [E] (rank << 16) | slot of expert e among the experts of its rank
    uint64_t *d_plan_cnt;       // [max_tokens] packed per-token counters; zero between plans
    uint32_t *d_plan_state;     // [MW_PLAN_STATE_WORDS] rows per destination, kept tokens, flags, workgroups done; zero between plans
    uint64_t *d_plan_keys;      // [min(max_tokens, 8192)] keys of the plan's two-launch form
    uint8_t *d_plan_idx;        // [min(max_tokens, 8192)] their tokens
    uint32_t *d_plan_bad;       // [64] its workgroups that saw an id outside the range
    uint64_t *d_sort_key;       // [max_tokens rounded up to 1024] sorted chunks of the large-batch plan (or null)
    uint32_t *d_sort_sec;       // same count: second sort word
    uint32_t *d_chunk_kept;     // [64] kept tokens per chunk
    uint64_t *d_row_cnt;        // [max_tokens] a packed row's counters (large-batch plan, or null)
    unsigned char *d_row_start; // [max_tokens] 1: a group starts at this packed row
    uint32_t ride_wait_limit;   // polls a riding plan's second half waits for its first
    uint32_t options;           // MW_OPT_*
    uint32_t *d_flags;      // [4] 1: receive flags, 2: receive workgroups done
    uint32_t *d_base;       // [L][R] first output row of (local expert, peer)
    mw_row_rec *d_recs;     // [max_recv_rows]
    uint32_t *d_cnt;        // [L][R] rows of peer p delivered to local expert le
    uint32_t *d_row_base;   // [R + 1] exclusive prefix of the peers' n_rows
    uint32_t *d_addr_cnt;   // [R] rows of peer p whose group names this rank
    mw_hit *d_hits;         // [max_recv_rows][Kd]
    int32_t *d_row_map;     // [max_tokens] mw_sim_deliver: kept row -> sender row
    int64_t recv_rows_hint; // rows the peers' buffers held at the last mw_get_recv_stats (0: unknown)
    // relay (only with cfg.max_hops > 0)
    int32_t n_hops;         // 0 until mw_set_forwarding
    uint64_t *d_hop_bits;   // [MW_MAX_HOPS][4] ranks served through each next hop
    int32_t *d_group_of_row;// [max_tokens]
    uint32_t *d_child_pos;  // [max_tokens][16, 32 or 64 by the hops] first child row of (group, hop) or kNoChild
    uint32_t *d_relay_flags;// flag word and the accounting sums behind it (mw_relay_acc)
    // measurement hook: optional event pairs recorded around single kernels
    hipEvent_t ev_start[MW_KERNEL_COUNT];
    hipEvent_t ev_stop[MW_KERNEL_COUNT];
};

// Records the context's timing events (if set) around one kernel launch.
struct mw_timed {
    mw_ctx *ctx; int k; hipStream_t s;
    mw_timed(mw_ctx *c, int kernel, hipStream_t st) : ctx(c), k(kernel), s(st)
    {
        if (ctx->ev_start[k]) (void)hipEventRecord(ctx->ev_start[k], s);
    }
    ~mw_timed()
    {
        if (ctx->ev_stop[k]) (void)hipEventRecord(ctx->ev_stop[k], s);
    }
};

#define MW_HIP_CHECK(expr)                         \
    do {                                           \
        hipError_t e_ = (expr);                    \
        if (e_ != hipSuccess) return MW_ERR_HIP;   \
    } while (0)

static inline int64_t mw_align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// Header in front of a packet's row: 4 bitmap words, source token, id count, the ids; whole
// 128-byte lines so that the row behind it starts on a cache line.
static inline int64_t mw_packet_header_bytes_of(int32_t top_k) { return mw_align_up(40 + 4 * (int64_t)top_k, 128); }

// ---- device helpers ---------------------------------------------------------------------
#ifdef __HIPCC__
// Streaming 16-byte accesses: payload rows are touched once, keep them out of the way of
// the small, reused index arrays.
__device__ __forceinline__ u32x4 mw_ld16(const u32x4 *p) { return __builtin_nontemporal_load(p); }
// The store is streaming and written through (sc0 sc1 nt): the lines leave the L2 as they are
// written, so the end of the kernel has nothing left to write back and the next launch on the
// stream starts about two microseconds sooner than with a plain non-temporal store.
__device__ __forceinline__ void mw_st16(u32x4 *p, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt" ::"v"(p), "v"(v) : "memory");
}
// The store of a row's chunk where rows are no whole number of cache lines apart.  Written through, a line of which a wave has only a
// part goes to memory by itself, and the other part again later; such rows have two of them in every wave's kilobyte.  They
// are stored streaming only, and the L2 puts the pieces of one CU together.  us for rows of 7392 bytes, written through /
// not: relay over 15 hops 44.5 / 42.0, a stream of relays 76.9 / 72.2 for two, of packets of 7520 bytes 47.4 / 43.4; a step of 4096
// such rows 92.4 / 89.6, mw_plan, mw_pack and mw_unpack 108.9 / 108.0; of 5280 bytes, relay 35.4 / 32.0.  Whole lines: relay of
// 7424 bytes 38.3 / 38.9.
__device__ __forceinline__ void mw_st16_part(u32x4 *p, u32x4 v)
{
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) u32x4 *)p);     // (global also where `p` was read from memory)
}
template <bool kPart>
__device__ __forceinline__ void mw_st16_as(u32x4 *p, u32x4 v)
{
    if constexpr (kPart) mw_st16_part(p, v);
    else mw_st16(p, v);
}
// The same load through a pointer that was read from memory: saying that it is a global
// address keeps it off the flat path, whose loads also count as LDS traffic and would make
// every later wait for a scalar load wait for the payload too.
typedef const __attribute__((address_space(1))) u32x4 *mw_gptr16;
__device__ __forceinline__ u32x4 mw_ld16_global(const void *row, int chunk)
{
    return __builtin_nontemporal_load((mw_gptr16)row + chunk);
}

// Wave-uniform values: "the value is needed in scalar registers here".  The compiler
// otherwise sinks every scalar load to its first use, one wait per load; pinning several
// values side by side makes it issue their loads together and wait once.
#define MW_PIN_S(x) asm volatile("" : "+s"(x))
#define MW_PIN_PTR(p) do { uint32_t lo_ = (uint32_t)(uintptr_t)(p); asm volatile("" : "+s"(lo_)); } while (0)
#define MW_PIN_S4(v) asm volatile("" : "+s"((v).x), "+s"((v).y), "+s"((v).z), "+s"((v).w))

// Workgroup barrier for data exchanged through LDS only.  __syncthreads() also waits until
// every global load and store of the wave has completed (about a microsecond each time a
// store or a prefetch is outstanding); this one orders LDS accesses and nothing else.
__device__ __forceinline__ void mw_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- publication between workgroups of ONE launch ------------------------------------------
// A workgroup that has produced (or finished reading) data another workgroup of the same launch
// depends on reports through a counter; the other side reads the counter and then the data.
//   producer   every lane: its stores / atomics;  mw_publish_barrier();  one lane: mw_report(counter)
//   consumer   one lane: reads the counter (mw_report's return value, or a poll followed by
//              mw_acquire_after_poll());  mw_consume_barrier();  every lane: reads the data
// Where ONE WAVE wrote all there is to publish its first lane reports behind mw_publish_wave(), while the other waves go on.
// If the report was the last the same wave may go on as the consumer without a workgroup barrier: mw_consume_wave()
// brings the counter's value from its first lane to all of them.  If its workgroup is to go on, that lane hands the value over
// in LDS and mw_consume_barrier() stands between it and every lane's reads, as above.
// In memory-model terms: the barrier orders every lane's accesses before the reporting lane's
// (workgroup scope); the report is a release (and, as a read-modify-write whose value decides who
// is last, an acquire) at agent scope; the consumer's counter read is an acquire at agent scope;
// happens-before is transitive over the two scopes, so everything the producer's lanes did is
// visible to every lane of the consumer after its barrier, whatever cache either side runs behind.
// (One wave: a release fence of every lane, the wave's barrier and an acquire take the place of the workgroup barrier in
// front of the report; behind it the wave's barrier and an agent-scope acquire fence of every lane.)
// The data itself is additionally written and read with agent-scope atomics, which are performed
// at the device's coherence point, so the release and acquire fences find next to nothing to
// write back or invalidate on their own account.
// MW_PUBLISH_FENCES 0 builds the same protocol from relaxed atomics and an explicit wait for all
// outstanding memory operations of every lane (s_waitcnt vmcnt(0)) in front of the barrier:
// correct on gfx950, where an agent-scope atomic or a write-through store is complete once
// acknowledged, but an argument about this hardware rather than about the memory model.
#ifndef MW_PUBLISH_FENCES
#define MW_PUBLISH_FENCES 0
#endif
__device__ __forceinline__ void mw_publish_barrier()
{
#if !MW_PUBLISH_FENCES
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    __syncthreads();
}
__device__ __forceinline__ uint32_t mw_report(uint32_t *counter)
{
#if MW_PUBLISH_FENCES
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
#else
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#endif
}
__device__ __forceinline__ void mw_publish_wave()
{
#if MW_PUBLISH_FENCES
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}
// `value`: what mw_report returned, in the wave's first lane.  Returns it in every lane.
__device__ __forceinline__ uint32_t mw_consume_wave(uint32_t value)
{
    value = (uint32_t)__builtin_amdgcn_readfirstlane((int)value);
#if MW_PUBLISH_FENCES
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#endif
    return value;
}
// Between the lane that read the counter and the lanes that read the data.  (LDS only without the fences: the wait for the
// counter's value is in front of the LDS write that says what it was.)
__device__ __forceinline__ void mw_consume_barrier()
{
#if MW_PUBLISH_FENCES
    __syncthreads();
#else
    mw_lds_barrier();
#endif
}
__device__ __forceinline__ void mw_acquire_after_poll()
{
#if MW_PUBLISH_FENCES
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#endif
}

// Scans and reductions inside a wave by data-parallel primitives: a shift inside rows of 16 lanes or a
// broadcast of one row's last lane into the next is an operand modifier of an ordinary vector
// instruction, where __shfl is a round trip through the LDS crossbar (six dependent ones a scan).
// With __shfl a block scan took 0.45-0.5 us, and every index and plan kernel is a chain of several:
// a 64-token stream step 10.5 -> 9.5 us, mw_plan + mw_pack + mw_unpack of 1000 fp8 tokens over 16 ranks
// 53.0 -> 50.7 us, of 4096 over 64 ranks 121.7 -> 118.8 us.
// Every lane of the wave must be active; lanes without a source keep the identity, 0.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t mw_dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRows, 0xf, false);
}
__device__ __forceinline__ uint32_t mw_row_incl_scan(uint32_t v)     // inside each row of 16 lanes
{
    v += mw_dpp<0x111, 0xf>(v);      // row_shr:1, 2, 4, 8
    v += mw_dpp<0x112, 0xf>(v);
    v += mw_dpp<0x114, 0xf>(v);
    v += mw_dpp<0x118, 0xf>(v);
    return v;
}
__device__ __forceinline__ uint32_t mw_wave_incl_scan(uint32_t v)
{
    v = mw_row_incl_scan(v);
    v += mw_dpp<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
    v += mw_dpp<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t mw_wave_sum(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)mw_wave_incl_scan(v), 63);
}
__device__ __forceinline__ uint32_t mw_wave_max(uint32_t v)
{
    v = max(v, mw_dpp<0x111, 0xf>(v));
    v = max(v, mw_dpp<0x112, 0xf>(v));
    v = max(v, mw_dpp<0x114, 0xf>(v));
    v = max(v, mw_dpp<0x118, 0xf>(v));
    v = max(v, mw_dpp<0x142, 0xa>(v));
    v = max(v, mw_dpp<0x143, 0xc>(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Exclusive prefix sum over one value per thread of a block (blockDim.x multiple of 64,
// at most 1024).  `wave_tot` is LDS scratch of 17 words.  Returns the exclusive prefix;
// *total receives the block total.  Ends with a barrier so the scratch can be reused.  The
// barriers order LDS only.  Every wave adds up the waves' totals for itself (one LDS read a
// lane and a 16-lane scan): a single thread walking them took a dependent LDS round trip per
// wave, a microsecond for 1024 lanes.
__device__ __forceinline__ uint32_t mw_block_exscan(uint32_t v, uint32_t *wave_tot, uint32_t *total)
{
    const int lane = threadIdx.x & 63, n_wave = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t inc = mw_wave_incl_scan(v);
    if (lane == 63) wave_tot[wave] = inc;
    mw_lds_barrier();
    const uint32_t t = mw_row_incl_scan((lane < n_wave) ? wave_tot[lane] : 0u);      // (at most 16 waves: one row)
    const uint32_t before = (wave > 0) ? (uint32_t)__builtin_amdgcn_readlane((int)t, wave - 1) : 0u;
    *total = (uint32_t)__builtin_amdgcn_readlane((int)t, n_wave - 1);
    mw_lds_barrier();
    return before + inc - v;
}
#endif

// payload and scale bytes of a row of `c` (checks the row format's constraints); returns a status
int32_t mw_row_geometry(const mw_config &c, int64_t *x_bytes, int64_t *s_bytes);

// kernels' host launchers (one per source file)
int32_t mw_launch_plan(mw_ctx *ctx, const int32_t *topk, int32_t T, uint64_t *mask, int32_t *perm,
                       mw_group_desc *desc, mw_send_stats *stats, hipStream_t s);
int32_t mw_launch_pack(mw_ctx *ctx, const void *x, const float *scales, const int32_t *topk,
                       const int32_t *perm, const mw_send_stats *stats, int32_t T, void *packed,
                       int32_t *row_src_token, int32_t *row_topk, hipStream_t s);
int32_t mw_launch_plan_pack(mw_ctx *ctx, const int32_t *topk, int32_t T, const void *x, const float *scales,
                            uint64_t *mask, int32_t *perm, mw_group_desc *desc, mw_send_stats *stats, void *packed,
                            int32_t *row_src_token, int32_t *row_topk, hipStream_t s);
int32_t mw_launch_unpack_index(mw_ctx *ctx, const void *peers, bool packets, int32_t P, int64_t cap,
                               int64_t *expert_offsets, mw_recv_stats *stats, hipStream_t s);
int32_t mw_launch_pack_quantize(mw_ctx *ctx, const void *x_bf16, const int32_t *topk, const int32_t *perm,
                                const mw_send_stats *stats, int32_t T, void *packed, int32_t *row_src_token,
                                int32_t *row_topk, hipStream_t s);
int32_t mw_launch_pack_packets(mw_ctx *ctx, const void *x, const float *scales, const int32_t *topk,
                               const uint64_t *mask, const int32_t *perm, const mw_send_stats *stats, int32_t T,
                               void *packets, hipStream_t s);
int32_t mw_launch_unpack_expand(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                int32_t *out_src_peer, int32_t *out_src_token, hipStream_t s);
int32_t mw_launch_unpack(mw_ctx *ctx, const mw_recv_peer *peers, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                         int32_t *out_src_peer, int32_t *out_src_token, int64_t *expert_offsets, mw_recv_stats *stats, hipStream_t s);
int32_t mw_launch_unpack_two(mw_ctx *ctx, const void *peers, bool packets, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                             int32_t *out_src_peer, int32_t *out_src_token, int64_t *expert_offsets, mw_recv_stats *stats, hipStream_t s);
int32_t mw_launch_unpack_expand_index_next(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                           int32_t *out_src_peer, int32_t *out_src_token, mw_ctx *next,
                                           const mw_recv_peer *next_peers, int32_t next_P, int64_t next_cap,
                                           int64_t *next_expert_offsets, mw_recv_stats *next_stats, hipStream_t s);
int32_t mw_launch_allgather_step(mw_ctx *ctx, const void *own_shard, int64_t shard_bytes, void *send_buf,
                                 mw_group_desc *desc, mw_send_stats *stats, const void *const *shards, void *out,
                                 hipStream_t s);
// the arguments of an mw_pack that rides in another launch (mw_stream_step)
struct mw_pack_call {
    const void *x; const float *scales; const int32_t *topk; const int32_t *perm; const mw_send_stats *stats;
    int32_t n_tokens; void *packed; int32_t *row_src_token; int32_t *row_topk;
};
int32_t mw_launch_unpack_expand_index_plan_next(mw_ctx *ctx, int32_t P, void *out_rows, float *out_scales, int64_t cap,
                                                int32_t *out_src_peer, int32_t *out_src_token, mw_ctx *next,
                                                const mw_recv_peer *next_peers, int32_t next_P, int64_t next_cap,
                                                int64_t *next_expert_offsets, mw_recv_stats *next_stats,
                                                const int32_t *next_topk, int32_t next_T, uint64_t *next_mask,
                                                int32_t *next_perm, mw_group_desc *next_desc,
                                                mw_send_stats *next_send_stats, const mw_pack_call *pack, hipStream_t s);
int32_t mw_launch_combine(mw_ctx *ctx, int32_t P, const void *y, int64_t cap, void *ret, int64_t ret_cap, hipStream_t s);
int32_t mw_launch_plan_allgather(mw_ctx *ctx, int64_t shard_bytes, mw_group_desc *desc,
                                 mw_send_stats *stats, hipStream_t s);
int32_t mw_launch_plan_allgather_split(mw_ctx *ctx, int64_t shard_bytes, int64_t direct_bytes, mw_group_desc *desc,
                                       mw_send_stats *stats, hipStream_t s);
int32_t mw_launch_gather_split(mw_ctx *ctx, const void *const *direct, const void *const *relayed,
                               int64_t shard_bytes, int64_t direct_bytes, void *out, hipStream_t s);
int32_t mw_launch_copy(mw_ctx *ctx, void *dst, const void *src, int64_t n_bytes, hipStream_t s);
int32_t mw_launch_gather_shards(mw_ctx *ctx, const void *const *shards, int64_t shard_bytes, void *out,
                                hipStream_t s);
int32_t mw_launch_relay_batch(const mw_relay_job *copy, int32_t n_copy, const mw_relay_job *index, int32_t n_index,
                              hipStream_t s);
int32_t mw_launch_relay(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children, int64_t cap,
                        mw_relay_stats *stats, hipStream_t s);
int32_t mw_launch_relay_index(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children, int64_t cap,
                              mw_relay_stats *stats, hipStream_t s);
int32_t mw_launch_relay_copy(mw_ctx *ctx, const mw_recv_peer *in, const mw_relay_child *children,
                             mw_relay_stats *stats, mw_ctx *next, const mw_recv_peer *next_in,
                             const mw_relay_child *next_children, int64_t next_cap, mw_relay_stats *next_stats,
                             hipStream_t s);
int32_t mw_launch_relay_packets_index(mw_ctx *ctx, const mw_recv_packets *in, int64_t cap, mw_relay_stats *stats,
                                      hipStream_t s);
int32_t mw_launch_relay_packets_copy(mw_ctx *ctx, const mw_recv_packets *in, void *const *children,
                                     mw_relay_stats *stats, mw_ctx *next, const mw_recv_packets *next_in,
                                     int64_t next_cap, mw_relay_stats *next_stats, hipStream_t s);
int32_t mw_launch_relay_packets(mw_ctx *ctx, const mw_recv_packets *in, void *const *children, int64_t cap,
                                mw_relay_stats *stats, hipStream_t s);
int32_t mw_launch_sim_deliver(mw_ctx *ctx, const mw_group_desc *desc, const mw_send_stats *stats,
                              int32_t T, const void *rows, const int32_t *src_token, const int32_t *topk,
                              int32_t dst_rank, mw_group_desc *desc_out, void *rows_out,
                              int32_t *src_token_out, int32_t *topk_out, uint32_t *counts, hipStream_t s);

#endif  // MW_INTERNAL_H_
