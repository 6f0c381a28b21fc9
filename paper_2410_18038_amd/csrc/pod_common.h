// Structures shared by the host planner and the gfx950 kernels.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define POD_HD __host__ __device__
#else
#define POD_HD
#endif

namespace pod {

constexpr int kWaveSize = 64;
constexpr int kWgThreads = 256;            // 4 wavefronts per workgroup, one per SIMD
constexpr int kWavesPerWg = 4;
constexpr int kDecodeStep = 16;            // decode units are cut at multiples of this many keys
// Shape of a prefill work item by head dimension.  Up to 128 channels a wavefront owns 32 packed
// (token, head-in-group) query rows and all output channels, a workgroup 128 rows, and K/V tiles
// hold 64 keys.  At 256 channels the accumulators and queries of 32 rows no longer fit a
// wavefront that shares its SIMD with another one, so two wavefronts share a row group: both
// compute its scores, each owns half of the output channels; a workgroup then covers 64 rows, and
// tiles hold 32 keys so that the four tile buffers still take 64 KB of LDS.
POD_HD constexpr int prefill_item_rows(int head_dim) { return head_dim == 256 ? 64 : 128; }
POD_HD constexpr int prefill_kv_tile(int head_dim) { return head_dim == 256 ? 32 : 64; }
// Keys per decode step of one wavefront: a step's K and V rows are one slot of the register ring
// (head_dim / 4 registers at 16 keys), which at 256 channels is halved to keep two slots.
POD_HD constexpr int decode_step_keys(int head_dim) { return head_dim == 256 ? 8 : 16; }
constexpr int kMaxGroup256 = 8;            // query heads per K/V head at head_dim 256 (the decode worker's query buffers)
constexpr int kMaxGroup = 16;              // query heads per K/V head a decode unit can hold
constexpr int kXcdQueues = 8;               // work is queued per XCD (one L2 each); a queue's counter is claimed mostly from its own XCD
constexpr int kSlotsPerUnit = 2;            // resident workgroups per compute unit (register and LDS budget)
constexpr int kChipUnits = 256;            // compute units of the chip (measured rules that hold for all of it)
constexpr int kCombineFetch = 8;            // splits a thread group of the combine kernel fetches together (independent loads)
constexpr int kCuSlots = 1024;             // hardware unit ids are sparse: (xcc << 6 | se << 4 | cu) < 1024

enum Role : int { kPrefill = 0, kDecode = 1, kNone = -1 };

// Cache layouts the kernels are specialised for: contiguous; paged with a power-of-two block size
// of at least 16 (a 16-key step then lies in one block, found with one scalar lookup and shifts);
// paged with any block size that is a multiple of the rows one load instruction covers (8, 4 or 2
// rows at 64, 128 or 256 channels: every load then lies in one block and block ids stay scalar, one
// per load); paged, any (a block id per lane, looked up with vector loads that the K/V loads wait for).
// Blocks of 24 keys, 15 / 5 heads, 2 chunks + 40 decodes at 0.5K-7K: 199 us by lane, 94 by row.
enum Layout : int { kLayoutContiguous = 0, kLayoutPaged16 = 1, kLayoutPagedRows = 2, kLayoutPagedAny = 3 };
inline Layout cache_layout(int block_size, int head_dim, int n_kv_heads)
{
    if (block_size <= 0) return kLayoutContiguous;
    // (byte offsets inside a block are 32 bits wide there)
    const bool small = (int64_t)block_size * n_kv_heads * head_dim * 2 < (int64_t)1 << 32;
    if (block_size >= 16 && (block_size & (block_size - 1)) == 0 && small) return kLayoutPaged16;
    return block_size % (kWaveSize / (head_dim / 8)) == 0 ? kLayoutPagedRows : kLayoutPagedAny;
}
// What the two kernels of the prefill-heavy configuration are built for.
inline bool built_for_prefill_heavy(int block_size, int head_dim, int n_kv_heads)
{
    const Layout layout = cache_layout(block_size, head_dim, n_kv_heads);
    return head_dim == 128 && (layout == kLayoutContiguous || layout == kLayoutPaged16);
}

// One prefill work item: a block of packed query rows of one K/V head over a key range.
// Packed row R of a request stands for token R / group, query head kv_head * group + R % group,
// so that the heads sharing a K/V head also share each staged K/V tile (Section 4.2.1 notes the
// query tile grows by the group size under grouped-query attention).
struct PrefillItem {
    int32_t req, kv_head, row0, n_rows;
    int32_t kv_begin, kv_end;              // keys [kv_begin, kv_end); causal limit applied inside
    int32_t prow0;                         // first partial row, or -1 when the item writes `out`
    int32_t split;
};

// One decode work unit: all query heads of one K/V head of one request over a token range.
// One wavefront runs it (the "virtual CTA" of Section 4.2.3).
struct DecodeUnit {
    int32_t req, kv_head, t0, t1;
    int32_t prow0;                         // first partial row (group rows), or -1
    int32_t split;                         // in the device's table, where units merge their groups, with the number of
                                           // splits << kSplitBits added
    int32_t q_start, cache_row;            // copied from the request: a unit starts with one lookup
};
constexpr int kMergeSplits = 8;            // the last unit of a group merges it itself up to this many splits,
constexpr int kMergeRows = 8;              // query heads
constexpr int kMergeDim = 128;             // and channels
constexpr int kSplitBits = 24;

// One group of output rows merged from split partials (host only; the kernel reads CombineRows).
struct CombineEntry {
    int32_t kind;                          // kPrefill or kDecode
    int32_t kv_head, row0, n_rows;
    int32_t n_splits, prow0, split_stride; // partial row of split s, row r: prow0 + s*split_stride + r
    int32_t q_start;                       // of the request
};

// One merged output row as the combine kernel reads it: everything in one 16-byte lookup.
struct CombineRow {
    int32_t prow;                          // partial row of split 0; split s is one item's or unit's rows further
    int32_t n_splits;
    uint32_t out_row_lo, out_row_hi;       // row of `out` counted in heads (token row * n_q_heads + query head);
                                           // the top bit is set for a decode row
};

// Counters at the head of the device workspace.  All zero between calls: the combine kernel, or in calls
// without one the last workgroup of the attention kernel, clears them.  Counters that many workgroups add to have a 128-byte
// line each: the memory system serves one atomic per line every 11 ns, whichever word it names
// (measured: 512 workgroups adding to eight words of one line take 7.4 us, on eight lines 2.7).
struct WsHeader {
    // Per compute unit: workgroups that have arrived on it so far in this launch (the ticket of
    // Section 4.1's listing).
    uint32_t cu_state[kCuSlots];
    uint32_t next_id[2][32];               // [op][0]: next decode seat; next work id of either operation (CTA-parallel launch)
    uint32_t done[2][32];                  // [0][0]: workgroups that have finished
    // Next prefill item of each per-XCD queue (offset inside the queue), claimed by workgroups.
    uint32_t next_pitem_xcd[kXcdQueues][32];
    // Next decode unit of each per-XCD queue (offset inside the queue), claimed by wavefronts.
    uint32_t next_dunit_xcd[kXcdQueues][32];
    // Units that have stored their partials, for the groups of a plan whose last units merge: the counter of a group
    // is the word whose index is its first decode partial row (one round of the chip's wavefronts has up to 1024 units of
    // kMergeRows rows, half of this).  The unit that merges clears it.
    uint32_t arrived[512 * 32];
};

// Set in the counter of an XCD's decode queue once a wavefront of that XCD has found every queue used up.
constexpr int kAllQueuesEmpty = 1 << 30;

// Which operation the workgroup holding `ticket` on hardware unit `unit` starts with: the ticket
// rule of Section 4.1 (ticket mod (p + d) < p means prefill).  A unit holds only kSlotsPerUnit
// workgroups at a time, so its own tickets would never get past the first entries of a longer
// pattern; unit u therefore counts from kSlotsPerUnit * u, which spreads the pattern over the
// chip (4:1 puts a decode workgroup on every fifth slot; 1:1 still gives every unit one of each).
// The workgroups of the fused kernel arrive together and stay until the work is done, so the
// ticket alone decides: the split does not depend on which of two simultaneous arrivals is seen
// first, and there is no departure to account for.
POD_HD inline int role_for_ticket(uint32_t ticket, int p, int d, int unit = 0)
{
    const int t = (int)(ticket & 0xfffffu) + kSlotsPerUnit * unit;
    return (t % (p + d)) < p ? kPrefill : kDecode;
}

// How the workgroups of a fused launch get their operation: by ticket (above), or, in a launch whose
// items and decode workers all fit the chip at once, by their index, prefill items or decode seats first.
enum RoleRule : int { kRolesByTicket = 0, kPrefillFirst = 1, kDecodeFirst = 2 };

// What workgroup b does under the second rule: prefill item (of the workgroup order) below n_pitems,
// decode seat + n_pitems from there on (workgroups beyond the last seat have nothing to do).
POD_HD inline int fixed_piece(int rule, int b, int n_pitems, int n_dwgs)
{
    if (rule == kPrefillFirst) return b;
    return b < n_dwgs ? n_pitems + b : b < n_dwgs + n_pitems ? b - n_dwgs : b;
}

// Optional execution trace: where each workgroup of an attention kernel ran, which operation it
// took first, when it switched to the other one and how many work items it processed in each.
struct TraceRecord {
    int32_t cu;                            // hardware unit id (xcc << 6 | se << 4 | cu)
    int32_t first_role;                    // kPrefill or kDecode
    int32_t n_first, n_second;             // items done in the first role, then in the other one
    uint64_t t_begin, t_switch, t_end;     // constant-rate device clock (100 MHz)
    uint64_t pad;
};

// Optional event log: one record per prefill item (written by the workgroup) and per decode unit
// (written by the wavefront).  The log starts with a 16-byte header whose first word counts the
// records appended so far; records beyond the capacity are counted but not stored.
struct EventRecord {
    int32_t kind;                          // kPrefill or kDecode
    int32_t item;                          // prefill item or decode unit index
    int32_t cu;                            // hardware unit id
    int32_t wg;                            // workgroup index * 4 + wavefront
    uint64_t t_begin, t_end;               // constant-rate device clock (100 MHz)
};

// Everything a kernel needs; passed by value.
struct KernelArgs {
    const void *prefill_q, *decode_q, *k_cache, *v_cache;
    const int32_t *seq_meta, *block_table;
    void *out;
    const PrefillItem *pitems;
    const PrefillItem *pitems_by_wg;       // the same items in workgroup order, for the kernels that run item blockIdx.x
    const int32_t *pitem_of_wg;            // their indices in `pitems` (what the event log names)
    const DecodeUnit *dunits;
    const CombineRow *crows;
    float *part_o;                         // [n_partial_rows][d]  un-normalised fp32 output
    float *part_ml;                        // [n_partial_rows][2]  running max (log2 domain), weight sum
    WsHeader *hdr;
    TraceRecord *trace;                    // optional: one record per workgroup of the attention kernels
    uint32_t *arrived;                     // decode units merge their groups (WsHeader::arrived), or null: the combine kernel does
    uint32_t *evlog;                       // optional: event log (16-byte header, then EventRecords)
    uint32_t evlog_cap;                    // records the event log can hold
    int64_t kv_seq_stride;
    // Cache strides in elements, the same three for the token-major and the head-major order:
    // between consecutive tokens of one head, between the heads of a sequence (or of a block), and
    // between blocks of a paged cache.
    int64_t head_stride, block_elems;
    int32_t tok_stride;
    int32_t n_prefill, n_q_heads, n_kv_heads, group;
    int32_t block_size, max_blocks_per_seq;
    int32_t bs_shift;                      // log2(block_size) when it is a power of two, else -1
    uint32_t bs_magic;                     // ceil(2^32 / block_size) for block sizes above 1 (block_of)
    int32_t n_crows, n_crows_prefill;      // merged rows, and how many of them (the first ones) are prefill rows
    int32_t combine_groups[2];             // [op]: thread groups of the combine kernel that share a row's splits
    int32_t n_pitems, n_dunits, n_dwgs;      // n_dwgs: decode worker workgroups
    int32_t n_prefill_rows;
    int32_t decode_prow0;                  // first decode partial row
    int32_t fused_grid;
    int32_t pq_begin[kXcdQueues + 1];      // prefill queue q holds items pq_begin[q] .. pq_begin[q+1]-1
    const int32_t *dq_begin;               // [kXcdQueues + 1]: decode queue q holds units dq_begin[q] .. dq_begin[q+1]-1
    int32_t n_static_seats;                // decode seats that start with four fixed units (units 0 .. 4*seats-1)
    int32_t n_dctas;                       // decode workgroups of the CTA-parallel launch: ceil(n_dunits / 4)
    int32_t combine_resets;                // the combine kernel of this call clears the counters, not the attention kernel
    int32_t single_unit;                   // a decode wavefront runs its fixed unit and claims none, whatever the queues hold
    int32_t fixed_roles;                   // CTA-parallel kernel: a RoleRule
    int32_t p_ratio, d_ratio;
    float scale_log2;                      // softmax_scale * log2(e)
};

}  // namespace pod
