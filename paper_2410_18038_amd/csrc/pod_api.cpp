// C ABI of the library (see include/pod_attn.h).
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/pod_attn.h"
#include "pod_common.h"
#include "pod_launch.h"
#include "pod_planner.h"

struct pod_attn_plan {
    pod::Plan p;
    uint64_t serial = 0;                    // unique per plan object of this process, never reused
};

namespace {

thread_local std::string g_last_error;
std::atomic<uint64_t> g_next_plan_serial{1};

// Which plan's work tables each GPU's static scratch holds (0 = none), for pod_attn_forward_static.
constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
uint64_t g_static_owner[kMaxDevices] = {0};

pod_status fail(pod_status code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

pod_status fail_hip(hipError_t e, const char *what)
{
    return fail(POD_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

int device_cu_count()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return 256; }
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return 256;
    }
    return n;
}

pod::KernelArgs make_args(const pod::Plan &p, const void *prefill_q, const void *decode_q,
                          const void *k_cache, const void *v_cache, const int32_t *seq_meta,
                          const int32_t *block_table, void *out, void *workspace)
{
    pod::KernelArgs a;
    std::memset(&a, 0, sizeof a);
    unsigned char *ws = (unsigned char *)workspace;
    a.prefill_q = prefill_q; a.decode_q = decode_q; a.k_cache = k_cache; a.v_cache = v_cache;
    a.seq_meta = seq_meta; a.block_table = block_table; a.out = out;
    a.hdr = (pod::WsHeader *)ws;
    a.pitems = (const pod::PrefillItem *)(ws + p.off_pitems);
    a.pitems_by_wg = (const pod::PrefillItem *)(ws + p.off_pitems_by_wg);
    a.pitem_of_wg = (const int32_t *)(ws + p.off_pitem_of_wg);
    a.dunits = (const pod::DecodeUnit *)(ws + p.off_dunits);
    a.crows = (const pod::CombineRow *)(ws + p.off_crows);
    a.n_crows = (int)p.merge_rows.size();
    a.n_crows_prefill = p.n_crows_prefill;
    for (int op : {pod::kPrefill, pod::kDecode}) a.combine_groups[op] = p.combine_groups[op];
    a.part_o = (float *)(ws + p.off_part_o);
    a.part_ml = (float *)(ws + p.off_part_ml);
    a.kv_seq_stride = p.prm.kv_seq_stride;
    {
        const int64_t d = p.prm.head_dim, hkv = p.prm.n_kv_heads, bs = p.prm.block_size;
        a.block_elems = bs * hkv * d;
        if (p.prm.kv_order == POD_KV_HEAD_MAJOR) {
            a.tok_stride = (int32_t)d;
            a.head_stride = bs > 0 ? bs * d : p.prm.kv_seq_stride / (hkv * d) * d;
        } else {
            a.tok_stride = (int32_t)(hkv * d);
            a.head_stride = d;
        }
    }
    a.n_prefill = p.prm.n_prefill;
    a.n_q_heads = p.prm.n_q_heads;
    a.n_kv_heads = p.prm.n_kv_heads;
    a.group = p.group;
    a.block_size = p.prm.block_size;
    a.max_blocks_per_seq = p.prm.max_blocks_per_seq;
    a.bs_shift = -1;
    if (p.prm.block_size > 0 && (p.prm.block_size & (p.prm.block_size - 1)) == 0) {
        int s = 0;
        while ((1 << s) < p.prm.block_size) ++s;
        a.bs_shift = s;
    }
    if (p.prm.block_size > 1) a.bs_magic = (uint32_t)(((uint64_t(1) << 32) + (uint64_t)p.prm.block_size - 1) / (uint64_t)p.prm.block_size);
    a.n_pitems = (int)p.pitems.size();
    a.n_dunits = (int)p.dunits.size();
    a.n_dwgs = p.n_dwgs;
    a.fused_grid = p.fused_grid;
    for (int q = 0; q <= pod::kXcdQueues; ++q) a.pq_begin[q] = p.pq_begin[q];
    // Every workgroup of a launch with decode work asks for a decode seat sooner or later and the
    // grid is never smaller than the number of seats, so all fixed units are run whatever
    // operation the workgroups start with.
    a.dq_begin = (const int32_t *)(ws + p.off_dq);
    // Units for one round of wavefronts or fewer are all run as fixed units, also the last up to three, which
    // the plan keeps in the queues: unit 4 * seat + v on wavefront v, and no wavefront claims anything.
    a.single_unit = a.n_dunits <= pod::kWavesPerWg * p.n_cus;
    a.n_static_seats = a.single_unit ? p.n_dwgs : p.n_static_seats;
    a.n_dctas = ((int)p.dunits.size() + pod::kWavesPerWg - 1) / pod::kWavesPerWg;
    a.fixed_roles = pod::kRolesByTicket;
    a.n_prefill_rows = (int)p.n_prefill_rows;
    a.decode_prow0 = (int)p.decode_prow0;
    a.p_ratio = p.p_ratio;
    a.d_ratio = p.d_ratio;
    a.scale_log2 = p.prm.softmax_scale * 1.4426950408889634f;
    a.trace = (pod::TraceRecord *)p.trace;
    a.evlog = (uint32_t *)p.evlog;
    a.evlog_cap = p.evlog ? (uint32_t)((p.evlog_bytes - 16) / sizeof(pod::EventRecord)) : 0u;
    return a;
}

// The two streams the two-kernel modes run their kernels on: one pair per GPU, created when it is first
// needed and kept until the process ends.  (A pair per plan would be spread over the few hardware queues a process
// has in creation order, and a later plan's pair can land on one queue, where its two kernels run one after the other.
// A second pair for the calls that take two kernels by themselves did: 1350 us instead of 1130.)
// Calls that ask for two streams share the pair, whoever makes them.  A fused call must not wait for what another
// stream does, so it takes two kernels by itself only while the pair holds no work of another caller's stream.
struct SideStreams {
    std::mutex enqueue;                     // held while a call enqueues: a wait refers to what its event was last recorded for
    hipStream_t st[2] = {};
    hipStream_t caller = nullptr;           // stream of the last call that enqueued here
};
SideStreams g_side[kMaxDevices];
std::mutex g_side_mu;                       // creation of streams, and the events of plans

// Creates what a two-kernel call of plan p needs on the current device.
pod_status ensure_side(pod::Plan &p, int *device)
{
    hipError_t e = hipGetDevice(device);
    if (e != hipSuccess) return fail_hip(e, "asking for the current device");
    if (*device < 0 || *device >= kMaxDevices) return fail(POD_ERR_UNSUPPORTED, "device index beyond what the library tracks");
    std::lock_guard<std::mutex> lock(g_side_mu);
    for (hipStream_t &st : g_side[*device].st)
        if (!st) {
            e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
            if (e != hipSuccess) { st = nullptr; return fail_hip(e, "creating side stream"); }
        }
    for (void *&ev : p.events)
        if (!ev) {
            hipEvent_t ne;
            e = hipEventCreateWithFlags(&ne, hipEventDisableTiming);
            if (e != hipSuccess) return fail_hip(e, "creating event");
            ev = ne;
            p.events_device = *device;
        }
    return POD_OK;
}

// May this fused call take the prefill-heavy configuration?  Then the lock that lets it enqueue on the pair is in
// `hold`.  Not where the records of the fused kernel are asked for, where streams or events would have to be
// created first, where a launch is being recorded (graph capture), or where the work would run otherwise on the side
// streams than on s: with a compute-unit mask or a priority of its own, or behind another stream's work.
bool heavy_is_ready(const pod::Plan &p, hipStream_t s, std::unique_lock<std::mutex> &hold)
{
    if (!p.heavy_pays || p.trace || p.evlog || s == hipStreamPerThread) return false;   // (that handle names many streams)
    auto usable = [&]() -> bool {
        int dev = -1, priority = 0, units = 0;
        uint32_t mask[pod::kChipUnits / 32] = {};
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
        {
            std::lock_guard<std::mutex> lock(g_side_mu);
            if (!p.events[2] || p.events_device != dev) return false;
        }
        auto recorded = [](hipStream_t x) {
            hipStreamCaptureStatus status = hipStreamCaptureStatusActive;
            return hipStreamIsCapturing(x, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
        };
        if (recorded(s) || hipStreamGetPriority(s, &priority) != hipSuccess || priority != 0 ||
            hipExtStreamGetCUMask(s, pod::kChipUnits / 32, mask) != hipSuccess)
            return false;
        for (uint32_t word : mask) units += __builtin_popcount(word);
        if (units != pod::kChipUnits) return false;
        SideStreams &side = g_side[dev];
        hold = std::unique_lock<std::mutex>(side.enqueue);
        if (side.caller != s)
            for (hipStream_t st : side.st)
                if (recorded(st) || hipStreamQuery(st) != hipSuccess) return false;
        side.caller = s;
        return true;
    };
    if (usable()) return true;
    (void)hipGetLastError();
    if (hold.owns_lock()) hold.unlock();
    return false;
}

// Clear the counters at the head of `workspace` (with a kernel, not a memset) and copy the plan's
// work tables behind them; returns when the copies have completed.
pod_status upload_tables(const pod::Plan &p, void *workspace, hipStream_t s)
{
    unsigned char *ws = (unsigned char *)workspace;
    hipError_t e = pod::clear_header((pod::WsHeader *)ws, s);
    if (e != hipSuccess) return fail_hip(e, "clearing workspace counters");
    struct Part { size_t off; const void *src; size_t bytes; };
    const Part parts[6] = {                                  // in the order they lie in
        {p.off_pitems, p.pitems.data(), p.pitems.size() * sizeof(pod::PrefillItem)},
        {p.off_pitems_by_wg, p.pitems_by_wg.data(), p.pitems_by_wg.size() * sizeof(pod::PrefillItem)},
        {p.off_pitem_of_wg, p.pitem_of_wg.data(), p.pitem_of_wg.size() * sizeof(int32_t)},
        {p.off_dunits, p.dunits.data(), p.dunits.size() * sizeof(pod::DecodeUnit)},
        {p.off_crows, p.merge_rows.data(), p.merge_rows.size() * sizeof(pod::CombineRow)},
        {p.off_dq, p.dq_begin, sizeof p.dq_begin}};
    // The tables lie behind each other in the workspace: one copy.  (Six before: preparing 48 decodes + 3
    // chunks took 143 us, 95 now; 32 decodes at 32K + a chunk 181, now 128.)
    const size_t bytes = p.off_part_o - p.off_pitems;
    const std::unique_ptr<unsigned char[]> tables(new (std::nothrow) unsigned char[bytes]);
    if (!tables) return fail(POD_ERR_INVALID_ARG, "out of host memory");
    size_t end = 0;                                          // the gaps up to the alignment of each table are cleared
    for (const Part &part : parts) {
        const size_t begin = part.off - p.off_pitems;
        std::memset(tables.get() + end, 0, begin - end);
        if (part.bytes > 0) std::memcpy(tables.get() + begin, part.src, part.bytes);
        end = begin + part.bytes;
    }
    std::memset(tables.get() + end, 0, bytes - end);
    pod::DecodeUnit *units = (pod::DecodeUnit *)(tables.get() + (p.off_dunits - p.off_pitems));
    for (size_t i = 0; i < p.unit_splits.size(); ++i) units[i].split |= p.unit_splits[i] << pod::kSplitBits;
    e = hipMemcpyAsync(ws + p.off_pitems, tables.get(), bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) { (void)hipStreamSynchronize(s); return fail_hip(e, "copying plan tables"); }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "waiting for plan upload");
    return POD_OK;
}

}  // namespace

extern "C" {

const char *pod_attn_last_error(void) { return g_last_error.c_str(); }
const char *pod_attn_version(void) { return "pod_attn 0.1 (gfx950)"; }

pod_status pod_attn_plan_create(const pod_attn_params *params, const int32_t *seq_meta_host,
                                pod_attn_plan **plan)
{
    if (!params || !plan) return fail(POD_ERR_INVALID_ARG, "params or plan is null");
    *plan = nullptr;
    const int n_cus = params->n_compute_units > 0 ? params->n_compute_units : device_cu_count();
    pod_attn_plan *obj = new (std::nothrow) pod_attn_plan();
    if (!obj) return fail(POD_ERR_INVALID_ARG, "out of host memory");
    std::string err;
    pod_status st;
    try {
        st = pod::build_plan(*params, seq_meta_host, n_cus, obj->p, err);
    } catch (const std::bad_alloc &) {
        st = POD_ERR_INVALID_ARG;
        err = "out of host memory";
    }
    if (st != POD_OK) {
        delete obj;
        return fail(st, err);
    }
    obj->serial = g_next_plan_serial.fetch_add(1);
    *plan = obj;
    return POD_OK;
}

void pod_attn_plan_destroy(pod_attn_plan *plan)
{
    if (!plan) return;
    for (void *&e : plan->p.events)
        if (e) { (void)hipEventDestroy((hipEvent_t)e); e = nullptr; }
    delete plan;
}

pod_status pod_attn_plan_info_get(const pod_attn_plan *plan, pod_attn_plan_info *info)
{
    if (!plan || !info) return fail(POD_ERR_INVALID_ARG, "plan or info is null");
    const pod::Plan &p = plan->p;
    info->n_prefill_items = (int32_t)p.pitems.size();
    info->n_decode_units = (int32_t)p.dunits.size();
    info->n_combine = (int32_t)p.centries.size();
    info->max_prefill_splits = p.max_psplits;
    info->max_decode_splits = p.max_dsplits;
    info->decode_chunk = p.decode_chunk;
    info->prefill_ratio = p.p_ratio;
    info->decode_ratio = p.d_ratio;
    info->fused_grid = p.fused_grid;
    info->n_compute_units = p.n_cus;
    info->n_prefill_rows = p.n_prefill_rows;
    info->n_partial_rows = p.n_partial_rows;
    info->workspace_bytes = (int64_t)p.ws_bytes;
    info->prefill_heavy_advised = p.heavy_advised ? 1 : 0;
    info->prefill_heavy_chosen = p.heavy_pays ? 1 : 0;
    return POD_OK;
}

pod_status pod_attn_plan_set_trace(pod_attn_plan *plan, void *trace, size_t trace_bytes)
{
    if (!plan) return fail(POD_ERR_INVALID_ARG, "plan is null");
    // one record per workgroup of the largest launch: the two stand-alone kernels together, or the fused round
    const size_t n_dctas = (plan->p.dunits.size() + pod::kWavesPerWg - 1) / pod::kWavesPerWg;
    const size_t n_records = std::max(plan->p.pitems.size() + n_dctas, (size_t)plan->p.fused_grid);
    const size_t need = n_records * sizeof(pod::TraceRecord);
    if (trace && trace_bytes < need) return fail(POD_ERR_WORKSPACE, "trace buffer too small");
    plan->p.trace = trace;
    plan->p.trace_bytes = trace ? trace_bytes : 0;
    return POD_OK;
}

pod_status pod_attn_plan_set_event_log(pod_attn_plan *plan, void *log, size_t log_bytes)
{
    if (!plan) return fail(POD_ERR_INVALID_ARG, "plan is null");
    if (log && log_bytes < 16 + sizeof(pod::EventRecord)) return fail(POD_ERR_WORKSPACE, "event log too small");
    if (log && ((uintptr_t)log & 15)) return fail(POD_ERR_INVALID_ARG, "event log must be 16-byte aligned");
    plan->p.evlog = log;
    plan->p.evlog_bytes = log ? log_bytes : 0;
    return POD_OK;
}

size_t pod_attn_workspace_size(const pod_attn_plan *plan) { return plan ? plan->p.ws_bytes : 0; }

pod_status pod_attn_plan_prefill_item(const pod_attn_plan *plan, int32_t index, int32_t out[8])
{
    if (!plan || !out || index < 0 || index >= (int32_t)plan->p.pitems.size())
        return fail(POD_ERR_INVALID_ARG, "prefill item index out of range");
    const pod::PrefillItem &it = plan->p.pitems[(size_t)index];
    const int32_t v[8] = {it.req, it.kv_head, it.row0, it.n_rows, it.kv_begin, it.kv_end, it.prow0, it.split};
    std::memcpy(out, v, sizeof v);
    return POD_OK;
}

pod_status pod_attn_plan_prefill_item_of_workgroup(const pod_attn_plan *plan, int32_t workgroup, int32_t out[8])
{
    if (!plan || !out || workgroup < 0 || workgroup >= (int32_t)plan->p.pitems_by_wg.size())
        return fail(POD_ERR_INVALID_ARG, "workgroup index out of range");
    const pod::PrefillItem &it = plan->p.pitems_by_wg[(size_t)workgroup];
    const int32_t v[8] = {it.req, it.kv_head, it.row0, it.n_rows, it.kv_begin, it.kv_end, it.prow0, it.split};
    std::memcpy(out, v, sizeof v);
    return POD_OK;
}

pod_status pod_attn_plan_decode_unit(const pod_attn_plan *plan, int32_t index, int32_t out[8])
{
    if (!plan || !out || index < 0 || index >= (int32_t)plan->p.dunits.size())
        return fail(POD_ERR_INVALID_ARG, "decode unit index out of range");
    const pod::DecodeUnit &u = plan->p.dunits[(size_t)index];
    const int32_t v[8] = {u.req, u.kv_head, u.t0, u.t1, u.prow0, u.split, u.q_start, u.cache_row};
    std::memcpy(out, v, sizeof v);
    return POD_OK;
}

pod_status pod_attn_plan_decode_queue(const pod_attn_plan *plan, int32_t q, int32_t *begin, int32_t *end)
{
    if (!plan || !begin || !end || q < 0 || q >= pod::kXcdQueues)
        return fail(POD_ERR_INVALID_ARG, "decode queue index out of range");
    *begin = plan->p.dq_begin[q];
    *end = plan->p.dq_begin[q + 1];
    return POD_OK;
}

pod_status pod_attn_plan_upload(const pod_attn_plan *plan, void *workspace, size_t workspace_bytes,
                                void *stream)
{
    if (!plan) return fail(POD_ERR_INVALID_ARG, "plan is null");
    const pod::Plan &p = plan->p;
    if (!workspace || workspace_bytes < p.ws_bytes) return fail(POD_ERR_WORKSPACE, "workspace missing or too small");
    if (((uintptr_t)workspace & 255u) != 0) return fail(POD_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    const pod_status st = upload_tables(p, workspace, (hipStream_t)stream);
    // What a fused call of this plan needs to take the prefill-heavy configuration is made here, so that the call itself
    // creates nothing.  Without it the fused kernel runs.
    int dev = -1;
    if (st == POD_OK && p.heavy_pays && ensure_side(const_cast<pod_attn_plan *>(plan)->p, &dev) != POD_OK) (void)hipGetLastError();
    return st;
}

static pod_status forward_impl(const void *prefill_q, const void *decode_q, const void *k_cache,
                               const void *v_cache, const int32_t *seq_meta, const int32_t *block_table,
                               void *out, const pod_attn_plan *plan, void *workspace,
                               size_t workspace_bytes, int32_t mode, void *stream, bool use_static)
{
    if (!plan) return fail(POD_ERR_INVALID_ARG, "plan is null");
    pod::Plan &p = const_cast<pod_attn_plan *>(plan)->p;
    const bool paged = p.prm.block_size > 0;
    const int n_req = p.prm.n_prefill + p.prm.n_decode;
    const bool no_combine = (mode & POD_MODE_FLAG_NO_COMBINE) != 0;
    const bool cta_parallel = (mode & POD_MODE_FLAG_CTA_PARALLEL) != 0;
    const bool heavy = (mode & POD_MODE_FLAG_PREFILL_HEAVY) != 0;
    mode &= ~(POD_MODE_FLAG_NO_COMBINE | POD_MODE_FLAG_CTA_PARALLEL | POD_MODE_FLAG_PREFILL_HEAVY);
    if (heavy && cta_parallel) return fail(POD_ERR_INVALID_ARG, "POD_MODE_FLAG_PREFILL_HEAVY and POD_MODE_FLAG_CTA_PARALLEL exclude each other");
    if (heavy && mode != POD_MODE_FUSED && mode != POD_MODE_DECODE_ONLY && mode != POD_MODE_PREFILL_ONLY)
        return fail(POD_ERR_INVALID_ARG, "POD_MODE_FLAG_PREFILL_HEAVY goes with POD_MODE_FUSED (or with one operation alone)");
    if (cta_parallel && mode != POD_MODE_FUSED)
        return fail(POD_ERR_INVALID_ARG, "POD_MODE_FLAG_CTA_PARALLEL goes with POD_MODE_FUSED only");
    if (mode < POD_MODE_FUSED || mode > POD_MODE_DECODE_ONLY) return fail(POD_ERR_INVALID_ARG, "unknown mode");
    if (n_req == 0) return POD_OK;
    if (!k_cache || !v_cache || !seq_meta || !out) return fail(POD_ERR_INVALID_ARG, "k_cache, v_cache, seq_meta or out is null");
    if (p.prm.n_prefill > 0 && !prefill_q) return fail(POD_ERR_INVALID_ARG, "prefill_q is null");
    if (p.prm.n_decode > 0 && !decode_q) return fail(POD_ERR_INVALID_ARG, "decode_q is null");
    if (paged && !block_table) return fail(POD_ERR_INVALID_ARG, "block_table is null for a paged cache");
    if (heavy && !pod::built_for_prefill_heavy(p.prm.block_size, p.prm.head_dim, p.prm.n_kv_heads))
        return fail(POD_ERR_UNSUPPORTED, "the prefill-heavy configuration is built for head_dim 128 and contiguous or "
                                         "power-of-two (>= 16) block caches, with blocks of less than 4 GB");
    if (use_static) {
        if (mode == POD_MODE_STREAMS || (heavy && mode == POD_MODE_FUSED))
            return fail(POD_ERR_UNSUPPORTED, "the two-stream mode creates streams and events; it is not available "
                                             "from the entry point that allocates nothing");
        if (p.ws_bytes > pod::kStaticScratchBytes)
            return fail(POD_ERR_WORKSPACE, "this batch needs " + std::to_string(p.ws_bytes) + " bytes of workspace, the "
                        "library's static scratch holds " + std::to_string(pod::kStaticScratchBytes) +
                        ": use pod_attn_forward with a workspace of the caller's");
    } else {
        if (!workspace || workspace_bytes < p.ws_bytes) return fail(POD_ERR_WORKSPACE, "workspace missing or too small");
        if (((uintptr_t)workspace & 255u) != 0) return fail(POD_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    }
    // every row is read and written in 16-byte pieces
    if ((((uintptr_t)prefill_q | (uintptr_t)decode_q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)out) & 15u) != 0)
        return fail(POD_ERR_INVALID_ARG, "prefill_q, decode_q, k_cache, v_cache and out must be 16-byte aligned");
    if ((((uintptr_t)seq_meta | (uintptr_t)block_table) & 3u) != 0)
        return fail(POD_ERR_INVALID_ARG, "seq_meta and block_table must be 4-byte aligned");
    if (use_static) {
        // This GPU's copy of the static array.  It is shared by every call on the GPU and keeps the
        // last call's contents: when it holds another plan's tables (or none), the counters are
        // cleared and this plan's tables copied in before the launch.
        int dev = 0;
        hipError_t de = hipGetDevice(&dev);
        if (de != hipSuccess) return fail_hip(de, "asking for the current device");
        if (dev < 0 || dev >= kMaxDevices) return fail(POD_ERR_UNSUPPORTED, "device index beyond what the static scratch tracks");
        de = pod::static_scratch(&workspace);
        if (de != hipSuccess) return fail_hip(de, "looking up the static scratch of this device");
        std::lock_guard<std::mutex> lock(g_static_mu);
        if (g_static_owner[dev] != plan->serial) {
            g_static_owner[dev] = 0;
            const pod_status up = upload_tables(p, workspace, (hipStream_t)stream);
            if (up != POD_OK) return up;
            g_static_owner[dev] = plan->serial;
        }
    }

    pod::KernelArgs a = make_args(p, prefill_q, decode_q, k_cache, v_cache, seq_meta, block_table, out, workspace);
    hipStream_t s = (hipStream_t)stream;
    const int dt = p.prm.dtype, hd = p.prm.head_dim;
    hipError_t e = hipSuccess;
    auto go = [&](int which, const pod::KernelArgs &args, hipStream_t on) {
        if (which == pod::kLaunchCombine && no_combine) return;
        if (e == hipSuccess) e = pod::launch(which, args, dt, hd, on);
    };

    // The combine pass only touches rows whose partials were produced in this call; the row list
    // holds the rows of prefill groups first, then those of decode groups.
    pod::KernelArgs only_p = a, only_d = a;
    only_p.n_crows = p.n_crows_prefill;
    only_d.n_crows_prefill = 0;
    only_d.crows = a.crows + p.n_crows_prefill;
    only_d.n_crows = a.n_crows - p.n_crows_prefill;

    // Where the decode units merge their groups the combine kernel is left with the prefill rows.  (The light decode
    // kernel does not merge.)
    std::unique_lock<std::mutex> side_held;
    const bool two_kernels = heavy || (mode == POD_MODE_FUSED && !cta_parallel && !use_static && heavy_is_ready(p, s, side_held));
    if (p.units_merge && !no_combine && !two_kernels) {
        a.arrived = a.hdr->arrived;
        a.n_crows = p.n_crows_prefill;
        only_d.n_crows = 0;
    }
    // The counters are cleared by the combine kernel of the call where it has one.
    if (!no_combine) {
        only_d.combine_resets = only_d.n_crows > 0;
        a.combine_resets = mode == POD_MODE_DECODE_ONLY ? only_d.combine_resets : a.n_crows > 0;
    }

    // Prefill kernel and decode kernel on the library's two side streams, forked from and joined
    // back into the caller's stream; the merge follows on the caller's stream.
    auto two_streams = [&](int prefill_kind, int decode_kind) -> pod_status {
        int dev = -1;
        const pod_status st = ensure_side(p, &dev);
        if (st != POD_OK) return st;
        SideStreams &side = g_side[dev];
        if (!side_held.owns_lock()) {
            side_held = std::unique_lock<std::mutex>(side.enqueue);
            side.caller = s;
        }
        const hipStream_t s0 = side.st[0], s1 = side.st[1];
        hipEvent_t fork = (hipEvent_t)p.events[0], j0 = (hipEvent_t)p.events[1], j1 = (hipEvent_t)p.events[2];
        auto chk = [&](hipError_t x) { if (e == hipSuccess) e = x; };
        chk(hipEventRecord(fork, s));
        chk(hipStreamWaitEvent(s0, fork, 0));
        chk(hipStreamWaitEvent(s1, fork, 0));
        go(prefill_kind, a, s0);
        go(decode_kind, a, s1);
        chk(hipEventRecord(j0, s0));
        chk(hipEventRecord(j1, s1));
        chk(hipStreamWaitEvent(s, j0, 0));
        chk(hipStreamWaitEvent(s, j1, 0));
        go(pod::kLaunchCombine, a, s);
        return POD_OK;
    };

    switch (mode) {
    case POD_MODE_FUSED:
        if (two_kernels) {
            // two prefill workgroups and one light decode workgroup per compute unit, from two kernels
            if (p.prm.n_prefill == 0 || p.prm.n_decode == 0) {
                go(p.prm.n_decode == 0 ? pod::kLaunchPrefillHeavy : pod::kLaunchDecodeLite, a, s);
                go(pod::kLaunchCombine, a, s);
            } else {
                const pod_status st = two_streams(pod::kLaunchPrefillHeavy, pod::kLaunchDecodeLite);
                if (st != POD_OK) return st;
            }
            break;
        }
        if (cta_parallel) {
            // one workgroup per work item: every decode workgroup is given its four units by index
            pod::KernelArgs c = a;
            c.n_static_seats = c.n_dctas;
            c.single_unit = 1;
            go(pod::kLaunchFusedCta, c, s);
        } else if (a.n_pitems == 0 || a.n_dunits == 0) {
            // One operation only: its own kernel does the same work without binding a role, and the
            // prefill one without claims.  Measured, fused kernel before: one decode of 6007 keys with 8
            // K/V heads 37.6 -> 34.2 us, four prompts of 100-700 tokens 69.7 -> 23.4 us, one of 8192
            // tokens 570 -> 552 us, 128 decodes at 2K-16K 811 -> 804 us.
            go(a.n_dunits == 0 ? pod::kLaunchPrefill : pod::kLaunchDecode, a, s);
        } else if (p.fixed_roles != pod::kRolesByTicket) {
            pod::KernelArgs c = a;
            c.fixed_roles = p.fixed_roles;
            c.n_dctas = c.fused_grid - c.n_pitems;
            go(pod::kLaunchFusedCta, c, s);
        } else {
            go(pod::kLaunchFused, a, s);
        }
        go(pod::kLaunchCombine, a, s);
        break;
    case POD_MODE_SERIAL:
        go(pod::kLaunchPrefill, a, s);
        go(pod::kLaunchDecode, a, s);
        go(pod::kLaunchCombine, a, s);
        break;
    case POD_MODE_PREFILL_ONLY:
        go(heavy ? pod::kLaunchPrefillHeavy : pod::kLaunchPrefill, a, s);
        go(pod::kLaunchCombine, only_p, s);
        break;
    case POD_MODE_DECODE_ONLY:
        go(heavy ? pod::kLaunchDecodeLite : pod::kLaunchDecode, a, s);
        go(pod::kLaunchCombine, only_d, s);
        break;
    case POD_MODE_STREAMS: {
        const pod_status st = two_streams(pod::kLaunchPrefill, pod::kLaunchDecode);
        if (st != POD_OK) return st;
        break;
    }
    default:
        break;
    }
    if (e != hipSuccess) {
        if (a.combine_resets) (void)pod::clear_header(a.hdr, s);       // the combine kernel may be what failed
        return fail_hip(e, "launching attention kernels");
    }
    return POD_OK;
}

pod_status pod_attn_forward(const void *prefill_q, const void *decode_q, const void *k_cache,
                            const void *v_cache, const int32_t *seq_meta, const int32_t *block_table,
                            void *out, const pod_attn_plan *plan, void *workspace,
                            size_t workspace_bytes, int32_t mode, void *stream)
{
    return forward_impl(prefill_q, decode_q, k_cache, v_cache, seq_meta, block_table, out, plan, workspace,
                        workspace_bytes, mode, stream, false);
}

pod_status pod_attn_forward_static(const void *prefill_q, const void *decode_q, const void *k_cache,
                                   const void *v_cache, const int32_t *seq_meta, const int32_t *block_table,
                                   void *out, const pod_attn_plan *plan, int32_t mode, void *stream)
{
    return forward_impl(prefill_q, decode_q, k_cache, v_cache, seq_meta, block_table, out, plan, nullptr, 0,
                        mode, stream, true);
}

static_assert(pod::kStaticScratchBytes == POD_ATTN_STATIC_SCRATCH_BYTES, "the header states the size of the static scratch");

int32_t pod_attn_role_for_ticket(int32_t ticket, int32_t prefill_ratio, int32_t decode_ratio, int32_t unit)
{
    if (ticket < 0 || unit < 0 || prefill_ratio < 0 || decode_ratio < 0 || prefill_ratio + decode_ratio <= 0) return -1;
    return pod::role_for_ticket((uint32_t)ticket, prefill_ratio, decode_ratio, unit);
}

// Host model of the fused launch.  Every actor is a small state machine whose steps are the
// atomic operations the device code performs, in the device's order; `order` decides whose step
// comes next, which stands for every timing the hardware could produce.
int32_t pod_attn_simulate_launch(const pod_attn_plan *plan, const int32_t *unit_of_wg, int32_t n_wgs,
                                 const int32_t *order, int32_t n_order, int32_t *first_role,
                                 int32_t *seat_of_wg, int32_t *item_owner, int32_t *unit_owner)
{
    if (!plan || n_wgs < 0 || n_order < 0 || (n_wgs > 0 && !unit_of_wg) || (n_order > 0 && !order)) return -1;
    const pod::Plan &p = plan->p;
    const int n_items = (int)p.pitems.size(), n_units = (int)p.dunits.size();
    for (int i = 0; i < n_items && item_owner; ++i) item_owner[i] = -1;
    for (int i = 0; i < n_units && unit_owner; ++i) unit_owner[i] = -1;
    constexpr int W = pod::kWavesPerWg, Q = pod::kXcdQueues;

    // the counters of the workspace header
    std::vector<uint32_t> cu_ticket(pod::kCuSlots, 0u);
    uint32_t next_seat = 0, next_pitem[Q] = {0}, next_dunit[Q] = {0};

    enum Phase { kBind, kPrefillClaims, kSeat, kDecodeWaves, kEnd };
    struct Wave { int cq = 0; bool started = false, done = false; };
    struct Wg {
        Phase phase = kBind;
        int first = pod::kNone, roles_done = 0, xcd = 0, seat = -1;
        int pq = 0;                            // prefill queue cursor
        bool plook = false;                    // that queue was found used up: look at all of them next
        Wave wave[W];
    };
    std::vector<Wg> wgs((size_t)n_wgs);
    int32_t owner_errors = 0;

    auto next_phase = [&](Wg &g) {
        // after a role has run dry: the other role, then the end
        ++g.roles_done;
        if (g.roles_done >= 2) { g.phase = kEnd; return; }
        const int next_role = g.first == pod::kPrefill ? pod::kDecode : pod::kPrefill;
        g.phase = next_role == pod::kPrefill ? kPrefillClaims : kSeat;
    };
    auto start_role = [&](Wg &g, int role) { g.phase = role == pod::kPrefill ? kPrefillClaims : kSeat; };
    auto wg_finished = [&](const Wg &g) { return g.phase == kEnd; };

    // One step of workgroup w's leader (actor 4w) or of its wavefront v (actor 4w + v) while the
    // workgroup is a decode worker.  Returns false when that actor has nothing to do right now.
    auto step = [&](int actor) -> bool {
        const int w = actor / W, v = actor % W;
        if (w < 0 || w >= n_wgs) return false;
        Wg &g = wgs[(size_t)w];
        switch (g.phase) {
        case kBind: {
            if (v != 0) return false;
            const unsigned cu = (unsigned)unit_of_wg[w] & (pod::kCuSlots - 1);
            if (p.fixed_roles != pod::kRolesByTicket) {
                // the workgroup index says it all: one prefill item, or a decode seat
                const int piece = pod::fixed_piece(p.fixed_roles, w, n_items, p.n_dwgs);
                g.roles_done = 1;               // no switch of operation
                g.first = piece < n_items ? pod::kPrefill : pod::kDecode;
                g.xcd = (int)(cu >> 6);
                if (first_role) first_role[w] = g.first;
                if (g.first == pod::kPrefill) {
                    const int item = p.pitem_of_wg[(size_t)piece];
                    if (item_owner) { if (item_owner[item] != -1) ++owner_errors; item_owner[item] = w; }
                    next_phase(g);
                } else {
                    const bool seated = piece - n_items < p.n_dwgs;
                    g.seat = seated ? piece - n_items : -1;
                    if (seat_of_wg) seat_of_wg[w] = g.seat;
                    g.phase = seated ? kDecodeWaves : kEnd;
                    for (Wave &x : g.wave) { x = Wave(); x.cq = g.xcd & (Q - 1); }
                }
                return true;
            }
            const uint32_t ticket = cu_ticket[cu]++;
            g.first = pod::role_for_ticket(ticket, p.p_ratio, p.d_ratio, (int)cu);
            g.xcd = (int)(cu >> 6);
            g.pq = g.xcd & (Q - 1);
            if (first_role) first_role[w] = g.first;
            start_role(g, g.first);
            return true;
        }
        case kPrefillClaims: {
            if (v != 0) return false;
            // one claim on the queue the workgroup is at, or, after that one was found used up, one
            // look at all queues: the nearest open one is next, and if none is open the operation is done
            auto len = [&](int q) { return p.pq_begin[q + 1] - p.pq_begin[q]; };
            if (g.plook) {
                g.plook = false;
                int d = 0;
                while (d < Q && (int)next_pitem[(g.pq + d) & (Q - 1)] >= len((g.pq + d) & (Q - 1))) ++d;
                if (d == Q) { next_phase(g); return true; }
                g.pq = (g.pq + d) & (Q - 1);
                return true;
            }
            const int k = len(g.pq) > 0 ? (int)next_pitem[g.pq]++ : len(g.pq);
            if (k < len(g.pq)) {
                const int item = p.pq_begin[g.pq] + k;
                if (item_owner) { if (item_owner[item] != -1) ++owner_errors; item_owner[item] = w; }
            } else {
                g.plook = true;
            }
            return true;
        }
        case kSeat: {
            if (v != 0) return false;
            g.seat = (int)next_seat++;
            if (seat_of_wg) seat_of_wg[w] = g.seat;
            if (g.seat < p.n_dwgs) {
                g.phase = kDecodeWaves;
                for (Wave &x : g.wave) { x = Wave(); x.cq = g.xcd & (Q - 1); }
            } else {
                next_phase(g);                  // every seat is taken: the seated workers stream the decode work
            }
            return true;
        }
        case kDecodeWaves: {
            Wave &x = g.wave[v];
            if (x.done) return false;
            auto own = [&](int unit) { if (unit_owner) { if (unit_owner[unit] != -1) ++owner_errors; unit_owner[unit] = actor; } };
            const bool one_round = n_units <= W * p.n_cus;
            if (!x.started && (one_round || g.seat < p.n_static_seats)) {
                x.started = true;
                x.done = one_round;             // nothing is left to claim
                if (g.seat * W + v < n_units) own(g.seat * W + v);   // the fixed first unit: no claim
            } else {
                x.started = true;
                // one claim on the queue the wavefront is at; a used-up queue sends it to the next
                // one with units, and back at its XCD's own queue it is done, as it is once another
                // wavefront of the XCD has come that far
                const int q0 = p.dq_begin[x.cq], q1 = p.dq_begin[x.cq + 1];
                const int k = (int)next_dunit[x.cq]++;
                if (k & pod::kAllQueuesEmpty) x.done = true;
                else if (k < q1 - q0) own(q0 + k);
                else {
                    const int home = g.xcd & (Q - 1);
                    do x.cq = (x.cq + 1) & (Q - 1);
                    while (x.cq != home && p.dq_begin[x.cq + 1] == p.dq_begin[x.cq]);
                    if (x.cq == home) {
                        next_dunit[home] |= pod::kAllQueuesEmpty;    // for the others of that XCD
                        x.done = true;
                    }
                }
            }
            bool all = true;
            for (const Wave &y : g.wave) all = all && y.done;
            if (all) next_phase(g);
            return true;
        }
        default:
            return false;
        }
    };

    int32_t steps = 0;
    for (int32_t i = 0; i < n_order; ++i)
        if (step(order[i])) ++steps;
    // whoever is not finished yet runs on, round-robin, until the launch has drained
    for (bool progress = true; progress;) {
        progress = false;
        for (int w = 0; w < n_wgs; ++w) {
            if (wg_finished(wgs[(size_t)w])) continue;
            for (int v = 0; v < W; ++v)
                if (step(w * W + v)) { ++steps; progress = true; }
        }
    }
    return owner_errors ? -2 : steps;
}

}  // extern "C"
