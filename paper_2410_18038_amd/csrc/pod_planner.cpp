// Host planner: validates a hybrid batch and cuts it into work items (paper Section 4.1: the
// numbers of prefill and decode workgroups are fixed on the host before the launch).
#include "pod_planner.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <numeric>

namespace pod {

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
int ceil_div(int a, int b) { return (a + b - 1) / b; }
int round_up(int a, int b) { return ceil_div(a, b) * b; }

std::string fmt(const char *f, long long a = 0, long long b = 0, long long c = 0)
{
    char buf[256];
    std::snprintf(buf, sizeof buf, f, a, b, c);
    return buf;
}

// Up to this many keys per wavefront the decode work is cut into one round of equal units, else into a wavefront's
// share with a taper.  us per call, taper / one round (8192-key requests): 128 channels (32 / 8 heads) at 260 keys per
// wavefront 37 / 27, at 400 46 / 39, at 640 67 / 60; 64 channels at 640 42 / 37; 256 channels at 260 57 / 49, at 400 75 /
// 71, at 640 between 128 / 110 and, beside a prefill chunk, 131 / 156: the line is the same number of bytes there.
// It is 320 keys beside prefill items on more than half of the compute units (384 items: 12000 keys of 32 heads 92 /
// 97; 256 channels at 310 keys 135 / 120), and where block ids are looked up per lane (24 decodes at 1K-6K
// beside 400 tokens 153 / 255; 256 channels, 43 at 0.4K-6K, 287 keys, 154 / 137).
int64_t one_round_share(int head_dim, bool few_items) { return few_items ? 640 * 128 / std::max(128, head_dim) : 320; }

// Keys of the longest decode unit of the automatic cut: about 1 MB of K/V (see "decode units" below).  Where
// block ids are looked up per lane a unit takes two to four times as long (the lookups are a second memory round
// trip in every step, and what they cost differs between wavefronts), so units are shorter to even that out.  us per
// call at 512 / 768 / 1024 / 2048 keys, blocks of one key: 32 decodes at 1K-4K of 32 / 32 heads 442 / 439 / 447 /
// 480; 64 at 2K-8K, 32 / 8 heads 479 / 485 / 493 / 514, of 64 channels 236 / 238 / 241 / 245; 16 at 4K-16K beside
// 512 tokens 302 / 304 / 352 / 319; 256 channels beside 1024 tokens 1029 / 1042 / 1063 / 1114.  768 makes half of
// the partial rows of 512.  (With blocks of 16 and 24 keys the same sizes are best between 1024 and 2048.)
int longest_unit(Layout layout, int head_dim)
{
    return layout == kLayoutPagedAny ? 768 : 2048 * 128 / std::max(128, head_dim);
}
constexpr int kLongestUnit = 2048;           // over all of them

// Where the tables lie in the workspace, given their lengths; returns the bytes it takes.
size_t lay_out(Plan &plan, size_t n_pitems, size_t n_dunits, size_t n_merge_rows, int64_t n_partial_rows)
{
    size_t off = align256(sizeof(WsHeader));
    plan.off_pitems = off;   off = align256(off + n_pitems * sizeof(PrefillItem));
    plan.off_pitems_by_wg = off; off = align256(off + n_pitems * sizeof(PrefillItem));
    plan.off_pitem_of_wg = off; off = align256(off + n_pitems * sizeof(int32_t));
    plan.off_dunits = off;   off = align256(off + n_dunits * sizeof(DecodeUnit));
    plan.off_crows = off;    off = align256(off + n_merge_rows * sizeof(CombineRow));
    plan.off_dq = off;       off = align256(off + sizeof plan.dq_begin);
    plan.off_part_o = off;   off = align256(off + (size_t)n_partial_rows * plan.prm.head_dim * sizeof(float));
    plan.off_part_ml = off;  off = align256(off + (size_t)n_partial_rows * 2 * sizeof(float));
    return off;
}

// First keys of the pieces a request of kv_len keys is cut into, and kv_len behind them.  One round of units:
// equal pieces of at most `chunk` keys.  A length given by the caller: the same, except that the last piece is
// cut again into a half and two quarters when those are still at least 128 keys (a request that fits one piece
// stays whole and needs no merge).  Otherwise a taper: pieces of at most `chunk` keys over the first half of the
// request, and a second half in pieces that halve down to max(chunk / 4, shortest).  Units are claimed
// longest first, so the short pieces are what is left at the end of a launch, when the wavefronts that
// are still busy decide when it ends.
enum class Cut { kEqual, kGiven, kTaper };
void cut_request(int kv_len, int chunk, int shortest, Cut how, std::vector<int> &cuts)
{
    cuts.clear();
    const int last = round_up(std::max(chunk / 4, shortest), kDecodeStep);     // shortest piece of a taper
    if (how == Cut::kTaper && kv_len > chunk + last / 2) {
        const int tail = kv_len / 2 >= 2 * last ? kv_len / 2 : 0;
        const int big = kv_len - tail, piece = round_up(ceil_div(big, ceil_div(big, chunk)), kDecodeStep);
        int t = 0;
        for (; t < big; t += piece) cuts.push_back(t);
        for (t = std::min(t, kv_len); t < kv_len;) {
            cuts.push_back(t);
            const int left = kv_len - t, half = std::min(chunk, left / 2 / kDecodeStep * kDecodeStep);
            t += half >= last ? half : left;
        }
    } else if (how == Cut::kTaper) {
        cuts.push_back(0);
    } else {
        const int tps = round_up(ceil_div(kv_len, ceil_div(kv_len, chunk)), kDecodeStep);
        for (int t = 0; t < kv_len; t += tps) cuts.push_back(t);
    }
    if (how == Cut::kGiven) {
        const int t_last = cuts.back(), len = kv_len - t_last;
        const int quarter = round_up(len / 4, kDecodeStep);
        const int half = (len - 2 * quarter) / kDecodeStep * kDecodeStep;    // cuts stay multiples of a step
        if (cuts.size() >= 2 && quarter >= 128 && half > 0 && half + quarter < len) {
            cuts.push_back(t_last + half);
            cuts.push_back(t_last + half + quarter);
        }
    }
    cuts.push_back(kv_len);
}

// Decode units when every request is cut into pieces of `chunk` keys.
int64_t units_of_length(const pod_attn_params &prm, const int32_t *seq_meta, int chunk)
{
    int64_t n = 0;
    for (int r = prm.n_prefill; r < prm.n_prefill + prm.n_decode; ++r)
        n += (int64_t)prm.n_kv_heads * ceil_div(seq_meta[4 * r + 2], chunk);
    return n;
}

}  // namespace

void role_ratio(int policy, int n_prefill_wgs, int n_decode_wgs, int &p, int &d)
{
    if (n_prefill_wgs <= 0 && n_decode_wgs <= 0) { p = 1; d = 1; return; }
    if (n_prefill_wgs <= 0) { p = 0; d = 1; return; }
    if (n_decode_wgs <= 0) { p = 1; d = 0; return; }
    if (policy == POD_POLICY_ALTERNATE) { p = 1; d = 1; return; }
    // Proportional (Section 4.1; Section 5.4.2 gives 50 prefill + 100 decode -> 1 : 2).
    const int kMaxSide = 8;
    if (n_decode_wgs >= n_prefill_wgs) {
        p = 1;
        d = std::min(kMaxSide, (int)std::lround((double)n_decode_wgs / n_prefill_wgs));
    } else {
        d = 1;
        p = std::min(kMaxSide, (int)std::lround((double)n_prefill_wgs / n_decode_wgs));
    }
    p = std::max(p, 1);
    d = std::max(d, 1);
}

pod_status build_plan(const pod_attn_params &prm, const int32_t *seq_meta, int n_cus, Plan &plan,
                      std::string &err)
{
    // ---- parameters --------------------------------------------------------------------
    if (prm.n_prefill < 0 || prm.n_decode < 0) { err = "negative request count"; return POD_ERR_INVALID_ARG; }
    if (prm.n_q_heads <= 0 || prm.n_kv_heads <= 0 || prm.n_q_heads % prm.n_kv_heads != 0) {
        err = "n_q_heads must be a positive multiple of n_kv_heads";
        return POD_ERR_INVALID_ARG;
    }
    const int group = prm.n_q_heads / prm.n_kv_heads;
    if (group > kMaxGroup) { err = "more than 16 query heads per K/V head"; return POD_ERR_UNSUPPORTED; }
    if (prm.head_dim != 64 && prm.head_dim != 128 && prm.head_dim != 256) { err = "head_dim must be 64, 128 or 256"; return POD_ERR_UNSUPPORTED; }
    if (prm.head_dim == 256 && group > kMaxGroup256) { err = "head_dim 256: more than 8 query heads per K/V head"; return POD_ERR_UNSUPPORTED; }
    if (prm.dtype != POD_F16 && prm.dtype != POD_BF16) { err = "dtype must be POD_F16 or POD_BF16"; return POD_ERR_UNSUPPORTED; }
    if (!(prm.softmax_scale > 0.f) || !std::isfinite(prm.softmax_scale)) {
        err = "softmax_scale must be positive and finite";
        return POD_ERR_INVALID_ARG;
    }
    if (prm.block_size < 0) { err = "negative block_size"; return POD_ERR_INVALID_ARG; }
    if (prm.n_cache_rows <= 0) { err = "n_cache_rows must be positive"; return POD_ERR_INVALID_ARG; }
    const bool paged = prm.block_size > 0;
    if (paged && (prm.max_blocks_per_seq <= 0 || prm.n_blocks <= 0)) {
        err = "paged cache needs max_blocks_per_seq and n_blocks";
        return POD_ERR_INVALID_ARG;
    }
    if (!paged && prm.kv_seq_stride <= 0) { err = "contiguous cache needs kv_seq_stride"; return POD_ERR_INVALID_ARG; }
    if (!paged && prm.kv_seq_stride % 8 != 0) { err = "kv_seq_stride must be a multiple of 8 elements (rows are read in 16-byte pieces)"; return POD_ERR_INVALID_ARG; }
    if (prm.kv_order != POD_KV_TOKEN_MAJOR && prm.kv_order != POD_KV_HEAD_MAJOR) { err = "unknown kv_order"; return POD_ERR_INVALID_ARG; }
    if (!paged && prm.kv_order == POD_KV_HEAD_MAJOR && prm.kv_seq_stride % ((int64_t)prm.n_kv_heads * prm.head_dim) != 0) {
        err = "head-major contiguous cache: kv_seq_stride must be a multiple of n_kv_heads * head_dim";
        return POD_ERR_INVALID_ARG;
    }
    if (prm.policy < POD_POLICY_AUTO || prm.policy > POD_POLICY_PROPORTIONAL) { err = "unknown policy"; return POD_ERR_INVALID_ARG; }
    if (prm.max_prefill_waves < 0 || prm.decode_chunk < 0 || prm.prefill_split_len < 0) {
        err = "negative tuning parameter";
        return POD_ERR_INVALID_ARG;
    }
    const int n_req = prm.n_prefill + prm.n_decode;
    if (n_req > 0 && seq_meta == nullptr) { err = "seq_meta is null"; return POD_ERR_INVALID_ARG; }
    if (n_cus <= 0) { err = "n_compute_units must be positive"; return POD_ERR_INVALID_ARG; }

    // ---- requests ----------------------------------------------------------------------
    const int64_t token_elems = (int64_t)prm.n_kv_heads * prm.head_dim;
    std::vector<std::pair<int, int>> spans;         // prefill (q_start, q_len)
    std::vector<char> decode_row_used((size_t)prm.n_decode, 0);
    int64_t n_prefill_rows = 0;
    for (int r = 0; r < n_req; ++r) {
        const int32_t *m = seq_meta + 4 * r;
        const int q_start = m[0], q_len = m[1], kv_len = m[2], row = m[3];
        if (q_len < 1) { err = fmt("request %lld: q_len must be >= 1", r); return POD_ERR_INVALID_ARG; }
        if (kv_len < q_len) { err = fmt("request %lld: kv_len %lld < q_len %lld", r, kv_len, q_len); return POD_ERR_INVALID_ARG; }
        if (q_start < 0) { err = fmt("request %lld: negative q_start", r); return POD_ERR_INVALID_ARG; }
        if (row < 0 || row >= prm.n_cache_rows) { err = fmt("request %lld: cache_row %lld out of range", r, row); return POD_ERR_INVALID_ARG; }
        if (paged) {
            if (ceil_div(kv_len, prm.block_size) > prm.max_blocks_per_seq) {
                err = fmt("request %lld: kv_len %lld needs more than max_blocks_per_seq blocks", r, kv_len);
                return POD_ERR_INVALID_ARG;
            }
        } else if ((int64_t)kv_len * token_elems > prm.kv_seq_stride) {
            err = fmt("request %lld: kv_len %lld does not fit in kv_seq_stride", r, kv_len);
            return POD_ERR_INVALID_ARG;
        }
        if (r < prm.n_prefill) {
            spans.emplace_back(q_start, q_len);
            n_prefill_rows = std::max<int64_t>(n_prefill_rows, (int64_t)q_start + q_len);
        } else {
            if (q_len != 1) { err = fmt("decode request %lld: q_len must be 1", r); return POD_ERR_INVALID_ARG; }
            if (q_start >= prm.n_decode) { err = fmt("decode request %lld: q_start out of range", r); return POD_ERR_INVALID_ARG; }
            if (decode_row_used[(size_t)q_start]) { err = fmt("decode request %lld: q_start used twice", r); return POD_ERR_INVALID_ARG; }
            decode_row_used[(size_t)q_start] = 1;
        }
    }
    // The prefill query ranges must tile [0, sum q_len): `out` holds exactly sum q_len prefill rows
    // followed by the decode rows, so a gap would push the decode rows past the end of a buffer
    // sized as documented, and an overlap would have two requests write one row.
    std::sort(spans.begin(), spans.end());
    int64_t next_row = 0;
    for (size_t i = 0; i < spans.size(); ++i) {
        if (spans[i].first != next_row) {
            err = spans[i].first < next_row ? "prefill query ranges overlap"
                                            : "prefill query ranges leave a gap (q_start must continue where the previous chunk ends)";
            return POD_ERR_INVALID_ARG;
        }
        next_row += spans[i].second;
    }
    // packed rows (token x head-in-group) are indexed with 32 bits
    if (n_prefill_rows * group > (int64_t)1 << 30) { err = "too many prefill rows"; return POD_ERR_INVALID_ARG; }

    plan = Plan();
    plan.prm = prm;
    plan.n_cus = n_cus;
    plan.group = group;
    plan.meta.assign(seq_meta, seq_meta + 4 * (size_t)n_req);
    plan.n_prefill_rows = n_prefill_rows;

    int64_t next_prow = 0;

    // ---- how much decode there is (decides the prefill split cap) ------------------------
    int64_t token_heads = 0;
    int longest_decode = 0;
    for (int r = prm.n_prefill; r < n_req; ++r) {
        token_heads += (int64_t)seq_meta[4 * r + 2] * prm.n_kv_heads;
        longest_decode = std::max(longest_decode, seq_meta[4 * r + 2]);
    }
    // Keys per streaming wavefront (there are four of those per compute unit).
    const int64_t n_waves = (int64_t)n_cus * kWavesPerWg;
    const int64_t share = (token_heads + n_waves - 1) / n_waves;
    // Does the decode work hold a worker on every compute unit for a good part of the launch?
    const int given_chunk = prm.decode_chunk > 0 ? round_up(prm.decode_chunk, kDecodeStep) : 0;
    const bool decode_on_every_unit = given_chunk > 0 ? units_of_length(prm, seq_meta, given_chunk) >= n_waves : share >= 512;

    // ---- prefill items -----------------------------------------------------------------
    // Row blocks of 128 packed rows per K/V head; split-KV only when there are too few blocks to
    // fill the chip, and never beyond `max_prefill_waves` chip-wide rounds (Section 4.2.4).
    {
        const int kPrefillRows = prefill_item_rows(prm.head_dim), kPrefillKvTile = prefill_kv_tile(prm.head_dim);
        int64_t base_items = 0;
        for (int r = 0; r < prm.n_prefill; ++r)
            base_items += (int64_t)prm.n_kv_heads * ceil_div(seq_meta[4 * r + 1] * group, kPrefillRows);
        // Default: two rounds of the chip, as in the paper; one, when a decode worker holds one of
        // the two slots of every unit for most of the launch, so that the items fill the other
        // slots once (measured on the ratio sweep: equal or up to 3 % faster, never slower; fewer
        // items also mean fewer partial rows to merge).
        const int waves = prm.max_prefill_waves > 0 ? prm.max_prefill_waves : (decode_on_every_unit ? 1 : 2);
        const int64_t cap_items = (int64_t)waves * n_cus;
        const int s_cap = base_items > 0 ? (int)std::max<int64_t>(1, cap_items / base_items) : 1;
        const int min_split = round_up(prm.prefill_split_len > 0 ? prm.prefill_split_len : 1024, kPrefillKvTile);
        for (int r = 0; r < prm.n_prefill; ++r) {
            const int q_len = seq_meta[4 * r + 1], kv_len = seq_meta[4 * r + 2];
            const int prefix = kv_len - q_len;
            const int rows_total = q_len * group;
            for (int kvh = 0; kvh < prm.n_kv_heads; ++kvh)
                for (int row0 = 0; row0 < rows_total; row0 += kPrefillRows) {
                    const int n_rows = std::min(kPrefillRows, rows_total - row0);
                    const int last_tok = (row0 + n_rows - 1) / group;
                    const int kmax = prefix + last_tok + 1;          // keys this block can see
                    const int n_tiles = ceil_div(kmax, kPrefillKvTile);
                    int s = std::min(s_cap, std::max(1, kmax / min_split));
                    const int tps = ceil_div(n_tiles, s);
                    s = ceil_div(n_tiles, tps);
                    int64_t prow_base = -1;
                    if (s > 1) {
                        prow_base = next_prow;
                        next_prow += (int64_t)s * kPrefillRows;
                        plan.centries.push_back(CombineEntry{kPrefill, kvh, row0, n_rows, s, (int32_t)prow_base,
                                                             kPrefillRows, seq_meta[4 * r]});
                    }
                    for (int i = 0; i < s; ++i) {
                        PrefillItem it;
                        it.req = r; it.kv_head = kvh; it.row0 = row0; it.n_rows = n_rows;
                        it.kv_begin = i * tps * kPrefillKvTile;
                        it.kv_end = std::min(kmax, (i + 1) * tps * kPrefillKvTile);
                        it.prow0 = s > 1 ? (int32_t)(prow_base + (int64_t)i * kPrefillRows) : -1;
                        it.split = i;
                        plan.pitems.push_back(it);
                    }
                    plan.max_psplits = std::max(plan.max_psplits, s);
                }
        }
        // One queue per XCD (each XCD has its own L2): items of one K/V head go to one queue, so
        // the workgroups that re-read that head's K/V tiles share an L2 and the re-reads do not
        // reach HBM.  Inside a queue: longest first, since ids are claimed in order.  A worker
        // whose own queue is empty takes items from the other queues.
        // With fewer (request, K/V head) streams than queues, a stream's row blocks are dealt over
        // several queues, so that every XCD has a queue of its own to start from.
        const int n_streams = prm.n_prefill * prm.n_kv_heads;
        const int per = n_streams > 0 && n_streams < kXcdQueues ? kXcdQueues / n_streams : 1;
        auto queue_of = [&](const PrefillItem &x) {
            const int stream = x.req * prm.n_kv_heads + x.kv_head;
            return (stream * per + (x.row0 / kPrefillRows) % per) % kXcdQueues;
        };
        std::vector<PrefillItem> dealt(plan.pitems.size());
        std::vector<int32_t> queue(plan.pitems.size());
        for (size_t i = 0; i < plan.pitems.size(); ++i) ++plan.pq_begin[(queue[i] = queue_of(plan.pitems[i])) + 1];
        for (int q = 0; q < kXcdQueues; ++q) plan.pq_begin[q + 1] += plan.pq_begin[q];
        {
            int at[kXcdQueues];
            std::copy(plan.pq_begin, plan.pq_begin + kXcdQueues, at);
            for (size_t i = 0; i < plan.pitems.size(); ++i) dealt[(size_t)at[queue[i]]++] = plan.pitems[i];
        }
        for (int q = 0; q < kXcdQueues; ++q)
            std::stable_sort(dealt.begin() + plan.pq_begin[q], dealt.begin() + plan.pq_begin[q + 1],
                             [](const PrefillItem &x, const PrefillItem &y) { return x.kv_end - x.kv_begin > y.kv_end - y.kv_begin; });
        plan.pitems = std::move(dealt);
        // Order for the kernels that take items by workgroup index (one workgroup per item, no
        // claims): workgroup b runs on XCD b % 8 (measured: the dispatcher deals them round-robin
        // without exception), so it gets the next item of queue b % 8 and a K/V head's tiles stay in
        // the L2 of the XCDs its queue belongs to.  Queues of unequal length: what is left over goes
        // to the workgroups whose own queue has run out.
        {
            const int n = (int)plan.pitems.size();
            std::vector<int32_t> &item = plan.pitem_of_wg;
            item.assign((size_t)n, 0);
            int next[kXcdQueues];
            for (int q = 0; q < kXcdQueues; ++q) next[q] = plan.pq_begin[q];
            std::vector<int> unfilled;
            for (int b = 0; b < n; ++b) {
                const int q = b % kXcdQueues;
                if (next[q] < plan.pq_begin[q + 1]) item[(size_t)b] = next[q]++;
                else unfilled.push_back(b);
            }
            size_t u = 0;
            for (int q = 0; q < kXcdQueues; ++q)
                while (next[q] < plan.pq_begin[q + 1]) item[(size_t)unfilled[u++]] = next[q]++;
            // Two rounds at once: workgroup b + n_cus joins workgroup b on its compute unit, and two long items
            // there slow each other down while other units run dry.  Within an XCD the second round is
            // therefore dealt shortest first.  (An XCD's own items come longest first; only items that were
            // left over from other queues are out of place, and are moved up.)
            if (n > n_cus && n <= 2 * n_cus) {
                auto keys = [&](int i) { return plan.pitems[(size_t)i].kv_end - plan.pitems[(size_t)i].kv_begin; };
                for (int x = 0; x < kXcdQueues; ++x) {
                    const int count = (n - x + kXcdQueues - 1) / kXcdQueues;
                    auto at = [&](int k) -> int32_t & { return item[(size_t)(x + k * kXcdQueues)]; };
                    for (int k = 1; k < count; ++k) {
                        const int32_t moved = at(k);
                        int j = k;
                        for (; j > 0 && keys(at(j - 1)) < keys(moved); --j) at(j) = at(j - 1);
                        at(j) = moved;
                    }
                    int lo = std::min(count, std::max(0, (n_cus - x + kXcdQueues - 1) / kXcdQueues)), hi = count - 1;
                    for (; lo < hi; ++lo, --hi) std::swap(at(lo), at(hi));
                }
            }
            plan.pitems_by_wg.reserve((size_t)n);
            for (int b = 0; b < n; ++b) plan.pitems_by_wg.push_back(plan.pitems[(size_t)item[(size_t)b]]);
        }
    }

    // ---- decode units ------------------------------------------------------------------
    {
        int longest_item = 0;                    // keys of the longest prefill item
        for (const PrefillItem &it : plan.pitems) longest_item = std::max(longest_item, it.kv_end - it.kv_begin);
        const int n_items = (int)plan.pitems.size();
        const Layout layout = cache_layout(prm.block_size, prm.head_dim, prm.n_kv_heads);
        const bool few_items = 2 * n_items <= n_cus && layout != kLayoutPagedAny;
        const bool one_round = prm.decode_chunk <= 0 && share <= one_round_share(prm.head_dim, few_items);
        const int shortest = std::max(64, 8 * group);    // at 8 * group keys a unit's partial rows are 1/8 of its K/V bytes
        std::vector<int> cuts;
        int chunk;
        if (given_chunk > 0) {
            chunk = given_chunk;
        } else if (one_round) {
            // Little work: what counts is the length of the one unit a wavefront runs (16 keys take about
            // 0.7 us), so requests are cut into equal pieces as short as one round of the chip allows.
            // us per call, units of at least 512 keys before: one decode of 6007 keys 31.9 -> 14.4,
            // three at 4K (8 heads per K/V head) 31.8 -> 18.1, 128 short ones 21.1 -> 15.0.
            //
            // Beside few prefill items (longer than a share) the round is that of the compute units without one: every workgroup then has
            // a unit to itself (see the roles by index), where an item that shares its unit with a worker takes up to
            // 40 % longer.  All units / those without an item: 300 + 1000 tokens beside 8 x 4000, 32 / 8 heads 47.4 /
            // 35.5; 128 + 1000 beside 8 x 4000, 256 channels 78 / 48; 96 items beside 12 x 8000, 8 / 1 heads 43.5 / 39.0.
            // Above half of the units (176 items, 8 x 1000: 25.9 / 26.2; 256 channels, 8 x 4000: 62 / 102) the workers need them all.
            const int64_t waves = few_items && longest_item > share ? (int64_t)kWavesPerWg * (n_cus - n_items) : n_waves;
            const int64_t own_share = (token_heads + waves - 1) / waves;
            // Cutting costs a merge, in the units or in a kernel of its own.  With the latter it is not worth it when the
            // requests are short: us whole / cut at 160 keys 10.2 / 10.9, at 176 11.4 / 10.8, at 250 14.6 / 10.8 (64
            // channels 8.3 / 11.5, 8.4 / 11.5, 10.3 / 11.4; 256 channels at 100 keys 17.0 / 14.6, at 250 34 / 15).
            // (That line is the merge kernel's.  Where the units merge, 112 keys would be it, at 128 8.8 / 8.4, at 160 10.2 /
            // 8.4; the rule does not tell the two apart.)  Nor when the prefill items beside them take longer than the
            // whole requests anyway (64 keys of an item take about 1.1 us, 16 of a unit 0.7, at 256 channels 2)
            // and need no merge themselves: items of 1128 keys beside 16 x 500 27.8 / 33.5, x 700 36 / 34;
            // of 2028 beside 16 x 700 44.6 / 50.7, 2 x 1000 50.1 / 48.1; of 128 beside 16 x 200 14.0 / 12.2; 256
            // channels, 1128 keys beside 16 x 300 41.2 / 44.0, x 400 53 / 44, 2028 beside 2 x 500 67.5 / 70.4, x 700
            // 86 / 71.  (Units whose block ids are looked up per lane take longer: cut from an eighth.)
            const int worth_merging = shortest + (prm.head_dim > 128 ? 16 : 112);
            const int beside_items = layout == kLayoutPagedAny ? longest_item / 8 + 150
                                                               : (prm.head_dim > 128 ? longest_item / 5 : longest_item / 5 * 2) + 100;
            // All of that holds where the workers have slots of their own.  With an item for every slot, the one
            // that a worker's slot gets starts when the worker is done and ends that much later: 512 items of 32K
            // keys beside 4 x 4096 of 4 heads 1128 us whole, 979 cut,
            // beside 16 x 4096 1146 / 976; 64 channels, 2048 + 6144 beside 1 x 3000 216 / 171.
            const int64_t whole_units = units_of_length(prm, seq_meta, longest_decode);
            const bool own_slots = n_items + (whole_units + kWavesPerWg - 1) / kWavesPerWg <= (int64_t)kSlotsPerUnit * n_cus;
            if (longest_decode <= worth_merging ||
                (longest_item > 0 && plan.centries.empty() && longest_decode <= beside_items && whole_units <= waves && own_slots))
                chunk = round_up(std::max(longest_decode, kDecodeStep), kDecodeStep);
            else {
                // the shortest length, in steps from `shortest`, that makes units for one round; two shares at the most
                const int64_t limit = std::min<int64_t>(longest_decode, 2 * own_share);
                int lo = 0, hi = limit > shortest ? (int)((limit - shortest + kDecodeStep - 1) / kDecodeStep) : 0;
                while (lo < hi) {
                    const int mid = (lo + hi) / 2;
                    if (units_of_length(prm, seq_meta, shortest + mid * kDecodeStep) <= waves) hi = mid;
                    else lo = mid + 1;
                }
                chunk = shortest + lo * kDecodeStep;
                // Up to kMergeSplits splits the units merge by themselves, which is worth any unit that the items beside it
                // outlast by far: cut to merge in a kernel of its own / in the units, items of 2028 keys beside 2 x 1000
                // 47.4 / 44.2, 1128 beside 16 x 700 with 4 K/V heads 31.0 / 27.7.  (Without items it is not: 3 x 677 in
                // 11 splits of 64 keys 9.4, in 8 of 96 10.0.)  Where they cannot merge, 256 channels or more than 8 query
                // heads per K/V head, the combine kernel still has fewer splits to fetch: items of 2028 keys beside 4 x 1500
                // 70.4 / 69.9 (16 / 8 heads of 256 channels), 1500 beside 2 x 1500 38.1 / 37.6 (9 / 1 heads of 128).
                const int piece = round_up(ceil_div(longest_decode, kMergeSplits), kDecodeStep);
                const int64_t workers = (units_of_length(prm, seq_meta, piece) + kWavesPerWg - 1) / kWavesPerWg;
                if (piece > chunk && plan.centries.empty() && longest_item > 0 && piece <= beside_items / 2 &&
                    n_items + workers <= (int64_t)kSlotsPerUnit * n_cus)
                    chunk = piece;
            }
        } else {
            // Enough work for every wavefront: pieces of at most one wavefront's share, and the second
            // half of every request in pieces that halve down to a quarter of that.  Wavefronts do not
            // stream at one rate (those of every second XCD get 10-20 % less), units are claimed longest
            // first, and the short ones are what is left to even that out at the end.  A piece is no
            // longer than about 1 MB of K/V: with long ones the slow wavefronts finish late (pieces of
            // 4096 keys instead of 2048, 64 x 4096 keys x 32 heads: 659 against 641 us; of 1296 against
            // 2592 keys of 256 channels: 464 against 483).  us per call, pieces of a quarter share or 768 keys
            // before: 8 decodes 62.6 -> 59.6, 512 + 16 decodes 140.7 -> 135.9, 256 channels 473 -> 464,
            // 15 / 5 heads 95 -> 86, 84 decodes at 0.5K-1K 66.8 -> 57.7.
            auto chunk_of = [&](int cap) { return round_up((int)std::min<int64_t>(std::max<int64_t>(share, shortest), cap), kDecodeStep); };
            const int coarse = chunk_of(kLongestUnit);
            const int cap = longest_unit(layout, prm.head_dim);
            chunk = chunk_of(cap);
            // Requests shorter than a piece stay whole.  Where they are most of the work and 1 to 1.4 (or 2 to 2.1; with one
            // or two heads per K/V head, whose partial rows are small, 1 to 1.6, 2 to 2.4 or 3 to 3.2) per wavefront, the last round keeps few wavefronts busy, and pieces of half the longest request (the taper
            // makes three or four of each) are faster.  (A wavefront streams up to 1.7 times as fast when others are
            // idle, so that fuller last rounds cost nothing.)  us whole / half, 32 / 8 heads of 2000 keys: 130
            // requests (1.02 per wavefront) 234 / 181, 160 (1.25) 248 / 217, 200 (1.56) 268 / 268, 250 (1.95) 323 / 331,
            // 300 (2.34) 402 / 395; of 1000 keys 123 / 100, 128 / 118, 139 / 145, 162 / 178, 204 / 211; 32 / 32 heads
            // of 2000 keys at 1.25, 1.56, 1.94, 2.34 249 / 213, 275 / 264, 327 / 321, 400 / 387; 8 / 1 heads at 1.25,
            // 1.56 246 / 227, 263 / 278.  Short pieces gain less: 160 of 500 keys 71 / 73, 64 channels 44 / 48, but
            // 256 channels 141 / 123 (200 of them, at 1.56, 144 / 150).
            {
                const int whole = chunk + round_up(std::max(chunk / 4, shortest), kDecodeStep) / 2;
                int64_t whole_token_heads = 0;
                for (int r = prm.n_prefill; r < n_req; ++r)
                    if (seq_meta[4 * r + 2] <= whole) whole_token_heads += (int64_t)seq_meta[4 * r + 2] * prm.n_kv_heads;
                const int64_t n_units = units_of_length(prm, seq_meta, whole), rounds = (n_units + n_waves - 1) / n_waves;
                const int64_t length = (int64_t)longest_decode * std::max(128, prm.head_dim);
                const int tenths = group <= 2 && length > 128 * 1024 ? 8 : 7;
                if (2 * whole_token_heads > token_heads && 10 * n_units < tenths * rounds * n_waves && length >= 96 * 1024)
                    chunk = chunk_of(std::min(cap, longest_decode / 2));
            }
            // Shorter units stream faster there but make more partial rows.  Where those are what keeps a
            // batch out of the library's own scratch, it is cut at 2048 keys.
            if (chunk < coarse) {
                size_t merged = 0;
                for (const CombineEntry &c : plan.centries) merged += (size_t)c.n_rows;
                auto bytes_at = [&](int length) {
                    size_t n_units = 0, n_rows = merged;
                    int64_t n_partials = next_prow;
                    for (int r = prm.n_prefill; r < n_req; ++r) {
                        cut_request(seq_meta[4 * r + 2], length, shortest, Cut::kTaper, cuts);
                        const size_t s = cuts.size() - 1;
                        n_units += s * (size_t)prm.n_kv_heads;
                        if (s > 1) { n_rows += (size_t)prm.n_q_heads; n_partials += (int64_t)s * prm.n_q_heads; }
                    }
                    return lay_out(plan, plan.pitems.size(), n_units, n_rows, n_partials);
                };
                if (bytes_at(chunk) > POD_ATTN_STATIC_SCRATCH_BYTES && bytes_at(coarse) <= POD_ATTN_STATIC_SCRATCH_BYTES)
                    chunk = coarse;
            }
        }
        plan.decode_chunk = chunk;
        plan.decode_prow0 = next_prow;
        const Cut how = given_chunk > 0 ? Cut::kGiven : one_round ? Cut::kEqual : Cut::kTaper;
        {
            size_t n_est = 0;
            for (int r = prm.n_prefill; r < n_req; ++r)
                n_est += (size_t)prm.n_kv_heads * (size_t)(seq_meta[4 * r + 2] / chunk + 5);
            plan.dunits.reserve(n_est);
            plan.centries.reserve(plan.centries.size() + (size_t)prm.n_decode * prm.n_kv_heads);
        }
        for (int r = prm.n_prefill; r < n_req; ++r) {
            cut_request(seq_meta[4 * r + 2], chunk, shortest, how, cuts);
            const int s_eff = (int)cuts.size() - 1;
            for (int kvh = 0; kvh < prm.n_kv_heads; ++kvh) {
                int64_t prow_base = -1;
                if (s_eff > 1) {
                    prow_base = next_prow;
                    next_prow += (int64_t)s_eff * group;
                    plan.centries.push_back(CombineEntry{kDecode, kvh, 0, group, s_eff, (int32_t)prow_base, group, seq_meta[4 * r]});
                }
                for (int i = 0; i < s_eff; ++i) {
                    DecodeUnit u;
                    u.req = r; u.kv_head = kvh;
                    u.t0 = cuts[(size_t)i];
                    u.t1 = cuts[(size_t)i + 1];
                    u.prow0 = s_eff > 1 ? (int32_t)(prow_base + (int64_t)i * group) : -1;
                    u.split = i; u.q_start = seq_meta[4 * r]; u.cache_row = seq_meta[4 * r + 3];
                    plan.dunits.push_back(u);
                }
                plan.max_dsplits = std::max(plan.max_dsplits, s_eff);
            }
        }
        // Longest first, in the given order among equals: dealt by length, since there are few lengths and many
        // units (comparisons took half of the time of planning a batch of short units); units of a length
        // beyond what the automatic cut makes are sorted.
        constexpr int kDealtByLength = 2 * kLongestUnit;
        auto length = [](const DecodeUnit &u) { return u.t1 - u.t0; };
        int longest = 0;
        for (const DecodeUnit &u : plan.dunits) longest = std::max(longest, length(u));
        if (longest <= kDealtByLength) {
            std::vector<int> at((size_t)longest + 2, 0);
            for (const DecodeUnit &u : plan.dunits) ++at[(size_t)(longest - length(u) + 1)];
            std::partial_sum(at.begin(), at.end(), at.begin());
            std::vector<DecodeUnit> sorted(plan.dunits.size());
            for (const DecodeUnit &u : plan.dunits) sorted[(size_t)at[(size_t)(longest - length(u))]++] = u;
            plan.dunits.swap(sorted);
        } else {
            std::stable_sort(plan.dunits.begin(), plan.dunits.end(),
                             [&](const DecodeUnit &x, const DecodeUnit &y) { return length(x) > length(y); });
        }
        // Decode workers are persistent: each of their wavefronts claims units until none is left.
        // One worker per compute unit: four streaming wavefronts per unit already keep HBM busy,
        // and a second worker on the unit makes the stream slower, not faster (measured: 681 ->
        // 656 us on a 4.3 GB batch; the eight wavefronts of a unit and the XCDs among each other
        // then get very unequal shares, and the slowest wavefronts decide when the launch ends).
        plan.n_dwgs = std::min(n_cus, ceil_div((int)plan.dunits.size(), kWavesPerWg));
        // With one unit a wavefront the unit that finishes a group last merges it, and no kernel follows for the decode
        // rows.  (With more units every one of them would wait for its stores in the middle of the stream; with
        // more splits or rows a single wavefront takes longer than the combine kernel.)  us per call, combine kernel /
        // in the units: 8 requests of 400 keys, 32 / 8 heads 9.3 / 8.6, 8 query heads on one K/V head 9.3 / 9.0, 16 of them
        // (64 channels) 9.8 / 10.7; 256 channels with two 14.7 / 14.6, with four 14.8 / 15.1.
        plan.units_merge = group <= kMergeRows && prm.head_dim <= kMergeDim && plan.max_dsplits >= 2 && plan.max_dsplits <= kMergeSplits &&
                           (int64_t)plan.dunits.size() <= (int64_t)kWavesPerWg * n_cus &&
                           next_prow - plan.decode_prow0 <= (int64_t)(sizeof(WsHeader::arrived) / sizeof(uint32_t));
        // The first workers to take a decode seat (one per compute unit) start with four fixed
        // units each, the longest ones, and claim nothing for them.  The other units are dealt
        // round-robin, still longest first, to one queue per XCD: a wavefront claims from the
        // queue of the XCD it runs on and moves to the next queue when that one is empty, so the
        // eight counters are each hit by an eighth of the chip.
        const int n_units = (int)plan.dunits.size();
        plan.n_static_seats = std::min(n_cus, n_units / kWavesPerWg);
        const int n_fixed = plan.n_static_seats * kWavesPerWg;
        std::vector<DecodeUnit> dealt;
        dealt.reserve((size_t)(n_units - n_fixed));
        for (int q = 0; q < kXcdQueues; ++q) {
            plan.dq_begin[q] = n_fixed + (int)dealt.size();
            for (int j = n_fixed + q; j < n_units; j += kXcdQueues) dealt.push_back(plan.dunits[(size_t)j]);
        }
        plan.dq_begin[kXcdQueues] = n_units;
        std::copy(dealt.begin(), dealt.end(), plan.dunits.begin() + n_fixed);
        if (plan.units_merge) {
            std::vector<uint8_t> n_splits((size_t)(next_prow - plan.decode_prow0), 0);     // by the group's first partial row
            for (int pass = 0; pass < 2; ++pass)
                for (const DecodeUnit &u : plan.dunits) {
                    uint8_t none = 0, &n = u.prow0 < 0 ? none : n_splits[(size_t)(u.prow0 - u.split * group - plan.decode_prow0)];
                    if (pass == 0) ++n;
                    else plan.unit_splits.push_back(n);
                }
        }
    }
    if (next_prow > (int64_t)1 << 30) { err = "too many partial rows"; return POD_ERR_INVALID_ARG; }
    plan.n_partial_rows = next_prow;

    // The output rows that are merged from partials, prefill rows first.
    {
        size_t n_rows = 0;
        for (const CombineEntry &c : plan.centries) n_rows += (size_t)c.n_rows;
        plan.merge_rows.reserve(n_rows);
    }
    for (const CombineEntry &c : plan.centries) {
        const uint64_t decode_bit = (uint64_t)(c.kind == kDecode) << 63;
        int64_t token_row = c.kind == kPrefill ? c.q_start + c.row0 / group : n_prefill_rows + c.q_start;
        int head = c.kind == kPrefill ? c.row0 % group : 0;               // inside the group
        for (int r = 0; r < c.n_rows; ++r) {
            const uint64_t out_row = (uint64_t)(token_row * prm.n_q_heads + c.kv_head * group + head) | decode_bit;
            plan.merge_rows.push_back(CombineRow{c.prow0 + r, c.n_splits, (uint32_t)out_row, (uint32_t)(out_row >> 32)});
            if (++head == group) { head = 0; ++token_row; }
        }
        if (c.kind == kPrefill) plan.n_crows_prefill = (int)plan.merge_rows.size();
    }

    // A group of the combine kernel fetches kCombineFetch splits at a time; as many groups share a row as
    // its splits need to be fetched at once, as far as a workgroup has groups.
    for (int op : {kPrefill, kDecode})
        while (plan.combine_groups[op] < kWgThreads / (prm.head_dim / 4) &&
               plan.combine_groups[op] * kCombineFetch < (op == kPrefill ? plan.max_psplits : plan.max_dsplits))
            plan.combine_groups[op] *= 2;

    // The ratio compares workgroup counts as the paper does (Section 4.1): decode work counts as the
    // workgroups it would fill at one wavefront per unit, up to one resident round.
    const int n_decode_ctas = std::min(2 * n_cus, ceil_div((int)plan.dunits.size(), kWavesPerWg));
    role_ratio(prm.policy, (int)plan.pitems.size(), n_decode_ctas, plan.p_ratio, plan.d_ratio);
    // Automatic policy: a unit seats one decode worker at most, so starting more than one of its
    // two workgroups in the decode role only leaves some units with two candidates for a seat and
    // others with none (measured on a 256-token chunk beside 256 decodes: 1812 against 1750 us).
    if (prm.policy == POD_POLICY_AUTO && plan.d_ratio > plan.p_ratio && plan.p_ratio > 0) plan.d_ratio = plan.p_ratio;
    // The fused launch is one resident round of workgroups (two per compute unit) that loop over
    // work, or fewer when the batch is smaller than that.
    plan.fused_grid = std::min(2 * n_cus, (int)plan.pitems.size() + plan.n_dwgs);
    // With a decode worker for every unit and some prefill work, the round is launched in full
    // even when the items are fewer than the remaining slots: every unit then gets one workgroup
    // that starts in each operation, and the decode seats are taken one per unit at once (a unit
    // that got a single workgroup would start it on prefill and be left without a decode worker).
    if (plan.n_dwgs == n_cus && !plan.pitems.empty()) plan.fused_grid = 2 * n_cus;
    // Where each prefill item and each decode worker has a workgroup and all of them are resident at once,
    // the hardware's own order puts one of each on a unit (it deals workgroups to the units in turn),
    // and binding by index saves the chain of ticket, seat and claim at the start (3-4 us, 256 seats being
    // handed out one per 11 ns) and the claims and seats after the last item.  us per call, by ticket / by index:
    // 4 items + 41 workers 17.1 / 13.5; 200 items (64 channels) 89.1 / 79.9; 140 (15 heads) 82.3 / 75.4; 224 (448
    // tokens + 16 decodes, 32 / 8 heads) 163.2 / 161.2.  With an item for every unit (225 to 256 items, 512 to 2048
    // tokens beside 16 to 120 decodes; ranges over 16 to 32 batches each): 64 channels 0.92 to 1.00 of the time by
    // ticket, 128 channels with 8 query heads per K/V head 0.93 to 0.99, with 4 0.97 to 1.00, with 2 0.98 to 1.05,
    // with one 0.99 to 1.02: the line is at 7/8 of the units there (few heads per K/V head mean much to stream, and
    // the older workgroup of a unit is a prefill one).  At 256 channels decode workers go first, for the
    // same reason: 256 items 471 / 452 (items first 471), 192 items 456 / 448 (461).  Workers first at up to 128
    // channels is within 2 % of items first but for 8 query heads per K/V head, 0.96 to 1.10 of the time by ticket.
    if (prm.policy == POD_POLICY_AUTO && !plan.pitems.empty() && plan.n_dwgs > 0) {
        const int n_items = (int)plan.pitems.size();
        int rule = kRolesByTicket;
        const int most_items = prm.head_dim < 128 || group >= 3 ? n_cus : n_cus / 8 * 7;
        if (n_items + plan.n_dwgs <= n_cus || (prm.head_dim <= 128 && n_items <= most_items)) rule = kPrefillFirst;
        else if (prm.head_dim > 128 && n_items <= n_cus && plan.n_dwgs == n_cus) rule = kDecodeFirst;
        plan.fixed_roles = rule;
    }

    // ---- which occupancy configuration suits the batch (Section 4.2.2) ----------------------
    // The prefill-heavy configuration pays when the prefill work outlasts the decode stream even
    // though that stream is the slower one there: matrix time of the prefill (at the datasheet
    // peak) above 1.2 x the time the batch's K/V bytes take at the HBM peak.
    {
        double pairs = 0.0, kv_tokens = 0.0;
        for (int r = 0; r < n_req; ++r) {
            const double q_len = seq_meta[4 * r + 1], kv_len = seq_meta[4 * r + 2];
            kv_tokens += kv_len;
            if (r < prm.n_prefill) pairs += q_len * (kv_len - q_len) + q_len * (q_len + 1.0) / 2.0;
        }
        const double flop_time = 4.0 * prm.head_dim * pairs * prm.n_q_heads / 2.5e15;
        const double byte_time = kv_tokens * prm.n_kv_heads * prm.head_dim * 4.0 / 8.0e12;
        const bool built = built_for_prefill_heavy(prm.block_size, prm.head_dim, prm.n_kv_heads);
        plan.heavy_advised = built && prm.n_prefill > 0 && prm.n_decode > 0 &&
                             flop_time > 1.2 * byte_time;
        // The automatic policy takes that configuration where it was ahead by more than its two streams and three
        // events cost (20 us a call): an item for every slot, so that decode workers of the fused launch hold up items,
        // enough prefill to make up for the light decode kernel, and enough decode to be worth hiding.
        // fused / prefill-heavy, us, by matrix time at the peak (us) and its ratio to the byte time of the decode
        // stream: 32 / 4 heads 2048 tokens at 32K beside 32 x 32K (426, 2.1) 1198 / 1114, 8192 tokens beside 32 x 32K
        // (220, 1.1) 743 / 659; 32 / 8 heads 4096 at 16K beside 32 x 32K (385, 0.95) 1181 / 1105, 8192 beside 32 x 8K (220,
        // 2.2) 620 / 580; 32 / 32 heads 2048 at 32K beside 16 x 4K (426, 3.2) 1089 / 1036.  Outside: ratio 0.54 (220)
        // 903 / 868, 0.24 (96) 579 / 692; 3.8 (385) 920 / 906, 6.6 (220) 539 / 549; 96 us of matrix time, ratio 1.9 268 /
        // 279; an item for every second slot (210, 1.04) 737 / 735.  (Towards long decode streams the two are level somewhere
        // between 0.24 and 0.54; the line keeps clear of that.)
        double decode_tokens = 0.0;
        for (int r = prm.n_prefill; r < n_req; ++r) decode_tokens += seq_meta[4 * r + 2];
        const double decode_time = decode_tokens * prm.n_kv_heads * prm.head_dim * 4.0 / 8.0e12;
        // (Rates and times are those of the whole chip.  A plan for fewer units keeps to the workgroups of its fused launch,
        // where the prefill kernel has one per item.)
        plan.heavy_pays = prm.policy == POD_POLICY_AUTO && built && prm.n_decode > 0 && n_cus == kChipUnits &&
                          (int)plan.pitems.size() >= kSlotsPerUnit * n_cus && flop_time >= 200e-6 &&
                          flop_time >= 0.8 * decode_time && flop_time <= 3.3 * decode_time;
        // Which of the two a fused call runs depends on what other streams do, and its bits must not: the light decode kernel
        // leaves merging to the combine kernel, which adds the weights in another order, so the units of the default
        // configuration do as well.  (Only decode units of a given length come here: cut by the planner, streams as long as
        // the rule asks for take several units a wavefront.  The combine kernel is 5 us of a launch of 500 and more.)
        if (plan.heavy_pays) {
            plan.units_merge = false;
            plan.unit_splits.clear();
        }
    }

    // ---- workspace layout --------------------------------------------------------------
    plan.ws_bytes = lay_out(plan, plan.pitems.size(), plan.dunits.size(), plan.merge_rows.size(), plan.n_partial_rows);
    return POD_OK;
}

}  // namespace pod
