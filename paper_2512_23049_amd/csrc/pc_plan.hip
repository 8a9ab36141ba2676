// Host side of the library: a call's validation and position resolution, the split of a batch into
// work items (prefill, per-call decode, shared decode), staging, and the launch of the plan builder.
#include "pc_host.h"

#include <numeric>
#include <type_traits>

int32_t pc_resolve(pc_cache *c, const pc_call *call, int idx, Resolved &out)
{
    if (!call) return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: null", idx);
    if (call->n_sel < 0 || (call->n_sel > 0 && !call->sel))
        return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: bad parent list", idx);
    if (call->n_q < 1) return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: n_q = %d must be >= 1", idx, call->n_q);
    const int64_t maxp = c->cfg.max_position;
    // a listed message becomes one (extent record, start) pair per extent that holds tokens
    out.sel.resize((size_t)call->n_sel);
    out.entry_start.resize((size_t)call->n_sel);
    size_t n_out = 0;
    int64_t nxt = 0, n_kv = 0, tiles = 0;
    const HostMsg *msgs = c->msgs.data();                // (raw pointers: long lists are resolved on every step of a decode loop)
    const int32_t n_msgs = (int32_t)c->msgs.size();
    const pc_sel *list = call->sel;
    int32_t *starts = out.entry_start.data();
    int2 *dst = out.sel.data();
    for (int e = 0; e < call->n_sel; ++e) {
        const int32_t m = list[e].msg_id;
        if ((uint32_t)m >= (uint32_t)n_msgs || !msgs[m].live || msgs[m].is_ext)
            return pc_fail(c, PC_ERR_BAD_MSG_ID, "call %d: parent %d names unknown message %d", idx, e, m);
        const HostMsg &hm = msgs[m];
        const int64_t len = hm.next < 0 ? hm.len : chain_len(c, m);
        const int64_t s = list[e].start_pos == PC_POS_AUTO ? nxt : (int64_t)list[e].start_pos;
        if (s < -maxp || s + len - 1 > maxp)
            return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: parent %d spans positions [%lld, %lld], limit is +-%lld", idx, e,
                        (long long)s, (long long)(s + len - 1), (long long)maxp);
        starts[e] = (int32_t)s;
        dst[n_out++] = make_int2(m, (int)s);
        tiles += (hm.len + PC_TILE - 1) / PC_TILE;
        if (hm.next >= 0) {                              // its further extents
            int64_t at = s + hm.len;
            for (int32_t r = hm.next; r >= 0; r = msgs[r].next) {
                const int32_t rl = msgs[r].len;
                if (rl > 0) {
                    out.sel.resize(out.sel.size() + 1);
                    dst = out.sel.data();
                    dst[n_out++] = make_int2(r, (int)at);
                }
                at += rl; tiles += (rl + PC_TILE - 1) / PC_TILE;
            }
        }
        nxt = s + len; n_kv += len;
    }
    out.sel.resize(n_out);
    out.self_msg = -1; out.self_len = 0;
    int64_t s_self = call->self_start == PC_POS_AUTO ? nxt : (int64_t)call->self_start;
    int64_t self_total = 0;
    if (call->self_msg >= 0) {
        if (!known(c, call->self_msg)) return pc_fail(c, PC_ERR_BAD_MSG_ID, "call %d: new message id %d unknown", idx, call->self_msg);
        self_total = chain_len(c, call->self_msg);
        if (call->n_q > self_total)
            return pc_fail(c, PC_ERR_SHAPE, "call %d: n_q = %d exceeds the new message's %lld tokens", idx, call->n_q, (long long)self_total);
        if (s_self < -maxp || s_self + self_total - 1 > maxp)
            return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: new message spans positions beyond +-%lld", idx, (long long)maxp);
        // The causal part lives in the message's last extent; the extents before it are seen whole by
        // every query row, like parents.
        const int32_t last = chain_last(c, call->self_msg);
        if (call->n_q > c->msgs[(size_t)last].len)
            return pc_fail(c, PC_ERR_SHAPE, "call %d: the %d query rows must lie in the new message's last extent (%d tokens)", idx,
                        call->n_q, c->msgs[(size_t)last].len);
        int64_t at = s_self;
        for (int32_t r = call->self_msg; r != last; r = c->msgs[(size_t)r].next) {
            const int32_t rl = c->msgs[(size_t)r].len;
            if (rl > 0) out.sel.push_back(make_int2(r, (int)at));
            at += rl; tiles += (rl + PC_TILE - 1) / PC_TILE;
        }
        out.self_msg = last;
        out.self_len = c->msgs[(size_t)last].len;
        out.self_start = (int32_t)at;
        n_kv += self_total; tiles += (out.self_len + PC_TILE - 1) / PC_TILE;
    } else if (call->self_msg != -1) {
        return pc_fail(c, PC_ERR_BAD_MSG_ID, "call %d: self_msg must be -1 or a message id", idx);
    } else if (s_self < -maxp || s_self + call->n_q - 1 > maxp) {
        return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: query positions beyond +-%lld", idx, (long long)maxp);
    }
    out.msg_start = (int32_t)s_self;
    if (out.self_msg < 0) out.self_start = (int32_t)s_self;
    out.n_q = call->n_q;
    out.q_pos.resize(call->n_q);
    const int64_t tok0 = out.self_msg >= 0 ? self_total - call->n_q : 0;
    for (int r = 0; r < call->n_q; ++r) {
        const int64_t p = call->q_pos ? (int64_t)call->q_pos[r] : s_self + tok0 + r;
        if (p < -maxp || p > maxp) return pc_fail(c, PC_ERR_INVALID_ARG, "call %d: query position %lld beyond +-%lld", idx, (long long)p, (long long)maxp);
        out.q_pos[r] = (int32_t)p;
    }
    if (n_kv > INT32_MAX / 2) return pc_fail(c, PC_ERR_SHAPE, "call %d: gathers %lld tokens, too many", idx, (long long)n_kv);
    out.n_kv = n_kv; out.tiles = (int32_t)tiles;
    return PC_OK;
}

PlanLayout make_layout(int n_calls, int total_q, int total_seg, int n_dec, int n_pre, int n_pre_pk,
                       int64_t part_rows, int64_t total_tiles, int H_q, int D,
                       size_t n_sh_groups = 0, size_t n_sh_segs = 0, size_t n_sh_items = 0, size_t n_sh_pos = 0,
                       size_t n_kg_items = 0, int64_t kg_tiles = 0, int H_kv = 1, size_t n_tok = 0,
                       size_t n_bwd_rb = 0, size_t n_bwd_keys = 0, size_t bwd_units = 0, size_t bwd_splits = 0, size_t part_esize = sizeof(uint16_t), size_t n_merge = 0)
{
    PlanLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
    // staged: arrays in 32-byte steps, nothing for a list that is empty (small blocks travel in the plan builder's arguments)
    auto put = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 32); return at; };
    L.calls = put(sizeof(PcCallDesc) * (size_t)n_calls);
    L.sel = put(sizeof(int2) * (size_t)total_seg);
    L.q_pos = put(sizeof(int32_t) * (size_t)total_q);
    L.merge_rows = put(sizeof(PcMergeRow) * n_merge);
    L.items_dec = put(sizeof(PcItem) * (size_t)n_dec);
    L.items_pre = put(sizeof(PcItem) * (size_t)n_pre);
    L.items_pk = put(sizeof(PcItem) * (size_t)n_pre_pk);
    L.sh_groups = put(sizeof(PcShGroup) * n_sh_groups);
    L.sh_segs = put(sizeof(PcShSeg) * n_sh_segs);
    L.sh_items = put(sizeof(PcShItem) * n_sh_items);
    L.sh_pos = put(sizeof(int32_t) * n_sh_pos);
    L.kg_items = put(sizeof(PcGatherItem) * n_kg_items);
    L.tok_items = put(sizeof(PcTokenItem) * n_tok);
    L.bwd_rb = put(sizeof(int2) * n_bwd_rb);
    L.bwd_keys = put(sizeof(PcBwdKeyItem) * n_bwd_keys);
    L.h2d_bytes = o;
    o = align_up(o, 256);
    L.segs = take(sizeof(PcSegment) * (size_t)std::max(total_seg, 1));
    L.seg_kvoff = take(sizeof(int32_t) * (size_t)std::max(total_seg, 1));
    L.rot_seg = take(sizeof(float2) * (size_t)std::max(total_seg, 1) * (D / 2));
    L.rot_q = take(sizeof(float2) * (size_t)std::max(total_q, 1) * (D / 2));
    L.rot_qw = take(D == 128 ? sizeof(float2) * (size_t)((std::max(total_q, 1) + 31) / 32) * 32 * (D / 2) : 0);   // whole blocks of 32 rows
    L.tiles = take(sizeof(PcTile) * (size_t)std::max<int64_t>(total_tiles, 1));
    L.sh_rot = take(sizeof(float2) * std::max<size_t>(n_sh_pos, 1) * (D / 2));
    L.part_o = take(part_esize * (size_t)std::max<int64_t>(part_rows, 1) * H_q * D);
    L.part_ml = take(sizeof(float) * (size_t)std::max<int64_t>(part_rows, 1) * H_q * 2);
    L.row_scalar = take(sizeof(float) * (size_t)std::max(total_q, 1) * H_q);      // one float per (row, head): the gradient path's Delta
    L.k_gather = take((size_t)std::max<int64_t>(kg_tiles, 0) * PC_TILE * (size_t)H_kv * (size_t)D * 2);   // bf16 keys ...
    L.v_gather = take((size_t)std::max<int64_t>(kg_tiles, 0) * PC_TILE * (size_t)H_kv * (size_t)D * 2);   // ... and values of the calls that gather
    L.kg_norm = take(sizeof(float) * (size_t)std::max<int64_t>(kg_tiles, 0) * (size_t)H_kv);             // ... and the largest key norm of each of their tiles
    L.bwd_qt = take(sizeof(float4) * 1024 * bwd_units);                          // gradient: per-unit buffers of one set of launches
    L.bwd_qp = take((size_t)4 * 8192 * bwd_units);
    L.bwd_delta = take(sizeof(float) * 32 * bwd_units * bwd_splits);
    L.bwd_dq = take(sizeof(float4) * 1024 * bwd_units * bwd_splits);
    L.bwd_stat = take(sizeof(float2) * 32 * bwd_units);
    L.total = o;
    return L;
}

// a decode call's parents in ascending cache-slot order; ties (a message listed twice) go by start
static void sort_by_slot(const pc_cache *c, Resolved &r)
{
    if (r.sel.size() < 2) return;
    // While ids ascend with slots (no freed span was ever refilled) and the list is long, one pass over
    // a table indexed by message id does it; a message listed twice sends the call to the general sort.
    if (c->slots_in_id_order && r.sel.size() * 8 > c->msgs.size()) {
        static thread_local std::vector<int32_t> where;
        static thread_local std::vector<int2> sorted;
        where.assign(c->msgs.size(), -1);
        bool twice = false;
        for (size_t e = 0; e < r.sel.size() && !twice; ++e) {
            int32_t &w = where[(size_t)r.sel[e].x];
            twice = w >= 0;
            w = (int32_t)e;
        }
        if (!twice) {
            sorted.clear();
            for (size_t m = 0; m < where.size(); ++m)
                if (where[m] >= 0) sorted.push_back(r.sel[(size_t)where[m]]);
            r.sel.assign(sorted.begin(), sorted.end());
            return;
        }
    }
    struct SortKey { uint64_t key; int2 v; };
    static thread_local std::vector<SortKey> keys;
    keys.resize(r.sel.size());
    for (size_t e = 0; e < r.sel.size(); ++e)
        keys[e] = {((uint64_t)(uint32_t)c->msgs[(size_t)r.sel[e].x].slot_start << 32) | ((uint32_t)r.sel[e].y ^ 0x80000000u), r.sel[e]};
    std::sort(keys.begin(), keys.end(), [](const SortKey &a, const SortKey &b) { return a.key < b.key; });
    for (size_t e = 0; e < r.sel.size(); ++e) r.sel[e] = keys[e].v;
}

// Shared decode (message-major): runs of consecutive one-row calls are cut into groups of up to
// 32 * 8 / g rows; a group whose calls overlap enough walks the union of their messages once.
struct SharedPlan {
    std::vector<char> in_shared;                 // per call
    std::vector<PcShGroup> groups;
    std::vector<PcShSeg> segs;
    std::vector<PcShItem> items;
    std::vector<char> wide;                      // per group: partial outputs in fp32
    std::vector<int32_t> pos;                    // rotation positions, q_pos - start + stored base, PC_SH_ABSENT where a row does not list the message
};

// The ways of a batch of one-row calls, in us a step with launches and merge.  Tiles (K and V of 32 keys, a KV head) are shared out over the
// compute units.  From 70 batches of 2 to 64 calls over 1 to 400 messages, 8 KV heads, 4 and 8 heads a KV head:
//   own walks     OWN_FIXED, with lists in pinned memory OWN_PINNED, and the longer of what one compute unit has to do (see one_splits) and the tiles:
//                 TILE_NEW a tile of the union, TILE_STEP a further pass over a message that every call lists (they meet it in step, in the L2),
//                 TILE_AGAIN one over any other
//   by message    RUN_FIXED, RUN_PART a part of the row that has most, and TILE_NEW a tile of the union or TILE_PASS a pass of PC_RUN_ROWS rows (16 / g at most)
//   shared walk   SHARED_FIXED and SHARED_TILE a tile of the groups' unions
// 64 calls over a system message and 8 of 512 others: 127 us by walks of their own, 111 by message; 8 over 100 of 300: 78 and 52; 16 over 20
// of 60 and a system message: 40 shared, 30 by message; 44 over 21 of 23 short ones: 44 shared, 30 own; 6 over 250: 63 own, 54 shared.
// In a batch with longer calls, whose launches are there anyway, a group takes the shared walk if its calls list SHARE_MIN times the
// tokens of the union: a union tile costs a workgroup 8.7 ns with the chip full, a tile streamed by one call 1.5 to 1.7.
constexpr double TILE_NEW = 0.79, TILE_AGAIN = 0.36, TILE_STEP = 0.15, TILE_PASS = 0.33, OWN_FIXED = 8.0, OWN_PINNED = 14.0, RUN_FIXED = 20.5, RUN_PART = 0.045,
                 SHARED_FIXED = 30.0, SHARED_TILE = 1.05;
// What they were not taken from: 1,020 drawn batches, 60 for each of 17 pairs of 1 to 32 KV heads and 1 to 8 heads a KV head, every one timed all three ways.
// The way chosen takes 1.028 times the least of the three in the mean (1.01 to 1.04 pair by pair, 1.73 at most), and 0.78 of what the sharing ratio
// alone had chosen; none over 15 us takes more than 1.03 of that.  One price is 14 to 25 % off (one deviation), the shared walk's too high where lists share
// much: SHARE_LEAN (it was taken with the rotations in a launch of their own, 3 us more).
constexpr double SHARE_LEAN = 0.8;
// What a step takes the host, in us: resolving, sorting and staging the lists of calls that walk on their own in one launch, and enqueuing it; and
// COLLECT_ENTRY for a union.  (5 calls over 996 of 1,228 messages, one KV head: 36 us a step, 52 with a union and walks of their own after all; 54
// over 110 of 157, two, 41 and 56; 20 over 298 of 1,154, two, 48 and 75.  Fitted to 18 batches of 5 to 155 calls, 775 to 16 thousand entries.)
constexpr double HOST_FIXED = 6.0, HOST_CALL = 0.1, HOST_ENTRY = 0.0055, COLLECT_ENTRY = 0.0045;
constexpr double RUN_START = 1.5;                        // a run's start and end, in passes
constexpr double SHARE_MIN = 6.0;
// entries of a group's rotation table, a row and a message of the union each: 512 bytes, 256 MB in all
constexpr size_t UNION_ENTRIES = (size_t)1 << 19;
// rows with more splits than this are merged by four lanes per 8 dimensions
constexpr int MERGE_MANY_SPLITS = 8;

// Lists that a thread keeps from one call to the next (fresh pages for them cost more than filling them) are given back when a batch made them
// longer than KEPT_BYTES each.
constexpr size_t KEPT_BYTES = (size_t)4 << 20;
template <typename T> static void keep(std::vector<T> &v) { if (v.capacity() * sizeof(T) > KEPT_BYTES) std::vector<T>().swap(v); }

// The union of the lists of some one-row calls: which messages there are, who lists each, and where.
struct Union {
    struct Seg { int32_t msg, occ, len, rows; int64_t slot; uint32_t vis[8]; };      // bit n of vis: row n lists it; rows: how many do
    std::vector<Seg> segs;                                // as they turn up
    std::vector<int32_t> pos;                             // [seg][row] q_pos - start + stored base, PC_SH_ABSENT where the row does not list it
    std::vector<int32_t> order;                           // segs in cache-slot order
    int n_rows = 0;
    int64_t call_tiles = 0, tiles = 0;
};

// (false: more messages than segs_max, or a position that 32 bits do not hold.  Raw pointers, one pass: the lists of long calls are collected on every step of a decode loop)
static bool collect_union(pc_cache *c, std::vector<Resolved> &res, int i, int n_rows, size_t segs_max, Union &un)
{
    const HostMsg *msgs = c->msgs.data();
    std::vector<std::pair<int64_t, int32_t>> extra;       // (msg << 20 | occurrence) -> seg, for repeats within a call
    un.segs.clear(); un.pos.clear();
    un.n_rows = n_rows; un.call_tiles = 0;
    bool far = false;
    auto listed = [&](int64_t p) {                       // (INT32_MIN is PC_SH_ABSENT)
        far |= p < -INT32_MAX || p > INT32_MAX;
        return (int32_t)p;
    };
    const uint32_t epoch = new_marks(c);                 // value: the message's place in segs
    pc_cache::Mark *marks = c->marks.data();
    Union::Seg *segs = un.segs.data();
    int32_t *pos = un.pos.data();
    auto add = [&](int32_t m, int32_t occ) {
        un.segs.push_back(Union::Seg{m, occ, msgs[m].len, 0, msgs[m].slot_start, {0, 0, 0, 0, 0, 0, 0, 0}});
        un.pos.resize(un.pos.size() + (size_t)n_rows, PC_SH_ABSENT);
        segs = un.segs.data(); pos = un.pos.data();
        return (int32_t)un.segs.size() - 1;
    };
    auto lookup = [&](int32_t m, int32_t occ) -> int32_t {              // -1: one too many
        if (occ == 0 && marks[m].epoch == epoch) return marks[m].value;
        const int64_t key = ((int64_t)m << 20) | occ;
        if (occ > 0) for (auto &kv : extra) if (kv.first == key) return kv.second;
        if (un.segs.size() >= segs_max) return -1;
        const int32_t u = add(m, occ);
        if (occ == 0) { marks[m] = pc_cache::Mark{epoch, u}; return u; }
        extra.push_back({key, u});
        return u;
    };
    for (int r = 0; r < n_rows; ++r) {
        Resolved &rc = res[(size_t)(i + r)];
        un.call_tiles += rc.tiles;
        // the union is sorted once, below: a call's own list is needed in slot order only where it names a message
        // twice (its occurrences are told apart by their starts)
        int32_t self_occ = 0;
        const int64_t q0 = rc.q_pos[0];
        const uint32_t word = (uint32_t)r >> 5, bit = 1u << (r & 31);
        uint32_t twice = 0;
        auto walk = [&](auto bounded) {                  // (bounded: every sum of a position, a start and a base fits 32 bits)
            for (const int2 *e = rc.sel.data(), *end = e + rc.sel.size(); e < end; ++e) {
                const HostMsg &hm = msgs[e->x];
                if (hm.len <= 0) continue;
                self_occ += e->x == rc.self_msg;
                int32_t u = marks[e->x].value;
                if (marks[e->x].epoch != epoch && (u = lookup(e->x, 0)) < 0) return false;      // (here: a row's list may be as long as the table of messages)
                uint32_t &vis = segs[u].vis[word];
                twice |= vis & bit;
                vis |= bit;
                int32_t &at = pos[(size_t)u * (size_t)n_rows + (size_t)r];
                if constexpr (decltype(bounded)::value) at = (int32_t)q0 - e->y + hm.base_pos;
                else at = listed(q0 - e->y + hm.base_pos);
            }
            return true;
        };
        // (a base is at most three largest positions out: that of a further extent)
        if (!(c->cfg.max_position <= INT32_MAX / 6 ? walk(std::true_type{}) : walk(std::false_type{}))) return false;
        auto enter = [&](int32_t u, int32_t start, int32_t base) {
            if (u < 0) return false;
            segs[u].vis[word] |= bit;
            pos[(size_t)u * (size_t)n_rows + (size_t)r] = listed(q0 - start + base);
            return true;
        };
        if (twice) {
            for (size_t u = 0; u < un.segs.size(); ++u) {             // the row again, from nothing
                segs[u].vis[word] &= ~bit;
                pos[u * (size_t)n_rows + (size_t)r] = PC_SH_ABSENT;
            }
            sort_by_slot(c, rc);
            int32_t prev = -1, occ = 0;
            for (const int2 &e : rc.sel) {
                occ = (e.x == prev) ? occ + 1 : 0;
                prev = e.x;
                if (msgs[e.x].len > 0 && !enter(lookup(e.x, occ), e.y, msgs[e.x].base_pos)) return false;
            }
        }
        // the call's own tail: one row, one token from the end -> all of it visible
        if (rc.self_msg >= 0 && rc.self_len > 0 && !enter(lookup(rc.self_msg, self_occ), rc.self_start, msgs[rc.self_msg].base_pos)) return false;
    }
    if (far) return false;
    un.tiles = 0;
    const int words = (n_rows + 31) / 32;                // (counted once, in the words there are: the processor's own count is not in the baseline this is built for)
    for (Union::Seg &u : un.segs) {
        un.tiles += (u.len + PC_TILE - 1) / PC_TILE;
        for (int w = 0; w < words; ++w) u.rows += __builtin_popcount(u.vis[w]);
    }
    return true;
}

static void order_union(Union &un)
{
    un.order.resize(un.segs.size());
    for (size_t u = 0; u < un.segs.size(); ++u) un.order[u] = (int32_t)u;
    const auto &usegs = un.segs;
    std::sort(un.order.begin(), un.order.end(), [&](int32_t a, int32_t b) {
        return usegs[(size_t)a].slot != usegs[(size_t)b].slot ? usegs[(size_t)a].slot < usegs[(size_t)b].slot
                                                              : usegs[(size_t)a].occ < usegs[(size_t)b].occ; });
}

static int rows_per_run(const pc_cache *c) { return std::max(1, std::min(PC_RUN_ROWS, 16 / c->g)); }

// Decode by message: what it needs whatever its runs are.  Queries go to LDS by direct loads of 16 bytes, whose addresses have to be multiples of
// that (the other ways load them into registers); angles are those of the short series.
static bool runs_possible(const pc_cache *c, const Planned &P, const Union &un)
{
    return rows_per_run(c) >= 2 && un.tiles > 0 && ((uintptr_t)P.q & 15) == 0 && c->cfg.max_position < 1 << 28 && c->cfg.rope_theta >= 1.f &&
           un.segs.size() * (size_t)un.n_rows <= 32768;
}
static size_t runs_layout(const pc_cache *c, int n_calls, size_t n_runs, int64_t n_parts, size_t n_tok, PlanLayout &L)
{
    const size_t off_merge = sizeof(PcMsgRun) * n_runs, off_tok = align_up(off_merge + sizeof(PcMergeRow) * (size_t)n_calls, 16);
    const size_t H_q = (size_t)c->cfg.n_q_heads;
    L = PlanLayout{};
    L.part_ml = align_up(sizeof(float) * (size_t)n_parts * H_q * (size_t)c->D, 256);
    const size_t bytes = off_tok + sizeof(PcTokenItem) * n_tok;
    // (a recorded call's launches leave its lists, the runs short, where the parts will be)
    const size_t parts = L.part_ml + sizeof(float) * 4 * (size_t)n_parts * H_q, recorded = align_up(sizeof(PcMsgRunShort) * n_runs + bytes - off_merge, 16);
    L.calls = align_up(std::max(parts, recorded), 256);  // the runs, then the rows to merge
    L.merge_rows = L.calls + off_merge;
    L.rot_seg = align_up(L.calls + bytes, 1024);
    L.total = L.rot_seg + n_runs * PC_RUN_ROWS * sizeof(float2) * 64;
    L.tok_items = off_tok;
    return bytes;
}
// the lists and parts fit what every caller has (a step's tokens left out: with them or without, a batch goes the same way)
static bool runs_fit(const pc_cache *c, int n_calls, size_t n_runs, int64_t n_parts)
{
    PlanLayout L;
    return n_runs < 65535 && runs_layout(c, n_calls, n_runs, n_parts, 0, L) <= HOST_READ_BYTES && L.total <= PC_STATIC_WS_BYTES;
}

// The splits of a call over T tiles in the one launch of a batch with so many (call, KV head) pairs: those with the least of ONE_TILE us a tile for each
// round of 256 workgroups, plus, if there is more than one, a merge of ONE_MERGE and ONE_PART a workgroup (us; 1 to 16 calls over 8 to 400 tiles, 1 to 32 splits:
// this choice is within 5 % of the best of them.  One call over 200 tiles: 63 us unsplit, 13.6 in 32; eight over 16: 11.7 unsplit, 13.3 in 2 or 4).
// (two rounds; further splits never pay.  Above PC_ONE_COUNTERS pairs there is none, and no counter in use)
constexpr double ONE_TILE = 0.28, ONE_MERGE = 2.0, ONE_PART = 0.009;
static int one_splits(int pairs, int T)
{
    const int most = std::min(std::max(1, std::min(MAX_SPLITS, 2 * PC_ONE_COUNTERS / pairs)), std::max(1, T / 4));
    int best = 1;
    double best_us = 1e30;
    for (int ns = 1; ns <= most; ++ns) {
        const int wgs = pairs * ns;
        const double us = ONE_TILE * ((T + ns - 1) / ns) * ((wgs + 255) / 256) + (ns > 1 ? ONE_MERGE + ONE_PART * wgs : 0.0);
        if (us < best_us) { best_us = us; best = ns; }
    }
    const int chunk = std::max(1, (T + best - 1) / best);
    return std::max(1, (T + chunk - 1) / chunk);
}

// What a batch's own walks cost: the launch, and the least that their tiles take, which is what the busiest compute unit has to do.  Under few KV heads
// that is more than the tiles shared out evenly: 36 calls over 3 of 10 messages and a long system message, 4 KV heads, 42 us for 27.  (510 drawn
// batches over 17 pairs of 1 to 32 KV heads and 1 to 8 heads a KV head: measured 0.88 to 1.56 times the price, pair by pair, by the tiles alone; so 0.85 to 1.09.)
struct OwnCost {
    double fixed, busiest;
    bool one_launch;                                     // as far as lists go that a wave cannot hold
    double with(double tiles_us) const { return fixed + std::max(busiest, tiles_us); }
};
static OwnCost own_cost(const pc_cache *c, const std::vector<Resolved> &res, size_t entries, int64_t all_tiles)
{
    const int n_calls = (int)res.size(), H_kv = c->cfg.n_kv_heads;
    size_t items = 0;
    int longest = 0;                                     // tiles of a split
    OwnCost k{0, 0, true};
    for (const Resolved &r : res) {
        const int ns = one_splits(n_calls * H_kv, r.tiles);
        items += (size_t)ns;
        longest = std::max(longest, (r.tiles + ns - 1) / ns);
        k.one_launch = k.one_launch && r.sel.size() < (size_t)ns * PC_ONE_SEGS;
    }
    const double wgs = (double)items * H_kv, rounds = std::ceil(wgs / 256);
    const bool pinned = (sizeof(PcOneCall) + 4) * (size_t)n_calls + sizeof(int2) * entries + sizeof(PcOneItem) * items > PC_ARG_BYTES;
    k.fixed = pinned ? OWN_PINNED : OWN_FIXED;
    k.busiest = ONE_TILE * std::max((double)longest, rounds * (double)all_tiles / (double)items) + (items > (size_t)n_calls ? ONE_MERGE + ONE_PART * wgs : 0.0);
    return k;
}

// what a batch's own walks and its runs by message cost
constexpr double NOT_BY_MESSAGE = 1e30;
struct DecodeCost { double own, by_message; int64_t passes, n_groups; };
static DecodeCost decode_cost(const pc_cache *c, const Planned &P, const Union &un, const OwnCost &oc)
{
    const int n_calls = un.n_rows, per_run = rows_per_run(c);
    const double per_cu = c->cfg.n_kv_heads / 256.0;
    int64_t again = 0, in_step = 0, listed = 0;
    DecodeCost k{0, 0, 0, 0};
    for (const Union::Seg &u : un.segs) {
        const int n = u.rows, t = (u.len + PC_TILE - 1) / PC_TILE, gr = (n + per_run - 1) / per_run;
        k.passes += (int64_t)gr * t; k.n_groups += gr; listed += n;
        (n == n_calls ? in_step : again) += (int64_t)(n - 1) * t;
    }
    k.own = oc.with(per_cu * (TILE_NEW * (double)un.tiles + TILE_AGAIN * (double)again + TILE_STEP * (double)in_step));
    k.by_message = RUN_FIXED + RUN_PART * (double)listed / n_calls + per_cu * std::max(TILE_PASS * ((double)k.passes + RUN_START * (double)k.n_groups), TILE_NEW * (double)un.tiles);
    // (a part per row that lists a message, and a run per group of them, are the least there is: for long lists that is all it takes to know, and
    // the search for the runs is not begun)
    if (!runs_possible(c, P, un) || !runs_fit(c, n_calls, (size_t)k.n_groups, listed)) k.by_message = NOT_BY_MESSAGE;
    return k;
}

static bool plan_runs(pc_cache *c, Planned &P, Union &un, const DecodeCost &cost, hipStream_t st, int32_t &rc);

// the splits of a group's union: as many as fill the chip together
static int shared_splits(const pc_cache *c, size_t n_groups, int T)
{
    const int64_t workgroups = (int64_t)n_groups * c->cfg.n_kv_heads;
    const int ns = std::max(1, std::min(MAX_SPLITS, c->decode_tiles_per_split > 0 ? (T + c->decode_tiles_per_split - 1) / c->decode_tiles_per_split
                                                                                  : (int)std::min<int64_t>((256 + workgroups - 1) / workgroups, std::max(1, T / 8))));
    const int chunk = std::max(1, (T + ns - 1) / ns);
    return std::max(1, (T + chunk - 1) / chunk);
}

// the calls of a union, the first of them `first`, as a group of the shared walk
static void add_group(SharedPlan &sp, Union &un, int first, int row0, bool wide)
{
    order_union(un);
    const int n_rows = un.n_rows;
    PcShGroup gr{};
    gr.seg_off = (int32_t)sp.segs.size(); gr.n_seg = (int32_t)un.segs.size();
    gr.row0 = row0; gr.n_rows = n_rows; gr.rot_off = (int32_t)sp.pos.size();
    gr.n_splits = 1; gr.part_off = 0;
    int32_t tile_off = 0;
    sp.segs.reserve(sp.segs.size() + un.segs.size());
    sp.pos.reserve(sp.pos.size() + un.pos.size());
    for (int32_t k : un.order) {
        const Union::Seg &u = un.segs[(size_t)k];
        PcShSeg sg{};
        sg.slot_start = (int32_t)u.slot; sg.len = u.len; sg.tile_off = tile_off;
        std::copy(u.vis, u.vis + 8, sg.vis);
        tile_off += (u.len + PC_TILE - 1) / PC_TILE;
        sp.segs.push_back(sg);
        const int32_t *row = un.pos.data() + (size_t)k * (size_t)n_rows;
        sp.pos.insert(sp.pos.end(), row, row + n_rows);
    }
    gr.n_tiles = tile_off;
    sp.groups.push_back(gr);
    sp.wide.push_back(wide);
    for (int k = 0; k < n_rows; ++k) sp.in_shared[(size_t)(first + k)] = 1;
}

static void drop_groups(SharedPlan &sp)
{
    std::fill(sp.in_shared.begin(), sp.in_shared.end(), 0);
    sp.groups.clear(); sp.wide.clear(); sp.segs.clear(); sp.pos.clear();
}

// The table of a group has an entry for every row and message of the union, listed or not, so that a batch the calls' own walks have room
// for may not fit the fixed workspace.
static bool groups_fit(const pc_cache *c, size_t n_groups, size_t rows, size_t segs, size_t entries, size_t items, int64_t part_rows)
{
    const PlanLayout l = make_layout((int)rows, (int)rows, 0, 0, 0, 0, part_rows, 0, c->cfg.n_q_heads, c->D, n_groups, segs, items, entries,
                                     0, 0, c->cfg.n_kv_heads, 0, 0, 0, 0, 0, sizeof(uint16_t), rows);
    return l.total <= PC_STATIC_WS_BYTES && l.h2d_bytes <= STAGE_BYTES;
}
// the groups so far, and one more of a union (null: none), as groups of a batch of n_groups
static bool groups_fit(const pc_cache *c, const SharedPlan &sp, size_t n_groups, const Union *more)
{
    size_t rows = 0, items = 0, segs = sp.segs.size(), entries = sp.pos.size();
    int64_t part_rows = 0;
    auto add = [&](int tiles, int n, int wide) {
        const int ns = shared_splits(c, n_groups, tiles);
        rows += (size_t)n; items += (size_t)ns;
        if (ns > 1) part_rows += ((int64_t)ns * n) << wide;
    };
    for (size_t i = 0; i < sp.groups.size(); ++i) add(sp.groups[i].n_tiles, sp.groups[i].n_rows, sp.wide[i]);
    if (more) { add((int)more->tiles, more->n_rows, 1); segs += more->segs.size(); entries += more->pos.size(); }
    return groups_fit(c, n_groups, rows, segs, entries, items, part_rows);
}
// the same for n_calls calls in n_groups groups of a size, each with a union of so many messages and tiles and fp32 parts
static bool even_groups_fit(const pc_cache *c, size_t n_calls, size_t n_groups, size_t segs, int64_t tiles)
{
    const int ns = shared_splits(c, n_groups, (int)std::min<int64_t>(tiles, INT32_MAX / 2));
    return groups_fit(c, n_groups, n_calls, n_groups * segs, n_calls * segs, n_groups * (size_t)ns, ns > 1 ? 2 * (int64_t)ns * (int64_t)n_calls : 0);
}

// What calls list together in tiles, over the tiles of their union, if any two have as much in common as the one with the longest list and the next one
static double likely_ratio(pc_cache *c, const std::vector<Resolved> &res)
{
    size_t at = 0;
    for (size_t i = 1; i < res.size(); ++i) if (res[i].tiles > res[at].tiles) at = i;
    const Resolved &a = res[at], &b = res[(at + 1) % res.size()];
    const uint32_t epoch = new_marks(c);
    for (const int2 &e : a.sel) c->marks[(size_t)e.x].epoch = epoch;
    int64_t common = 0;
    for (const int2 &e : b.sel) common += c->marks[(size_t)e.x].epoch == epoch ? (c->msgs[(size_t)e.x].len + PC_TILE - 1) / PC_TILE : 0;
    const double n = (double)res.size(), p = (double)common / std::max(1, b.tiles);
    return p > 0 ? n * std::min(p, 1.0) / (1 - std::pow(1 - std::min(p, 1.0), n)) : 1;
}

enum class Way { OWN, BY_MESSAGE, SHARED, BY_RATIO };

// The way of a batch of nothing but one-row calls (the shared walk's groups, or the runs, are planned when this returns); BY_RATIO: as in a mixed batch.
static Way cheapest_way(pc_cache *c, Planned &P, int rows_max, SharedPlan &sp, Union &un, hipStream_t st, int32_t &rc)
{
    std::vector<Resolved> &res = P.res;
    const int n_calls = (int)res.size();
    const double per_cu = c->cfg.n_kv_heads / 256.0;
    size_t entries = 0, most_sel = 0;
    int64_t all_tiles = 0;
    int32_t most_tiles = 0;
    for (const Resolved &r : res) {
        entries += r.sel.size() + (r.self_msg >= 0 ? 1 : 0); most_sel = std::max(most_sel, r.sel.size()); all_tiles += r.tiles; most_tiles = std::max(most_tiles, r.tiles);
    }
    // (what no other way can undercut, whatever its calls share, is not collected: 0.5 to 1.5 us of a step of 10 to 30 short calls)
    if (OWN_PINNED + per_cu * TILE_NEW * (double)all_tiles < 1.2 * RUN_FIXED) return Way::OWN;
    // The longest list is the least a union can be, and the other two ways gain the most on walks of their own there
    const OwnCost oc = own_cost(c, res, entries, all_tiles);
    const double longest = (double)most_tiles;
    const double on_own = oc.with(per_cu * (TILE_NEW * longest + TILE_AGAIN * ((double)all_tiles - longest)));
    const double by_shared = ((double)all_tiles >= SHARE_MIN * longest ? SHARE_LEAN : 1.0) * (SHARED_FIXED + SHARED_TILE * per_cu * longest);
    const double by_message = RUN_FIXED + RUN_PART * (double)entries / n_calls + TILE_NEW * per_cu * longest;
    if (on_own < by_shared && 0.95 * on_own < by_message) return Way::OWN;
    // Long lists of short messages under few KV heads: the host takes longer than the GPU whichever way it is, and least if nothing is collected
    const double host = HOST_FIXED + HOST_CALL * n_calls + HOST_ENTRY * (double)entries;
    if (oc.one_launch && oc.with(per_cu * TILE_AGAIN * (double)all_tiles) < host) return Way::OWN;
    // (where it takes longer with a union, the union is collected if two of the lists have so much in common that it may be short)
    if (oc.one_launch && on_own < host + COLLECT_ENTRY * (double)entries && likely_ratio(c, res) < SHARE_MIN) return Way::OWN;
    const int n_groups = (n_calls + rows_max - 1) / rows_max;
    double own = oc.with(per_cu * TILE_AGAIN * (double)all_tiles), lean = 1;
    // (calls that make several groups of the shared walk are collected once more for it: 53 calls over 234 messages, whose host work is all of a
    // step, took 104 us and then 128)
    const bool whole = n_calls <= 256 && (n_groups == 1 || entries <= 2048);
    if (whole) {
        if (!collect_union(c, res, 0, n_calls, UNION_ENTRIES / (size_t)n_calls, un)) return n_groups == 1 ? Way::OWN : Way::BY_RATIO;
        const DecodeCost cost = decode_cost(c, P, un, oc);
        if ((double)un.call_tiles >= SHARE_MIN * (double)un.tiles) lean = SHARE_LEAN;
        const double shared = lean * (SHARED_FIXED + SHARED_TILE * per_cu * (double)un.tiles * (double)n_groups);
        own = cost.own;
        if (!c->host_only && cost.by_message < 0.95 * std::min(own, shared) && plan_runs(c, P, un, cost, st, rc)) return Way::BY_MESSAGE;
        if (rc != PC_OK || own < SHARED_FIXED) return Way::OWN;
    }
    // Groups of a size, or full ones and a rest, as the ratio forms them.  One that the ratio would not have formed, or not have given this walk (two calls
    // behind a full group: walks, and a launch, of their own), keeps its partial outputs in fp32, as the calls' own walks do, and takes it if
    // there is room for that.  (6 calls over 300 messages of 5 tiles, each listed by 5 of them, 8 heads a KV head: 118 us a step on their own.
    // 101 calls over 152 of 170, three groups and five calls: 176, with these in the walk 101.  139 over 14 of 15, 4 heads and 4 KV heads: in
    // groups of 64, 64 and 11 45, of 47 and 46 41.)
    bool even = n_groups > 1 && n_calls % rows_max != 0 && even_groups_fit(c, (size_t)n_calls, (size_t)n_groups, most_sel, most_tiles);
    double shared = SHARED_FIXED;                        // with what does not take the walk beside it
    bool any_wide = false, any_own = false;
    for (int i = 0, n_rows; i < n_calls; i += n_rows) {
        const int left = (n_calls - i + rows_max - 1) / rows_max;
        n_rows = even ? (n_calls - i + left - 1) / left : std::min(rows_max, n_calls - i);
        if (!(whole && n_rows == n_calls) && !collect_union(c, res, i, n_rows, UNION_ENTRIES / (size_t)n_rows, un)) return Way::BY_RATIO;
        if (even && i == 0 && !even_groups_fit(c, (size_t)n_calls, (size_t)n_groups, un.segs.size(), un.tiles)) {
            even = false;                                // (known from the first of them)
            n_rows = 0;
            continue;
        }
        const bool enough = !even && n_rows >= 2 && (double)un.call_tiles >= SHARE_MIN * (double)un.tiles;
        const bool take = un.tiles > 0 && un.tiles < INT32_MAX / 2 && (enough || groups_fit(c, sp, (size_t)n_groups, &un));
        shared += take ? SHARED_TILE * per_cu * (double)un.tiles : OWN_FIXED + per_cu * TILE_AGAIN * (double)un.call_tiles;
        if (own < lean * shared) return Way::OWN;
        if (take) add_group(sp, un, i, i, !enough);
        any_wide = any_wide || (take && !enough);
        any_own = any_own || !take;
    }
    if (sp.groups.empty()) return Way::OWN;
    // (with calls on their own beside it a group has more splits than was assumed)
    return any_wide && (any_own || !groups_fit(c, sp, sp.groups.size(), nullptr)) ? Way::BY_RATIO : Way::SHARED;
}

// rc != PC_OK: an error.  True: the whole batch goes by message (P.runs_*), and nothing else is to be planned
static bool plan_shared(pc_cache *c, Planned &P, const std::vector<int> &q_off, int g, SharedPlan &sp, hipStream_t st, int32_t &rc)
{
    std::vector<Resolved> &res = P.res;
    const int n_calls = (int)res.size();
    sp.in_shared.assign((size_t)n_calls, 0);
    if (c->decode_sharing == 1 || !(g == 1 || g == 2 || g == 4 || g == 8)) return false;
    const int rows_max = 32 * (8 / g);
    static thread_local Union un;
    struct Kept { ~Kept() { keep(un.segs); keep(un.pos); keep(un.order); } } kept;
    bool alone = c->decode_sharing == 0 && n_calls > 1 && c->decode_tiles_per_split == 0;
    for (const Resolved &r : res) alone = alone && r.n_q == 1;
    if (alone) {
        const Way way = cheapest_way(c, P, rows_max, sp, un, st, rc);
        if (way != Way::SHARED) drop_groups(sp);
        if (way != Way::BY_RATIO) return way == Way::BY_MESSAGE;
    }
    for (int i = 0; i < n_calls;) {
        if (res[i].n_q != 1) { ++i; continue; }
        int j = i;
        while (j < n_calls && res[j].n_q == 1 && j - i < rows_max) ++j;
        const int n_rows = j - i;
        // (the union holds each call's list: calls that list less than SHARE_MIN times the longest list cannot take this walk)
        int64_t sum_tiles = 0, longest = 0;
        for (int r = i; r < j; ++r) { sum_tiles += res[(size_t)r].tiles; longest = std::max<int64_t>(longest, res[(size_t)r].tiles); }
        if ((c->decode_sharing == 2 || (double)sum_tiles >= SHARE_MIN * (double)longest) &&
            collect_union(c, res, i, n_rows, UNION_ENTRIES / (size_t)n_rows, un) && un.tiles > 0 && un.tiles < INT32_MAX / 2 &&
            (c->decode_sharing == 2 || (n_rows >= 2 && (double)un.call_tiles >= SHARE_MIN * (double)un.tiles)))
            add_group(sp, un, i, q_off[(size_t)i], false);
        i = j;
    }
    return false;
}

// A decode batch by message (pc_decode_runs_bf16_kernel), if its lists and parts fit (decode_cost has seen to the rest).
static bool plan_runs(pc_cache *c, Planned &P, Union &un, const DecodeCost &cost, hipStream_t st, int32_t &rc)
{
    const int n_calls = un.n_rows, H_kv = c->cfg.n_kv_heads, per_run = rows_per_run(c);
    order_union(un);
    // the least share of tiles, and of runs' starts and ends, with which so many waves take all of them
    const double total = (double)cost.passes + RUN_START * (double)cost.n_groups;
    const int most_waves = std::max(1, std::min(PC_RUN_WAVES, 2048 / H_kv));
    auto take_of = [](double room, int left) { return std::min(left, std::max(1, (int)(room - RUN_START))); };
    double share = std::max(6.0, total / most_waves + 0.5);
    int n_waves = 0;
    size_t n_runs = 0;
    int64_t n_parts = 0;
    for (;; share *= 1.03) {
        n_waves = 1; n_runs = 0; n_parts = 0;
        double used = 0;
        for (int32_t k : un.order) {
            const Union::Seg &u = un.segs[(size_t)k];
            const int T = (u.len + PC_TILE - 1) / PC_TILE;
            for (int left = u.rows; left > 0; left -= per_run)
                for (int t = 0; t < T;) {
                    if (used + RUN_START + 1 > share) { ++n_waves; used = 0; }         // (less than a start and a tile left: the next wave)
                    const int take = take_of(share - used, T - t);
                    used += RUN_START + take; t += take;
                    ++n_runs; n_parts += std::min(left, per_run);
                }
        }
        if (n_waves <= most_waves) break;
    }
    if (!runs_fit(c, n_calls, n_runs, n_parts)) return false;
    static thread_local std::vector<PcMsgRun> runs;
    runs.clear();
    std::vector<int32_t> parts((size_t)n_calls, 0);
    int wave = 0;
    double used = 0;
    P.run_starts.first[0] = 0;
    for (int32_t k : un.order) {
        const Union::Seg &u = un.segs[(size_t)k];
        const int32_t *pos = un.pos.data() + (size_t)k * (size_t)n_calls;
        const int T = (u.len + PC_TILE - 1) / PC_TILE;
        PcMsgRun run{};
        run.msg = u.msg;
        int n = 0;
        auto emit = [&]() {
            for (int t = 0; t < T;) {
                if (used + RUN_START + 1 > share) { P.run_starts.first[++wave] = (uint16_t)runs.size(); used = 0; }
                const int take = take_of(share - used, T - t);
                run.tile0 = t; run.size = take | n << 28;
                for (int i = 0; i < n; ++i) run.part[i] = parts[(size_t)run.row[i]]++;
                runs.push_back(run);
                used += RUN_START + take;
                t += take;
            }
            n = 0;
        };
        for (int b = 0; b < (n_calls + 31) / 32; ++b)
            for (uint32_t v = u.vis[b]; v; v &= v - 1) {
                const int row = 32 * b + __builtin_ctz(v);
                run.row[n] = row;
                run.pos[n] = pos[row] - c->msgs[(size_t)u.msg].base_pos;
                if (++n == per_run) emit();
            }
        if (n > 0) emit();
    }
    P.run_starts.first[++wave] = (uint16_t)runs.size();
    // a call's parts lie one after the other, in slot order
    std::vector<int32_t> part0((size_t)n_calls);
    int32_t part_rows = 0;
    for (int i = 0; i < n_calls; ++i) { part0[(size_t)i] = part_rows; part_rows += parts[(size_t)i]; }
    for (PcMsgRun &r : runs)
        for (int i = 0; i < r.size >> 28; ++i) r.part[i] += part0[(size_t)r.row[i]];
    const size_t bytes = runs_layout(c, n_calls, runs.size(), part_rows, P.tok_items.size(), P.lay), off_merge = P.lay.merge_rows - P.lay.calls, off_tok = P.lay.tok_items;
    P.n_runs = (int)runs.size();
    char *rest;                                          // what is behind the runs
    if (pc_recorded(st)) {
        static_assert(PC_STATIC_WS_BYTES / (4 * 128 + 16) < 1 << 16, "a part's number in 16 bits: those of 128 dimensions and one head that fit");
        const size_t off_rest = sizeof(PcMsgRunShort) * runs.size();
        P.recorded.resize(align_up(off_rest + bytes - off_merge, 16));
        PcMsgRunShort *to = (PcMsgRunShort *)P.recorded.data();
        for (const PcMsgRun &r : runs) {
            PcMsgRunShort s{r.msg, r.tile0, r.size, {}, {}, {}};
            for (int i = 0; i < r.size >> 28; ++i) { s.row[i] = (uint8_t)r.row[i]; s.part[i] = (uint16_t)r.part[i]; s.pos[i] = r.pos[i]; }
            *to++ = s;
        }
        rest = P.recorded.data() + off_rest;
    } else {
        rc = pc_stage_acquire(c, bytes, &P.runs_slot);
        if (rc != PC_OK) return false;
        std::memcpy(P.runs_slot->host, runs.data(), off_merge);
        rest = (char *)P.runs_slot->host + off_merge;
    }
    PcMergeRow *rows = (PcMergeRow *)rest;
    for (int i = 0; i < n_calls; ++i) rows[i] = PcMergeRow{i, 2 * part0[(size_t)i], parts[(size_t)i] | PC_MERGE_WIDE, 1};
    P.runs_bytes = bytes;
    P.n_merge_rows = n_calls; P.n_merge_few = 0;
    if (!P.tok_items.empty()) std::memcpy(rest + (off_tok - off_merge), P.tok_items.data(), sizeof(PcTokenItem) * P.tok_items.size());
    P.runs = PcRuns{c->table_dev, nullptr, nullptr, n_waves};
    return true;
}

// Tokens of a call's parents; tiles of its new message (its last extent)
static int64_t parent_tokens(const pc_cache *c, const Resolved &r)
{
    int64_t n = 0;
    for (const int2 &e : r.sel) n += c->msgs[(size_t)e.x].len;
    return n;
}
static int own_tiles_of(const Resolved &r) { return r.self_msg >= 0 ? (r.self_len + PC_TILE - 1) / PC_TILE : 0; }
// Gather: a call with many query rows reads its keys and values from a packed copy (the gather pass: keys
// turned to the call's positions, no padding between messages), which moves 8192 bytes per listed token once
// (about 1.8 ns) and saves the turns of the queries at every message, the ragged tile at every message's end
// and the per-tile lookups: 15 to 25 % of the attention's own time, which is rows x heads x 0.47 ps per token.
// The copy pays from rows x query heads of about 20 thousand on; taken from 32768 on.  (Not with a fixed
// workspace, which the copy may not fit into.)
static bool gathers(const pc_cache *c, const Planned &P, const Resolved &r)
{
    return r.tiles > 0 && !P.fixed_ws && (c->key_gather == 2 || (c->key_gather == 0 && (int64_t)r.n_q * c->cfg.n_q_heads >= 32768));
}
// Tiles the prefill kernel walks for a call: those of the copy, or those of the cache
static int walked_tiles(const pc_cache *c, const Planned &P, const Resolved &r)
{
    return gathers(c, P, r) ? (int)((parent_tokens(c, r) + PC_TILE - 1) / PC_TILE) + own_tiles_of(r) : r.tiles;
}

// Tiles a split of the batch's prefill calls takes.  A workgroup fills a compute unit and takes about a start and an end of
// PRE_FIXED and PRE_TILE a tile (packed walk: PRE_TILE_PACKED), so a launch takes rounds of 256 of them: more splits shorten
// a round until there is one more of them, and their parts are written, read again and added by one more launch.
// (us; measured over 20 to 512 rows, 0.3 to 30 thousand tokens, one to four calls.  The rule before, as many splits as
// reach 256 workgroups, 16 tiles at least, put 1.1 rounds where one does: 200 rows x 64 heads over 3000 tokens
// 49 us for 5 splits of 56 groups, 33 us for 4.)
constexpr double PRE_FIXED = 9.0, PRE_TILE = 1.0, PRE_TILE_PACKED = 0.75, MERGE_FIXED = 4.5, PART_BYTES_US = 3.5e6;
constexpr int PRE_LEAST = 4;                             // tiles of a split: below, the start is all there is
// Partial results of a group (8 units of 32 rows: outputs of 2 bytes, a maximum and a sum) in one split; twice that in fp32.
// part_max: bytes all of them may take.
constexpr int64_t GROUP_PART_BYTES = 8 * 32 * (128 * 2 + 8);
static int prefill_chunk(const pc_cache *c, const Planned &P, const SharedPlan &sp, int64_t pre_groups, int64_t part_max)
{
    if (pre_groups >= 256) return INT32_MAX;             // the chip is full (prefill_tail sees to the last round)
    struct Shape { int64_t groups; int n_q, tiles; };    // consecutive calls of the same rows and tiles
    std::vector<Shape> shapes;
    int longest = 0;
    bool packed = false;
    for (size_t i = 0; i < P.res.size(); ++i) {
        const Resolved &r = P.res[i];
        if (sp.in_shared[i] || (int64_t)r.n_q * c->g <= 16) continue;
        const int64_t groups = (int64_t)((((r.n_q + 31) / 32) * c->g + P.pre_waves - 1) / P.pre_waves) * c->cfg.n_kv_heads;
        const int tiles = walked_tiles(c, P, r);
        if (!shapes.empty() && shapes.back().tiles == tiles && shapes.back().n_q == r.n_q) shapes.back().groups += groups;
        else shapes.push_back(Shape{groups, r.n_q, tiles});
        longest = std::max(longest, tiles);
        packed |= gathers(c, P, r);
    }
    const double tile = packed ? PRE_TILE_PACKED : PRE_TILE;
    int best = std::max(longest, 1), last = 0;
    double best_us = 0;
    const int most = (int)std::min<int64_t>({(int64_t)MAX_SPLITS, (int64_t)longest / PRE_LEAST, std::max<int64_t>(2, 1024 / pre_groups)});
    for (int k = 1; k <= std::max(most, 1); ++k) {
        const int chunk = (std::max(longest, 1) + k - 1) / k;
        if (chunk == last) continue;
        last = chunk;
        int64_t wgs = 0, part = 0;
        for (const Shape &sh : shapes) {
            const int ns = std::max(1, (sh.tiles + chunk - 1) / chunk);
            wgs += sh.groups * ns;
            if (ns > 1) part += sh.groups * ns * (sh.tiles < 32 ? 2 : 1);
        }
        if (k > 1 && part * GROUP_PART_BYTES > part_max) continue;
        // (8 * 32 * 128 partial outputs of 2 bytes, or 4, written and read)
        const double us = (double)((wgs + 255) / 256) * (PRE_FIXED + tile * chunk) + (part ? MERGE_FIXED + (double)part * 131072.0 / PART_BYTES_US : 0.0);
        if (k == 1 || us < best_us) { best_us = us; best = chunk; }
    }
    return best;
}

// A batch of more than 256 prefill groups runs in rounds, and a last round of a few groups takes as long as a full one: 280
// groups, 2 rounds for 1.1 rounds of work.  The items of that last round are split, so that it fills the chip as well.
// Returns how many of the last items (each n_kv_heads groups) are split, and into how many parts.
static std::pair<int, int> prefill_tail(const pc_cache *c, const Planned &P, const SharedPlan &sp, int64_t pre_groups, int64_t part_max)
{
    const int H_kv = c->cfg.n_kv_heads, g = c->g, per_round = 256 / H_kv;
    // (a row's heads must lie in one item, and a round hold whole items)
    if (pre_groups <= 256 || 8 % g != 0 || 256 % H_kv != 0 || c->prefill_tiles_per_split != 0) return {0, 1};
    int tiles = 0, kinds = 0;
    for (size_t i = 0; i < P.res.size(); ++i) {
        const Resolved &r = P.res[i];
        if (sp.in_shared[i] || (int64_t)r.n_q * g <= 16) continue;
        tiles = std::max(tiles, walked_tiles(c, P, r));
        kinds |= gathers(c, P, r) ? 2 : 1;
    }
    const int tail = (int)(pre_groups / H_kv % per_round);
    if (tail == 0 || kinds == 3) return {0, 1};          // (two kinds of calls are two launches)
    int best = 1;
    double best_us = 0;
    for (int k = 1; k <= std::min({MAX_SPLITS, tiles / PRE_LEAST, std::max(1, 4 * per_round / tail)}); ++k) {
        if (k > 1 && (int64_t)tail * H_kv * k * 2 * GROUP_PART_BYTES > part_max) break;
        const double us = (double)((tail * k + per_round - 1) / per_round) * (PRE_FIXED + (kinds == 2 ? PRE_TILE_PACKED : PRE_TILE) * ((tiles + k - 1) / k)) +
                          (k > 1 ? MERGE_FIXED + (double)tail * H_kv * k * 262144.0 / PART_BYTES_US : 0.0);
        if (k == 1 || us < best_us) { best_us = us; best = k; }
    }
    return {best > 1 ? tail : 0, best};
}

// Work items of the gradient of a bf16 batch.  An item of the row-major walk is 8 units (32-row block x head): a workgroup of
// the Delta kernel, two of dq's, each of which fills a compute unit.  It gets as many splits of the tiles as fill whole rounds of
// 256 items.  The key-major kernel takes 4 key tiles a workgroup and splits their units: a workgroup costs KEY_FIXED us (keys
// turned and cut into pieces at the start, an atomic per gradient element at the end) and KEY_UNIT a unit, and a launch ends
// between the even share of a compute unit (workgroups of unlike lengths fill each other's gaps) and the whole rounds of the longest
// ones: the mean of the two.  Fitted to the step's time over 22 batches of 1 to 8 calls (1 to 32 row blocks, 7 to 104 tiles) with
// 4 to 128 units a workgroup: where the choice was among the measured ones it is 0.3 % behind the best in the mean, 3 % at most.
// The rule before (even share and half a longest workgroup, 8 units at least) was 2 and 9 % behind.  Steps of 41 batches, 20 of them
// not in the fit: 1.02 times as fast in the mean, 0.985 (launch-bound ones whose plan did not change) to 1.09 (one call of 320 rows
// over 100 tiles 357 -> 329 us, 1000 rows 802 -> 776, 43 and 31 rows over 8 and 16 tiles 131 -> 120).  Splits of the row-major
// walk: within 3 % of the best of 1, 2, 3, 4, 5, 6, 8 and 12 in 16 batches.
// Per-unit buffers take 64 KB a unit (16 more per further split, of which there are several only in batches of few units).  A
// batch with more units than BWD_UNITS (256 MB) is cut into even runs of row blocks with launches of their own, inside a call
// only where whole workgroups of 8 units end.  2048 rows x 64 heads over 4000 tokens, 4096 x 128 over themselves, six calls of
// 700 x 64 over 2000: 4.50, 7.66, 4.79 ms in runs of 4096 units, 4.50, 7.74, 4.63 of 8192, 4.71, 8.60, 5.06 of 2048.
constexpr int64_t BWD_UNITS = 4096;
constexpr double KEY_FIXED = 30.0, KEY_UNIT = 3.0, ROWS_FIXED = 15.0, ROWS_TILE = 3.0;
struct BwdPlan { std::vector<PcItem> items; std::vector<PcBwdKeyItem> keys; std::vector<int2> row_blocks; size_t units = 0, splits = 1; };

static void plan_backward(const pc_cache *c, Planned &P, std::vector<PcCallDesc> &cds, BwdPlan &bp, int64_t max_units)
{
    const int g = c->g, H_q = c->cfg.n_q_heads, H_kv = c->cfg.n_kv_heads;
    const int step = 8 / std::gcd(8, g);                 // row blocks of whole workgroups
    bp = BwdPlan{};
    P.chunks.clear();
    int64_t groups = 0, blocks = 0;
    int most_units = 1;
    for (const Resolved &r : P.res) {
        blocks += (r.n_q + 31) / 32;
        groups += (int64_t)(((r.n_q + 31) / 32) * g + 7) / 8 * H_kv;
        most_units = std::max(most_units, (r.n_q + 31) / 32 * g);
    }
    const int64_t most_blocks = std::max<int64_t>(step, max_units / H_q / step * step), runs = (blocks + most_blocks - 1) / most_blocks;
    const int rb_max = (int)std::max<int64_t>(step, (int64_t)align_up((size_t)((blocks + runs - 1) / runs), (size_t)step));
    // tiles of the call in front of its own, and the first row block that sees one of four tiles from t on
    auto parents_of = [](const Resolved &r) { return r.tiles - (r.self_msg >= 0 ? (r.self_len + PC_TILE - 1) / PC_TILE : 0); };
    auto first_block = [&](const Resolved &r, int t) { return t >= parents_of(r) ? std::max(0, ((t - parents_of(r)) * PC_TILE - (r.self_len - r.n_q)) / 32) : 0; };
    int key_units = most_units;                          // units a key-major workgroup takes
    double best_us = 0;
    for (int k = 1; k <= 16 && (k == 1 || most_units / k >= 4); ++k) {
        const int u = (most_units + k - 1) / k;
        int64_t workgroups = 0, total = 0;               // (units of all of them together)
        int longest = 0;
        for (const Resolved &r : P.res) {
            const int n_rb = (r.n_q + 31) / 32;
            auto add = [&](int64_t fours, int n) {       // so many groups of four tiles that n units see
                const int sp = (n + u - 1) / u;
                workgroups += fours * sp * H_kv; total += fours * n * H_kv;
                longest = std::max(longest, (n + sp - 1) / sp);
            };
            int t = (parents_of(r) + 3) / 4 * 4;
            if (t > 0 && n_rb > 0) add(t / 4, n_rb * g);
            for (; t < r.tiles && first_block(r, t) < n_rb; t += 4) add(1, (n_rb - first_block(r, t)) * g);
        }
        const double even = (KEY_FIXED * workgroups + KEY_UNIT * total) / 256, rounds = (double)runs * ((workgroups + 256 * runs - 1) / (256 * runs));
        const double us = 0.5 * even + 0.5 * rounds * (KEY_FIXED + KEY_UNIT * longest);
        if (k == 1 || us < best_us) { best_us = us; key_units = u; }
    }
    // splits of the row-major walk: the fewest rounds of 256 workgroups, each a start (ROWS_FIXED) and its tiles long
    int row_splits = 1, most_tiles = 0;
    for (const Resolved &r : P.res) most_tiles = std::max(most_tiles, r.tiles);
    groups = (groups + runs - 1) / runs;                 // (of a run)
    for (int k = 1; k <= std::min(MAX_SPLITS, most_tiles / 8); ++k) {
        if (k > 1 && std::min<int64_t>(rb_max, blocks) * H_q * (3 + k) > 4 * max_units) break;      // (64 KB a unit for k = 1, 16 a split)
        const double us = (double)((groups * k + 255) / 256) * (ROWS_FIXED + ROWS_TILE * ((most_tiles + k - 1) / k));
        if (k == 1 || us < best_us) { best_us = us; row_splits = k; }
        if (groups * k > 1024) break;
    }
    Planned::BwdChunk ch{0, 0, 0, 0, 0, 0};
    auto close = [&]() {
        if (ch.n_rb == 0) return;
        ch.n_items = (int)bp.items.size() - ch.item0; ch.n_keys = (int)bp.keys.size() - ch.key0;
        bp.units = std::max(bp.units, (size_t)ch.n_rb * (size_t)H_q);
        P.chunks.push_back(ch);
        ch = Planned::BwdChunk{ch.rb0 + ch.n_rb, 0, (int)bp.items.size(), 0, (int)bp.keys.size(), 0};
    };
    for (size_t i = 0; i < P.res.size(); ++i) {
        const Resolved &r = P.res[i];
        PcCallDesc &cd = cds[i];
        const int n_rb = (r.n_q + 31) / 32, T = r.tiles, parent_tiles = parents_of(r), self_tiles = T - parent_tiles;
        const int ns = std::max(1, std::min(row_splits, T / 8));
        cd.n_splits = ns;
        cd.rb_off = (int32_t)bp.row_blocks.size();
        bp.splits = std::max(bp.splits, (size_t)ns);
        for (int b = 0; b < n_rb; ++b) bp.row_blocks.push_back(make_int2((int)i, b));
        for (int b0 = 0; b0 < n_rb;) {
            if (ch.n_rb > 0 && ch.n_rb + std::min(n_rb - b0, step) > rb_max) close();
            int nb = n_rb - b0;
            if (nb > rb_max - ch.n_rb) nb = (rb_max - ch.n_rb) / step * step;             // (at least a step: see close above; rb_max is a multiple of it)
            if (nb == 0) { close(); continue; }
            const int b1 = b0 + nb;
            // rows by tiles: a split's share is cut at the causal limit of the workgroup's last row
            for (int u0 = b0 * g; u0 < b1 * g; u0 += 8) {
                int Tg = T;
                if (r.self_msg >= 0) {
                    const int last_unit = std::min(u0 + 7, b1 * g - 1);
                    const int lim = (r.self_len - r.n_q) + std::min(32 * (last_unit / g) + 31, r.n_q - 1);
                    Tg = parent_tiles + std::min(self_tiles, lim / PC_TILE + 1);
                }
                const int chunk = std::max(1, (Tg + ns - 1) / ns);
                for (int s = 0; s < ns; ++s) {
                    PcItem it{}; it.call = (int32_t)i; it.unit0 = u0; it.split = s; it.tile_tab0 = cd.tile_off;
                    it.tile_begin = std::min(Tg, s * chunk); it.tile_end = s == ns - 1 ? Tg : std::min(Tg, (s + 1) * chunk);
                    bp.items.push_back(it);
                }
            }
            // tiles by units: own tiles are seen from the block of their first key on
            for (int t = 0; t < T; t += 4) {
                const int first = std::max(b0, first_block(r, t));
                if (first >= b1) continue;
                const int n_rt = (b1 - first) * g;
                const int sp = (n_rt + key_units - 1) / key_units, per = (n_rt + sp - 1) / sp;
                for (int a = 0; a < n_rt; a += per)
                    bp.keys.push_back(PcBwdKeyItem{(int32_t)i, t, std::min(4, T - t), first * g + a, first * g + std::min(n_rt, a + per), {0, 0, 0}});
            }
            ch.n_rb += nb;
            b0 = b1;
        }
    }
    close();
}

// Work items of an fp32 batch.  A workgroup takes 32 (row, head) columns of a KV head and all of its tiles (eight waves, an
// eighth each) unless the batch has fewer such blocks than half the compute units: then the tiles are split over as many
// workgroups as fill the chip once, 16 tiles (two a wave) at least, and a second launch adds the parts.  A wave's tile is
// 6 us at D = 128 beside the other wave of its SIMD, the merge launch 5, and every split writes its part to memory.
static void plan_f32(const pc_cache *c, const Planned &P, std::vector<PcCallDesc> &cds, bool may_split, std::vector<PcItem> &items, int64_t &part_rows)
{
    const int g = c->g, H_kv = c->cfg.n_kv_heads;
    auto blocks_of = [&](const Resolved &r) { return ((int64_t)r.n_q * g + 31) / 32; };
    int64_t groups = 0;
    for (const Resolved &r : P.res) groups += blocks_of(r) * H_kv;
    items.clear();
    part_rows = 0;
    for (size_t i = 0; i < P.res.size(); ++i) {
        const Resolved &r = P.res[i];
        PcCallDesc &cd = cds[i];
        const int T = r.tiles, self_tiles = r.self_msg >= 0 ? (r.self_len + PC_TILE - 1) / PC_TILE : 0;
        const int ns = may_split ? (int)std::max<int64_t>(1, std::min<int64_t>({256 / std::max<int64_t>(groups, 1), (int64_t)T / 16, (int64_t)MAX_SPLITS})) : 1;
        cd.n_splits = ns; cd.part_off = 0;
        if (ns > 1) { cd.part_off = (int32_t)part_rows; part_rows += (int64_t)ns * cd.n_q; }
        for (int64_t b = 0; b < blocks_of(r); ++b) {
            int Tg = T;
            if (r.self_msg >= 0) {                       // cut at the causal limit of the block's last row
                const int last_row = (int)(std::min<int64_t>(32 * b + 31, (int64_t)r.n_q * g - 1) / g);
                Tg = T - self_tiles + std::min(self_tiles, (r.self_len - r.n_q + last_row) / PC_TILE + 1);
            }
            const int chunk = std::max(1, (Tg + ns - 1) / ns);
            for (int s = 0; s < ns; ++s) {
                PcItem it{}; it.call = (int32_t)i; it.unit0 = (int32_t)b; it.split = s; it.tile_tab0 = cd.tile_off;
                it.tile_begin = std::min(Tg, s * chunk); it.tile_end = std::min(Tg, (s + 1) * chunk);
                items.push_back(it);
            }
        }
    }
}

// Key-major work items of the gradient of an fp32 batch: 4 key tiles a workgroup (one a wave), which fills a compute unit,
// and the column blocks that see them split until the chip is full twice over, two blocks a split at least (a split ends in
// one atomic per element of its tiles' dK and dV, about what one more block costs), or into as many splits as fill the chip once, where that is
// more (two calls of 11 and 14 blocks, 24 groups of four tiles: 10 splits, of which 6 and 7 have blocks to take, two each).
static void plan_backward_keys_f32(const pc_cache *c, const Planned &P, std::vector<PcBwdKeyItem> &keys)
{
    const int g = c->g;
    int64_t quads = 0;
    for (const Resolved &r : P.res) quads += (int64_t)((r.tiles + 3) / 4) * c->cfg.n_kv_heads;
    for (size_t i = 0; i < P.res.size(); ++i) {
        const Resolved &r = P.res[i];
        const int T = r.tiles, self_tiles = r.self_msg >= 0 ? (r.self_len + PC_TILE - 1) / PC_TILE : 0, parent_tiles = T - self_tiles;
        const int blocks = (int)(((int64_t)r.n_q * g + 31) / 32);
        for (int t = 0; t < T; t += 4) {
            int first = 0;                               // own tiles are seen from the block of their first key's row on
            if (t >= parent_tiles) first = (int)((int64_t)std::max(0, (t - parent_tiles) * PC_TILE - (r.self_len - r.n_q)) * g / 32);
            if (first >= blocks) continue;
            const int n = blocks - first;
            const int sp = (int)std::max<int64_t>({1, std::min<int64_t>((512 + quads - 1) / quads, n / 2), std::min<int64_t>(256 / quads, n)});
            const int per = (n + sp - 1) / sp;
            for (int a = 0; a < n; a += per)
                keys.push_back(PcBwdKeyItem{(int32_t)i, t, std::min(4, T - t), first + a, first + std::min(n, a + per), {0, 0, 0}});
        }
    }
}

// A batch of nothing but decode calls that walk their own lists goes to one launch (pc_decode_one_bf16_kernel) when no split takes
// its tiles from more messages than a wave has lanes (it looks them up one a lane, once) and every token of a decode step is the
// last one of exactly one call's new message.  Not where the splits are tuned by hand, nor where lists or tables might not fit what pc_attend_static has, so that
// it refuses what it refused.  rc != PC_OK: an error; else false: the plan builder's way.  Fills P.one_*.
// (us a step of 64 calls over 9 messages each: 136 the plan builder's way, 131; of 5 over 220: 141 and 93.  Batches that share
// enough stay with the shared walk: 14 calls over 27 messages each of 40: 38 us there, 47 in one launch of their own walks.)
static bool plan_one(pc_cache *c, Planned &P, hipStream_t st, int32_t &rc)
{
    const int n_calls = (int)P.res.size(), g = c->g, H_kv = c->cfg.n_kv_heads, H_q = c->cfg.n_q_heads;
    if (c->decode_tiles_per_split != 0 || n_calls > 4095 || c->cfg.max_position >= 1 << 28 || c->cfg.rope_theta < 1.f) return false;
    size_t n_seg = 0, n_q = 0, n_tiles = 0;
    for (const Resolved &r : P.res) {
        if (r.n_q * g > 16 || r.tiles >= 1 << 24 || r.sel.size() > 4094) return false;
        n_tiles += (size_t)r.tiles;
        n_seg += r.sel.size() + (r.self_msg >= 0 ? 1 : 0);
        n_q += (size_t)r.n_q;
    }
    {   // at most what the plan builder's way stages and keeps under the plain rule
        const size_t wgs = (size_t)(n_calls * H_kv) + 256, staged = 64 * (size_t)n_calls + 8 * n_seg + 20 * n_q + 32 * ((size_t)n_calls + 256) + 16 * P.tok_items.size();
        const size_t tables = n_seg * 548 + n_q * (1536 + 4 * (size_t)H_q) + n_tiles * sizeof(PcTile) + wgs * 16 * 264;
        if (staged > HOST_READ_BYTES || staged + tables > PC_STATIC_WS_BYTES - (1 << 20)) return false;
    }
    size_t n_items = 0;
    std::vector<int> splits((size_t)n_calls);
    for (int i = 0; i < n_calls; ++i) {
        n_items += (size_t)(splits[(size_t)i] = one_splits(n_calls * H_kv, P.res[(size_t)i].tiles));
        // (some split has more: known here before any list is sorted)
        if (P.res[(size_t)i].sel.size() + (P.res[(size_t)i].self_msg >= 0 ? 1 : 0) > (size_t)splits[(size_t)i] * PC_ONE_SEGS) return false;
    }
    const size_t off_sel = sizeof(PcOneCall) * (size_t)n_calls, off_items = off_sel + sizeof(int2) * n_seg;
    const size_t off_q_pos = off_items + sizeof(PcOneItem) * n_items, bytes = off_q_pos + sizeof(int32_t) * n_q;
    std::vector<int32_t> tok((size_t)n_calls, -1);
    if (!P.tok_items.empty()) {
        const uint32_t epoch = new_marks(c);             // value: the call that has it as its new message and no token for it yet, -1: several
        for (int i = 0; i < n_calls; ++i)
            if (P.res[(size_t)i].self_msg >= 0) {
                pc_cache::Mark &mk = c->marks[(size_t)P.res[(size_t)i].self_msg];
                mk = pc_cache::Mark{epoch, mk.epoch == epoch ? -1 : i};
            }
        for (size_t k = 0; k < P.tok_items.size(); ++k) {
            const PcTokenItem &t = P.tok_items[k];
            pc_cache::Mark &mk = c->marks[(size_t)t.msg];
            if (mk.epoch != epoch || mk.value < 0 || t.new_len != c->msgs[(size_t)t.msg].len) return false;
            tok[(size_t)mk.value] = (int32_t)k;
            mk.value = -1;
        }
    }
    // which messages a split takes its tiles from (before a slot of the ring is taken: the plan builder's way takes one itself)
    std::vector<PcOneItem> items;
    items.reserve(n_items);
    for (int i = 0; i < n_calls; ++i) {
        Resolved &r = P.res[(size_t)i];
        sort_by_slot(c, r);                              // (as in pc_plan_and_stage)
        const int T = r.tiles, ns = splits[(size_t)i], n_sel = (int)r.sel.size(), n = n_sel + (r.self_msg >= 0 ? 1 : 0);
        const int chunk = std::max(1, (T + ns - 1) / ns);
        auto tiles_of = [&](int e) { return ((e < n_sel ? c->msgs[(size_t)r.sel[(size_t)e].x].len : r.self_len) + PC_TILE - 1) / PC_TILE; };
        int e = 0, before = 0;                           // an entry, and the tiles before it
        for (int s = 0; s < ns; ++s) {
            while (e + 1 < n && before + tiles_of(e) <= s * chunk) before += tiles_of(e++);
            int last = e;
            for (int end = before + (n > 0 ? tiles_of(e) : 0); last + 1 < n && end < std::min(T, (s + 1) * chunk); end += tiles_of(++last)) {}
            const int count = n > 0 ? last - e + 1 : 0;
            if (count > PC_ONE_SEGS) return false;
            PcOneItem it{};
            it.call = (uint32_t)i; it.split = (uint32_t)s; it.seg0 = (uint32_t)e; it.tile0 = (uint32_t)before; it.n_seg = (uint32_t)count;
            items.push_back(it);
        }
    }
    char *h = (char *)P.one_blob.w;
    if (bytes > PC_ARG_BYTES && pc_recorded(st)) {
        P.recorded.resize(align_up(bytes, 16));
        h = P.recorded.data();
    } else if (bytes > PC_ARG_BYTES) {                   // (a slot of the ring holds four times HOST_READ_BYTES: nothing is allocated)
        rc = pc_stage_acquire(c, bytes, &P.one_slot);
        if (rc != PC_OK) return false;
        h = (char *)P.one_slot->host;
    }
    PcOneCall *calls = (PcOneCall *)h;
    int2 *sel = (int2 *)(h + off_sel);
    int32_t *q_pos = (int32_t *)(h + off_q_pos);
    std::memcpy(h + off_items, items.data(), sizeof(PcOneItem) * items.size());
    int64_t part_rows = 0;
    int seg_off = 0, q_off = 0;
    for (int i = 0; i < n_calls; ++i) {
        const Resolved &r = P.res[(size_t)i];
        const int T = r.tiles, ns = splits[(size_t)i], n_sel = (int)r.sel.size(), n = n_sel + (r.self_msg >= 0 ? 1 : 0);
        PcOneCall &oc = calls[i];
        oc.seg_off = (uint16_t)seg_off; oc.n_seg = (uint16_t)n; oc.n_q = (uint16_t)r.n_q; oc.n_splits = (uint16_t)ns;
        oc.q_off = q_off; oc.self_len = r.self_msg >= 0 ? r.self_len : 0; oc.n_tiles = T; oc.chunk = std::max(1, (T + ns - 1) / ns);
        oc.part_off = (int32_t)part_rows; oc.tok = tok[(size_t)i];
        if (ns > 1) part_rows += (int64_t)ns * r.n_q;
        std::copy(r.sel.begin(), r.sel.end(), sel + seg_off);
        if (r.self_msg >= 0) sel[seg_off + n_sel] = make_int2(r.self_msg, r.self_start);
        std::copy(r.q_pos.begin(), r.q_pos.end(), q_pos + q_off);
        seg_off += n; q_off += r.n_q;
    }
    P.lay = PlanLayout{};
    P.lay.part_ml = align_up(sizeof(float) * (size_t)part_rows * H_q * c->D, 256);       // (part_o comes first)
    P.lay.calls = align_up(P.lay.part_ml + sizeof(float) * 2 * (size_t)part_rows * H_q, 256);       // (a recorded call's lists)
    P.lay.total = P.lay.calls + P.recorded.size();
    P.total_seg = seg_off;
    P.one_bytes = bytes;
    P.one.lists = P.one_slot ? P.one_slot->host : nullptr;
    P.one.off_sel = (int32_t)off_sel; P.one.off_q_pos = (int32_t)off_q_pos; P.one.off_items = (int32_t)off_items; P.one.n_items = (int32_t)n_items;
    P.one.table = c->table_dev; P.one.inv_freq = c->inv_freq_dev;
    // (like the workspaces: a replay of a captured pc_attend_static may run beside a pc_attend)
    P.one.counters = c->counters_dev + (P.fixed_ws ? PC_ONE_COUNTERS : 0);
    P.one.tok_k = (const uint16_t *)P.tok_k; P.one.tok_v = (const uint16_t *)P.tok_v;
    return true;
}

// the tokens of a decode step, whose items lie at `items`, for a launch that appends them
static PcTokenWork token_work(const pc_cache *c, const Planned &P, const PcTokenItem *items)
{
    PcTokenWork tok;
    if (P.tok_items.empty()) return tok;
    tok.items = items; tok.n = (int)P.tok_items.size();
    tok.k = P.tok_k; tok.v = P.tok_v; tok.k_store = c->k_store; tok.v_store = c->v_store;
    tok.slots = c->slots; tok.n_kv_heads = c->cfg.n_kv_heads; tok.D = c->D; tok.dtype = c->cfg.dtype;
    return tok;
}

// every call's entries fit a wave, and their angles the short series (see rope_small)
static bool self_plans(const pc_cache *c, const std::vector<PcCallDesc> &cds)
{
    if (c->cfg.max_position >= 1 << 28 || c->cfg.rope_theta < 1.f) return false;
    for (const PcCallDesc &cd : cds) if (cd.n_seg > PC_SELF_SEGS) return false;
    return true;
}

int32_t pc_plan_and_stage(pc_cache *c, const pc_call *calls, int32_t n_calls, bool want_items,
                              hipStream_t st, Planned &P)
{
    P.n_calls = n_calls;
    P.res.resize((size_t)n_calls);
    for (int i = 0; i < n_calls; ++i) {
        const int32_t rc = pc_resolve(c, &calls[i], i, P.res[i]);
        if (rc != PC_OK) return rc;
        P.total_q += P.res[i].n_q;
    }
    const int g = c->g, H_kv = c->cfg.n_kv_heads;
    const bool bf16 = c->cfg.dtype == PC_BF16;
    // work-group shape of the prefill kernel: 8 row units (32 rows x 1 q head each) per group
    P.pre_waves = 8;
    std::vector<PcCallDesc> cds((size_t)n_calls);
    std::vector<PcItem> dec, pre, pre_pk;
    std::vector<PcGatherItem> kg;
    int64_t kg_tiles = 0;
    int64_t part_rows = 0, total_tiles = 0;
    int q_off = 0, seg_off = 0;
    // groups of one-row calls that share enough of their messages take the shared walk, or the whole batch goes by message
    int32_t rc = PC_OK;
    static thread_local SharedPlan sp;
    struct Kept { ~Kept() { keep(sp.segs); keep(sp.pos); } } kept;
    sp.in_shared.assign((size_t)n_calls, 0);
    sp.groups.clear(); sp.wide.clear(); sp.segs.clear(); sp.items.clear(); sp.pos.clear();
    if (want_items && bf16) {
        std::vector<int> q_offs((size_t)n_calls);
        for (int i = 0, o = 0; i < n_calls; ++i) { q_offs[(size_t)i] = o; o += P.res[(size_t)i].n_q; }
        if (plan_shared(c, P, q_offs, g, sp, st, rc)) {
            if (!P.fixed_ws) {
                rc = pc_ensure_ws(c, P.lay.total, st);
                if (rc != PC_OK) return rc;
            }                                            // (it fits every fixed workspace, see plan_runs)
            P.ws = P.fixed_ws ? P.fixed_ws : c->ws;
            P.runs.runs = (const PcMsgRun *)((char *)P.ws + P.lay.calls);
            P.runs.rot = (const float2 *)((char *)P.ws + P.lay.rot_seg);
            ProfScope ps(c, 1, st);
            const bool recorded = !P.runs_slot;
            if (recorded) pc_launch_store_args(P.recorded.data(), P.recorded.size(), P.ws, st);
            char *from = recorded ? (char *)P.ws : (char *)P.runs_slot->host, *lists = (char *)P.ws + P.lay.calls;
            const size_t off_rest = sizeof(PcMsgRun) * (size_t)P.n_runs, saved = recorded ? (sizeof(PcMsgRun) - sizeof(PcMsgRunShort)) * (size_t)P.n_runs : 0;
            const PcTokenWork tok = token_work(c, P, (const PcTokenItem *)(from + P.lay.tok_items - saved));
            pc_launch_runs_prepare(from, lists, P.runs_bytes - off_rest, P.n_runs, recorded, c->scale * 1.4426950408889634f, tok, c->inv_freq_dev, c->table_dev,
                                   (float2 *)((char *)P.ws + P.lay.rot_seg), st);
            PC_HIP(c, hipGetLastError());
            P.tok_done = !P.tok_items.empty();
            return PC_OK;
        }
        if (rc != PC_OK) return rc;
    }
    if (want_items && bf16 && !c->host_only && sp.groups.empty() && plan_one(c, P, st, rc)) {
        if (!P.fixed_ws) {
            rc = pc_ensure_ws(c, P.lay.total, st);
            if (rc != PC_OK) return rc;
        } else if (P.lay.total > P.fixed_cap)
            return pc_fail(c, PC_ERR_NO_SPACE, "attend: this batch needs %zu bytes of workspace, the fixed one holds %zu", P.lay.total, P.fixed_cap);
        P.ws = P.fixed_ws ? P.fixed_ws : c->ws;
        if (!P.recorded.empty()) {
            pc_launch_store_args(P.recorded.data(), P.recorded.size(), (char *)P.ws + P.lay.calls, st);
            PC_HIP(c, hipGetLastError());
            P.one.lists = (char *)P.ws + P.lay.calls;
        }
        return PC_OK;
    }
    if (rc != PC_OK) return rc;
    // first pass: how many prefill groups without splitting (to decide on KV splits)
    int64_t pre_groups = 0, dec_groups = 0;
    if (want_items && bf16)
        for (int i = 0; i < n_calls; ++i) {
            const Resolved &r = P.res[(size_t)i];
            if (sp.in_shared[(size_t)i]) continue;
            if (r.n_q * g > 16) pre_groups += (int64_t)((((r.n_q + 31) / 32) * g + P.pre_waves - 1) / P.pre_waves) * H_kv;
            else dec_groups += H_kv;
        }
    auto pre_groups_of = [&](const Resolved &r) { return (((r.n_q + 31) / 32) * g + P.pre_waves - 1) / P.pre_waves; };
    // the plain rule: as many splits as bring the batch to 256 workgroups, of 16 of the tiles that are walked at least
    auto plain_splits = [](int64_t groups, int tiles) { return (int)std::min<int64_t>((256 + groups - 1) / groups, std::max(1, tiles / 16)); };
    int pre_chunk = 1;                                   // tiles a prefill split takes
    std::pair<int, int> tail{0, 1};                      // last prefill items that are split, and into how many parts
    int64_t pre_part_rows = 0;                           // partial rows of prefill items among part_rows
    std::vector<PcMergeRow> tail_rows;
    // splits of a call over the tiles it walks, none of them empty.  small: the rules as they stand; else the plain rule
    auto whole_splits = [](int tiles, int ns) {
        ns = std::max(1, std::min(MAX_SPLITS, ns));
        const int chunk = std::max(1, (tiles + ns - 1) / ns);
        return std::max(1, (tiles + chunk - 1) / chunk);
    };
    // Decode: as few splits as fill the chip (256 workgroups): the kernel is bound by memory, and every split beyond
    // that only adds partial results to write and merge.  A split has 4 tiles at least, one a wave: a small
    // call is a chain of latencies, which shorter runs of tiles shorten by more than the merge launch costs from
    // 16 tiles on (4 calls over 1300 tokens, 8 KV heads: 18 + 5 us at 16 tiles a split, 10 + 5 at 4).
    auto decode_splits = [&](int T, bool small) {
        const int least = small ? (T >= 16 ? 4 : T + 1) : 16;
        return whole_splits(T, c->decode_tiles_per_split > 0 ? (T + c->decode_tiles_per_split - 1) / c->decode_tiles_per_split
                                                             : (int)std::min<int64_t>((256 + dec_groups - 1) / dec_groups, std::max(1, T / least)));
    };
    auto prefill_splits = [&](int Tc, bool small) {
        return whole_splits(Tc, c->prefill_tiles_per_split > 0 ? (Tc + c->prefill_tiles_per_split - 1) / c->prefill_tiles_per_split
                                : small ? (int)(((int64_t)Tc + pre_chunk - 1) / pre_chunk) : plain_splits(pre_groups, Tc));
    };
    // small_splits: the rules for the number of splits as they stand.  Without it: the plain rule (see below).
    auto plan_calls = [&](bool small_splits) {
        dec.clear(); pre.clear(); pre_pk.clear(); kg.clear(); sp.items.clear(); tail_rows.clear();
        int64_t items_left = pre_groups / H_kv;          // prefill items still to come
        kg_tiles = part_rows = pre_part_rows = total_tiles = 0;
        q_off = seg_off = 0;
        for (int i = 0; i < n_calls; ++i) {
            Resolved &r = P.res[i];
            PcCallDesc &cd = cds[i];
            // a call served by the shared walk needs no segments, tiles or rotation rows of its own: the plan
            // builder sees it as a call that lists nothing
            const bool own_plan = !sp.in_shared[(size_t)i];
            cd.sel_off = seg_off; cd.n_sel = own_plan ? (int)r.sel.size() : 0;
            cd.self_msg = own_plan ? r.self_msg : -1; cd.self_start = r.self_start;
            cd.n_q = r.n_q; cd.q_off = q_off; cd.seg_off = seg_off; cd.n_seg = cd.n_sel + (cd.self_msg >= 0 ? 1 : 0);
            cd.self_len = own_plan ? r.self_len : 0; cd.n_splits = 1; cd.part_off = 0; cd.tile_off = (int32_t)total_tiles;
            cd.kg_tile0 = -1; cd.n_par = 0; cd.rb_off = 0; cd.part_wide = 0;
            if (own_plan) total_tiles += r.tiles;
            q_off += cd.n_q; seg_off += cd.n_seg;
            if (!want_items || !bf16 || !own_plan) continue;
            const int T = r.tiles;
            int wide = 0;
            if (r.n_q * g <= 16) {                       // decode-shaped: all rows x heads of a KV head in one wave
                // Attention does not depend on the order the keys are visited in (each keeps its own
                // position), so a decode call walks its parents in ascending cache-slot order: calls that
                // share messages then touch them at about the same time and the later ones hit in L2.
                sort_by_slot(c, r);
                const int ns = decode_splits(T, small_splits), chunk = std::max(1, (T + ns - 1) / ns);
                cd.n_splits = ns;
                wide = ns > 1 && small_splits && c->decode_tiles_per_split == 0 && plain_splits(dec_groups, T) == 1;
                for (int s = 0; s < ns; ++s) {
                    PcItem it{}; it.call = i; it.unit0 = 0; it.tile_begin = s * chunk; it.tile_end = std::min(T, (s + 1) * chunk); it.split = s;
                    it.tile_tab0 = cd.tile_off;
                    dec.push_back(it);
                }
            } else {
                const int own_tiles = own_tiles_of(r);
                const int64_t n_par = parent_tokens(c, r);
                const int p_tiles = (int)((n_par + PC_TILE - 1) / PC_TILE);
                const bool packed = gathers(c, P, r) && kg_tiles + p_tiles + own_tiles < ((int64_t)1 << 24);
                if (packed) {
                    cd.kg_tile0 = (int32_t)kg_tiles; cd.n_par = (int32_t)n_par;
                    kg.push_back(PcGatherItem{i, (int32_t)kg_tiles, p_tiles + own_tiles, (int32_t)n_par});
                    kg_tiles += p_tiles + own_tiles;
                }
                const int Tc = packed ? p_tiles + own_tiles : T;        // tiles the attention kernel walks for this call
                const int units = ((r.n_q + 31) / 32) * g;
                const int groups = pre_groups_of(r);
                const int ns = prefill_splits(Tc, small_splits);
                cd.n_splits = ns;
                // A group of row units walks the parents' tiles and the tiles of the new message up to the
                // causal limit of its last row (the kernel relies on tile_end being cut there); its splits
                // divide THAT count evenly, so the groups with early rows do not end up with a nearly empty
                // last split.
                const int parent_tiles = Tc - own_tiles;
                wide = ns > 1 && small_splits && c->prefill_tiles_per_split == 0 && plain_splits(pre_groups, Tc) == 1;
                for (int gidx = 0; gidx < groups; ++gidx, --items_left) {
                    int Tg = Tc;
                    if (r.self_msg >= 0) {
                        const int last_unit = std::min(gidx * P.pre_waves + P.pre_waves - 1, units - 1);
                        const int lim = (r.self_len - r.n_q) + std::min(32 * (last_unit / g) + 31, r.n_q - 1);   // last own token seen
                        Tg = parent_tiles + std::min(own_tiles, lim / PC_TILE + 1);
                    }
                    // partial rows: those of the whole call, or of an item of the last round alone
                    int parts = ns, row0 = 0, n_rows = r.n_q;
                    int64_t part0 = part_rows;
                    if (small_splits && items_left <= tail.first) {
                        parts = tail.second;
                        wide = 1;
                        row0 = 32 * (gidx * P.pre_waves / g);
                        n_rows = std::min(r.n_q - row0, 32 * P.pre_waves / g);
                        for (int q = 0; q < n_rows; ++q)
                            tail_rows.push_back(PcMergeRow{cd.q_off + row0 + q, (int32_t)(part_rows + 2 * q), parts | PC_MERGE_WIDE, n_rows});
                        part_rows += 2 * (int64_t)parts * n_rows;
                        pre_part_rows += 2 * (int64_t)parts * n_rows;
                    }
                    const int chunk_g = std::max(1, (Tg + parts - 1) / parts);
                    for (int s = 0; s < parts; ++s) {
                        PcItem it{}; it.call = i; it.unit0 = gidx * P.pre_waves; it.split = s; it.tile_tab0 = cd.tile_off;
                        it.tile_begin = std::min(Tg, s * chunk_g);
                        it.tile_end = s == parts - 1 ? Tg : std::min(Tg, (s + 1) * chunk_g);
                        it.n_splits = parts;
                        it.part_base = (int32_t)(part0 + (((int64_t)s * n_rows - row0) << wide));
                        (packed ? pre_pk : pre).push_back(it);
                    }
                }
            }
            // Partial results are fp32 where the plain rule would not have split the rows at all, so that no sum is held in fewer
            // bits for being split; the others, fp16, are bound by the bytes they move (512 rows x 32 heads in 4 splits: 17 MB,
            // 8 us).
            cd.part_wide = wide;
            if (cd.n_splits > 1) {
                const int64_t n = ((int64_t)cd.n_splits * cd.n_q) << cd.part_wide;
                cd.part_off = (int32_t)part_rows;
                part_rows += n;
                if (r.n_q * g > 16) pre_part_rows += n;
            }
        }
        // shared groups: as many splits of the union as fill the chip together
        for (size_t gi = 0; gi < sp.groups.size(); ++gi) {
            PcShGroup &gr = sp.groups[gi];
            const int T = gr.n_tiles;
            const int ns = shared_splits(c, sp.groups.size(), T), chunk = std::max(1, (T + ns - 1) / ns);
            gr.n_splits = ns;
            if (ns > 1) { gr.part_off = (int32_t)part_rows; part_rows += ((int64_t)ns * gr.n_rows) << sp.wide[gi]; }
            int seg = 0;                                     // the message that owns a split's first tile (splits ascend)
            for (int sidx = 0; sidx < ns; ++sidx) {
                const int t0 = sidx * chunk;
                while (seg + 1 < gr.n_seg && sp.segs[(size_t)gr.seg_off + (size_t)seg + 1].tile_off <= t0) ++seg;
                sp.items.push_back(PcShItem{(int32_t)gi, t0, std::min(T, (sidx + 1) * chunk), sidx, seg, sp.wide[gi], {0, 0}});
            }
        }
    };
    // the batch's work items; part_max: bytes the partial results of its prefill calls may take
    auto plan_items = [&](bool small_splits, int64_t part_max) {
        if (want_items && bf16 && c->prefill_tiles_per_split == 0) {
            if (pre_groups > 0) pre_chunk = prefill_chunk(c, P, sp, pre_groups, part_max);
            tail = prefill_tail(c, P, sp, pre_groups, part_max);
        }
        plan_calls(small_splits);
        if (want_items && !bf16) plan_f32(c, P, cds, small_splits, pre, part_rows);
    };
    BwdPlan bp;
    plan_items(true, INT64_MAX);
    if (P.backward && bf16) plan_backward(c, P, cds, bp, BWD_UNITS);
    if (P.backward && !bf16) {
        plan_f32(c, P, cds, false, pre, part_rows);
        plan_backward_keys_f32(c, P, bp.keys);
        P.n_bwd_keys = (int)bp.keys.size();
    }
    if (P.backward && bf16) pre = std::move(bp.items);   // (the gradient's row-major items are staged where the prefill items go)
    if (sp.pos.size() > (size_t)INT32_MAX / 2) return pc_fail(c, PC_ERR_SHAPE, "attend: shared decode table too large");
    auto layout_of = [&](size_t n_dec, size_t n_pre, int64_t n_part, size_t n_merge, size_t n_tok) {
        return make_layout(n_calls, P.total_q, seg_off, (int)n_dec, (int)n_pre, (int)pre_pk.size(), n_part, total_tiles, c->cfg.n_q_heads, c->D,
                           sp.groups.size(), sp.segs.size(), sp.items.size(), sp.pos.size(), kg.size(), kg_tiles, H_kv, n_tok,
                           bp.row_blocks.size(), bp.keys.size(), bp.units, bp.splits, bf16 ? sizeof(uint16_t) : sizeof(float), n_merge);
    };
    auto layout = [&](size_t n_tok) {
        size_t n_merge = 0;
        for (int i = 0; i < n_calls && want_items; ++i) if (cds[(size_t)i].n_splits > 1) n_merge += (size_t)cds[(size_t)i].n_q;
        for (const PcShGroup &gr : sp.groups) if (gr.n_splits > 1) n_merge += (size_t)gr.n_rows;
        return layout_of(dec.size(), pre.size(), part_rows, n_merge + tail_rows.size(), n_tok);
    };
    // pc_attend_static takes a batch that fits its workspace under the plain rule, which bounds the partial results, and
    // returns pc_attend's bits: where the partial results of the splits above would not fit as well, both keep those of the
    // prefill calls to what is left of that workspace, or take the plain rule.  (The same sizes decide in both: a decode
    // step's tokens and a ring slot that has grown are left out.  A call that gathers has other bits in any case.)
    if (want_items && !c->host_only && (P.fixed_ws || kg.empty())) {
        auto fits = [](const PlanLayout &l) { return l.total <= PC_STATIC_WS_BYTES && l.h2d_bytes <= STAGE_BYTES; };
        const PlanLayout small = layout(0);
        const int64_t other = (int64_t)small.total - pre_part_rows * c->cfg.n_q_heads * (c->D * 2 + 8);
        const size_t tables = (small.part_o - small.segs) + (small.total - small.row_scalar);     // the same under every rule
        if (P.fixed_ws || (!fits(small) && tables <= PC_STATIC_WS_BYTES)) {
            // the layout under the plain rule, counted: planning a batch twice more for it took a quarter of the host time of a
            // static call (200 one-row calls over 20 messages: 57 us, 42 counted)
            size_t n_dec = 0, n_pre = 0, n_merge = 0;
            int64_t rows = 0;
            for (int i = 0; i < n_calls; ++i) {
                const Resolved &r = P.res[(size_t)i];
                if (sp.in_shared[(size_t)i]) continue;
                int ns = 1;
                if (!bf16) n_pre += (size_t)(((int64_t)r.n_q * g + 31) / 32);
                else if (r.n_q * g <= 16) n_dec += (size_t)(ns = decode_splits(r.tiles, false));
                else n_pre += (size_t)(ns = prefill_splits(r.tiles, false)) * (size_t)pre_groups_of(r);
                if (ns > 1) { rows += (int64_t)ns * r.n_q; n_merge += (size_t)r.n_q; }
            }
            for (size_t i = 0; i < sp.groups.size(); ++i) {
                const PcShGroup &gr = sp.groups[i];
                if (gr.n_splits > 1) { rows += ((int64_t)gr.n_splits * gr.n_rows) << sp.wide[i]; n_merge += (size_t)gr.n_rows; }
            }
            const PlanLayout plain = layout_of(n_dec, n_pre, rows, n_merge, 0);
            const bool refused = P.fixed_ws && (plain.total > P.fixed_cap || plain.h2d_bytes > c->stage[c->stage_next].cap);
            if (refused) plan_items(false, INT64_MAX);
            else if (!fits(small) && plain.total <= PC_STATIC_WS_BYTES) {
                plan_items(true, (int64_t)PC_STATIC_WS_BYTES - other);
                if (!fits(layout(0))) plan_items(false, INT64_MAX);
            }
        }
    }
    P.lay = layout(P.tok_items.size());
    if (P.backward && bf16 && !c->host_only && P.lay.total > c->ws_cap &&
        (P.lay.total >= c->ws_refused || pc_ensure_ws(c, P.lay.total, st) != PC_OK)) {
        // the device has no room for that (and is not asked again): shorter runs, in the workspace there is
        c->ws_refused = std::min(c->ws_refused, P.lay.total);
        for (int64_t units = BWD_UNITS / 2; units >= 8 && P.lay.total > c->ws_cap; units /= 2) {
            plan_backward(c, P, cds, bp, units);
            pre = std::move(bp.items);
            P.lay = layout(0);
        }
    }
    // An fp32 batch with short lists: the attention launch plans for itself.  (Rows and entries of a workgroup: a region of 20 KB or so each; not a decode
    // step's, whose tokens the plan builder appends.)
    if (want_items && !bf16 && !P.backward && !c->host_only && P.tok_items.empty() && P.lay.h2d_bytes <= PC_ARG_BYTES && self_plans(c, cds)) {
        int most_seg = 1, most_tiles = 1;
        for (const PcCallDesc &cd : cds) most_seg = std::max(most_seg, cd.n_seg);
        for (const PcItem &it : pre) most_tiles = std::max(most_tiles, it.tile_end - it.tile_begin);
        PcSelf S{};
        S.off_rot = (int32_t)align_up(sizeof(PcTile) * (size_t)most_tiles, 256);
        S.off_rot_q = S.off_rot + (int32_t)align_up(sizeof(float2) * (size_t)c->half * (size_t)most_seg, 256);
        S.stride = S.off_rot_q + (int64_t)align_up(sizeof(float2) * (size_t)c->half * (size_t)(32 / g + 2), 256);
        const size_t regions = (size_t)S.stride * pre.size() * (size_t)H_kv;
        if (regions <= (size_t)8 << 20 && P.lay.total + regions <= PC_STATIC_WS_BYTES) {
            S.n16 = (int32_t)((P.lay.h2d_bytes + 15) / 16);
            S.off_calls = (int32_t)P.lay.calls; S.off_items = (int32_t)P.lay.items_pre; S.off_sel = (int32_t)P.lay.sel; S.off_q_pos = (int32_t)P.lay.q_pos;
            S.table = c->table_dev; S.inv_freq = c->inv_freq_dev;
            P.self = S;
            P.self_at = P.lay.total;
            P.lay.total += regions;
        }
    }
    P.total_seg = seg_off;
    P.n_dec = (int)dec.size(); P.n_pre = (int)pre.size(); P.n_pre_pk = (int)pre_pk.size();
    P.n_sh_items = (int)sp.items.size(); P.sh_wide = std::find(sp.wide.begin(), sp.wide.end(), 1) != sp.wide.end(); P.n_sh_pos = sp.pos.size();
    P.n_kg_items = (int)kg.size(); P.kg_tiles = kg_tiles;
    if (part_rows > INT32_MAX) return pc_fail(c, PC_ERR_SHAPE, "attend: partial buffer too large");
    if (total_tiles > INT32_MAX / 2) return pc_fail(c, PC_ERR_SHAPE, "attend: too many KV tiles");
    if (c->host_only) return PC_OK;

    if (P.fixed_ws) {                                    // nothing may be allocated: the plan fits or the call fails
        if (P.lay.total > P.fixed_cap)
            return pc_fail(c, PC_ERR_NO_SPACE, "attend: this batch needs %zu bytes of workspace, the fixed one holds %zu",
                           P.lay.total, P.fixed_cap);
        if (P.lay.h2d_bytes > c->stage[c->stage_next].cap)
            return pc_fail(c, PC_ERR_NO_SPACE, "attend: this batch stages %zu bytes of descriptors, the pinned ring slot holds %zu",
                           P.lay.h2d_bytes, c->stage[c->stage_next].cap);
        P.ws = P.fixed_ws;
    } else {
        rc = pc_ensure_ws(c, P.lay.total, st);
        if (rc != PC_OK) return rc;
        P.ws = c->ws;
    }
    StageSlot *slot = nullptr;
    PcArgBlob &blob = P.one_blob;
    // (Batches with shared groups stay with the ring, where they were measured: they need six calls at least over the same
    // messages, and their lists, 50 bytes a message and 4 more a row of it, seldom fit.)
    const bool in_args = P.lay.h2d_bytes <= PC_ARG_BYTES && P.n_sh_items == 0;
    const bool recorded = !in_args && pc_recorded(st);
    if (recorded) P.recorded.resize(P.lay.h2d_bytes);
    if (!in_args && !recorded) {
        rc = pc_stage_acquire(c, P.lay.h2d_bytes, &slot);
        if (rc != PC_OK) return rc;
    }
    char *h = in_args ? (char *)blob.w : recorded ? P.recorded.data() : (char *)slot->host;
    std::memcpy(h + P.lay.calls, cds.data(), sizeof(PcCallDesc) * cds.size());
    int2 *hs = (int2 *)(h + P.lay.sel);
    int32_t *hq = (int32_t *)(h + P.lay.q_pos);
    PcMergeRow *hm = (PcMergeRow *)(h + P.lay.merge_rows);
    for (int i = 0; i < n_calls; ++i) {
        const Resolved &r = P.res[i];
        if (cds[i].n_sel > 0) std::memcpy(hs + cds[i].seg_off, r.sel.data(), sizeof(int2) * (size_t)cds[i].n_sel);
        if (cds[i].self_msg >= 0) hs[cds[i].seg_off + cds[i].n_sel] = make_int2(cds[i].self_msg, cds[i].self_start);
        std::memcpy(hq + cds[i].q_off, r.q_pos.data(), sizeof(int32_t) * r.q_pos.size());
    }
    // rows to merge: those with few splits first, then those with many (they get four lanes per 8 dimensions)
    for (int pass = 0; pass < 2 && want_items; ++pass) {
        auto wanted = [&](int n_splits) { return n_splits > 1 && (n_splits > MERGE_MANY_SPLITS) == (pass == 1); };
        for (int i = 0; i < n_calls; ++i)
            if (wanted(cds[i].n_splits))
                for (int q = 0; q < P.res[i].n_q; ++q)
                    hm[P.n_merge_rows++] = PcMergeRow{cds[i].q_off + q, cds[i].part_off + (q << cds[i].part_wide),
                                                      cds[i].n_splits | (cds[i].part_wide ? PC_MERGE_WIDE : 0), P.res[i].n_q};
        if (!tail_rows.empty() && wanted(tail.second))
            for (const PcMergeRow &mr : tail_rows) hm[P.n_merge_rows++] = mr;
        for (size_t i = 0; i < sp.groups.size(); ++i) {
            const PcShGroup &gr = sp.groups[i];
            if (wanted(gr.n_splits))
                for (int q = 0; q < gr.n_rows; ++q)
                    hm[P.n_merge_rows++] = PcMergeRow{gr.row0 + q, gr.part_off + (q << sp.wide[i]), gr.n_splits | (sp.wide[i] ? PC_MERGE_WIDE : 0), gr.n_rows};
        }
        if (pass == 0) P.n_merge_few = P.n_merge_rows;
    }
    if (!dec.empty()) std::memcpy(h + P.lay.items_dec, dec.data(), sizeof(PcItem) * dec.size());
    if (!pre.empty()) std::memcpy(h + P.lay.items_pre, pre.data(), sizeof(PcItem) * pre.size());
    if (!pre_pk.empty()) std::memcpy(h + P.lay.items_pk, pre_pk.data(), sizeof(PcItem) * pre_pk.size());
    if (!kg.empty()) std::memcpy(h + P.lay.kg_items, kg.data(), sizeof(PcGatherItem) * kg.size());
    if (!P.tok_items.empty()) std::memcpy(h + P.lay.tok_items, P.tok_items.data(), sizeof(PcTokenItem) * P.tok_items.size());
    if (!bp.row_blocks.empty()) std::memcpy(h + P.lay.bwd_rb, bp.row_blocks.data(), sizeof(int2) * bp.row_blocks.size());
    if (!bp.keys.empty()) std::memcpy(h + P.lay.bwd_keys, bp.keys.data(), sizeof(PcBwdKeyItem) * bp.keys.size());
    if (!sp.items.empty()) {
        std::memcpy(h + P.lay.sh_groups, sp.groups.data(), sizeof(PcShGroup) * sp.groups.size());
        std::memcpy(h + P.lay.sh_segs, sp.segs.data(), sizeof(PcShSeg) * sp.segs.size());
        std::memcpy(h + P.lay.sh_items, sp.items.data(), sizeof(PcShItem) * sp.items.size());
        std::memcpy(h + P.lay.sh_pos, sp.pos.data(), sizeof(int32_t) * sp.pos.size());
    }
    if (P.self.n16 > 0) {                                // (h2d_bytes fit the arguments, and the block starts the workspace: lists keep their offsets)
        P.self.ws = (uint4 *)P.ws;
        P.self.regions = (char *)P.ws + P.self_at;
        return PC_OK;
    }
    // A block too large for the arguments is read by the plan builder where it is and copied to the workspace by further
    // blocks of the same launch (a copy in front of it took 4 us on the stream, 8 from 16 KB on, and a gap); beyond
    // HOST_READ_BYTES the copy engine is the faster way.
    const bool in_place = !in_args && !recorded && P.lay.h2d_bytes <= HOST_READ_BYTES;
    if (recorded) {
        pc_launch_store_args(h, P.lay.h2d_bytes, P.ws, st);
        PC_HIP(c, hipGetLastError());
    } else if (!in_args && !in_place) {
        PC_HIP(c, hipMemcpyAsync(P.ws, h, P.lay.h2d_bytes, hipMemcpyHostToDevice, st));
        if (P.merge_releases && P.n_merge_rows > 0) P.merge_slot = slot;
        else { const int32_t rc = pc_stage_release(c, slot, st); if (rc != PC_OK) return rc; }
    }
    {
        ProfScope ps(c, 1, st);
        char *w = (char *)P.ws, *from = in_place ? h : w;
        const PcTokenWork tok = token_work(c, P, (const PcTokenItem *)(from + P.lay.tok_items));
        PcShTurns turns;
        if (P.n_sh_items > 0) turns = PcShTurns{(const int32_t *)(from + P.lay.sh_pos), (int)P.n_sh_pos, (float2 *)(w + P.lay.sh_rot)};
        auto *calls_at = (const PcCallDesc *)(from + P.lay.calls);
        auto *sel_at = (const int2 *)(from + P.lay.sel);
        auto *q_pos_at = (const int32_t *)(from + P.lay.q_pos);
        auto *segs = (PcSegment *)(w + P.lay.segs);
        auto *seg_kvoff = (int32_t *)(w + P.lay.seg_kvoff);
        auto *rot_seg = (float2 *)(w + P.lay.rot_seg), *rot_q = (float2 *)(w + P.lay.rot_q);
        auto *rot_qw = c->cfg.head_dim == 128 ? (float2 *)(w + P.lay.rot_qw) : nullptr;
        auto *tiles = (PcTile *)(w + P.lay.tiles);
        // a block writes 256 tiles in one go: the longest call decides, within reason for a batch of many
        int longest = 0;
        for (const PcCallDesc &cd : cds) if (cd.n_seg > 0) longest = std::max(longest, P.res[(size_t)(&cd - cds.data())].tiles);
        const int tile_blocks = std::max(1, std::min((longest + 255) / 256, std::max(1, 256 / n_calls)));
        // (the shared walk turns a query by its whole angle: where nothing else is launched no row's own rotation is read)
        const int rot_rows = P.n_sh_items > 0 && P.n_dec == 0 && P.n_pre == 0 && P.n_pre_pk == 0 ? 0 : P.total_q;
        if (in_args)
            pc_launch_build_plan_arg(blob, P.ws, P.lay.h2d_bytes, calls_at, n_calls, sel_at, q_pos_at, c->table_dev, c->inv_freq_dev, c->half, P.total_seg,
                                     rot_rows, segs, seg_kvoff, rot_seg, rot_q, rot_qw, tiles, tile_blocks, tok, st);
        else
            pc_launch_build_plan(calls_at, n_calls, sel_at, q_pos_at, c->table_dev, c->inv_freq_dev, c->half, P.total_seg,
                                 rot_rows, segs, seg_kvoff, rot_seg, rot_q, rot_qw, tiles, tile_blocks, tok, turns, in_place ? h : nullptr, P.ws, P.lay.h2d_bytes, st);
        PC_HIP(c, hipGetLastError());
        P.tok_done = !P.tok_items.empty();
        if (in_place) {                                  // the ring slot is free again once the plan builder is done
            if (P.merge_releases && P.n_merge_rows > 0) P.merge_slot = slot;
            else { const int32_t rc = pc_stage_release(c, slot, st); if (rc != PC_OK) return rc; }
        }
    }
    return PC_OK;
}

extern "C" {

int32_t pc_resolve_call(pc_cache *c, const pc_call *call, int32_t *starts_out, int32_t *self_start_out, int64_t *n_kv)
{
    if (!c) return PC_ERR_INVALID_ARG;
    Resolved r;
    const int32_t rc = pc_resolve(c, call, 0, r);
    if (rc != PC_OK) return rc;
    if (starts_out) for (size_t e = 0; e < r.entry_start.size(); ++e) starts_out[e] = r.entry_start[e];
    if (self_start_out) *self_start_out = r.msg_start;
    if (n_kv) *n_kv = r.n_kv;
    return PC_OK;
}

}  // extern "C"
