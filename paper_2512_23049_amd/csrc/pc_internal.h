// Structures shared by the host side of the library and its kernels.
#ifndef PC_INTERNAL_H_
#define PC_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#define PC_TILE 32            // keys per KV tile; equals the slot alignment, so a
                              // tile never straddles two messages
#define PC_VGROUP 8           // V is stored key-transposed in groups of 8 slots

// Device copy of one message-table entry (Sec. 2.4: message id -> physical span).
struct PcMsgEntry {
    int32_t slot_start;       // first slot (multiple of PC_TILE)
    int32_t len;              // tokens stored
    int32_t base_pos;         // the stored key of token t is turned to position base_pos + t
                              // (0 after an append; moved by pc_reposition)
    int32_t pad;
};

// One message of a batched append (staged by the host).
struct PcAppendItem {
    const void *k, *v;        // device, [len, H_kv, D] each
    int32_t msg;
    int32_t slot_start;
    int32_t len;
    int32_t rows;             // >= len: slots written; those behind the last token get zeros (see pc_append_rows)
};

// One token appended to an existing message (staged by the host).
struct PcTokenItem {
    int32_t msg;              // message that grows
    int32_t slot;             // physical slot the token goes to
    int32_t pos;              // base_pos + in-message index: what its key is turned to
    int32_t new_len;          // the message's length once this token is in
};

// (cos, sin) of a rotation by x radians, |x| < 2^30, rounded to fp32 from fp64: x is taken to the nearest multiple of pi/2 (two
// pieces of it; the product by the first is exact inside the fused operation) and the Taylor series of both functions are summed on
// [-pi/4, pi/4]: the sine to 2.0e-14 (x^13), the cosine to 1.1e-15 (x^14; with x^12 alone 3.9e-13, and 5 of the whole numbers below 2^24 had another
// fp32 sine or cosine than the nearest one, now none).  The device library's sincos takes every argument and every bit: some three times
// the instructions, and branches that wait for their code.  Angles are below 2^30 wherever this is called, see rope_turn.
__device__ __forceinline__ float2 rope_small(double x)
{
    const double q = __builtin_rint(x * 0.63661977236758134308);              // 2 / pi
    double r = __builtin_fma(-q, 1.57079632679489655800, x);                  // pi/2 in fp64, and what is left of it
    r = __builtin_fma(-q, 6.12323399573676603587e-17, r);
    const double z = r * r;
    double s = __builtin_fma(z, 1. / 6227020800., -1. / 39916800.);
    s = __builtin_fma(z, s, 1. / 362880.);
    s = __builtin_fma(z, s, -1. / 5040.);
    s = __builtin_fma(z, s, 1. / 120.);
    s = __builtin_fma(z, s, -1. / 6.);
    s = __builtin_fma(r * z, s, r);
    double c = __builtin_fma(z, -1. / 87178291200., 1. / 479001600.);
    c = __builtin_fma(z, c, -1. / 3628800.);
    c = __builtin_fma(z, c, 1. / 40320.);
    c = __builtin_fma(z, c, -1. / 720.);
    c = __builtin_fma(z, c, 1. / 24.);
    c = __builtin_fma(z, c, -0.5);
    c = __builtin_fma(z, c, 1.);
    const int n = (int)q;                                // quarter turns
    const float fs = (float)((n & 1) ? c : s), fc = (float)((n & 1) ? s : c);
    return make_float2(((n + 1) & 2) ? -fc : fc, (n & 2) ? -fs : fs);
}
// The rotation of a position by a frequency.  (A cache may be created with theta < 1, whose frequencies have no such bound.)
__device__ __forceinline__ float2 rope_angle(double x)
{
    if (__builtin_expect(!(__builtin_fabs(x) < 0x1.0p+30), 0)) {
        double s, c;
        sincos(x, &s, &c);
        return make_float2((float)c, (float)s);
    }
    return rope_small(x);
}
__device__ __forceinline__ float2 rope_turn(int pos, double freq) { return rope_angle((double)pos * freq); }

// A decode step's token: one frequency's pair of its key, turned.  The launches that append tokens and the decode launch that
// writes them itself store the same bits: the roundings are spelled out.
__device__ __forceinline__ float2 turn_token(float x, float y, float c, float s)
{
    return make_float2(__builtin_fmaf(x, c, -(y * s)), __builtin_fmaf(x, s, y * c));
}

// Small host-built lists travel in a kernel's arguments: no staging buffer, copy or event (a copy and its event cost the host
// 8 us and the stream 3 us of copy kernel and a gap).  The limit of a kernel's arguments is 4 KB.
#define PC_ARG_BYTES 3584
struct PcArgBlob { uint4 w[PC_ARG_BYTES / 16]; };

#define PC_TOKEN_PACK 128     // token items that travel in a kernel's arguments (2 KB)
struct PcTokenPack { PcTokenItem it[PC_TOKEN_PACK]; };

// One message of a batched position update (staged by the host).
struct PcMoveItem {
    int32_t msg;
    int32_t slot_start;
    int32_t len;
    int32_t delta;            // positions the stored keys are turned by
    int32_t new_base;
    int32_t pad[3];
};

// One call of a batch as staged by the host.
struct PcCallDesc {
    int32_t sel_off;          // first entry in the packed (msg, start) list (= seg_off: the new message is a call's last entry there)
    int32_t n_sel;
    int32_t self_msg;         // -1: none
    int32_t self_start;       // resolved
    int32_t n_q;
    int32_t q_off;            // first packed query row
    int32_t seg_off;          // first segment of this call in the segment arrays
    int32_t n_seg;            // n_sel + (self_msg >= 0)
    int32_t self_len;         // tokens in the new message (0 if none)
    int32_t n_splits;         // KV splits of this call's work items
    int32_t part_off;         // first partial row (units of rows) when n_splits > 1
    int32_t tile_off;         // first entry of this call in the tile table
    int32_t kg_tile0;         // -1, or the call's first tile in the gather buffers: its keys (turned to the positions
                              // the call gives them) and values were copied there token after token, the parents'
                              // part padded to whole tiles, then the new message
    int32_t n_par;            // tokens of the parents' part (all segments but the new message)
    int32_t rb_off;           // gradient: the call's first 32-row block among those of the batch
    int32_t part_wide;        // bf16 caches, n_splits > 1: 1 = partial outputs in fp32, a row takes two units of part_off
};

// One call whose keys the gather pass copies (staged by the host).
struct PcGatherItem {
    int32_t call;
    int32_t kg_tile0;         // its first tile in the gathered-keys buffer
    int32_t n_tiles;          // tiles of its copy: ceil(n_par / 32) + ceil(self_len / 32)
    int32_t n_par;            // tokens of the parents' part
};

// A gathered segment = one whole message placed at pos_start (built on device).
struct PcSegment {
    int32_t slot_start;
    int32_t len;
    int32_t pos_start;        // position the call assigns to the message's first token
    int32_t tile_off;         // KV tiles of this call before this segment
    int32_t rot_pos;          // pos_start - the message's stored base: what the queries are turned back by
    int32_t same_rot;         // 1: rot_pos equals that of the segment before (no new turn of the queries)
    int32_t pad[2];
};

// One 32-key KV tile of a call's gathered sequence (built on device from the segments).
#define PC_TILE_FRESH 0x100   // first tile of a segment whose query rotation differs from the one before
#define PC_TILE_SELF  0x200   // tile of the new message (causal limit applies)
struct PcTile {
    int32_t slot0;            // first physical slot of the tile (multiple of PC_TILE)
    int32_t key0;             // in-message index of its first token
    int32_t seg;              // segment index within the call
    int32_t valid_flags;      // low byte: tokens that exist (1..32); PC_TILE_* flags above
};

// One workgroup's share of an attention launch.
struct PcItem {
    int32_t call;
    int32_t unit0;            // prefill: first row unit of the workgroup; decode: 0; fp32: block of 32 (row, head) columns
    int32_t tile_begin;       // KV tile range [begin, end) within the call
    int32_t tile_end;
    int32_t split;            // split index within the call
    int32_t tile_tab0;        // the call's first entry in the tile table (a copy of its PcCallDesc::tile_off, so that
                              // the first tile descriptors can be requested without waiting for the call descriptor)
    int32_t n_splits;         // prefill: splits of this item's rows
    int32_t part_base;        // prefill, n_splits > 1: partial row of the call's row 0 in this split (row r: part_base + (r << part_wide))
};

// Gradient, key-major kernel: one workgroup's key tiles and units (bf16: 32-row block x head of the KV head, head fastest;
// fp32: block of 32 (row, head) columns).
struct PcBwdKeyItem {
    int32_t call;
    int32_t tile0;            // first of up to 4 consecutive tiles of the call
    int32_t n_tiles;
    int32_t rt_begin, rt_end; // units [begin, end) of the call
    int32_t pad[3];
};

// ---- a decode batch in one launch: its lists, calls first, travel in the kernel's arguments or lie in pinned memory ----
struct PcOneCall {
    uint16_t seg_off, n_seg;  // its entries of the (msg, start) list; the new message is the last one if self_len > 0
    uint16_t n_q, n_splits;
    int32_t q_off;            // first packed query row
    int32_t self_len;         // tokens of the new message (0: none)
    int32_t n_tiles, chunk;   // KV tiles, and how many a split takes
    int32_t part_off;         // first partial row (fp32; split s is n_q rows further) when n_splits > 1
    int32_t tok;              // row of the step's tokens that is the new message's last token, -1: none
};
struct PcOneItem {
    uint32_t call : 12, split : 8;
    uint32_t seg0 : 12;       // the call's entry that owns the split's first tile
    uint32_t tile0 : 24;      // the call's tiles before that entry
    uint32_t n_seg : 8;       // entries the split's tiles come from
};
#define PC_ONE_SEGS 64        // most of them (a wave holds them, one a lane)
#define PC_ONE_COUNTERS 256   // (call, KV head) pairs of a batch whose calls are split (two splits each: two rounds of workgroups)

// ---- a decode batch by message: a wave streams a run of tiles of one message for up to PC_RUN_ROWS of the one-row calls that list it ----
#define PC_RUN_ROWS 4
#define PC_RUN_WAVES 1024     // most waves a KV head's runs are shared out over (their first runs travel in the kernel's arguments)
struct PcMsgRun {             // one cache line
    int32_t msg;
    int32_t tile0;            // first tile of the run within the message
    int32_t size;             // tiles of the run | rows << 28
    int32_t pad;
    int32_t row[PC_RUN_ROWS];     // packed query rows
    int32_t part[PC_RUN_ROWS];    // fp32 partial rows of the run's results
    int32_t pos[PC_RUN_ROWS];     // the rows' positions minus the positions their calls give the message's first token
};
// The same for lists that are recorded into a graph, whose launches each bring PC_ARG_BYTES of them (0.9 us a launch): 40 bytes
struct PcMsgRunShort { int32_t msg, tile0, size; uint8_t row[PC_RUN_ROWS]; uint16_t part[PC_RUN_ROWS]; int32_t pos[PC_RUN_ROWS]; };
struct PcRunStarts { uint16_t first[PC_RUN_WAVES + 2]; };       // wave w of a KV head takes the runs [first[w], first[w + 1])

#define PC_MERGE_WIDE 0x10000     // partial outputs in fp32 (bf16 caches)
// One output row whose KV splits the merge kernel combines (staged by the host).
struct PcMergeRow {
    int32_t row;              // packed query row
    int32_t part_row0;        // partial row of split 0 (split s is n_q rows further; twice that if the rows are fp32, see PcCallDesc::part_wide)
    int32_t n_splits;         // | PC_MERGE_WIDE
    int32_t n_q;
};

// ---- shared decode: a group of one-row calls walks the union of its calls' messages once ----
#define PC_SH_ABSENT INT32_MIN    // rotation-table entry of a (message, row) pair the row's call does not list

// One message of a group's union list, in cache-slot order (staged by the host).
struct PcShSeg {
    int32_t slot_start;
    int32_t len;
    int32_t tile_off;         // KV tiles of the union before this message
    int32_t pad;
    uint32_t vis[8];          // bit n of word b: row 32*b + n of the group lists this message
};

// One group: consecutive one-row calls (staged by the host).
struct PcShGroup {
    int32_t seg_off, n_seg;   // its messages in the PcShSeg array
    int32_t n_tiles;          // KV tiles of the union
    int32_t row0;             // packed query row of the group's first call
    int32_t n_rows;           // calls in the group (<= 32 * 8 / g)
    int32_t rot_off;          // entry (message s, row r) of the rotation table is rot_off + s * n_rows + r
    int32_t part_off;         // first partial row when n_splits > 1 (split s is n_rows rows further; twice that if the rows are fp32)
    int32_t n_splits;
};

struct PcShItem {
    int32_t group;
    int32_t tile_begin, tile_end;     // range of the union's tiles
    int32_t split;
    int32_t seg_begin;                // message of the union that owns tile_begin
    int32_t part_wide;                // 1 = partial outputs in fp32, a row takes two units of its group's part_off
    int32_t pad[2];
};

struct PcShLaunch {
    const PcShGroup *groups;
    const PcShSeg   *segs;
    const PcShItem  *items;
    const float2    *rot;     // [entries][D/2] (cos, sin)((q_pos - start + stored base) * theta_i)
};

// Everything an attention kernel needs, passed by value.
struct PcLaunch {
    const PcCallDesc *calls;
    const PcSegment  *segs;
    const float2     *rot_seg;    // [total_seg][D/2] (cos, sin)((pos_start - stored base) * theta_i)
    const float2     *rot_q;      // [total_q][D/2]   (cos, sin)(q_pos * theta_i)
    const float2     *rot_qw;     // the same values laid out for the bf16 prefill kernel's lanes (D = 128 only, else null):
                                  // pair 16 ks + 8 hh + 2 jq + e of row R at float2 index
                                  // ((R / 32 * 1024 + ks * 256 + jq * 64 + hh * 32 + R % 32) * 2 + e
    const PcItem     *items;
    const PcTile     *tiles;      // [total tiles] per-call tile tables
    const void       *k_store;    // [H_kv][slots][D]            K turned to its in-message index
    const void       *v_store;    // bf16: [H_kv][slots/8][D][8] ; f32: [H_kv][slots][D]
    const void       *q;          // [total_q][H_q][D]
    void             *out;        // [total_q][H_q][D]
    float            *lse;        // [total_q][H_q] or null
    uint16_t         *part_o;     // [part rows][H_q][D]   partial outputs, each normalised by its own sum: fp16, or fp32 in rows of two units; fp32 caches: fp32, not normalised
    float            *part_ml;    // [part rows][H_q][2]   running max (scaled log2 domain), sum
    void             *k_gather;   // [H_kv][kg_slots][D]       keys of the calls that gather, turned to their positions
    void             *v_gather;   // [H_kv][kg_slots/8][D][8]  their values, in the cache's group-of-8 layout
    int64_t           kg_slots;   // slots of that buffer per KV head (32 per gathered tile)
    float            *kg_norm;    // [H_kv][kg_slots/32]       per tile of that buffer: the largest squared norm of its keys (as stored, bf16)
    int64_t           slots;      // capacity in slots (stride between KV heads)
    int32_t           n_q_heads, n_kv_heads;
    float             scale_log2; // softmax scale * log2(e)
};

// A decode batch in one launch: what the kernel needs besides its lists and PcLaunch.
struct PcOne {
    PcMsgEntry   *table;
    const double *inv_freq;
    const uint16_t *tok_k, *tok_v;    // [tokens][H_kv][D] rows the step appends
    uint32_t     *counters;           // [call][H_kv] splits that are done: zero between launches
    const void   *lists;              // in pinned host memory or the workspace, or null: in the arguments
    int32_t       off_sel, off_q_pos, off_items;      // within the lists, in bytes
    int32_t       n_items;
};

// A decode batch by message: what the kernel needs besides PcLaunch.
struct PcRuns {
    const PcMsgEntry *table;
    const PcMsgRun   *runs;
    const float2     *rot;            // [run][PC_RUN_ROWS][D/2] (cos, sin) of the row's position as seen from the message's stored keys, times the scores' scale
    int32_t           n_waves;
};

// An attention launch that plans for itself: every workgroup makes the tiles and rotations it needs, in a region of the workspace of its
// own, from the batch's lists in the kernel's arguments (offsets of the staged block).
struct PcSelf {
    int32_t off_calls, off_items, off_sel, off_q_pos, n16;        // n16: pieces of 16 bytes in the block, which workgroup 0 leaves in the workspace for the merge
    int32_t off_rot, off_rot_q;       // within a region: (cos, sin) of the call's entries, then of the workgroup's rows (its tiles come first)
    int64_t stride;                   // bytes of a region
    const PcMsgEntry *table;
    const double *inv_freq;
    uint4   *ws;
    char    *regions;
};
#define PC_SELF_SEGS 64               // most entries of a call: a wave looks them up one a lane

// Gradient of a bf16 batch: what its kernels need besides PcLaunch (whose items are the row-major kernels').  A unit is
// a 32-row block of one head; the blocks [rb0, rb0 + n_rb) are processed by one set of launches, and the per-unit
// buffers are indexed by (block - rb0) * n_q_heads + head.
struct PcBwd {
    const int2         *row_blocks;   // [blocks of the batch] (call, block within the call)
    const PcBwdKeyItem *key_items;
    int32_t             rb0, n_rb;
    int64_t             n_units;      // n_rb * n_q_heads
    float4             *q_turned;     // [unit][4 ks][4][64 lanes] queries turned by their positions, fp32: lane (n, hh) of entry
                                      // (ks, j): row n, dims 16 ks + 8 hh + 4 j + 0..3 (j < 2) and their partners 64 up (j >= 2)
    uint16_t           *q_pieces;     // [unit][4][32 rows][128] the same as three bf16 pieces; fourth: the output gradients
    float              *delta_part;   // [split][unit][32]
    float4             *dq_part;      // [split][unit][16][64 lanes]
    float2             *stat;         // [unit][32] (lse * log2 e, Delta)
    const float        *lse;
    const uint16_t     *d_out;
    float              *d_q, *d_k, *d_v;
    float               scale;
};

#endif
