// Launch wrappers of the kernels (internal to the library).
#ifndef PC_KERNELS_H_
#define PC_KERNELS_H_

#include "pc_internal.h"

// rows >= len: slots written, zeros behind the last token
void pc_launch_append(int dtype, const void *k, const void *v, int len, int rows, int n_kv_heads, int D,
                      int64_t slot_start, int64_t slots, const double *inv_freq, void *k_store,
                      void *v_store, PcMsgEntry *table, int msg_id, hipStream_t st);

// several whole messages in one launch
// (host_items: the same list in host memory, or null; short lists are then passed in the kernel's arguments and `items` is not read)
void pc_launch_append_batch(int dtype, const PcAppendItem *items, const PcAppendItem *host_items, int n_items, int max_rows, int n_kv_heads, int D,
                            int64_t slots, const double *inv_freq, void *k_store, void *v_store, PcMsgEntry *table,
                            hipStream_t st);

// n tokens (rows of k, v: [n, H_kv, D]) into the slots the items name
void pc_launch_append_tokens(int dtype, const PcTokenItem *items, int n, const void *k, const void *v, int n_kv_heads,
                             int D, int64_t slots, const double *inv_freq, void *k_store, void *v_store,
                             PcMsgEntry *table, hipStream_t st);

// the same for at most PC_TOKEN_PACK items, passed in the kernel's arguments (no staging copy)
void pc_launch_append_tokens_packed(int dtype, const PcTokenPack &pack, int n, const void *k, const void *v, int n_kv_heads,
                                    int D, int64_t slots, const double *inv_freq, void *k_store, void *v_store,
                                    PcMsgEntry *table, hipStream_t st);

// zero the rows of n_slots slots from slot_start on (both multiples of the tile) of the K or the V store, every KV head
void pc_launch_zero_span(int dtype, void *store, int64_t slots, int n_kv_heads, int D, int64_t slot_start, int64_t n_slots,
                           hipStream_t st);

// turn the stored keys of one message by delta positions, in place
void pc_launch_reposition(int dtype, int len, int n_kv_heads, int D, int64_t slot_start, int64_t slots, int delta,
                          int new_base, const double *inv_freq, void *k_store, PcMsgEntry *table, int msg_id,
                          hipStream_t st);

// the same for a staged list of messages, one launch (blockIdx.y = message)
void pc_launch_reposition_batch(int dtype, const PcMoveItem *items, int n_items, int n_kv_heads, int D, int64_t slots,
                                const double *inv_freq, void *k_store, PcMsgEntry *table, hipStream_t st);

// tok (may be empty): tokens the same launch appends to existing messages (a decode step: one launch for both)
struct PcTokenWork {
    const PcTokenItem *items = nullptr; int n = 0;
    const void *k = nullptr, *v = nullptr;        // [n, H_kv, D] rows in item order
    void *k_store = nullptr, *v_store = nullptr;
    int64_t slots = 0; int n_kv_heads = 0, D = 0, dtype = 0;
};
// The rotations of a shared decode walk: n positions, PC_SH_ABSENT where a row does not list the message, to [n][64] (cos, sin).
struct PcShTurns { const int32_t *pos = nullptr; int n = 0; float2 *rot = nullptr; };
// tile_blocks: blocks that share out a call's tile table
void pc_launch_build_plan(const PcCallDesc *calls, int n_calls, const int2 *sel, const int32_t *q_pos,
                          PcMsgEntry *table, const double *inv_freq, int half, int total_seg,
                          int total_q, PcSegment *segs, int32_t *seg_kvoff, float2 *rot_seg,
                          float2 *rot_q, float2 *rot_qw, PcTile *tiles, int tile_blocks, const PcTokenWork &tok, const PcShTurns &turns, const void *staged, void *ws, size_t h2d_bytes,
                          hipStream_t st);
// (staged != null: calls, sel, q_pos, tok.items and turns.pos lie in that block of pinned host memory, which the kernel copies to the workspace)
// the same with the staged block (h2d_bytes <= PC_ARG_BYTES, at the start of the workspace) in the kernel's arguments: calls,
// sel, q_pos and tok.items are addresses within the workspace, which the kernel fills for the kernels behind it
void pc_launch_build_plan_arg(const PcArgBlob &blob, void *ws, size_t h2d_bytes, const PcCallDesc *calls, int n_calls, const int2 *sel, const int32_t *q_pos,
                              PcMsgEntry *table, const double *inv_freq, int half, int total_seg,
                              int total_q, PcSegment *segs, int32_t *seg_kvoff, float2 *rot_seg,
                              float2 *rot_q, float2 *rot_qw, PcTile *tiles, int tile_blocks, const PcTokenWork &tok, hipStream_t st);

// `bytes` of host memory to dst (16-byte aligned) through kernels' arguments, read before the function returns
void pc_launch_store_args(const void *host, size_t bytes, void *dst, hipStream_t st);

void pc_launch_expand_tables(const PcSegment *segs, const int32_t *seg_kvoff, int n_seg, int64_t n_kv,
                             int32_t *kv_slot, int32_t *kv_pos, hipStream_t st);

// split_lanes: 1, or 4 for rows with many splits (their splits are shared out over four lanes)
// done.at != null: done.value goes there (pinned host memory), as what came before this launch on the stream is done
struct PcMergeDone { uint32_t *at = nullptr; uint32_t value = 0; };
void pc_launch_merge(int dtype, const PcMergeRow *merge_rows, int n_merge_rows, int split_lanes, bool many, const uint16_t *part_o,
                     const float *part_ml, void *out, float *lse, int n_q_heads, int D, const PcMergeDone &done, hipStream_t st);

// fp32 caches: the work items L.items (unit0: block of 32 (row, head) columns of the KV head), partials in fp32; then the
// rows whose tiles were split
void pc_launch_attend_f32(const PcLaunch &L, int n_items, int D, hipStream_t st);
// the same for a launch that plans for itself, from the staged block in its arguments
void pc_launch_attend_f32_self(const PcArgBlob &blob, const PcLaunch &L, const PcSelf &S, int n_items, int D, hipStream_t st);
void pc_launch_merge_f32(const PcMergeRow *rows, int n_rows, const void *part_o, const float *part_ml, void *out, float *lse, int n_q_heads, int D,
                         hipStream_t st);

// gradient of the attention for fp32 caches; d_k collects the gradient w.r.t. the stored keys until the finalize pass
// (row-major items L.items as in pc_launch_attend_f32, unsplit; key-major items over blocks of 32 columns)
void pc_launch_attend_bwd_f32(const PcLaunch &L, int n_items, const PcBwdKeyItem *key_items, int n_key_items, int D, const float *lse,
                              const float *d_out, float scale, float *delta, float *d_q, float *d_k, float *d_v, hipStream_t st);
// the same for bf16 caches on the matrix cores: the row blocks [B.rb0, B.rb0 + B.n_rb), their row-major work items L.items
// and key-major work items B.key_items
void pc_launch_attend_bwd_bf16(const PcLaunch &L, const PcBwd &B, int n_items, int n_key_items, hipStream_t st);
// (host_msgs: the same list in host memory, or null; short lists are passed in the kernel's arguments and `msgs` is not read)
void pc_launch_grad_keys_finalize(const PcMsgEntry *msgs, const PcMsgEntry *host_msgs, int n_msgs, int n_kv_heads, int D, const double *inv_freq,
                                  float *d_k, hipStream_t st);

// keys (turned to the positions their call gives them) and values of the listed calls, token after token, into
// L.k_gather / L.v_gather
void pc_launch_gather(const PcLaunch &L, const PcGatherItem *items, int n_items, int64_t n_tiles, const int32_t *seg_kvoff,
                      hipStream_t st);

// bf16 MFMA kernels (D = 128)
void pc_launch_decode_bf16(const PcLaunch &L, int n_items, hipStream_t st);
// a batch of decode calls: plan, token append, attention and merge in one launch (blob: bytes of its lists, unless O.lists has them)
void pc_launch_decode_one_bf16(const PcArgBlob &blob, size_t bytes, const PcLaunch &L, const PcOne &O, hipStream_t st);
// lists (runs first, `rest` bytes behind them; short_runs: as PcMsgRunShort) to the workspace, the runs' rotations, and a step's tokens into the cache, in one launch
void pc_launch_runs_prepare(const void *lists, void *to, size_t rest, int n_runs, bool short_runs, float scale, const PcTokenWork &tok, const double *inv_freq, PcMsgEntry *table,
                            float2 *rot, hipStream_t st);
// a decode batch by message (H_kv n_waves waves); its parts, fp32, are added by pc_launch_merge
void pc_launch_decode_runs_bf16(const PcLaunch &L, const PcRuns &O, const PcRunStarts &starts, hipStream_t st);
void pc_launch_prefill_bf16(const PcLaunch &L, int n_items, bool packed, hipStream_t st);   // packed: the items of calls that gathered

// shared decode (wide: some items have part_wide set)
void pc_launch_decode_shared_bf16(const PcLaunch &L, const PcShLaunch &S, int n_items, bool wide, hipStream_t st);

#endif
