// The plan of one workgroup, made by the workgroup itself (device code shared by the attention kernels that plan for themselves).
//
// A small batch is a chain of launches, and the plan builder's is 4 us of it, most of that the start and the end of a kernel.  Here every workgroup
// looks its call's entries up (one a lane), and writes the tiles of its range and the rotations of their messages and of its rows where the
// walk reads them: to memory of its own, which comes back from the L2 (about 1 us; registers and LDS belong to the walk).
#ifndef PC_SELF_PLAN_H_
#define PC_SELF_PLAN_H_

#include "pc_kernels.h"

namespace {

// A work item and a call of the block in the kernel's arguments (field by field: scalar loads into scalar registers)
__device__ __forceinline__ PcItem self_item(const __attribute__((address_space(4))) char *args, const PcSelf &S, int i)
{
    const auto *p = reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(args + S.off_items) + i * (int)(sizeof(PcItem) / 4);
    PcItem it;
    it.call = p[0]; it.unit0 = p[1]; it.tile_begin = p[2]; it.tile_end = p[3]; it.split = p[4]; it.tile_tab0 = p[5]; it.n_splits = p[6]; it.part_base = p[7];
    return it;
}
__device__ __forceinline__ PcCallDesc self_call(const __attribute__((address_space(4))) char *args, const PcSelf &S, int i)
{
    const auto *p = reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(args + S.off_calls) + i * (int)(sizeof(PcCallDesc) / 4);
    PcCallDesc cd;
    cd.sel_off = p[0]; cd.n_sel = p[1]; cd.self_msg = p[2]; cd.self_start = p[3]; cd.n_q = p[4]; cd.q_off = p[5]; cd.seg_off = p[6]; cd.n_seg = p[7];
    cd.self_len = p[8]; cd.n_splits = p[9]; cd.part_off = p[10]; cd.tile_off = p[11]; cd.kg_tile0 = p[12]; cd.n_par = p[13]; cd.rb_off = p[14]; cd.part_wide = p[15];
    return cd;
}

// THREADS threads; HALF frequencies.  The range [tile_begin, tile_end) of the call; rows [row0, row0 + n_rows) of it.  Ends with a barrier behind which
// what was written can be read (vector stores and scalar loads meet in the L2; nobody has read these lines before in this launch).
// early(slot_of): called as soon as the entries are known; slot_of(t) is the first slot of the call's tile t (uniform over the wave).
template <int HALF, int THREADS, class Early>
__device__ __forceinline__ void wg_plan(const PcSelf &S, const __attribute__((address_space(4))) char *args, const PcCallDesc &cd, int tile_begin, int tile_end,
                                        int row0, int n_rows, char *region, Early early)
{
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double freq = S.inv_freq[lane % HALF];
    int slot = 0, len = 0, rot = 0;
    if (lane < cd.n_seg) {
        const i32x2 ms = reinterpret_cast<const __attribute__((address_space(4))) i32x2 *>(args + S.off_sel)[cd.seg_off + lane];
        const PcMsgEntry me = S.table[ms.x];
        slot = me.slot_start; rot = ms.y - me.base_pos;
        len = lane < cd.n_sel ? me.len : cd.self_len;    // (the new message is the last entry)
    }
    const int tiles = (len + PC_TILE - 1) / PC_TILE;
    int first = tiles;                                   // the call's tiles before the lane's entry
    for (int off = 1; off < cd.n_seg; off <<= 1) {
        const int x = __shfl_up(first, off);
        if (lane >= off) first += x;
    }
    first -= tiles;
    early([&](int t) __attribute__((always_inline)) {
        const int e = 63 - (int)__builtin_clzll(__builtin_amdgcn_ballot_w64(lane < cd.n_seg && first <= t) | 1ull);
        return __builtin_amdgcn_readlane(slot, e) + (t - __builtin_amdgcn_readlane(first, e)) * PC_TILE;
    });
    const int before = __shfl_up(rot, 1);
    const bool fresh = lane == 0 || before != rot;
    PcTile *out = reinterpret_cast<PcTile *>(region);
    for (int t0 = tile_begin; t0 < tile_end; t0 += THREADS) {
        const int t = t0 + (int)threadIdx.x;
        int e = 0;
        for (int k = 1; k < cd.n_seg; ++k) e = __builtin_amdgcn_readlane(first, k) <= t ? k : e;       // (an empty entry is passed over: the next one starts where it does)
        PcTile tl;
        tl.key0 = (t - __shfl(first, e)) * PC_TILE;
        tl.slot0 = __shfl(slot, e) + tl.key0;
        tl.seg = e;
        const int left = __shfl(len, e) - tl.key0, is_fresh = __shfl((int)fresh, e);
        tl.valid_flags = min(left, PC_TILE) | (tl.key0 == 0 && is_fresh ? PC_TILE_FRESH : 0) | (cd.self_msg >= 0 && e == cd.n_seg - 1 ? PC_TILE_SELF : 0);
        if (t < tile_end) out[t - tile_begin] = tl;
    }
    constexpr int PER = 64 / HALF;                       // entries a wave makes at a time
    const int i = lane % HALF, sub = lane / HALF;
    float2 *rot_seg = reinterpret_cast<float2 *>(region + S.off_rot), *rot_q = reinterpret_cast<float2 *>(region + S.off_rot_q);
    const auto *q_pos = reinterpret_cast<const __attribute__((address_space(4))) int32_t *>(args + S.off_q_pos) + cd.q_off + row0;
    // (those of a tile of the range; an entry whose tiles all lie outside is not asked for)
    const uint64_t wanted = __builtin_amdgcn_ballot_w64(lane < cd.n_seg && first < tile_end && first + tiles > tile_begin);
#pragma unroll 1
    for (int e0 = wave * PER; e0 < cd.n_seg + n_rows; e0 += THREADS / HALF) {
        const int e = e0 + sub, r = e - cd.n_seg;
        const int from_entry = __shfl(rot, e < cd.n_seg ? e : 0);
        if (e >= cd.n_seg + n_rows || (r < 0 && !((wanted >> e) & 1))) continue;
        const int pos = r < 0 ? from_entry : q_pos[r];
        const float2 cs = rope_small((double)pos * freq);        // (the host keeps positions times frequencies below 2^29)
        if (r < 0) rot_seg[e * HALF + i] = cs;
        else rot_q[r * HALF + i] = cs;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// a pointer as it is behind the barrier: loads through it stay there, whatever the compiler takes for constant memory
template <typename T> __device__ __forceinline__ T *behind(T *p)
{
    asm volatile("" : "+s"(p)::"memory");
    return p;
}

}  // namespace

#endif
