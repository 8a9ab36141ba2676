// bf16 MFMA attention kernels for gfx950: split-K decode (the prefill kernel is in
// pc_kernels_prefill.hip and shares the formulation described here).
//
// Both work on the transposed problem: scores S^T = K~ . Q^T (rows = keys, columns =
// query rows), so that the softmax statistics of a query row live in one lane column and
// the probabilities come out of the first MFMA already in the register layout the second
// MFMA (O^T = V^T . P^T) wants for its B operand.  V is stored key-transposed in groups of
// 8 slots, so the A operand of the second MFMA is one 16-byte load per lane.
//
// Keys are stored turned to b + t (in-message index t, base b = 0 unless the message was
// repositioned); a message placed at start s then needs the query turned by (q_pos - s + b):
// <R(p)q, R(s+t)k> = <R(p-s+b)q, R(b+t)k>.  The query is turned once by p (table rot_q) and
// once more per segment by -(s - b) (table rot_seg).
#include "pc_mfma_common.h"

// ----------------------------------------------------------------------------------------
// K4: split-K decode.  One workgroup of 4 waves per (work item, KV head); the g query heads
// of the KV head times the call's (few) query rows are the <= 16 columns of 16x16x32 MFMAs.
// Each wave streams a contiguous run of 32-key tiles straight from HBM into registers
// (K rows as MFMA A operands, V groups as A operands of the second MFMA), double buffered.
// Two workgroups per CU (256 registers per wave): the kernel lives on bytes in flight, and
// with one workgroup per CU (what an unconstrained register allocation gives) it reached
// only four fifths of the bandwidth it reaches with two.
// ----------------------------------------------------------------------------------------
// maximum over the lane pairs (l, l ^ 16) and (l, l ^ 32) without a trip through LDS: the swap
// instructions exchange 16- resp. 32-lane rows between their two operands
__device__ __forceinline__ float max_lanes_xor16(float x)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_lanes_xor32(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// One 16-byte-per-lane direct load: lane l's 16 bytes land at lds_wave_base + 16*l (see pc_kernels_prefill.hip)
__device__ __forceinline__ void dma16(const void *gbase_uniform, unsigned lane_off, unsigned lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(lds_wave_base), "v"(lane_off), "s"(gbase_uniform) : "memory", "m0");
}

struct DecTile {
    uint4 k[2][4];      // [16-key half][d step of 32]
    uint4 v[8];         // [16-d block]
    int seg;            // which rotation row turns the query for it
    int key0;           // first in-message token of the tile
    int valid;          // tokens of the tile that exist (1..32)
    bool fresh;         // first tile of a segment whose query rotation differs from the one before
    bool self;          // a tile of the new message (by message: a run's last one)
    bool there;         // (by message) there is such a tile
};

// Sixteen loads whatever the tile: loads under conditions of their own make the compiler wait for all that is in flight, the next tile
// included, before it uses any of it.  Keys and groups of values past the tile's end read the last one
// that exists (no further line of memory); drop_dead takes the values out.  A uniform address and a 32-bit offset a lane.
__device__ __forceinline__ void dec_load(DecTile &T, const uint16_t *__restrict__ kb, const uint16_t *__restrict__ vb,
                                         int slot0, int valid, int lane)
{
    const int m = lane & 15, a = lane >> 4, last = max(valid - 1, 0);
    const char *kt = reinterpret_cast<const char *>(kb + (int64_t)slot0 * PC_D), *vt = reinterpret_cast<const char *>(vb + (int64_t)slot0 * PC_D);
#pragma unroll
    for (int tau = 0; tau < 2; ++tau) {
        const unsigned at = (unsigned)(min(8 * (m >> 2) + 4 * tau + (m & 3), last) * (PC_D * 2) + 16 * a);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) T.k[tau][ks] = ldg16(kt + at + 64 * ks);
    }
    const unsigned at = (unsigned)(min(a, last / PC_VGROUP) * (PC_D * PC_VGROUP * 2) + m * (PC_VGROUP * 2));
#pragma unroll
    for (int db = 0; db < 8; ++db) T.v[db] = ldg16(vt + at + 16 * db * (PC_VGROUP * 2));
}
// the groups of values that hold no token, as zeros: what stands in for them may be infinite, and their probabilities are zero
__device__ __forceinline__ void drop_dead(DecTile &T, int lane)
{
    const bool dead = 8 * (lane >> 4) >= T.valid;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
        T.v[db].x = dead ? 0u : T.v[db].x; T.v[db].y = dead ? 0u : T.v[db].y;
        T.v[db].z = dead ? 0u : T.v[db].z; T.v[db].w = dead ? 0u : T.v[db].w;
    }
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// The walk of one workgroup: this wave's run of tiles of the columns (row, head) of KV head kh, then its NW waves' results
// combined and written: the finished rows if the call is not split, else the split's part.
// describe(t): {slot0, key0, rotation row, valid | flags} of the call's tile t.  Rotation rows (cos, sin): seg_rot(row of the
// tile), q_rot(query row of the call, f), which calls f once to request the wave's first tile.
// ONE: the launch merges its splits itself; a part is fp32 then and is stored at agent scope, for the workgroup that merges.
struct DecCall { int n_q, q_off, self_lim0, n_splits, split, part_off, part_wide; };      // self_lim0: own tokens before the query rows
template <bool ONE, int NW, class Describe, class SegRot, class QRot>
__device__ __forceinline__ void decode_walk(const PcLaunch &L, const DecCall cd, int kh, int tile, int tile_stop, Describe describe, SegRot seg_rot, QRot q_rot,
                                            float (&s_acc)[NW][16][PC_D + 4], float (&s_m)[NW][16], float (&s_l)[NW][16])
{
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, a = lane >> 4;
    const int n_cols = cd.n_q * g;
    const int qr = n / g, qj = n - qr * g;               // column -> (query row, head in group)
    const bool col_ok = n < n_cols;
    const int R = cd.q_off + (col_ok ? qr : 0);
    const int h = kh * g + (col_ok ? qj : 0);
    const int self_lim = cd.self_lim0 + qr;              // last own token this column sees
    i32x4 next_desc = describe(tile);                    // {slot0, key0, seg, valid | flags}

    const uint16_t *kb = (const uint16_t *)L.k_store + (int64_t)kh * L.slots * PC_D;
    const uint16_t *vb = (const uint16_t *)L.v_store + (int64_t)kh * L.slots * PC_D;
    auto fetch = [&](DecTile &T, int t) __attribute__((always_inline)) {       // t is the tile next_desc describes
        const i32x4 d = next_desc;
        next_desc = describe(t + 1);
        T.seg = d.z; T.key0 = d.y; T.valid = d.w & 0xFF; T.fresh = (d.w & PC_TILE_FRESH) != 0; T.self = (d.w & PC_TILE_SELF) != 0;
        dec_load(T, kb, vb, d.x, T.valid, lane);
    };
    // query turned by its own position, kept in fp32: element (ks, j) is dim 32*ks + 8*a + j
    float qh[4][8];
    DecTile A, B;
    {
        const uint16_t *qp = (const uint16_t *)L.q + ((int64_t)R * L.n_q_heads + h) * PC_D + 8 * a;
        uint4 raw[2][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) { raw[ks][0] = ldg16(qp + 32 * ks); raw[ks][1] = ldg16(qp + 32 * ks + 64); }
        const float2 *rq = q_rot(col_ok ? qr : 0, [&]() __attribute__((always_inline)) {
            if (tile < tile_stop) fetch(A, tile);
            if (tile + 1 < tile_stop) fetch(B, tile + 1);
        }) + 8 * a;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint4 lo = raw[ks][0], hi = raw[ks][1];
            const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float x = (j & 1) ? bf_hi(lw[j >> 1]) : bf_lo(lw[j >> 1]);
                const float y = (j & 1) ? bf_hi(hw[j >> 1]) : bf_lo(hw[j >> 1]);
                const float2 cs = rq[32 * ks + j];
                // (the softmax scale, times log2 e, rides on the query: scores come out of the MFMA ready for exp2)
                qh[ks][j] = col_ok ? (x * cs.x - y * cs.y) * L.scale_log2 : 0.f;
                qh[ks + 2][j] = col_ok ? (x * cs.y + y * cs.x) * L.scale_log2 : 0.f;
            }
        }
    }

    float m_run = -INFINITY, l_run = 0.f;
    f32x4 acc[8];
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db] = (f32x4){0.f, 0.f, 0.f, 0.f};

    int cur_seg = -1;
    bf16x8 qop[4];
    auto compute = [&](DecTile &T) __attribute__((always_inline)) {
        if (T.fresh || cur_seg < 0) {                    // turn the query by -(segment start - stored base): a new
            cur_seg = T.seg;                             // rotation starts here, or the wave starts inside a segment
            const float2 *rs = seg_rot(cur_seg) + 8 * a;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                uint32_t lo[4], hi[4];
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const float2 c0 = rs[32 * ks + j], c1 = rs[32 * ks + j + 1];
                    const float x0 = qh[ks][j], y0 = qh[ks + 2][j], x1 = qh[ks][j + 1], y1 = qh[ks + 2][j + 1];
                    lo[j >> 1] = pack_bf16(x0 * c0.x + y0 * c0.y, x1 * c1.x + y1 * c1.y);
                    hi[j >> 1] = pack_bf16(y0 * c0.x - x0 * c0.y, y1 * c1.x - x1 * c1.y);
                }
                qop[ks] = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
                qop[ks + 2] = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            }
        }
        f32x4 s[2];
#pragma unroll
        for (int tau = 0; tau < 2; ++tau) {
            s[tau] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                s[tau] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.k[tau][ks]), qop[ks], s[tau], 0, 0, 0);
        }
        // lane holds keys 8a + 0..7 of column n
        const int lim = T.self ? min(T.valid, self_lim - T.key0 + 1) : T.valid;
        float sc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[j] = s[j >> 2][j & 3];
        if (T.valid < PC_TILE || T.self) {      // ragged or causal tile (uniform over the wave): mask
#pragma unroll
            for (int j = 0; j < 8; ++j) sc[j] = (8 * a + j < lim) ? sc[j] : -INFINITY;
            drop_dead(T, lane);
        }
        float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
        mx = max_lanes_xor16(mx);
        mx = max_lanes_xor32(mx);
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        // the row sum is taken over the probabilities as the second MFMA sees them (rounded to bf16): the
        // rounding then cancels between numerator and denominator (a row with a single key returns its V exactly)
        uint32_t pk[4];
        float ps = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pk[j] = pack_bf16(__builtin_amdgcn_exp2f(sc[2 * j] - m_safe), __builtin_amdgcn_exp2f(sc[2 * j + 1] - m_safe));
            ps += bf_lo(pk[j]) + bf_hi(pk[j]);
        }
        l_run = l_run * alpha + ps;
        m_run = m_new;
        const bool rescale = __builtin_amdgcn_ballot_w64(alpha != 1.f) != 0;   // rare once the running maxima have settled
        const bf16x8 pop = __builtin_bit_cast(bf16x8, make_uint4(pk[0], pk[1], pk[2], pk[3]));
        if (rescale) {
#pragma unroll
            for (int db = 0; db < 8; ++db) acc[db] *= alpha;
        }
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.v[db]), pop, acc[db], 0, 0, 0);
    };

    // A tile is requested as soon as its registers are free, two tiles ahead.  The long part of the walk has no way through it but one: where a
    // path on which a tile was not requested joins, the compiler waits for all that is in flight.  (us a step: 64 calls over 146 tiles of 10
    // messages each 131 -> 127, one over 770 of 151 26.3 -> 25.8, four over 24 of 5 10.9 -> 10.7.)
    // (Not behind the plan builder, whose rotations come from memory: 11 registers too many.)
    if (ONE && tile + 3 < tile_stop) {
        __builtin_amdgcn_s_waitcnt(0x4F70);              // vmcnt(16): the first tile is there
        do {
            compute(A);
            fetch(A, tile + 2);
            compute(B);
            fetch(B, tile + 3);
            tile += 2;
        } while (tile + 3 < tile_stop);
    }
    while (tile < tile_stop) {                           // three tiles or fewer, the first two of them requested
        compute(A);
        if (tile + 2 < tile_stop) fetch(A, tile + 2);
        if (++tile >= tile_stop) break;
        compute(B);
        if (!ONE && tile + 2 < tile_stop) fetch(B, tile + 2);
        ++tile;
    }

    // combine lane groups, then the waves
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (a == 0) { s_m[wave][n] = m_run; s_l[wave][n] = l_run; }
    int at = threadIdx.x;
    asm volatile("" : "+v"(at));                         // (the address is made here: in front of the loop its registers would be spilled)
    f32x4 *const to = reinterpret_cast<f32x4 *>(&s_acc[at >> 6][at & 15][(at >> 4 & 3) * 4]);      // dims 16 db + 4 a + 0..3 of column n
#pragma unroll
    for (int db = 0; db < 8; ++db) to[4 * db] = acc[db];
    __syncthreads();
    for (int idx = threadIdx.x; idx < n_cols * (PC_D / 2); idx += 64 * NW) {
        const int col = idx / (PC_D / 2), d = 2 * (idx - col * (PC_D / 2));
        float mm = s_m[0][col];
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, s_m[w][col]);
        float o0 = 0.f, o1 = 0.f, l = 0.f;
        if (mm > -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float sc = (s_m[w][col] > -INFINITY) ? exp2f(s_m[w][col] - mm) : 0.f;
                const float2 x = *reinterpret_cast<const float2 *>(&s_acc[w][col][d]);
                o0 += x.x * sc;
                o1 += x.y * sc;
                l += s_l[w][col] * sc;
            }
        }
        const float x0 = l > 0.f ? o0 / l : 0.f, x1 = l > 0.f ? o1 / l : 0.f;
        const int r = col / g, hq = kh * g + (col - r * g);
        const int64_t Rr = cd.q_off + r;
        if (cd.n_splits == 1) {
            *reinterpret_cast<uint32_t *>((uint16_t *)L.out + (Rr * L.n_q_heads + hq) * PC_D + d) = pack_bf16(x0, x1);
            if (L.lse && d == 0) L.lse[Rr * L.n_q_heads + hq] = (l > 0.f) ? (mm + log2f(l)) * 0.6931471805599453f : -INFINITY;
        } else if constexpr (ONE) {
            const int64_t pr = (int64_t)cd.part_off + (int64_t)cd.split * cd.n_q + r;
            uint64_t *po = reinterpret_cast<uint64_t *>(L.part_o) + ((pr * L.n_q_heads + hq) * PC_D + d) / 2;
            __hip_atomic_store(po, (uint64_t)__float_as_uint(x0) | (uint64_t)__float_as_uint(x1) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (d == 0)
                __hip_atomic_store(reinterpret_cast<uint64_t *>(L.part_ml) + pr * L.n_q_heads + hq,
                                   (uint64_t)__float_as_uint(mm) | (uint64_t)__float_as_uint(l) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const int64_t pr = (int64_t)cd.part_off + (((int64_t)cd.split * cd.n_q + r) << cd.part_wide);
            if (cd.part_wide) *reinterpret_cast<float2 *>(reinterpret_cast<float *>(L.part_o + pr * L.n_q_heads * PC_D) + hq * PC_D + d) = make_float2(x0, x1);
            else *reinterpret_cast<uint32_t *>(L.part_o + (pr * L.n_q_heads + hq) * PC_D + d) = pack_f16(x0, x1);
            if (d == 0) *reinterpret_cast<float2 *>(L.part_ml + (pr * L.n_q_heads + hq) * 2) = make_float2(mm, l);
        }
    }
}

__global__ __launch_bounds__(256, 2) void pc_decode_bf16_kernel(PcLaunch L)
{
    __shared__ __attribute__((aligned(16))) float s_acc[4][16][PC_D + 4];
    __shared__ float s_m[4][16], s_l[4][16];

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const PcItem item = L.items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int wave = threadIdx.x >> 6;
    // this wave's contiguous run of tiles
    const int per_wave = (item.tile_end - item.tile_begin + 3) >> 2;
    const int tile = item.tile_begin + wave * per_wave;
    const int tile_stop = min(item.tile_end, tile + per_wave);
    // Where a tile lives comes from the call's tile table (written by the plan builder), read with a
    // scalar load one tile ahead of the loads it steers; the first one is requested in front of
    // the query, so that the wave's first K/V loads do not wait behind a search through the segments.
    const PcTile *tile_tab = L.tiles + item.tile_tab0;   // (from the work item: requested beside the call descriptor, not behind it)
    auto describe = [&](int t) {
        const int tc = __builtin_amdgcn_readfirstlane(max(0, min(t, item.tile_end - 1)));
        if (item.tile_end <= 0) return (i32x4){0, 0, 0, 0};                   // a call that sees nothing has no table
        return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(tile_tab + tc));
    };
    const DecCall dc{cd.n_q, cd.q_off, cd.self_len - cd.n_q, cd.n_splits, item.split, cd.part_off, cd.part_wide};
    decode_walk<false, 4>(L, dc, kh, tile, tile_stop, describe,
                       [&](int seg) { return L.rot_seg + (int64_t)(cd.seg_off + seg) * (PC_D / 2); },
                       [&](int r, auto first_tile) { first_tile(); return L.rot_q + (int64_t)(cd.q_off + r) * (PC_D / 2); }, s_acc, s_m, s_l);
}

// The splits of a (call, KV head) merged by one workgroup of ONE_WAVES waves, as pc_merge_kernel does it for a row: 16 * SL threads a
// column, eight dimensions and one of SL parts of the splits each, in split order.  What counts is one round trip to memory: SL
// is as large as the threads allow, and eight splits of a part are requested together.
#define ONE_WAVES 4
__device__ __forceinline__ void merge_cols(const PcLaunch &L, const DecCall &cd, int kh)
{
    const int g = L.n_q_heads / L.n_kv_heads, n_cols = cd.n_q * g;
    const int SL = n_cols > 8 ? 1 : n_cols > 4 ? 2 : 4;  // (16 columns at most, 256 threads)
    static_assert(ONE_WAVES * 64 == 256, "as SL has it");
    const int sub = threadIdx.x & 15, sg = (threadIdx.x >> 4) & (SL - 1), col = (int)threadIdx.x / (16 * SL);
    const int part = (cd.n_splits + SL - 1) / SL, s_begin = sg * part, s_end = col < n_cols ? min(s_begin + part, cd.n_splits) : 0;
    const int r = col / g, h = kh * g + (col - r * g);
    const int64_t at0 = ((int64_t)cd.part_off + r) * L.n_q_heads + h, step = (int64_t)cd.n_q * L.n_q_heads;
    const float2 *ml_at = reinterpret_cast<const float2 *>(L.part_ml) + at0;
    const float4 *o_at = reinterpret_cast<const float4 *>(L.part_o) + at0 * (PC_D / 4) + 2 * sub;
    float m = -INFINITY, l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int s0 = s_begin; s0 < s_end; s0 += 8) {
        float2 ml[8];
        float4 v[8][2];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ml[u] = make_float2(-INFINITY, 0.f);
            v[u][0] = v[u][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s0 + u < s_end) {
                ml[u] = ml_at[(s0 + u) * step];
                v[u][0] = o_at[(s0 + u) * step * (PC_D / 4)];
                v[u][1] = o_at[(s0 + u) * step * (PC_D / 4) + 1];
            }
        }
        float m_new = m;
#pragma unroll
        for (int u = 0; u < 8; ++u) m_new = fmaxf(m_new, ml[u].x);
        if (m_new == -INFINITY) continue;
        const float keep = m > -INFINITY ? exp2f(m - m_new) : 0.f;
        l *= keep;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] *= keep;
        m = m_new;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float w = ml[u].x > -INFINITY ? ml[u].y * exp2f(ml[u].x - m) : 0.f;
            l += w;
#pragma unroll
            for (int k = 0; k < 2; ++k) { o[4 * k] += v[u][k].x * w; o[4 * k + 1] += v[u][k].y * w; o[4 * k + 2] += v[u][k].z * w; o[4 * k + 3] += v[u][k].w * w; }
        }
    }
    // parts 0+1 and 2+3 (16 lanes apart), then the two halves (32 apart); the swaps give both values of a pair to both lanes
    auto fold = [&](auto swap) __attribute__((always_inline)) {
        const auto mm = swap(m), ll = swap(l);
        m = fmaxf(mm.x, mm.y);
        const float w0 = mm.x > -INFINITY ? exp2f(mm.x - m) : 0.f, w1 = mm.y > -INFINITY ? exp2f(mm.y - m) : 0.f;
        l = ll.x * w0 + ll.y * w1;
#pragma unroll
        for (int j = 0; j < 8; ++j) { const auto x = swap(o[j]); o[j] = x.x * w0 + x.y * w1; }
    };
    if (SL > 1) fold([](float x) { const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                                   return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1])); });
    if (SL > 2) fold([](float x) { const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                                   return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1])); });
    if (sg != 0 || col >= n_cols) return;
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const int64_t Rr = (int64_t)(cd.q_off + r) * L.n_q_heads + h;
    *reinterpret_cast<uint4 *>((uint16_t *)L.out + Rr * PC_D + 8 * sub) =
        make_uint4(pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv), pack_bf16(o[4] * inv, o[5] * inv), pack_bf16(o[6] * inv, o[7] * inv));
    if (L.lse && sub == 0) L.lse[Rr] = l > 0.f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

// A batch of decode calls in ONE launch: no plan builder in front, no merge behind.  Such a batch is a chain of latencies:
// as three launches, 4 calls over 700 tokens took 4.2 us of plan, 8 of attention and 3.6 of merge, most of each the start and
// the end of a kernel; one launch takes 11.  The lists come in the kernel's arguments, or are read in pinned memory (a few
// hundred bytes a workgroup; the plan builder did the same, then copied them for the others).  Every wave looks the split's messages
// up in the device table itself, one a lane (the host says which entry owns the split's first tile), and finds a tile's place
// by a ballot over them; the rotations of the split's messages and query rows are shared out over the waves and computed into
// LDS while the first tiles are on their way (fp64, rounded to fp32, as in the plan builder).  A decode step's new token is
// written by the wave that reads it.  The workgroup whose split of a (call, KV head) is done last merges them, in split order
// whichever comes last.  (By time stamps of a workgroup's first wave, for 4 calls over 700 tokens and one over 23 thousand:
// 1.4 and 1.6 us until it knows its tiles, 1.9 and 3.1 for rotations and queries, 0.28 a tile and workgroup -- 57 GB/s is what
// a compute unit draws with these loads, with four waves or eight --, 1.0 and 1.6 to combine the waves, 1.4 to publish a part
// and learn that it is the last, 2.3 and 3.5 to merge.)
template <int BYTES> struct PcArgs { uint4 w[BYTES / 16]; };
template <> struct PcArgs<0> {};
template <int BYTES>
__global__ __launch_bounds__(64 * ONE_WAVES, 2) void pc_decode_one_bf16_kernel(const PcArgs<BYTES> blob, PcLaunch L, PcOne O)
{
    __shared__ __attribute__((aligned(16))) float s_acc[ONE_WAVES][16][PC_D + 4];
    __shared__ float s_m[ONE_WAVES][16], s_l[ONE_WAVES][16];
    __shared__ float2 s_rot[PC_ONE_SEGS + 16][PC_D / 2]; // (cos, sin) of the split's messages, then of the query rows' positions
    __shared__ int s_last;

    typedef const __attribute__((address_space(4))) char *KernArg;
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    typedef int i32x8 __attribute__((ext_vector_type(8)));
    typedef const __attribute__((address_space(4))) i32x2 *KernArg2;
    const KernArg args = BYTES ? (KernArg)__builtin_amdgcn_kernarg_segment_ptr() : (KernArg)(uintptr_t)O.lists;
    const int kh = blockIdx.x % L.n_kv_heads;            // consecutive workgroups (one per XCD) take different KV heads
    const PcOneItem item = __builtin_bit_cast(PcOneItem, ((KernArg2)(args + O.off_items))[blockIdx.x / L.n_kv_heads]);
    const int call = item.call, split = item.split;
    const PcOneCall cd = __builtin_bit_cast(PcOneCall, ((const __attribute__((address_space(4))) i32x8 *)args)[call]);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile_begin = split * cd.chunk, tile_end = min(cd.n_tiles, tile_begin + cd.chunk);
    const int per_wave = (tile_end - tile_begin + ONE_WAVES - 1) / ONE_WAVES;
    const int tile = tile_begin + wave * per_wave;
    const int tile_stop = min(tile_end, tile + per_wave);
    const double freq = O.inv_freq[lane];                // (a lane is a frequency pair wherever rotations are made)

    // the split's messages, one a lane
    const bool have = lane < item.n_seg;
    int m = 0, m_slot = 0, m_len = 0, m_rot = 0, m_base = 0;
    if (have) {
        const i32x2 ms = ((KernArg2)(args + O.off_sel))[cd.seg_off + item.seg0 + lane];
        m = ms.x;
        const PcMsgEntry me = O.table[m];
        m_slot = me.slot_start; m_base = me.base_pos; m_rot = ms.y - me.base_pos;
        // (the new message's length comes from the host: its last token may be appended by this launch)
        m_len = (cd.self_len > 0 && item.seg0 + lane == cd.n_seg - 1) ? cd.self_len : me.len;
    }
    const int tiles = (m_len + PC_TILE - 1) / PC_TILE;
    int m_tile = tiles;
    for (int off = 1; off < item.n_seg; off <<= 1) {
        const int x = __shfl_up(m_tile, off);
        if (lane >= off) m_tile += x;
    }
    m_tile += item.tile0 - tiles;                        // the call's tiles before the lane's message
    const int self_lane = cd.self_len > 0 ? cd.n_seg - 1 - item.seg0 : -1;
    auto describe = [&](int t) {
        const int e = 63 - (int)__builtin_clzll(__builtin_amdgcn_ballot_w64(have && m_tile <= t) | 1ull);
        i32x4 d;
        d.y = (t - __builtin_amdgcn_readlane(m_tile, e)) * PC_TILE;
        d.x = __builtin_amdgcn_readlane(m_slot, e) + d.y;
        d.z = e;
        d.w = min(__builtin_amdgcn_readlane(m_len, e) - d.y, PC_TILE) | (d.y == 0 ? PC_TILE_FRESH : 0) | (e == self_lane ? PC_TILE_SELF : 0);
        return d;
    };
    // the step's token goes to the call's last tile, which one wave alone reads
    const bool token = cd.tok >= 0 && tile < tile_stop && tile_stop == cd.n_tiles;
    uint16_t tok[4];                                     // lane = dims lane and lane + 64 of the KV head's row: K, then V
    if (token) {
        const int64_t row = ((int64_t)cd.tok * L.n_kv_heads + kh) * PC_D + lane;
        tok[0] = O.tok_k[row]; tok[1] = O.tok_k[row + PC_D / 2]; tok[2] = O.tok_v[row]; tok[3] = O.tok_v[row + PC_D / 2];
    }
    // (the host keeps positions below 2^28 and frequencies at most 1: a start less a stored base stays below 2^29, or 2^30 behind a message of 2^28 tokens)
    if (token) {
        const int at = cd.self_len - 1;
        const float2 cs = rope_small((double)(__builtin_amdgcn_readlane(m_base, self_lane) + at) * freq);
        const int64_t slot = __builtin_amdgcn_readlane(m_slot, self_lane) + at;
        const float2 turned = turn_token(bf_lo(tok[0]), bf_lo(tok[1]), cs.x, cs.y);
        uint16_t *kd = (uint16_t *)const_cast<void *>(L.k_store) + (kh * L.slots + slot) * PC_D + lane;
        kd[0] = to_bf16(turned.x);
        kd[PC_D / 2] = to_bf16(turned.y);
        uint16_t *vd = (uint16_t *)const_cast<void *>(L.v_store) + ((kh * L.slots + slot) / PC_VGROUP * PC_D + lane) * PC_VGROUP + slot % PC_VGROUP;
        vd[0] = tok[2];
        vd[PC_D / 2 * PC_VGROUP] = tok[3];
        if (kh == 0 && lane == 0) O.table[__builtin_amdgcn_readlane(m, self_lane)].len = cd.self_len;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");              // the token is written before this wave reads its tile
    }
    auto prepare = [&](int r, auto first_tiles) __attribute__((always_inline)) {
        first_tiles();
        typedef const __attribute__((address_space(4))) int32_t *KernArgInt;
        const KernArgInt q_pos = (KernArgInt)(args + O.off_q_pos) + cd.q_off;
        const int n_ent = item.n_seg + cd.n_q;
#pragma unroll 1
        for (int e = wave; e < n_ent; e += ONE_WAVES) {
            const int pos = e < item.n_seg ? __builtin_amdgcn_readlane(m_rot, e) : q_pos[e - item.n_seg];
            s_rot[e < item.n_seg ? e : e - item.n_seg + PC_ONE_SEGS][lane] = rope_small((double)pos * freq);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): the rows are in LDS (tiles may still be on their way)
        asm volatile("s_barrier" ::: "memory");
        return (const float2 *)s_rot[PC_ONE_SEGS + r];
    };
    const DecCall dc{cd.n_q, cd.q_off, cd.self_len - cd.n_q, cd.n_splits, split, cd.part_off, 1};
    decode_walk<true, ONE_WAVES>(L, dc, kh, tile, tile_stop, describe, [&](int seg) { return (const float2 *)s_rot[seg]; }, prepare, s_acc, s_m, s_l);
    if (cd.n_splits == 1) return;

    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wave's part is out
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        // (wraps to zero with the last split: ready for the next launch)
        s_last = atomicInc(&O.counters[call * L.n_kv_heads + kh], (unsigned)cd.n_splits - 1) == (unsigned)cd.n_splits - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    merge_cols(L, dc, kh);
}

void pc_launch_decode_one_bf16(const PcArgBlob &blob, size_t bytes, const PcLaunch &L, const PcOne &O, hipStream_t st)
{
    const dim3 grid((unsigned)O.n_items * L.n_kv_heads);
    auto launch = [&](auto args) {
        __builtin_memcpy(args.w, blob.w, sizeof args < bytes ? sizeof args : bytes);
        pc_decode_one_bf16_kernel<<<grid, 64 * ONE_WAVES, 0, st>>>(args, L, O);
    };
    // (three forms: the host copies all of a launch's arguments, 0.1 us of a step of 1 to 4 calls between the two sizes: passes of
    // 16 steps 131 and 134, 143 and 144, 176.5 and 178 us)
    if (O.lists) pc_decode_one_bf16_kernel<<<grid, 64 * ONE_WAVES, 0, st>>>(PcArgs<0>(), L, O);
    else if (bytes <= 768) launch(PcArgs<768>());
    else launch(PcArgs<PC_ARG_BYTES>());
}

__device__ __forceinline__ int pick(int i, int a, int b, int c, int d) { return i < 2 ? (i == 0 ? a : b) : (i == 2 ? c : d); }

// A batch of one-row decode calls by message.  Calls that list the same messages out of step (64 calls over a common system message and
// 8 of 512 others each) fetch most of them once per call when every call walks its own list, yet leave most of the 16 columns of the matrix
// instructions empty.  Here the messages are the work: every wave streams an even share of all tiles, run after run in slot order,
// and a run's columns are the heads of up to PC_RUN_ROWS calls that list the message.  A run ends in an fp32 part per (row, head), which
// the merge launch adds in slot order.  Waves are on their own: no barrier, nothing shared but the L2s.
__global__ __launch_bounds__(256, 2) void pc_decode_runs_bf16_kernel(const PcRunStarts starts, PcLaunch L, PcRuns O)
{
    // each wave's requested run: the rotations of its rows, and its columns' queries (chunk c of 16 bytes of column n at c ^ n)
    __shared__ __attribute__((aligned(1024))) float2 s_rot[4][PC_RUN_ROWS][PC_D / 2];
    __shared__ __attribute__((aligned(1024))) uint4 s_q[4][16][16];
    typedef int i32x8 __attribute__((ext_vector_type(8)));
    const int kh = blockIdx.x % L.n_kv_heads;            // consecutive workgroups (one per XCD) take different KV heads
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, a = lane >> 4;
    const int w = 4 * (blockIdx.x / L.n_kv_heads) + wave;
    if (w >= O.n_waves) return;
    const auto *firsts = (const __attribute__((address_space(4))) uint16_t *)__builtin_amdgcn_kernarg_segment_ptr();
    const int first = __builtin_amdgcn_readfirstlane(firsts[w]), end = __builtin_amdgcn_readfirstlane(firsts[w + 1]);
    if (first >= end) return;
    // column n: row n / g of the run, head n % g of the group (g is 1, 2, 4 or 8 here)
    const int g = L.n_q_heads / L.n_kv_heads, lg = __builtin_ctz(g);
    auto fresh_lane = [&]() __attribute__((always_inline)) { int l = lane; asm volatile("" : "+v"(l)); return l; };
    // (scalar loads; what is uniform over the wave is said to be, wherever the compiler cannot see it)
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    auto load_run = [&](int i) __attribute__((always_inline)) { return *reinterpret_cast<const __attribute__((address_space(4))) i32x8 *>(reinterpret_cast<uintptr_t>(O.runs + uniform(i))); };
    auto load_parts = [&](int i) __attribute__((always_inline)) { return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(&O.runs[uniform(i)].part)); };
    auto load_entry = [&](int m) __attribute__((always_inline)) { return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(O.table + uniform(m))); };

    const uint16_t *kb = (const uint16_t *)L.k_store + (int64_t)kh * L.slots * PC_D;
    const uint16_t *vb = (const uint16_t *)L.v_store + (int64_t)kh * L.slots * PC_D;
    // The requests' place: the run being requested, and the one behind it.  A tile is requested while the one before it is computed.
    int at_run = first, at_tile = 0, left = 0, slot = 0, len = 0, run_rows = 0;
    i32x8 ahead = load_run(first);
    i32x4 entry = load_entry(ahead[0]);
    int rows = 0, p0 = 0, p1 = 0, p2 = 0, p3 = 0;        // of the run being computed, and their parts
    const unsigned lds_rot = (unsigned)(size_t)&s_rot[0][0][0] + wave * (unsigned)sizeof(s_rot[0]);
    const unsigned lds_q = (unsigned)(size_t)&s_q[0][0][0] + wave * (unsigned)sizeof(s_q[0]);
    auto fetch = [&](DecTile &T) __attribute__((always_inline)) {
        T.fresh = false;
        if (left == 0 && at_run < end) {
            T.fresh = true;
            slot = uniform(entry.x); len = uniform(entry.y);
            at_tile = uniform(ahead[1]); left = uniform(ahead[2]) & 0xFFFFFFF; run_rows = uniform(ahead[2]) >> 28;
            // (the lane anew, here and below: held across the loop, addresses that follow from it cost registers that tiles in flight need)
            const int ln = fresh_lane(), r0 = uniform(ahead[4]), r1 = uniform(ahead[5]), r2 = uniform(ahead[6]), r3 = uniform(ahead[7]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {                // columns 4 i + lane / 16
                const int col = 4 * i + (ln >> 4), cr = col >> lg, c0 = cr < run_rows ? cr : 0;
                dma16(L.q, (unsigned)((pick(c0, r0, r1, r2, r3) * L.n_q_heads + kh * g + (col & (g - 1))) * (PC_D * 2) + (((ln & 15) ^ col) << 4)), lds_q + i * 1024);
            }
            const float2 *rot = O.rot + (int64_t)uniform(at_run) * PC_RUN_ROWS * (PC_D / 2);
            dma16(rot, 16 * ln, lds_rot);                // rows 0 and 1, 2 and 3
            dma16(rot + PC_D, 16 * ln, lds_rot + 1024);
            if (++at_run < end) ahead = load_run(at_run);
        }
        // (behind the wave's last tile: a line of it)
        T.there = left > 0;
        const int key0 = T.there ? at_tile * PC_TILE : 0;
        T.valid = T.there ? min(len - key0, PC_TILE) : 1;
        dec_load(T, kb, vb, slot + key0, T.valid, lane);
        ++at_tile;
        T.self = --left == 0;                            // (the run's last tile)
        left = max(left, 0);
    };
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 acc[8];
    bf16x8 qop[4];
    auto clear = [&]() __attribute__((always_inline)) {
        m_run = -INFINITY; l_run = 0.f;
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    };
    // the requested run becomes the computed one: its columns' queries turned by where their calls see them from the message, scaled
    auto begin = [&]() __attribute__((always_inline)) {
        rows = run_rows;
        const i32x4 parts = load_parts(at_run - 1);
        p0 = uniform(parts.x); p1 = uniform(parts.y); p2 = uniform(parts.z); p3 = uniform(parts.w);
        // (in LDS once all but the 16 requests of the run's first tile, which are behind them, are done)
        __builtin_amdgcn_s_waitcnt(0x4F70);              // vmcnt(16)
        asm volatile("" ::: "memory");
        const int ln = fresh_lane(), n = ln & 15, a = ln >> 4, ri = n >> lg;
        const bool ok = ri < rows;
        const float2 *rq = &s_rot[wave][ok ? ri : 0][8 * a];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint4 lo = s_q[wave][n][(4 * ks + a) ^ n], hi = s_q[wave][n][(4 * ks + a + 8) ^ n];
            const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
            uint32_t pl[4], ph[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 c0 = rq[32 * ks + 2 * j], c1 = rq[32 * ks + 2 * j + 1];
                const float x0 = bf_lo(lw[j]), x1 = bf_hi(lw[j]), y0 = bf_lo(hw[j]), y1 = bf_hi(hw[j]);
                pl[j] = ok ? pack_bf16(x0 * c0.x - y0 * c0.y, x1 * c1.x - y1 * c1.y) : 0u;
                ph[j] = ok ? pack_bf16(x0 * c0.y + y0 * c0.x, x1 * c1.y + y1 * c1.x) : 0u;
            }
            qop[ks] = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
            qop[ks + 2] = __builtin_bit_cast(bf16x8, make_uint4(ph[0], ph[1], ph[2], ph[3]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // (read before the next run's come)
        if (at_run < end) entry = load_entry(ahead[0]);
        clear();
    };
    auto compute = [&](DecTile &T) __attribute__((always_inline)) {
        f32x4 s[2];
#pragma unroll
        for (int tau = 0; tau < 2; ++tau) {
            s[tau] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                s[tau] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.k[tau][ks]), qop[ks], s[tau], 0, 0, 0);
        }
        float sc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[j] = s[j >> 2][j & 3];
        if (T.valid < PC_TILE) {                         // (one row a call, its message's last token: a row sees all there is)
#pragma unroll
            for (int j = 0; j < 8; ++j) sc[j] = (8 * a + j < T.valid) ? sc[j] : -INFINITY;
            drop_dead(T, lane);
        }
        float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
        mx = max_lanes_xor16(mx);
        mx = max_lanes_xor32(mx);
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        uint32_t pk[4];
        float ps = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {                    // (the row sum over the rounded probabilities, as in decode_walk)
            pk[j] = pack_bf16(__builtin_amdgcn_exp2f(sc[2 * j] - m_safe), __builtin_amdgcn_exp2f(sc[2 * j + 1] - m_safe));
            ps += bf_lo(pk[j]) + bf_hi(pk[j]);
        }
        l_run = l_run * alpha + ps;
        m_run = m_new;
        const bool rescale = __builtin_amdgcn_ballot_w64(alpha != 1.f) != 0;
        const bf16x8 pop = __builtin_bit_cast(bf16x8, make_uint4(pk[0], pk[1], pk[2], pk[3]));
        if (rescale) {
#pragma unroll
            for (int db = 0; db < 8; ++db) acc[db] *= alpha;
        }
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, T.v[db]), pop, acc[db], 0, 0, 0);
        if (!T.self) return;
        // the run's part
        l_run += __shfl_xor(l_run, 16);
        l_run += __shfl_xor(l_run, 32);
        const int ln = fresh_lane(), ri = (ln & 15) >> lg, rh = ln & 15 & (g - 1), a = ln >> 4;
        if (ri < rows) {
            const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
            const int part = pick(ri, p0, p1, p2, p3);
            const int h = kh * g + rh;
            f32x4 *po = reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(L.part_o) + ((int64_t)part * L.n_q_heads + h) * PC_D + 4 * a);     // dims 16 db + 4 a + 0..3
#pragma unroll
            for (int db = 0; db < 8; ++db) po[4 * db] = acc[db] * inv;
            if (a == 0) *reinterpret_cast<float2 *>(L.part_ml + (2 * (int64_t)part * L.n_q_heads + h) * 2) = make_float2(m_run, l_run);
        }
    };
    // Two tiles are in flight.  A run's queries and rotations have one place in LDS: they are requested with its first tile, which is when the
    // run before it, whose place it is, has been begun.
    DecTile A, B;
    fetch(A);
    begin();
    fetch(B);
    do {                                                 // (one way out, as in decode_walk)
        compute(A);
        if (B.fresh) begin();
        fetch(A);
        if (B.there) compute(B);
        if (A.fresh) begin();
        fetch(B);
    } while (A.there);
}

void pc_launch_decode_runs_bf16(const PcLaunch &L, const PcRuns &O, const PcRunStarts &starts, hipStream_t st)
{
    pc_decode_runs_bf16_kernel<<<(unsigned)((O.n_waves + 3) / 4 * L.n_kv_heads), 256, 0, st>>>(starts, L, O);
}

void pc_launch_decode_bf16(const PcLaunch &L, int n_items, hipStream_t st)
{
    if (n_items <= 0) return;
    dim3 grid((unsigned)n_items * L.n_kv_heads);
    pc_decode_bf16_kernel<<<grid, 256, 0, st>>>(L);
}

