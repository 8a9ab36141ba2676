// Gradient of the attention for bf16 caches on the matrix cores (gfx950), at fp32 precision.
//
// What is computed, per query row r and head, with p_j = exp(s_j - LSE) from the forward's LSE and dp_j = dO . v_j:
//   Delta = sum_j p_j dp_j,  ds_j = p_j (dp_j - Delta),  dq += scale ds_j K_j,  dK_j += scale ds_j q,  dV_j += p_j dO
// (Sec. 2.4: in fine-tuning a position update is applied without destroying the keys, so that gradients flow through
// it).  Inputs are bf16, everything between them and the fp32 gradients is fp32.
//
// fp32 from bf16 matrix instructions.  A product of two bf16 numbers is exact in fp32, so a bf16 MFMA is an fp32
// dot product of its operands, and a number of 24 significant bits is the exact sum of three bf16 pieces of 8 (round,
// subtract, round, subtract, round).  A product of an fp32 factor with a bf16 one (dq: ds K, dV: p dO, the scores of
// the row-major kernels: turned query times stored key) takes three MFMAs and is exact; two fp32 factors (dK: ds
// times turned query, and the scores of the key-major kernel) take the six whose pieces' orders sum to at most two:
// what is left out is below 2^-24 of a product, what rounding it to fp32 costs at most.  Three to six
// bf16 MFMAs run at 2.5 to 5 times the rate of the fp32 ones.
//
// Kernels, in launch order:
//   prep      per (32-row block, head): the queries turned by their positions, as fp32 in the lanes' order and as three
//             bf16 pieces, and the output gradients, rows past the call's end as zeros
//   delta     per (8 row units, KV head, split of the tiles): Delta partials        (32 MFMAs a tile and unit)
//   dq        per half of those units, the same walk with Delta known: dq partials  (56)
//   finish    sum of the dq partials, turned back by the rows' positions
//   keys      per (4 key tiles, KV head, split of the row units): dK and dV         (128)
// A unit is 32 rows of one head, a tile 32 keys.  The walks are bound by the matrix pipe (216 MFMAs of 32 cycles per
// unit and tile).  Four calls of 150 to 320 rows over about 2000 tokens each, 32/8 heads, least and mean us of a kernel trace
// of 16 passes: prep 12 / 12, delta 100 / 106, dq 181 / 189 to 199, finish 9 / 9, keys 312 / 327 (with one wave a unit or tile
// dq 201 / 209, keys 354 / 373; plain vector kernels, a thread per key and an FMA per product, took 31.4 ms).  delta: 46 us of
// it are the pipe, 9 the turns; running the vector work of one of a SIMD's two waves beside the matrix work of the other took
// 3 off.  keys: longest workgroups first, 9 us more.
//
// All operands that a product needs with its indices the other way round (V by dimension, keys, queries and output
// gradients by token) come from the same LDS tile through ds_read_b64_tr_b16: within 16 lanes, lane l points at row
// l / 4, columns 4 (l % 4) .. + 3 of a 4 x 16 block and receives column l, rows 0 .. 3.
#include "pc_pieces.h"

#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)
#define TILE_BYTES 8192

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) bf16x8 *lds_frag;
typedef __attribute__((address_space(3))) s16x4 *lds_tr;
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8 frag4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return __builtin_bit_cast(bf16x8, make_uint4(a, b, c, d)); }
__device__ __forceinline__ bf16x8 read_tr(unsigned at0, unsigned at1)       // rows 0..3 and 4..7 of the lane's column
{
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)at0);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr)(uintptr_t)at1);
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    return frag4(x.x, x.y, y.x, y.y);
}
// the largest finite numbers in the place of infinities, zeros in the place of NaN
__device__ __forceinline__ bf16x8 finite8(bf16x8 x)
{
    uint4 u = __builtin_bit_cast(uint4, x);
    uint32_t *w = reinterpret_cast<uint32_t *>(&u);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t lo = w[j] & 0x7FFFu, hi = w[j] & 0x7FFF0000u;
        w[j] = lo > 0x7F80u ? w[j] & 0xFFFF0000u : w[j] - (lo == 0x7F80u ? 1u : 0u);
        w[j] = hi > 0x7F800000u ? w[j] & 0xFFFFu : w[j] - (hi == 0x7F800000u ? 0x10000u : 0u);
    }
    return __builtin_bit_cast(bf16x8, u);
}
// The 4-byte direct load beside dma16; completion is awaited with an explicit s_waitcnt vmcnt(n).
__device__ __forceinline__ void dma4(const void *gbase_uniform, unsigned lane_off, unsigned lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 ::"s"(lds_wave_base), "v"(lane_off), "s"(gbase_uniform) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }
__device__ __forceinline__ void ring_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Swizzle of a row-major tile [32 rows][16 chunks of 16 bytes]: chunk c of row r sits at position c ^ swz(r).  The
// 16 rows of a fragment read hit different banks, and so do the 4 consecutive rows of a transposing one.
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// Fragment addresses of a row-major tile at LDS offset `tile`:
//   by row:    lane's row `row` (any), dims 16 ks + 8 hh + 0..7
//   by column: lane's dim 32 db + (lane & 31), rows 16 s + 8 hh + 0..7
struct RowMajor {
    unsigned row_at, col_at[2];
    __device__ RowMajor(int row, int lane)
    {
        const int hh = lane >> 5, nh = (lane >> 4) & 1, l = lane & 15;
        row_at = (unsigned)(row * 256 + ((hh ^ swz(row)) << 4));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int key = 8 * hh + 4 * e + (l >> 2);
            col_at[e] = (unsigned)(key * 256 + (((2 * nh + ((l & 3) >> 1)) ^ swz(key)) << 4) + (l & 1) * 8);
        }
    }
    __device__ bf16x8 by_row(unsigned tile, int ks) const { return *(lds_frag)(uintptr_t)((row_at ^ (ks << 5)) + tile); }
    __device__ bf16x8 by_col(unsigned tile, int s, int db) const
    {
        return read_tr((col_at[0] ^ (db << 6)) + tile + s * 4096, (col_at[1] ^ (db << 6)) + tile + s * 4096);
    }
    // the same with the addresses of a tile made once: `at` the tile's position behind them, a constant
    struct Cols { unsigned base[4][2]; };
    __device__ Cols cols(unsigned tile) const
    {
        Cols c;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                c.base[db][e] = (col_at[e] ^ (db << 6)) + tile;
                asm volatile("" : "+v"(c.base[db][e]));  // (or every read gets an addition of its own)
            }
        return c;
    }
    static __device__ bf16x8 by_col(const Cols &c, unsigned at, int s, int db) { return read_tr(c.base[db][0] + (at + s * 4096), c.base[db][1] + (at + s * 4096)); }
};
// the row of the first product's left operand this lane reads: rows are permuted so that result registers 0..7 / 8..15
// of a lane are rows 8 hh + 0..7 / 16 + 8 hh + 0..7, the order in which the second product takes them
__device__ __forceinline__ int perm_row(int n) { return 16 * (n >> 4) + 8 * ((n >> 2) & 1) + 4 * ((n >> 3) & 1) + (n & 3); }

// Values by key from a tile in the V store's order, [4 groups][128 dims][8 keys], chunk (group, dim) at position
// 128 group + (dim ^ 4 (group & 1)): lane's key, dims 16 ks + 8 hh + 0..7.  PERM: the lane's key is perm_row(lane & 31).
template <bool PERM>
struct ValuesByKey {
    unsigned at[2];
    __device__ ValuesByKey(int lane)
    {
        const int hh = lane >> 5, nh = (lane >> 4) & 1, l = lane & 15, c4 = l & 3;
        const int grp = 2 * nh + (PERM ? (c4 & 1) : (c4 >> 1)), half = PERM ? (c4 >> 1) : (c4 & 1);
#pragma unroll
        for (int e = 0; e < 2; ++e) at[e] = (unsigned)((grp * 128 + 8 * hh + 4 * (e ^ (grp & 1)) + (l >> 2)) * 16 + half * 8);
    }
    __device__ bf16x8 get(unsigned tile, int ks) const { return read_tr(at[0] + tile + ks * 256, at[1] + tile + ks * 256); }
};
__device__ __forceinline__ int v_src_chunk(int pos) { return (pos & ~127) | ((pos & 127) ^ (4 * ((pos >> 7) & 1))); }   // what belongs at a position

__device__ __forceinline__ i32x4 scalar16(const void *p)                    // (wave-uniform address)
{
    return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(p));
}

}  // namespace

// ----------------------------------------------------------------------------------------------------------- prep
// A thread takes eight low dims of a row and their partners 64 up.
__global__ __launch_bounds__(256) void pc_bwd_prep_kernel(PcLaunch L, PcBwd B)
{
    const int rbl = blockIdx.x, h = blockIdx.y;
    const int2 rb = B.row_blocks[B.rb0 + rbl];
    const PcCallDesc cd = L.calls[rb.x];
    const int r = threadIdx.x >> 3, c = threadIdx.x & 7;
    const int row = 32 * rb.y + r;
    const int64_t unit = (int64_t)rbl * L.n_q_heads + h;
    float x[8], y[8];
    uint4 glo = make_uint4(0, 0, 0, 0), ghi = glo;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = y[j] = 0.f;
    // (a row that saw nothing, or a score that is not a number, has no gradient: it is taken as zeros)
    if (row < cd.n_q && B.lse[(int64_t)(cd.q_off + row) * L.n_q_heads + h] > -INFINITY) {
        const int64_t R = cd.q_off + row, at = (R * L.n_q_heads + h) * PC_D + 8 * c;
        const uint4 lo = ldg16((const uint16_t *)L.q + at), hi = ldg16((const uint16_t *)L.q + at + 64);
        glo = ldg16(B.d_out + at); ghi = ldg16(B.d_out + at + 64);
        const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
        const float4 *rot = reinterpret_cast<const float4 *>(L.rot_q + R * (PC_D / 2) + 8 * c);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4 cs = rot[u];
            const float a0 = bf_lo(lw[u]), a1 = bf_hi(lw[u]), b0 = bf_lo(hw[u]), b1 = bf_hi(hw[u]);
            x[2 * u] = a0 * cs.x - b0 * cs.y; y[2 * u] = a0 * cs.y + b0 * cs.x;
            x[2 * u + 1] = a1 * cs.z - b1 * cs.w; y[2 * u + 1] = a1 * cs.w + b1 * cs.z;
        }
    }
    float4 *qt = B.q_turned + unit * 1024 + (c >> 1) * 256 + (c & 1) * 32 + r;
    qt[0] = make_float4(x[0], x[1], x[2], x[3]); qt[64] = make_float4(x[4], x[5], x[6], x[7]);
    qt[128] = make_float4(y[0], y[1], y[2], y[3]); qt[192] = make_float4(y[4], y[5], y[6], y[7]);
    const Pieces px = split8<false>(x), py = split8<false>(y);
    unsigned char *dst = (unsigned char *)B.q_pieces + unit * (4 * TILE_BYTES) + r * 256 + c * 16;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        *reinterpret_cast<bf16x8 *>(dst + i * TILE_BYTES) = px.p[i];
        *reinterpret_cast<bf16x8 *>(dst + i * TILE_BYTES + 128) = py.p[i];
    }
    *reinterpret_cast<uint4 *>(dst + 3 * TILE_BYTES) = glo;
    *reinterpret_cast<uint4 *>(dst + 3 * TILE_BYTES + 128) = ghi;
}

// ----------------------------------------------------------------------------------------------- row-major kernels
// Delta.  A workgroup is 8 waves = 8 consecutive units (heads of a KV head fastest), which share the staged K and V tiles: a
// ring of four, requested three tiles ahead by direct loads, one barrier a tile.  S^T = K Q^T and dP^T = V dO^T leave a
// row's values in one lane column.  The turned queries (three pieces) live in registers and are made anew from the fp32 copy
// at every segment; the output gradients are read from LDS, which is what keeps the kernel at two waves per SIMD.
__global__ __launch_bounds__(512, 1) void pc_bwd_delta_kernel(PcLaunch L, PcBwd B)
{
    constexpr int RING = 4, AHEAD = 3;
    __shared__ __attribute__((aligned(1024))) unsigned char s_k[RING][TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char s_v[RING][TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char s_g[8][TILE_BYTES];       // output gradients of the 8 units

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const PcItem item = L.items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_units = ((cd.n_q + 31) >> 5) * g;
    const bool unit_ok = item.unit0 + wave < n_units;
    const int unit = unit_ok ? item.unit0 + wave : item.unit0;
    const int ub = unit / g, h = kh * g + (unit - ub * g);
    const int row = 32 * ub + n;
    const bool row_ok = unit_ok && row < cd.n_q;
    const int self_lim = cd.self_len - cd.n_q + row;     // last own token this row sees
    const int blk_lim_lo = cd.self_len - cd.n_q + 32 * ub;
    const int64_t U = (int64_t)(cd.rb_off + ub - B.rb0) * L.n_q_heads + h;

    // the row's scalars; rows that saw nothing or do not exist get a log-sum-exp of +inf, which makes their p zero
    float lse2 = INFINITY;
    if (row_ok) {
        const float v = B.lse[(int64_t)(cd.q_off + row) * L.n_q_heads + h];
        if (v > -INFINITY) lse2 = v * 1.4426950408889634f;
    }

    const bool some_dead = __builtin_amdgcn_ballot_w64(row_ok && lse2 == INFINITY) != 0;
    const RowMajor rk(perm_row(n), lane), rg(n, lane);
    const ValuesByKey<true> rv(lane);
    const unsigned lds_k = (unsigned)(uintptr_t)&s_k[0][0], lds_v = (unsigned)(uintptr_t)&s_v[0][0], lds_g = (unsigned)(uintptr_t)&s_g[0][0] + wave * TILE_BYTES;
    const unsigned k_src = (threadIdx.x >> 4) * 256 + (((threadIdx.x & 15) ^ swz(threadIdx.x >> 4)) << 4);
    const unsigned v_src = (unsigned)v_src_chunk(threadIdx.x) * 16;
    const unsigned char *kb = (const unsigned char *)L.k_store + (int64_t)kh * L.slots * PC_D * 2;
    const unsigned char *vb = (const unsigned char *)L.v_store + (int64_t)kh * L.slots * PC_D * 2;
    const PcTile *tab = L.tiles + item.tile_tab0;
    const int last = item.tile_end - 1;
    auto describe = [&](int t) { return scalar16(tab + __builtin_amdgcn_readfirstlane(min(t, last))); };   // {slot0, key0, seg, valid | flags}
    auto request = [&](const i32x4 &d, int slot) {
        const int64_t at = (int64_t)__builtin_amdgcn_readfirstlane(d.x) * 256;
        dma16(kb + at, k_src, lds_k + slot * TILE_BYTES + wave * 1024);
        dma16(vb + at, v_src, lds_v + slot * TILE_BYTES + wave * 1024);
    };

    bf16x8 qp[3][8];
    auto turn = [&](int seg) __attribute__((always_inline)) {       // the unit's queries turned by -(start - base) of a segment
        const float4 *qt = B.q_turned + U * 1024 + hh * 32 + n;
        const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + seg) * (PC_D / 2) + 8 * hh);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const float4 xa = qt[ks * 256], xb = qt[ks * 256 + 64], ya = qt[ks * 256 + 128], yb = qt[ks * 256 + 192];
            const float x[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w}, y[8] = {ya.x, ya.y, ya.z, ya.w, yb.x, yb.y, yb.z, yb.w};
            float u[8], v[8];
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const float4 cs = rs[8 * ks + (j >> 1)];
                u[j] = x[j] * cs.x + y[j] * cs.y; v[j] = y[j] * cs.x - x[j] * cs.y;
                u[j + 1] = x[j + 1] * cs.z + y[j + 1] * cs.w; v[j + 1] = y[j + 1] * cs.z - x[j + 1] * cs.w;
            }
            const Pieces pu = split8<false>(u), pv = split8<false>(v);
#pragma unroll
            for (int i = 0; i < 3; ++i) { qp[i][ks] = pu.p[i]; qp[i][ks + 4] = pv.p[i]; }
        }
    };
    float dsum = 0.f;
    const int t0 = item.tile_begin, t1 = item.tile_end;
    if (t0 < t1) {
        {   // the unit's output gradients: 4 rows per instruction, whole lines
            const unsigned char *src = (const unsigned char *)B.q_pieces + __builtin_amdgcn_readfirstlane((int)U) * (int64_t)(4 * TILE_BYTES) + 3 * TILE_BYTES;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 4 * i + (lane >> 4);
                dma16(src, (unsigned)(r * 256 + (((lane & 15) ^ swz(r)) << 4)), lds_g + i * 1024);
            }
        }
        i32x4 d[AHEAD + 1];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) { d[i] = describe(t0 + i); request(d[i], i); }
        int cur = -1;
        for (int t = t0; t < t1; ++t) {
            const int slot = (t - t0) & (RING - 1);
            wait_vm<2 * (AHEAD - 1)>();                  // this wave's share of tile t has landed (and everything older)
            ring_barrier();                              // ... every wave's has, and tile t - 1 is no longer read
            const int seg = __builtin_amdgcn_readfirstlane(d[0].z), flags = __builtin_amdgcn_readfirstlane(d[0].w), key0 = __builtin_amdgcn_readfirstlane(d[0].y);
            if (cur < 0 || (flags & PC_TILE_FRESH)) {
                if (unit_ok) turn(seg);
                cur = seg;
            }
            d[AHEAD] = describe(t + AHEAD);
            request(d[AHEAD], (slot + AHEAD) & (RING - 1));
            if (unit_ok) {
                const unsigned kt = lds_k + slot * TILE_BYTES, vt = lds_v + slot * TILE_BYTES;
                f32x16 s, dp;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 k = rk.by_row(kt, ks);
                    s = MFMA32(k, qp[2][ks], s);
                    s = MFMA32(k, qp[1][ks], s);
                    s = MFMA32(k, qp[0][ks], s);
                }
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) dp = MFMA32(rv.get(vt, ks), rg.by_row(lds_g, ks), dp);
                const int valid = flags & 0xFF;
                const bool self = (flags & PC_TILE_SELF) != 0;
                float w[16];                             // p dp
#pragma unroll
                for (int r = 0; r < 16; ++r)             // (the maximum: an infinite key times a piece that is 0 is a NaN, see the key-major kernel)
                    w[r] = ex2(fmaxf(__builtin_fmaf(s[r], L.scale_log2, -lse2), -1e30f)) * dp[r];
                // (masked behind the product: the value of a token behind the row's own is the caller's and need not be finite)
                if (valid < PC_TILE || some_dead || (self && key0 + PC_TILE - 1 > blk_lim_lo)) {      // ragged or causal tile (uniform)
                    const int lim = lse2 == INFINITY ? 0 : self ? min(valid, self_lim - key0 + 1) : valid;
#pragma unroll
                    for (int r = 0; r < 16; ++r) w[r] = (16 * (r >> 3) + 8 * hh + (r & 7) < lim) ? w[r] : 0.f;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) dsum += w[r];
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) d[i] = d[i + 1];
        }
        wait_vm<0>();
    }
    dsum += __shfl_xor(dsum, 32);
    if (unit_ok && hh == 0) B.delta_part[((int64_t)item.split * B.n_units + U) * 32 + n] = dsum;
}

// dq, with Delta known.  Two waves a unit, on the same SIMD: the first holds the unit's turned queries and output gradients and
// makes ds = p (dp - Delta), which it leaves in LDS in fp32; the second follows one tile behind and adds dq^T = K^T dS^T, collected
// in the frame of the segment's keys and turned into the rows' frame whenever the rotation changes, by adding to the unit's
// fp32 partial in memory.  (With one wave a unit, eight units a workgroup, both waves of a SIMD did their matrix work and then
// their vector work at the same time, and all waited while any of them turned its queries or its sums: 201 us at
// least, now 181, for the batch above.)  A workgroup takes half of an item's eight units; ring of four tiles: the one of the
// second waves, that of the first, two on their way.  All 256 registers are in use, 4 of the wave's values are spilled (20 bytes).
__global__ __launch_bounds__(512, 2) void pc_bwd_dq_kernel(PcLaunch L, PcBwd B)
{
    constexpr int RING = 4, AHEAD = 2, W_BYTES = 4096;
    __shared__ __attribute__((aligned(1024))) unsigned char s_k[RING][TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char s_v[RING][TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char s_w[2][4][W_BYTES];       // ds of two tiles: float4 j of lane l at 1024 j + 16 l

    const int kh = blockIdx.x % L.n_kv_heads;
    const int idx = blockIdx.x / L.n_kv_heads;
    const PcItem item = L.items[idx >> 1];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int pair = wave & 3, unit0 = item.unit0 + 4 * (idx & 1);
    const bool is_dq = wave >= 4;                        // the second wave of the unit
    const int n_units = ((cd.n_q + 31) >> 5) * g;
    if (unit0 >= n_units) return;                        // (the whole workgroup)
    const bool unit_ok = unit0 + pair < n_units;
    const int unit = unit_ok ? unit0 + pair : unit0;
    const int ub = unit / g, h = kh * g + (unit - ub * g);
    const int64_t U = (int64_t)(cd.rb_off + ub - B.rb0) * L.n_q_heads + h;

    const RowMajor rk(perm_row(n), lane);
    const unsigned lds_k = (unsigned)(uintptr_t)&s_k[0][0], lds_v = (unsigned)(uintptr_t)&s_v[0][0];
    const unsigned k_src = (threadIdx.x >> 4) * 256 + (((threadIdx.x & 15) ^ swz(threadIdx.x >> 4)) << 4);
    const unsigned v_src = (unsigned)v_src_chunk(threadIdx.x) * 16;
    const unsigned char *kb = (const unsigned char *)L.k_store + (int64_t)kh * L.slots * PC_D * 2;
    const unsigned char *vb = (const unsigned char *)L.v_store + (int64_t)kh * L.slots * PC_D * 2;
    const PcTile *tab = L.tiles + item.tile_tab0;
    const int t0 = item.tile_begin, t1 = item.tile_end, last = t1 - 1;
    float4 *part = B.dq_part + ((int64_t)item.split * B.n_units + U) * 1024 + lane;
    if (t0 >= t1) {                                      // nothing to see: a partial of zeros, and the row's scalars
        if (is_dq && unit_ok)
#pragma unroll
            for (int i = 0; i < 16; ++i) part[64 * i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    auto describe = [&](int t) { return scalar16(tab + __builtin_amdgcn_readfirstlane(min(t, last))); };   // {slot0, key0, seg, valid | flags}
    auto request = [&](const i32x4 &d, int slot) {
        const int64_t at = (int64_t)__builtin_amdgcn_readfirstlane(d.x) * 256;
        dma16(kb + at, k_src, lds_k + slot * TILE_BYTES + wave * 1024);
        dma16(vb + at, v_src, lds_v + slot * TILE_BYTES + wave * 1024);
    };
    i32x4 d[AHEAD + 1];
    if (t0 < t1)
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) { d[i] = describe(t0 + i); request(d[i], i); }
    // tile t, of the first waves: it and its successor have landed (so that fragments can be read a tile ahead), the second waves
    // have its predecessor's ds, and nobody reads the one before that, whose slot the next request takes
    auto next_tile = [&](int t) {
        __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0), lgkmcnt(0)
        ring_barrier();
        if (t < t1 && (__builtin_amdgcn_readfirstlane(d[0].w) & PC_TILE_SELF)) {
            // A tile of the new message (uniform over the workgroup): a zero takes a key that stands behind a row's own
            // token out of dq only while it is finite, which the caller's tokens need not be.  (A row that sees such a
            // key has no gradient, or, where its score is -inf, a probability of 0: a score of -1e38 gives the same.)
            uint4 *chunk = reinterpret_cast<uint4 *>(&s_k[(t - t0) & (RING - 1)][0]) + threadIdx.x;
            const bf16x8 raw = __builtin_bit_cast(bf16x8, *chunk);
            *chunk = __builtin_bit_cast(uint4, finite8(raw));
            __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0)
            ring_barrier();
        }
        d[AHEAD] = describe(t + AHEAD);
        request(d[AHEAD], (t - t0 + AHEAD) & (RING - 1));
    };

    if (!is_dq) {
        const int row = 32 * ub + n;
        const bool row_ok = unit_ok && row < cd.n_q;
        const int self_lim = cd.self_len - cd.n_q + row; // last own token this row sees
        const int blk_lim_lo = cd.self_len - cd.n_q + 32 * ub;
        // the row's scalars; rows that saw nothing or do not exist get a log-sum-exp of +inf, which makes their p zero
        float lse2 = INFINITY, delta = 0.f;
        if (row_ok) {
            const float v = B.lse[(int64_t)(cd.q_off + row) * L.n_q_heads + h];
            if (v > -INFINITY) lse2 = v * 1.4426950408889634f;
            for (int s = 0; s < cd.n_splits; ++s) delta += B.delta_part[((int64_t)s * B.n_units + U) * 32 + n];
        }
        if (unit_ok && item.split == 0 && hh == 0) B.stat[U * 32 + n] = make_float2(lse2, delta);
        if (t0 >= t1) return;
        const bool some_dead = __builtin_amdgcn_ballot_w64(row_ok && lse2 == INFINITY) != 0;
        const ValuesByKey<true> rv(lane);
        bf16x8 go[8];                                    // the unit's output gradients: the lane's row, dims 16 ks + 8 hh + 0..7
        {
            const unsigned char *src = (const unsigned char *)B.q_pieces + U * (4 * TILE_BYTES) + 3 * TILE_BYTES + n * 256 + hh * 16;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) go[ks] = __builtin_bit_cast(bf16x8, ldg16(src + 32 * ks));
        }
        bf16x8 qp[3][8];
        auto turn = [&](int seg) __attribute__((always_inline)) {       // the unit's queries turned by -(start - base) of a segment
            const float4 *qt = B.q_turned + U * 1024 + hh * 32 + n;
            const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + seg) * (PC_D / 2) + 8 * hh);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const float4 xa = qt[ks * 256], xb = qt[ks * 256 + 64], ya = qt[ks * 256 + 128], yb = qt[ks * 256 + 192];
                const float x[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w}, y[8] = {ya.x, ya.y, ya.z, ya.w, yb.x, yb.y, yb.z, yb.w};
                float u[8], v[8];
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const float4 cs = rs[8 * ks + (j >> 1)];
                    u[j] = x[j] * cs.x + y[j] * cs.y; v[j] = y[j] * cs.x - x[j] * cs.y;
                    u[j + 1] = x[j + 1] * cs.z + y[j + 1] * cs.w; v[j + 1] = y[j + 1] * cs.z - x[j + 1] * cs.w;
                }
                const Pieces pu = split8<false>(u), pv = split8<false>(v);
#pragma unroll
                for (int i = 0; i < 3; ++i) { qp[i][ks] = pu.p[i]; qp[i][ks + 4] = pv.p[i]; }
            }
        };
        int cur = -1;
        bf16x8 kf[8];                                    // the tile's keys, read while its predecessor is worked on
        for (int t = t0; t < t1; ++t) {
            next_tile(t);
            const int slot = (t - t0) & (RING - 1);
            const int seg = __builtin_amdgcn_readfirstlane(d[0].z), flags = __builtin_amdgcn_readfirstlane(d[0].w), key0 = __builtin_amdgcn_readfirstlane(d[0].y);
            if (cur < 0 || (flags & PC_TILE_FRESH)) {
                if (unit_ok) turn(seg);
                cur = seg;
            }
            if (unit_ok) {
                const unsigned kt = lds_k + slot * TILE_BYTES, vt = lds_v + slot * TILE_BYTES, kn = lds_k + ((slot + 1) & (RING - 1)) * TILE_BYTES;
                if (t == t0 || (flags & PC_TILE_SELF))   // (a tile of the new message was made finite since)
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) kf[ks] = rk.by_row(kt, ks);
                f32x16 s, dp;
                bf16x8 vf[4];
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    s = MFMA32(kf[ks], qp[2][ks], s);
                    s = MFMA32(kf[ks], qp[1][ks], s);
                    s = MFMA32(kf[ks], qp[0][ks], s);
                    if (ks >= 4) vf[ks - 4] = rv.get(vt, ks - 4);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    dp = MFMA32(vf[ks & 3], go[ks], dp);
                    if (ks < 4) vf[ks] = rv.get(vt, ks + 4);
                    kf[ks] = rk.by_row(kn, ks);          // (behind the last tile: what the ring holds there, which is not used)
                    __builtin_amdgcn_sched_barrier(0);
                }
                const int valid = flags & 0xFF;
                const bool self = (flags & PC_TILE_SELF) != 0;
                float w[16];                             // p (dp - Delta)
#pragma unroll
                for (int r = 0; r < 16; ++r)             // (the maximum: an infinite key times a piece that is 0 is a NaN, see the key-major kernel)
                    w[r] = ex2(fmaxf(__builtin_fmaf(s[r], L.scale_log2, -lse2), -1e30f)) * (dp[r] - delta);
                // (masked behind the product: the value of a token behind the row's own is the caller's and need not be finite)
                if (valid < PC_TILE || some_dead || (self && key0 + PC_TILE - 1 > blk_lim_lo)) {      // ragged or causal tile (uniform)
                    const int lim = lse2 == INFINITY ? 0 : self ? min(valid, self_lim - key0 + 1) : valid;
#pragma unroll
                    for (int r = 0; r < 16; ++r) w[r] = (16 * (r >> 3) + 8 * hh + (r & 7) < lim) ? w[r] : 0.f;
                }
                float4 *out = reinterpret_cast<float4 *>(&s_w[(t - t0) & 1][pair][0]) + lane;
#pragma unroll
                for (int j = 0; j < 4; ++j) out[64 * j] = make_float4(w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]);
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) d[i] = d[i + 1];
        }
        next_tile(t1);                                   // (the second waves' last tile)
        wait_vm<0>();
        return;
    }
    if (t0 >= t1) return;
    f32x16 acc[4];
    bool first = true;                                   // nothing written to the unit's dq partial yet
    auto clear = [&]() {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    };
    // dq of the segment, turned by +(start - base), into the partial: float4 (db, q4) of a lane is dims 32 db + 8 q4 + 4 hh + 0..3
    auto flush = [&](int seg) __attribute__((always_inline)) {
        const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + seg) * (PC_D / 2) + 4 * hh);
        // (all of the old partial is requested before any of the new one is stored: a store in between would make each
        // load wait for the one before it, eight round trips to memory instead of one)
        float4 old[16];
        if (!first)
#pragma unroll
            for (int i = 0; i < 16; ++i) old[i] = part[i * 64];
        else
#pragma unroll
            for (int i = 0; i < 16; ++i) old[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float4 c0 = rs[16 * db + 4 * q4], c1 = rs[16 * db + 4 * q4 + 1];
                const float cx[4] = {c0.x, c0.z, c1.x, c1.z}, sx[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = acc[db][4 * q4 + i] * B.scale, b = acc[db + 2][4 * q4 + i] * B.scale;
                    float *ol = reinterpret_cast<float *>(&old[db * 4 + q4]), *oh = reinterpret_cast<float *>(&old[db * 4 + q4 + 8]);
                    ol[i] += a * cx[i] - b * sx[i]; oh[i] += a * sx[i] + b * cx[i];
                }
            }
#pragma unroll
        for (int i = 0; i < 16; ++i) part[i * 64] = old[i];
        first = false;
    };
    clear();
    int cur = -1;
    next_tile(t0);                                       // (the first waves' first tile)
    bf16x8 kf[2][4];
    auto read_keys = [&](int t) {
        const unsigned kt = lds_k + ((t - t0) & (RING - 1)) * TILE_BYTES;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int db = 0; db < 4; ++db) kf[st][db] = rk.by_col(kt, st, db);
    };
    read_keys(t0);
    for (int t = t0; t < t1; ++t) {
        const int seg = __builtin_amdgcn_readfirstlane(d[0].z), flags = __builtin_amdgcn_readfirstlane(d[0].w);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) d[i] = d[i + 1];
        next_tile(t + 1);
        if (!unit_ok) continue;
        if (cur < 0 || (flags & PC_TILE_FRESH)) {
            if (cur >= 0) { flush(cur); clear(); }
            cur = seg;
        }
        const float4 *in = reinterpret_cast<const float4 *>(&s_w[(t - t0) & 1][pair][0]) + lane;
        float w[16];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 x = in[64 * j];
            w[4 * j] = x.x; w[4 * j + 1] = x.y; w[4 * j + 2] = x.z; w[4 * j + 3] = x.w;
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const Pieces ds = split8<false>(w + 8 * st);
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                acc[db] = MFMA32(kf[st][db], ds.p[2], acc[db]);
                acc[db] = MFMA32(kf[st][db], ds.p[1], acc[db]);
                acc[db] = MFMA32(kf[st][db], ds.p[0], acc[db]);
            }
        }
        read_keys(t + 1);                                // (behind the last tile: not used)
    }
    wait_vm<0>();
    if (unit_ok) flush(cur);
}

// dq: the splits' partials summed in order and turned back by the row's own position
__global__ __launch_bounds__(256) void pc_bwd_finish_kernel(PcLaunch L, PcBwd B)
{
    __shared__ float s_o[32][PC_D + 4];
    const int rbl = blockIdx.x, h = blockIdx.y;
    const int2 rb = B.row_blocks[B.rb0 + rbl];
    const PcCallDesc cd = L.calls[rb.x];
    const int64_t U = (int64_t)rbl * L.n_q_heads + h;
    const int lane = threadIdx.x & 63, n = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = (threadIdx.x >> 6) + 4 * i;        // (db, q4) of the lower half
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        for (int s = 0; s < cd.n_splits; ++s) {
            const float4 *p = B.dq_part + ((int64_t)s * B.n_units + U) * 1024 + lane;
            const float4 u = p[k * 64], v = p[(k + 8) * 64];
            a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
            b.x += v.x; b.y += v.y; b.z += v.z; b.w += v.w;
        }
        const int d = 32 * (k >> 2) + 8 * (k & 3) + 4 * hh;
        *reinterpret_cast<float4 *>(&s_o[n][d]) = a;
        *reinterpret_cast<float4 *>(&s_o[n][d + 64]) = b;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {                        // 16 threads per row: 4 dims and their partners
        const int r = (threadIdx.x >> 4) + 16 * i, c = threadIdx.x & 15;
        const int row = 32 * rb.y + r;
        if (row >= cd.n_q) continue;
        const int64_t R = cd.q_off + row;
        float4 a = *reinterpret_cast<const float4 *>(&s_o[r][4 * c]), b = *reinterpret_cast<const float4 *>(&s_o[r][4 * c + 64]);
        if (!(B.stat[U * 32 + r].x < INFINITY)) a = b = make_float4(0.f, 0.f, 0.f, 0.f);       // the row saw nothing
        const float4 *rot = reinterpret_cast<const float4 *>(L.rot_q + R * (PC_D / 2) + 4 * c);
        const float4 c0 = rot[0], c1 = rot[1];
        float *out = B.d_q + (R * L.n_q_heads + h) * PC_D + 4 * c;
        *reinterpret_cast<float4 *>(out) = make_float4(a.x * c0.x + b.x * c0.y, a.y * c0.z + b.y * c0.w, a.z * c1.x + b.z * c1.y, a.w * c1.z + b.w * c1.w);
        *reinterpret_cast<float4 *>(out + 64) = make_float4(b.x * c0.x - a.x * c0.y, b.y * c0.z - a.y * c0.w, b.z * c1.x - a.z * c1.y, b.w * c1.z - a.w * c1.w);
    }
}

// ----------------------------------------------------------------------------------------------------- key-major
// A workgroup takes four 32-key tiles of the call (each one placement of a message), with two waves a tile that sit on the
// same SIMD: the first holds the tile's keys turned to the call's positions (three pieces) and the sums of dV, and makes the
// probabilities, which it leaves in LDS in fp32; the second holds the values and the sums of dK and follows one unit behind.  The
// units of this KV head go by, staged through LDS in a ring of three (queries in three pieces, output gradients, row
// scalars: 32 KB a unit).  Keys, values and both sums fill 256 registers: with one wave a tile, one a SIMD, all of that wave's
// vector work and every wait for LDS stood in its matrix work's way (3.9 us a unit, 128 MFMAs of 32 cycles = 1.8; with two waves
// a tile 3.1, which is 1.4 PFLOP/s of the 1.73 that a bare MFMA loop reaches on such operands).  Here the keys are turned, not the queries: the waves of a workgroup hold tiles of different messages, and the
// staged queries then serve all of them.  At the end dK is turned back to the stored frame and both sums meet those of the
// tokens' other placements (other calls, repeated listings, other splits of the units) through one fp32 atomic per
// element, whole cache lines at a time.
__global__ __launch_bounds__(512, 2) void pc_bwd_keys_kernel(PcLaunch L, PcBwd B)
{
    constexpr int RING = 3, STAGE = 4 * TILE_BYTES, P_BYTES = 4096, TURN = 32 * (PC_D + 4) * 4;
    constexpr int MEM = RING * STAGE + 2 * 4 * P_BYTES > 8 * TURN ? RING * STAGE + 2 * 4 * P_BYTES : 8 * TURN;
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[MEM];   // ring, probabilities of two units; at the end the sums being turned round
    __shared__ __attribute__((aligned(256))) float2 s_stat[RING][32];

    const int kh = blockIdx.x % L.n_kv_heads;
    const PcBwdKeyItem item = B.key_items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int tile = wave & 3;
    const bool is_dk = wave >= 4;                        // the second wave of the tile
    const bool active = tile < item.n_tiles;
    const i32x4 d = scalar16(L.tiles + cd.tile_off + item.tile0 + (active ? tile : 0));
    const int slot0 = __builtin_amdgcn_readfirstlane(d.x), key0 = __builtin_amdgcn_readfirstlane(d.y);
    const int seg = __builtin_amdgcn_readfirstlane(d.z), flags = __builtin_amdgcn_readfirstlane(d.w);
    const bool self = (flags & PC_TILE_SELF) != 0;
    const int tok0 = cd.self_len - cd.n_q;

    const unsigned lds_q = (unsigned)(uintptr_t)&s_mem[0], lds_stat = (unsigned)(uintptr_t)&s_stat[0][0];
    const unsigned q_src = (unsigned)((threadIdx.x >> 4) * 256 + (((threadIdx.x & 15) ^ swz(threadIdx.x >> 4)) << 4));
    const int64_t u_base = (int64_t)(cd.rb_off - B.rb0) * L.n_q_heads + kh * g;
    int req_rt = item.rt_begin, req_rb = item.rt_begin / g, req_h = item.rt_begin - req_rb * g, req_slot = 0;
    auto request = [&]() {                               // the next unit, if there is one
        if (req_rt >= item.rt_end) return;
        const int64_t u = u_base + (int64_t)req_rb * L.n_q_heads + req_h;
        ++req_rt;
        if (++req_h == g) { req_h = 0; ++req_rb; }
        const unsigned char *src = (const unsigned char *)B.q_pieces + u * STAGE;
#pragma unroll
        for (int i = 0; i < 4; ++i) dma16(src + i * TILE_BYTES, q_src, lds_q + req_slot * STAGE + i * TILE_BYTES + wave * 1024);
        if (wave == 0) dma4(B.stat + u * 32, lane * 4, lds_stat + req_slot * 256);
        req_slot = req_slot + 1 == RING ? 0 : req_slot + 1;
    };
    // the values, through the ring's last slot
    if (is_dk) {
        const unsigned char *vb = (const unsigned char *)L.v_store + ((int64_t)kh * L.slots + slot0) * PC_D * 2;
        const unsigned at = lds_q + (RING - 1) * STAGE + tile * TILE_BYTES;
#pragma unroll
        for (int i = 0; i < 8; ++i) dma16(vb, (unsigned)v_src_chunk(64 * i + lane) * 16, at + i * 1024);
    }
    request();
    const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + seg) * (PC_D / 2));
    const RowMajor rq(perm_row(n), lane);
    f32x16 sum[4];                                       // dV, or dK
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[db][r] = 0.f;
    // the probabilities of a unit: float4 j of lane l at 1024 j + 16 l
    float4 *const s_p = reinterpret_cast<float4 *>(&s_mem[RING * STAGE + tile * P_BYTES]) + lane;
    uint64_t odd = 0;                                    // second wave: keys whose values are not finite
    // A unit's turn: every wave's share of it has landed, the probabilities of the unit before are written, and the slot of the
    // one before that, which the next request takes, is no longer read.
    auto next_unit = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0), lgkmcnt(0)
        ring_barrier();
        request();
    };
    int rb = item.rt_begin / g, left = (rb + 1) * g - item.rt_begin, slot = 0, odd_unit = 0;      // row block, its units still to come, ring slot

    if (!is_dk) {
        // the keys turned by +(start - base): lane = key, dims 16 ks + 8 hh + 0..7
        bf16x8 kp[3][8];
        {
            const uint16_t *kr = (const uint16_t *)L.k_store + ((int64_t)kh * L.slots + slot0 + n) * PC_D + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const uint4 lo = ldg16(kr + 16 * ks), hi = ldg16(kr + 16 * ks + 64);
                const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
                float x[8], y[8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 cs = rs[8 * ks + 4 * hh + u];
                    const float a0 = bf_lo(lw[u]), a1 = bf_hi(lw[u]), b0 = bf_lo(hw[u]), b1 = bf_hi(hw[u]);
                    x[2 * u] = a0 * cs.x - b0 * cs.y; y[2 * u] = a0 * cs.y + b0 * cs.x;
                    x[2 * u + 1] = a1 * cs.z - b1 * cs.w; y[2 * u + 1] = a1 * cs.w + b1 * cs.z;
                }
                const Pieces px = split8<false>(x), py = split8<false>(y);
#pragma unroll
                for (int i = 0; i < 3; ++i) { kp[i][ks] = px.p[i]; kp[i][ks + 4] = py.p[i]; }
            }
        }
        for (int rt = item.rt_begin; rt < item.rt_end; ++rt) {
            next_unit();
            const int row0 = tok0 + 32 * rb;             // own token of the block's first row
            const unsigned qt = lds_q + slot * STAGE;
            const float4 *st = reinterpret_cast<const float4 *>(&s_stat[slot][8 * hh]);
            float4 *const pw = s_p + odd_unit * (4 * P_BYTES / 16);
            if (--left == 0) { ++rb; left = g; }
            slot = slot + 1 == RING ? 0 : slot + 1;
            odd_unit ^= 1;
            if (!active || (self && key0 > row0 + 31)) continue;        // (uniform over the wave: no row of the block sees the tile)
            const int lim = self && key0 + PC_TILE - 1 > row0 ? key0 + n - row0 : -1;      // the first row that sees the lane's key
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const bf16x8 a0 = rq.by_row(qt, ks), a1 = rq.by_row(qt + TILE_BYTES, ks), a2 = rq.by_row(qt + 2 * TILE_BYTES, ks);
                s = MFMA32(a2, kp[0][ks], s);
                s = MFMA32(a1, kp[1][ks], s);
                s = MFMA32(a0, kp[2][ks], s);
                s = MFMA32(a1, kp[0][ks], s);
                s = MFMA32(a0, kp[1][ks], s);
                s = MFMA32(a0, kp[0][ks], s);
            }
            // register r: row 16 (r / 8) + 8 hh + r % 8 of the block
            float p[16];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float4 x = st[(r >> 3) * 8 + ((r & 7) >> 1)];
                // (The maximum takes a NaN to a probability of 0.  A row that saw a NaN or +inf has no gradient, see prep; where a row
                // that has one meets an infinite key its score is -inf, which the pieces' products turn into NaN.)
                p[r] = ex2(fmaxf(__builtin_fmaf(s[r], L.scale_log2, -x.x), -1e30f));
                p[r + 1] = ex2(fmaxf(__builtin_fmaf(s[r + 1], L.scale_log2, -x.z), -1e30f));
            }
            // (no branch for the few causal tiles: it would cut the block the scheduler mixes matrix and vector work in)
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = (16 * (r >> 3) + 8 * hh + (r & 7) >= lim) ? p[r] : 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) pw[j * 64] = make_float4(p[4 * j], p[4 * j + 1], p[4 * j + 2], p[4 * j + 3]);
            const RowMajor::Cols qc = rq.cols(qt);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const Pieces pp = split8<false>(p + 8 * half);
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    const bf16x8 a = RowMajor::by_col(qc, 3 * TILE_BYTES, half, db);
                    sum[db] = MFMA32(a, pp.p[2], sum[db]);
                    sum[db] = MFMA32(a, pp.p[1], sum[db]);
                    sum[db] = MFMA32(a, pp.p[0], sum[db]);
                }
            }
        }
        next_unit();                                     // (the second waves' last unit)
    } else {
        bf16x8 vf[8];
        wait_vm<0>();                                    // (each brought its own tile's)
        {
            const ValuesByKey<false> rv(lane);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) vf[ks] = rv.get(lds_q + (RING - 1) * STAGE + tile * TILE_BYTES, ks);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(vf[ks]));    // (read before the slot is requested again)
        }
        // A value that is not finite makes dp a NaN for every row of a block, and no zero takes the rows without a gradient out of
        // dK again (a select per probability would: 24 us of 740 for a training step).  It is taken as zeros here, and its key's
        // dK is a NaN at the end if a row with a gradient sees it.
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const uint4 u = __builtin_bit_cast(uint4, vf[ks]);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 4; ++j) bad |= (w[j] & 0x7F80u) == 0x7F80u || (w[j] & 0x7F800000u) == 0x7F800000u;
            odd |= __builtin_amdgcn_ballot_w64(bad);
            if (bad) vf[ks] = frag4(0, 0, 0, 0);
        }
        next_unit();                                     // (the first waves' first unit)
        for (int rt = item.rt_begin; rt < item.rt_end; ++rt) {
            next_unit();
            const int row0 = tok0 + 32 * rb;
            const unsigned qt = lds_q + slot * STAGE;
            const float4 *st = reinterpret_cast<const float4 *>(&s_stat[slot][8 * hh]);
            const float4 *const pr = s_p + odd_unit * (4 * P_BYTES / 16);
            if (--left == 0) { ++rb; left = g; }
            slot = slot + 1 == RING ? 0 : slot + 1;
            odd_unit ^= 1;
            if (!active || (self && key0 > row0 + 31)) continue;
            f32x16 dp;
#pragma unroll
            for (int r = 0; r < 16; ++r) dp[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) dp = MFMA32(rq.by_row(qt + 3 * TILE_BYTES, ks), vf[ks], dp);
            float w[16];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float4 x = st[(r >> 3) * 8 + ((r & 7) >> 1)];
                w[r] = dp[r] - x.y;
                w[r + 1] = dp[r + 1] - x.w;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 p = pr[j * 64];
                w[4 * j] *= p.x; w[4 * j + 1] *= p.y; w[4 * j + 2] *= p.z; w[4 * j + 3] *= p.w;
            }
            const RowMajor::Cols qc = rq.cols(qt);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const Pieces ds = split8<false>(w + 8 * half);
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    const bf16x8 a0 = RowMajor::by_col(qc, 0, half, db), a1 = RowMajor::by_col(qc, TILE_BYTES, half, db), a2 = RowMajor::by_col(qc, 2 * TILE_BYTES, half, db);
                    sum[db] = MFMA32(a2, ds.p[0], sum[db]);
                    sum[db] = MFMA32(a1, ds.p[1], sum[db]);
                    sum[db] = MFMA32(a0, ds.p[2], sum[db]);
                    sum[db] = MFMA32(a1, ds.p[0], sum[db]);
                    sum[db] = MFMA32(a0, ds.p[1], sum[db]);
                    sum[db] = MFMA32(a0, ds.p[0], sum[db]);
                }
            }
        }
    }
    ring_barrier();                                      // the ring is free: each wave turns its sums round in 17 KB of it
    if (!active) return;
    if (odd != 0) {
        bool hit = false;
        for (int rt = item.rt_begin; rt < item.rt_end; ++rt) {
            const int b = rt / g;
            const float2 *stat = B.stat + (u_base + (int64_t)b * L.n_q_heads + (rt - b * g)) * 32;
            for (int r = 0; r < 32; ++r) hit |= stat[r].x < INFINITY && (!self || key0 + n <= tok0 + 32 * b + r);
        }
        if (hit && (((odd | odd >> 32) >> n) & 1) != 0)
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[db][r] = __builtin_nanf("");
    }
    float *stg = reinterpret_cast<float *>(&s_mem[wave * TURN]);
    const int valid = flags & 0xFF;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int dim = 32 * db + 8 * q4 + 4 * hh;
            float lo[4], hi[4];
            if (is_dk) {                                 // dK back to the stored frame
                const float4 c0 = rs[dim >> 1], c1 = rs[(dim >> 1) + 1];
                const float cx[4] = {c0.x, c0.z, c1.x, c1.z}, sx[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = sum[db][4 * q4 + i] * B.scale, b = sum[db + 2][4 * q4 + i] * B.scale;
                    lo[i] = a * cx[i] + b * sx[i]; hi[i] = b * cx[i] - a * sx[i];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) { lo[i] = sum[db][4 * q4 + i]; hi[i] = sum[db + 2][4 * q4 + i]; }
            }
            *reinterpret_cast<float4 *>(stg + n * (PC_D + 4) + dim) = make_float4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<float4 *>(stg + n * (PC_D + 4) + dim + 64) = make_float4(hi[0], hi[1], hi[2], hi[3]);
        }
    // (a wave's own LDS writes and reads are ordered; the other waves use other parts)
    float *out = (is_dk ? B.d_k : B.d_v) + ((int64_t)slot0 * L.n_kv_heads + kh) * PC_D + lane;
    for (int k = 0; k < valid; ++k) {
        const int64_t at = (int64_t)k * L.n_kv_heads * PC_D;
        unsafeAtomicAdd(out + at, stg[k * (PC_D + 4) + lane]);
        unsafeAtomicAdd(out + at + 64, stg[k * (PC_D + 4) + lane + 64]);
    }
}

void pc_launch_attend_bwd_bf16(const PcLaunch &L, const PcBwd &B, int n_items, int n_key_items, hipStream_t st)
{
    if (B.n_rb <= 0) return;
    const dim3 blocks((unsigned)B.n_rb, (unsigned)L.n_q_heads);
    pc_bwd_prep_kernel<<<blocks, 256, 0, st>>>(L, B);
    const unsigned rows = (unsigned)n_items * L.n_kv_heads;
    pc_bwd_delta_kernel<<<rows, 512, 0, st>>>(L, B);
    pc_bwd_dq_kernel<<<2 * rows, 512, 0, st>>>(L, B);
    pc_bwd_finish_kernel<<<blocks, 256, 0, st>>>(L, B);
    if (n_key_items > 0) pc_bwd_keys_kernel<<<(unsigned)n_key_items * L.n_kv_heads, 512, 0, st>>>(L, B);
}
