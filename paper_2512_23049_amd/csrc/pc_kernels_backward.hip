// Gradient of the attention for fp32 caches on the fp32 matrix instructions (gfx950), and the finalize pass of both cache
// types (bf16 caches: pc_kernels_bwd_mfma.hip).
//
// Per query row r and head, with p_j = exp(s_j - LSE) from the forward's LSE and dp_j = dO . v_j:
//   Delta = sum_j p_j dp_j,  ds_j = p_j (dp_j - Delta),  dq += scale ds_j K_j,  dK_j += scale ds_j q,  dV_j += p_j dO
// (Sec. 2.4: in fine-tuning a position update is applied non-destructively, so gradients flow through it to the cached
// keys.)  Products and sums are fp32 throughout: v_mfma_f32_32x32x2_f32, whose operands a lane holds one float of (row or
// column lane % 32, index lane / 32 of two) and whose result has 16 rows a lane, 8 (r / 4) + 4 (lane / 32) + r % 4.  The
// order of the summed index is free, so register r of a product is the operand of the next one for the two indices it
// stands for, and the other operand is read in 16-byte pieces, whichever way round it is needed.
//
// Two kernels.  rows: 32 (row, head) columns of a KV head against the call's tiles, twice: Delta, then dq.  keys: a wave
// owns one 32-key tile of the call, its keys turned to the call's positions, and the sums of dK and dV, while the call's
// column blocks go by.  A row that saw nothing has no gradient: its queries and output gradients are taken as zeros.
// Bound: the matrix rate, 576 MFMAs of 64 cycles per 32 x 32 block at D = 128 (half at D = 64).  Two calls of 50 to 110
// rows over 550 keys, 8/2 heads, D = 64: rows 52, keys 29 us; 212 and 390 us with a wave per (row, head) and a thread per
// quarter key, an FMA per product.  That size is bound by latency: 44 workgroups of rows, three tiles a wave.
#include "pc_mfma_common.h"

#define MFMA_F32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0)

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int W> struct Vec;                             // W consecutive floats of a row
template <> struct Vec<2> { using type = float2; };
template <> struct Vec<4> { using type = float4; };

// two pairs (a, b) turned by (cos, sin) c.x, c.y and c.z, c.w, forwards or back
__device__ __forceinline__ void turn2(float &a0, float &b0, float &a1, float &b1, float4 c)
{
    const float x0 = a0 * c.x - b0 * c.y, y0 = a0 * c.y + b0 * c.x, x1 = a1 * c.z - b1 * c.w, y1 = a1 * c.w + b1 * c.z;
    a0 = x0; b0 = y0; a1 = x1; b1 = y1;
}
__device__ __forceinline__ float4 conj2(float4 c) { return make_float4(c.x, -c.y, c.z, -c.w); }
__device__ __forceinline__ void turn4(float4 &a, float4 &b, float4 c0, float4 c1)
{
    turn2(a.x, b.x, a.y, b.y, c0);
    turn2(a.z, b.z, a.w, b.w, c1);
}
__device__ __forceinline__ i32x4 tile_at(const PcTile *tab, int t)
{
    return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(tab + __builtin_amdgcn_readfirstlane(t)));
}

}  // namespace

// ------------------------------------------------------------------------------------------------------------ rows
// A workgroup is 8 waves, two per SIMD, over the same 32 columns; each walks a contiguous eighth of the item's tiles.  The
// queries are turned to a segment's frame at every new rotation, made anew from memory; dq is collected in that frame and
// turned back into the wave's own part of LDS.  The waves' parts are added in order.
#define NW 8
template <int D>
__global__ __launch_bounds__(64 * NW, 1) void pc_bwd_rows_f32_kernel(PcLaunch L, const float *__restrict__ lse, const float *__restrict__ d_out,
                                                                     float scale, float *__restrict__ d_q, float *__restrict__ delta_out)
{
    constexpr int NJ = D / 8, VW = D / 32, HALF = D / 2, PITCH = D + 4;
    __shared__ __attribute__((aligned(16))) float s_dq[NW][32 * PITCH];
    __shared__ __attribute__((aligned(16))) float s_g[32 * PITCH];          // the columns' output gradients
    __shared__ float s_delta[NW][32];
    using VV = typename Vec<VW>::type;

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const PcItem item = L.items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_cols = cd.n_q * g, col0 = item.unit0 * 32;                  // column c: query row c / g, head c % g of the group
    const int per_wave = (item.tile_end - item.tile_begin + NW - 1) / NW;
    const int t0 = item.tile_begin + wave * per_wave, t1 = min(item.tile_end, t0 + per_wave);
    const PcTile *tab = L.tiles + item.tile_tab0;

    auto row_head = [&](int col) { return (int64_t)(cd.q_off + col / g) * L.n_q_heads + kh * g + col % g; };
    auto alive = [&](int col) { return col < n_cols && lse[row_head(col)] > -INFINITY; };
    for (int e = threadIdx.x; e < 32 * (D / 4); e += 64 * NW) {
        const int c = e / (D / 4), i = 4 * (e % (D / 4));
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (alive(col0 + c)) {
            const float *p = d_out + row_head(col0 + c) * D + i;
            x = make_float4(p[0], p[1], p[2], p[3]);
        }
        *reinterpret_cast<float4 *>(s_g + c * PITCH + i) = x;
    }
    const bool live = alive(col0 + n);
    const int64_t rh = row_head(live ? col0 + n : col0);
    const float row_lse = live ? lse[rh] : 0.f;
    const int row = (col0 + n) / g;
    const int self_lim = cd.self_len - cd.n_q + row;     // last own token this column sees
    const int lo_lim = cd.self_len - cd.n_q + col0 / g;  // ... the item's first column
    const float *qrow = (const float *)L.q + rh * D + 4 * hh;
    const float4 *rq = reinterpret_cast<const float4 *>(L.rot_q + (live ? (int64_t)(cd.q_off + row) : (int64_t)cd.q_off) * HALF) + 2 * hh;
    const float *kb = (const float *)L.k_store + (int64_t)kh * L.slots * D, *vb = (const float *)L.v_store + (int64_t)kh * L.slots * D;
    __syncthreads();

    float4 q[NJ];
    auto turn = [&](int seg) __attribute__((always_inline)) {               // queries turned by their position less (start - stored base)
        const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + seg) * HALF) + 2 * hh;
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
            if (live) {
                const float *p = qrow + 8 * j;
                a = make_float4(p[0], p[1], p[2], p[3]);
                b = make_float4(p[HALF], p[HALF + 1], p[HALF + 2], p[HALF + 3]);
            }
            turn4(a, b, rq[4 * j], rq[4 * j + 1]);
            turn4(a, b, conj2(rs[4 * j]), conj2(rs[4 * j + 1]));
            q[j] = a; q[j + NJ / 2] = b;
        }
    };
    // the product of a tile's rows (K or V by key) with the columns' operand, in two chains
    auto by_key = [&](const float *tile, auto operand) __attribute__((always_inline)) {
        const float *p = tile + n * D + 4 * hh;
        float4 x[2][4];
        auto load = [&](int c) {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[c & 1][j] = *reinterpret_cast<const float4 *>(p + 8 * (4 * c + j));
        };
        f32x16 s0, s1;
#pragma unroll
        for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
        load(0); load(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NJ / 4; ++c) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x16 &s = (j & 1) ? s1 : s0;
                const float4 a = x[c & 1][j], b = operand(4 * c + j);
                s = MFMA_F32(a.x, b.x, s);
                s = MFMA_F32(a.y, b.y, s);
                s = MFMA_F32(a.z, b.z, s);
                s = MFMA_F32(a.w, b.w, s);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (c + 2 < NJ / 4) load(c + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        return s0 + s1;
    };
    bool causal = false;
    int lim = 0;
    auto scores = [&](const i32x4 &d, f32x16 &p, f32x16 &dp) __attribute__((always_inline)) {
        p = by_key(kb + (int64_t)d.x * D, [&](int j) { return q[j]; });
        const int valid = d.w & 0xFF, key0 = d.y;
        const bool self = (d.w & PC_TILE_SELF) != 0;
        causal = self && key0 + valid - 1 > lo_lim;      // some column does not see some key
        lim = self ? min(valid, self_lim - key0 + 1) : valid;
        if (!live) lim = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = expf(fmaf(p[r], scale, -row_lse));
        dp = by_key(vb + (int64_t)d.x * D, [&](int j) { return *reinterpret_cast<const float4 *>(s_g + n * PITCH + 8 * j + 4 * hh); });
    };
    auto seen = [&](int r) { return 8 * (r >> 2) + 4 * hh + (r & 3) < lim; };

    float delta = 0.f;
    int cur = -1;
    for (int t = t0; t < t1; ++t) {
        const i32x4 d = tile_at(tab, t);
        if (cur < 0 || (d.w & PC_TILE_FRESH)) { cur = d.z; turn(cur); }
        f32x16 p, dp;
        scores(d, p, dp);
#pragma unroll
        for (int r = 0; r < 16; ++r) delta += seen(r) ? p[r] * dp[r] : 0.f;
    }
    delta += __shfl_xor(delta, 32);
    if (hh == 0) s_delta[wave][n] = delta;
    __syncthreads();
    delta = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) delta += s_delta[w][n];
    if (wave == 0 && hh == 0 && col0 + n < n_cols) delta_out[row_head(col0 + n)] = live ? delta : 0.f;

    f32x16 acc[VW];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < VW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    };
    bool first = true;
    // dq of a segment, turned by +(start - base), into the wave's part of LDS: element (i, r) is dim VW (8 (r / 4) + 4 hh + r % 4) + i
    auto flush = [&](int seg) __attribute__((always_inline)) {
        const float2 *rs = L.rot_seg + (int64_t)(cd.seg_off + seg) * HALF;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int dim = VW * (8 * (r >> 2) + 4 * hh + (r & 3));
            float lo[VW], hi[VW];
#pragma unroll
            for (int i = 0; i < VW; i += 2) {
                lo[i] = acc[i][r]; lo[i + 1] = acc[i + 1][r]; hi[i] = acc[i][r + 8]; hi[i + 1] = acc[i + 1][r + 8];
                turn2(lo[i], hi[i], lo[i + 1], hi[i + 1], *reinterpret_cast<const float4 *>(rs + dim + i));
            }
            float *pl = &s_dq[wave][n * PITCH + dim], *ph = pl + HALF;
#pragma unroll
            for (int i = 0; i < VW; ++i) {
                pl[i] = first ? lo[i] : pl[i] + lo[i];
                ph[i] = first ? hi[i] : ph[i] + hi[i];
            }
        }
        first = false;
    };
    clear();
    cur = -1;
    for (int t = t0; t < t1; ++t) {
        const i32x4 d = tile_at(tab, t);
        if (cur < 0 || (d.w & PC_TILE_FRESH)) {
            if (cur >= 0) { flush(cur); clear(); }
            cur = d.z;
            turn(cur);
        }
        f32x16 p, dp;
        scores(d, p, dp);
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = seen(r) ? p[r] * (dp[r] - delta) * scale : 0.f;
        constexpr int VP = 16 / VW;                      // keys (registers of the scores) of a piece of K
        VV x[2][VP];
        const float *kr = kb + ((int64_t)d.x + 4 * hh) * D + VW * n;        // register r: key 8 (r / 4) + 4 hh + r % 4
        auto load = [&](int c) {
#pragma unroll
            for (int i = 0; i < VP; ++i) { const int r = VP * c + i; x[c & 1][i] = *reinterpret_cast<const VV *>(kr + (8 * (r >> 2) + (r & 3)) * D); }
        };
        load(0); load(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 16 / VP; ++c) {
            float k[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) k[e] = reinterpret_cast<const float *>(&x[c & 1][0])[e];
            if (causal)                                  // a zero takes a later token of the caller's out of the sum only while it is finite
#pragma unroll
                for (int e = 0; e < 16; ++e) k[e] = fabsf(k[e]) < INFINITY ? k[e] : 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e % VW] = MFMA_F32(k[e], p[VP * c + e / VW], acc[e % VW]);
            __builtin_amdgcn_sched_barrier(0);
            if ((c + 2) * VP < 16) load(c + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (cur >= 0) flush(cur);
    __syncthreads();
    const int n_waves = min(NW, per_wave > 0 ? (item.tile_end - item.tile_begin + per_wave - 1) / per_wave : 0);        // those that had tiles
    for (int e = threadIdx.x; e < 32 * (D / 8); e += 64 * NW) {             // 4 pairs of a column a step
        const int c = e / (D / 8), i = 4 * (e % (D / 8)), col = col0 + c;
        if (col >= n_cols) break;                        // (columns ascend with e)
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        if (alive(col)) {
            for (int w = 0; w < n_waves; ++w) {
                const float4 x = *reinterpret_cast<const float4 *>(&s_dq[w][c * PITCH + i]), y = *reinterpret_cast<const float4 *>(&s_dq[w][c * PITCH + i + HALF]);
                a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
                b.x += y.x; b.y += y.y; b.z += y.z; b.w += y.w;
            }
            const float4 *rot = reinterpret_cast<const float4 *>(L.rot_q + (int64_t)(cd.q_off + col / g) * HALF + i);
            turn4(a, b, conj2(rot[0]), conj2(rot[1]));   // back through the row's own position
        }
        float *o = d_q + row_head(col) * D + i;
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
        o[HALF] = b.x; o[HALF + 1] = b.y; o[HALF + 2] = b.z; o[HALF + 3] = b.w;
    }
}

// ------------------------------------------------------------------------------------------------------------ keys
// A workgroup is 4 waves, one per SIMD with all of its 512 registers.  The column blocks (queries turned by their
// positions, output gradients, row scalars) are made in LDS by all of it, the next block's loads in flight under the
// present one's products.  The sums meet those of the tokens' other placements (other calls, repeated listings, other
// splits of the blocks) through one fp32 atomic per element, whole cache lines at a time.
template <int D>
__global__ __launch_bounds__(256, 1) void pc_bwd_keys_f32_kernel(PcLaunch L, const PcBwdKeyItem *__restrict__ items, const float *__restrict__ lse,
                                                                 const float *__restrict__ d_out, const float *__restrict__ delta, float scale,
                                                                 float *__restrict__ d_k, float *__restrict__ d_v)
{
    constexpr int NJ = D / 8, VW = D / 32, HALF = D / 2, PITCH = D + 4, NP = HALF / 32;       // NP: float4 of pairs a thread stages
    __shared__ __attribute__((aligned(16))) float s_blk[2][2][32 * PITCH];  // [buffer][queries, output gradients]
    __shared__ __attribute__((aligned(16))) float s_lse[2][32], s_del[2][32];
    __shared__ __attribute__((aligned(16))) int s_lim[2][32];
    using VV = typename Vec<VW>::type;

    const int kh = blockIdx.x % L.n_kv_heads;
    const PcBwdKeyItem item = items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_cols = cd.n_q * g;
    const bool active = wave < item.n_tiles;
    const i32x4 d = tile_at(L.tiles + cd.tile_off, item.tile0 + (active ? wave : 0));
    const int slot0 = d.x, key0 = d.y, valid = d.w & 0xFF;
    const bool self = (d.w & PC_TILE_SELF) != 0;

    // staging: thread = (column, NP pieces of 4 pairs)
    const int sc = threadIdx.x >> 3, sp = 4 * (threadIdx.x & 7);
    float4 qa[NP], qb[NP], ga[NP], gb[NP], ra[NP], rb[NP];
    float st_lse = INFINITY, st_del = 0.f;
    auto fetch = [&](int u) {
        const int col = 32 * u + sc;
        st_lse = INFINITY; st_del = 0.f;                 // no such column, or a row that saw nothing: p = 0
#pragma unroll
        for (int i = 0; i < NP; ++i) qa[i] = qb[i] = ga[i] = gb[i] = ra[i] = rb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (u >= item.rt_end || col >= n_cols) return;
        const int64_t R = cd.q_off + col / g, rh = R * L.n_q_heads + kh * g + col % g;
        const float x = lse[rh];
        if (!(x > -INFINITY)) return;
        st_lse = x; st_del = delta[rh];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float *q = (const float *)L.q + rh * D + sp + 32 * i, *o = d_out + rh * D + sp + 32 * i;
            const float4 *rot = reinterpret_cast<const float4 *>(L.rot_q + R * HALF + sp + 32 * i);
            qa[i] = make_float4(q[0], q[1], q[2], q[3]); qb[i] = make_float4(q[HALF], q[HALF + 1], q[HALF + 2], q[HALF + 3]);
            ga[i] = make_float4(o[0], o[1], o[2], o[3]); gb[i] = make_float4(o[HALF], o[HALF + 1], o[HALF + 2], o[HALF + 3]);
            ra[i] = rot[0]; rb[i] = rot[1];
        }
    };
    auto put = [&](int u, int buf) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            turn4(qa[i], qb[i], ra[i], rb[i]);
            float *q = &s_blk[buf][0][sc * PITCH + sp + 32 * i], *o = &s_blk[buf][1][sc * PITCH + sp + 32 * i];
            *reinterpret_cast<float4 *>(q) = qa[i]; *reinterpret_cast<float4 *>(q + HALF) = qb[i];
            *reinterpret_cast<float4 *>(o) = ga[i]; *reinterpret_cast<float4 *>(o + HALF) = gb[i];
        }
        if (sp == 0) { s_lse[buf][sc] = st_lse; s_del[buf][sc] = st_del; s_lim[buf][sc] = cd.self_len - cd.n_q + (32 * u + sc) / g; }
    };
    fetch(item.rt_begin);

    // the wave's keys turned by +(start - base) and its values: lane = key, dims 8 j + 4 hh + 0..3
    float4 k[NJ], v[NJ];
    const float2 *rs = L.rot_seg + (int64_t)(cd.seg_off + d.z) * HALF;
    {
        const float *kr = (const float *)L.k_store + ((int64_t)kh * L.slots + slot0 + n) * D + 4 * hh;
        const float *vr = (const float *)L.v_store + ((int64_t)kh * L.slots + slot0 + n) * D + 4 * hh;
#pragma unroll
        for (int j = 0; j < NJ; ++j) { k[j] = *reinterpret_cast<const float4 *>(kr + 8 * j); v[j] = *reinterpret_cast<const float4 *>(vr + 8 * j); }
#pragma unroll
        for (int j = 0; j < NJ / 2; ++j) {
            const float4 *c = reinterpret_cast<const float4 *>(rs + 8 * j + 4 * hh);
            turn4(k[j], k[j + NJ / 2], c[0], c[1]);
        }
    }
    f32x16 dk[VW], dv[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) dk[i][r] = dv[i][r] = 0.f;
    put(item.rt_begin, 0);
    __syncthreads();

    for (int u = item.rt_begin; u < item.rt_end; ++u) {
        const int buf = (u - item.rt_begin) & 1;
        fetch(u + 1);
        const int first_lim = s_lim[buf][0], last_lim = s_lim[buf][31];
        if (active && !(self && key0 > last_lim)) {      // (uniform over the wave: some row of the block sees the tile)
            const float *bq = s_blk[buf][0], *bg = s_blk[buf][1];
            auto rows = [&](const float *b, const float4 *o) __attribute__((always_inline)) {
                f32x16 s0, s1;
#pragma unroll
                for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const float4 a = *reinterpret_cast<const float4 *>(b + n * PITCH + 8 * j + 4 * hh);
                    f32x16 &s = (j & 1) ? s1 : s0;
                    s = MFMA_F32(a.x, o[j].x, s);
                    s = MFMA_F32(a.y, o[j].y, s);
                    s = MFMA_F32(a.z, o[j].z, s);
                    s = MFMA_F32(a.w, o[j].w, s);
                }
                return s0 + s1;
            };
            f32x16 p = rows(bq, k);                      // register r: column 8 (r / 4) + 4 hh + r % 4 of the block
            f32x16 w = rows(bg, v);
            const bool causal = self && key0 + PC_TILE - 1 > first_lim;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = 8 * (r >> 2) + 4 * hh + (r & 3);
                // (the maximum: the components of an infinite key are turned into NaN; a row with a log-sum-exp saw it at a score of -inf)
                const float x = expf(fmaxf(fmaf(p[r], scale, -s_lse[buf][c]), -1e30f));
                const bool ok = s_lse[buf][c] < INFINITY && (!causal || key0 + n <= s_lim[buf][c]);
                p[r] = ok ? x : 0.f;
                w[r] = ok ? x * (w[r] - s_del[buf][c]) * scale : 0.f;
            }
            auto cols = [&](const float *b, const f32x16 &o, f32x16 *acc) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const VV a = *reinterpret_cast<const VV *>(b + (8 * (r >> 2) + 4 * hh + (r & 3)) * PITCH + VW * n);
                    const float *x = reinterpret_cast<const float *>(&a);
#pragma unroll
                    for (int i = 0; i < VW; ++i) acc[i] = MFMA_F32(x[i], o[r], acc[i]);
                }
            };
            cols(bg, p, dv);
            cols(bq, w, dk);
        }
        if (u + 1 < item.rt_end) put(u + 1, buf ^ 1);    // (last read before the barrier behind the block before this one)
        __syncthreads();
    }
    if (!active) return;
    // element (i, r) is dim VW (8 (r / 4) + 4 hh + r % 4) + i of key n: turned round through the wave's quarter of the block buffers
    float *stg = &s_blk[0][0][0] + wave * 32 * PITCH;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int dim = VW * (8 * (r >> 2) + 4 * hh + (r & 3));
            float lo[VW], hi[VW];
#pragma unroll
            for (int i = 0; i < VW; i += 2) {
                const f32x16 *a = which == 0 ? dk : dv;
                lo[i] = a[i][r]; lo[i + 1] = a[i + 1][r]; hi[i] = a[i][r + 8]; hi[i + 1] = a[i + 1][r + 8];
                if (which == 0) turn2(lo[i], hi[i], lo[i + 1], hi[i + 1], conj2(*reinterpret_cast<const float4 *>(rs + dim + i)));    // back to the stored frame
            }
#pragma unroll
            for (int i = 0; i < VW; ++i) { stg[n * PITCH + dim + i] = lo[i]; stg[n * PITCH + dim + HALF + i] = hi[i]; }
        }
        // (a wave's own LDS writes and reads are ordered; the other waves use other parts)
        float *out = (which == 0 ? d_k : d_v) + ((int64_t)slot0 * L.n_kv_heads + kh) * D + lane;
        for (int key = 0; key < valid; ++key)
#pragma unroll
            for (int i = 0; i < D; i += 64) unsafeAtomicAdd(out + (int64_t)key * L.n_kv_heads * D + i, stg[key * PITCH + lane + i]);
    }
}

void pc_launch_attend_bwd_f32(const PcLaunch &L, int n_items, const PcBwdKeyItem *key_items, int n_key_items, int D, const float *lse,
                              const float *d_out, float scale, float *delta, float *d_q, float *d_k, float *d_v, hipStream_t st)
{
    if (n_items <= 0) return;
    const unsigned rows = (unsigned)n_items * L.n_kv_heads, keys = (unsigned)n_key_items * L.n_kv_heads;
    if (D == 64) {
        pc_bwd_rows_f32_kernel<64><<<rows, 64 * NW, 0, st>>>(L, lse, d_out, scale, d_q, delta);
        if (keys > 0) pc_bwd_keys_f32_kernel<64><<<keys, 256, 0, st>>>(L, key_items, lse, d_out, delta, scale, d_k, d_v);
    } else {
        pc_bwd_rows_f32_kernel<128><<<rows, 64 * NW, 0, st>>>(L, lse, d_out, scale, d_q, delta);
        if (keys > 0) pc_bwd_keys_f32_kernel<128><<<keys, 256, 0, st>>>(L, key_items, lse, d_out, delta, scale, d_k, d_v);
    }
}

// d_k holds the gradient with respect to the stored keys K~_t = R(base + t) k_t; the gradient with
// respect to k_t is R(base + t)^T of it (Sec. 2.4 "Position Updates", transposed).  blockIdx.y names the message; a thread
// takes one rotation pair of a token and turns it for every KV head: the fp64 sincos is what the kernel spends its time on
// (one per head and pair, as before, took 55 us for 5500 tokens x 8 heads; now 12).
__global__ __launch_bounds__(256) void pc_grad_keys_finalize_kernel(const PcMsgEntry *__restrict__ msgs, int n_kv_heads, int D,
                                                                    const double *__restrict__ inv_freq, float *__restrict__ d_k)
{
    const PcMsgEntry m = msgs[blockIdx.y];
    const int half = D / 2;
    const int64_t n = (int64_t)m.len * half;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * 256) {
        const int i = (int)(idx % half), t = (int)(idx / half);
        float *row = d_k + (int64_t)(m.slot_start + t) * n_kv_heads * D + i;
        double sn, cs;
        sincos((double)(m.base_pos + t) * inv_freq[i], &sn, &cs);
        const float c = (float)cs, z = (float)sn;
#pragma unroll 4
        for (int kh = 0; kh < n_kv_heads; ++kh, row += D) {
            const float a = row[0], b = row[half];
            row[0] = a * c + b * z;
            row[half] = -a * z + b * c;
        }
    }
}

void pc_launch_grad_keys_finalize(const PcMsgEntry *msgs, int n_msgs, int n_kv_heads, int D, const double *inv_freq,
                                  float *d_k, hipStream_t st)
{
    for (int first = 0; first < n_msgs; first += 65535) {              // grid.y is limited to 65535
        const int n = n_msgs - first < 65535 ? n_msgs - first : 65535;
        dim3 grid(64, (unsigned)n);                      // 256 tokens of 64 pairs a step
        pc_grad_keys_finalize_kernel<<<grid, 256, 0, st>>>(msgs + first, n_kv_heads, D, inv_freq, d_k);
    }
}
