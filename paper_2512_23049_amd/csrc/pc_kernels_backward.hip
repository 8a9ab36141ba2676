// Gradient of the attention for fp32 caches on the bf16 matrix instructions (gfx950), at fp32 precision, and the finalize pass of both cache
// types (bf16 caches: pc_kernels_bwd_mfma.hip).
//
// Per query row r and head, with p_j = exp(s_j - LSE) from the forward's LSE and dp_j = dO . v_j:
//   Delta = sum_j p_j dp_j,  ds_j = p_j (dp_j - Delta),  dq += scale ds_j K_j,  dK_j += scale ds_j q,  dV_j += p_j dO
// (Sec. 2.4: in fine-tuning a position update is applied non-destructively, so gradients flow through it to the cached
// keys.)  Products and sums are fp32 throughout, on the bf16 matrix instructions: an fp32 number is the exact sum of three bf16
// pieces, and six MFMAs over them are an fp32 product (see pc_pieces.h).  A result has 16 rows a lane, 8 (r / 4) + 4 (lane / 32) +
// r % 4; the order of the summed index is free, so registers 8 kk .. 8 kk + 7 of a product, cut, are the operand of the next one
// for the indices they stand for, as long as the other operand is read in that order.  Queries, keys, values and output gradients are
// cut times UP = 2^16, so that the smallest numbers have their pieces; scores and dp carry it twice, sums of ds K and ds q three times, those of
// p dO twice (p is cut times UP as well), and powers of two take it back exactly.  (Values or output gradients of 1e-34 without it: dK 6e-5 to 9e-5
// from fp64, dq 8e-6; of 1e-36 with it 2.2e-7 to 2.9e-7.)  A sum that overflows for it, or meets an Inf or NaN, is made again on the fp32 instruction.
//
// Two kernels.  rows: 32 (row, head) columns of a KV head against the call's tiles: Delta and dq.  keys: a wave owns one 32-key tile of
// the call, its keys turned to the call's positions, and the sums of dK and dV, while the call's column blocks go by.  A
// row that saw nothing has no gradient: its queries and output gradients are taken as zeros.  Two calls of 82 and 109 rows over
// 600 keys, 8/2 heads, D = 64: rows 26, keys 22 us, with the fp32 instruction 52 and 28, with a wave per (row, head) and a thread per
// quarter key 212 and 390; one call of 15 rows over 90 keys, 8/2 heads, D = 128: 17.5 and 19 (25.7 and 33).  Such sizes are
// bound by latency: 50 workgroups of rows, three tiles a wave.  Distances to fp64 in the 2-norm over 14 batches: dq 3.1e-7 to
// 4.5e-7, dK 3.3e-7 to 4.4e-7, dV 2.9e-7 to 4.1e-7 (3.7e-7 to 4.7e-7, 3.7e-7 to 4.6e-7, 3.4e-7 to 4.3e-7 with the fp32 instruction); dq
// 1.8e-7 to 3.9e-7 over 67 others since its sums are centred and a tile's product is added to them.
#include "pc_pieces.h"

#include <cstring>
#include <type_traits>

#define MFMA_F32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0)

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int W> struct Vec;                             // W consecutive floats of a row
template <> struct Vec<1> { using type = float; };
template <> struct Vec<2> { using type = f32x2; };
template <> struct Vec<4> { using type = f32x4; };

// e^x as 2^(h + l): h the product with log2 e, l what rounding it leaves out, so that the result is off by what x is off by
__device__ __forceinline__ float exp_x(float x)
{
    const float h = x * 1.4426950408889634f, l = fmaf(x, 1.4426950408889634f, -h) + x * 1.9259629911266175e-8f;
    const float e = __builtin_amdgcn_exp2f(h);
    return fmaf(e, l * 0.6931471805599453f, e);
}
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
// A workgroup is one wave a SIMD (D = 128: all of its 512 registers) or two over the same 32 columns, whose queries (turned by their positions) and output
// gradients lie in LDS as pieces; each wave walks a contiguous part of the item's tiles, once: its keys are turned to the call's
// positions, and with w = p (dp - c) it collects sum p, sum w, sum w K and sum p K.  Once the waves' Delta = sum w + c sum p have met,
// dq = scale (sum w K - (Delta - c) sum p K)  (a second walk with Delta known would make the scores again: five products a tile, not four).
// The centre c of a column is the wave's mean of dp under p, so that the sums grow and round like those of the centred terms p (dp - Delta):
// values or output gradients with a common part make dp large against its spread, and keys have a mean under p.  It moves,
// and the sums with it, whenever the walk is half as long again, and where sum w is more than half of sum |w|.  (1300 keys, D = 128, values
// 3 + N(0,1), keys with +-1 a channel: dq 1.9e-6 from fp64, 4.9e-6 with c = 0, 2.0e-6 with two walks on the fp32 instruction.)
// A product for sum w K is made from zero and added: a matrix instruction that takes the long sum along rounds it several times,
// six times a product (100 thousand keys, D = 128: 1.0e-6 from fp64, 3.0e-6 with the sum taken along, 2.1e-6 with two walks on the fp32
// instruction; a million, D = 64: 2.6e-6, 1.3e-5, 6.7e-6).  sum p K is all but cancelled by the centre and takes it along.
// The vector work of a product's pieces stands beside the matrix work of the one before.  Two calls of 82 and 109 rows over 600
// keys, 8/2 heads, D = 64: 26 us (52 with the fp32 instruction and two walks).
template <int D> constexpr int row_waves = D == 64 ? 8 : 4;
template <int D>
__global__ __launch_bounds__(64 * row_waves<D>, 1) void pc_bwd_rows_f32_kernel(PcLaunch L, const float *__restrict__ lse, const float *__restrict__ d_out,
                                                                               float scale, float *__restrict__ d_q, float *__restrict__ delta_out)
{
    constexpr int NW = row_waves<D>, NJ = D / 8, VW = D / 32, HW = VW / 2, HALF = D / 2, PITCH = D + 4, NP = D / 32, PIECES_B = 3 * 2 * NP * 1024;
    // during the walk: the columns' queries and output gradients in pieces, each wave's present tile of keys; then the waves' dq
    constexpr int MEM = 2 * PIECES_B + NW * RowTile<D>::BYTES, MEM_END = 4 * (NW + 1) * 32 * PITCH;
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[MEM > MEM_END ? MEM : MEM_END];
    __shared__ __attribute__((aligned(16))) float2 s_rot[NW][HALF];         // the rotation of each wave's segment
    __shared__ float s_delta[NW][32];
    __shared__ int s_odd;
    bf16x8 (*const s_qp)[2 * NP][64] = reinterpret_cast<bf16x8 (*)[2 * NP][64]>(s_mem);     // [piece][16 dims][lane]
    bf16x8 (*const s_gp)[2 * NP][64] = reinterpret_cast<bf16x8 (*)[2 * NP][64]>(s_mem + PIECES_B);
    float (*const s_dq)[32 * PITCH] = reinterpret_cast<float (*)[32 * PITCH]>(s_mem);
    using VV = typename Vec<VW>::type;

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const PcItem item = L.items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_cols = cd.n_q * g, col0 = item.unit0 * 32;                  // column c: query row c / g, head c % g of the group
    // (waves 0 to 3 are on four SIMDs: what does not divide by the waves goes to the first ones)
    const int n_tiles = item.tile_end - item.tile_begin;
    const int t0 = item.tile_begin + wave * (n_tiles / NW) + min(wave, n_tiles % NW), t1 = t0 + n_tiles / NW + (wave < n_tiles % NW);
    const PcTile *tab = L.tiles + item.tile_tab0;
    const float *kb = (const float *)L.k_store + (int64_t)kh * L.slots * D, *vb = (const float *)L.v_store + (int64_t)kh * L.slots * D;
    const RowTile<D> keys(s_mem + 2 * PIECES_B + wave * RowTile<D>::BYTES, lane);           // the present tile's keys
    f32x4 rot;                                           // two pairs of a segment's rotation
    const unsigned rot_at = lane & (HALF / 2 - 1);
    auto load_rot = [&](const i32x4 &d) {
        unsigned at = 16 * rot_at;
        asm volatile("" : "+v"(at));
        rot = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(L.rot_seg + (int64_t)(cd.seg_off + d.z) * HALF) + at);
    };
    auto put_rot = [&]() { reinterpret_cast<f32x4 *>(s_rot[wave])[rot_at] = rot * UP; };     // (a wave's own LDS accesses are in order)
    auto describe = [&](int t) { return tile_at(tab, min(t, item.tile_end - 1)); };
    i32x4 next = {0, 0, 0, 0};
    if (t0 < t1) { next = describe(t0); keys.request(kb + (int64_t)next.x * D); load_rot(next); }
    if (threadIdx.x == 0) s_odd = 0;

    auto row_head = [&](int col) { return (int64_t)(cd.q_off + col / g) * L.n_q_heads + kh * g + col % g; };
    auto alive = [&](int col) { return col < n_cols && lse[row_head(col)] > -INFINITY; };
    for (int e = threadIdx.x; e < 32 * (HALF / 8); e += 64 * NW) {          // 8 pairs of a column a step
        const int c = e / (HALF / 8), i = 8 * (e % (HALF / 8));
        float x[8], y[8], u[8], w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = y[j] = u[j] = w[j] = 0.f;
        if (alive(col0 + c)) {
            const int64_t at = row_head(col0 + c) * D + i;
            const float *q = (const float *)L.q + at, *o = d_out + at;
            const float4 *rq = reinterpret_cast<const float4 *>(L.rot_q + (int64_t)(cd.q_off + (col0 + c) / g) * HALF + i);
#pragma unroll
            for (int j = 0; j < 8; ++j) { x[j] = q[j]; y[j] = q[j + HALF]; u[j] = o[j] * UP; w[j] = o[j + HALF] * UP; }
#pragma unroll
            for (int j = 0; j < 8; j += 2) turn2(x[j], y[j], x[j + 1], y[j + 1], up(rq[j / 2]));
        }
        const Pieces px = split8(x), py = split8(y), pu = split8(u), pw = split8(w);
#pragma unroll
        for (int z = 0; z < 3; ++z) {
            s_qp[z][i / 16][(i / 8 % 2) * 32 + c] = px.p[z]; s_qp[z][i / 16 + NP][(i / 8 % 2) * 32 + c] = py.p[z];
            s_gp[z][i / 16][(i / 8 % 2) * 32 + c] = pu.p[z]; s_gp[z][i / 16 + NP][(i / 8 % 2) * 32 + c] = pw.p[z];
        }
    }
    const bool live = alive(col0 + n);
    const float row_lse = live ? lse[row_head(col0 + n)] : 0.f;
    const int row = (col0 + n) / g;
    const int self_lim = cd.self_len - cd.n_q + row;     // last own token this column sees
    const int lo_lim = cd.self_len - cd.n_q + col0 / g;  // ... the item's first column
    const bool some_dead = __builtin_amdgcn_ballot_w64(!live) != 0;

    // step j of the keys: dims 16 j + 8 hh + 0..7 of the lane's key and their partners, turned, into x and y
    f32x4 k[4];
    const unsigned dim_at = keys.lds + 4 * hh * (D * 4) + ((((HW * n) / 4) ^ (4 * hh)) << 4) + (HW * n) % 4 * 4;
    const unsigned row_at = keys.lds + ((n * (D * 4) + ((n % RowTile<D>::CHUNKS) << 4)) ^ (hh << 5));
    auto read_k = [&](int p) {
        unsigned at = row_at;
        asm volatile("" : "+v"(at));                     // (one register, not one for every chunk)
#pragma unroll
        for (int j = 0; j < 4; ++j) k[j] = from_lds<f32x4>(at ^ ((4 * p + (j & 1) + (j >> 1) * (HALF / 4)) << 4));
    };
    float x[8], y[8];
    auto turn = [&](int p) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { x[j] = reinterpret_cast<const float *>(&k[0])[j]; y[j] = reinterpret_cast<const float *>(&k[2])[j]; }
#pragma unroll
        for (int j = 0; j < 8; j += 2) turn2(x[j], y[j], x[j + 1], y[j + 1], *reinterpret_cast<const float4 *>(&s_rot[wave][16 * p + 8 * hh + j]));
    };
    bf16x8 bn[3];                                        // the next product's right operand
    auto load_b = [&](bf16x8 (*s)[2 * NP][64], int j) {
#pragma unroll
        for (int z = 0; z < 3; ++z) bn[z] = s[z][j][lane];
    };
    Pieces kx;
    if (t0 < t1) {
        put_rot();
        wait_vm0();
        read_k(0);
        turn(0);
        kx = split8(x);
    }
    __syncthreads();

    float delta = 0.f, centre = 0.f, sum_w = 0.f, sum_p = 0.f, abs_w = 0.f;               // (sums of the lane's keys)
    int due = t0;                                        // the tile at which the centre moves next
    f32x16 acc_w[VW], acc_p[VW];                         // sum w K and sum p K: block i (partners: i + HW), row nn: dim HW nn + i (+ HALF)
#pragma unroll
    for (int i = 0; i < VW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_w[i][r] = acc_p[i][r] = 0.f;
    if (t0 < t1) load_b(s_qp, 0);
    for (int t = t0; t < t1; ++t) {
        const i32x4 d = next;
        next = describe(t + 1);
        f32x4 v[2 * NP][2];                              // step j of the values: dims 16 j + 8 hh + 0..7 of the lane's key
        {
            const float *vt = vb + (int64_t)d.x * D;     // (wave uniform)
            unsigned v_at = 4 * (n * D + 8 * hh);
            asm volatile("" : "+v"(v_at));               // (a 32-bit offset to a uniform address, not a pointer a lane)
#pragma unroll
            for (int j = 0; j < 2 * NP; ++j)
#pragma unroll
                for (int u = 0; u < 2; ++u) v[j][u] = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(vt + (16 * j + 4 * u)) + v_at);
        }
        load_rot(next);
        auto value = [&](int j) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = v[j][e / 4][e % 4] * UP;
        };
        f32x16 s, s1, dp, dp1;                           // (two chains of D / 2 terms round less than one of D)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = s1[r] = dp[r] = dp1[r] = 0.f;
        Pieces va;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            __builtin_amdgcn_sched_barrier(0);
            if (p + 1 < NP) read_k(p + 1);
            bf16x8 b[3] = {bn[0], bn[1], bn[2]};
            load_b(s_qp, p + NP);
            s = product(kx, b, s);
            const Pieces ky = split8(y);
            beside<6, 7>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int z = 0; z < 3; ++z) b[z] = bn[z];
            if (p + 1 < NP) load_b(s_qp, p + 1);
            else load_b(s_gp, 0);
            s1 = product(ky, b, s1);
            if (p + 1 < NP) {
                turn(p + 1);
                kx = split8(x);
            } else {
#pragma unroll
                for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(v[0][u]));           // (or they are cut, and waited for, as soon as they are requested)
                value(0);
                va = split8(x);
            }
            beside<6, 12>();
        }
        // the tile's keys once more, by dims: the lane's dims HW n .. + HW - 1 and their partners of key 8 (r / 4) + 4 hh + r % 4
        float kc[16][VW];
        float cs[2 * HW];                                // their rotation
        unsigned dim_now = dim_at;
        asm volatile("" : "+v"(dim_now));
        auto by_dim = [&](int r) {
            constexpr int CHUNKS = RowTile<D>::CHUNKS;
            const int c = 8 * (r >> 2) + (r & 3);        // (the key but for the lane's 4 hh)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const auto x = from_lds<typename Vec<HW>::type>((dim_now ^ (((u * (HALF / 4)) ^ (c % CHUNKS)) << 4)) + c * (D * 4));
#pragma unroll
                for (int i = 0; i < HW; ++i) kc[r][u * HW + i] = reinterpret_cast<const float *>(&x)[i];
            }
        };
#pragma unroll
        for (int j = 0; j < 2 * NP; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if (j == 1) s += s1;                         // (16 registers less)
            bf16x8 b[3] = {bn[0], bn[1], bn[2]};
            if (j + 1 < 2 * NP) load_b(s_gp, j + 1);
#pragma unroll
            for (int r = 16 / (2 * NP) * j; r < 16 / (2 * NP) * (j + 1); ++r) by_dim(r);
            f32x16 &c = (j & 1) ? dp1 : dp;
            c = product(va, b, c);
            if (j + 1 < 2 * NP) {
                value(j + 1);
                va = split8(x);
            }
            beside<6, 8>();
        }
#pragma unroll
        for (int i = 0; i < 2 * HW; ++i) cs[i] = reinterpret_cast<const float *>(&s_rot[wave][HW * n])[i];
        __builtin_amdgcn_sched_barrier(0);
        dp += dp1;
        const int valid = d.w & 0xFF, key0 = d.y;
        const bool self = (d.w & PC_TILE_SELF) != 0;
        float ps[16], w[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ps[r] = exp_x(fmaf(s[r], scale * (1.f / (UP * UP)), -row_lse));
        if (valid < PC_TILE || some_dead || (self && key0 + valid - 1 > lo_lim)) {        // (uniform over the wave)
            const int lim = !live ? 0 : self ? min(valid, self_lim - key0 + 1) : valid;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool seen = 8 * (r >> 2) + 4 * hh + (r & 3) < lim;
                ps[r] = seen ? ps[r] : 0.f;
                dp[r] = seen ? dp[r] : 0.f;
            }
        }
        auto sum16 = [](auto f) __attribute__((always_inline)) {            // (a tile's terms in pairs: a chain of them would round 16 times as often)
            float a[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) a[r] = f(r) + f(r + 8);
            return ((a[0] + a[4]) + (a[1] + a[5])) + ((a[2] + a[6]) + (a[3] + a[7]));
        };
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = ps[r] * (dp[r] - centre);
        sum_p += sum16([&](int r) { return ps[r]; });
        sum_w += sum16([&](int r) { return w[r]; });
        abs_w += sum16([&](int r) { return fabsf(w[r]); });
        if (t >= due || __builtin_amdgcn_ballot_w64(fabsf(sum_w) > 0.5f * abs_w) != 0) {
            due = t + 1 + (t - t0) / 2;
            const float all_w = sum_w + __shfl_xor(sum_w, 32), all_p = sum_p + __shfl_xor(sum_p, 32);      // of the column: both halves of the wave
            const float moved = centre + (all_p > 1e-30f ? all_w * __builtin_amdgcn_rcpf(all_p) : 0.f), by = moved - centre;
            centre = moved;
            sum_w = fmaf(-by, sum_p, sum_w);
            abs_w = fmaxf(fmaf(-fabsf(by), sum_p, abs_w), 0.f);             // (what it is at least)
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = fmaf(-by, ps[r], w[r]);
#pragma unroll
            for (int i = 0; i < VW; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_w[i][r] = fmaf(-by, acc_p[i][r], acc_w[i][r]);
        }
        // the next tile's keys: everything the wave has asked memory for has landed, and the present tile has been read
        asm volatile("" : "+v"(rot));
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < t1) keys.request(kb + (int64_t)next.x * D);
        auto column = [&](int kk, int i) __attribute__((always_inline)) {   // pair block i of keys 16 kk + ..: x the lower dims, y their partners
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                x[j] = kc[8 * kk + j][i]; y[j] = kc[8 * kk + j][HW + i]; x[j + 1] = kc[8 * kk + j + 1][i]; y[j + 1] = kc[8 * kk + j + 1][HW + i];
                turn2(x[j], y[j], x[j + 1], y[j + 1], make_float4(cs[2 * i], cs[2 * i + 1], cs[2 * i], cs[2 * i + 1]));
            }
        };
        f32x16 zero16;
#pragma unroll
        for (int r = 0; r < 16; ++r) zero16[r] = 0.f;
        Pieces pw = split8(w), pp = split8(ps), pw1, pp1;
        column(0, 0);
        kx = split8(x);
#pragma unroll
        for (int u = 0; u < 2 * HW; ++u) {               // (16 keys, pair block)
            const int kk = u / HW, i = u % HW;
            __builtin_amdgcn_sched_barrier(0);
            acc_w[i] += product(kx, pw.p, zero16);
            acc_p[i] = product(kx, pp.p, acc_p[i]);
            const Pieces ky = split8(y);
            if (u == 0) pw1 = split8(w + 8);
            beside<12, 8>();
            __builtin_amdgcn_sched_barrier(0);
            if (u + 1 == 2 * HW) {
                put_rot();
                wait_vm0();
                read_k(0);
            }
            acc_w[HW + i] += product(ky, pw.p, zero16);
            acc_p[HW + i] = product(ky, pp.p, acc_p[HW + i]);
            if (u == 0) pp1 = split8(ps + 8);
            if (u + 1 < 2 * HW) column((u + 1) / HW, (u + 1) % HW);
            else {                                       // (behind the last tile the present one is turned and cut once more, and not used)
                turn(0);
                load_b(s_qp, 0);
            }
            kx = split8(x);
            if (i + 1 == HW) { pw = pw1; pp = pp1; }
            beside<12, 8>();
        }
    }
    delta = fmaf(centre, sum_p, sum_w);
    delta += __shfl_xor(delta, 32);
    if (hh == 0) s_delta[wave][n] = delta;
    // The pieces of an Inf or NaN are not its parts: if a wave met one, be it behind a row's own token, all walk their tiles
    // again on the fp32 instruction.
    float odd = 0.f * delta;
#pragma unroll
    for (int i = 0; i < VW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd = fmaf(acc_w[i][r], 0.f, fmaf(acc_p[i][r], 0.f, odd));
    if (__builtin_amdgcn_ballot_w64(odd != 0.f) != 0 && lane == 0) s_odd = 1;
    __syncthreads();
    // (what follows is addressed anew: with the walk's own addresses the compiler keeps 40 registers for it through the walk, in scratch)
    unsigned tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int end_n = tid & 31, end_hh = (tid >> 5) & 1;
    if (s_odd == 0) {
        delta = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) delta += s_delta[w][end_n];
        const float off = delta - centre, down = scale * (1.f / (UP * UP * UP));
        if (t0 < t1)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float *p = &s_dq[wave][end_n * PITCH + HW * (8 * (r >> 2) + 4 * end_hh + (r & 3))];
#pragma unroll
                for (int i = 0; i < HW; ++i) {
                    p[i] = fmaf(-off, acc_p[i][r], acc_w[i][r]) * down;
                    p[HALF + i] = fmaf(-off, acc_p[HW + i][r], acc_w[HW + i][r]) * down;
                }
            }
        delta *= 1.f / (UP * UP);
    } else {
        // the queries are turned to a segment's frame at every new rotation; dq is collected in that frame and turned back into the
        // wave's own part of LDS
        const int n = end_n, hh = end_hh, row = (col0 + n) / g, self_lim = cd.self_len - cd.n_q + row;
        const bool live = alive(col0 + n);
        const int64_t rh = row_head(live ? col0 + n : col0);
        const float row_lse = live ? lse[rh] : 0.f;
        float *const s_g = reinterpret_cast<float *>(s_mem) + NW * 32 * PITCH;               // the columns' output gradients
        for (int e = tid; e < 32 * (D / 4); e += 64 * NW) {
            const int c = e / (D / 4), i = 4 * (e % (D / 4));
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            if (alive(col0 + c)) {
                const float *p = d_out + row_head(col0 + c) * D + i;
                z = make_float4(p[0], p[1], p[2], p[3]);
            }
            *reinterpret_cast<float4 *>(s_g + c * PITCH + i) = z;
        }
        __syncthreads();
        const float *qrow = (const float *)L.q + rh * D + 4 * hh;
        const float4 *rq = reinterpret_cast<const float4 *>(L.rot_q + (live ? (int64_t)(cd.q_off + row) : (int64_t)cd.q_off) * HALF) + 2 * hh;

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

        delta = 0.f;
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
    }
    if (tid < 32 && col0 + end_n < n_cols) delta_out[row_head(col0 + end_n)] = alive(col0 + end_n) ? delta : 0.f;
    __syncthreads();
    const int n_waves = min(NW, n_tiles);                // those that had tiles
    for (int e = tid; e < 32 * (D / 8); e += 64 * NW) {             // 4 pairs of a column a step
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
// A workgroup is 4 waves, one per SIMD with all of its 512 registers.  A wave owns one 32-key tile, its keys (turned to the call's
// positions) and values in pieces.  The column blocks (queries turned by their positions and output gradients in pieces, row
// scalars) are made in LDS by all of it, the next block's loads in flight under the present one's first products and its pieces
// cut beside the second ones.  Products that sum over columns take their left operand from the same LDS tiles through
// ds_read_b64_tr_b16: within 16 lanes, lane l points at row l / 4, columns 4 (l % 4) .. + 3 of a 4 x 16 block and receives column l,
// rows 0 .. 3.  The sums meet those of the tokens' other placements (other calls, repeated listings, other splits of the
// blocks) through one fp32 atomic per element, whole cache lines at a time.  Two calls of 82 and 109 rows over 600 keys, 8/2 heads,
// D = 64: 22 us (28 with the fp32 instruction).  D = 128 fills the 512 registers; 13 stand in scratch memory, 4 of them read in the loop.
typedef short s16x4 __attribute__((ext_vector_type(4)));
// A bf16 tile of 32 rows of D in LDS: chunk c (16 bytes) of row r sits at position c ^ swz(r) of the row; the rows of a fragment
// read, and the four rows of a transposing one, hit different banks.
template <int D>
struct PieceTile {
    static constexpr int BYTES = 64 * D;
    static __device__ int swz(int r) { return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 3) << 1) | ((r >> 3) & 1); }
    unsigned row_at, col_at[2][2];
    __device__ explicit PieceTile(int lane)
    {
        const int n = lane & 31, hh = lane >> 5, nh = (lane >> 4) & 1, l = lane & 15;
        row_at = (unsigned)(n * (2 * D) + ((hh ^ swz(n)) << 4));
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int e = 0; e < 2; ++e) {                // rows 16 kk + 8 e + 4 hh + 0..3
                const int r = 16 * kk + 8 * e + 4 * hh + (l >> 2);
                col_at[kk][e] = (unsigned)(r * (2 * D) + (((2 * nh + ((l & 3) >> 1)) ^ swz(r)) << 4) + (l & 1) * 8);
            }
    }
    // lane's row lane % 32, dims 16 ks + 8 (lane / 32) + 0..7
    __device__ bf16x8 by_row(const unsigned char *t, int ks) const { return *reinterpret_cast<const bf16x8 *>(t + (row_at ^ (ks << 5))); }
    // lane's dim 32 db + lane % 32, rows 16 kk + 8 (j / 4) + 4 (lane / 32) + j % 4
    __device__ bf16x8 by_col(const unsigned char *t, int kk, int db) const
    {
        typedef __attribute__((address_space(3))) s16x4 *Tr;
        const unsigned at = (unsigned)(uintptr_t)t;
        const uint2 x = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Tr)(uintptr_t)(at + (col_at[kk][0] ^ (db << 6)))));
        const uint2 y = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Tr)(uintptr_t)(at + (col_at[kk][1] ^ (db << 6)))));
        return __builtin_bit_cast(bf16x8, make_uint4(x.x, x.y, y.x, y.y));
    }
    // where dims dim .. dim + 3 of a row lie
    static __device__ unsigned at(int row, int dim) { return (unsigned)(row * (2 * D) + (((dim >> 3) ^ swz(row)) << 4) + 2 * (dim & 7)); }
};
template <int D>
__global__ __launch_bounds__(256, 1) void pc_bwd_keys_f32_kernel(PcLaunch L, const PcBwdKeyItem *__restrict__ items, const float *__restrict__ lse,
                                                                 const float *__restrict__ d_out, const float *__restrict__ delta, float scale,
                                                                 float *__restrict__ d_k, float *__restrict__ d_v)
{
    constexpr int NK = D / 16, VW = D / 32, HALF = D / 2, PITCH = D + 4, NP = HALF / 32;      // NP: float4 of pairs a thread stages
    using Tile = PieceTile<D>;
    constexpr int MEM = 2 * 2 * 3 * Tile::BYTES, MEM_END = 4 * 4 * 32 * PITCH;
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[MEM > MEM_END ? MEM : MEM_END];      // [buffer][queries, output gradients][piece]
    __shared__ __attribute__((aligned(16))) float s_lse[2][32], s_del[2][32];
    __shared__ __attribute__((aligned(16))) int s_lim[2][32];
    auto tile = [&](int buf, int which, int z) { return s_mem + ((buf * 2 + which) * 3 + z) * Tile::BYTES; };

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
    const Tile frag(lane);

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
            ra[i] = up(rot[0]); rb[i] = up(rot[1]);
        }
    };
    auto put4 = [&](int buf, int which, int dim, float4 v) __attribute__((always_inline)) {
        uint32_t lo[3], hi[3];
        split2(v.x, v.y, lo); split2(v.z, v.w, hi);
#pragma unroll
        for (int z = 0; z < 3; ++z) *reinterpret_cast<uint2 *>(tile(buf, which, z) + Tile::at(sc, dim)) = make_uint2(lo[z], hi[z]);
    };
    auto put = [&](int u, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            turn4(qa[i], qb[i], ra[i], rb[i]);
            put4(buf, 0, sp + 32 * i, qa[i]); put4(buf, 0, sp + 32 * i + HALF, qb[i]);
            put4(buf, 1, sp + 32 * i, up(ga[i])); put4(buf, 1, sp + 32 * i + HALF, up(gb[i]));
        }
        if (sp == 0) { s_lse[buf][sc] = st_lse; s_del[buf][sc] = st_del * (UP * UP); s_lim[buf][sc] = cd.self_len - cd.n_q + (32 * u + sc) / g; }
    };
    fetch(item.rt_begin);

    // the wave's keys turned by +(start - base) and its values: lane = key, dims 16 j + 8 hh + 0..7
    Pieces k[NK], v[NK];
    const float2 *rs = L.rot_seg + (int64_t)(cd.seg_off + d.z) * HALF;
    {
        const float *kr = (const float *)L.k_store + ((int64_t)kh * L.slots + slot0 + n) * D + 8 * hh;
        const float *vr = (const float *)L.v_store + ((int64_t)kh * L.slots + slot0 + n) * D + 8 * hh;
#pragma unroll
        for (int j = 0; j < NK / 2; ++j) {
            float x[8], y[8], u[8], w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { x[e] = kr[16 * j + e]; y[e] = kr[16 * j + e + HALF]; u[e] = vr[16 * j + e] * UP; w[e] = vr[16 * j + e + HALF] * UP; }
#pragma unroll
            for (int e = 0; e < 8; e += 2) turn2(x[e], y[e], x[e + 1], y[e + 1], up(*reinterpret_cast<const float4 *>(rs + 16 * j + 8 * hh + e)));
            k[j] = split8(x); k[j + NK / 2] = split8(y); v[j] = split8(u); v[j + NK / 2] = split8(w);
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
        const bool seen = active && !(self && key0 > last_lim);             // (uniform over the wave: some row of the block sees the tile)
        const bool causal = self && key0 + PC_TILE - 1 > first_lim;
        // p times UP and ds times UP twice of the block: register r: column 8 (r / 4) + 4 hh + r % 4
        auto weights = [&](f32x16 &p, f32x16 &w) __attribute__((always_inline)) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float4 l4 = *reinterpret_cast<const float4 *>(&s_lse[buf][8 * q4 + 4 * hh]), d4 = *reinterpret_cast<const float4 *>(&s_del[buf][8 * q4 + 4 * hh]);
                const int4 m4 = *reinterpret_cast<const int4 *>(&s_lim[buf][8 * q4 + 4 * hh]);
                const float ll[4] = {l4.x, l4.y, l4.z, l4.w}, dd[4] = {d4.x, d4.y, d4.z, d4.w};
                const int mm[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 4 * q4 + i;
                    const float x = UP * exp_x(fmaf(p[r], scale * (1.f / (UP * UP)), -ll[i]));
                    const bool ok = ll[i] < INFINITY && (!causal || key0 + n <= mm[i]);
                    p[r] = ok ? x : 0.f;
                    w[r] = ok ? x * (w[r] - dd[i]) * (scale * (1.f / UP)) : 0.f;
                }
            }
        };
        f32x16 p, w;
        if (seen) {
            f32x16 s1, w1;                               // (two chains of D / 2 terms round less than one of D)
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = s1[r] = w[r] = w1[r] = 0.f;
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                Pieces a;
#pragma unroll
                for (int z = 0; z < 3; ++z) a.p[z] = frag.by_row(tile(buf, 0, z), j);
                f32x16 &c = (j & 1) ? s1 : p;
                c = product(a, k[j].p, c);
            }
#pragma unroll
            for (int j = 0; j < NK; ++j) {
                Pieces a;
#pragma unroll
                for (int z = 0; z < 3; ++z) a.p[z] = frag.by_row(tile(buf, 1, z), j);
                f32x16 &c = (j & 1) ? w1 : w;
                c = product(a, v[j].p, c);
            }
            p += s1;
            w += w1;
            weights(p, w);
        }
        if (u + 1 < item.rt_end) put(u + 1, buf ^ 1);    // (last read before the barrier behind the block before this one)
        if (seen) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                float x[8], y[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) { x[j] = p[8 * kk + j]; y[j] = w[8 * kk + j]; }
                const Pieces pp = split8(x), pw = split8(y);
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    Pieces a, b;
#pragma unroll
                    for (int z = 0; z < 3; ++z) { a.p[z] = frag.by_col(tile(buf, 1, z), kk, i); b.p[z] = frag.by_col(tile(buf, 0, z), kk, i); }
                    dv[i] = product(a, pp.p, dv[i]);
                    dk[i] = product(b, pw.p, dk[i]);
                }
            }
        }
        __syncthreads();
    }
    if (!active) return;
    // The pieces of an Inf or NaN are not its parts, nor are those of a number that rounds to one in bf16 (3.4e38).  Whatever holds one, a query, an output
    // gradient, a key or a value, it leaves a NaN in the sums that it belongs to: such a wave goes through its column blocks again, on the fp32
    // instruction, with the caller's numbers.
    float odd = 0.f;
#pragma unroll
    for (int i = 0; i < VW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            odd = fmaf(dk[i][r], 0.f, fmaf(dv[i][r], 0.f, odd));
            dk[i][r] *= 1.f / (UP * UP * UP);
            dv[i][r] *= 1.f / (UP * UP);
        }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd != 0.f) != 0, 0)) {
#pragma unroll
        for (int i = 0; i < VW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) dk[i][r] = dv[i][r] = 0.f;
        const float *kr = (const float *)L.k_store + ((int64_t)kh * L.slots + slot0 + n) * D, *vr = (const float *)L.v_store + ((int64_t)kh * L.slots + slot0 + n) * D;
        auto turned = [&](const float *v, const float2 *rot, int dim) {     // one dim of a row, turned
            const int i = dim & (HALF - 1);
            const float a = v[i], b = v[i + HALF];
            const float2 cs = rot[i];
            return dim < HALF ? a * cs.x - b * cs.y : a * cs.y + b * cs.x;
        };
        struct Column { int64_t rh; const float2 *rot; float lse, delta; int lim; };
        auto column = [&](int col) {                     // (no such column, or a row that saw nothing: a log-sum-exp of +inf)
            const int cc = min(col, n_cols - 1);
            Column r;
            r.rh = (int64_t)(cd.q_off + cc / g) * L.n_q_heads + kh * g + cc % g;
            r.rot = L.rot_q + (int64_t)(cd.q_off + cc / g) * HALF;
            const float x = lse[r.rh];
            r.lse = col < n_cols && x > -INFINITY ? x : INFINITY;
            r.delta = r.lse < INFINITY ? delta[r.rh] : 0.f;
            r.lim = cd.self_len - cd.n_q + col / g;
            return r;
        };
        auto q_at = [&](const Column &c, int dim) { const float v = turned((const float *)L.q + c.rh * D, c.rot, dim); return c.lse < INFINITY ? v : 0.f; };
        auto g_at = [&](const Column &c, int dim) { const float v = d_out[c.rh * D + dim]; return c.lse < INFINITY ? v : 0.f; };
#pragma unroll 1
        for (int u = item.rt_begin; u < item.rt_end; ++u) {
            const int first_lim = cd.self_len - cd.n_q + 32 * u / g, last_lim = cd.self_len - cd.n_q + (32 * u + 31) / g;
            if (self && key0 > last_lim) continue;
            const bool causal = self && key0 + PC_TILE - 1 > first_lim;
            const Column own = column(32 * u + n);
            f32x16 p, w, p1, w1;
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = w[r] = p1[r] = w1[r] = 0.f;
#pragma unroll 1
            for (int j = 0; j < HALF; j += 2) {
                p = MFMA_F32(q_at(own, j + hh), turned(kr, rs, j + hh), p);
                w = MFMA_F32(g_at(own, j + hh), vr[j + hh], w);
                p1 = MFMA_F32(q_at(own, j + HALF + hh), turned(kr, rs, j + HALF + hh), p1);
                w1 = MFMA_F32(g_at(own, j + HALF + hh), vr[j + HALF + hh], w1);
            }
            p += p1;
            w += w1;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const Column c = column(32 * u + 8 * (r >> 2) + 4 * hh + (r & 3));
                // (the maximum: an infinite key makes a NaN; a row with a log-sum-exp saw it at a score of -inf)
                const float x = exp_x(fmaxf(fmaf(p[r], scale, -c.lse), -1e30f));
                const bool ok = c.lse < INFINITY && (!causal || key0 + n <= c.lim);
                const float pp = ok ? x : 0.f, ww = ok ? x * (w[r] - c.delta) * scale : 0.f;
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    dv[i] = MFMA_F32(g_at(c, 32 * i + n), pp, dv[i]);
                    dk[i] = MFMA_F32(q_at(c, 32 * i + n), ww, dk[i]);
                }
            }
        }
    }
    // element (i, r) is dim 32 i + 8 (r / 4) + 4 hh + r % 4 of key n: turned round through the wave's quarter of the block buffers
    float *stg = reinterpret_cast<float *>(s_mem) + wave * 32 * PITCH;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        const f32x16 *a = which == 0 ? dk : dv;
#pragma unroll
        for (int i = 0; i < VW / 2; ++i)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int dim = 32 * i + 8 * q4 + 4 * hh;
                float4 lo = make_float4(a[i][4 * q4], a[i][4 * q4 + 1], a[i][4 * q4 + 2], a[i][4 * q4 + 3]);
                float4 hi = make_float4(a[i + VW / 2][4 * q4], a[i + VW / 2][4 * q4 + 1], a[i + VW / 2][4 * q4 + 2], a[i + VW / 2][4 * q4 + 3]);
                if (which == 0) {                        // back to the stored frame
                    const float4 *c = reinterpret_cast<const float4 *>(rs + dim);
                    turn4(lo, hi, conj2(c[0]), conj2(c[1]));
                }
                *reinterpret_cast<float4 *>(stg + n * PITCH + dim) = lo;
                *reinterpret_cast<float4 *>(stg + n * PITCH + dim + HALF) = hi;
            }
        // (a wave's own LDS writes and reads are ordered; the other waves use other parts)
        float *out = (which == 0 ? d_k : d_v) + ((int64_t)slot0 * L.n_kv_heads + kh) * D + lane;
        for (int k0 = 0; k0 < valid; k0 += 8) {          // (eight rows' LDS reads together)
            float z[8][D / 64];
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int i = 0; i < D / 64; ++i) z[e][i] = stg[(k0 + e) * PITCH + lane + 64 * i];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k0 + e < valid)
#pragma unroll
                    for (int i = 0; i < D / 64; ++i) unsafeAtomicAdd(out + (int64_t)(k0 + e) * L.n_kv_heads * D + 64 * i, z[e][i]);
        }
    }
}

void pc_launch_attend_bwd_f32(const PcLaunch &L, int n_items, const PcBwdKeyItem *key_items, int n_key_items, int D, const float *lse,
                              const float *d_out, float scale, float *delta, float *d_q, float *d_k, float *d_v, hipStream_t st)
{
    if (n_items <= 0) return;
    const unsigned rows = (unsigned)n_items * L.n_kv_heads, keys = (unsigned)n_key_items * L.n_kv_heads;
    if (D == 64) {
        pc_bwd_rows_f32_kernel<64><<<rows, 64 * row_waves<64>, 0, st>>>(L, lse, d_out, scale, d_q, delta);
        if (keys > 0) pc_bwd_keys_f32_kernel<64><<<keys, 256, 0, st>>>(L, key_items, lse, d_out, delta, scale, d_k, d_v);
    } else {
        pc_bwd_rows_f32_kernel<128><<<rows, 64 * row_waves<128>, 0, st>>>(L, lse, d_out, scale, d_q, delta);
        if (keys > 0) pc_bwd_keys_f32_kernel<128><<<keys, 256, 0, st>>>(L, key_items, lse, d_out, delta, scale, d_k, d_v);
    }
}

// d_k holds the gradient with respect to the stored keys K~_t = R(base + t) k_t; the gradient with
// respect to k_t is R(base + t)^T of it (Sec. 2.4 "Position Updates", transposed).  blockIdx.y names the message; a thread
// takes one rotation pair of a token and turns it for every KV head: the fp64 sincos is what the kernel spends its time on
// (one per head and pair, as before, took 55 us for 5500 tokens x 8 heads; now 12).
// List: a device pointer, or the messages themselves as the kernel's first arguments (the copy of 12 of them and its event took 6 us of a step of 90).
template <typename List>
__global__ __launch_bounds__(256) void pc_grad_keys_finalize_kernel(const List msgs, int n_kv_heads, int D, const double *__restrict__ inv_freq, float *__restrict__ d_k)
{
    PcMsgEntry m;
    if constexpr (std::is_same<List, PcArgBlob>::value) {
        static_assert(sizeof(PcMsgEntry) == 16, "");
        const auto *p = (const __attribute__((address_space(4))) int32_t *)__builtin_amdgcn_kernarg_segment_ptr() + 4 * blockIdx.y;
        m.slot_start = p[0]; m.len = p[1]; m.base_pos = p[2];
    } else m = msgs[blockIdx.y];
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

void pc_launch_grad_keys_finalize(const PcMsgEntry *msgs, const PcMsgEntry *host_msgs, int n_msgs, int n_kv_heads, int D, const double *inv_freq,
                                  float *d_k, hipStream_t st)
{
    if (host_msgs) {                                     // (the caller checked that they fit)
        PcArgBlob blob;
        std::memcpy(blob.w, host_msgs, sizeof(PcMsgEntry) * (size_t)n_msgs);
        pc_grad_keys_finalize_kernel<PcArgBlob><<<dim3(64, (unsigned)n_msgs), 256, 0, st>>>(blob, n_kv_heads, D, inv_freq, d_k);
        return;
    }
    for (int first = 0; first < n_msgs; first += 65535) {              // grid.y is limited to 65535
        const int n = n_msgs - first < 65535 ? n_msgs - first : 65535;
        dim3 grid(64, (unsigned)n);                      // 256 tokens of 64 pairs a step
        pc_grad_keys_finalize_kernel<const PcMsgEntry *><<<grid, 256, 0, st>>>(msgs + first, n_kv_heads, D, inv_freq, d_k);
    }
}
