// Attention of fp32 caches on the bf16 matrix instructions (gfx950), at fp32 precision.
//
// The transposed problem of the bf16 kernels: scores S^T = K~ . Q^T (rows = 32 keys, columns = 32 (query row, head) pairs
// of one KV head), O^T = V^T . P^T.  An fp32 number is the exact sum of three bf16 pieces and a product of two bf16 numbers is
// exact in fp32, so six bf16 MFMAs over the pieces are an fp32 product (see split8): a tile takes 96 of them, of 32 cycles (D = 128),
// where v_mfma_f32_32x32x2_f32 took 128 of 64.  A result has 16 rows a lane: 8 (r / 4) + 4 (lane / 32) + r % 4, and the order of
// the summed index is free as long as both operands agree: registers 8 kk .. 8 kk + 7 of the scores are the right operand of
// the second product for the keys they stand for, and a lane reads those keys' values straight from memory, 16 bytes at a time.
//
// A workgroup is 8 waves, two per SIMD, over the same 32 columns; each walks a contiguous eighth of the item's tiles and
// the results meet in LDS.  The columns' queries are turned by their positions, cut and kept in LDS; each wave turns its keys by
// (start - stored base) and cuts them, and its values, as they come.  Bound: instruction issue.  Turning and cutting a tile are
// 1000 vector instructions beside 96 MFMAs, about 4.5 cycles each of a SIMD's for its two waves together (6.5 thousand cycles a
// tile and wave, 3 thousand of them matrix work).  A call with few columns is split over the tiles as well (see
// pc_plan_and_stage) and pc_merge_f32_kernel adds the parts.
//
// 200 rows over 1400 keys, 32/8 heads, D = 128: 49 us (77 with the fp32 instruction); 32 rows over 160 keys, 4/2 heads, D = 64:
// 13.0 -> 10.4 us, all of it latency.  Distance to fp64 in the 2-norm 1.7e-7 to 3.0e-7 over ten shapes (2.2e-7 to 3.7e-7 with the
// fp32 instruction: its chains are four times as long).
#include "pc_pieces.h"
#include "pc_self_plan.h"

#define NW 8                  // waves of a workgroup
#define MFMA_F32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0)

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float other_half(float x)                        // the value of lane ^ 32
{
    return __shfl_xor(x, 32);
}
template <int W> struct Vec;                                                // W consecutive floats of a row
template <> struct Vec<2> { using type = f32x2; };
template <> struct Vec<4> { using type = f32x4; };

}  // namespace

// SELF: the launch plans for itself
template <int D, bool SELF>
__device__ __forceinline__ void attend_f32(const PcLaunch &L, const PcSelf &S)
{
    constexpr int NJ = D / 8, VW = D / 32, HALF = D / 2, PITCH = D + 4, NP = D / 32;        // NP: steps of 16 dims and their partners
    // during the walk: the columns' queries turned by their positions, in pieces, and each wave's present tile of keys; then the waves' results
    __shared__ __attribute__((aligned(1024))) unsigned char s_mem[3 * 2 * NP * 1024 + NW * RowTile<D>::BYTES];
    __shared__ __attribute__((aligned(16))) float2 s_rot[NW][HALF];         // the rotation of each wave's segment
    __shared__ float s_m[NW][32], s_l[NW][32];
    __shared__ int s_again;
    bf16x8 (*const s_qp)[2 * NP][64] = reinterpret_cast<bf16x8 (*)[2 * NP][64]>(s_mem);     // [piece][16 dims][lane]
    float (*const s_acc)[32 * PITCH] = reinterpret_cast<float (*)[32 * PITCH]>(s_mem);
    static_assert(sizeof(float) * NW * 32 * PITCH <= sizeof s_mem, "");

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const auto *args = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();      // SELF: the lists
    PcItem item;
    PcCallDesc cd;
    if constexpr (SELF) {
        item = self_item(args, S, blockIdx.x / L.n_kv_heads);
        cd = self_call(args, S, item.call);
    } else {
        item = L.items[blockIdx.x / L.n_kv_heads];
        cd = L.calls[item.call];
    }
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_cols = cd.n_q * g;
    const int col0 = item.unit0 * 32;       // column c: query row c / g, head c % g of the group
    // this wave's contiguous run of tiles
    const int n_tiles = item.tile_end - item.tile_begin;
    // (waves 0 to 3 are on four SIMDs: what does not divide by eight goes to the first ones)
    const int t0 = item.tile_begin + wave * (n_tiles / NW) + min(wave, n_tiles % NW), t1 = t0 + n_tiles / NW + (wave < n_tiles % NW);
    if (threadIdx.x == 0) s_again = 0;

    using VV = typename Vec<VW>::type;
    const float *kb = (const float *)L.k_store + (int64_t)kh * L.slots * D, *vb = (const float *)L.v_store + (int64_t)kh * L.slots * D;
    const unsigned v_at = 4 * hh * D + VW * n;           // within a tile: the lane's dims VW n + 0..VW-1
    const RowTile<D> keys(s_mem + 3 * 2 * NP * 1024 + wave * RowTile<D>::BYTES, lane);      // the present tile's keys
    auto request_k = [&](int slot0) { keys.request(kb + (int64_t)slot0 * D); };
    const PcTile *tab = L.tiles + item.tile_tab0;
    const float2 *rot_seg = L.rot_seg + (int64_t)cd.seg_off * HALF, *rot_q = L.rot_q + (int64_t)cd.q_off * HALF;      // of the call's entries, of its rows
    if constexpr (SELF) {
        if (blockIdx.x == 0 && (int)threadIdx.x < S.n16) {
            typedef int i32x4a __attribute__((ext_vector_type(4)));
            const i32x4a w = reinterpret_cast<const __attribute__((address_space(4))) i32x4a *>(args)[threadIdx.x];
            S.ws[threadIdx.x] = make_uint4((unsigned)w.x, (unsigned)w.y, (unsigned)w.z, (unsigned)w.w);
        }
        char *region = S.regions + (int64_t)blockIdx.x * S.stride;
        const int row0 = col0 / g;
        wg_plan<HALF, 64 * NW>(S, args, cd, item.tile_begin, item.tile_end, row0, min((col0 + 31) / g, cd.n_q - 1) - row0 + 1, region,
                               [&](auto slot_of) __attribute__((always_inline)) { if (t0 < t1) request_k(slot_of(t0)); });
        region = behind(region);
        tab = reinterpret_cast<const PcTile *>(region) - item.tile_begin;
        rot_seg = reinterpret_cast<const float2 *>(region + S.off_rot);
        rot_q = reinterpret_cast<const float2 *>(region + S.off_rot_q) - row0 * HALF;
    }
    auto describe = [&](int t) {
        const int tc = __builtin_amdgcn_readfirstlane(max(0, min(t, item.tile_end - 1)));
        if (item.tile_end <= 0) return (i32x4){0, 0, 0, 0};                 // a call that sees nothing has no table
        return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(tab + tc));
    };
    i32x4 next = describe(t0);                           // {slot0, key0, seg, valid | flags}
    f32x4 k[4];                                          // step p of the present tile: dims 16 p + 8 hh + 0..7 of the lane's key and their partners
    const unsigned row_at = keys.lds + ((n * (D * 4) + ((n % RowTile<D>::CHUNKS) << 4)) ^ (hh << 5));
    auto read_k = [&](int p) {
        unsigned at = row_at;
        asm volatile("" : "+v"(at));                     // (one register, not one for every chunk)
#pragma unroll
        for (int j = 0; j < 4; ++j) k[j] = from_lds<f32x4>(at ^ ((4 * p + (j & 1) + (j >> 1) * (HALF / 4)) << 4));
    };
    f32x4 rot;                                           // two pairs of a segment's rotation
    const unsigned rot_at = lane & (HALF / 2 - 1);
    auto load_rot = [&](const i32x4 &d) {
        unsigned at = 16 * rot_at;
        asm volatile("" : "+v"(at));                     // (a 32-bit offset to a uniform address, not a pointer a lane)
        rot = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(rot_seg + (int64_t)d.z * HALF) + at);
    };
    auto put_rot = [&]() { reinterpret_cast<f32x4 *>(s_rot[wave])[rot_at] = rot * UP; };     // (a wave's own LDS accesses are in order)
    if (t0 < t1) { if constexpr (!SELF) request_k(next.x); load_rot(next); }

    for (int e = threadIdx.x; e < 32 * (HALF / 8); e += 64 * NW) {          // 8 pairs of a column a step
        const int c = e / (HALF / 8), i = 8 * (e % (HALF / 8));
        float x[8], y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = y[j] = 0.f;
        if (col0 + c < n_cols) {
            const int col = col0 + c;
            const int64_t R = cd.q_off + col / g;
            const float *q = (const float *)L.q + (R * L.n_q_heads + kh * g + col % g) * D + i;
            const float4 *rot = reinterpret_cast<const float4 *>(rot_q + (int64_t)(col / g) * HALF + i);
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const float4 cs = up(rot[j / 2]);
                const float x0 = q[j], x1 = q[j + 1], y0 = q[j + HALF], y1 = q[j + HALF + 1];
                x[j] = x0 * cs.x - y0 * cs.y; x[j + 1] = x1 * cs.z - y1 * cs.w;
                y[j] = x0 * cs.y + y0 * cs.x; y[j + 1] = x1 * cs.w + y1 * cs.z;
            }
        }
        const Pieces px = split8(x), py = split8(y);
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            s_qp[w][i / 16][(i / 8 % 2) * 32 + c] = px.p[w];
            s_qp[w][i / 16 + NP][(i / 8 % 2) * 32 + c] = py.p[w];
        }
    }
    float x[8], y[8];
    auto turn = [&](int p) __attribute__((always_inline)) {                 // step p of the keys, in k, into x, y
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            const float4 cs = *reinterpret_cast<const float4 *>(&s_rot[wave][16 * p + 8 * hh + j]);
            const float *kx = reinterpret_cast<const float *>(&k[0]) + j, *ky = reinterpret_cast<const float *>(&k[2]) + j;
            x[j] = kx[0] * cs.x - ky[0] * cs.y; x[j + 1] = kx[1] * cs.z - ky[1] * cs.w;
            y[j] = kx[0] * cs.y + ky[0] * cs.x; y[j + 1] = kx[1] * cs.w + ky[1] * cs.z;
        }
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

    const int row = (col0 + n) / g;
    const int self_lim = cd.self_len - cd.n_q + row;     // last own token this column sees
    const int lo_lim = cd.self_len - cd.n_q + col0 / g;              // ... the item's first column
    const bool sees = t0 < t1 && !((next.w & PC_TILE_SELF) != 0 && next.y > self_lim);      // a key of the wave's
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 acc[VW];
    auto clear = [&]() {
        m_run = -INFINITY; l_run = 0.f;
#pragma unroll
        for (int i = 0; i < VW; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    };
    clear();
    // scores scaled and masked, the running maximum and sum, the accumulators' factor: s becomes the probabilities
    auto softmax = [&](f32x16 &s, float scale, const i32x4 &d, bool causal) __attribute__((always_inline)) {
        const int valid = d.w & 0xFF, lim = (d.w & PC_TILE_SELF) ? min(valid, self_lim - d.y + 1) : valid;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] *= scale;
        if (valid < PC_TILE || causal) {                 // (uniform over the wave)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = (8 * (r >> 2) + 4 * hh + (r & 3) < lim) ? s[r] : -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = fmaxf(mx, other_half(mx));
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
        const float alpha = ex2(m_run - m_safe);
        m_run = m_new;
        float ps = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[r] = ex2(s[r] - m_safe); ps += s[r]; }
        l_run = l_run * alpha + ps;
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {               // rare once the running maxima have settled
#pragma unroll
            for (int i = 0; i < VW; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] *= alpha;
        }
    };
    // some column of the item does not see some key of the tile
    auto on_limit = [&](const i32x4 &d) { return (d.w & PC_TILE_SELF) != 0 && d.y + (d.w & 0xFF) - 1 > lo_lim; };

    // The walk.  Every product of pieces stands beside the vector work that makes the pieces of the next one (`beside` pins the
    // order: a matrix instruction, a few vector ones): keys are turned and cut a step of 16 + 16 dims ahead, values a block ahead.
    bf16x8 qn[3];                                        // the next product's right operand
    auto load_q = [&](int j) {
#pragma unroll
        for (int w = 0; w < 3; ++w) qn[w] = s_qp[w][j][lane];
    };
    if (t0 < t1) load_q(0);
    for (int t = t0; t < t1; ++t) {
        const i32x4 d = next;
        next = describe(t + 1);
        VV v[16];                                        // register r: key 8 (r / 4) + 4 hh + r % 4
        const float *vt = vb + (int64_t)d.x * D;         // (wave uniform)
        auto load_v = [&](int half) {
#pragma unroll
            for (int r = 8 * half; r < 8 * half + 8; ++r) v[r] = *reinterpret_cast<const VV *>(vt + (8 * (r >> 2) + (r & 3)) * D + v_at);
        };
        auto column = [&](int i) {                       // block i % VW of the values of keys 16 (i / VW) + ...
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = reinterpret_cast<const float *>(&v[8 * (i / VW) + j])[i % VW];
        };
        f32x16 s, s1;                                    // (two chains of D / 2 terms round less than one of D)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = s1[r] = 0.f;
        Pieces vp;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            __builtin_amdgcn_sched_barrier(0);
            if (p == NP / 4) { load_v(0); load_rot(next); }
            if (p == NP / 2) load_v(1);
            if (p + 1 < NP) read_k(p + 1);
            bf16x8 qc[3] = {qn[0], qn[1], qn[2]};
            load_q(p + NP);
            s = product(kx, qc, s);
            const Pieces ky = split8(y);
            beside<6, 7>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int w = 0; w < 3; ++w) qc[w] = qn[w];
            if (p + 1 < NP) load_q(p + 1);
            s1 = product(ky, qc, s1);
            if (p + 1 < NP) {
                turn(p + 1);
                kx = split8(x);
            } else {
                column(0);
                vp = split8(x);
            }
            beside<6, 12>();
        }
        __builtin_amdgcn_sched_barrier(0);
        s += s1;
        softmax(s, L.scale_log2 * (1.f / (UP * UP)), d, on_limit(d));
        // the next tile's keys: the values and the rotation have landed by then, so that no wait for them waits for the keys as well
        // (behind the last tile the present one is turned and cut once more, and not used)
#pragma unroll
        for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(v[r]));
        asm volatile("" : "+v"(rot));
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < t1) request_k(next.x);
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = s[j];
        Pieces pr = split8(x), pr1;
#pragma unroll
        for (int i = 0; i < 2 * VW; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 == 2 * VW) {
                put_rot();
                wait_vm0();
                read_k(0);
            }
            acc[i % VW] = product(vp, pr.p, acc[i % VW]);
            if (i == 0) {
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = s[8 + j];
                pr1 = split8(x);
            }
            if (i + 1 < 2 * VW) {
                column(i + 1);
                vp = split8(x);
            } else {
                turn(0);
                kx = split8(x);
                load_q(0);
            }
            if (i + 1 == VW) pr = pr1;
            beside<6, 8>();
        }
    }
    // The waves' results meet in LDS: element (i, r) of a lane is dim VW (8 (r / 4) + 4 hh + r % 4) + i of column n; then 16 threads a column take
    // dims 4 sub + 64 i.
    //
    // The pieces of an Inf or NaN are not its parts, nor are those of a number that rounds to one in bf16 (3.4e38): a workgroup that met one, be it in
    // a query, a key that counts or the value of a token behind a row's own, which no probability of zero takes out of a
    // product, walks its tiles again on the fp32 instruction, with the caller's queries.  So does one with a result below 2^-100 that is not
    // zero, whose values may be below 2^-110 and have bits behind their pieces' last ones, and one with a wave whose column sees keys and has met none:
    // their scores may be below -2^96, infinities times UP twice.  What no number gives is found in the results: 8 (4) of them a thread there,
    // 64 (32) in the waves' accumulators, which took 0.8 us to look through in the first example above.
    // There a probability of zero takes a key out of the second product only while its value is finite.  What lies behind a
    // message's last token is (the store is kept that way), but a later token of the new message is the caller's own
    // data: in a tile on the causal limit an Inf or NaN is left out and added at the end, for the columns that see its key.
    // (addressed anew: with the walk's own addresses the compiler keeps registers for all of this through the walk)
    unsigned tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int c = tid >> 4, sub = tid & 15, end_col = col0 + c;
    const int end_n = tid & 31, end_hh = (tid >> 5) & 1;
    bool odd = false;
    for (bool slow = false;; slow = true) {
        __syncthreads();                                 // (the queries' pieces make room for the results)
        l_run += other_half(l_run);
        if (end_hh == 0) { s_m[wave][end_n] = m_run; s_l[wave][end_n] = l_run; }
        if (sees && m_run == -INFINITY) s_again = 1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            VV z;
            float *x = reinterpret_cast<float *>(&z);
#pragma unroll
            for (int i = 0; i < VW; ++i) x[i] = acc[i][r];
            *reinterpret_cast<VV *>(&s_acc[wave][end_n * PITCH + VW * (8 * (r >> 2) + 4 * end_hh + (r & 3))]) = z;
        }
        if (__builtin_amdgcn_ballot_w64(odd) != 0) {     // (the probability has no say in an Inf or NaN; a wave's own LDS accesses are in order)
            for (int t = t0; t < t1; ++t) {
                const i32x4 d = describe(t);
                if (!(d.w & PC_TILE_SELF) || d.y + (d.w & 0xFF) - 1 <= lo_lim) continue;
                const int lim = min(d.w & 0xFF, self_lim - d.y + 1);
                const float *vr = (const float *)L.v_store + ((int64_t)kh * L.slots + d.x) * D;
                for (int e = end_hh; e < lim * D; e += 2) {
                    const float x = vr[e];
                    if (!(fabsf(x) < INFINITY)) s_acc[wave][end_n * PITCH + e % D] += x;
                }
            }
        }
        __syncthreads();
        float mm = s_m[0][c], l = 0.f;
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, s_m[w][c]);
        float4 o[D / 64];
#pragma unroll
        for (int i = 0; i < D / 64; ++i) o[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (mm > -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (!(s_m[w][c] > -INFINITY)) { l += s_l[w][c]; continue; }        // saw nothing: a sum of 0 (or NaN, which stays)
                const float f = ex2(s_m[w][c] - mm);
                l = fmaf(s_l[w][c], f, l);
#pragma unroll
                for (int i = 0; i < D / 64; ++i) {
                    const float4 a = *reinterpret_cast<const float4 *>(&s_acc[w][c * PITCH + 64 * i + 4 * sub]);
                    o[i].x = fmaf(a.x, f, o[i].x); o[i].y = fmaf(a.y, f, o[i].y); o[i].z = fmaf(a.z, f, o[i].z); o[i].w = fmaf(a.w, f, o[i].w);
                }
            }
        } else if (!slow) {
#pragma unroll
            for (int w = 0; w < NW; ++w) l += s_l[w][c]; // (only a NaN is seen in it)
        }
        bool again = false;
        if (end_col < n_cols) {
            const int r = end_col / g, h = kh * g + end_col % g;
            again = !(l < INFINITY);
            const bool whole = cd.n_splits == 1;
            const int64_t at = (whole ? (int64_t)(cd.q_off + r) : (int64_t)cd.part_off + (int64_t)item.split * cd.n_q + r) * L.n_q_heads + h;
#pragma unroll
            for (int i = 0; i < D / 64; ++i) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = fabsf((&o[i].x)[j]);
                    again |= !(x < INFINITY) || (x < 0x1p-100f && x > 0.f);
                }
                if (whole) {
                    if (l > 0.f) { o[i].x /= l; o[i].y /= l; o[i].z /= l; o[i].w /= l; }
                    else o[i] = make_float4(0.f, 0.f, 0.f, 0.f);            // nothing visible (or a NaN score)
                    float *out = (float *)L.out + at * D + 64 * i + 4 * sub;
                    out[0] = o[i].x; out[1] = o[i].y; out[2] = o[i].z; out[3] = o[i].w;
                } else *reinterpret_cast<float4 *>((float *)L.part_o + at * D + 64 * i + 4 * sub) = o[i];
            }
            if (sub == 0) {
                if (!whole) { L.part_ml[at * 2] = mm; L.part_ml[at * 2 + 1] = l; }
                else if (L.lse) L.lse[at] = (l > 0.f) ? (mm + log2f(l)) * 0.6931471805599453f : -INFINITY;
            }
        }
        if (slow) return;
        if (again) s_again = 1;
        __syncthreads();
        if (__builtin_expect(s_again == 0, 1)) return;
        const int n = end_n, hh = end_hh;
        const unsigned v_at = 4 * hh * D + VW * n;
        const bool there = col0 + n < n_cols;
        const int col = there ? col0 + n : col0;
        const float *qr = (const float *)L.q + ((int64_t)(cd.q_off + col / g) * L.n_q_heads + kh * g + col % g) * D + 4 * hh;
        const float4 *rq = reinterpret_cast<const float4 *>(rot_q + (int64_t)(col / g) * HALF) + 2 * hh;
        auto query = [&](float4 &a, float4 &b, int j) {  // dims 8 j + 4 hh + 0..3 of the lane's column and their partners, turned by its position
            a = b = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!there) return;
            const float4 c0 = rq[4 * j], c1 = rq[4 * j + 1];
            const float x[4] = {qr[8 * j], qr[8 * j + 1], qr[8 * j + 2], qr[8 * j + 3]};
            const float y[4] = {qr[8 * j + HALF], qr[8 * j + HALF + 1], qr[8 * j + HALF + 2], qr[8 * j + HALF + 3]};
            a = make_float4(x[0] * c0.x - y[0] * c0.y, x[1] * c0.z - y[1] * c0.w, x[2] * c1.x - y[2] * c1.y, x[3] * c1.z - y[3] * c1.w);
            b = make_float4(x[0] * c0.y + y[0] * c0.x, x[1] * c0.w + y[1] * c0.z, x[2] * c1.y + y[2] * c1.x, x[3] * c1.w + y[3] * c1.z);
        };
        clear();
        for (int t = t0; t < t1; ++t) {
            const i32x4 d = describe(t);
            const bool causal = on_limit(d);
            const float4 *rs = reinterpret_cast<const float4 *>(rot_seg + (int64_t)d.z * HALF) + 2 * hh;
            const float *kr = kb + ((int64_t)d.x + n) * D + 4 * hh, *vr = vb + (int64_t)d.x * D + v_at;
            f32x16 s, s1;                                // (two chains, as above)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = s1[r] = 0.f;
#pragma unroll 1
            for (int j = 0; j < NJ / 2; ++j) {           // the queries turned by -(segment start - stored base)
                float4 a, b;
                query(a, b, j);
                const float4 c0 = rs[4 * j], c1 = rs[4 * j + 1], x = *reinterpret_cast<const float4 *>(kr + 8 * j), y = *reinterpret_cast<const float4 *>(kr + 8 * j + HALF);
                s = MFMA_F32(x.x, a.x * c0.x + b.x * c0.y, s); s = MFMA_F32(x.y, a.y * c0.z + b.y * c0.w, s);
                s = MFMA_F32(x.z, a.z * c1.x + b.z * c1.y, s); s = MFMA_F32(x.w, a.w * c1.z + b.w * c1.w, s);
                s1 = MFMA_F32(y.x, b.x * c0.x - a.x * c0.y, s1); s1 = MFMA_F32(y.y, b.y * c0.z - a.y * c0.w, s1);
                s1 = MFMA_F32(y.z, b.z * c1.x - a.z * c1.y, s1); s1 = MFMA_F32(y.w, b.w * c1.z - a.w * c1.w, s1);
            }
            s += s1;
            softmax(s, L.scale_log2, d, causal);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const VV vv = *reinterpret_cast<const VV *>(vr + (8 * (r >> 2) + (r & 3)) * D);
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    float x = reinterpret_cast<const float *>(&vv)[i];
                    const bool skip = causal && !(fabsf(x) < INFINITY);
                    odd |= skip;
                    x = skip ? 0.f : x;
                    acc[i] = MFMA_F32(x, s[r], acc[i]);
                }
            }
        }
    }
}

template <int D>
__global__ __launch_bounds__(64 * NW, 1) void pc_attend_f32_kernel(PcLaunch L) { attend_f32<D, false>(L, PcSelf{}); }
// (the lists come first: the start of the kernel's arguments)
template <int D>
__global__ __launch_bounds__(64 * NW, 1) void pc_attend_f32_self_kernel(const PcArgBlob blob, PcLaunch L, PcSelf S) { attend_f32<D, true>(L, S); }

// The splits of a row added in order: one thread per (row, head, 4 dims), every split's sums and outputs requested before
// any is used (four at a time).
template <int D>
__global__ __launch_bounds__(256) void pc_merge_f32_kernel(const PcMergeRow *__restrict__ rows, const float *__restrict__ part_o,
                                                           const float *__restrict__ part_ml, float *__restrict__ out,
                                                           float *__restrict__ lse, int n_q_heads, int64_t n)
{
    const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (tid >= n) return;
    const int dim = 4 * (int)(tid % (D / 4));
    const int64_t pair = tid / (D / 4);
    const int h = (int)(pair % n_q_heads);
    const PcMergeRow mr = rows[pair / n_q_heads];
    float m = -INFINITY, l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < mr.n_splits; s0 += 4) {
        float2 ml[4];
        float4 a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ml[u] = make_float2(-INFINITY, 0.f);
            a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s0 + u < mr.n_splits) {
                const int64_t at = ((int64_t)mr.part_row0 + (int64_t)(s0 + u) * mr.n_q) * n_q_heads + h;
                ml[u] = *reinterpret_cast<const float2 *>(part_ml + at * 2);
                a[u] = *reinterpret_cast<const float4 *>(part_o + at * D + dim);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!(ml[u].x > -INFINITY)) { l += ml[u].y; continue; }         // saw nothing: a sum of 0 (or NaN, which stays)
            const float mn = fmaxf(m, ml[u].x), f = ex2(m - mn), w = ex2(ml[u].x - mn);
            o.x = fmaf(o.x, f, a[u].x * w); o.y = fmaf(o.y, f, a[u].y * w); o.z = fmaf(o.z, f, a[u].z * w); o.w = fmaf(o.w, f, a[u].w * w);
            l = fmaf(l, f, ml[u].y * w);
            m = mn;
        }
    }
    const int64_t at = (int64_t)mr.row * n_q_heads + h;
    if (l > 0.f) { o.x /= l; o.y /= l; o.z /= l; o.w /= l; }
    else o = make_float4(0.f, 0.f, 0.f, 0.f);
    float *dst = out + at * D + dim;
    dst[0] = o.x; dst[1] = o.y; dst[2] = o.z; dst[3] = o.w;
    if (lse && dim == 0) lse[at] = (l > 0.f) ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

void pc_launch_attend_f32(const PcLaunch &L, int n_items, int D, hipStream_t st)
{
    if (n_items <= 0) return;
    const unsigned grid = (unsigned)n_items * L.n_kv_heads, block = 64 * NW;
    if (D == 64) pc_attend_f32_kernel<64><<<grid, block, 0, st>>>(L);
    else pc_attend_f32_kernel<128><<<grid, block, 0, st>>>(L);
}

void pc_launch_attend_f32_self(const PcArgBlob &blob, const PcLaunch &L, const PcSelf &S, int n_items, int D, hipStream_t st)
{
    if (n_items <= 0) return;
    const unsigned grid = (unsigned)n_items * L.n_kv_heads, block = 64 * NW;
    if (D == 64) pc_attend_f32_self_kernel<64><<<grid, block, 0, st>>>(blob, L, S);
    else pc_attend_f32_self_kernel<128><<<grid, block, 0, st>>>(blob, L, S);
}

void pc_launch_merge_f32(const PcMergeRow *rows, int n_rows, const void *part_o, const float *part_ml, void *out, float *lse, int n_q_heads, int D,
                         hipStream_t st)
{
    const int64_t n = (int64_t)n_rows * n_q_heads * (D / 4);
    if (n <= 0) return;
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (D == 64) pc_merge_f32_kernel<64><<<grid, 256, 0, st>>>(rows, (const float *)part_o, part_ml, (float *)out, lse, n_q_heads, n);
    else pc_merge_f32_kernel<128><<<grid, 256, 0, st>>>(rows, (const float *)part_o, part_ml, (float *)out, lse, n_q_heads, n);
}
