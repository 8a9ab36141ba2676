// Attention of fp32 caches on the fp32 matrix instructions (gfx950).
//
// The transposed problem of the bf16 kernels: scores S^T = K~ . Q^T (rows = 32 keys, columns = 32 (query row, head) pairs
// of one KV head), O^T = V^T . P^T, both with v_mfma_f32_32x32x2_f32, whose products and sums are plain fp32.  Its operands
// are one float a lane (row or column lane % 32, index lane / 32 of the two), its result has 16 rows a lane:
// 8 (r / 4) + 4 (lane / 32) + r % 4.  Register r of the scores is therefore the right operand of the second product for the
// two keys of that register, and neither product needs its operands in any particular order of the summed index: a lane
// reads K and V straight from memory, 16 bytes at a time, and no operand passes through LDS but the queries' master copy.
//
// A workgroup is 8 waves, two per SIMD, over the same 32 columns; each walks a contiguous eighth of the item's tiles and
// the results meet in LDS.  A tile is 128 MFMAs of 64 cycles (D = 128, 64 at D = 64), 3.4 us, against 32 KB of loads in
// small pieces: one wave's loads, softmax and turns of the queries run under the other's matrix work.  A call with few columns is split over the tiles as well (see
// pc_plan_and_stage) and pc_merge_f32_kernel adds the parts.  Bound: the fp32 matrix rate, 157 TFLOP/s nominal.
//
// 200 rows over 1400 keys, 32/8 heads, D = 128: 78 us (1115 us with one wave per (row, head), a lane per key and an FMA per
// product); 40 us of them are matrix work, the rest is the start (work item, queries, first tile: one round trip to
// memory after the other), the turns of the queries and 56 idle compute units of 256.  32 rows over 160 keys, 4/2 heads,
// D = 64: 16.6 -> 12.6 us, all of it latency.
#include "pc_mfma_common.h"

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
template <> struct Vec<2> { using type = float2; };
template <> struct Vec<4> { using type = float4; };

}  // namespace

template <int D>
__global__ __launch_bounds__(64 * NW, 1) void pc_attend_f32_kernel(PcLaunch L)
{
    constexpr int NJ = D / 8, VW = D / 32, HALF = D / 2, PITCH = D + 4;
    __shared__ __attribute__((aligned(16))) float s_q[32 * PITCH];          // the columns' queries turned by their positions
    __shared__ __attribute__((aligned(16))) float s_acc[NW][32 * PITCH];
    __shared__ float s_m[NW][32], s_l[NW][32];

    const int kh = blockIdx.x % L.n_kv_heads;          // consecutive workgroups (one per XCD) take different KV heads
    const PcItem item = L.items[blockIdx.x / L.n_kv_heads];
    const PcCallDesc cd = L.calls[item.call];
    const int g = L.n_q_heads / L.n_kv_heads;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int n_cols = cd.n_q * g;
    const int col0 = item.unit0 * 32;       // column c: query row c / g, head c % g of the group

    // this wave's contiguous run of tiles
    const int per_wave = (item.tile_end - item.tile_begin + NW - 1) / NW;
    const int t0 = item.tile_begin + wave * per_wave, t1 = min(item.tile_end, t0 + per_wave);
    const PcTile *tab = L.tiles + item.tile_tab0;
    auto describe = [&](int t) {
        const int tc = __builtin_amdgcn_readfirstlane(max(0, min(t, item.tile_end - 1)));
        if (item.tile_end <= 0) return (i32x4){0, 0, 0, 0};                 // a call that sees nothing has no table
        return *reinterpret_cast<const __attribute__((address_space(4))) i32x4 *>(reinterpret_cast<uintptr_t>(tab + tc));
    };
    i32x4 next = describe(t0);                           // {slot0, key0, seg, valid | flags}

    for (int e = threadIdx.x; e < 32 * (HALF / 4); e += 64 * NW) {          // 4 pairs of a column a step
        const int c = e / (HALF / 4), i = 4 * (e % (HALF / 4));
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
        if (col0 + c < n_cols) {
            const int col = col0 + c;
            const int64_t R = cd.q_off + col / g;
            const float *q = (const float *)L.q + (R * L.n_q_heads + kh * g + col % g) * D;
            const float4 x = make_float4(q[i], q[i + 1], q[i + 2], q[i + 3]);
            const float4 y = make_float4(q[i + HALF], q[i + HALF + 1], q[i + HALF + 2], q[i + HALF + 3]);
            const float4 *rot = reinterpret_cast<const float4 *>(L.rot_q + R * HALF + i);
            const float4 c0 = rot[0], c1 = rot[1];
            a = make_float4(x.x * c0.x - y.x * c0.y, x.y * c0.z - y.y * c0.w, x.z * c1.x - y.z * c1.y, x.w * c1.z - y.w * c1.w);
            b = make_float4(x.x * c0.y + y.x * c0.x, x.y * c0.w + y.y * c0.z, x.z * c1.y + y.z * c1.x, x.w * c1.w + y.w * c1.z);
        }
        *reinterpret_cast<float4 *>(s_q + c * PITCH + i) = a;
        *reinterpret_cast<float4 *>(s_q + c * PITCH + i + HALF) = b;
    }
    __syncthreads();

    using VV = typename Vec<VW>::type;
    const float *kb = (const float *)L.k_store + (int64_t)kh * L.slots * D + n * D + 4 * hh;          // lane's key row, dims 8 j + 4 hh + 0..3
    const float *vb = (const float *)L.v_store + (int64_t)kh * L.slots * D + 4 * hh * D + VW * n;     // lane's dims VW n + 0..VW-1
    const int row = (col0 + n) / g;
    const int self_lim = cd.self_len - cd.n_q + row;     // last own token this column sees
    const int lo_lim = cd.self_len - cd.n_q + col0 / g;              // ... the item's first column
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 acc[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    float4 q[NJ];
    int cur = -1;
    bool odd = false;                                    // an Inf or NaN was left out
    for (int t = t0; t < t1; ++t) {
        const i32x4 d = next;
        if (t + 1 < t1) next = describe(t + 1);
        // K and V come in pieces of 16 registers, two of them in flight
        float4 k[2][4];
        const float *kr = kb + (int64_t)d.x * D;
        auto load_k = [&](int p) {
#pragma unroll
            for (int j = 0; j < 4; ++j) k[p & 1][j] = *reinterpret_cast<const float4 *>(kr + 8 * (4 * p + j));
        };
        load_k(0); load_k(1);
        __builtin_amdgcn_sched_barrier(0);
        if (cur < 0 || (d.w & PC_TILE_FRESH)) {          // turn the queries by -(segment start - stored base)
            cur = d.z;
            const float4 *rs = reinterpret_cast<const float4 *>(L.rot_seg + (int64_t)(cd.seg_off + cur) * HALF) + 2 * hh;
#pragma unroll
            for (int j = 0; j < NJ / 2; ++j) {
                const float4 a = *reinterpret_cast<const float4 *>(s_q + n * PITCH + 8 * j + 4 * hh);
                const float4 b = *reinterpret_cast<const float4 *>(s_q + n * PITCH + HALF + 8 * j + 4 * hh);
                const float4 c0 = rs[4 * j], c1 = rs[4 * j + 1];
                q[j] = make_float4(a.x * c0.x + b.x * c0.y, a.y * c0.z + b.y * c0.w, a.z * c1.x + b.z * c1.y, a.w * c1.z + b.w * c1.w);
                q[j + NJ / 2] = make_float4(b.x * c0.x - a.x * c0.y, b.y * c0.z - a.y * c0.w, b.z * c1.x - a.z * c1.y, b.w * c1.z - a.w * c1.w);
            }
        }
        f32x16 s, s1;                                    // (two chains of D / 2 terms round less than one of D)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = s1[r] = 0.f;
#pragma unroll
        for (int p = 0; p < NJ / 4; ++p) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x16 &c = (j & 1) ? s1 : s;
                const float4 x = k[p & 1][j], y = q[4 * p + j];
                c = MFMA_F32(x.x, y.x, c);
                c = MFMA_F32(x.y, y.y, c);
                c = MFMA_F32(x.z, y.z, c);
                c = MFMA_F32(x.w, y.w, c);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (p + 2 < NJ / 4) load_k(p + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        constexpr int VP = 16 / VW;                      // keys (registers of the scores) of a piece of V
        VV v[2][VP];
        const float *vr = vb + (int64_t)d.x * D;         // register r: key 8 (r / 4) + 4 hh + r % 4
        auto load_v = [&](int p) {
#pragma unroll
            for (int i = 0; i < VP; ++i) { const int r = VP * p + i; v[p & 1][i] = *reinterpret_cast<const VV *>(vr + (8 * (r >> 2) + (r & 3)) * D); }
        };
        load_v(0);
        if constexpr (VP < 16) load_v(1);
        __builtin_amdgcn_sched_barrier(0);
        s += s1;
        const int valid = d.w & 0xFF, key0 = d.y;
        const bool self = (d.w & PC_TILE_SELF) != 0;
        const bool causal = self && key0 + valid - 1 > lo_lim;      // some column does not see some key
        const int lim = self ? min(valid, self_lim - key0 + 1) : valid;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] *= L.scale_log2;
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
        // A probability of zero takes a key out of the second product only while its value is finite.  What lies behind a
        // message's last token is (the store is kept that way), but a later token of the new message is the caller's own
        // data: in a tile on the causal limit an Inf or NaN is left out here and added at the end, for the columns that
        // see its key.
#pragma unroll
        for (int p = 0; p < 16 / VP; ++p) {
            float x[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = reinterpret_cast<const float *>(&v[p & 1][0])[e];
            if (causal)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const bool ok = fabsf(x[e]) < INFINITY;
                    odd |= !ok;
                    x[e] = ok ? x[e] : 0.f;
                }
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e % VW] = MFMA_F32(x[e], s[VP * p + e / VW], acc[e % VW]);
            __builtin_amdgcn_sched_barrier(0);
            if ((p + 2) * VP < 16) load_v(p + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // the waves' results: element (i, r) of a lane is dim VW (8 (r / 4) + 4 hh + r % 4) + i of column n
    l_run += other_half(l_run);
    if (hh == 0) { s_m[wave][n] = m_run; s_l[wave][n] = l_run; }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        VV o;
        float *x = reinterpret_cast<float *>(&o);
#pragma unroll
        for (int i = 0; i < VW; ++i) x[i] = acc[i][r];
        *reinterpret_cast<VV *>(&s_acc[wave][n * PITCH + VW * (8 * (r >> 2) + 4 * hh + (r & 3))]) = o;
    }
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {         // (the probability has no say in an Inf or NaN; a wave's own LDS accesses are in order)
        for (int t = t0; t < t1; ++t) {
            const i32x4 d = describe(t);
            if (!(d.w & PC_TILE_SELF) || d.y + (d.w & 0xFF) - 1 <= lo_lim) continue;
            const int lim = min(d.w & 0xFF, self_lim - d.y + 1);
            const float *vr = (const float *)L.v_store + ((int64_t)kh * L.slots + d.x) * D;
            for (int e = hh; e < lim * D; e += 2) {
                const float x = vr[e];
                if (!(fabsf(x) < INFINITY)) s_acc[wave][n * PITCH + e % D] += x;
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * (D / 4); e += 64 * NW) {
        const int c = e / (D / 4), dim = 4 * (e % (D / 4));
        const int col = col0 + c;
        if (col >= n_cols) break;                        // (columns ascend with e)
        float mm = s_m[0][c], l = 0.f;
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, s_m[w][c]);
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        if (mm > -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (!(s_m[w][c] > -INFINITY)) { l += s_l[w][c]; continue; }        // saw nothing: a sum of 0 (or NaN, which stays)
                const float f = ex2(s_m[w][c] - mm);
                const float4 a = *reinterpret_cast<const float4 *>(&s_acc[w][c * PITCH + dim]);
                o.x = fmaf(a.x, f, o.x); o.y = fmaf(a.y, f, o.y); o.z = fmaf(a.z, f, o.z); o.w = fmaf(a.w, f, o.w);
                l = fmaf(s_l[w][c], f, l);
            }
        }
        const int r = col / g, h = kh * g + col % g;
        if (cd.n_splits == 1) {
            const int64_t at = (int64_t)(cd.q_off + r) * L.n_q_heads + h;
            if (l > 0.f) { o.x /= l; o.y /= l; o.z /= l; o.w /= l; }
            else o = make_float4(0.f, 0.f, 0.f, 0.f);    // nothing visible (or a NaN score)
            float *out = (float *)L.out + at * D + dim;
            out[0] = o.x; out[1] = o.y; out[2] = o.z; out[3] = o.w;
            if (L.lse && dim == 0) L.lse[at] = (l > 0.f) ? (mm + log2f(l)) * 0.6931471805599453f : -INFINITY;
        } else {
            const int64_t at = ((int64_t)cd.part_off + (int64_t)item.split * cd.n_q + r) * L.n_q_heads + h;
            *reinterpret_cast<float4 *>((float *)L.part_o + at * D + dim) = o;
            if (dim == 0) { L.part_ml[at * 2] = mm; L.part_ml[at * 2 + 1] = l; }
        }
    }
}

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

void pc_launch_merge_f32(const PcMergeRow *rows, int n_rows, const void *part_o, const float *part_ml, void *out, float *lse, int n_q_heads, int D,
                         hipStream_t st)
{
    const int64_t n = (int64_t)n_rows * n_q_heads * (D / 4);
    if (n <= 0) return;
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (D == 64) pc_merge_f32_kernel<64><<<grid, 256, 0, st>>>(rows, (const float *)part_o, part_ml, (float *)out, lse, n_q_heads, n);
    else pc_merge_f32_kernel<128><<<grid, 256, 0, st>>>(rows, (const float *)part_o, part_ml, (float *)out, lse, n_q_heads, n);
}
