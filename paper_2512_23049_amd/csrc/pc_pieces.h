// fp32 products on the bf16 matrix instructions: device helpers shared by the kernels of fp32 caches (gfx950).
#ifndef PC_PIECES_H_
#define PC_PIECES_H_

#include "pc_mfma_common.h"

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));

// Eight fp32 numbers as three bf16 pieces each, whose sum the number is (round, subtract, round, subtract, round).  A product
// of two bf16 numbers is exact in fp32, so six products of pieces, those whose orders sum to at most two, are a product of fp32
// numbers: what is left out is below 2^-24 of it, what rounding it to fp32 costs at most (a fifth of 2^-25 in the mean square).  Six bf16 MFMAs take
// 192 cycles for 32 x 32 x 16, the fp32 instruction 512.
// The pieces' exponents end at both ends: above 3.396e38 the first one is an infinity (the kernels look for what is not finite in their
// results), below 2^-110 the last ones fall below 2^-133, bf16's least number.  Operands are cut times UP where that costs nothing or little: then
// every fp32 number has its pieces, the subnormal ones too, and the upper end is at 5.2e33.
constexpr float UP = 0x1p16f;
__device__ __forceinline__ float4 up(float4 v) { return make_float4(v.x * UP, v.y * UP, v.z * UP, v.w * UP); }
struct Pieces { bf16x8 p[3]; };
// PIN: without it the compiler rounds the lower number of a pair a second time, by an instruction of its own, which takes fewer registers: the
// bf16 caches' gradient, whose walk of dq fills its 256 (20 of them in scratch with PIN, 180 -> 208 us), goes without.
template <bool PIN = true>
__device__ __forceinline__ void split2(float a, float b, uint32_t (&w)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        w[i] = pack_bf16(a, b);
        if constexpr (PIN) asm("" : "+v"(w[i]));
        a -= bf_lo(w[i]);
        b -= bf_hi(w[i]);
    }
}
template <bool PIN = true>
__device__ __forceinline__ Pieces split8(const float *v)
{
    uint32_t w[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j) split2<PIN>(v[2 * j], v[2 * j + 1], w[j]);
    Pieces r;
#pragma unroll
    for (int i = 0; i < 3; ++i) r.p[i] = __builtin_bit_cast(bf16x8, make_uint4(w[0][i], w[1][i], w[2][i], w[3][i]));
    return r;
}
#define MFMA_BF(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)
__device__ __forceinline__ f32x16 product(const Pieces &a, const bf16x8 (&b)[3], f32x16 c)     // small terms first
{
    c = MFMA_BF(a.p[2], b[0], c); c = MFMA_BF(a.p[0], b[2], c); c = MFMA_BF(a.p[1], b[1], c);
    c = MFMA_BF(a.p[1], b[0], c); c = MFMA_BF(a.p[0], b[1], c);
    return MFMA_BF(a.p[0], b[0], c);
}
// N times: a matrix instruction, then V vector ones
template <int N, int V>
__device__ __forceinline__ void beside()
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
}

// One 16-byte per lane direct load: lane l's bytes land at lds_wave_base + 16 l.  Assembly, so that the compiler keeps no
// record of the LDS write and does not drain every request in front of later LDS reads; completion is awaited with wait_vm0().
__device__ __forceinline__ void dma16(const void *gbase_uniform, unsigned lane_off, unsigned lds_wave_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(lds_wave_base), "v"(lane_off), "s"(gbase_uniform) : "memory", "m0");
}
__device__ __forceinline__ void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <typename T> __device__ __forceinline__ T from_lds(unsigned at) { return *reinterpret_cast<const __attribute__((address_space(3))) T *>((uintptr_t)at); }

// A wave's tile of 32 fp32 rows of D, brought to LDS by direct loads of whole rows (a lane that fetches its own row's pieces
// touches 32 lines an instruction: two cycles each of the CU's memory pipeline).  Chunk c (16 bytes) of row r sits at position
// c ^ (r % CHUNKS) of the row: 16 lanes that read one chunk of 16 rows hit different banks.
template <int D>
struct RowTile {
    static constexpr int BYTES = 32 * D * 4, CHUNKS = D / 4;
    unsigned lds, src;
    __device__ RowTile(unsigned char *mem, int lane) : lds((unsigned)(uintptr_t)mem),
        src((lane / CHUNKS) * (D * 4) + (((lane % CHUNKS) ^ (lane / CHUNKS)) << 4)) {}
    __device__ void request(const float *rows) const     // (wave uniform)
    {
        constexpr int STEP = 64 / CHUNKS;                // rows of an instruction
        unsigned src = this->src;
        asm volatile("" : "+v"(src));                    // (or the exclusive ors below wait in registers, or in scratch, from tile to tile)
#pragma unroll
        for (int i = 0; i < 32 / STEP; ++i) dma16(rows + STEP * i * D, src ^ (((STEP * i) % CHUNKS) << 4), lds + i * 1024);
    }
};

}  // namespace

#endif
