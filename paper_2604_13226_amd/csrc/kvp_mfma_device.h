// kvp_mfma_device.h -- what the bf16 matrix-core attention kernels share: tile loads straight into
// LDS, lane exchanges, the rotation of a chunk pair.
#pragma once
#include "kvp_device.h"

namespace kvp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void *lds_void_p;
typedef __attribute__((address_space(1))) const void *glb_void_p;

__device__ __forceinline__ uint32_t pack_bf16_hw(float a, float b)
{
    floatx2 f = {a, b};
    bf16x2 v = __builtin_convertvector(f, bf16x2);  // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}

// wait until at most n of this wave's vector-memory operations are outstanding
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// x of lane l and of lane l ^ 32, without a trip through the LDS crossbar: the half-swap
// leaves lanes 0..31 of the first result with x[l], of the second with x[l + 32], and the
// upper lanes with the same pair.  The second operand is made opaque to the compiler: given
// the same value twice it was seen to use the first result for both.
__device__ __forceinline__ void xhalf_pair(float x, float &lo, float &hi)
{
    uint32_t u = __builtin_bit_cast(uint32_t, x), w = u;
    asm volatile("" : "+v"(w));
    const auto r = __builtin_amdgcn_permlane32_swap(u, w, false, false);
    uint32_t r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1));
    lo = __builtin_bit_cast(float, r0);
    hi = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ float xhalf_max(float x)
{
    float lo, hi;
    xhalf_pair(x, lo, hi);
    return fmaxf(lo, hi);
}
__device__ __forceinline__ float xhalf_sum(float x)
{
    float lo, hi;
    xhalf_pair(x, lo, hi);
    return lo + hi;
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// HBM -> LDS without staging registers: each lane names its own 16 global bytes (a
// wave-uniform base plus a per-lane 32-bit byte offset); the wavefront's 64 x 16 B land
// contiguously at the wave-uniform LDS byte address lds_addr.  Written as inline assembly so
// that the compiler's wait-count insertion does not treat every later LDS read as dependent
// on every outstanding load: the waits are explicit (wait_vmcnt + wg_barrier) in the loop.
// `stream`: the rows will not be read again soon by anyone (no other work item shares them
// through the L2): the load carries the non-temporal hint, which a plain streaming read of HBM
// was measured to reward with 7.0 instead of 6.3 TB/s.
// (A compile-time choice: selected at run time, every load became a branch between two copies of
// the instruction, and the tile loads could no longer be issued between the matrix instructions.)
template <bool STREAM>
__device__ __forceinline__ void load_to_lds_16(const void *sbase, uint32_t voff, uint32_t lds_addr)
{
    if (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}
// A 16-byte global load whose wait is ours to place: before the first use of a load it knows,
// the compiler waits for every load issued up to there, the tile loads included (it cannot
// count those), so the query-side loads are made opaque to it as well and waited for by count.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4_t load16_nowait(const void *p)
{
    u32x4_t v;
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(v) : "v"(p) : "memory");
    return v;
}
// a pointer the program knows to be wave-uniform, made so for the compiler too
__device__ __forceinline__ const char *uniform_ptr(const void *p)
{
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char *)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
// Stores that go on to memory at once (sc1), for what a later launch reads on another XCD.  (A line that stays dirty in the L2
// leaves it at the end of the launch, all of them together.)  `bytes` from `base` on, both wave-uniform, can be written.
struct ThroughStore {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ ThroughStore(void *base, int bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(base), 0, bytes, 0x00027000)) {}
    __device__ __forceinline__ void put16(int at, const u32x4_t &v) const { __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, at, 0, 16); }
};
// same with a full per-lane address
__device__ __forceinline__ void load_to_lds_16(const void *gptr, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}

// If the running reference maximum lags the true row maximum by at most this many
// powers of two, the accumulators are not rescaled (probabilities then reach at most 2^8,
// harmless in fp32 accumulators and scale-free in bf16); the final (m, l, O) stay consistent
// because all three are relative to the same reference.
constexpr float RESCALE_SLACK = 8.f;

// v with zeros in place of its infinities and NaNs; `dropped` becomes non-zero if there are any
__device__ __forceinline__ bf16x8 drop_nonfinite(const bf16x8 &v, uint32_t &dropped)
{
    const uint4 u = __builtin_bit_cast(uint4, v);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t bad = ((w[i] & 0x7F80u) == 0x7F80u ? 0xFFFFu : 0u) | ((w[i] & 0x7F800000u) == 0x7F800000u ? 0xFFFF0000u : 0u);
        dropped |= bad;
        w[i] &= ~bad;
    }
    return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// the largest magnitudes, as bits, of the even and of the odd elements: 0x7F80 and above are infinities and NaNs
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void max_magnitude(ushort2_t &m, const uint4 &v)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(ushort2_t, w[i] & 0x7FFF7FFFu));
}
// the float of these bits if it is an infinity or a NaN, else zero
__device__ __forceinline__ float nonfinite_only(uint32_t bits) { return (bits & 0x7F800000u) == 0x7F800000u ? __uint_as_float(bits) : 0.f; }

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// One 16-byte chunk pair of a head vector rotated by the (cos, sin) pairs in cs4 (Eq. 1): element i of
// the low chunk pairs with element i of the high chunk.  Products and sums are rounded separately, as
// in the gather kernel.
__device__ __forceinline__ void rotate_chunk_pair(const uint4 &ulo, const uint4 &uhi, const float4 (&cs4)[4], uint4 &olo, uint4 &ohi)
{
#pragma clang fp contract(off)
    const uint32_t wl[4] = {ulo.x, ulo.y, ulo.z, ulo.w}, wh[4] = {uhi.x, uhi.y, uhi.z, uhi.w};
    uint32_t ol[4], oh[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float lo2[2], hi2[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float x = __uint_as_float(u ? (wl[j] & 0xFFFF0000u) : (wl[j] << 16));
            const float y = __uint_as_float(u ? (wh[j] & 0xFFFF0000u) : (wh[j] << 16));
            const float c = u ? cs4[j].z : cs4[j].x, sn = u ? cs4[j].w : cs4[j].y;
            const float xc = x * c, ys = y * sn, yc = y * c, xs = x * sn;
            lo2[u] = xc - ys;
            hi2[u] = yc + xs;
        }
        ol[j] = (uint32_t)f32_to_bf16(lo2[0]) | ((uint32_t)f32_to_bf16(lo2[1]) << 16);
        oh[j] = (uint32_t)f32_to_bf16(hi2[0]) | ((uint32_t)f32_to_bf16(hi2[1]) << 16);
    }
    olo = make_uint4(ol[0], ol[1], ol[2], ol[3]);
    ohi = make_uint4(oh[0], oh[1], oh[2], oh[3]);
}

// The same for the query, which nothing is compared with bit for bit: sums are fused.  SCALED: cs4 holds
// the pairs times the score scale already (where one lane scales them for four), else the results are
// multiplied.
template <bool SCALED>
__device__ __forceinline__ void rotate_query_pair(const uint4 &ulo, const uint4 &uhi, const float4 (&cs4)[4], float scale, uint4 &olo, uint4 &ohi)
{
    const float k = SCALED ? 1.f : scale;
    const uint32_t wl[4] = {ulo.x, ulo.y, ulo.z, ulo.w}, wh[4] = {uhi.x, uhi.y, uhi.z, uhi.w};
    uint32_t ol[4], oh[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x0 = __uint_as_float(wl[j] << 16), x1 = __uint_as_float(wl[j] & 0xFFFF0000u);
        const float y0 = __uint_as_float(wh[j] << 16), y1 = __uint_as_float(wh[j] & 0xFFFF0000u);
        const float l0 = __builtin_fmaf(x0, cs4[j].x, -(y0 * cs4[j].y)), l1 = __builtin_fmaf(x1, cs4[j].z, -(y1 * cs4[j].w));
        const float h0 = __builtin_fmaf(y0, cs4[j].x, x0 * cs4[j].y), h1 = __builtin_fmaf(y1, cs4[j].z, x1 * cs4[j].w);
        ol[j] = SCALED ? pack_bf16_hw(l0, l1) : pack_bf16_hw(l0 * k, l1 * k);
        oh[j] = SCALED ? pack_bf16_hw(h0, h1) : pack_bf16_hw(h0 * k, h1 * k);
    }
    olo = make_uint4(ol[0], ol[1], ol[2], ol[3]);
    ohi = make_uint4(oh[0], oh[1], oh[2], oh[3]);
}
__device__ __forceinline__ float4 scale_cs(const float4 &v, float scale, float sin_scale)
{
    return make_float4(v.x * scale, v.y * sin_scale, v.z * scale, v.w * sin_scale);
}

// v of lane J of this lane's group of four
template <int J> __device__ __forceinline__ float4 quad_lane(const float4 &v)
{
    auto bc = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x55 * J, 0xF, 0xF, true)); };
    return make_float4(bc(v.x), bc(v.y), bc(v.z), bc(v.w));
}

enum { SRC_CONTIG = 0, SRC_PAGED = 1, SRC_PACKETS = 2 };

}  // namespace kvp
