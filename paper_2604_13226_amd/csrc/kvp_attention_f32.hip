// kvp_attention_f32.hip -- K3 for fp32 stores (head_dim 64, 128 or 256): query-prefill attention on
// the fp32 matrix instructions (Sec. 4.2.1 step 4; Fig. 2(d)).
//
// Bound: the fp32 matrix pipe (64 cycles per 32x32x2 MFMA, 157 TFLOP/s over the chip): a 32-row tile of
// K and V costs a wave 2 x D/2 of them, 8192 cycles at head_dim 128, against 32 KB to fetch.  That
// leaves time enough to take K and V straight into registers, with no LDS and no barrier in the
// loop, and one wave per SIMD hides its loads under its own matrix work.
//
// One workgroup = 4 wavefronts = one work item: up to 32 packed (query token, query head) rows of
// one KV head over one kv range.  All four waves own the same 32 rows and take every fourth 32-row
// tile of the range, so a range is four times longer than a wave's share of it: a quarter of the
// partial rows that four row waves over shorter ranges would write (the row blocks of a head
// re-read its tiles through the L2: 16 bytes per cycle and CU, a quarter of what it delivers).
// Their (m, l, O) are merged through LDS at the end.
//
//   S^T = K Q^T      v_mfma_f32_32x32x2_f32; a k-step takes columns 8 j + i and 8 j + 4 + i (the lane
//                    halves h = 0, 1), so K and Q come as 16-byte pieces: lane (n, h) holds columns
//                    8 j + 4 h .. +3 of row n
//   O^T += V^T P^T   P^T is the accumulator itself: register r of lane half h is kv row
//                    8 (r / 4) + 4 h + r % 4, so the k-step of register r multiplies those two rows
//                    of V; block i of the output holds columns VW R + i (R the matrix row), so one
//                    piece of VW neighbouring columns per lane feeds VW blocks
//
// The query side of the layer is part of it: every workgroup rotates its own query rows, and those
// whose range reaches the query rows append K_new / V_new first.  (Several may: same bytes.)
//
// Measured (2.9K rows of context, 32 query rows, 32 / 8 heads of 128 columns): 27 us per layer, of which
// the three tiles of a wave are 12; one wave per row with fp32 vector arithmetic and a lane
// reduction per score took 1062.  Error against float64 there: 2.0e-7 of the result, 7.0e-7 before.
// 256 columns spill 34 to 36 registers (140 to 148 bytes of scratch per lane) and take 52 us per layer over
// the same rows with 16 / 4 heads, 873 before.
#include "kvp_device.h"

#include <type_traits>

namespace kvp {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int F32_WAVES = 4;
constexpr int F32_TILE = 32;  // kv rows per tile

// Row stride of a wave's O in LDS (floats): 4 past D, so that the 16-byte writes of lanes in
// neighbouring rows fall into different banks.
__host__ __device__ constexpr int f32_lds_stride(int d) { return d + 4; }
__host__ __device__ constexpr int f32_lds_floats(int d) { return F32_WAVES * 32 * f32_lds_stride(d) + 2 * F32_WAVES * 32; }

__device__ __forceinline__ float comp(const float4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

template <int D, bool PAGED>
__global__ __launch_bounds__(64 * F32_WAVES, 1) void attention_f32_kernel(AttnArgs a)
{
    constexpr int NK = D / 8;               // 16-byte pieces of a K / Q row per lane
    constexpr int EB = D / 32;              // 32-column blocks of the output
    constexpr int VW = EB < 4 ? EB : 4;     // neighbouring columns of V per piece
    constexpr int NP = EB / VW;             // pieces per V row and lane
    static_assert(D == 64 || D == 128 || D == 256, "shape");
    extern __shared__ __attribute__((aligned(16))) float f32_lds[];
    const AttnItem it = a.items[blockIdx.x];
    if (it.n_rows <= 0) return;  // padding item of the launch order
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;

    // element offset of cache row `row` (PAGED: by the item's block ids in LDS)
    int *blk_ids = (int *)(f32_lds + f32_lds_floats(D));
    const int shift = a.cache.block_shift, blk0 = it.kv_begin >> shift;
    const int n_blk = ((it.kv_end - 1) >> shift) - blk0 + 1;
    if (PAGED) {
        for (int i = tid; i < n_blk; i += 64 * F32_WAVES) blk_ids[i] = a.cache.block_table[(int64_t)it.req * a.cache.max_blocks + blk0 + i];
        __syncthreads();
    }
    const int64_t head_base = PAGED ? (int64_t)a.layer * a.cache.layer_stride
                                    : (int64_t)it.req * a.cache.req_stride + (int64_t)a.layer * a.cache.layer_stride + (int64_t)it.kv_head * a.cache.t_cap * D;
    auto row_off = [&](int row) -> int64_t {
        if (!PAGED) return head_base + (int64_t)row * D;
        const int b = blk_ids[(row >> shift) - blk0];
        return head_base + ((((int64_t)b * a.n_kv + it.kv_head) << shift) + (row & ((1 << shift) - 1))) * D;
    };

    // ---- append: K_new rotated to its position, V_new as it is, before any tile is read
    const int tail_lo = it.kv_begin > it.ctx_len ? it.kv_begin - it.ctx_len : 0;
    const int n_tail = it.kv_end - it.ctx_len - tail_lo;  // > 0 only for items that reach the query rows
    if (n_tail > 0) {
#pragma clang fp contract(off)  // separately rounded products and sums, as the gather kernel
        constexpr int UPR = D / 8;  // units of 4 columns and their partners per row
        for (int u = tid; u < n_tail * UPR; u += 64 * F32_WAVES) {
            const int qr = tail_lo + u / UPR, e = 4 * (u % UPR);
            const int64_t src = ((int64_t)(it.q_off + qr) * a.n_kv + it.kv_head) * D + e, dst = row_off(it.ctx_len + qr) + e;
            const float4 x = *(const float4 *)((const float *)a.k_new + src), y = *(const float4 *)((const float *)a.k_new + src + D / 2);
            const float4 v0 = *(const float4 *)((const float *)a.v_new + src), v1 = *(const float4 *)((const float *)a.v_new + src + D / 2);
            float4 cs01 = make_float4(1.f, 0.f, 1.f, 0.f), cs23 = cs01;
            if (!a.prerotated) {
                const float4 *cs = (const float4 *)(a.cs + (int64_t)(it.pos0 + qr) * (D / 2) + e);
                cs01 = cs[0];
                cs23 = cs[1];
            }
            float4 lo, hi;
            float p, q;
            p = x.x * cs01.x; q = y.x * cs01.y; lo.x = p - q; p = y.x * cs01.x; q = x.x * cs01.y; hi.x = p + q;
            p = x.y * cs01.z; q = y.y * cs01.w; lo.y = p - q; p = y.y * cs01.z; q = x.y * cs01.w; hi.y = p + q;
            p = x.z * cs23.x; q = y.z * cs23.y; lo.z = p - q; p = y.z * cs23.x; q = x.z * cs23.y; hi.z = p + q;
            p = x.w * cs23.z; q = y.w * cs23.w; lo.w = p - q; p = y.w * cs23.z; q = x.w * cs23.w; hi.w = p + q;
            *(float4 *)((float *)a.cache.k + dst) = lo;
            *(float4 *)((float *)a.cache.k + dst + D / 2) = hi;
            *(float4 *)((float *)a.cache.v + dst) = v0;
            *(float4 *)((float *)a.cache.v + dst + D / 2) = v1;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's stores have reached the L2
        __syncthreads();                     // ... and so have every other wave's
    }

    // ---- tiles: rows past the range repeat its last row (their scores are masked)
    const int n_tiles = (it.kv_end - it.kv_begin + F32_TILE - 1) / F32_TILE;
    // Loads run KA pieces (of NK) and VA rows (of 16) ahead of the MFMAs that use them: the whole tile
    // where the registers hold it, a quarter of it (2048 cycles of matrix work) at 256 columns.
    constexpr int KA = D == 256 ? NK / 4 : NK, VA = D == 256 ? 4 : 16;
    auto k_row = [&](int ti) -> const float * {
        const int row = it.kv_begin + ti * F32_TILE + n;
        return (const float *)a.cache.k + row_off(row < it.kv_end ? row : it.kv_end - 1) + 4 * h;
    };
    float4 kr[KA];
    float4 vr[VA][NP];
    auto load_v = [&](int ti, int r) {
        const int row = it.kv_begin + ti * F32_TILE + 8 * (r >> 2) + 4 * h + (r & 3);
        const float *p = (const float *)a.cache.v + row_off(row < it.kv_end ? row : it.kv_end - 1) + VW * n;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            if (VW == 4) {
                vr[r % VA][q] = *(const float4 *)(p + 128 * q);
            } else {
                const float2 t = *(const float2 *)p;
                vr[r % VA][q] = make_float4(t.x, t.y, 0.f, 0.f);
            }
        }
    };
    if (wave < n_tiles) {
        const float *kp = k_row(wave);
#pragma unroll
        for (int j = 0; j < KA; ++j) kr[j] = *(const float4 *)(kp + 8 * j);
    }

    // ---- this lane's query row: B operand of S^T = K Q^T, rotated, times log2(e) / sqrt(d)
    const bool row_ok = n < it.n_rows;
    const int m = it.m0 + (row_ok ? n : 0);
    const int t = m / a.g, hq = it.kv_head * a.g + m % a.g;
    const int vis = row_ok ? it.ctx_len + t + 1 : 0;         // kv rows [0, vis) are visible
    const int limit = vis < it.kv_end ? vis : it.kv_end;
    const int wave_limit = it.ctx_len + it.m0 / a.g + 1;     // the smallest `vis` of the block (rows are ordered by token)
    float4 qr[NK];
    {
        const float *qp = (const float *)a.q + ((int64_t)(it.q_off + t) * a.n_q_heads + hq) * D + 4 * h;
#pragma unroll
        for (int j = 0; j < NK; ++j) qr[j] = *(const float4 *)(qp + 8 * j);
        const float4 *cs = (const float4 *)(a.cs + (int64_t)(a.prerotated ? 0 : it.pos0 + t) * (D / 2) + 4 * h);  // (position 0 rotates nothing)
        const float sc = row_ok ? a.scale_log2e : 0.f;
#pragma unroll
        for (int j = 0; j < NK / 2; ++j) {
            const float4 c01 = cs[4 * j], c23 = cs[4 * j + 1], x = qr[j], y = qr[j + NK / 2];
            qr[j] = make_float4((x.x * c01.x - y.x * c01.y) * sc, (x.y * c01.z - y.y * c01.w) * sc,
                                (x.z * c23.x - y.z * c23.y) * sc, (x.w * c23.z - y.w * c23.w) * sc);
            qr[j + NK / 2] = make_float4((y.x * c01.x + x.x * c01.y) * sc, (y.y * c01.z + x.y * c01.w) * sc,
                                         (y.z * c23.x + x.z * c23.y) * sc, (y.w * c23.z + x.w * c23.w) * sc);
        }
    }

    f32x16 oacc[EB];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[eb][r] = 0.f;
    float m_i = -INFINITY, l_i = 0.f;
    constexpr bool ALL_FINITE = D == 256;  // every tile that way (two copies of the loop body do not fit the registers)
    bool dropped = false;  // infinities or NaNs of V were left out
    for (int ti = wave; ti < n_tiles; ti += F32_WAVES) {
#pragma unroll
        for (int r = 0; r < VA; ++r) load_v(ti, r);  // arrive under the S MFMAs
        const float *kp = k_row(ti);
        const float *kn = k_row(ti + F32_WAVES < n_tiles ? ti + F32_WAVES : ti);  // (the last tile loads itself again, from the L2)
        __builtin_amdgcn_sched_barrier(0);
        // (four partial sums over the columns, two at 256: a chain of 64 additions each would round
        // further from the exact score than the generic kernel's tree of lanes)
        constexpr int NS = D == 256 ? 2 : 4;
        f32x16 sp[NS];
#pragma unroll
        for (int c = 0; c < NS; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) sp[c][r] = 0.f;
#pragma unroll
        for (int j = 0; j < NK; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sp[i % NS] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(kr[j % KA], i), comp(qr[j], i), sp[i % NS], 0, 0, 0);
            kr[j % KA] = *(const float4 *)(j + KA < NK ? kp + 8 * (j + KA) : kn + 8 * (j + KA - NK));
            __builtin_amdgcn_sched_barrier(0);
        }
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = NS == 4 ? (sp[0][r] + sp[1][r]) + (sp[2 % NS][r] + sp[3 % NS][r]) : sp[0][r] + sp[1][r];

        const int kv0 = it.kv_begin + ti * F32_TILE;
        const bool masked = kv0 + F32_TILE > wave_limit || kv0 + F32_TILE > it.kv_end;  // wave-uniform: last tiles only
        if (masked) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kv0 + 8 * (r >> 2) + 4 * h + (r & 3) >= limit) s[r] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = fmaxf(m_i, fmaxf(mx, __shfl_xor(mx, 32, 64)));
        const float ref = mx == -INFINITY ? 0.f : mx;
        if (__any(mx > m_i)) {
            const float alpha = __builtin_amdgcn_exp2f(m_i - ref);  // 0 for a row's first visible tile
            l_i *= alpha;
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[eb][r] *= alpha;
            m_i = mx;
        }
        float p[16], sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            p[r] = __builtin_amdgcn_exp2f(s[r] - ref);
            sum += p[r];
        }
        l_i += sum;
        // A masked tile's zero probabilities times an infinity or NaN of V would be NaN: there such elements
        // stay out of the matrix product (as zeros) and are added at the end to the rows that see them.
        uint32_t bad = 0;
        auto pv = [&](auto drop) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (decltype(drop)::value) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int eb = 0; eb < EB; ++eb) {
                    float v = comp(vr[r % VA][eb / VW], eb % VW);
                    if (decltype(drop)::value) {
                        // all ones if the exponent is: in integer arithmetic, a compare mask per element is a scalar pair
                        uint32_t nf = 0u - ((__builtin_amdgcn_ubfe(__float_as_uint(v), 23, 8) + 1u) >> 8);
                        asm("" : "+v"(nf));
                        bad |= nf;
                        v = __uint_as_float(__float_as_uint(v) & ~nf);
                    }
                    oacc[eb] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, p[r], oacc[eb], 0, 0, 0);
                }
                if (VA < 16 && r + VA < 16) {
                    load_v(ti, r + VA);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (ALL_FINITE || masked) {
            pv(std::true_type{});
            dropped |= __any(bad != 0);
        } else {
            pv(std::false_type{});
        }
    }
    l_i += __shfl_xor(l_i, 32, 64);  // the lane halves saw different kv rows

    // ---- merge the four waves' (m, l, O) and write the rows
    constexpr int LS = f32_lds_stride(D);
    float *xo = f32_lds + wave * 32 * LS, *xm = f32_lds + F32_WAVES * 32 * LS, *xl = xm + F32_WAVES * 32;
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float *o = xo + n * LS + 32 * VW * q + VW * (8 * (r >> 2) + 4 * h + (r & 3));
            if (VW == 4) *(float4 *)o = make_float4(oacc[VW * q][r], oacc[VW * q + 1][r], oacc[(VW * q + 2) % EB][r], oacc[(VW * q + 3) % EB][r]);
            else *(float2 *)o = make_float2(oacc[0][r], oacc[1][r]);
        }
    if (h == 0) {
        xm[wave * 32 + n] = m_i;
        xl[wave * 32 + n] = l_i;
    }
    dropped = __syncthreads_or(dropped);
    const int seen_end = wave_limit < it.kv_end ? wave_limit : it.kv_end;  // the masked tiles start with the tile this row is in
    const int masked0 = it.kv_begin + (!ALL_FINITE && seen_end > it.kv_begin ? (seen_end - it.kv_begin) / F32_TILE * F32_TILE : 0);
    for (int u = tid; u < it.n_rows * (D / 4); u += 64 * F32_WAVES) {
        const int rr = u / (D / 4), e = 4 * (u % (D / 4));
        float mm = -INFINITY, l = 0.f;
#pragma unroll
        for (int w = 0; w < F32_WAVES; ++w) mm = fmaxf(mm, xm[w * 32 + rr]);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < F32_WAVES; ++w) {
            const float mw = xm[w * 32 + rr];
            const float wt = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - mm);
            const float4 o = *(const float4 *)(f32_lds + (w * 32 + rr) * LS + e);
            l += xl[w * 32 + rr] * wt;
            if (wt != 0.f) { acc.x += o.x * wt; acc.y += o.y * wt; acc.z += o.z * wt; acc.w += o.w * wt; }
        }
        if (dropped) {
            const int end = it.ctx_len + (it.m0 + rr) / a.g + 1 < it.kv_end ? it.ctx_len + (it.m0 + rr) / a.g + 1 : it.kv_end;
#pragma unroll 1
            for (int kv = masked0; kv < end; ++kv) {
                const float4 x = *(const float4 *)((const float *)a.cache.v + row_off(kv) + e);
                acc.x += __builtin_fabsf(x.x) < INFINITY ? 0.f : x.x;
                acc.y += __builtin_fabsf(x.y) < INFINITY ? 0.f : x.y;
                acc.z += __builtin_fabsf(x.z) < INFINITY ? 0.f : x.z;
                acc.w += __builtin_fabsf(x.w) < INFINITY ? 0.f : x.w;
            }
        }
        if (it.part_slot < 0) {
            const int mr = it.m0 + rr;
            const float inv = 1.f / l;  // the row always sees itself, so l > 0
            float *op = (float *)a.out + ((int64_t)(it.q_off + mr / a.g) * a.n_q_heads + it.kv_head * a.g + mr % a.g) * D + e;
            *(float4 *)op = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        } else {
            float *pp = (float *)((char *)a.partials + (int64_t)it.part_slot * part_slot_bytes(a.bm, D, 0));
            *(float4 *)(pp + (int64_t)rr * D + e) = acc;
            if (e == 0) {
                pp[(int64_t)a.bm * D + rr] = mm;
                pp[(int64_t)a.bm * D + a.bm + rr] = l;
            }
        }
    }
}

template <int D, bool PAGED> static int launch_f32(const AttnArgs &a, void *stream)
{
    constexpr int lds_bytes = f32_lds_floats(D) * 4 + (PAGED ? MFMA_MAX_ITEM_BLOCKS * 4 : 0);
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)attention_f32_kernel<D, PAGED>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    hipLaunchKernelGGL((attention_f32_kernel<D, PAGED>), dim3(a.n_items), dim3(64 * F32_WAVES), lds_bytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_attention_f32(const AttnArgs &a, void *stream)
{
    if (a.bm != ATTN_F32_BM) return (int)hipErrorInvalidValue;
    const bool paged = a.cache.layout != 0;
    if (a.d == 64) return paged ? launch_f32<64, true>(a, stream) : launch_f32<64, false>(a, stream);
    if (a.d == 128) return paged ? launch_f32<128, true>(a, stream) : launch_f32<128, false>(a, stream);
    if (a.d == 256) return paged ? launch_f32<256, true>(a, stream) : launch_f32<256, false>(a, stream);
    return (int)hipErrorInvalidValue;
}

}  // namespace kvp
