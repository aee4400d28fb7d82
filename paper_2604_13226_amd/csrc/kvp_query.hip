// kvp_query.hip -- K2: query-side RoPE + append; generic (any dtype, any head_dim)
// split-KV attention; K4: split-KV combine.  (Sec. 4.2.1 step 4; Fig. 2(d).)
#include "kvp_device.h"

#include <utility>

namespace kvp {

// ---------------------------------------------------------------------------------
// K2.  One thread per (query row, head, pair i): rotates Q and K_new from position 0 to
// ctx_len + t, writes the rotated Q to the workspace (store dtype), the rotated K_new and
// the raw V_new to cache rows ctx_len + t.
// ---------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a)
{
#pragma clang fp contract(off)
    const int half = a.d / 2;
    const int heads = a.n_q_heads + a.n_kv;
    const int64_t total = (int64_t)a.tot_q * heads * half;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        int i = (int)(idx % half);
        int64_t rh = idx / half;
        int hh = (int)(rh % heads);
        int row = (int)(rh / heads);
        int req = a.row_req[row];
        ReqMeta m = a.reqs[req];
        const int row_in_req = row - m.q_off;
        int pos = m.pos0 + row_in_req;            // the token's position
        const int cache_row = m.ctx_len + row_in_req;  // the cache row its K / V go to
        float c = 1.f, s = 0.f;
        if (!a.prerotated) {
            float2 t = a.cs[(int64_t)pos * half + i];
            c = t.x;
            s = t.y;
        }
        if (hh < a.n_q_heads) {
            int64_t o = ((int64_t)row * a.n_q_heads + hh) * a.d;
            const T *src = (const T *)a.q + o;
            T *dst = (T *)a.q_rot + o;
            float x = ld_elem(src + i), y = ld_elem(src + half + i);
            float xc = x * c, ys = y * s, yc = y * c, xs = x * s;
            st_elem(dst + i, (xc - ys) * a.q_scale);
            st_elem(dst + half + i, (yc + xs) * a.q_scale);
        } else {
            int h = hh - a.n_q_heads;
            int64_t o = ((int64_t)row * a.n_kv + h) * a.d;
            const T *ks = (const T *)a.k_new + o;
            const T *vs = (const T *)a.v_new + o;
            int64_t co = cache_row_off(a.cache, req, a.layer, h, cache_row, a.n_kv, a.d);
            T *kd = (T *)a.cache.k + co;
            T *vd = (T *)a.cache.v + co;
            float x = ld_elem(ks + i), y = ld_elem(ks + half + i);
            float xc = x * c, ys = y * s, yc = y * c, xs = x * s;
            st_elem(kd + i, xc - ys);
            st_elem(kd + half + i, yc + xs);
            vd[i] = vs[i];
            vd[half + i] = vs[half + i];
        }
    }
}

int launch_append(int dtype, const AppendArgs &a, void *stream)
{
    if (a.tot_q == 0) return 0;
    int64_t total = (int64_t)a.tot_q * (a.n_q_heads + a.n_kv) * (a.d / 2);
    unsigned blocks = (unsigned)((total + 255) / 256);
    if (blocks > 65536u) blocks = 65536u;
    if (dtype == 1) hipLaunchKernelGGL((append_kernel<bf16_t>), dim3(blocks), dim3(256), 0, (hipStream_t)stream, a);
    else hipLaunchKernelGGL((append_kernel<float>), dim3(blocks), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Generic attention: one wavefront per packed row, lanes own head_dim/64 columns
// (head_dim <= 256), online softmax over the item's kv range in fp32.  Slow but
// shape-agnostic: whatever the matrix-core kernels do not take.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T>
__global__ __launch_bounds__(256) void attention_generic_kernel(AttnArgs a)
{
    const AttnItem it = a.items[blockIdx.x];
    if (it.n_rows <= 0) return;  // padding item of the launch order
    const AttnGroup gp = a.groups[it.group];
    const ReqMeta rq = a.reqs[gp.req];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int d = a.d;
    const T *kc = (const T *)a.cache.k;
    const T *vc = (const T *)a.cache.v;

    for (int rr = wave; rr < gp.n_rows; rr += 4) {
        const int m = gp.m0 + rr;
        const int t = m / a.g, hq = gp.kv_head * a.g + m % a.g;
        const T *qp = (const T *)a.q_rot + ((int64_t)(rq.q_off + t) * a.n_q_heads + hq) * d;
        float q[4], o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int e = lane + 64 * j;
            q[j] = e < d ? ld_elem(qp + e) : 0.f;
            o[j] = 0.f;
        }
        float mx = -INFINITY, l = 0.f;
        int vis_end = rq.ctx_len + t + 1;  // causal among the query rows, full over the prefix
        int end = it.kv_end < vis_end ? it.kv_end : vis_end;
        // UB rows per trip: all their K and V loads are issued before the first is used, so a
        // trip costs one memory round trip instead of UB
        constexpr int UB = 8;
        for (int u0 = it.kv_begin; u0 < end; u0 += UB) {
            float kk[UB][4], v[UB][4];
#pragma unroll
            for (int i = 0; i < UB; ++i) {
                const int u = u0 + i < end ? u0 + i : end - 1;  // rows past the range repeat the last one (unused)
                const int64_t off = cache_row_off(a.cache, gp.req, a.layer, gp.kv_head, u, a.n_kv, d);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int e = lane + 64 * j;
                    kk[i][j] = e < d ? ld_elem(kc + off + e) : 0.f;
                    v[i][j] = e < d ? ld_elem(vc + off + e) : 0.f;
                }
            }
#pragma unroll
            for (int i = 0; i < UB; ++i) {
                if (u0 + i >= end) break;  // wave-uniform
                float part = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) part += q[j] * kk[i][j];
                float sc = wave_sum(part) * a.scale_log2e;
                float mn = fmaxf(mx, sc);
                float alpha = exp2f(mx - mn);  // exp2f(-inf) = 0 on the first row
                float p = exp2f(sc - mn);
                l = l * alpha + p;
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = o[j] * alpha + p * v[i][j];
                mx = mn;
            }
        }
        if (gp.n_splits == 1) {
            T *op = (T *)a.out + ((int64_t)(rq.q_off + t) * a.n_q_heads + hq) * d;
            float inv = 1.f / l;  // the row always sees itself, so l > 0
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int e = lane + 64 * j;
                if (e < d) st_elem(op + e, o[j] * inv);
            }
        } else {
            float *pp = (float *)((char *)a.partials + (int64_t)(gp.part0 + it.split) * part_slot_bytes(a.bm, d, 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int e = lane + 64 * j;
                if (e < d) pp[(int64_t)rr * d + e] = o[j];
            }
            if (lane == 0) {
                pp[(int64_t)a.bm * d + rr] = mx;
                pp[(int64_t)a.bm * d + a.bm + rr] = l;
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// K4.  Merge the splits of one group by log-sum-exp:
//   m = max m_i;  l = sum l_i 2^(m_i - m);  O = sum O~_i 2^(m_i - m) / l.
// A split that saw no visible row has m_i = -inf, l_i = 0 and contributes nothing.
// ---------------------------------------------------------------------------------
// fp32 rows that lie one behind the other (the fp32, the narrow and the generic kernel's, the MFMA kernel's at 64 columns):
// one wave per packed row.  A partial row is CPR pieces of 16 bytes, and the 64 lanes hold the pieces of
// G = 64 / CPR splits at a time.  The first NB pieces of every lane are requested before anything is known about
// the group.  Nothing of the merge passes through LDS: the maximum and the sum over the splits'
// (m, l) are lane permutes, a split's weight reaches its lanes by a broadcast within sixteen lanes (or a read into a
// scalar register), and the G partial sums of a column are added by half and quarter swaps that leave
// every lane NC / G columns of the row to write.
//
// Bound: latency -- a launch (1.6 us in a chain of empty kernels), the arguments, one trip for the
// partial rows, the merge.  A layer of a step, with shuffles through LDS for all of that, 8-byte loads, two-byte
// stores and the whole AttnArgs to fetch, and now: one token at 8K 13.3 -> 12.5 us (24 splits).  Up to eight
// splits had a kernel with a thread per piece and the (m, l) in LDS: fp32, 2.3K rows 35.2 -> 34.0 us; 64 columns, four
// paged requests 27.6 -> 26.9.
constexpr int COMBINE_ROWS = 4;         // rows (waves) per workgroup
constexpr int COMBINE_MAX_SPLITS = 64;  // the planner's bound on splits per group

struct CombineArgs {
    const char *partials;
    void *out;
    const AttnGroup *groups;
    int32_t slot_bytes, rows_bytes, part_stride, bm, n_q_heads, g;
    int32_t rows_first;  // combine_pieces_kernel: the row blocks run along blockIdx.x, the groups along y
};

__device__ __forceinline__ float opaque(float x) { asm volatile("" : "+v"(x)); return x; }
template <int CTRL> __device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// (the second operand is made opaque: given the same value twice, the compiler was seen to use the first result for both)
__device__ __forceinline__ void swap32(float &x, float &y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
    x = opaque(__builtin_bit_cast(float, (uint32_t)r[0]));
    y = opaque(__builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ void swap16(float &x, float &y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
    x = opaque(__builtin_bit_cast(float, (uint32_t)r[0]));
    y = opaque(__builtin_bit_cast(float, (uint32_t)r[1]));
}
template <typename F> __device__ __forceinline__ float over_lanes(float x, F f)  // f over all 64 lanes, in every lane
{
    x = f(x, dpp<0xB1>(x));   // lane ^ 1
    x = f(x, dpp<0x4E>(x));   // lane ^ 2
    x = f(x, dpp<0x141>(x));  // mirrored within eight
    x = f(x, dpp<0x140>(x));  // mirrored within sixteen
    float y = opaque(x);
    swap16(x, y);
    x = f(x, y);
    y = opaque(x);
    swap32(x, y);
    return f(x, y);
}
// the maximum over the lanes that have this one's place in their quad: of four quads, eight, or all sixteen
template <int QUADS> __device__ __forceinline__ float max_over_quads(float x)
{
    x = fmaxf(x, dpp<0x124>(x));  // turned by four within sixteen
    x = fmaxf(x, dpp<0x128>(x));  // and by eight
    if constexpr (QUADS > 4) {
        float y = opaque(x);
        swap16(x, y);
        x = fmaxf(x, y);
    }
    if constexpr (QUADS > 8) {
        float y = opaque(x);
        swap32(x, y);
        x = fmaxf(x, y);
    }
    return x;
}
// w of lane CPR * (this lane / CPR) + I
template <int CPR, int I> __device__ __forceinline__ float split_weight(float w, int sg)
{
    if constexpr (CPR == 16) return dpp<0x150 + I>(w);
    const float w0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), I));
    if constexpr (CPR == 64) return w0;
    const float w1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), 32 + I % 32));
    return sg ? w1 : w0;
}
template <typename P> __device__ __forceinline__ void add_piece(float (&acc)[16 / sizeof(P)], uint4 v, float w)
{
    if (w == 0.f) v = make_uint4(0u, 0u, 0u, 0u);  // (a split without visible rows, or none: it may hold anything)
    P e[16 / sizeof(P)];
    __builtin_memcpy(e, &v, 16);
#pragma unroll
    for (int j = 0; j < (int)(16 / sizeof(P)); ++j) acc[j] = __builtin_fmaf((float)e[j], w, acc[j]);
}
template <int CPR, int... I>
__device__ __forceinline__ void add_pieces(float (&acc)[4], const uint4 *v, float w, int sg, std::integer_sequence<int, I...>)
{
    (add_piece<float>(acc, v[I], split_weight<CPR, I>(w, sg)), ...);
}

template <typename T, int D, int NB>
__global__ __launch_bounds__(256) void combine_wave_kernel(CombineArgs a)
{
    constexpr int CPR = D / 4, G = 64 / CPR, NC = 4, NCO = NC / G;
    static_assert(CPR <= 64 && NB <= CPR && NCO >= 1, "shape");
    const int lane = threadIdx.x & 63, sg = lane / CPR, c = lane % CPR;
    const int rr = (int)blockIdx.y * COMBINE_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int stride = a.part_stride, rc = rr < a.bm ? rr : a.bm - 1;
    // Group gi's partial slots start at gi * stride, so the first loads below do not wait for
    // the group's record; slots and rows the group does not use hold stale bytes of the
    // workspace (in bounds: the addresses are clamped into the group's slots) and get weight zero.
    const char *base = a.partials + (int64_t)blockIdx.x * stride * a.slot_bytes;
    const int ms = G * c + sg;  // this lane's split
    float mi, li;
    {
        const float *ml = (const float *)(base + (int64_t)(ms < stride ? ms : stride - 1) * a.slot_bytes + a.rows_bytes) + rc;
        mi = ml[0];
        li = ml[a.bm];
    }
    const char *row = base + (int64_t)rc * (D * 4) + 16 * c;
    uint4 v[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int sp = G * i + sg;
        v[i] = *(const uint4 *)(row + (int64_t)(sp < stride ? sp : stride - 1) * a.slot_bytes);
    }
    const AttnGroup gp = a.groups[blockIdx.x];
    const int ns = gp.n_splits;
    if (ns <= 1 || rr >= gp.n_rows) return;
    if (ms >= ns) { mi = -INFINITY; li = 0.f; }
    const float mx = over_lanes(mi, [](float x, float y) { return fmaxf(x, y); });
    const float w = mi == -INFINITY ? 0.f : exp2f(mi - mx);
    const float inv = 1.f / over_lanes(li * w, [](float x, float y) { return x + y; });
    float acc[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[j] = 0.f;
    add_pieces<CPR>(acc, v, w, sg, std::make_integer_sequence<int, NB>{});
    constexpr int BATCH = 8;  // later pieces go out BATCH per lane at a time, all before the first is used
    for (int s0 = G * NB; s0 < ns; s0 += G * BATCH) {
        uint4 u[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int sp = s0 + G * i + sg;
            u[i] = *(const uint4 *)(row + (int64_t)(sp < ns ? sp : ns - 1) * a.slot_bytes);
        }
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int sp = s0 + G * i + sg;
            const float ws = __shfl(w, sg * CPR + (s0 / G + i < CPR ? s0 / G + i : CPR - 1), 64);
            add_piece<float>(acc, u[i], sp < ns ? ws : 0.f);
        }
    }
    int col = NC * c;
    if constexpr (G >= 2) {
        col += (lane >> 5) * (NC / 2);
#pragma unroll
        for (int j = 0; j < NC / 2; ++j) {
            swap32(acc[j], acc[j + NC / 2]);
            acc[j] += acc[j + NC / 2];
        }
    }
    if constexpr (G == 4) {
        col += ((lane >> 4) & 1) * (NC / 4);
#pragma unroll
        for (int j = 0; j < NC / 4; ++j) {
            swap16(acc[j], acc[j + NC / 4]);
            acc[j] += acc[j + NC / 4];
        }
    }
    const int m = gp.m0 + rr;
    const int t = m / a.g, hq = gp.kv_head * a.g + m % a.g;
    T o[NCO];
#pragma unroll
    for (int j = 0; j < NCO; ++j) st_elem(o + j, acc[j] * inv);
    T *op = (T *)a.out + ((int64_t)(gp.q_off + t) * a.n_q_heads + hq) * D + col;
    __builtin_memcpy(__builtin_assume_aligned(op, sizeof o), o, sizeof o);
}

// The MFMA kernel's rows: fp16 of 128 columns, scaled per row by a power of two that m and l carry along, or fp32 of 256.
// They lie as its accumulators do (part_piece_at), pieces of neighbouring rows next to each other: a workgroup merges
// 16 ZC pieces of four rows, a quad of lanes reads a piece of each, and wave w takes every fourth split from w on.  Each lane
// reads the (m, l) of its splits itself, and the sixteen lanes of a row read all splits' m between them: weights are relative to
// the group's maximum in every wave, so that the waves' sums, which pass through LDS once, only need adding.  (Relative to a
// wave's own they would overflow, or keep an infinity, where the split does not count.)  (A wave per row, as above, takes 64
// places of this layout with every load: 8K context, 27 splits, 26.6 us per layer of a step, so 26.1; with whole rows 26.3.)
template <typename P, int D, int NB, int ZC>
__global__ __launch_bounds__(256) void combine_pieces_kernel(CombineArgs a)
{
    constexpr int NC = 16 / (int)sizeof(P), W = 16 * NC * ZC;  // columns of a piece, and of a workgroup
    constexpr int RS = W + 4;  // (row stride in LDS: the four rows of a quad in banks of their own)
    __shared__ __attribute__((aligned(16))) float xo[4][4][RS];
    __shared__ float xl[4][4];
    constexpr int NM = (4 * NB + 15) / 16, QUADS = NB < 4 ? 4 * NB : 16;  // (up to eight splits, fewer quads hold all m)
    const int lane = threadIdx.x & 63, row = lane & 3, c = lane >> 2;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int stride = a.part_stride;
    // Eight neighbouring rows lie in the same lines: the two workgroups that read them are on one XCD (every eighth workgroup).
    const uint32_t x = blockIdx.x, gi = a.rows_first ? blockIdx.y : x;
    const int r0 = 4 * (int)(a.rows_first ? x / 16 * 16 + x % 8 * 2 + x / 8 % 2 : blockIdx.y);  // (a slot has a multiple of 64 rows)
    const char *base = a.partials + (int64_t)gi * stride * a.slot_bytes;
    const char *piece = base + part_piece_at(D * (int)sizeof(P), r0 + row, 16 * ZC * (int)blockIdx.z + c), *ml = base + a.rows_bytes + (r0 + row) * 8;
    float m[NM];
    float2 s[NB];
    uint4 v[NB][ZC];
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        const int sp = 16 * i + c % QUADS;
        m[i] = *(const float *)(ml + __umul24(sp < stride ? sp : stride - 1, a.slot_bytes));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int sp = 4 * i + wave;
        const int64_t at = (int64_t)(sp < stride ? sp : stride - 1) * a.slot_bytes;
        s[i] = *(const float2 *)(ml + at);
#pragma unroll
        for (int z = 0; z < ZC; ++z) v[i][z] = *(const uint4 *)(piece + at + 8192 * z);
    }
    const AttnGroup gp = a.groups[gi];
    const int ns = gp.n_splits;
    if (ns <= 1 || r0 >= gp.n_rows) return;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        if (16 * i + c % QUADS >= ns) m[i] = -INFINITY;
        mx = fmaxf(mx, m[i]);
    }
    mx = fmaxf(max_over_quads<QUADS>(mx), -3.4028235e38f);  // (finite, so that a split without visible rows has weight zero below)
    bool low = false;  // weights below 2^-126, for which the instruction alone gives zero
#pragma unroll
    for (int i = 0; i < NM; ++i) low |= m[i] - mx < -126.f && m[i] > -INFINITY;
    float wt[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (4 * i + wave >= ns) s[i] = make_float2(-INFINITY, 0.f);
        wt[i] = __builtin_amdgcn_exp2f(s[i].x - mx);
    }
    if (__any(low)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) wt[i] = exp2f(opaque(s[i].x) - mx);
    }
    float l = 0.f, acc[ZC][NC] = {};
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        l += s[i].y * wt[i];
#pragma unroll
        for (int z = 0; z < ZC; ++z) add_piece<P>(acc[z], v[i][z], wt[i]);
    }
#pragma unroll
    for (int z = 0; z < ZC; ++z) {
        float *x = &xo[wave][row][16 * NC * z + (NC == 8 ? 16 * (c >> 1) + 4 * (c & 1) : 4 * c)];
        *(float4 *)x = make_float4(acc[z][0], acc[z][1], acc[z][2], acc[z][3]);
        if constexpr (NC == 8) *(float4 *)(x + 8) = make_float4(acc[z][4], acc[z][5], acc[z][6], acc[z][7]);
    }
    if (c == 0) xl[wave][row] = l;
    __syncthreads();
    const int rr = r0 + wave;  // each wave writes one of the rows
    if (rr >= gp.n_rows) return;
    constexpr int NO = W / 64;  // columns that a lane writes
    float out[NO] = {}, sum = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        float o[NO];
        __builtin_memcpy(o, __builtin_assume_aligned(&xo[w][wave][NO * lane], 4 * NO), 4 * NO);
        sum += xl[w][wave];
#pragma unroll
        for (int j = 0; j < NO; ++j) out[j] += o[j];
    }
    const float inv = 1.f / sum;
    const int pr = gp.m0 + rr;
    const int tok = pr / a.g, hq = gp.kv_head * a.g + pr % a.g;
    bf16_t *op = (bf16_t *)a.out + ((int64_t)(gp.q_off + tok) * a.n_q_heads + hq) * D + W * (int)blockIdx.z + NO * lane;
    bf16_t u[NO];
#pragma unroll
    for (int j = 0; j < NO; ++j) u[j] = f32_to_bf16(out[j] * inv);
    __builtin_memcpy(__builtin_assume_aligned(op, sizeof u), u, sizeof u);
}

// Other head dims (the generic attention kernel's): a wave per row, a column per lane, split by split.
template <typename T>
__global__ __launch_bounds__(256) void combine_any_kernel(AttnArgs a)
{
    const int lane = threadIdx.x & 63;
    const int rr = (int)blockIdx.y * COMBINE_ROWS + (threadIdx.x >> 6);
    const AttnGroup gp = a.groups[blockIdx.x];
    const int d = a.d, ns = gp.n_splits;
    if (ns <= 1 || rr >= gp.n_rows) return;
    const int64_t slot_b = part_slot_bytes(a.bm, d, 0);
    const char *base = (const char *)a.partials + (int64_t)blockIdx.x * a.part_stride * slot_b;
    const float *ml = (const float *)(base + part_rows_bytes(a.bm, d, 0)) + rr;
    const float *row = (const float *)base + (int64_t)rr * d;
    const int64_t slot = slot_b / 4;  // in floats
    float mi = -INFINITY, lv = 0.f;
    if (lane < ns) { mi = ml[lane * slot]; lv = ml[lane * slot + a.bm]; }
    float mx = mi;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    const float w = (mi == -INFINITY) ? 0.f : exp2f(mi - mx);
    const float inv = 1.f / wave_sum(lv * w);
    const int m = gp.m0 + rr;
    const int t = m / a.g, hq = gp.kv_head * a.g + m % a.g;
    T *op = (T *)a.out + ((int64_t)(gp.q_off + t) * a.n_q_heads + hq) * d;
    for (int e0 = 0; e0 < d; e0 += 64) {  // (every lane runs every trip: the weights travel by lane shuffles)
        const int e = e0 + lane;
        const bool on = e < d;
        float acc = 0.f;
        for (int sp = 0; sp < ns; ++sp) {
            const float ws = __shfl(w, sp, 64), x = row[sp * slot + (on ? e : 0)];
            if (ws != 0.f) acc += x * ws;  // (a split without visible rows has weight 0 and may hold anything)
        }
        if (on) st_elem(op + e, acc * inv);
    }
}

static CombineArgs combine_args(const AttnArgs &a, int f16)
{
    CombineArgs c;
    c.partials = (const char *)a.partials;
    c.out = a.out;
    c.groups = a.groups;
    c.slot_bytes = (int32_t)part_slot_bytes(a.bm, a.d, f16);
    c.rows_bytes = (int32_t)part_rows_bytes(a.bm, a.d, f16);
    c.part_stride = a.part_stride;
    c.bm = a.bm;
    c.n_q_heads = a.n_q_heads;
    c.g = a.g;
    c.rows_first = 0;
    return c;
}

// Pieces requested up front: for the launch's largest split count, rounded up.  (A second round trip costs 2 us; the
// variant for 24 splits is 0.2 us slower than that for 16 where 12 are needed.  256 columns of fp32: no more
// than 24, the pieces fill the registers.)
template <typename T, int D> static void launch_combine_wave(const AttnArgs &a, dim3 grid, hipStream_t st)
{
    constexpr int G = 64 * 4 / D;
    const CombineArgs c = combine_args(a, 0);
    if (a.part_stride <= 4) launch(combine_wave_kernel<T, D, 4 / G>, grid, dim3(256), 0, st, c);
    else if (a.part_stride <= 8) launch(combine_wave_kernel<T, D, 8 / G>, grid, dim3(256), 0, st, c);
    else if (a.part_stride <= 16) launch(combine_wave_kernel<T, D, 16 / G>, grid, dim3(256), 0, st, c);
    else if (a.part_stride <= 24 || D == 256) launch(combine_wave_kernel<T, D, 24 / G>, grid, dim3(256), 0, st, c);
    else if (a.part_stride <= 32) launch(combine_wave_kernel<T, D, (D < 256 ? 32 : 24) / G>, grid, dim3(256), 0, st, c);
    else launch(combine_wave_kernel<T, D, (D < 256 ? 40 : 24) / G>, grid, dim3(256), 0, st, c);
}

template <typename P, int D, int ZC> static void launch_combine_zc(const CombineArgs &c, dim3 grid, hipStream_t st)
{
    if (c.part_stride <= 4) launch(combine_pieces_kernel<P, D, 1, ZC>, grid, dim3(256), 0, st, c);
    else if (c.part_stride <= 8) launch(combine_pieces_kernel<P, D, 2, ZC>, grid, dim3(256), 0, st, c);
    else if (c.part_stride <= 16) launch(combine_pieces_kernel<P, D, 4, ZC>, grid, dim3(256), 0, st, c);
    else if constexpr (ZC == 1) {
        if (c.part_stride <= 24) launch(combine_pieces_kernel<P, D, 6, ZC>, grid, dim3(256), 0, st, c);
        else if (c.part_stride <= 32) launch(combine_pieces_kernel<P, D, 8, ZC>, grid, dim3(256), 0, st, c);
        else if (c.part_stride <= 40) launch(combine_pieces_kernel<P, D, 10, ZC>, grid, dim3(256), 0, st, c);
        else launch(combine_pieces_kernel<P, D, 16, ZC>, grid, dim3(256), 0, st, c);
    }
}

template <typename P, int D> static void launch_combine_pieces(const AttnArgs &a, dim3 grid, hipStream_t st)
{
    CombineArgs c = combine_args(a, sizeof(P) == 2);
    // 256 columns: all 64 pieces of the rows in one workgroup for up to sixteen splits (of more they would fill the registers), from
    // three workgroups to a CU on; fewer are dealt out in quarters.  (Per layer, in one and in quarters: 16 / 4 heads, 3K rows, 8
    // query rows 22.1 and 21.1 us; six requests of 32 / 8 heads, 13 query rows, 624 workgroups 27.9 and 27.6; eight with 12, 768, 50.6 and
    // 51.5; eight with 39, 4096, 87.2 and 93.7.)
    constexpr int Z = D * (int)sizeof(P) / 256;
    const bool quarters = Z > 1 && (a.part_stride > 16 || (int64_t)grid.x * grid.y < 768);
    // As many groups as a multiple of eight: a group's workgroups are on one XCD, that of its items where those keep to one.  Others:
    // sixteen workgroups take 64 rows of a group, two on each XCD.  (Group by group there too, two XCDs read each line: per layer, 3.4K
    // rows of 28 / 4 heads with 76 query rows 18.0 us, so 15.6, and by whole rows, a wave each, 16.2; 16 / 2 heads, 145 query
    // rows over 6K 22.9, 19.9 and 20.5; in place, 160 over 3K of 28 / 4 heads 26.4, 23.2 and 24.5.)
    c.rows_first = grid.x % 8 != 0 && grid.x < 65536;
    if (c.rows_first) grid = dim3((grid.y + 15) / 16 * 16, grid.x);
    if (quarters) grid.z = Z;
    if (quarters) launch_combine_zc<P, D, 1>(c, grid, st);
    else launch_combine_zc<P, D, Z>(c, grid, st);
}

template <typename T> static void launch_combine_fp32_rows(const AttnArgs &a, dim3 grid, hipStream_t st)
{
    if (a.d == 64) launch_combine_wave<T, 64>(a, grid, st);
    else if (a.d == 128) launch_combine_wave<T, 128>(a, grid, st);
    else if (a.d == 256) launch_combine_wave<T, 256>(a, grid, st);
    else hipLaunchKernelGGL((combine_any_kernel<T>), grid, dim3(256), 0, st, a);
}

int launch_combine(int dtype, const AttnArgs &a, void *stream)
{
    if (a.n_groups == 0) return 0;
    const int rows = a.max_group_rows > 0 && a.max_group_rows < a.bm ? a.max_group_rows : a.bm;
    hipStream_t st = (hipStream_t)stream;
    if (a.part_stride > COMBINE_MAX_SPLITS) return (int)hipErrorInvalidValue;
    const dim3 grid((unsigned)a.n_groups, (unsigned)((rows + COMBINE_ROWS - 1) / COMBINE_ROWS));
    if (a.part_pieces) {  // the MFMA kernel's partial rows (bf16 stores only)
        if (dtype != 1 || a.part_f16 != (a.d == 128)) return (int)hipErrorInvalidValue;
        if (a.d == 128) launch_combine_pieces<_Float16, 128>(a, grid, st);
        else if (a.d == 256) launch_combine_pieces<float, 256>(a, grid, st);
        else return (int)hipErrorInvalidValue;
    } else if (dtype == 1) {
        launch_combine_fp32_rows<bf16_t>(a, grid, st);
    } else {
        launch_combine_fp32_rows<float>(a, grid, st);
    }
    return (int)hipGetLastError();
}

int launch_attention_mfma(const AttnArgs &a, void *stream);  // kvp_attention_mfma.hip
int launch_attention_f32(const AttnArgs &a, void *stream);   // kvp_attention_f32.hip
int launch_attention_narrow(const AttnArgs &a, void *stream);  // kvp_attention_narrow.hip

int launch_attention(int dtype, const AttnArgs &a, int kernel_kind, void *stream)
{
    if (a.n_items == 0) return 0;
    if (kernel_kind == ATTN_MFMA) return launch_attention_mfma(a, stream);
    if (kernel_kind == ATTN_NARROW) return dtype == 1 ? launch_attention_narrow(a, stream) : (int)hipErrorInvalidValue;
    if (kernel_kind == ATTN_F32) return dtype == 0 ? launch_attention_f32(a, stream) : (int)hipErrorInvalidValue;
    if (dtype == 1) hipLaunchKernelGGL((attention_generic_kernel<bf16_t>), dim3(a.n_items), dim3(256), 0, (hipStream_t)stream, a);
    else hipLaunchKernelGGL((attention_generic_kernel<float>), dim3(a.n_items), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace kvp
