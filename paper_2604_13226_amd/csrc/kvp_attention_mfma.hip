// kvp_attention_mfma.hip -- K3: query-prefill attention on the bf16 matrix cores
// (Sec. 4.2.1 step 4; Fig. 2(d): full over the packet prefix, causal among the query rows).
//
// One workgroup = 4 wavefronts = one work item: rows [m0, m0+128) of the packed
// (query token, query head) rows that share one KV head, over one kv range (split-KV).
// Wave w owns 32 rows.  K/V tiles of 64 rows travel HBM -> LDS directly
// (global_load_lds_dwordx4, no staging registers) through a ring of STAGES tiles, so
// STAGES-1 tiles are in flight while one is being consumed.  Per tile:
//
//   S^T = K Q^T      v_mfma_f32_32x32x16_bf16, A = K rows from LDS (16-byte reads),
//                    B = Q^T held in registers for the whole item
//   online softmax   a lane owns one query row (a column of S^T): row max / row sum are
//                    in-lane reductions plus one exchange with lane ^ 32
//   O^T += V^T P^T   A = V^T read out of the row-major V tile with the transposing LDS
//                    read (ds_read_b64_tr_b16), B = P^T taken from the S^T accumulators in
//                    place: the kv order inside each 16-row k-step is whatever the
//                    accumulator layout gives, applied to both operands.
//
// LDS tiles are unpadded (a direct load writes 64 lanes x 16 B contiguously); bank
// conflicts are avoided by choosing WHICH 16-byte chunk of a row each lane fetches:
// K row r keeps logical chunk c at physical chunk c ^ (r & 15), V row r at c ^ 4 (r & 3) (64
// columns, two rows to a pass over the banks: c ^ (r / 2 & 7) and c ^ 4 (r / 2 & 1)).
//
// The kernel also does the query side of the layer (Sec. 4.2.1 step 4): every workgroup
// rotates its own 128 query rows to positions ctx_len + t in registers (the RoPE partner of
// element e is e + 64, which the MFMA operand layout keeps in the same lane), and the
// workgroups whose kv range reaches into the query rows first rotate K_new, write it and
// V_new to the cache rows ctx_len + t, and only then start loading tiles.  Several
// workgroups may write the same rows: they write the same bytes.
//
// HBM traffic: every K/V row of the range is read once per group of 128 packed rows.
#include "kvp_mfma_device.h"

namespace kvp {

constexpr int BN = 64;   // kv rows per tile
constexpr int stage_bytes(int d) { return 2 * BN * d * 2; }  // K tile then V tile

// A tile record of the in-place path, read through the scalar cache: the records are written by
// the host before the launch and never by a kernel, and the index is the same in every lane.  (As
// an ordinary load this was a vector load, and the wait for it -- placed by the compiler, who cannot
// count the tile loads in flight -- drained the whole prefetch ring at every tile.)
__device__ __forceinline__ AttnTile load_tile_record(const AttnTile *tiles, int idx)
{
    typedef const __attribute__((address_space(4))) int32_t *const_i32_p;
    const_i32_p p = (const_i32_p)(uintptr_t)(tiles + __builtin_amdgcn_readfirstlane(idx));
    int32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = p[i];
    AttnTile t;
    __builtin_memcpy(&t, w, sizeof t);
    return t;
}
static_assert(sizeof(AttnTile) == 8 * sizeof(int32_t), "eight words");

// A micro-benchmark that includes this file with -DKVP_TIMING gets per-workgroup time stamps and
// per-wave phase totals through two file-scope pointers it sets itself; the library is never
// built that way, and its kernel arguments are the same in either build.
#ifdef KVP_TIMING
__device__ unsigned long long *kvp_timing_stamps;  // [item][32]
__device__ unsigned long long *kvp_timing_phases;  // [item][8 waves][8]
#define KVP_STAMP(slot) do { if (threadIdx.x == 0 && (slot) < 32 && kvp_timing_stamps) kvp_timing_stamps[blockIdx.x * 32 + (slot)] = wall_clock64(); } while (0)
// per-wave cycle totals of the tile loop's phases
#define KVP_PHASE_DECL unsigned long long ph_acc[6] = {0, 0, 0, 0, 0, 0}, ph_last = __builtin_readcyclecounter()
#define KVP_PHASE(i) do { const unsigned long long t_ = __builtin_readcyclecounter(); ph_acc[i] += t_ - ph_last; ph_last = t_; } while (0)
#define KVP_PHASE_WRITE do { if ((threadIdx.x & 63) == 0 && kvp_timing_phases) for (int i_ = 0; i_ < 6; ++i_) kvp_timing_phases[(blockIdx.x * 8 + (threadIdx.x >> 6)) * 8 + i_] = ph_acc[i_]; } while (0)
#else
#define KVP_STAMP(slot) do {} while (0)
#define KVP_PHASE_DECL do {} while (0)
#define KVP_PHASE(i) do {} while (0)
#define KVP_PHASE_WRITE do {} while (0)
#endif

// The query is held rotated and (128 columns) multiplied by log2(e)/sqrt(d), so S = K Q^T is in log2
// units.  The S accumulators start at -m_ref: after the MFMAs they hold s - m_ref and the
// probabilities are exp2 of them with no further arithmetic.
//
// SRC_CONTIG / SRC_PAGED: an item's [kv_begin, kv_end) are cache rows.
// SRC_PACKETS: no cache exists; [kv_begin, kv_end) index a.tiles, each tile up to 64 rows of
// one stored packet (read in place from the arena) or of the query rows (rotated K_new in
// a.k_tail, V_new as given).  The keys of a stored packet stay at their local positions;
// instead the query is rotated by (ctx_len + t) - Delta_j for that packet's tiles, which
// gives the same scores (Eq. 1: scores depend on the position difference only).
//
// NW wavefronts per workgroup in KS groups of RW = NW / KS; a wave owns 32 packed rows, a
// group owns BM = 32 RW rows, and all NW waves share the loading of every K/V tile.
//   NW 4, KS 1, 2 stages: two workgroups share a CU (small row blocks, many items);
//   NW 8, KS 1, 4 stages: each K/V row is fetched once per 256 packed rows, three tiles in
//                         flight, one workgroup per CU;
//   NW 8, KS 2, 4 stages: 128 rows, the two groups take alternate tiles of the item's range
//                         (an in-workgroup split-KV that halves the serial chain of a
//                         latency-bound item) and merge their (m, l, O) through LDS.
template <int D, int STAGES, int SRC, int NW, int KS, bool NTL, bool QUAD>
__device__ __forceinline__ void attention_body(const AttnArgs &a)
{
    constexpr int ROW_BYTES = D * 2;
    constexpr int TILE_BYTES = BN * ROW_BYTES;  // of K, same for V
    constexpr int STAGE_BYTES = 2 * TILE_BYTES;
    constexpr int CH = D / 8;      // 16-byte chunks per row
    constexpr int RPI = 64 / CH;   // rows one load instruction of a wave fills
    constexpr int NKS = D / 16;    // k-steps of S^T = K Q^T
    constexpr int EB = D / 32;     // 32-column blocks of O
    constexpr int RW = NW / KS;    // waves per group (a group owns 32 RW rows)
    constexpr int NT = 64 * NW;    // threads
    constexpr int NI = BN / RPI / NW;  // K (and V) load instructions per wave per tile
    constexpr int PR = STAGES / KS - 1;  // rounds (of KS tiles) loaded ahead
    static_assert(STAGES % KS == 0 && PR >= 1, "stages");
    // Head dims other than 128: a probability goes into the product as two bf16 numbers, its leading eight
    // bits and the rest (16 bits together); the row sum and the partial rows are fp32.  The query is rotated
    // only, and the scores are scaled as they leave the matrix cores (one multiplication per score): scaled
    // before it is rounded to bf16, a query that came rotated, or a column that turns so slowly that
    // its values hardly change, would be rounded where the product can take it exactly.
    constexpr bool SPLIT_P = D != 128;
    const float q_scale = SPLIT_P ? 1.f : a.scale_log2e, s_scale = SPLIT_P ? a.scale_log2e : 1.f;
    const float above = RESCALE_SLACK / s_scale;  // the slack in the accumulators' units
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    KVP_STAMP(0);
    const AttnItem it = a.inl.n ? attn_inline_item(a.inl, blockIdx.x, a.n_kv, a.part_stride) : a.items[blockIdx.x];
    if (it.n_rows <= 0) return;  // padding item of the launch order
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_r = wave % RW, grp = wave / RW;  // row wave inside its group, group
    const int n = lane & 31, h = lane >> 5;
    const int g = a.g;

    const bf16_t *kc = (const bf16_t *)a.cache.k;
    const bf16_t *vc = (const bf16_t *)a.cache.v;
    const int n_tiles = SRC == SRC_PACKETS ? it.kv_end - it.kv_begin : (it.kv_end - it.kv_begin + BN - 1) / BN;

    // Paged layout: block ids come through the scalar cache, like the tile records above.  (They were kept in LDS, fetched
    // behind a barrier and read there in front of every load instruction: per layer of a step, 3.4K rows 16.1 -> 15.5 us, 8K
    // 27.8 -> 27.25, four requests of 64 columns 23.7 -> 23.2 with the quads below; long launches within 1 %.)
    typedef const __attribute__((address_space(4))) int32_t *const_i32_p;
    const const_i32_p blk_ids = SRC == SRC_PAGED ? (const_i32_p)(uintptr_t)uniform_ptr(a.cache.block_table + (int64_t)it.req * a.cache.max_blocks) : nullptr;
    // contiguous layout: wave-uniform byte address of the item's first K / V row
    const int64_t contig_off = SRC == SRC_CONTIG
                                   ? (int64_t)it.req * a.cache.req_stride + (int64_t)a.layer * a.cache.layer_stride +
                                         ((int64_t)it.kv_head * a.cache.t_cap + it.kv_begin) * D
                                   : 0;
    const char *k_item = (const char *)(kc + contig_off);
    const char *v_item = (const char *)(vc + contig_off);
    const int64_t paged_base = (int64_t)a.layer * a.cache.layer_stride;
    // rows of the query's own V (a.v_new) for this head; packets: and of its K (rotated, in a.k_tail)
    const int64_t tail_off = ((int64_t)it.q_off * a.n_kv + it.kv_head) * D;

    // direct HBM -> LDS load of tile tj: wave w, instruction i fills tile rows
    // RPI (NW i + w) .. + RPI - 1 (1 KiB contiguous in LDS); lane l owns slot (row + l / CH, chunk l % CH)
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
    const int slot_row = lane / CH, slot_chunk = lane % CH;
    // tile row r keeps logical chunk c of K at chunk c ^ k_swz(r), of V at c ^ 4 v_swz(r)
    auto k_swz = [](int r) -> int { return D == 64 ? (r >> 1) & 7 : r & 15; };
    auto v_swz = [](int r) -> int { return D == 64 ? (r >> 1) & 1 : r & 3; };
    // logical chunks this lane fetches; the same for every instruction of a wave while NW RPI is a multiple of 16
    const int k_chunk0 = slot_chunk ^ k_swz(RPI * wave + slot_row), v_chunk = slot_chunk ^ (4 * v_swz(RPI * wave + slot_row));
    const int last_tile_rows = it.kv_end - it.kv_begin - (n_tiles - 1) * BN;  // 1..64 (cache modes)
    // The loads of tile tj: NI parts per wave, each one K and one V load instruction.  tile_src
    // is the scalar part (where the tile's rows are), issue_part the per-lane part.
    struct TileSrc {
        const char *kt, *vt;   // wave-uniform byte address of the tile's first K / V row
        uint32_t row_bytes;    // distance between rows
        int max_r;             // last row of the tile that exists (rows past it repeat it; they are masked later)
        int blk[NI];           // paged: the block of each load instruction's rows
    };
    auto tile_src = [&](int tj) -> TileSrc {
        TileSrc ts;
        if (SRC == SRC_PACKETS) {
            const AttnTile td = load_tile_record(a.tiles, it.kv_begin + tj);
            if (td.kind == 0) {
                // stride < 0: a compressed packet, src_base is this layer's own part of the blob
                // ([K: Hkv x rows][V: Hkv x rows], rows = -stride)
                const bool own_layer = td.stride < 0;
                const int stride = own_layer ? -td.stride : td.stride;
                const int64_t slice = ((int64_t)(own_layer ? 0 : a.layer) * a.n_kv + it.kv_head) * stride + td.row0;
                ts.kt = (const char *)((const bf16_t *)a.arena + td.src_base + slice * D);
                ts.vt = ts.kt + (int64_t)(own_layer ? 1 : a.n_layers_total) * a.n_kv * stride * ROW_BYTES;
                ts.row_bytes = ROW_BYTES;
            } else {
                ts.kt = (const char *)((const bf16_t *)a.k_tail + tail_off + (int64_t)td.row0 * a.n_kv * D);
                ts.vt = (const char *)((const bf16_t *)a.v_new + tail_off + (int64_t)td.row0 * a.n_kv * D);
                ts.row_bytes = (uint32_t)(a.n_kv * ROW_BYTES);
            }
            ts.kt = uniform_ptr(ts.kt);
            ts.vt = uniform_ptr(ts.vt);
            ts.max_r = td.n_rows - 1;
            return ts;
        }
        ts.max_r = tj == n_tiles - 1 ? last_tile_rows - 1 : BN - 1;
        ts.row_bytes = ROW_BYTES;
        if (SRC == SRC_CONTIG) {
            ts.kt = uniform_ptr(k_item + (int64_t)tj * TILE_BYTES);
            ts.vt = uniform_ptr(v_item + (int64_t)tj * TILE_BYTES);
        } else {
            // The RPI rows of one instruction lie in one block (blocks hold a multiple of 16 rows, items start at a
            // multiple of 16), clamped rows included, so the block is the same for the whole wave.
            ts.kt = ts.vt = nullptr;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r0 = RPI * (NW * i + wave), row = it.kv_begin + tj * BN + (r0 < ts.max_r ? r0 : ts.max_r);
                ts.blk[i] = blk_ids[__builtin_amdgcn_readfirstlane(row >> a.cache.block_shift)];
            }
        }
        return ts;
    };
    auto issue_part = [&](const TileSrc &ts, int tj, int i) {
        const uint32_t st = lds_base + (uint32_t)((tj % STAGES) * STAGE_BYTES);
        int r = RPI * (NW * i + wave) + slot_row;
        const int k_chunk = NW * RPI % 16 ? slot_chunk ^ k_swz(r) : k_chunk0;
        r = r < ts.max_r ? r : ts.max_r;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(st + (uint32_t)(RPI * (NW * i + wave) * ROW_BYTES));  // (wave-uniform)
        if (SRC != SRC_PAGED) {
            // (uniform_ptr again: should the compiler have moved the address to vector registers, it
            // comes back to scalar ones, which the instruction needs; otherwise this folds away)
            load_to_lds_16<NTL>(uniform_ptr(ts.kt), (uint32_t)r * ts.row_bytes + 16 * k_chunk, dst);
            load_to_lds_16<NTL>(uniform_ptr(ts.vt), (uint32_t)r * ts.row_bytes + 16 * v_chunk, dst + TILE_BYTES);
        } else {
            // the block id is wave-uniform: the address is a scalar base plus a 32-bit lane offset
            const int b = ts.blk[i];
            const int64_t blk_off = paged_base + (((int64_t)b * a.n_kv + it.kv_head) << a.cache.block_shift) * D;
            const int slot = (it.kv_begin + tj * BN + r) & ((1 << a.cache.block_shift) - 1);
            const char *kt = uniform_ptr((const char *)(kc + blk_off));
            const char *vt = uniform_ptr((const char *)(vc + blk_off));
            load_to_lds_16<NTL>(kt, (uint32_t)(slot * ROW_BYTES + 16 * k_chunk), dst);
            load_to_lds_16<NTL>(vt, (uint32_t)(slot * ROW_BYTES + 16 * v_chunk), dst + TILE_BYTES);
        }
    };
    auto issue = [&](int tj) {
        const TileSrc ts = tile_src(tj);
#pragma unroll
        for (int i = 0; i < NI; ++i) issue_part(ts, tj, i);
    };
    // Infinities and NaNs of V among the query rows stay out of the tiles, as zeros: times the zero probability
    // of a row that does not see them, or of the copies that fill a ragged tile, they would be NaN.  The rows
    // that do see them get them at the end, added to what was written.  The append looks for them while it copies
    // V_new to the cache (a word per wave, in LDS behind the tiles); without a cache there is no such copy, and
    // each wave looks at its part of the tiles with query rows as they land.  clean_from: the item's first
    // tile with query rows, if there is something to look for.  (Cost, per layer: 8K context 28.2 -> 28.4 us, 2.9K
    // rows 18.4 -> 18.5, in place 19.3 -> 19.4.  Looking at every tile as it lands cost 0.5 to 0.9 us, adding to
    // the accumulators before they are written 0.2 to 0.4.)
    int *const found = (int *)(lds + STAGES * STAGE_BYTES);
    int clean_from = n_tiles;
    // this wave's part of tile tj, landed and seen by no other wave yet
    auto clean_v = [&](int tj) {
        char *vt = lds + (tj % STAGES) * STAGE_BYTES + TILE_BYTES + wave * (RPI * ROW_BYTES) + lane * 16;
        uint4 v[NI];
        ushort2_t v_max = {0, 0};
#pragma unroll
        for (int i = 0; i < NI; ++i) v[i] = *(const uint4 *)(vt + i * (NW * RPI * ROW_BYTES));
#pragma unroll
        for (int i = 0; i < NI; ++i) max_magnitude(v_max, v[i]);
        if (!__any(v_max[0] >= 0x7F80u || v_max[1] >= 0x7F80u)) return;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            uint32_t bad = 0;
            const bf16x8 w = drop_nonfinite(__builtin_bit_cast(bf16x8, v[i]), bad);
            if (bad && (SRC == SRC_PACKETS || it.kv_begin + tj * BN + RPI * (NW * i + wave) + slot_row >= it.ctx_len)) *(bf16x8 *)(vt + i * (NW * RPI * ROW_BYTES)) = w;
        }
        if (SRC == SRC_PACKETS) found[wave] = 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // this lane's query row
    const int rr = 32 * wave_r + n;
    const bool row_ok = rr < it.n_rows;
    const bool wave_active = 32 * wave_r < it.n_rows;  // wave-uniform
    const int m = it.m0 + (row_ok ? rr : 0);
    const int t = m / g, hq = it.kv_head * g + m % g;
    const int limit = row_ok ? it.ctx_len + t + 1 : 0;  // cache modes: kv rows [0, limit) are visible
    // smallest limit among the wave's rows (rows are ordered by query token)
    const int wave_limit = it.ctx_len + (it.m0 + 32 * wave_r) / g + 1;

    // B operand of S^T = K Q^T: lane holds Q[m][16 ks + 8 h .. +7] for every k-step ks, rotated by
    // `rel` positions and multiplied by q_scale.  Element 16 ks + 8 h + j (ks < NKS / 2)
    // pairs with the same slot of ks + NKS / 2, so the rotation stays inside the lane.
    // KS = 2: the two groups hold the same rows; each loads and rotates half of the k-steps, and they
    // exchange the results through LDS.
    constexpr int NKH = NKS / 2;
    constexpr int NQP = NKH / KS;  // partner pairs of k-steps a wave rotates: grp NQP .. + NQP - 1
    bf16x8 qf[NKS];
    const bf16_t *qp = (const bf16_t *)a.q + ((int64_t)(it.q_off + t) * a.n_q_heads + hq) * D + 8 * h;
    const int q_pos = a.prerotated ? 0 : it.pos0 + t;  // rotation the query still needs
    // QUAD, a multiple of four query heads to a KV head: the four lanes of a quad hold rows of one token: each
    // loads a quarter of its (cos, sin) pairs, scales it, and the rotation takes the rest from its
    // neighbours.  (A workgroup of 128 rows pulls 48 KB through the CU's texture unit before it can start,
    // not 96.  Four heads, 128 rows, per layer: 2.9K rows 20.2 -> 20.0 us, 8K 29.9 -> 29.8, pruned 26.6 ->
    // 26.3.  A template argument: chosen at run time, the in-place variant held both versions' registers
    // and spilled.)
    auto rotate_k_step = [&](const uint4 &lo, const uint4 &hi, const float4 &cs_own, uint4 &olo, uint4 &ohi) {  // cs_own: scaled
        const float4 cs4[4] = {quad_lane<0>(cs_own), quad_lane<1>(cs_own), quad_lane<2>(cs_own), quad_lane<3>(cs_own)};
        rotate_query_pair<true>(lo, hi, cs4, 1.f, olo, ohi);
    };
    auto directed = [&](const float4 &v, float sign) -> float4 {  // (only a packet can lie ahead of the query's own position)
        return SRC == SRC_PACKETS ? make_float4(v.x, v.y * sign, v.z, v.w * sign) : v;
    };
    u32x4_t qraw[2 * NQP], csraw[4 * NQP];
    auto q_issue = [&](int delta) {  // 3 D / 16 / KS loads: the raw query row and the (cos, sin) of its rotation
        const bf16_t *qsrc = (row_ok ? qp : (const bf16_t *)a.q + 8 * h) + 16 * NQP * grp;  // idle lanes read row 0 (and drop it)
#pragma unroll
        for (int ks = 0; ks < NQP; ++ks) {
            qraw[ks] = load16_nowait(qsrc + 16 * ks);
            qraw[ks + NQP] = load16_nowait(qsrc + 16 * (ks + NKH));
        }
        const int rel = row_ok ? q_pos - delta : 0;
        const float4 *csr = (const float4 *)(a.cs + (int64_t)(rel < 0 ? -rel : rel) * (D / 2) + 8 * h + 16 * NQP * grp);
        if (QUAD) {
#pragma unroll
            for (int ks = 0; ks < NQP; ++ks) csraw[ks] = load16_nowait(csr + 8 * ks + (lane & 3));
            return;
        }
#pragma unroll
        for (int ks = 0; ks < NQP; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) csraw[4 * ks + j] = load16_nowait(csr + 8 * ks + j);
    };
    // `younger`: tiles whose loads were issued after q_issue and may still be on their way
    auto q_finish = [&](int delta, int younger) {
        if (younger >= 3) wait_vmcnt<3 * 2 * NI>();
        else if (younger == 2) wait_vmcnt<2 * 2 * NI>();
        else if (younger == 1) wait_vmcnt<2 * NI>();
        else wait_vmcnt<0>();
        // the registers are valid from here on: keep every use below this point
#pragma unroll
        for (int i = 0; i < 2 * NQP; ++i) asm volatile("" : "+v"(qraw[i]));
#pragma unroll
        for (int i = 0; i < 4 * NQP; ++i) asm volatile("" : "+v"(csraw[i]));
        const int rel = row_ok ? q_pos - delta : 0;
        const float sign = rel < 0 ? -1.f : 1.f;
        char *qx = lds + (STAGES - 1) * STAGE_BYTES + wave_r * (64 * 16) + lane * 16;  // KS = 2: [NKS][RW][64 lanes]; no tile is in this stage yet
        static_assert(KS == 1 || KS * PR < STAGES, "the last stage is free until the loop");
        auto keep = [&](int ks, const uint4 &olo, const uint4 &ohi) {
            if (KS == 2) {
                *(uint4 *)(qx + (ks + NQP * grp) * (RW * 64 * 16)) = olo;
                *(uint4 *)(qx + (ks + NQP * grp + NKH) * (RW * 64 * 16)) = ohi;
            } else {
                qf[ks] = __builtin_bit_cast(bf16x8, olo);
                qf[ks + NKH] = __builtin_bit_cast(bf16x8, ohi);
            }
        };
        const float sc = row_ok ? q_scale : 0.f;  // (idle lanes: zeros, whatever their registers hold)
        if (QUAD) {
#pragma unroll
            for (int ks = 0; ks < NQP; ++ks) {
                uint4 olo, ohi;
                rotate_k_step(__builtin_bit_cast(uint4, qraw[ks]), __builtin_bit_cast(uint4, qraw[ks + NQP]),
                              scale_cs(__builtin_bit_cast(float4, csraw[ks]), sc, sc * sign), olo, ohi);
                keep(ks, olo, ohi);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < NQP; ++ks) {
                float4 cs4[4];  // (cos, sin) pairs of elements 16 ks + 8 h + 2 j, + 1
#pragma unroll
                for (int j = 0; j < 4; ++j) cs4[j] = directed(__builtin_bit_cast(float4, csraw[4 * ks + j]), sign);
                uint4 olo, ohi;
                rotate_query_pair<false>(__builtin_bit_cast(uint4, qraw[ks]), __builtin_bit_cast(uint4, qraw[ks + NQP]), cs4, sc, olo, ohi);
                keep(ks, olo, ohi);
            }
        }
        if (KS == 2) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wg_barrier();
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)(qx + ks * (RW * 64 * 16));
        }
        // pinned: nothing of this is recomputed or waited for inside the tile loop
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));
    };
    // Re-rotation inside the tile loop (in-place packet reads, at every packet boundary; and the only
    // rotation of 256 columns): plain loads, whose wait the compiler places (it drains the tile loads in flight as well).
    auto reload_q = [&](int delta) {
        uint4 qr[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qr[ks] = row_ok ? *(const uint4 *)(qp + 16 * ks) : make_uint4(0, 0, 0, 0);
        const int rel = row_ok ? q_pos - delta : 0;
        const float sign = rel < 0 ? -1.f : 1.f;
        const float4 *csr = (const float4 *)(a.cs + (int64_t)(rel < 0 ? -rel : rel) * (D / 2) + 8 * h);
        const float sc = q_scale;
        float4 own[NKH];
        if (QUAD) {
#pragma unroll
            for (int ks = 0; ks < NKH; ++ks) own[ks] = csr[8 * ks + (lane & 3)];
        }
#pragma unroll
        for (int ks = 0; ks < NKH; ++ks) {
            float4 cs4[4];
            if (QUAD) {
                own[ks] = scale_cs(own[ks], sc, sc * sign);
                cs4[0] = quad_lane<0>(own[ks]);
                cs4[1] = quad_lane<1>(own[ks]);
                cs4[2] = quad_lane<2>(own[ks]);
                cs4[3] = quad_lane<3>(own[ks]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) cs4[j] = directed(csr[8 * ks + j], sign);
            }
            uint4 olo, ohi;
            rotate_query_pair<QUAD>(qr[ks], qr[ks + NKH], cs4, sc, olo, ohi);
            qf[ks] = __builtin_bit_cast(bf16x8, olo);
            qf[ks + NKH] = __builtin_bit_cast(bf16x8, ohi);
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));
    };
    int cur_delta = SRC == SRC_PACKETS && n_tiles > 0 ? load_tile_record(a.tiles, it.kv_begin).pos : 0;
    KVP_STAMP(1);
    // (256 columns: the loads in flight would not fit the vector registers, and one the compiler moved
    // to an accumulation register before its data has arrived would be lost: plain loads there)
    constexpr bool OWN_WAIT = D <= 128;
    if (OWN_WAIT) q_issue(cur_delta);  // first, so that the query arrives ahead of the tiles
    // a first tile that cannot contain query rows can start its trip right away
    const bool early0 = n_tiles > 0 && (SRC == SRC_PACKETS ? load_tile_record(a.tiles, it.kv_begin).kind == 0 : it.kv_begin + BN <= it.ctx_len);
    if (early0) issue(0);

    // ---- query rows inside this item's range: rotate K_new to its row's position and
    // append K_new / V_new before any tile load can touch those rows
    {
        int tail_lo, n_tail;  // query rows [tail_lo, tail_lo + n_tail) relative to ctx_len
        if (SRC == SRC_PACKETS) {
            // an item that reaches the query tiles writes all of this head's rotated K_new rows
            const bool has_tail = n_tiles > 0 && load_tile_record(a.tiles, it.kv_end - 1).kind != 0;
            tail_lo = 0;
            n_tail = has_tail ? it.n_q : 0;
        } else {
            tail_lo = (it.kv_begin > it.ctx_len ? it.kv_begin : it.ctx_len) - it.ctx_len;
            n_tail = it.kv_end - it.ctx_len - tail_lo;  // > 0 only for items that reach the query rows
        }
        if (n_tail > 0) {
            bf16_t *kcw = SRC == SRC_PACKETS ? (bf16_t *)a.k_tail : (bf16_t *)a.cache.k;
            bf16_t *vcw = (bf16_t *)a.cache.v;
            // Work units: CH / 2 K chunk pairs per row (rotate, store) and, with a cache, CH V chunks per
            // row (copy).  A thread takes two K units and four V units per trip and issues all their
            // loads before it uses the first, so the append costs one memory round trip per trip
            // (32 query rows: one trip) instead of one per unit.
            auto unit_dst = [&](int qr, int64_t src) -> int64_t {
                const int row = it.ctx_len + qr;  // cache row of the query token
                if (SRC == SRC_PACKETS) return src;
                if (SRC == SRC_CONTIG) return contig_off + (int64_t)(row - it.kv_begin) * D;
                const int b = a.cache.block_table[(int64_t)it.req * a.cache.max_blocks + (row >> a.cache.block_shift)];
                const int slot = row & ((1 << a.cache.block_shift) - 1);
                return paged_base + ((((int64_t)b * a.n_kv + it.kv_head) << a.cache.block_shift) + slot) * D;
            };
            const int n_k = n_tail * (CH / 2), n_v = SRC == SRC_PACKETS ? 0 : n_tail * CH;
            ushort2_t v_max = {0, 0};  // largest magnitudes of V_new, as bits
            // (loads are unconditional, from units clamped into range; only the stores are guarded)
            for (int s0 = 0; 2 * s0 * NT < n_k || 4 * s0 * NT < n_v; ++s0) {
                if (4 * s0 * NT + tid >= n_v && 2 * s0 * NT + tid >= n_k) continue;  // (a thread without a unit: few query rows)
                uint4 vv0, vv1, vv2, vv3;
                int64_t vd0, vd1, vd2, vd3;
                auto v_load = [&](int j, uint4 &vv, int64_t &vd) -> bool {
                    const int idx = (4 * s0 + j) * NT + tid;
                    const int ic = idx < n_v ? idx : (n_v > 0 ? n_v - 1 : 0);
                    const int qr = tail_lo + ic / CH, e = 8 * (ic % CH);
                    const int64_t src = ((int64_t)(it.q_off + qr) * a.n_kv + it.kv_head) * D;
                    vd = unit_dst(qr, src) + e;
                    vv = n_v > 0 ? *(const uint4 *)((const bf16_t *)a.v_new + src + e) : make_uint4(0, 0, 0, 0);
                    return idx < n_v;
                };
                const bool von0 = v_load(0, vv0, vd0), von1 = v_load(1, vv1, vd1), von2 = v_load(2, vv2, vd2), von3 = v_load(3, vv3, vd3);
                struct KUnit { uint4 ulo, uhi; float4 c0, c1, c2, c3; int64_t dst; bool on; };
                auto k_load = [&](int j) -> KUnit {
                    KUnit u;
                    const int idx = (2 * s0 + j) * NT + tid;
                    const int ic = idx < n_k ? idx : n_k - 1;
                    const int qr = tail_lo + ic / (CH / 2), e = 8 * (ic % (CH / 2));
                    const int pos = it.pos0 + qr;     // the token's position
                    const int64_t src = ((int64_t)(it.q_off + qr) * a.n_kv + it.kv_head) * D;
                    u.dst = unit_dst(qr, src) + e;
                    u.ulo = *(const uint4 *)((const bf16_t *)a.k_new + src + e);
                    u.uhi = *(const uint4 *)((const bf16_t *)a.k_new + src + D / 2 + e);
                    const float4 *csr = (const float4 *)(a.cs + (int64_t)pos * (D / 2) + e);
                    u.c0 = csr[0]; u.c1 = csr[1]; u.c2 = csr[2]; u.c3 = csr[3];
                    u.on = idx < n_k;
                    return u;
                };
                const KUnit k0 = k_load(0), k1 = k_load(1);
                max_magnitude(v_max, vv0);
                max_magnitude(v_max, vv1);
                max_magnitude(v_max, vv2);
                max_magnitude(v_max, vv3);
                if (von0) *(uint4 *)(vcw + vd0) = vv0;
                if (von1) *(uint4 *)(vcw + vd1) = vv1;
                if (von2) *(uint4 *)(vcw + vd2) = vv2;
                if (von3) *(uint4 *)(vcw + vd3) = vv3;
                auto k_store = [&](const KUnit &u) {
                    if (!u.on) return;
                    const float4 one = make_float4(1.f, 0.f, 1.f, 0.f);
                    const float4 cs4[4] = {a.prerotated ? one : u.c0, a.prerotated ? one : u.c1, a.prerotated ? one : u.c2, a.prerotated ? one : u.c3};
                    uint4 olo, ohi;
                    rotate_chunk_pair(u.ulo, u.uhi, cs4, olo, ohi);
                    *(uint4 *)(kcw + u.dst) = olo;
                    *(uint4 *)(kcw + u.dst + D / 2) = ohi;
                };
                k_store(k0);
                k_store(k1);
            }
            const bool nonfinite = __any(v_max[0] >= 0x7F80u || v_max[1] >= 0x7F80u);
            if (lane == 0) found[wave] = nonfinite;
            wait_vmcnt<0>();   // this wave's stores have reached the L2
            // The same wait once more, in the form the compiler's own wait bookkeeping understands:
            // without it the compiler takes the loads and stores above for still outstanding when the
            // tile loop is entered and puts a full vmcnt(0) in front of every tile's first MFMA -- which
            // waits for every tile load in flight and turns a four-stage ring into a one-deep prefetch.
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters left alone
            __syncthreads();   // ... and so have every other wave's
            if (SRC == SRC_PACKETS) {  // (each wave looks at its part of the tiles as they land)
                const AttnTile last = load_tile_record(a.tiles, it.kv_end - 1);
                clean_from = n_tiles > last.row0 / BN + 1 ? n_tiles - (last.row0 / BN + 1) : 0;
            } else {
                int any = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) any |= found[w];
                if (__builtin_amdgcn_readfirstlane(any)) clean_from = it.ctx_len > it.kv_begin ? (it.ctx_len - it.kv_begin) / BN : 0;
            }
        }
    }

#pragma unroll
    for (int s = 0; s < KS * PR; ++s)
        if (s < n_tiles && !(s == 0 && early0)) issue(s);

    if (OWN_WAIT) q_finish(cur_delta, n_tiles < KS * PR ? n_tiles : KS * PR);
    else reload_q(cur_delta);
    KVP_STAMP(2);

    floatx16 oacc[EB];
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[eb][r] = 0.f;
    float m_ref = -INFINITY, l_i = 0.f;  // reference max (in the accumulators' units) and running sum
    // -m_ref in all 16 slots (every accumulator of a lane belongs to the same query row): the
    // first S MFMA of a tile takes it as its C operand, so S - m_ref costs no extra instruction.
    // Rewritten only when the reference moves; pinned so that it is not rebuilt per tile.
    // (The in-place packet variant and 256 columns have no registers to spare and rebuild it per tile.)
    constexpr bool KEEP_CINIT = SRC != SRC_PACKETS && D <= 128;
    floatx16 cinit;
#pragma unroll
    for (int r = 0; r < 16; ++r) cinit[r] = 0.f;
    if (KEEP_CINIT) asm volatile("" : "+v"(cinit));

    const int tr_row = (lane & 15) >> 2;
    const int tr_x = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);  // 16-byte chunk inside the 64-byte column group
    const int tr_half = 8 * (lane & 1);


    // Where the tiles are that a round requests.  Paged: looked up at the end of the round before it, so that the block ids
    // arrive under the wait for the tiles (a scalar load outstanding turns the next wait for an LDS read into
    // a wait for everything: 8K rows 27.5 -> 27.25 us per layer of a step).  Elsewhere there is nothing to wait for, or (in place) the
    // registers are short: 17.7 -> 18.05, with 28 / 4 heads over a cache 22.95 -> 23.6.
    constexpr bool LOOK_AHEAD = SRC == SRC_PAGED;
    TileSrc rsrc[KS];
    auto look_up = [&](int rd) {
#pragma unroll
        for (int k2 = 0; k2 < KS; ++k2)
            if (KS * (rd + PR) + k2 < n_tiles) rsrc[k2] = tile_src(KS * (rd + PR) + k2);
    };
    if (LOOK_AHEAD) look_up(0);

    const int n_rounds = (n_tiles + KS - 1) / KS;
    KVP_PHASE_DECL;
    for (int rd = 0; rd < n_rounds; ++rd) {
        KVP_PHASE(5);
        // round rd's tiles have landed once only the loads of the rounds issued after it remain
        {
            const int hi = KS * (rd + PR) < n_tiles ? KS * (rd + PR) : n_tiles;
            const int lo = KS * (rd + 1) < n_tiles ? KS * (rd + 1) : n_tiles;
            const int younger = hi - lo;  // tiles issued after this round, 0 .. KS (PR - 1)
            if (younger >= 3) wait_vmcnt<3 * 2 * NI>();
            else if (younger == 2) wait_vmcnt<2 * 2 * NI>();
            else if (younger == 1) wait_vmcnt<2 * NI>();
            else wait_vmcnt<0>();
        }
        if (KS * rd + KS > clean_from) {  // (rare)
#pragma unroll 1
            for (int k2 = 0; k2 < KS; ++k2)
                if (KS * rd + k2 >= clean_from && KS * rd + k2 < n_tiles) clean_v(KS * rd + k2);
        }
        KVP_STAMP(4 + 2 * rd);
        KVP_PHASE(0);
        wg_barrier();  // every wave's part of the round is in LDS; everyone is done with round rd-1
        KVP_STAMP(5 + 2 * rd);
        KVP_PHASE(1);
        auto refill = [&]() {  // the stages round rd-1 used take round rd+PR
#pragma unroll
            for (int k2 = 0; k2 < KS; ++k2)
                if (KS * (rd + PR) + k2 < n_tiles) issue(KS * (rd + PR) + k2);
        };
        const int ti = KS * rd + grp;  // this group's tile of the round
        if (ti >= n_tiles || !wave_active) {  // nothing to compute: only help to load
            refill();
            continue;
        }

        const int kv0 = it.kv_begin + ti * BN;
        const char *kl = lds + (ti % STAGES) * STAGE_BYTES;
        const char *vl = kl + TILE_BYTES;
        AttnTile td;
        if (SRC == SRC_PACKETS) {
            td = load_tile_record(a.tiles, it.kv_begin + ti);
            if (td.pos != cur_delta && wave_active) {  // the tile belongs to another packet: re-rotate the query
                cur_delta = td.pos;
                reload_q(cur_delta);
            }
        }

        // ---- S^T - m_ref = K Q^T - m_ref : 2 blocks of 32 kv rows x 32 query rows
        floatx16 sacc[2];
        if (!KEEP_CINIT) {
            const float c = m_ref == -INFINITY ? 0.f : -m_ref;
#pragma unroll
            for (int r = 0; r < 16; ++r) cinit[r] = c;
        }
        // K fragments run AHEAD k-steps in front of the MFMAs that use them: the first AHEAD k-steps'
        // fragments are requested up front, and each k-step's MFMA pair is followed by the request
        // for the fragments AHEAD steps on, so the matrix pipe starts after a quarter of the tile has
        // arrived from LDS instead of all of it (the four waves of a workgroup reach this point
        // together, and 64 KB of fragment reads keep the LDS busy for about as long as the 16 MFMAs
        // keep the matrix pipe).
        // The next tile loads -- they refill the stages the previous round used, which every wave
        // left before the barrier above -- are issued between the matrix instructions too, one part
        // (a K and a V load with their address arithmetic) behind each of the first k-steps' MFMA
        // pair: the matrix pipe is busy for 64 cycles per pair, about what a part takes to issue.
        {
            constexpr int AHEAD = 2;  // (2, 3, 4, 6 and 8 k-steps measured: 2 is the fastest by a little, and holds the fewest registers)
            constexpr int N_PARTS = KS * NI;
            static_assert(N_PARTS <= NKS, "one part per k-step");
            if (!LOOK_AHEAD) look_up(rd);
            uint4 kf[2 * AHEAD];
            auto read_k = [&](int kstep) {
                const int coff = 16 * ((2 * kstep + h) ^ k_swz(n));
                kf[2 * (kstep % AHEAD)] = *(const uint4 *)(kl + n * ROW_BYTES + coff);
                kf[2 * (kstep % AHEAD) + 1] = *(const uint4 *)(kl + (32 + n) * ROW_BYTES + coff);
            };
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) read_k(i);
            __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the matrix code
#pragma unroll
            for (int kstep = 0; kstep < NKS; ++kstep) {
                const bool head = kstep == 0;  // compile-time: the tile's first k-step
                const int sl = 2 * (kstep % AHEAD);
                sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[sl]), qf[kstep], head ? cinit : sacc[0], 0, 0, 0);
                sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[sl + 1]), qf[kstep], head ? cinit : sacc[1], 0, 0, 0);
                if (kstep + AHEAD < NKS) read_k(kstep + AHEAD);
                if (kstep < N_PARTS) {
                    const int k2 = kstep / NI, tj = KS * (rd + PR) + k2;
                    if (tj < n_tiles) issue_part(rsrc[k2], tj, kstep % NI);
                }
                __builtin_amdgcn_sched_barrier(0);  // what follows a pair stays behind it
            }
        }
        KVP_PHASE(2);

        // ---- online softmax; accumulator r of block kb is tile row 32 kb + 8 (r/4) + 4 h + r%4
        if (SRC == SRC_PACKETS) {
            if (td.kind != 0 || td.n_rows < BN) {  // wave-uniform: query tiles and ragged packet ends
                const int vis = td.kind != 0 ? (row_ok ? t - td.row0 + 1 : 0) : BN;  // causal among query rows
                const int lim = vis < td.n_rows ? vis : td.n_rows;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (32 * kb + 8 * (r >> 2) + 4 * h + (r & 3) >= lim) sacc[kb][r] = -INFINITY;
            }
        } else if (kv0 + BN > wave_limit || kv0 + BN > it.kv_end) {  // wave-uniform: tail tiles only
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    int kv = kv0 + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3);
                    if (kv >= limit || kv >= it.kv_end) sacc[kb][r] = -INFINITY;
                }
        }
        float mx = max3(sacc[0][0], sacc[1][0], sacc[0][1]);
        mx = max3(mx, sacc[1][1], sacc[0][2]);
#pragma unroll
        for (int r = 2; r < 15; ++r) mx = max3(mx, sacc[1][r], sacc[0][r + 1]);
        mx = fmaxf(mx, sacc[1][15]);
        mx = xhalf_max(mx);  // row max relative to m_ref
        // The reference moves when a row sees its first visible entry (it becomes that
        // tile's maximum) and afterwards only when the maximum outgrows the slack.
        // (Head dims other than 128 set the reference the slack above the maximum: no weight exceeds one, so V
        // near the top of bf16's range overflows no earlier than in the generic kernel.)
        const bool first = m_ref == -INFINITY;
        const bool move = first ? mx > -INFINITY : mx > (SPLIT_P ? 0.f : RESCALE_SLACK);
        if (__any(move)) {  // wave-uniform; rare once the maxima settle
            const float delta = move ? (SPLIT_P ? mx + above : mx) : 0.f;
            const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-delta * s_scale);  // first: O = l = 0
            m_ref = first ? (move ? delta : -INFINITY) : m_ref + delta;
            l_i *= alpha;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) sacc[kb][r] -= delta;
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[eb][r] *= alpha;
            if (KEEP_CINIT) {
                const float c = m_ref == -INFINITY ? 0.f : -m_ref;
#pragma unroll
                for (int r = 0; r < 16; ++r) cinit[r] = c;
                asm volatile("" : "+v"(cinit));
            }
        }

        // ---- P = exp2(S - m_ref) and O^T += V^T P^T, one 32-row block at a time so that the
        // exponentials of block 1 run while the matrix cores accumulate block 0.
        // k-step j of block kb covers tile rows 32 kb + 16 j + [0, 16); P^T slots 0..7 of
        // lane-half h are rows 4h+{0..3} and 8+4h+{0..3} of that step, so the two transposing
        // reads fetch exactly those rows of V for column 32 eb + n.
        KVP_PHASE(3);
        float rs0 = 0.f, rs1 = 0.f;
        const bf16x2 bf16_ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
        typedef __attribute__((address_space(3))) short4v *lds_s4;
        short4v vfr[2][2 * EB];  // V fragments of one k-step: [buffer][2 eb + lo/hi]
        auto read_v = [&](int step, int buf) {  // step = 2 kb + j
            const char *vp = vl + (16 * step + 4 * h + tr_row) * ROW_BYTES + tr_half;
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) {
                const int coff = 16 * (4 * (eb ^ v_swz(tr_row)) + tr_x);
                vfr[buf][2 * eb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(vp + coff));
                vfr[buf][2 * eb + 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(vp + 8 * ROW_BYTES + coff));
            }
        };
        read_v(0, 0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            uint32_t pk[8], pl[8];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                float p0 = __builtin_amdgcn_exp2f(sacc[kb][r] * s_scale);
                float p1 = __builtin_amdgcn_exp2f(sacc[kb][r + 1] * s_scale);
                if (SPLIT_P) {
                    // Cut, not rounded, so that the rest is never negative; 2^-23 of p on top keeps it above zero
                    // where p is (both parts times an infinity of V then agree), and only there: a masked
                    // entry's p is zero, and so is what its row of V, however large, is multiplied by.
                    constexpr float ABOVE = 1.f + 0x1p-23f;
                    pk[r >> 1] = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302);
                    const float q0 = __builtin_fmaf(p0, ABOVE, -__uint_as_float(__float_as_uint(p0) & 0xFFFF0000u));
                    const float q1 = __builtin_fmaf(p1, ABOVE, -__uint_as_float(__float_as_uint(p1) & 0xFFFF0000u));
                    pl[r >> 1] = pack_bf16_hw(q0, q1);
                    rs0 += p0;
                    rs1 += p1;
                    continue;
                }
                pk[r >> 1] = pack_bf16_hw(p0, p1);
                // the row sum takes the rounded values, i.e. exactly what multiplies V
                const bf16x2 pp = __builtin_bit_cast(bf16x2, pk[r >> 1]);
                if (r & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pp, bf16_ones, rs1, false);
                else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pp, bf16_ones, rs0, false);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int step = 2 * kb + j;
                if (step + 1 < 4) read_v(step + 1, (step + 1) & 1);  // next k-step's V lands under these MFMAs
                uint4 pu = make_uint4(pk[4 * j], pk[4 * j + 1], pk[4 * j + 2], pk[4 * j + 3]);
                bf16x8 pf = __builtin_bit_cast(bf16x8, pu);
                bf16x8 pg = pf;
                if (SPLIT_P) pg = __builtin_bit_cast(bf16x8, make_uint4(pl[4 * j], pl[4 * j + 1], pl[4 * j + 2], pl[4 * j + 3]));
#pragma unroll
                for (int eb = 0; eb < EB; ++eb) {
                    union { short4v s[2]; bf16x8 v; } vf;
                    vf.s[0] = vfr[step & 1][2 * eb];
                    vf.s[1] = vfr[step & 1][2 * eb + 1];
                    oacc[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pf, oacc[eb], 0, 0, 0);
                    if (SPLIT_P) oacc[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pg, oacc[eb], 0, 0, 0);
                }
            }
        }
        l_i += rs0 + rs1;  // this lane's half of the row; the halves are added once, at the end
        if (LOOK_AHEAD) look_up(rd + 1);
        KVP_PHASE(4);
    }
    KVP_PHASE_WRITE;
    l_i = xhalf_sum(l_i);
    m_ref *= s_scale;  // log2 units from here on
    KVP_STAMP(30);

    // KS = 2: both groups go on with half of the columns each (EBO blocks from column col0 on).  (Shared query
    // and halves, against one group that merges and writes everything: 8K context as two-group items 31.3 ->
    // 30.0 us per layer; one token over 8 contexts of 16.9K rows 89.3 -> 87.8.)
    constexpr int EBO = EB / KS;
    const int col0 = KS == 2 ? 32 * EBO * grp : 0;
    if (KS == 2) {
        static_assert(KS == 1 || D == 128, "the two-group shape's LDS layout");
        // ---- merge the two groups' (m, l, O) of each row through LDS (the tile stages are free once
        // every wave has left the loop): each group hands over the columns the other goes on with.
        wg_barrier();
        float *xo = (float *)lds;                      // [2][4 EBO][RW][64 lanes][4]
        float *xm = xo + 2 * 4 * EBO * RW * 64 * 4;    // [2][RW][64] m, then [2][RW][64] l
        auto hand_over = [&](const floatx16 *o) {
#pragma unroll
            for (int q = 0; q < 4 * EBO; ++q)
                *(float4 *)(xo + (((grp * 4 * EBO + q) * RW + wave_r) * 64 + lane) * 4) =
                    make_float4(o[q >> 2][4 * (q & 3)], o[q >> 2][4 * (q & 3) + 1], o[q >> 2][4 * (q & 3) + 2], o[q >> 2][4 * (q & 3) + 3]);
        };
        if (grp == 0) {
            hand_over(oacc + EBO % EB);
        } else {
            hand_over(oacc);
#pragma unroll
            for (int eb = 0; eb < EBO; ++eb) oacc[eb] = oacc[eb + EB - EBO];
        }
        xm[(grp * RW + wave_r) * 64 + lane] = m_ref;
        xm[((2 + grp) * RW + wave_r) * 64 + lane] = l_i;
        __syncthreads();
        const float m1 = xm[((1 - grp) * RW + wave_r) * 64 + lane], l1 = xm[((3 - grp) * RW + wave_r) * 64 + lane];
        const float mm = fmaxf(m_ref, m1);
        const float a0 = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref - mm);
        const float a1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
        m_ref = mm;
        l_i = grp == 0 ? l_i * a0 + l1 * a1 : l1 * a1 + l_i * a0;
#pragma unroll
        for (int q = 0; q < 4 * EBO; ++q) {
            const float4 o1 = *(const float4 *)(xo + ((((1 - grp) * 4 * EBO + q) * RW + wave_r) * 64 + lane) * 4);
            floatx16 &o = oacc[q >> 2];
            const int r = 4 * (q & 3);
            o[r] = o[r] * a0 + o1.x * a1;
            o[r + 1] = o[r + 1] * a0 + o1.y * a1;
            o[r + 2] = o[r + 2] * a0 + o1.z * a1;
            o[r + 3] = o[r + 3] * a0 + o1.w * a1;
        }
    }

    // ---- epilogue: lane holds O[m][32 eb + 8 (r/4) + 4 h + r%4]
    if (row_ok) {
        if (it.part_slot < 0) {
            bf16_t *op = (bf16_t *)a.out + ((int64_t)(it.q_off + t) * a.n_q_heads + hq) * D;
            const float inv = 1.f / l_i;
#pragma unroll
            for (int eb = 0; eb < EBO; ++eb)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    uint2 u;
                    u.x = pack_bf16_hw(oacc[eb][4 * q4] * inv, oacc[eb][4 * q4 + 1] * inv);
                    u.y = pack_bf16_hw(oacc[eb][4 * q4 + 2] * inv, oacc[eb][4 * q4 + 3] * inv);
                    *(uint2 *)(op + col0 + 32 * eb + 8 * q4 + 4 * h) = u;
                }
        }
    }
    if constexpr (D == 64) {
        if (it.part_slot >= 0 && row_ok) {  // fp32 rows, then m and l of each row
            float *pp = (float *)((char *)a.partials + (int64_t)it.part_slot * part_slot_bytes(a.bm, D, 0));
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *(float4 *)(pp + (int64_t)rr * D + 32 * eb + 8 * q4 + 4 * h) =
                        make_float4(oacc[eb][4 * q4], oacc[eb][4 * q4 + 1], oacc[eb][4 * q4 + 2], oacc[eb][4 * q4 + 3]);
            if (h == 0) {
                pp[(int64_t)a.bm * D + rr] = m_ref;
                pp[(int64_t)a.bm * D + a.bm + rr] = l_i;
            }
        }
    } else if constexpr (SPLIT_P) {
        // 256 columns: as the accumulators lie, then (m, l) of each row.  (Row by row, a layer of a step over 2K rows took 32.3 us,
        // now 30.7; four paged requests of 3 to 8 passages 58.8 and 57.9.  64 columns: a launch that is not split became 2 % slower.)
        if (it.part_slot >= 0 && row_ok) {
            char *pp = (char *)a.partials + (int64_t)it.part_slot * part_slot_bytes(a.bm, D, 0);
            const int own = part_piece_at(4 * D, rr, h);
            auto piece = [&](int j) -> u32x4_t {
                const floatx16 &o = oacc[j >> 2];
                const int r = 4 * (j & 3);
                return __builtin_bit_cast(u32x4_t, make_float4(o[r], o[r + 1], o[r + 2], o[r + 3]));
            };
            if (NW == 4 && a.merged_elsewhere) {
                const ThroughStore through(pp, (int)part_rows_bytes(a.bm, D, 0));
#pragma unroll
                for (int j = 0; j < 4 * EB; ++j) through.put16(own + 1024 * j, piece(j));
            } else {
#pragma unroll
                for (int j = 0; j < 4 * EB; ++j) *(u32x4_t *)(pp + own + 1024 * j) = piece(j);
            }
            if (h == 0) ((float2 *)(pp + part_rows_bytes(a.bm, D, 0)))[rr] = make_float2(m_ref, l_i);
        }
    } else if (it.part_slot >= 0) {
        // A slot holds a.bm rows of D fp16 values (the launch's largest row block; BM <= a.bm), then
        // (m, l) of each row in fp32.  A row of the split's unnormalised O goes out as fp16 scaled
        // by a power of two 2^-e that brings its largest magnitude below 1; m + e and l 2^-e go with
        // it, which is the same partial result relative to another reference, so the merge's
        // algebra does not change.  Eleven significant bits relative to the row's maximum, where the
        // bf16 output keeps eight.
        char *pp = (char *)a.partials + (int64_t)it.part_slot * part_slot_bytes(a.bm, D, 1);
        float amax = 0.f;
#pragma unroll
        for (int eb = 0; eb < EBO; ++eb)
#pragma unroll
            for (int r = 0; r < 16; ++r) amax = fmaxf(amax, __builtin_fabsf(oacc[eb][r]));
        amax = xhalf_max(amax);
        if (KS == 2) {  // the row's other columns are with the other group
            float *xa = (float *)(lds + 68 * 1024);
            xa[(grp * RW + wave_r) * 64 + lane] = amax;
            __syncthreads();
            amax = fmaxf(amax, xa[((1 - grp) * RW + wave_r) * 64 + lane]);
        }
        int e = amax > 0.f ? __builtin_amdgcn_frexp_expf(amax) : 0;  // amax = f 2^e with f in [0.5, 1)
        e = e < -100 ? -100 : (e > 120 ? 120 : e);                   // (keeps l 2^-e and 2^-e itself in range)
        const float sc = __builtin_ldexpf(1.f, -e);
        typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
        auto pack4 = [&](int eb, int q4) -> uint2 {  // four neighbouring columns of this lane's row
            const floatx2 lo = {oacc[eb][4 * q4] * sc, oacc[eb][4 * q4 + 1] * sc};
            const floatx2 hi = {oacc[eb][4 * q4 + 2] * sc, oacc[eb][4 * q4 + 3] * sc};
            return make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, halfx2)),
                              __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, halfx2)));
        };
        // Written as the accumulators lie (part_piece_at): a store instruction fills a whole KiB, and nothing passes
        // through LDS.  (KS = 2: half of the columns each.)
        if (row_ok) {
            const int own = part_piece_at(2 * D, 32 * wave_r + n, 4 * EBO * (KS == 2 ? grp : 0) + h);
            auto piece = [&](int j) -> u32x4_t {
                const uint2 lo = pack4(j >> 1, 2 * (j & 1)), hi = pack4(j >> 1, 2 * (j & 1) + 1);
                return u32x4_t{lo.x, lo.y, hi.x, hi.y};
            };
            static_assert(KS == 2 || EBO == EB, "2 EBO pieces, 1024 bytes apart");
            if (NW == 4 && a.merged_elsewhere) {
                const ThroughStore through(pp, (int)part_rows_bytes(a.bm, D, 1));
#pragma unroll
                for (int j = 0; j < 2 * EBO; ++j) through.put16(own + 1024 * j, piece(j));
            } else {
#pragma unroll
                for (int j = 0; j < 2 * EBO; ++j) *(u32x4_t *)(pp + own + 1024 * j) = piece(j);
            }
        }
        if (row_ok && h == 0 && grp == 0) {
            float2 *ml = (float2 *)(pp + part_rows_bytes(a.bm, D, 1));
            ml[rr] = make_float2(m_ref == -INFINITY ? -INFINITY : m_ref + (float)e, l_i * sc);
        }
    }
    KVP_STAMP(31);

    if (clean_from < n_tiles) {
        // Add what the rows see of the infinities and NaNs left out to what was written (weights are
        // positive, so an infinity needs none).
        int j0 = it.kv_begin - it.ctx_len, j1 = it.kv_end - it.ctx_len;  // query rows in the item's range
        if (SRC == SRC_PACKETS) {
            const AttnTile last = load_tile_record(a.tiles, it.kv_end - 1);
            j0 = last.row0 - (n_tiles - 1 - clean_from) * BN;
            j1 = last.row0 + last.n_rows;
        }
        if (j0 < 0) j0 = 0;
        wait_vmcnt<0>();
        __syncthreads();  // the rows are written
        if (SRC == SRC_PACKETS) {
            int any = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) any |= found[w];
            if (!__builtin_amdgcn_readfirstlane(any)) return;
        }
        char *pp = (char *)a.partials + (it.part_slot < 0 ? 0 : (int64_t)it.part_slot * part_slot_bytes(a.bm, D, SPLIT_P ? 0 : 1));
#pragma unroll 1
        for (int u = tid; u < it.n_rows * D; u += NT) {
            const int r = u / D, e = u % D, tr = (it.m0 + r) / g;
            float x = 0.f;
#pragma unroll 1
            for (int j = j0; j < j1 && j <= tr; ++j)
                x += nonfinite_only((uint32_t)*((const bf16_t *)a.v_new + tail_off + (int64_t)j * a.n_kv * D + e) << 16);
            if (x == 0.f) continue;
            bf16_t *op = (bf16_t *)a.out + ((int64_t)(it.q_off + tr) * a.n_q_heads + it.kv_head * g + (it.m0 + r) % g) * D + e;
            if (it.part_slot < 0) *op = f32_to_bf16(ld_elem(op) + x);
            else if (D == 64) *((float *)pp + (int64_t)r * D + e) += x;
            else if (SPLIT_P) *(float *)(pp + part_piece_at(4 * D, r, e >> 2) + 4 * (e & 3)) += x;
            else *(_Float16 *)(pp + part_piece_at(2 * D, r, e / 16 * 2 + (e >> 2 & 1)) + 2 * (e & 3) + (e & 8)) += (_Float16)x;
        }
    }
}

// (256 columns: twice the accumulators and query registers, one wave per SIMD, no register spilled; with a
// second copy of the output product in the loop 22 to 30 were, and the layer above took 59 us)
template <int D, int STAGES, int SRC, int NW, int KS, bool NTL, bool QUAD>
__global__ __launch_bounds__(64 * NW, D == 256 ? 1 : 2) void attention_mfma_kernel(AttnArgs a)
{
    attention_body<D, STAGES, SRC, NW, KS, NTL, QUAD>(a);
}

// 8 waves, 4 stages, the row block chosen item by item: 256 packed rows, or (AttnItem::half_block)
// at most 128 rows handled by two wave groups that take alternate tiles.  A launch of 256-row
// blocks uses it when some groups -- the last rows of a request -- fill at most half a block:
// such an item then holds its compute unit for half the time.
template <int SRC, bool QUAD>
__global__ __launch_bounds__(512, 2) void attention_mfma_mixed_kernel(AttnArgs a)
{
    const bool half = a.inl.n ? false : a.items[blockIdx.x].half_block != 0;  // (regular launches have no half blocks)
    if (half) attention_body<128, 4, SRC, 8, 2, false, QUAD>(a);
    else attention_body<128, 4, SRC, 8, 1, false, QUAD>(a);
}

static int launch_kernel(void (*kernel)(AttnArgs), bool &attr_set, int lds_bytes, int threads, const AttnArgs &a, void *stream)
{
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return (int)e;
        attr_set = true;
    }
    launch(kernel, dim3(a.n_items), dim3(threads), lds_bytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

template <int D, int SRC, int NW, int KS, int STAGES, bool NTL, bool QUAD> static int launch_variant_nt(const AttnArgs &a, void *stream)
{
    constexpr int lds_bytes = STAGES * stage_bytes(D) + NW * 4;
    static bool attr_set = false;
    return launch_kernel(attention_mfma_kernel<D, STAGES, SRC, NW, KS, NTL, QUAD>, attr_set, lds_bytes, 64 * NW, a, stream);
}

// (a.nt_loads: the streaming hint on the tile loads, streams_rows in the planner)
template <int SRC, int NW, int KS, int STAGES> static int launch_variant(const AttnArgs &a, void *stream)
{
    const bool quad = a.g % 4 == 0;
    if (a.nt_loads)
        return quad ? launch_variant_nt<128, SRC, NW, KS, STAGES, true, true>(a, stream) : launch_variant_nt<128, SRC, NW, KS, STAGES, true, false>(a, stream);
    return quad ? launch_variant_nt<128, SRC, NW, KS, STAGES, false, true>(a, stream) : launch_variant_nt<128, SRC, NW, KS, STAGES, false, false>(a, stream);
}

template <int SRC, bool QUAD> static int launch_mixed_as(const AttnArgs &a, void *stream)
{
    constexpr int lds_bytes = 4 * stage_bytes(128) + 8 * 4;
    static bool attr_set = false;
    return launch_kernel(attention_mfma_mixed_kernel<SRC, QUAD>, attr_set, lds_bytes, 512, a, stream);
}

template <int SRC> static int launch_mixed(const AttnArgs &a, void *stream)
{
    return a.g % 4 == 0 ? launch_mixed_as<SRC, true>(a, stream) : launch_mixed_as<SRC, false>(a, stream);
}

template <int NW, int KS, int STAGES> static int launch_nw(const AttnArgs &a, void *stream)
{
    if (a.tiles) return launch_variant<SRC_PACKETS, NW, KS, STAGES>(a, stream);
    return a.cache.layout != 0 ? launch_variant<SRC_PAGED, NW, KS, STAGES>(a, stream)
                               : launch_variant<SRC_CONTIG, NW, KS, STAGES>(a, stream);
}

// Head dims 64 and 256: 128-row blocks of 4 waves.  A tile of 64 columns is half as large, so four
// stages fit where two of 128 columns do; of 256 columns two stages fill the CU's LDS.  (The generic
// kernel served these dims before, with a lane reduction and a block-table walk per score.  Four requests of
// 2K-row paged contexts, 16-64 query rows, per layer: 64 columns 3890 us there, 20.4 here, of which some 4
// keep its precision -- the second bf16 part of P, fp32 partial rows, scores scaled in fp32; 256
// columns 4710 and 43.)
template <int D, int STAGES> static int launch_other_dim(const AttnArgs &a, void *stream)
{
    if (a.bm != 128 || a.tiles) return (int)hipErrorInvalidValue;
    const bool quad = D == 64 && a.g % 4 == 0;  // (256 columns load with plain loads)
    if (a.cache.layout != 0)
        return quad ? launch_variant_nt<D, SRC_PAGED, 4, 1, STAGES, false, D == 64>(a, stream) : launch_variant_nt<D, SRC_PAGED, 4, 1, STAGES, false, false>(a, stream);
    return quad ? launch_variant_nt<D, SRC_CONTIG, 4, 1, STAGES, false, D == 64>(a, stream) : launch_variant_nt<D, SRC_CONTIG, 4, 1, STAGES, false, false>(a, stream);
}

// a.bm selects the row block (128 columns): 256 packed rows (8 waves; a.mixed: with half blocks among them,
// see above) or 128.  128-row blocks run as 4 waves
// with two tile stages (two workgroups per CU), or -- a.split_in_wg, chosen when the launch
// has at most one item per CU -- as 8 waves in two groups that take alternate tiles.
int launch_attention_mfma(const AttnArgs &a, void *stream)
{
    if (a.d == 64) return launch_other_dim<64, 4>(a, stream);
    if (a.d == 256) return launch_other_dim<256, 2>(a, stream);
    if (a.d != 128 || (a.bm != 128 && a.bm != 256)) return (int)hipErrorInvalidValue;
    if (a.bm == 256 && a.mixed) {
        if (a.tiles) return launch_mixed<SRC_PACKETS>(a, stream);
        return a.cache.layout != 0 ? launch_mixed<SRC_PAGED>(a, stream) : launch_mixed<SRC_CONTIG>(a, stream);
    }
    if (a.bm == 256) return launch_nw<8, 1, 4>(a, stream);
    return a.split_in_wg ? launch_nw<8, 2, 4>(a, stream) : launch_nw<4, 1, 2>(a, stream);
}

}  // namespace kvp
