// HIP kernels for gfx950 (CDNA4, wave64): K/V commit (scatter), attention over a paged
// session cache (bf16 MFMA kernel and an fp32 FMA kernel), cross-split log-sum-exp combine,
// gather.  What they compute is defined in include/sk.h; the data layout in sk_internal.h.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "sk_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float sk_f32x4;
typedef __attribute__((ext_vector_type(4))) short sk_s16x4;

#define SK_NEG_INF (-__builtin_inff())
#define SK_LN2 0.6931471805599453f

// ---------------------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float sk_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float sk_log2(float x) { return __builtin_amdgcn_logf(x); }

// Value of lane (i ^ 32) next to the lane's own, with one v_permlane32_swap (no LDS round trip):
// swapping a register with a copy of itself leaves {x[i % 32], x[i % 32 + 32]} in every lane.
struct sk_halves { float lo, hi; };
__device__ __forceinline__ sk_halves sk_both_halves(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return sk_halves{__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// The same for lane (i ^ 16).
__device__ __forceinline__ sk_halves sk_row_pairs(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return sk_halves{__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// Maximum / sum over the 64 lanes, in every lane, without LDS: partners within a quad, quad against quad (mirrored halves
// of a row, whose quads hold one value each by then), half rows, rows, row pairs.  Six dependent vector instructions where
// six shuffles are round trips to the LDS unit, some 100 cycles each.
template <int CTRL> __device__ __forceinline__ float sk_dpp(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float sk_wave_max(float x)
{
    x = fmaxf(x, sk_dpp<0xB1>(x)); x = fmaxf(x, sk_dpp<0x4E>(x)); x = fmaxf(x, sk_dpp<0x141>(x)); x = fmaxf(x, sk_dpp<0x140>(x));
    { const sk_halves h = sk_row_pairs(x); x = fmaxf(h.lo, h.hi); }
    { const sk_halves h = sk_both_halves(x); return fmaxf(h.lo, h.hi); }
}
__device__ __forceinline__ float sk_wave_sum(float x)
{
    x += sk_dpp<0xB1>(x); x += sk_dpp<0x4E>(x); x += sk_dpp<0x141>(x); x += sk_dpp<0x140>(x);
    { const sk_halves h = sk_row_pairs(x); x = h.lo + h.hi; }
    { const sk_halves h = sk_both_halves(x); return h.lo + h.hi; }
}

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f)
{   // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ int sk_divide(const int n, const sk_div d)
{
    return d.mul ? (int)(__umulhi((uint32_t)n, d.mul) >> d.shift) : n;
}

// Requests every 64-byte line of a kernel's argument block at once.  The arguments lie in memory that nothing
// has read yet; left to the compiler they are fetched field by field as the code branches, each first touch of
// a line a round trip of its own in front of the kernel's first useful load (with the divisions below done by
// multiplication and the first tiles requested before the query operand is waited for: first tile in LDS at 2.2
// instead of 3.0 us after a workgroup's start, a 32-token query at 32K 40.2 -> 39.2 us).
template <unsigned BYTES>
__device__ __forceinline__ void sk_touch_arguments()
{
    typedef const __attribute__((address_space(4))) uint32_t* args_ptr;
    const args_ptr a = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr unsigned LINES = (BYTES + 63) / 64;
    uint32_t x[LINES];
#pragma unroll
    for (unsigned i = 0; i < LINES; ++i) x[i] = a[i * 16];
#pragma unroll
    for (unsigned i = 0; i < LINES; ++i) asm volatile("" : : "s"(x[i]));
}

// An argument at byte OFFSET of the block, read from here on and not earlier: left to itself the compiler reads what a loop
// uses in front of it, and the wait for that is one for every scalar load in flight, the first block ids among them.
template <class T, unsigned OFFSET>
__device__ __forceinline__ T sk_late_argument()
{
    typedef const __attribute__((address_space(4))) unsigned char* args_ptr;
    args_ptr a = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr() + OFFSET;
    asm volatile("" : "+s"(a));
    return *(const T*)a;
}

// Work item of workgroup b.  Regular mode derives it from the launch parameters: consecutive
// workgroups differ in KV head first (so with 8 KV heads a head stays on one XCD and its K/V
// stay in that XCD's L2), then in row tile, then in split.
template <bool MAY_BE_F32 = true>
__device__ __forceinline__ int sk_tile_parts(const sk_launch& P, int tok0, int ntok, int* kv_vis_out)
{
    if (MAY_BE_F32 && P.own_mode == SK_OWN_F32) {               // cached keys padded to whole 16-key tiles, then the call's own tokens
        int own = P.own_cnt;
        if (P.pos0 < SK_NO_CAUSAL) own = tok0 + ntok < own ? tok0 + ntok : own;
        *kv_vis_out = ((P.kv_len + 15) & ~15) + own;
        const int np = sk_divide(*kv_vis_out + P.chunk - 1, P.by_chunk);
        return np < 1 ? 1 : np;
    }
    int kv_vis = P.kv_len;
    if (P.pos0 < SK_NO_CAUSAL) {
        int last = P.pos0 + tok0 + ntok;       // last position + 1
        kv_vis = last < kv_vis ? last : kv_vis;
    }
    *kv_vis_out = kv_vis;
    int np = sk_divide(kv_vis + P.chunk - 1, P.by_chunk);
    if (P.eph_cnt[0] > 0 || P.eph_cnt[1] > 0) np += 1;      // uncommitted tokens: own part
    return np < 1 ? 1 : np;
}

__device__ __forceinline__ bool sk_decode_work(const sk_launch& P, int b, sk_work& w)
{
    if (P.mode == SK_MODE_LIST) { w = P.work[b]; return true; }
    const int Hkv = P.g.Hkv;
    const int rest = sk_divide(b, P.by_heads), head = b - rest * Hkv;
    const int split = sk_divide(rest, P.by_tiles);
    int tile = rest - split * P.n_tiles;
    // The last tokens of a chunk see the most keys: they start first, so that a launch of more workgroups than the
    // chip holds ends with its short ones (2,600 tokens into an empty session, 328 workgroups of 1 to 41 iterations on
    // 256 CUs: append and 16-token query 115.6 -> 99.8 us).
    if (P.pos0 < SK_NO_CAUSAL) tile = P.n_tiles - 1 - tile;
    int tok0 = tile * P.tok_per_tile;
    int ntok = P.n_tok - tok0; ntok = ntok < P.tok_per_tile ? ntok : P.tok_per_tile;
    int kv_vis;
    int np = sk_tile_parts<false>(P, tok0, ntok, &kv_vis);
    if (split >= np) return false;
    bool has_eph = (P.eph_cnt[0] > 0 || P.eph_cnt[1] > 0);
    bool eph_part = has_eph && (split == np - 1);
    w.tbl_off = P.tbl_off; w.kv_head = head; w.q_tok0 = tok0; w.n_tok = ntok; w.pos0 = P.pos0 < SK_NO_CAUSAL ? P.pos0 + tok0 : P.pos0;
    w.kv_step = 0;
    if (eph_part) { w.kv_begin = 0; w.kv_end = 0; }
    else if (P.interleave) {          // every split's first piece exists: the host keeps splits <= kv_len / 256
        w.kv_begin = split * 64;
        w.kv_end = kv_vis;
        w.kv_step = (np - (has_eph ? 1 : 0)) * 64;
    } else {
        w.kv_begin = split * P.chunk;
        int e = w.kv_begin + P.chunk;
        w.kv_end = e < kv_vis ? e : kv_vis;
    }
    w.part = np == 1 ? -1 : (tile * P.n_splits + split) * Hkv + head;         // a tile of one part is written directly
    w.unit = tile * Hkv + head; w.part0 = tile * P.n_splits * Hkv + head; w.n_parts = np;
    w.hole_lo = P.hole_lo; w.hole_hi = P.hole_hi;
    w.tok_period = 0; w.sub_blocks = 0; w.once = P.kv_once;
    for (int i = 0; i < 2; ++i) {
        w.eph_blk[i] = P.eph_blk[i]; w.eph_cnt[i] = eph_part ? P.eph_cnt[i] : 0; w.eph_pos0[i] = P.eph_pos0[i];
    }
    return true;
}

// A run of keys the kernel walks through in 16-token groups: either cached tokens of a session
// (through its block table) or an uncommitted segment in the staging area (through a slice of
// an identity table, so both kinds are addressed the same way).
struct sk_seg {
    const unsigned char* base;   // + head offset already applied
    const int32_t* table;        // block of token t = table[t >> log2B]
    int64_t blk_stride;
    int32_t v_off, B, log2B;
    int32_t begin, end;          // token indices; begin is a multiple of 16
    int32_t step;                // iteration i covers the 64 keys from begin + i * step (64: one contiguous run)
    int32_t iterations;
    int32_t pos_shift;           // absolute position = token index + pos_shift
    int32_t hole_lo, hole_n;     // tokens [hole_lo, hole_lo + hole_n) are evicted: streamed, never attended to
    int32_t once;                // 1: no other workgroup of the launch reads these keys (load them non-temporal)
};

// Segment s of a work item: 0 = cached tokens, 1 = first uncommitted segment, 2 + k = second
// uncommitted segment of sub-sequence k (k = 0 unless the tile packs several sequences).
__device__ __forceinline__ sk_seg sk_make_seg(const sk_launch& P, const sk_work& w, int s)
{
    sk_seg g;
    if (s == 0) {
        g.base = P.g.kv + (int64_t)w.kv_head * P.g.head_stride;
        g.table = P.g.tables + w.tbl_off; g.blk_stride = P.g.blk_stride;
        g.v_off = P.g.v_off; g.B = P.g.B; g.log2B = P.g.log2B;
        g.begin = w.kv_begin; g.end = w.kv_end; g.pos_shift = 0;
        g.step = w.kv_step > 0 ? (int)w.kv_step : 64;
        g.iterations = w.kv_step > 0 ? sk_divide(g.end - g.begin + g.step - 1, P.by_step) : (g.end - g.begin + 63) >> 6;
        g.hole_lo = w.hole_lo; g.hole_n = w.hole_hi - w.hole_lo;
        g.once = w.once;
    } else {
        g.base = P.g.eph + (int64_t)w.kv_head * P.g.eph_head_stride;
        g.table = P.g.eph_ident + (s == 1 ? w.eph_blk[0] : w.eph_blk[1] + (s - 2) * w.sub_blocks); g.blk_stride = P.g.eph_blk_stride;
        g.v_off = P.g.eph_v_off; g.B = 16; g.log2B = 4;
        g.begin = 0; g.end = (s == 1 ? w.eph_cnt[0] : w.eph_cnt[1]); g.pos_shift = (s == 1 ? w.eph_pos0[0] : w.eph_pos0[1]);
        g.step = 64; g.iterations = (g.end + 63) >> 6;
        g.hole_lo = 0; g.hole_n = 0;
        g.once = 0;
    }
    return g;
}

__device__ __forceinline__ const unsigned char* sk_group_base(const sk_seg& g, int tg)
{   // base of the block holding the 16-token group that starts at token tg (tg < g.end)
    // Block tables are only written by the commit kernel of an earlier launch, so inside an
    // attention kernel they are constant: reading them through the constant address space makes
    // the lookup a scalar load (it must not count as a vector memory operation, see below).
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    const int blk = ((const_i32_ptr)(uintptr_t)g.table)[tg >> g.log2B];
    return g.base + (int64_t)blk * g.blk_stride;
}

// One wave merges the split partials of one output row (partial row prow0 of the first split, the
// others pstride rows apart):
//   M = max_s m_s ; w_s = 2^(m_s - M) ; O = sum_s O_s w_s / sum_s l_s w_s ; LSE = (M + log2 sum_s lx_s w_s) ln 2
// Lane s holds the statistics of splits s, s + 64, ..; every lane two output dimensions (one when
// d = 64).  The splits are added in index order whoever does this (the combine kernel, or a
// workgroup of the attention kernel, here), with explicit FMAs, so the result depends on the partials only.
// Rows are read 16 splits at a time, the next ones requested before the current ones are used.  The partials were
// written by other workgroups of the same launch (with write-through
// stores); they are read with device-scope loads, which see them wherever the reader runs, so the
// reader needs no cache invalidate (measured at over 10 us when every workgroup issues one).
__device__ __forceinline__ float sk_ld_partial(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <int D>
__device__ __forceinline__ void sk_merge_row(const sk_launch& P, const size_t prow0, const size_t pstride, const int n_parts,
                                             const size_t orow, const int lane)
{
    constexpr int BATCH = 16, d = D;
    constexpr bool two = D == 128;
    const float* obase = P.part_o + prow0 * d + lane;          // dimensions of a lane: lane and lane + 64
    const size_t ostride = pstride * d;
    const float* mlbase = P.part_ml + prow0 * 4;
    const size_t mlstride = pstride * 4;
    auto load_o = [&](const int s, float& x0, float& x1) __attribute__((always_inline)) {
        const float* op = obase + (size_t)s * ostride;
        x0 = sk_ld_partial(op); x1 = two ? sk_ld_partial(op + 64) : 0.f;
    };
    float M = SK_NEG_INF;
    if (n_parts > 64) {              // rare: the maximum needs its own pass
        for (int s = lane; s < n_parts; s += 64) M = fmaxf(M, sk_ld_partial(mlbase + (size_t)s * mlstride));
        M = sk_wave_max(M);
    }
    float L = 0.f, Lx = 0.f, a0 = 0.f, a1 = 0.f;
    for (int base = 0; base < n_parts; base += 64) {
        const int cnt = n_parts - base < 64 ? n_parts - base : 64;
        float x0[BATCH], x1[BATCH], y0[BATCH], y1[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            x0[j] = 0.f; x1[j] = 0.f;
            if (j < cnt) load_o(base + j, x0[j], x1[j]);
        }
        float m_s = SK_NEG_INF, l_s = 0.f, lx_s = 0.f;
        if (lane < cnt) {
            const float* mp = mlbase + (size_t)(base + lane) * mlstride;
            m_s = sk_ld_partial(mp); l_s = sk_ld_partial(mp + 1); lx_s = sk_ld_partial(mp + 2);
        }
        if (n_parts <= 64) M = sk_wave_max(m_s);
        const float wgt = (m_s == SK_NEG_INF) ? 0.f : sk_exp2(m_s - M);
        L = fmaf(l_s, wgt, L); Lx = fmaf(lx_s, wgt, Lx);
        for (int j0 = 0; j0 < cnt; j0 += BATCH) {
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {           // request the next batch
                y0[j] = 0.f; y1[j] = 0.f;
                if (j0 + BATCH + j < cnt) load_o(base + j0 + BATCH + j, y0[j], y1[j]);
            }
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                const float wj = __shfl(wgt, j0 + j, 64);    // 0 for splits past the end
                a0 = fmaf(x0[j], wj, a0); a1 = fmaf(x1[j], wj, a1);
            }
#pragma unroll
            for (int j = 0; j < BATCH; ++j) { x0[j] = y0[j]; x1[j] = y1[j]; }
        }
    }
    L = sk_wave_sum(L); Lx = sk_wave_sum(Lx);
    const float inv = 1.0f / L;
    if (P.out_dtype == 0) {
        float* o = (float*)P.out + orow * d + lane;
        o[0] = a0 * inv;
        if (two) o[64] = a1 * inv;
    } else {
        uint16_t* o = (uint16_t*)P.out + orow * d + lane;
        o[0] = f32_to_bf16_bits(a0 * inv);
        if (two) o[64] = f32_to_bf16_bits(a1 * inv);
    }
    if (P.lse && lane == 0) P.lse[orow] = (M + sk_log2(Lx)) * SK_LN2;
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA attention kernel, head_dim D = 128 (described below) or 64 (the same with four instead
// of eight 16-dim slices of the first contraction and two instead of four 32-dim blocks of the
// second, tiles of half the bytes, and a 256-row instance whose waves do not take turns).
//
// Workgroup = NRG row groups x NPH key phases = 4 or 8 waves: a row group owns 32 query rows, a
// phase owns every NPH-th key tile.  Instances: <4,1,2> 128-row tile; <2,2,2> 64-row tile, the two
// phases merged through LDS at the end; <4,2,2> 128-row tile, eight waves as four row groups x two
// phases; <8,1,4> 256-row tile, eight waves in two groups that take turns on the matrix pipe and
// the vector ALU (head_dim 64: eight waves that interleave both; described at the segment loop).
// Head_dim 64 has no <4,2,2>: with two or three workgroups on a CU the four waves overlap as well (one instance of 32 tokens at
// 131,072 cached, eight waves, one workgroup a CU 65.5 us; four waves, two workgroups 62.0).
//
// Keys move HBM -> LDS with direct-to-LDS loads (global_load_lds_dwordx4), never through
// registers, into a ring of NSS iterations of two 32-key tiles (K 8 KiB + V^T 8 KiB each): 64 KiB
// with two workgroups per CU, or 128 KiB with one (half of each at head_dim 64).  One iteration consumes two tiles (64 keys:
// both by every wave when NPH = 1, one per phase when NPH = 2) while the others are in flight,
// which is what covers the HBM latency.  A direct-to-LDS load writes lane i's 16 bytes at
// base + 16 i, so the bank swizzle is applied to the *source* address each lane picks:
//   K   : LDS row rho holds global 16-byte chunk (c ^ (rho & 15)) at chunk position c,
//   V^T : LDS row dd of a 16-key group holds the two 8-key halves swapped when bit 3 of dd is set.
// The sixteen loads of one tile are issued by four waves (4 instructions each); a wave waits on
// its own vmcnt and a workgroup barrier publishes the tile.  Nothing else in the loop is a vector
// memory instruction (block-table entries are scalar loads), so the outstanding-load count a
// wave waits for is exact.
// Tiles past the end of a segment re-read its last 16-key group (always valid memory); their
// keys are masked by position.  The commit kernel zero-fills V behind the last committed key of
// a 16-key group, so a masked key never contributes 0 * garbage.
//
// Per 32 keys a wave issues
//   S^T[32 keys][32 rows]  = K[32][128] * Q^T[128][32]        8 x mfma_f32_32x32x16_bf16
//   O^T[128][32 rows]     += V^T[128][32 keys] * P^T[32][32]  8 x mfma_f32_32x32x16_bf16
// With S transposed a lane owns one query row (lane % 32) and 16 keys of it, so the row maximum
// and sum need one cross-lane exchange (lane ^ 32, v_permlane32_swap) and P feeds the second contraction straight
// from registers.  Key row rho of the first product is loaded from key tau(rho) (bits 2 and 3
// swapped) so that the 8 P values a lane hands to one PV instruction belong to 8 consecutive
// keys, which are one 16-byte read of V^T.
// Softmax runs in the log2 domain in fp32 against a reference maximum that is only raised when a weight
// may exceed 2^8 (step_softmax), which bounds the weights and makes accumulator rescaling rare; the
// result is the same up to rounding.
// ---------------------------------------------------------------------------------------------
#define SK_TILE 32                 // keys per tile
#define SK_TILE_BYTES 16384        // K 8 KiB | V^T 8 KiB
#define SK_RESCALE_SLACK 8.0f      // log2 of the largest weight before the reference maximum is raised
#define SK_SUM_LIMIT 256.0f        // 2^slack: no weight of a lane whose sum of weights stays below exceeds it

template <int N> struct sk_int { static constexpr int value = N; };
typedef __attribute__((address_space(3))) void* sk_lds_ptr;
// LDS operand addresses are kept in the LDS address space explicitly: through a generic pointer
// the compiler may fall back to flat loads, which also count as vector memory operations.
typedef const __attribute__((address_space(3))) unsigned char* sk_lds_cptr;
typedef __attribute__((ext_vector_type(4))) unsigned sk_u32x4;       // one 16-byte MFMA operand
typedef const __attribute__((address_space(3))) sk_u32x4* sk_lds_u4ptr;
typedef const __attribute__((address_space(1))) void* sk_glb_ptr;

// s_waitcnt vmcnt(n) only (gfx9 encoding: vmcnt = simm16[3:0] | simm16[15:14] << 4)
#define SK_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))

#define SK_LGKMCNT0 0xc07f       // s_waitcnt lgkmcnt(0) only

// Workgroup barrier that orders LDS traffic only.  __syncthreads() would also wait for every
// outstanding global load, i.e. drain the ring of tiles in flight.
__device__ __forceinline__ void sk_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One direct-to-LDS load of 16 bytes per lane: lane i's data lands at lds_addr + IMM + 16 i.
// Written as inline assembly so that the compiler's automatic wait insertion does not drain the
// tiles in flight before every LDS read; the waits are placed by hand (SK_WAIT_VMCNT).
template <unsigned IMM, bool STREAM>
__device__ __forceinline__ void sk_dma16(const void* base, unsigned lane_off, unsigned lds_addr)
{   // address = base (scalar registers) + lane_off (one VGPR, unsigned)
    // STREAM marks the data as used once (cache policy "non-temporal"): it passes through the caches
    // without displacing what other kernels left there.
    if (STREAM)
        asm volatile("s_add_u32 m0, %0, %3\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     : : "s"(lds_addr), "v"(lane_off), "s"(base), "n"(IMM) : "memory", "m0", "scc");
    else
        asm volatile("s_add_u32 m0, %0, %3\n\tglobal_load_lds_dwordx4 %1, %2"
                     : : "s"(lds_addr), "v"(lane_off), "s"(base), "n"(IMM) : "memory", "m0", "scc");
}

// 16-byte store that is written through to memory at once (cache policy "system coherent"), so that
// the split partials never sit as dirty lines in one XCD's L2: the workgroups that merge them may run
// on another XCD, and a release fence wide enough for that would have to walk the whole L2 for dirty
// lines (measured: about 25 us per kernel).  Through a buffer resource, whose bounds drop what lies behind `bytes`: rows
// that are not there need no branch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t sk_bounded(float* base, const int bytes) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000); }
__device__ __forceinline__ void sk_store16_through(const __amdgpu_buffer_rsrc_t to, const unsigned offset, const float4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(sk_u32x4, v), to, offset, 0, 17);      // sc0 sc1
}

// Pool blocks holding the 16-key groups that wave `sub` loads of the tile that starts at key t0 (scalar loads): both, or with
// head_dim 64 group sub >> 1 alone.  Groups past the end of the segment fall back to its last group.
struct sk_tile_blocks { uint32_t blk[2]; };
template <int D>
__device__ __forceinline__ sk_tile_blocks sk_lookup_tile(const sk_seg& g, int t0, int last_group, int sub)
{
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
    sk_tile_blocks b;
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
        int tg = t0 + 16 * (D == 128 ? j : sub >> 1);
        tg = tg < last_group ? tg : last_group;
        b.blk[j] = (uint32_t)((const_i32_ptr)(uintptr_t)g.table)[(unsigned)tg >> g.log2B];
    }
    return b;
}

// Keeps a segment's first block ids together.
template <int D>
__device__ __forceinline__ void sk_together(const sk_tile_blocks& b)
{
#pragma unroll
    for (int j = 0; j < D / 64; ++j) asm volatile("" : : "s"(b.blk[j]));
}

// Issues the four direct-to-LDS loads with which one of four waves contributes to one tile: a K
// and a V^T load for each of the tile's two 16-key groups.  The address arithmetic per load is
// kept short, because a wave issues it in between its vector or matrix work: the block's byte
// offset is a shift (a block of this kernel holds B * 512 bytes per head), the lane-dependent
// part of the address is one VGPR per kind of load, the same for every tile of a segment:
//   K   : the wave fills LDS rows 16 j + 4 sub .. + 3 of group j; lane -> (row rr, chunk position),
//         source chunk (position ^ rr):        koff = rr * 256 + ((lane & 15) ^ rr) * 16
//   V^T : the wave fills dims 32 sub .. + 31 of group j; lane -> (dim dd, half position),
//         source half (position ^ bit 3 of dd): voff = V offset in the block + dd * 32 + (half ^ ((dd >> 3) & 1)) * 16
// and the 16-key group's offset inside a block of more than 16 tokens is added to those.
// In LDS the sixteen 1 KiB units of a tile (K units 0-7, V^T units 8-15) lie US bytes apart, with
// the same unit of the other tiles of the ring in between; `unit_addr` is the address of unit `sub`.
// With head_dim 64 a tile has half the bytes, eight units: K units 0-3 (rows of 128 bytes, eight to a unit), V^T units
// 4-7 (of each 16-key group two).  Wave sub loads K unit sub and V^T unit sub, both of group sub >> 1.
template <unsigned US, int J, int D, bool MAY_STREAM>
__device__ __forceinline__ void sk_issue_group(const sk_seg& g, int t0, int last_group, uint32_t blk,
                                               unsigned unit_addr, unsigned koff, unsigned voff, int j)
{
    constexpr int LOG2_TOK_BYTES = D == 128 ? 8 : 7;       // K bytes per token and head = V^T bytes per token
    int tg = t0 + 16 * j;                                   // j: the group; the constant J with head_dim 128
    tg = tg < last_group ? tg : last_group;
    // the group's place in the block: 256 (128) bytes per token for K, 4 (2) KiB per 16-token group for V^T
    const unsigned char* bb = g.base + ((uint64_t)blk << (g.log2B + LOG2_TOK_BYTES + 1)) + (((unsigned)tg & (unsigned)(g.B - 1)) << LOG2_TOK_BYTES);
    constexpr unsigned KU = J * 4 * US, VU = (D / 16 + J * 4) * US;
    if (MAY_STREAM && g.once) {       // uniform over the workgroup
        sk_dma16<KU, true>(bb, koff, unit_addr);
        sk_dma16<VU, true>(bb, voff, unit_addr);
    } else {
        sk_dma16<KU, false>(bb, koff, unit_addr);
        sk_dma16<VU, false>(bb, voff, unit_addr);
    }
}
template <unsigned US, int D, bool MAY_STREAM>
__device__ __forceinline__ void sk_issue_tile(const sk_seg& g, int t0, int last_group, const sk_tile_blocks& tb,
                                              unsigned unit_addr, unsigned koff, unsigned voff, int sub)
{
    if (D == 128) {
        sk_issue_group<US, 0, D, MAY_STREAM>(g, t0, last_group, tb.blk[0], unit_addr, koff, voff, 0);
        sk_issue_group<US, 1, D, MAY_STREAM>(g, t0, last_group, tb.blk[1], unit_addr, koff, voff, 1);
    } else sk_issue_group<US, 0, D, MAY_STREAM>(g, t0, last_group, tb.blk[0], unit_addr, koff, voff, sub >> 1);
}

// Writes a query's own K/V (at most SK_STAGE_TOKENS tokens, packed rows where the caller has them) into the staging
// blocks of the workgroup's KV head, as the commit kernel lays them out: K rows as they are, V^T through LDS, V zero
// behind the last token of a 16-token group.  The workgroup of the own part, the only one of the launch that reads
// them, does this before it attends to them.
// Bound: two round trips to memory, in a workgroup with one iteration to do while the others walk the cache: the
// launch that staged them took 3 us and a gap (23 tokens at 14,800 cached 25.8 -> 23.1 us; five tokens of a 28/4-head
// layer behind an append 52.6 -> 50.3; 16 tokens behind the append that opens a session 99.8 -> 97.4).
template <int D, int NTHREADS>
__device__ __forceinline__ void sk_stage_own(const sk_launch& P, const sk_work& w, unsigned char* lds, const int tid)
{
    constexpr int CPR = D / 8, LD = D + 8;                  // 16-byte chunks of a row; LDS row length
    uint16_t* vt = (uint16_t*)lds;
    const int cnt = w.eph_cnt[0], n_groups = (cnt + 15) >> 4;
    unsigned char* base = (unsigned char*)P.g.eph + (int64_t)w.kv_head * P.g.eph_head_stride + (int64_t)w.eph_blk[0] * P.g.eph_blk_stride;
    for (int i = tid; i < cnt * CPR; i += NTHREADS) {
        const int row = i / CPR, cc = i % CPR;
        const size_t src = ((size_t)row * P.g.Hkv + w.kv_head) * (D * 2) + cc * 16;
        const uint4 x = *(const uint4*)((const unsigned char*)P.own_k + src), y = *(const uint4*)((const unsigned char*)P.own_v + src);
        *(uint4*)(base + (int64_t)(row >> 4) * P.g.eph_blk_stride + (row & 15) * (D * 2) + cc * 16) = x;
        *(uint4*)(vt + row * LD + cc * 8) = y;
    }
    __syncthreads();
    for (int i = tid; i < n_groups * 2 * D; i += NTHREADS) {
        const int grp = i / (2 * D), dim = (i % (2 * D)) >> 1, t0 = grp * 16 + (i & 1) * 8;      // eight tokens of one dimension
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = t0 + j < cnt ? vt[(t0 + j) * LD + dim] : 0u;
        *(uint4*)(base + (int64_t)grp * P.g.eph_blk_stride + P.g.eph_v_off + dim * 32 + (i & 1) * 16) =
            make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    }
    SK_WAIT_VMCNT(0);                                       // this wave's stores have completed (the barrier alone orders LDS)
    __syncthreads();                                        // so have the others'; LDS is free again
}

template <int NRG, int NPH, int NSS, int D>
__device__ __forceinline__ void sk_attn_bf16_body(const sk_launch P)
{
    static_assert(D == 128 || D == 64, "head_dim");
    constexpr int NKS = D / 16;              // 16-dim slices of the QK^T contraction
    constexpr int NMT = D / 32;              // 32-dim blocks of the output
    constexpr int NW = NRG * NPH;            // waves: 4 or 8
    constexpr int TPI = 2;                   // tiles per iteration (64 keys)
    constexpr int TPW = TPI / NPH;           // tiles per wave per iteration
    // eight waves either as two groups of row groups that take turns (LOCKSTEP, 256 rows), or as two key
    // phases per row group running freely (128 rows: half the arithmetic per wave of the four-wave
    // 128-row instance, two waves per SIMD)
    constexpr bool LOCKSTEP = NW == 8 && NPH == 1 && D == 128, PIPELINED = NW == 8 && NPH == 1 && D == 64;
    // how the reference maximum is kept (step_softmax); at head_dim 128 the four-wave 128-row instance has no registers
    // to keep the scores of two tiles beside their V^T operands
    constexpr bool LAZY_MAX = LOCKSTEP || TPW == 1 || D == 64;
    constexpr int NLG = NW / 4;              // groups of four waves; each loads whole tiles
    static_assert(NW == 4 || ((LOCKSTEP || PIPELINED) && NSS == 4) || (NW == 8 && NPH == 2 && NSS == 2), "four waves, or eight as described");
    static_assert(NSS == 2 || NSS == 4, "ring depth in iterations: 64 KiB (two workgroups per CU) or 128 KiB (one)");
    // The ring holds NSS iterations of TPI tiles.  Its 1 KiB units are interleaved: unit u of tile t
    // of ring slot s sits at (u * TPI * NSS + t * NSS + s) KiB, so that from a lane's per-unit base
    // address every tile of the ring is within reach of the 16-bit offset field of an LDS read.
    constexpr unsigned US = TPI * NSS * 1024;                 // bytes from unit u to unit u + 1
#define SK_SLOT_OFF(s, t) (((t) * NSS + (s)) * 1024)          // tile t of ring slot s, relative to unit bases
    // The epilogue takes a 32 x D tile of floats per wave, which is more than the ring where two key phases share one; the
    // phases' row statistics lie behind both.
    constexpr unsigned RING_BYTES = NSS * TPI * SK_TILE_BYTES * D / 128;
    constexpr unsigned XCH_BYTES = NW * 32 * D * 4;
    constexpr unsigned STAT_BYTES = NPH > 1 ? NW * 32 * 16 : 0;
    __shared__ __attribute__((aligned(16))) unsigned char lds[(RING_BYTES > XCH_BYTES ? RING_BYTES : XCH_BYTES) + STAT_BYTES];

    sk_touch_arguments<sizeof(sk_launch)>();
    sk_work w;
    if (!sk_decode_work(P, blockIdx.x, w)) return;

    const unsigned lds_base = (unsigned)(uintptr_t)(sk_lds_ptr)lds;   // LDS byte address of the ring
    const int tid = threadIdx.x, lane = tid & 63;
    if (P.own_k && w.eph_cnt[0] > 0) sk_stage_own<D, 64 * NW>(P, w, lds, tid);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // in a scalar register
    const int rg = wave % NRG, ph = wave / NRG;
    // Eight waves work as two groups of four that alternate between the matrix pipe and the vector
    // ALU (see the segment loop).  Waves i and i + 4 of a workgroup share a SIMD, so a SIMD holds
    // one wave of each group.  `sub` is the wave's index among the four that load a tile.
    const int grp = LOCKSTEP ? (wave >> 2) : 0;
    const int lg = NLG == 1 ? 0 : (wave >> 2);                     // which tiles of an iteration this wave helps to load (free-running path)
    const int sub = wave & 3;
    const unsigned unit_base = lds_base + sub * US;                // LDS address of this wave's unit of ring slot 0, tile 0
    const int half = PIPELINED ? (wave >> 2) : 0;

    // The block ids a wave's first loads of a segment need, requested together and as the first thing: one by one, each in front of
    // its loads, they are round trips one behind the other.  With the query operand beside them, the first loads right behind and no
    // division on the way the 64-row instance takes 9.2 instead of 10.2 us at 2,600 cached tokens (with the epilogue below) and 80.9
    // instead of 84.4 at 131,072 (right behind an append to the same session; in a stream of queries 85.8 instead of 86.7).
    constexpr int NPRE = PIPELINED ? 5 : LOCKSTEP ? 4 : NSS * (TPI / NLG);
    sk_tile_blocks pre[NPRE];
    auto look_up = [&](const sk_seg& g) __attribute__((always_inline)) {
        const int last_group = g.end > 0 ? (g.end - 1) & ~15 : 0;
#pragma unroll
        for (int i = 0; i < NPRE; ++i) {
            int t = PIPELINED ? g.begin + (half - 1 + 2 * i) * SK_TILE : LOCKSTEP ? g.begin + (1 - grp) * SK_TILE + i * g.step
                              : g.begin + (i / (TPI / NLG)) * g.step + (NLG > 1 ? lg : i % TPI) * SK_TILE;
            if (PIPELINED && i == 0) t = t > g.begin ? t : g.begin;
            pre[i] = sk_lookup_tile<D>(g, t, last_group, sub);
        }
    };
    // Lane-dependent parts of a wave's DMA source addresses in a segment
    // (head_dim 64: lane -> (row rr of eight, chunk position of eight), source chunk (position ^ rr),
    // the wave's rows and dims being those of unit sub & 1 of group sub >> 1).
    const int krow = D == 128 ? sub * 4 + (lane >> 4) : (sub & 1) * 8 + (lane >> 3);
    const unsigned koff = D == 128 ? (unsigned)(krow * 256 + (((lane & 15) ^ krow) << 4))
                                   : (unsigned)(krow * 128 + (((lane & 7) ^ (krow & 7)) << 4));
    const int vdd = (D == 128 ? sub : sub & 1) * 32 + (lane >> 1);
    const unsigned voff0 = (unsigned)(vdd * 32 + ((((lane & 1) ^ ((vdd >> 3) & 1))) << 4));
    // head_dim 64, 256-row tiles: a wave's load of the K tile / V^T tile at key t0: unit `sub`, of group sub >> 1 (128 bytes per token for
    // K and for V^T), and the address of an iteration's ring slot
    auto group_base = [&](const sk_seg& g, const int last_group, const int t0, const sk_tile_blocks& tb) __attribute__((always_inline)) {
        int tg = t0 + 16 * (sub >> 1);
        tg = tg < last_group ? tg : last_group;
        return g.base + ((uint64_t)tb.blk[0] << (g.log2B + 8)) + (((unsigned)tg & (unsigned)(g.B - 1)) << 7);
    };
    auto slot_addr_of = [&](const int it) __attribute__((always_inline)) { return unit_base + (unsigned)((((it + 3) & 3) * 2 + half) * 1024); };
    // A segment's first loads, those of the iterations in front of its loop (the loops say which): their block ids have arrived.
    // The query operand has too: the compiler's wait for it, which does not know of these loads, would be one for all of
    // them behind here, and drain the ring on every iteration inside a loop.
    auto issue_first = [&](const sk_seg& g) __attribute__((always_inline)) {
        const int last_group = (g.end - 1) & ~15;
        const unsigned voff = (unsigned)g.v_off + voff0;
        if constexpr (PIPELINED) {          // "iterations" -4 .. -1 (tiles in front of the segment are not loaded)
#pragma unroll
            for (int it = -4; it < 0; ++it) {
                const int t_k = g.begin + (half + 2 * it + 7) * SK_TILE;
                if (it > -4 || half == 1) sk_dma16<0, false>(group_base(g, last_group, t_k, pre[it + 4]), koff, slot_addr_of(it));
                if (it > -3 || (it == -3 && half == 1)) sk_dma16<NKS * US, false>(group_base(g, last_group, t_k - 2 * SK_TILE, pre[it + 3]), voff, slot_addr_of(it));
            }
        } else if constexpr (LOCKSTEP) {    // iterations 0, 1 (group 1: and 2)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < 2 || grp == 1)
                    sk_issue_tile<US, D, false>(g, g.begin + (1 - grp) * SK_TILE + i * g.step, last_group, pre[i], unit_base + SK_SLOT_OFF(i, 1 - grp), koff, voff, sub);
        } else {                            // iterations 0 .. NSS - 2
#pragma unroll
            for (int a = 0; a < NSS - 1; ++a)
                if (a < g.iterations) {
#pragma unroll
                    for (int p = 0; p < TPI; ++p) {
                        if (NLG > 1 && (p % NLG) != lg) continue;
                        sk_issue_tile<US, D, true>(g, g.begin + a * g.step + p * SK_TILE, last_group, pre[a * (TPI / NLG) + p / NLG], unit_base + SK_SLOT_OFF(a, p), koff, voff, sub);
                    }
                }
        }
    };
    sk_seg g = sk_make_seg(P, w, 0);
    look_up(g);
    __builtin_amdgcn_sched_barrier(0);         // requested here, not behind the query operand's addresses

    const int r = lane & 31, kg = lane >> 5;
    // Row i of a tile is head i % G of token i / G (any group size up to 128; rows past the last
    // whole token of a tile are idle).  Rows are below 256, so the division is a multiplication by
    // ceil(2^16 / G) and a shift, exactly.
    const int G = P.g.G;
    const unsigned g_magic = P.g.g_magic;
    auto div_g = [&](const int row) __attribute__((always_inline)) { return (int)(((unsigned)row * g_magic) >> 16); };
    const int row_in_tile = rg * 32 + r;
    const int tok_local = div_g(row_in_tile);
    const int hq = w.kv_head * G + (row_in_tile - tok_local * G);
    const bool row_valid = tok_local < w.n_tok;

    // Q^T operand: lane (row r, k-group kg) keeps Q[row][16*ks + 8*kg .. +7] for ks = 0..7.  It is on its way beside the block
    // ids, and waited for with them, in front of the first loads into LDS: behind them the compiler's wait, which does not know of those,
    // would be one for all of them (the 256-row kernel, 64 tokens of 32/8 heads at 2,600 cached: 13.5 -> 13.8 us from its first workgroup's
    // start to its last one's end).
    bf16x8 qreg[NKS];
    {
        // Rows past the tile re-read its first token's head row; what they compute goes nowhere.
        const uint4* qp = (const uint4*)((const unsigned char*)P.q +
                          ((size_t)(w.q_tok0 + (row_valid ? tok_local : 0)) * P.g.Hq + hq) * (D * 2));
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qreg[ks] = __builtin_bit_cast(bf16x8, qp[ks * 2 + kg]);
    }
#pragma unroll
    for (int i = 0; i < NPRE; ++i) sk_together<D>(pre[i]);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : : "v"(qreg[ks]));
    if (g.end > g.begin) issue_first(g);

    // positions of the first and last valid token of this wave (wave-uniform); with a group size that
    // does not divide 32 a token's rows can lie in two waves
    const int wave_tok_first = div_g(rg * 32);
    int wave_tok_last = div_g(rg * 32 + 31);
    if (wave_tok_last > w.n_tok - 1) wave_tok_last = w.n_tok - 1;
    const bool wave_has_rows = wave_tok_first < w.n_tok;
    const bool causal = w.pos0 < SK_NO_CAUSAL;
    // A tile may pack several sequences of tok_period tokens each (questions of a batch): token t of
    // the tile is token t % tok_period of sequence t / tok_period, all sequences start at pos0, and
    // each has its own second uncommitted segment.  A wave's rows belong to one sequence (the host
    // only packs when 32 rows divide a sequence's rows).
    int n_sub = 1, wave_sub = 0, t_row = row_valid ? tok_local : wave_tok_last, t_min = wave_tok_first, t_max = wave_tok_last;
    if (w.tok_period > 0) {
        const unsigned period = (unsigned)w.tok_period;
        n_sub = (int)(((unsigned)w.n_tok + period - 1) / period);
        wave_sub = (int)((unsigned)wave_tok_first / period);
        t_row = (int)((unsigned)t_row % period); t_min = (int)((unsigned)t_min % period); t_max = (int)((unsigned)t_max % period);
    }
    const int p_row = causal ? w.pos0 + t_row : 0x7fffffff;
    const int p_wave_min = causal ? w.pos0 + t_min : 0x7fffffff;
    const int p_wave_max = causal ? w.pos0 + t_max : 0x7fffffff;

    f32x16 oacc[NMT];
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[mt][v] = 0.f;
    float m_ref = SK_NEG_INF;
    sk_f32x4 l_acc = {0.f, 0.f, 0.f, 0.f};          // sum of the weights as rounded: element 0 (the others are not kept to the reference)
    sk_s16x4 ones4 = {0x3f80, 0x3f80, 0x3f80, 0x3f80};          // bf16 ones
    if (!LOCKSTEP) asm volatile("" : "+v"(ones4));
    float lx_run = 0.f;                  // sum of the weights before rounding: what the log-sum-exp is taken from
    const float c_scale = P.g.scale_log2e;
    // key tau(rho): swap bits 2 and 3 of the S^T row index
    const int tau = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);

    // lane-dependent LDS addresses of the MFMA operands inside a tile (the XOR swizzles make them
    // irregular in ks, so they are kept in registers; tile and ring-slot offsets are immediates)
    sk_lds_cptr kptr[NKS];
    sk_lds_cptr vptr[NMT];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)       // K row tau is row tau % 4 of unit tau / 4 (head_dim 64: row tau % 8 of unit tau / 8)
        kptr[ks] = D == 128 ? (sk_lds_cptr)lds + SK_SLOT_OFF(0, ph * TPW) + (tau >> 2) * US + (tau & 3) * 256 + (((ks * 2 + kg) ^ (tau & 15)) << 4)
                            : (sk_lds_cptr)lds + SK_SLOT_OFF(0, ph * TPW) + (tau >> 3) * US + (tau & 7) * 128 + (((ks * 2 + kg) ^ (tau & 7)) << 4);
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt) {
        const int dd = mt * 32 + r;
        vptr[mt] = (sk_lds_cptr)lds + SK_SLOT_OFF(0, ph * TPW) + (D / 16 + mt) * US + r * 32 + ((kg ^ ((dd >> 3) & 1)) << 4);   // 16-key group q: + NMT q units
    }

#pragma unroll 1
    for (int s = 0; s < 2 + n_sub; ++s) {
        if (s > 0) g = sk_make_seg(P, w, s);
        if (g.end <= g.begin) continue;
        if (s > 0) {
            sk_lds_barrier();                  // ring free (previous segment fully consumed)
            look_up(g);
            issue_first(g);
        }
        const int niter = g.iterations;          // iteration i: keys from g.begin + i * g.step
        const int last_group = (g.end - 1) & ~15;
        // last position of the segment this wave's rows may see; nothing of another sequence's segment
        const int seg_last_pos = (s >= 2 && s - 2 != wave_sub) ? (int)0x80000000 : g.end - 1 + g.pos_shift;
        const int lim_wave_min = p_wave_min < seg_last_pos ? p_wave_min : seg_last_pos;
        const int lim_wave_max = p_wave_max < seg_last_pos ? p_wave_max : seg_last_pos;
        const int lim_row = p_row < seg_last_pos ? p_row : seg_last_pos;

        const unsigned voff = (unsigned)g.v_off + voff0;

        // ---- the three steps of one iteration (64 keys) for this wave; the ring slot is a
        // compile-time constant so that it folds into the offset field of the LDS instructions ----
        f32x16 sacc[TPW];          // S^T of the iteration in flight
        sk_u32x4 va[TPW][2][NMT];       // its V^T operands (four waves)
        sk_u32x4 va0[4];              // V^T operands of the first 16 keys (eight waves)
        bf16x8 pb[TPW][2];         // its P^T operands

        // first key position of the wave's tiles of iteration `it`, and whether it has work there
        auto first_pos = [&](const int it) __attribute__((always_inline)) { return g.begin + it * g.step + ph * TPW * SK_TILE + g.pos_shift; };
        auto is_active = [&](const int it) __attribute__((always_inline)) {
            return wave_has_rows && g.begin + it * g.step + ph * TPW * SK_TILE < g.end && first_pos(it) <= lim_wave_max;
        };

        // S^T = K Q^T, TPW independent accumulator chains
        // (`soff`: byte offset of the ring slot read, a constant when the loop is unrolled over the slots)
        auto step_scores = [&](const int soff) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) sacc[t][v] = 0.f;
            sk_u32x4 ka[TPW][NKS];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    ka[t][ks] = *(sk_lds_u4ptr)(kptr[ks] + soff + SK_SLOT_OFF(0, t));
            __builtin_amdgcn_s_setprio(2);     // the wave feeding the matrix pipe goes first
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    sacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[t][ks]), qreg[ks], sacc[t], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            // all LDS reads first, then the MFMAs back to back (two independent chains)
            __builtin_amdgcn_sched_group_barrier(0x100, NKS * TPW, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NKS * TPW, 0);
        };
        auto load_v_tile = [&](const int t, const int soff) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt)
                    va[t][q][mt] = *(sk_lds_u4ptr)(vptr[mt] + soff + SK_SLOT_OFF(0, t) + q * NMT * US);
        };
        // a tile is masked when it crosses a causal or end-of-segment limit, or touches evicted tokens
        auto needs_mask = [&](const int it) __attribute__((always_inline)) {
            const int pos_first = first_pos(it);
            return pos_first + TPW * SK_TILE - 1 > lim_wave_min ||
                   (pos_first < g.hole_lo + g.hole_n && pos_first + TPW * SK_TILE > g.hole_lo);
        };
        auto mask_scores = [&](const int it) __attribute__((always_inline)) {
            const int pos_first = first_pos(it);
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int pos = pos_first + t * SK_TILE + 16 * (v >> 3) + 8 * kg + (v & 7);
                    const bool vis = pos <= lim_row && (unsigned)(pos - g.hole_lo) >= (unsigned)g.hole_n;
                    sacc[t][v] = vis ? sacc[t][v] : SK_NEG_INF;
                }
        };
        // The row sum that normalises the output is taken over the weights as the matrix pipe sees
        // them (rounded to bf16), with fp32 accumulation: numerator and
        // denominator of the output then carry the same weights, so a row that one key dominates
        // keeps that key's value to fp32 accuracy whatever the rounding of its weight (with the lazy
        // maximum that weight is not 1).  The log-sum-exp is taken from the unrounded weights
        // (lx_run), so it does not carry the rounding.
        // Four weights of the lane at a time, in the smallest matrix instruction (sixteen 4 x 4 products: with ones on the
        // left, every lane's own four weights are summed; 8 cycles of the matrix pipe), beside the products that use the
        // same weights.  (v_dot2_f32_bf16 sums two, and takes three times its 4.9 cycles while the other wave of the SIMD keeps
        // the matrix pipe busy.  The instance whose groups take turns sums by it all the same, in the vector slot: with it a
        // 48-session step takes 4.12 ms, with the small products in the matrix slot 4.19.)
        auto add_weights = [&](const bf16x8 p, const int h) __attribute__((always_inline)) {
            typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
            l_acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones4, __builtin_bit_cast(sk_s16x4, (uint64_t)__builtin_bit_cast(u64x2, p)[h]), l_acc, 0, 0, 0);
        };
        // P = exp2(s * scale - m) for the reference maximum m as it stands, and the lane's sum of it (unrounded)
        auto weights = [&](const float neg_m) __attribute__((always_inline)) -> float {
            float lx0 = 0.f, lx1 = 0.f;
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const float p0 = sk_exp2(fmaf(sacc[t][v], c_scale, neg_m)), p1 = sk_exp2(fmaf(sacc[t][8 + v], c_scale, neg_m));
                    pb[t][0][v] = (__bf16)p0;
                    pb[t][1][v] = (__bf16)p1;
                    lx0 += p0; lx1 += p1;
                }
            return lx0 + lx1;
        };
        // Softmax of one iteration.  The row maximum is not looked for in every tile: the weights are formed
        // against the reference maximum as it stands, and only when their sum says that one of them may
        // exceed 2^8 (or when there is no reference yet: the sum is then infinite or NaN) does
        // the wave find the tile's maximum, raise the reference, rescale and form them again.  That leaves
        // 16 maxima and a cross-lane exchange out of the vector work of nearly every iteration (256-token
        // append at 32,512 tokens: 128.9 -> 124.4 us; 512 at 130,560: 939 -> 915 us).
        auto step_softmax = [&]() __attribute__((always_inline)) {
            float lx = 0.f;
            bool look = true;
            if (LAZY_MAX) {
                lx = weights(-m_ref);
                look = __any(!(lx <= SK_SUM_LIMIT));
            }
            if (look) {
                float mt_ = SK_NEG_INF;
#pragma unroll
                for (int t = 0; t < TPW; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) mt_ = fmaxf(mt_, sacc[t][v]);
                { const sk_halves h = sk_both_halves(mt_); mt_ = fmaxf(h.lo, h.hi) * c_scale; }      // log2 units (c_scale > 0)
                const bool raise = mt_ > m_ref + (LAZY_MAX ? 0.f : SK_RESCALE_SLACK);
                if (LAZY_MAX || __any(raise)) {
                    const float alpha = raise ? sk_exp2(m_ref - mt_) : 1.0f;
                    l_acc[0] *= alpha; lx_run *= alpha;
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                        for (int v = 0; v < 16; ++v) oacc[mt][v] *= alpha;
                    m_ref = raise ? mt_ : m_ref;
                }
                lx = weights(m_ref == SK_NEG_INF ? 0.f : -m_ref);      // no key seen yet: all weights 0
            }
            lx_run += lx;
            if constexpr (LOCKSTEP) {
                const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
                float ls0 = 0.f, ls1 = 0.f;
#pragma unroll
                for (int t = 0; t < TPW; ++t)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        ls0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t][q], pb[t][q], 0, 1), ones, ls0, false);
                        ls1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t][q], pb[t][q], 2, 3), ones, ls1, false);
                        ls0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t][q], pb[t][q], 4, 5), ones, ls0, false);
                        ls1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[t][q], pb[t][q], 6, 7), ones, ls1, false);
                    }
                l_acc[0] += ls0 + ls1;
            }
        };
        // O^T += V^T P^T for one tile
        auto pv_tile = [&](const int t) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[t][q][mt]), pb[t][q], oacc[mt], 0, 0, 0);
                    if (mt < 2) add_weights(pb[t][q], mt);
                }
        };

        if constexpr (!LOCKSTEP && !PIPELINED) {
            // ---- free-running waves: every wave walks S, softmax, PV of an iteration in turn; overlap of
            // matrix and vector work comes from the other wave of the SIMD (the other workgroup on the
            // CU for the four-wave instances, the other key phase for the eight-wave one) ----
            constexpr int LPW = 4 * TPI / NLG;   // direct-to-LDS loads per wave per iteration (tile p is loaded by wave group p % NLG)
            // block ids of the next refill are looked up one iteration ahead of their use
            sk_tile_blocks nb[TPI];
#pragma unroll
            for (int p = 0; p < TPI; ++p) nb[p] = pre[(NSS - 1) * (TPI / NLG) + p / NLG];

            // `slot` is the ring slot the iteration reads; the slot read by the previous iteration is
            // refilled with iteration it + NSS - 1.  With the two-slot ring the loop is unrolled over the
            // slots (the slot offsets fold into the LDS instructions); a four-slot ring takes the slot at
            // run time (one copy of the loop body).  The instances in use have two slots: with
            // four (three iterations in flight, 128 KiB, one workgroup per CU) a query is slower, as its first tile comes behind three times
            // the bytes of all CUs (kernel, us: 16 tokens at 131,072 cached 80.9 -> 94.0, 32 at 32,768 29.0 -> 30.1, 23 at 14,800 16.4 -> 18.8).
            auto iteration = [&](const int it, const int slot) __attribute__((always_inline)) {
                // this wave's loads of iteration `it` have landed: everything but the loads of the
                // (at most NSS - 2) later iterations already issued
                const int later = niter - 1 - it;
                if (NSS == 2 || later <= 0) SK_WAIT_VMCNT(0);
                else if (later == 1) SK_WAIT_VMCNT(LPW);
                else SK_WAIT_VMCNT(2 * LPW);
                sk_lds_barrier();
                if (it + NSS - 1 < niter) {
#pragma unroll
                    for (int p = 0; p < TPI; ++p) {
                        if (NLG > 1 && (p % NLG) != lg) continue;
                        sk_issue_tile<US, D, true>(g, g.begin + (it + NSS - 1) * g.step + p * SK_TILE, last_group, nb[p],
                                                       unit_base + SK_SLOT_OFF((slot + NSS - 1) % NSS, p), koff, voff, sub);
                    }
                    if (it + NSS < niter) {
#pragma unroll
                        for (int p = 0; p < TPI; ++p)
                            nb[p] = sk_lookup_tile<D>(g, g.begin + (it + NSS) * g.step + (NLG > 1 ? lg : p) * SK_TILE, last_group, sub);
                    }
                }
                if (!is_active(it)) return;
                step_scores(slot * 1024);
#pragma unroll
                for (int t = 0; t < TPW; ++t) load_v_tile(t, slot * 1024);   // requested now: their LDS latency hides behind the softmax
                if (needs_mask(it)) mask_scores(it);
                step_softmax();
#pragma unroll
                for (int t = 0; t < TPW; ++t) pv_tile(t);
            };
            if constexpr (NSS == 2) {
                for (int it = 0; it < niter; it += 2) {
                    iteration(it, 0);
                    if (it + 1 < niter) iteration(it + 1, 1);
                }
            } else {
#pragma unroll 1
                for (int it = 0; it < niter; ++it) iteration(it, it & (NSS - 1));
            }
        } else if constexpr (PIPELINED) {
            // ---- eight waves, each of which interleaves matrix and vector work instruction by instruction.  A stage
            // is one tile: S of the next tile and P V of the last one (matrix instructions, alternating, so that neither chain
            // waits for itself) with the weights of this one in between; the operand of a matrix instruction is read from
            // LDS eight of them ahead.  An iteration is two stages with one workgroup barrier in front.
            // Ring: a tile's K is read one stage before its weights and its V^T one stage behind, so K tile i lies in
            // slot i - 1 and V^T tile i in slot i + 1 (mod 8): iteration j reads slots 2j and 2j + 1 of both.  In iteration j a
            // wave issues its loads of the K tiles 2j + 7, 2j + 8 and the V^T tiles 2j + 5, 2j + 6 (one of each, by
            // `half`), whose slots iteration j - 1 has read for the last time; it waits for them before the barrier of
            // iteration j + 2, whose second stage reads ahead into iteration j + 3.
            // Bound: issue.  A vector instruction beside matrix instructions of the same SIMD takes 8.8 cycles instead of 4.9
            // (v_exp_f32 12.7 instead of 8.8; v_dot2_f32_bf16 14.8, hence add_weights): a stage of a SIMD's two waves takes about
            // 1,200 cycles for 576 of matrix and 700 of vector instructions.  256 tokens of 32/8 heads at 32,512 cached, with the
            // combine and the commit kernel: 96.5 us with 128-row tiles of four waves that walk S, softmax and P V in turn, 88.4
            // with these; 512 at 130,560: 665 -> 618; the last ones of 2,600 into an empty session 63.4 -> 60.9.
            constexpr int LPW = 2;               // direct-to-LDS loads per wave and iteration: one of K, one of V^T
            constexpr int NP = 2 * NKS;          // matrix instructions of a stage
            constexpr int VP = 16 / NP;          // weights formed beside each
            static_assert(NKS == 4 && NMT == 2, "a stage has as many matrix instructions of either product; a tile is eight units, two loads of each of four waves");
            const int n_iter = niter;
            // Iterations that any row of this wave sees a key of.  In the others it loads its share of the tiles and computes
            // nothing: a weight of 0 times an infinite value would be NaN, and reach rows of questions and of tokens that lie in
            // front of that value (the 32 keys of one tile, and the two tiles of an iteration, are not told apart).
            const int first_0 = g.begin + g.pos_shift;
            int n_live = !wave_has_rows || lim_wave_max < first_0 ? 0 : (int)((unsigned)(lim_wave_max - first_0) / (2 * SK_TILE)) + 1;
            n_live = n_live < n_iter ? n_live : n_iter;
            auto& kc = kptr;                     // operand addresses: they follow the iteration through the ring
            auto& vc = vptr;
            f32x16 sc[2];
            sk_u32x4 pw[2][2];
            sk_u32x4 op[8];

            // block ids of the K tile loaded next and of the V tile, which is the K tile of the iteration before
            int t_k = g.begin + (half + 7) * SK_TILE;
            sk_tile_blocks kb = pre[4], vb = pre[3];
            auto issue_k = [&](const unsigned slot_addr) __attribute__((always_inline)) { sk_dma16<0, false>(group_base(g, last_group, t_k, kb), koff, slot_addr); };
            auto issue_v = [&](const unsigned slot_addr) __attribute__((always_inline)) { sk_dma16<NKS * US, false>(group_base(g, last_group, t_k - 2 * SK_TILE, vb), voff, slot_addr); };
            auto next_blocks = [&]() __attribute__((always_inline)) {
                t_k += 2 * SK_TILE;
                vb = kb;
                kb = sk_lookup_tile<D>(g, t_k, last_group, sub);
            };

            // tiles that need a mask
            const int last_0 = g.begin + g.pos_shift + SK_TILE - 1;             // last position of tile 0
            const int n_free = lim_wave_min < last_0 ? 0 : (int)((unsigned)(lim_wave_min - last_0) / SK_TILE) + 1;
            int hole_t = 0, hole_ts = 0;
            if (g.hole_n > 0 && g.hole_lo < g.end && g.hole_lo + g.hole_n > g.begin) {
                hole_t = g.hole_lo > g.begin ? (g.hole_lo - g.begin) / SK_TILE : 0;
                hole_ts = (g.hole_lo + g.hole_n - g.begin) / SK_TILE + 1 - hole_t;
            }
            auto mask_tile = [&](const int t, f32x16& s) __attribute__((always_inline)) {
                if (!(t >= n_free || (unsigned)(t - hole_t) < (unsigned)hole_ts)) return;
                const int pos_first = g.begin + t * SK_TILE + g.pos_shift;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int pos = pos_first + 16 * (v >> 3) + 8 * kg + (v & 7);
                    const bool vis = pos <= lim_row && (unsigned)(pos - g.hole_lo) >= (unsigned)g.hole_n;
                    s[v] = vis ? s[v] : SK_NEG_INF;
                }
            };
            // operand of position p of a stage: even, K slice p / 2; odd, V^T block p / 2 (16-key group, then 32 dims)
            auto ld_op = [&](const int p, const int off) __attribute__((always_inline)) -> sk_u32x4 {
                if ((p & 1) == 0) return *(sk_lds_u4ptr)(kc[p >> 1] + off);
                const int i = p >> 1;
                return *(sk_lds_u4ptr)(vc[i % NMT] + off + (i / NMT) * NMT * US);
            };
            // One stage: S of the next tile, the weights of this one, P V of the last one, instruction by instruction.
            auto stage = [&](auto half_const, auto pv_const, const int tile, const int delta, const f32x16& zero, f32x16& cur, f32x16& nxt,
                             sk_u32x4 (&p_old)[2], sk_u32x4 (&p_new)[2], auto extra) __attribute__((always_inline)) {
                constexpr int HALF = decltype(half_const)::value;
                constexpr bool PV = decltype(pv_const)::value != 0;
                if (PV || HALF == 1) mask_tile(tile, cur);
                const float neg_m = -m_ref;
                float x[17], e[16], lx0 = 0.f, lx1 = 0.f;
                auto pair = [&](const int i) __attribute__((always_inline)) {
                    uint32_t w2 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)e[2 * i], (__bf16)e[2 * i + 1]});
                    asm volatile("" : "+v"(w2));         // here, not behind the branch below
                    p_new[i >> 2][i & 3] = w2;
                };
                x[0] = fmaf(cur[0], c_scale, neg_m);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    if ((p & 1) == 0) nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[p & 7]), qreg[p >> 1], p == 0 ? zero : nxt, 0, 0, 0);
                    else if (PV) {
                        const int i = p >> 1;
                        oacc[i % NMT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[p & 7]), __builtin_bit_cast(bf16x8, p_old[i / NMT]), oacc[i % NMT], 0, 0, 0);
                        if (i % NMT < 2) add_weights(__builtin_bit_cast(bf16x8, p_old[i / NMT]), i % NMT);
                    }
                    // the operand of eight positions later
                    if (p + 8 < NP) op[p & 7] = ld_op(p + 8, HALF * 1024);
                    else {
                        const int t = p + 8 - NP, i = t >> 1;
                        if (HALF == 1) {
                            if ((t & 1) == 0) kc[i] += delta;
                            else if (i < NMT) vc[i] += delta;
                        }
                        op[p & 7] = ld_op(t, HALF == 0 ? 1024 : 0);
                    }
#pragma unroll
                    for (int u = 0; u < VP; ++u) {
                        const int v = p * VP + u;
                        if (v < 15) x[v + 1] = fmaf(cur[v + 1], c_scale, neg_m);
                        e[v] = sk_exp2(x[v]);
                        if (v >= 1) { if (v & 1) lx0 += e[v - 1]; else lx1 += e[v - 1]; }
                        if (v >= 2 && (v & 1) == 0) pair(v / 2 - 1);
                    }
                    extra(p);
                    __builtin_amdgcn_sched_barrier(0);
                }
                lx1 += e[15];
                pair(7);
                float lx = lx0 + lx1;
                if (__builtin_expect(__any(!(lx <= SK_SUM_LIMIT)), 0)) {
                    float mt_ = SK_NEG_INF;
#pragma unroll
                    for (int v = 0; v < 16; ++v) mt_ = fmaxf(mt_, cur[v]);
                    { const sk_halves h = sk_both_halves(mt_); mt_ = fmaxf(h.lo, h.hi) * c_scale; }
                    const bool raise = mt_ > m_ref;
                    const float alpha = raise ? sk_exp2(m_ref - mt_) : 1.0f;
                    l_acc[0] *= alpha; lx_run *= alpha;
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                        for (int v = 0; v < 16; ++v) oacc[mt][v] *= alpha;
                    m_ref = raise ? mt_ : m_ref;
                    const float neg = m_ref == SK_NEG_INF ? 0.f : -m_ref;
                    lx0 = lx1 = 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        e[v] = sk_exp2(fmaf(cur[v], c_scale, neg));
                        if (v & 1) lx1 += e[v]; else lx0 += e[v];
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) pair(i);
                    lx = lx0 + lx1;
                }
                lx_run += lx;
            };
            f32x16 zero;
#pragma unroll
            for (int v = 0; v < 16; ++v) zero[v] = 0.f;

            // S of tile 0, and the first reference: a row's maximum over its first two tiles, the 64 keys the other instances take it
            // from.  The more keys it is taken from, the more often the row's largest weight is exactly 1 and not rounded: error
            // against 64 bits over the first tile alone and over two, 1,500 tokens of 32/8 heads into an empty session 1.30e-3 and
            // 1.27e-3, 300 behind 2,600 1.62e-3 and 1.60e-3, 256 behind 32,512 1.658e-3 and 1.656e-3.
            if (half == 1) SK_WAIT_VMCNT(5);
            else SK_WAIT_VMCNT(4);
            sk_lds_barrier();
            // K tile 0 lies in slot 7, tile 1 in slot 0 (a tile's K one slot below its number, its V one above)
            if (n_live > 0) {
                auto scores = [&](const int off) __attribute__((always_inline)) {
                    sk_u32x4 k0[NKS];
#pragma unroll
                    for (int i = 0; i < NKS; ++i) k0[i] = *(sk_lds_u4ptr)(kc[i] + off);
                    f32x16 s0 = zero;
#pragma unroll
                    for (int i = 0; i < NKS; ++i) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k0[i]), qreg[i], s0, 0, 0, 0);
                    return s0;
                };
                sc[0] = scores(7 * 1024);
                mask_tile(0, sc[0]);                 // (the first stage does not again)
                if (__any(m_ref == SK_NEG_INF)) {
                    float mt_ = SK_NEG_INF;
#pragma unroll
                    for (int v = 0; v < 16; ++v) mt_ = fmaxf(mt_, sc[0][v]);
                    if (first_0 + SK_TILE <= lim_wave_max) {
                        f32x16 s1 = scores(0);
                        mask_tile(1, s1);
#pragma unroll
                        for (int v = 0; v < 16; ++v) mt_ = fmaxf(mt_, s1[v]);
                    }
                    { const sk_halves h = sk_both_halves(mt_); mt_ = fmaxf(h.lo, h.hi) * c_scale; }
                    m_ref = m_ref == SK_NEG_INF ? mt_ : m_ref;
                }
            }
            auto begin_iteration = [&]() __attribute__((always_inline)) {
                SK_WAIT_VMCNT(LPW);
                sk_lds_barrier();
            };
            auto iteration = [&](auto pv_const, const int it) __attribute__((always_inline)) {
                const unsigned sa = slot_addr_of(it);
                const int delta = ((it + 1) & 3) == 0 ? -6 * 1024 : 2 * 1024;
                stage(sk_int<0>{}, pv_const, 2 * it, delta, zero, sc[0], sc[1], pw[1], pw[0], [&](const int p) __attribute__((always_inline)) {
                    if (p == 3) issue_k(sa);
                });
                stage(sk_int<1>{}, sk_int<1>{}, 2 * it + 1, delta, zero, sc[1], sc[0], pw[0], pw[1], [&](const int p) __attribute__((always_inline)) {
                    if (p == 3) issue_v(sa);
                    if (p == NP - 3) next_blocks();
                });
            };
            if (n_live > 0) {
                begin_iteration();
#pragma unroll
                for (int p = 0; p < 8; ++p) op[p] = ld_op(p, 0);
                iteration(sk_int<0>{}, 0);
#pragma unroll 1
                for (int it = 1; it < n_live; ++it) {
                    begin_iteration();
                    iteration(sk_int<1>{}, it);
                }
                // P V of the last tile: its V^T lies where the next iteration's first stage would read it (loaded three
                // iterations ahead, so the barrier in front of this iteration has published it)
#pragma unroll
                for (int i = 0; i < 2 * NMT; ++i) {
                    oacc[i % NMT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ld_op(2 * i + 1, 0)), __builtin_bit_cast(bf16x8, pw[1][i / NMT]), oacc[i % NMT], 0, 0, 0);
                    if (i % NMT < 2) add_weights(__builtin_bit_cast(bf16x8, pw[1][i / NMT]), i % NMT);
                }
#pragma unroll
                for (int i = 0; i < NKS; ++i) kc[i] -= (n_live & 3) * 2048;
#pragma unroll
                for (int i = 0; i < NMT; ++i) vc[i] -= (n_live & 3) * 2048;
            }
#pragma unroll 1
            for (int it = n_live; it < n_iter; ++it) {          // the same loads, waits and barriers
                begin_iteration();
                const unsigned sa = slot_addr_of(it);
                issue_k(sa);
                issue_v(sa);
                next_blocks();
            }
            SK_WAIT_VMCNT(0);                    // nothing is still on its way into the ring
            sk_lds_barrier();
        } else {
            // ---- eight waves in two groups of four that take turns.  Every wave alternates between
            // a matrix slot (P V of iteration j-1, then S of iteration j) and a vector slot (softmax
            // of iteration j), with a workgroup barrier in front of each; group 1 runs the same
            // sequence one barrier behind group 0, so that whenever one group is in a matrix slot the
            // other is in a vector slot.  A SIMD holds one wave of each group: its matrix pipe and
            // its vector ALU are busy at the same time.
            //   barrier number    2j              2j+1            2j+2
            //   group 0           | PV(j-1) S(j)  | softmax(j)    | PV(j) S(j+1)
            //   group 1           | softmax(j-1)  | PV(j-1) S(j)  | softmax(j)
            // Iteration i lives in ring slot i % 4 and is read between barriers 2i and 2i+4.  Group
            // 0 loads the second tile of every iteration, group 1 the first; a wave issues the loads
            // of iteration j + 2 + grp at the start of its vector slot j (after barrier 2j+1+grp >=
            // 2(j + grp - 2) + 4, so the ring slot is free) and waits for its loads of iteration i
            // before its barrier number 2i, after which the whole iteration is in LDS.
            // The ring slot is a run-time value here (one copy of the loop body): the operand
            // addresses of the current slot are rebuilt from the per-unit bases once per iteration.
            // Every wave does every iteration (rows or keys that do not count are masked): the slots
            // are synchronised, so skipping work would not save time.
            // Bound: the matrix slot (its operands come from LDS, and the two kinds of slot overlap only partly) at the clock the
            // chip holds under it: at 32,512 cached tokens an iteration takes about 3,000 cycles for 2,048 of matrix
            // instructions per SIMD (counters: matrix pipe busy 0.62 of the cycles), 256 tokens 122-124 us = 1.10-1.12 PFLOP/s;
            // 512 at 130,560 run at 1.18-1.22 where the bare matrix loop holds 1.85 and a library product of 8192^3 1.41.
            constexpr int LPW = 4;               // direct-to-LDS loads per wave per iteration (one tile)
            const int my_tile = 1 - grp;
            const int ahead = 2 + grp;           // iterations loaded before the loop (issue_first)
            // Loads are issued for `ahead` iterations past the end too (they re-read the segment's last
            // group and nothing reads them), so that the number of loads in flight at each wait is a constant.
            int t_next = g.begin + my_tile * SK_TILE + ahead * g.step;
            sk_tile_blocks nb = grp == 1 ? pre[3] : pre[2];
            auto issue_next = [&](const int slot) __attribute__((always_inline)) {
                sk_issue_tile<US, D, false>(g, t_next, last_group, nb, unit_base + SK_SLOT_OFF(slot, my_tile), koff, voff, sub);
                t_next += g.step;
                nb = sk_lookup_tile<D>(g, t_next, last_group, sub);
            };
            SK_WAIT_VMCNT(LPW);                  // iteration 0 has landed (group 1: and iteration 1)
            if (grp == 1) sk_lds_barrier();      // group 1 stays one barrier behind
            // Matrix slot: eight groups of four matrix instructions, P V of the previous iteration
            // (V^T through vp, the pointers of its ring slot) and S of the current one (K through
            // kc).  Operands stream from LDS two groups ahead of their use, into the registers that
            // earlier groups have released (the scheduling barriers keep that order); the first
            // group's were read in the vector slot.  KIND 0: first slot of a segment, S only;
            // 2: last slot, P V only.
            auto matrix_slot = [&](auto kind_const, const int j, const sk_lds_cptr (&kc)[8], const sk_lds_cptr (&vp)[4])
                                   __attribute__((always_inline)) {
                constexpr int KIND = decltype(kind_const)::value;
                auto ld_v = [&](sk_u32x4 (&o)[4], const int t, const int q) __attribute__((always_inline)) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) o[mt] = *(sk_lds_u4ptr)(vp[mt] + SK_SLOT_OFF(0, t) + q * 4 * US);
                };
                auto mm_v = [&](const sk_u32x4 (&o)[4], const int t, const int q) __attribute__((always_inline)) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt)
                        oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o[mt]), pb[t][q], oacc[mt], 0, 0, 0);
                };
                auto ld_k = [&](sk_u32x4 (&o)[4], const int kk) __attribute__((always_inline)) {      // ks = 2 kk, 2 kk + 1; both tiles
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = *(sk_lds_u4ptr)(kc[kk * 2 + (i >> 1)] + SK_SLOT_OFF(0, i & 1));
                };
                auto mm_k = [&](const sk_u32x4 (&o)[4], const int kk) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        sacc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o[i]), qreg[kk * 2 + (i >> 1)], sacc[i & 1], 0, 0, 0);
                };
                auto clear_scores = [&]() __attribute__((always_inline)) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int v = 0; v < 16; ++v) sacc[t][v] = 0.f;
                };
#define SK_SB __builtin_amdgcn_sched_barrier(0)
                sk_u32x4 o1[4], o2[4], o3[4], o4[4], o5[4], o6[4], o7[4];
                if (KIND == 1) {
                    ld_v(o1, 0, 1); ld_v(o2, 1, 0); SK_SB;
                    mm_v(va0, 0, 0); SK_SB; ld_v(o3, 1, 1); SK_SB;
                    mm_v(o1, 0, 1); SK_SB; ld_k(o4, 0); SK_SB;
                    mm_v(o2, 1, 0); SK_SB; ld_k(o5, 1); SK_SB;
                    mm_v(o3, 1, 1); SK_SB; ld_k(o6, 2); SK_SB;
                    clear_scores(); mm_k(o4, 0); SK_SB; ld_k(o7, 3); SK_SB;
                    mm_k(o5, 1); SK_SB;
                    mm_k(o6, 2); SK_SB;
                    mm_k(o7, 3);
                } else if (KIND == 0) {
                    ld_k(o4, 0); ld_k(o5, 1); ld_k(o6, 2); ld_k(o7, 3);
                    clear_scores();
                    mm_k(o4, 0); mm_k(o5, 1); mm_k(o6, 2); mm_k(o7, 3);
                } else {
                    ld_v(o1, 0, 1); ld_v(o2, 1, 0); ld_v(o3, 1, 1);
                    mm_v(va0, 0, 0); mm_v(o1, 0, 1); mm_v(o2, 1, 0); mm_v(o3, 1, 1);
                }
#undef SK_SB
            };
            // Iterations that need a mask: those that reach past what the wave's first row may see, and those
            // that touch evicted tokens.
            const int last_0 = g.begin + g.pos_shift + TPI * SK_TILE - 1;       // last position of iteration 0
            const int n_free = lim_wave_min < last_0 ? 0 : (int)((unsigned)(lim_wave_min - last_0) / (unsigned)g.step) + 1;      // iterations the limit leaves whole
            int hole_it = 0, hole_its = 0;
            if (g.hole_n > 0 && g.hole_lo < g.end && g.hole_lo + g.hole_n > g.begin) {
                hole_it = g.hole_lo > g.begin ? (g.hole_lo - g.begin) / g.step : 0;
                hole_its = (g.hole_lo + g.hole_n - g.begin) / g.step + 1 - hole_it;
            }
            auto mask_iteration = [&](const int j) __attribute__((always_inline)) {
                if (j >= n_free || (unsigned)(j - hole_it) < (unsigned)hole_its) mask_scores(j);
            };
            // Vector slot: softmax of iteration j, and the operands of the first group of matrix
            // instructions of the slot that follows (V^T, first 16 keys of the iteration).
            auto vector_slot = [&](const int j, const sk_lds_cptr (&vc)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) va0[mt] = *(sk_lds_u4ptr)(vc[mt]);
                __builtin_amdgcn_sched_barrier(0);
                mask_iteration(j);
                step_softmax();
                // (the scalar loads of the block ids have long arrived; said here, so that the matrix slot's
                // waits for its LDS operands need not allow for them and can count)
                __builtin_amdgcn_s_waitcnt(SK_LGKMCNT0);
            };
            sk_lds_cptr kc[8];          // K operand addresses in the ring slot of the current iteration
            sk_lds_cptr vc[4];          // V^T operand addresses in it (the next matrix slot reads them as "previous")
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) kc[ks] = kptr[ks];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) vc[mt] = vptr[mt];
            // slots of iteration 0 (ring slot 0): S only
            sk_lds_barrier();
            matrix_slot(sk_int<0>{}, 0, kc, vc);
            if (grp == 1) SK_WAIT_VMCNT(LPW);
            sk_lds_barrier();
            issue_next(ahead);
            vector_slot(0, vc);
#pragma unroll 1
            for (int j = 1; j < niter; ++j) {
                sk_lds_cptr vp[4];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) { vp[mt] = vc[mt]; vc[mt] = vptr[mt] + (j & 3) * 1024; }
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) kc[ks] = kptr[ks] + (j & 3) * 1024;
                // a wave waits for its own loads of the iteration that is published by its next barrier of
                // even number; those of one later iteration stay in flight
                if (grp == 0) SK_WAIT_VMCNT(LPW);
                sk_lds_barrier();                                  // barrier 2j (group 0), 2j+1 (group 1)
                __builtin_amdgcn_s_setprio(2);                     // the wave feeding the matrix pipe goes first (1.8 % of the kernel)
                matrix_slot(sk_int<1>{}, j, kc, vp);
                __builtin_amdgcn_s_setprio(0);
                if (grp == 1) SK_WAIT_VMCNT(LPW);
                sk_lds_barrier();                                  // barrier 2j+1 (group 0), 2j+2 (group 1)
                issue_next((j + ahead) & 3);
                vector_slot(j, vc);
            }
            // slots after the last iteration: P V only
            sk_lds_barrier();
            matrix_slot(sk_int<2>{}, niter, kc, vc);
            SK_WAIT_VMCNT(0);                    // nothing is still on its way into the ring
            sk_lds_barrier();
            if (grp == 0) sk_lds_barrier();      // the barrier group 1 took first
        }
    }

    float l_tot; { const sk_halves h = sk_both_halves(l_acc[0]); l_tot = h.lo + h.hi; }
    float lx_tot; { const sk_halves h = sk_both_halves(lx_run); lx_tot = h.lo + h.hi; }

    // ---- epilogue: rows go out through LDS so that every store instruction writes whole rows ----
    // A lane holds 4-float pieces of ONE row (its accumulators are O^T); written as they are, a store
    // instruction would touch 64 different 128-byte lines.  Each wave writes its 32 x D tile to LDS (the ring is
    // idle by then), XOR-swizzled by row so both directions are conflict-free.  With two key phases the waves first tell each
    // other their reference maxima, scale by them, and the rows of both are added on the way out: every wave stores half of
    // its row group's rows.
    // Bound: round trips of a wave to LDS.  The values of a batch of stores are read before the first of them goes out: with
    // each read in front of its store that was 16 round trips, 1.8 us of a workgroup; the phases merged in registers by half of the waves, and only those storing, took another 1.8.
    const bool direct = w.part < 0;
    const int nrows = w.n_tok * G;
    float factor = 1.0f;
    constexpr unsigned STATS = RING_BYTES > XCH_BYTES ? RING_BYTES : XCH_BYTES;         // behind the ring: it may still be read
    if (NPH > 1) {
        float4* stat = (float4*)(lds + STATS) + (ph * NRG + rg) * 32 + r;
        if (kg == 0) *stat = make_float4(m_ref, l_tot, lx_tot, 0.f);
        __syncthreads();                              // every wave is done reading key tiles, and has written its statistics
        const float4 other = *((const float4*)(lds + STATS) + ((ph ^ 1) * NRG + rg) * 32 + r);
        const float M = fmaxf(m_ref, other.x);
        const float a_own = (m_ref == SK_NEG_INF) ? 0.f : sk_exp2(m_ref - M);
        const float a_other = (other.x == SK_NEG_INF) ? 0.f : sk_exp2(other.x - M);
        factor = a_own;
        l_tot = l_tot * a_own + other.y * a_other;
        lx_tot = lx_tot * a_own + other.z * a_other;
        m_ref = M;
    } else __syncthreads();                           // every wave is done reading key tiles
    if (direct) factor *= 1.0f / l_tot;
    {
        float* tr = (float*)lds + wave * (32 * D);
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int c4 = mt * 8 + q4 * 2 + kg;
                *(float4*)(tr + r * D + ((c4 ^ r) & (D / 4 - 1)) * 4) =
                    make_float4(oacc[mt][q4 * 4 + 0] * factor, oacc[mt][q4 * 4 + 1] * factor, oacc[mt][q4 * 4 + 2] * factor, oacc[mt][q4 * 4 + 3] * factor);
            }
        const size_t orow_lane = ((size_t)(w.q_tok0 + tok_local) * P.g.Hq + hq);
        if (row_valid && kg == 0 && ph == 0) {
            if (direct) { if (P.lse) P.lse[orow_lane] = (m_ref + sk_log2(lx_tot)) * SK_LN2; }
            else sk_store16_through(sk_bounded(P.part_ml + (size_t)w.part * P.rows_per_slot * 4, nrows * 16), row_in_tile * 16, make_float4(m_ref, l_tot, lx_tot, 0.f));
        }
    }
    if (NPH > 1) __syncthreads();                     // the other phase's rows are there too
    {
        // a row is D / 4 chunks of four floats: a store instruction writes two rows (four at head_dim 64)
        constexpr int CPR = D / 4, RPI = 64 / CPR, ROWS = 32 / NPH, NIT = ROWS / RPI, BATCH = NIT < 8 ? NIT : 8;
        const int c4 = lane & (CPR - 1);
        const float* tr = (const float*)lds + rg * (32 * D);
#pragma unroll
        for (int b0 = 0; b0 < NIT; b0 += BATCH) {
            // the row order is rotated by the workgroup index: workgroups that finish together (short
            // contexts) would otherwise all write the same offset of their partial slots, which lie a
            // power of two apart, at the same time, and crowd onto a few memory channels
            auto row_of = [&](const int i) __attribute__((always_inline)) { return ph * ROWS + ((b0 + i + (int)blockIdx.x) & (NIT - 1)) * RPI + lane / CPR; };
            float4 val[BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int row = row_of(i), at = row * D + ((c4 ^ row) & (D / 4 - 1)) * 4;
                val[i] = *(const float4*)(tr + at);
                if (NPH > 1) {
                    const float4 y = *(const float4*)(tr + NRG * 32 * D + at);
                    val[i].x += y.x; val[i].y += y.y; val[i].z += y.z; val[i].w += y.w;
                }
            }
            if (!direct) {
                const __amdgpu_buffer_rsrc_t to = sk_bounded(P.part_o + (size_t)w.part * P.rows_per_slot * D, nrows * D * 4);
#pragma unroll
                for (int i = 0; i < BATCH; ++i) sk_store16_through(to, (unsigned)(rg * 32 + row_of(i)) * (D * 4) + c4 * 16, val[i]);
                continue;
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int rit = rg * 32 + row_of(i);           // row inside the tile
                if (rit >= nrows) continue;
                const int tok2 = div_g(rit);
                const size_t orow = ((size_t)(w.q_tok0 + tok2) * P.g.Hq + w.kv_head * G + (rit - tok2 * G));
                if (P.out_dtype == 0) *(float4*)((float*)P.out + orow * D + c4 * 4) = val[i];
                else {
                    const uint32_t lo = f32_to_bf16_bits(val[i].x) | ((uint32_t)f32_to_bf16_bits(val[i].y) << 16);
                    const uint32_t hi = f32_to_bf16_bits(val[i].z) | ((uint32_t)f32_to_bf16_bits(val[i].w) << 16);
                    *(uint2*)((uint16_t*)P.out + orow * D + c4 * 4) = make_uint2(lo, hi);
                }
            }
        }
    }
    asm volatile("" : : : "memory");                  // the partial's stores are issued in front of the wait,
    SK_WAIT_VMCNT(0);                                 // and behind it they have completed
    if (direct || !P.fuse) return;

    // ---- in-kernel merge of the split partials ----
    // The workgroups of one (row tile, KV head) are a unit.  Each has written its partial above; it
    // now arrives at the unit's counter and waits, for a bounded number of polls, until all have
    // arrived; then every workgroup of the unit merges its own share of the tile's rows (split k the
    // rows k * rps ..), reading the other partials through the L2.  A workgroup that gives up waiting
    // says so in the counter's high bits and leaves; the last workgroup to arrive (which never waits,
    // so the scheme needs no two workgroups to be resident together) then merges every share.  Who
    // merges a row does not change its value: sk_merge_row adds the splits in index order.
    __syncthreads();                                  // the whole partial is written (and LDS is free again)
    volatile int* flag = (volatile int*)lds;
    uint32_t* cnt = P.sync + 2 * (size_t)w.unit;
    uint32_t left = 0;
    // Release: every thread has waited for its write-through stores and passed the barrier above, so
    // the partial is in memory before the arrival below.  Acquire: the merge reads the partials with
    // device-scope loads, issued after the counter has said that everybody has arrived (the fence below
    // only keeps the compiler and this workgroup's waves from reading earlier).
    if (tid == 0) {
        if (P.merge_fences) __threadfence();
        const uint32_t np = (uint32_t)w.n_parts;
        const uint32_t old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int state;                                    // 0: leave, 1: merge the own share, 2: merge every share
        if ((old & 0xffffu) + 1u == np) state = (old >> 16) ? 2 : 1;
        else {
            state = 0;
            for (int i = 0; i < P.wait_polls; ++i) {
                __builtin_amdgcn_s_sleep(4);
                if ((__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffffu) == np) { state = 1; break; }
            }
            if (state == 0) {
                // gave up.  The mark and the last arrival are atomic operations on one word: either the last
                // arriver sees the mark (and merges this share), or this sees that everybody has arrived.
                const uint32_t o2 = __hip_atomic_fetch_add(cnt, 0x10000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((o2 & 0xffffu) == np) state = 1;
            }
        }
        if (P.merge_fences) __threadfence(); else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        // departure (this workgroup will not look at the arrival counter again), requested now so that
        // its round trip runs beside the merge; the answer is needed at the very end only
        left = __hip_atomic_fetch_add(cnt + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = state;
    }
    __syncthreads();
    const int state = *flag;
    if (state != 0) {
        const int rps = (nrows + w.n_parts - 1) / w.n_parts;
        const int k_own = (w.part - w.part0) / P.g.Hkv;
        const int k_lo = state == 2 ? 0 : k_own, k_hi = state == 2 ? w.n_parts : k_own + 1;
        for (int k = k_lo; k < k_hi; ++k) {
            const int row_end = (k + 1) * rps < nrows ? (k + 1) * rps : nrows;
            for (int row = k * rps + wave; row < row_end; row += NW) {
                const int tok3 = div_g(row);
                const size_t orow = (size_t)(w.q_tok0 + tok3) * P.g.Hq + w.kv_head * G + (row - tok3 * G);
                sk_merge_row<D>(P, (size_t)w.part0 * P.rows_per_slot + row, (size_t)P.g.Hkv * P.rows_per_slot, w.n_parts, orow, lane);
            }
        }
    }
    // the last workgroup of the unit to depart clears the counters for the next launch
    if (tid == 0) {
        if (left + 1u == (uint32_t)w.n_parts) {
            __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(cnt + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// The kernels proper: head_dim 128 (all four instances) and head_dim 64 (all but <4,2,2>).
template <int NRG, int NPH, int NSS>
__global__ __launch_bounds__(64 * NRG * NPH, NRG * NPH == 8 ? 1 : 2) void sk_attn_bf16_d128(const sk_launch P)
{
    sk_attn_bf16_body<NRG, NPH, NSS, 128>(P);
}
template <int NRG, int NPH, int NSS>
__global__ __launch_bounds__(64 * NRG * NPH, 2) void sk_attn_bf16_d64(const sk_launch P)
{
    sk_attn_bf16_body<NRG, NPH, NSS, 64>(P);
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA attention kernel for calls of at most 32 query rows per KV head (a decoded token, a short
// question): what such a call takes is latency, not rate, so everything between the launch and the
// result is kept short.
//
// A workgroup is four waves that share nothing until the end: wave w takes the 32-key tiles w, w + 4, .. of
// the workgroup's keys, straight from memory into the operand registers of the matrix instructions
// (sixteen 16-byte loads per lane and tile, all in flight at once; no LDS ring, no barrier in the loop),
// with the arithmetic and register layout of the kernel above.  The four partial results meet in LDS.
// The call's own K/V (a query's, or a chunk being appended: at most 32 tokens) are read where the caller
// has them, as one more tile of the last part, so no staging launch stands in front; an append's commit
// runs in further workgroups of the same launch.
//
// The parts of a row tile are merged by the workgroup that finishes last (P.fuse), which reads the others'
// partials through the L2 it shares with them: the launch maps all parts of a KV head to one XCD, so their
// ordinary stores are visible there once they have completed.  That they did run on one XCD is checked, not
// assumed: every workgroup adds its XCD number and its square to the unit's 64-bit arrival word (one
// device-scope atomic), and the last one merges only if n * sum(x^2) == sum(x)^2, i.e. all x are equal.
// If not, it computes every part again by itself, one after the other and each as its own workgroup did, and
// merges those (the slots get the bytes they hold already): the result is the same to the last bit wherever the
// parts ran.  Nobody waits for anybody.
//
// Bound: round trips.  One query token with its own K/V at 2,600 cached tokens: one launch of 6.6 us where a staging,
// an attention and a combine kernel took 17.3 back to back.  By time stamps: 0.6 us from a workgroup's start to its block ids, 1.9 to the
// end of its keys, 1.2 for the meeting in LDS, 0.6 for the arrival and 1.4 for the merge (two round trips, a third behind 16 parts).
// 10.7 MB of cache at the rate of a plain read would be 1.7 us.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned sk_xcd_id() { return (unsigned)__builtin_amdgcn_s_getreg((3 << 11) | 20); }    // HW_REG_XCC_ID, bits 3:0

template <int D>
__device__ __forceinline__ void sk_commit_group(const sk_geom& g, const void* k, const void* v, const sk_scatter& it, const int head,
                                                int32_t* tables_rw, unsigned char* kv_rw, uint16_t* vt);

// What a workgroup of the kernels below does once its four waves have laid their accumulators side by side in LDS
// (tr[wave][row][16-byte chunk ^ row], stat[wave][row] = (m, l, lx, -)): brings them to the common row maxima, adds
// the four up, writes the rows out (n_parts == 1) or to the slot of `part` (slot0 + part * Hkv), and, with P.fuse,
// arrives at `unit` and merges the unit's parts if it is the last one there.  False: the parts did not run on
// one XCD and this workgroup has to compute them all, part 0 first (`alone` from then on).  `orow_of`: row of the
// tile -> row of out / lse.
template <int D, int ROWS, class OutRow>
__device__ __forceinline__ bool sk_meet(const sk_launch& P, float4 (*tr)[ROWS][D / 4], float4 (*stat)[ROWS], int* decision, const int tid,
                                        const int nrows, const int part, const bool alone, const int slot0, const int n_parts, const int unit,
                                        const OutRow orow_of)
{
    const bool whole = n_parts == 1;
    constexpr int CPR = D / 4;
    auto put_row = [&](const int row, const int c4, const float4 x, const float inv, const float lse) __attribute__((always_inline)) {
        const size_t orow = orow_of(row);
        if (P.out_dtype == 0) *(float4*)((float*)P.out + orow * D + c4 * 4) = make_float4(x.x * inv, x.y * inv, x.z * inv, x.w * inv);
        else {
            const uint32_t lo = f32_to_bf16_bits(x.x * inv) | ((uint32_t)f32_to_bf16_bits(x.y * inv) << 16);
            const uint32_t hi = f32_to_bf16_bits(x.z * inv) | ((uint32_t)f32_to_bf16_bits(x.w * inv) << 16);
            *(uint2*)((uint16_t*)P.out + orow * D + c4 * 4) = make_uint2(lo, hi);
        }
        if (P.lse && c4 == 0) P.lse[orow] = lse;
    };
    __syncthreads();
    const size_t prow = (size_t)(slot0 + part * P.g.Hkv) * P.rows_per_slot;
    for (int i = tid; i < nrows * CPR; i += 256) {
        const int row = i / CPR, c4 = i % CPR;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f), st[4];
        float m = SK_NEG_INF, l = 0.f, lx = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) { st[w] = stat[w][row]; m = fmaxf(m, st[w].x); }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 y = tr[w][row][(c4 ^ row) & (CPR - 1)];
            const float a = st[w].x == SK_NEG_INF ? 0.f : sk_exp2(st[w].x - m);
            x.x = fmaf(y.x, a, x.x); x.y = fmaf(y.y, a, x.y); x.z = fmaf(y.z, a, x.z); x.w = fmaf(y.w, a, x.w);
            l = fmaf(st[w].y, a, l); lx = fmaf(st[w].z, a, lx);
        }
        if (whole) put_row(row, c4, x, 1.0f / l, (m + sk_log2(lx)) * SK_LN2);
        else {
            *(float4*)(P.part_o + (prow + row) * D + c4 * 4) = x;
            if (c4 == 0) *((float4*)P.part_ml + prow + row) = make_float4(m, l, lx, 0.f);
        }
    }
    if (whole || !P.fuse) return true;

    // ---- arrival; the last workgroup of the unit merges ----
    SK_WAIT_VMCNT(0);                                 // this thread's part of the partial has reached the L2
    __syncthreads();
    if (alone) {
        if (part + 1 < n_parts) return false;
    } else {
        if (tid == 0) {
            const unsigned long long x = sk_xcd_id();
            unsigned long long* word = (unsigned long long*)P.sync + (size_t)unit * 16;      // a 128-byte line per unit: each is one XCD's
            const unsigned long long add = 1ull | (x << 16) | ((x * x) << 36);
            const unsigned long long got = __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
            int d = 0;
            if ((int)(got & 0xffffu) == n_parts) {
                const unsigned long long sum = (got >> 16) & 0xfffffu, sq = got >> 36;
                d = (!(P.distrust & 1) && (unsigned long long)n_parts * sq == sum * sum) ? 1 : ((P.distrust & 2) ? 0 : 2);
                __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // ready for the next launch
            }
            *decision = d;
        }
        __syncthreads();
        const int d = *decision;
        if (d == 0) return true;
        if (d == 2) return false;
    }
    // The CPR lanes that merge a row (a 16-byte piece each) find its weights by themselves: lane c holds the statistics of parts c, c + CPR, ..,
    // maxima and sums go over the lanes without LDS, the weights through a corner of LDS that only this wave uses.  Nobody waits for another
    // wave, and the first parts' rows are requested beside the statistics: two round trips to the L2 for up to 16 parts, one more for every
    // 16 further ones.  (Against statistics loaded by all, two barriers and rounds of eight, a decoded token at 2,600 cached, 21 parts:
    // 8.31 -> 6.61 us.)  The rounds are short loops: code that runs once per launch costs its instruction fetches.
    constexpr int STAT = 64 / CPR > 0 ? 64 / CPR : 1, ROUND = 16;      // at most 64 parts (can_merge)
    const size_t pstep = (size_t)P.g.Hkv * P.rows_per_slot;
    const unsigned row0 = (unsigned)(slot0 * P.rows_per_slot);
    const unsigned step = (unsigned)(pstep * D * 4);                   // bytes from part to part
    // (buffer loads return zeros behind the unit's last part, so that no round needs a branch around its loads)
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(P.part_o + (size_t)row0 * D, 0, (int)((unsigned)n_parts * step), 0x00020000);
    const __amdgpu_buffer_rsrc_t stats = __builtin_amdgcn_make_buffer_rsrc(P.part_ml + (size_t)row0 * 4, 0, (int)((unsigned)n_parts * (unsigned)(pstep * 16)), 0x00020000);
    const int c = tid & (CPR - 1);
    float* const wgt = (float*)&tr[0][0][0] + (tid / CPR) * 64;        // [lane group][part]
#pragma unroll 1
    for (int i = tid; i < nrows * CPR; i += 256) {
        const int row = i / CPR;
        float4 ml[STAT], x[ROUND];
#pragma unroll
        for (int j = 0; j < STAT; ++j)
            ml[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(stats, (unsigned)(c + j * CPR) * (unsigned)(pstep * 16) + (unsigned)row * 16, 0, 0));
#pragma unroll
        for (int j = 0; j < ROUND; ++j) x[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(parts, (unsigned)j * step + (unsigned)i * 16, 0, 0));
        float M = SK_NEG_INF, L = 0.f, Lx = 0.f;
#pragma unroll
        for (int j = 0; j < STAT; ++j) M = fmaxf(M, c + j * CPR < n_parts ? ml[j].x : SK_NEG_INF);
        M = fmaxf(M, sk_dpp<0xB1>(M)); M = fmaxf(M, sk_dpp<0x4E>(M)); M = fmaxf(M, sk_dpp<0x141>(M)); M = fmaxf(M, sk_dpp<0x140>(M));
        if (CPR == 32) { const sk_halves h = sk_row_pairs(M); M = fmaxf(h.lo, h.hi); }
#pragma unroll
        for (int j = 0; j < STAT; ++j) {
            const float a = c + j * CPR >= n_parts || ml[j].x == SK_NEG_INF ? 0.f : sk_exp2(ml[j].x - M);
            wgt[c + j * CPR] = a;
            L = fmaf(ml[j].y, a, L); Lx = fmaf(ml[j].z, a, Lx);
        }
        L += sk_dpp<0xB1>(L); L += sk_dpp<0x4E>(L); L += sk_dpp<0x141>(L); L += sk_dpp<0x140>(L);
        Lx += sk_dpp<0xB1>(Lx); Lx += sk_dpp<0x4E>(Lx); Lx += sk_dpp<0x141>(Lx); Lx += sk_dpp<0x140>(Lx);
        if (CPR == 32) {
            { const sk_halves h = sk_row_pairs(L); L = h.lo + h.hi; }
            { const sk_halves h = sk_row_pairs(Lx); Lx = h.lo + h.hi; }
        }
        __builtin_amdgcn_wave_barrier();                  // the weights of a row come from the lanes of this wave: no read is moved in front of them
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
        for (int p0 = 0;;) {
#pragma unroll
            for (int j = 0; j < ROUND; j += 4) {
                const float4 w4 = *(const float4*)(wgt + p0 + j);
                const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    acc.x = fmaf(x[j + k].x, w[k], acc.x); acc.y = fmaf(x[j + k].y, w[k], acc.y);
                    acc.z = fmaf(x[j + k].z, w[k], acc.z); acc.w = fmaf(x[j + k].w, w[k], acc.w);
                }
            }
            p0 += ROUND;
            if (p0 >= n_parts) break;
#pragma unroll
            for (int j = 0; j < ROUND; ++j) x[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(parts, (unsigned)(p0 + j) * step + (unsigned)i * 16, 0, 0));
        }
        put_row(row, c, acc, 1.0f / L, (M + sk_log2(Lx)) * SK_LN2);
    }
    return true;
}

// The kernel's arguments, as they lie in memory.
struct sk_small_args {
    const int32_t* table; const unsigned char *q, *kv;
    uint32_t head_pages; int32_t Hkv; uint32_t shape, pad_mul, g_magic; int32_t n_parts, chunk, kv_len;
    sk_launch P;
    sk_commit C;
};
// Byte offset at which argument N of a kernel lies in its argument block: each behind the one in front, aligned as its type.
template <int N, class... A>
constexpr size_t sk_argument_offset(void (*)(A...))
{
    constexpr size_t size[] = {sizeof(A)...}, align[] = {alignof(A)...};
    size_t at = 0;
    for (int i = 0; i < N; ++i) at = (at + align[i] - 1) / align[i] * align[i] + size[i];
    return (at + align[N] - 1) / align[N] * align[N];
}
// The first arguments are in registers when a wave starts: what the first loads need (`table`: of the session; `shape`: see
// sk_launch_attention_small), which go out before the argument block, that nobody has read yet, has arrived.
template <int D>
__global__ __launch_bounds__(256, 2) void sk_attn_bf16_small(const int32_t* const table, const unsigned char* const q, const unsigned char* const kv,
                                                             const uint32_t head_pages, const int32_t Hkv, const uint32_t shape, const uint32_t pad_mul,
                                                             const uint32_t g_magic, const int32_t n_parts, const int32_t chunk, const int32_t kv_len,
                                                             const sk_launch, const sk_commit)
{
    constexpr int NKS = D / 16, NMT = D / 32, NWV = 4, CPR = D / 4;      // CPR: float4 chunks of an output row
    constexpr int ROWB = D * 2, LOG2_TOK_BYTES = D == 128 ? 8 : 7;
    __shared__ float4 tr[NWV][32][CPR];
    __shared__ float4 stat[NWV][32];
    __shared__ int decision;
    const int G = shape & 255, log2B = (shape >> 8) & 15, n_tok = (shape >> 18) & 63, own_cnt = shape >> 24 & 63;
    // workgroup -> (part, KV head); the heads of a part are padded to a multiple of the XCD count
    const int head_pad = (shape >> 17) & 1 ? (Hkv + 7) & ~7 : Hkv;
    int part = sk_divide(blockIdx.x, sk_div{pad_mul, (int)(shape >> 12) & 31});
    const int head = blockIdx.x - part * head_pad;
    if (__builtin_expect(part >= n_parts, 0)) {                                // the commit of an append
        const sk_launch P = sk_late_argument<sk_launch, offsetof(sk_small_args, P)>();
        typedef const __attribute__((address_space(4))) unsigned char* args_ptr;
        const sk_commit& C = *(const sk_commit*)((args_ptr)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(sk_small_args, C));
        const int i = blockIdx.x - C.first_wg, item = sk_divide(i, P.by_heads);
        sk_commit_group<D>(P.g, P.own_k, P.own_v, C.item[item], i - item * Hkv, C.tables_rw, C.kv_rw, (uint16_t*)&tr[0][0][0]);
        return;
    }
    if (head >= Hkv) return;
    bool alone = false;                                   // the parts ran on several XCDs: this workgroup computes them all
    for (;;) {
        // (opaque, or everything below that depends on the lane only is computed before the first load is
        // requested: the loop almost never runs twice)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int r = lane & 31, kg = lane >> 5;
        const int nrows = n_tok * G;
        auto div_g = [&](const int row) __attribute__((always_inline)) { return (int)(((unsigned)row * g_magic) >> 16); };
        const int tok = div_g(r < nrows ? r : 0), hq = head * G + (r < nrows ? r - tok * G : 0);
        const int tau = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);      // key of S^T row r (bits 2 and 3 swapped)

        int k_begin = 0, k_end = kv_len;
        if (n_parts > 1) {
            k_begin = part * chunk;
            k_end = k_begin + chunk < k_end ? k_begin + chunk : k_end;
        }
        const int n_cached = k_end > k_begin ? (k_end - k_begin + 31) >> 5 : 0;
        const int last_group = k_end > 0 ? (k_end - 1) & ~15 : 0;

        bf16x8 qreg[NKS];
        sk_u32x4 ka[NKS], va[2][NMT];
        // the two 16-key groups of cached tile t: their block ids, requested at once, and the base of each group's K (its V^T lies v_off further)
        auto group_at = [&](const int t, const int j) __attribute__((always_inline)) {
            const int tg = k_begin + t * 32 + 16 * j;
            return tg < last_group ? tg : last_group;
        };
        auto group_id = [&](const int t, const int j) __attribute__((always_inline)) {
            typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
            return (uint32_t)((const_i32_ptr)(uintptr_t)table)[(unsigned)group_at(t, j) >> log2B];
        };
        auto group_base = [&](const int t, const int j, const uint32_t blk) __attribute__((always_inline)) -> const unsigned char* {
            return kv + (int64_t)head * ((int64_t)head_pages << 12) + ((uint64_t)blk << (log2B + LOG2_TOK_BYTES + 1)) +
                   (((unsigned)group_at(t, j) & ((1u << log2B) - 1)) << LOG2_TOK_BYTES);
        };
        auto load_k = [&](const unsigned char* b0, const unsigned char* b1) __attribute__((always_inline)) {
            const unsigned char* p = ((r & 16) ? b1 : b0) + (tau & 15) * ROWB + kg * 16;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) ka[ks] = *(const sk_u32x4*)(p + ks * 32);
        };
        auto load_v = [&](const unsigned char* b0, const unsigned char* b1) __attribute__((always_inline)) {
            const unsigned voff = ((unsigned)ROWB << log2B) + (unsigned)(r * 32 + kg * 16);
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt) {
                va[0][mt] = *(const sk_u32x4*)(b0 + voff + mt * 1024);
                va[1][mt] = *(const sk_u32x4*)(b1 + voff + mt * 1024);
            }
        };
        uint32_t id0 = group_id(wave, 0), id1 = group_id(wave, 1);
        __builtin_amdgcn_sched_barrier(0);
        {
            const sk_u32x4* qp = (const sk_u32x4*)(q + ((size_t)tok * (Hkv * G) + hq) * ROWB);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) qreg[ks] = __builtin_bit_cast(bf16x8, qp[ks * 2 + kg]);
        }
        const unsigned char *b0 = group_base(wave, 0, id0), *b1 = group_base(wave, 1, id1);
        if (wave < n_cached) { load_k(b0, b1); load_v(b0, b1); }
        sk_touch_arguments<offsetof(sk_small_args, C)>();
        const sk_launch P = sk_late_argument<sk_launch, offsetof(sk_small_args, P)>();
        const float c_scale = P.g.scale_log2e;

        f32x16 oacc[NMT];
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[mt][v] = 0.f;
        float m_ref = SK_NEG_INF, l_run = 0.f, lx_run = 0.f;
        f32x16 sacc;
        bf16x8 pb[2];
        auto scores = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[ks]), qreg[ks], sacc, 0, 0, 0);
        };
        auto mask = [&](const int k0, const int limit, const int hole_lo, const int hole_n) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int key = k0 + 16 * (v >> 3) + 8 * kg + (v & 7);
                const bool vis = key <= limit && (unsigned)(key - hole_lo) >= (unsigned)hole_n;
                sacc[v] = vis ? sacc[v] : SK_NEG_INF;
            }
        };
        // Clears the values behind the first `left` keys of the tile.  Where the tile ends inside a 16-token group, the commit
        // of this launch may be writing the slots behind its end: their weight of 0 must not meet what is found there.
        auto drop_values = [&](const int left) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int key = 16 * q + 8 * kg + 2 * j;
                    const uint32_t keep = (key < left ? 0xffffu : 0u) | (key + 1 < left ? 0xffff0000u : 0u);
#pragma unroll
                    for (int mt = 0; mt < NMT; ++mt) va[q][mt][j] &= keep;
                }
        };
        auto softmax = [&]() __attribute__((always_inline)) {
            float mx = SK_NEG_INF;
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[v]);
            { const sk_halves h = sk_both_halves(mx); mx = fmaxf(h.lo, h.hi) * c_scale; }
            const bool raise = mx > m_ref + SK_RESCALE_SLACK;
            if (__any(raise)) {
                const float alpha = raise ? sk_exp2(m_ref - mx) : 1.0f;
                l_run *= alpha; lx_run *= alpha;
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[mt][v] *= alpha;
                m_ref = raise ? mx : m_ref;
            }
            const float neg_m = m_ref == SK_NEG_INF ? 0.f : -m_ref;
            float lx0 = 0.f, lx1 = 0.f;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const float p0 = sk_exp2(fmaf(sacc[v], c_scale, neg_m)), p1 = sk_exp2(fmaf(sacc[8 + v], c_scale, neg_m));
                pb[0][v] = (__bf16)p0; pb[1][v] = (__bf16)p1;
                lx0 += p0; lx1 += p1;
            }
            lx_run += lx0 + lx1;
            const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
            float ls0 = 0.f, ls1 = 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {        // the row sum over the weights as the matrix pipe sees them (see above)
                ls0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[q], pb[q], 0, 1), ones, ls0, false);
                ls1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[q], pb[q], 2, 3), ones, ls1, false);
                ls0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[q], pb[q], 4, 5), ones, ls0, false);
                ls1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[q], pb[q], 6, 7), ones, ls1, false);
            }
            l_run += ls0 + ls1;
        };
        auto values = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt)
                    oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[q][mt]), pb[q], oacc[mt], 0, 0, 0);
        };

#pragma unroll 1
        for (int t = wave; t < n_cached; t += NWV) {
            const bool more = t + NWV < n_cached;
            if (more) {
                id0 = group_id(t + NWV, 0); id1 = group_id(t + NWV, 1);
                b0 = group_base(t + NWV, 0, id0); b1 = group_base(t + NWV, 1, id1);
            }
            scores();
            if (more) load_k(b0, b1);
            const int k0 = k_begin + t * 32;          // keys past the end of the part and evicted keys do not count
            if (k0 + 32 > k_end || (k0 < P.hole_hi && k0 + 32 > P.hole_lo)) mask(k0, k_end - 1, P.hole_lo, P.hole_hi - P.hole_lo);
            softmax();
            if (k0 + 32 > k_end) drop_values(k_end - k0);
            values();
            if (more) load_v(b0, b1);
        }
        // The call's own tokens: one tile, for a wave that has no cached one when the launch is cut into parts.
        if (part == n_parts - 1 && own_cnt > 0 && wave == (n_cached & (NWV - 1))) {
            const int key = tau < own_cnt ? tau : own_cnt - 1;
            const unsigned char* p = (const unsigned char*)P.own_k + ((size_t)key * Hkv + head) * ROWB + kg * 16;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) ka[ks] = *(const sk_u32x4*)(p + ks * 32);
            // token-major values: the rows go through this wave's quarter of the exchange area, where eight keys of
            // one dimension are eight 2-byte reads; zero past the end
            uint4* rows = (uint4*)&tr[wave][0][0];
#pragma unroll
            for (int i = 0; i < 32 * ROWB / 16 / 64; ++i) {
                const int c = i * 64 + lane, vkey = c / (ROWB / 16), cc = c % (ROWB / 16);
                uint4 x = make_uint4(0, 0, 0, 0);
                if (vkey < own_cnt) x = *(const uint4*)((const unsigned char*)P.own_v + ((size_t)vkey * Hkv + head) * ROWB + cc * 16);
                rows[c] = x;
            }
            scores();
            mask(0, P.pos0 < SK_NO_CAUSAL ? tok : own_cnt - 1, 0, 0);
            softmax();
            const uint16_t* vt = (const uint16_t*)rows + 8 * kg * D + r;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        va[q][mt][j] = (uint32_t)vt[(16 * q + 2 * j) * D + mt * 32] | ((uint32_t)vt[(16 * q + 2 * j + 1) * D + mt * 32] << 16);
                }
            values();
        }

        // ---- the four waves meet: accumulators and row statistics side by side in LDS ----
        float l_tot, lx_tot;
        { const sk_halves h = sk_both_halves(l_run); l_tot = h.lo + h.hi; }
        { const sk_halves h = sk_both_halves(lx_run); lx_tot = h.lo + h.hi; }
        if (r < nrows) {
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int c4 = mt * 8 + q4 * 2 + kg;
                    tr[wave][r][(c4 ^ r) & (CPR - 1)] = make_float4(oacc[mt][q4 * 4 + 0], oacc[mt][q4 * 4 + 1], oacc[mt][q4 * 4 + 2], oacc[mt][q4 * 4 + 3]);
                }
            if (kg == 0) stat[wave][r] = make_float4(m_ref, l_tot, lx_tot, 0.f);
        }
        if (sk_meet<D, 32>(P, tr, stat, &decision, tid, nrows, part, alone, head, n_parts, head,
                           [&](const int row) __attribute__((always_inline)) {
                               const int t2 = div_g(row);
                               return (size_t)t2 * P.g.Hq + head * G + (row - t2 * G);
                           })) return;
        part = alone ? part + 1 : 0;
        alone = true;
    }
}

// ---------------------------------------------------------------------------------------------
// fp32 attention kernel (fp32 pools): every product on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 accumulation).  Tile of up to 16 query rows; four waves that take the 16-key tiles w, w + 4, ..
// straight from memory into registers and meet in LDS at the end, as in sk_attn_bf16_small.
//   S^T[16 keys][16 rows] = K Q^T: lane (c = lane % 16, g = lane / 16) holds K[c] and Q[c] at dims 16 j + 4 g .. + 3
//     (any order of the contraction will do, so a load instruction reads 64 consecutive bytes of a row);
//   the lane then owns row c and keys 4 g .. 4 g + 3, whose weights are, register by register, the B operand of
//   O^T[16 dims][16 rows] += V^T P^T with the keys 4 g + i of step i; the A operand is V[4 g + i] at dims 4 c .. 4 c + 3
//     (+ 64): one 16-byte load serves four of the 16-dim blocks, whose row c then is dim 4 c + block.
// In single-session calls the call's own K/V are read where the caller has them, as further keys behind the
// cached ones (padded to whole tiles), and a short commit runs in the same launch; in batched calls they come from
// the staging area.  Rows past the end of a tile's keys re-read the last one; they count as zeros.
// Bound: round trips and launches at the sizes in use: a 64-token append at 960 cached tokens (4 heads of 64 dims) 29.1
// -> 8.1 us in a stream of appends, a cache-only 16-token query at 1,024 25.2 -> 7.7 (a commit or nothing, an fp32-FMA kernel
// of 24 / 20.6 us and a combine kernel of 4.4 / 3.9 before; one launch now).
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) float sk_acc4;

// Maximum / sum over the four lanes c, c + 16, c + 32, c + 48.
__device__ __forceinline__ float sk_max_over_groups(float x)
{
    { const sk_halves h = sk_row_pairs(x); x = fmaxf(h.lo, h.hi); }
    { const sk_halves h = sk_both_halves(x); x = fmaxf(h.lo, h.hi); }
    return x;
}
__device__ __forceinline__ float sk_sum_over_groups(float x)
{
    { const sk_halves h = sk_row_pairs(x); x = h.lo + h.hi; }
    { const sk_halves h = sk_both_halves(x); x = h.lo + h.hi; }
    return x;
}

__device__ __forceinline__ void sk_commit_group_f32(const sk_geom& g, const void* k, const void* v, const sk_scatter& it, const int head,
                                                    int32_t* tables_rw, unsigned char* base);

template <int D>
__global__ __launch_bounds__(256, 2) void sk_attn_f32(const sk_launch P, const sk_commit C)
{
    constexpr int NJ = D / 16, NH = D / 64, CPR = D / 4, ROWB = D * 4;
    __shared__ float4 tr[4][16][CPR];
    __shared__ float4 stat[4][16];
    __shared__ int decision;
    sk_touch_arguments<sizeof(sk_launch) + offsetof(sk_commit, item)>();
    const int Hkv = P.g.Hkv, G = P.g.G;
    if (__builtin_expect((int)blockIdx.x >= C.first_wg, 0)) {                  // the commit of an append
        const int i = blockIdx.x - C.first_wg, item = sk_divide(i, P.by_heads);
        sk_commit_group_f32(P.g, P.own_k, P.own_v, C.item[item], i - item * Hkv, C.tables_rw, C.kv_rw);
        return;
    }
    // the row tile, and its keys: cached [k_begin, k_end), then own tokens [o_begin, o_end) (where the caller has them) or
    // staged segments
    const bool listed = P.mode == SK_MODE_LIST;
    sk_work w;
    int part = 0, unit = 0, n_parts = 1, vis = 0;
    if (listed) { w = P.work[blockIdx.x]; n_parts = w.n_parts; }
    else {
        part = sk_divide(blockIdx.x, P.by_pad); unit = blockIdx.x - part * P.head_pad;
        if (unit >= P.n_tiles * Hkv) return;
        const int tile = sk_divide(unit, P.by_heads);
        w.kv_head = unit - tile * Hkv;
        w.q_tok0 = tile * P.tok_per_tile;
        w.n_tok = P.n_tok - w.q_tok0 < P.tok_per_tile ? P.n_tok - w.q_tok0 : P.tok_per_tile;
        n_parts = sk_tile_parts(P, w.q_tok0, w.n_tok, &vis);
        if (part >= n_parts) return;
        w.tbl_off = P.tbl_off; w.pos0 = P.pos0 < SK_NO_CAUSAL ? P.pos0 + w.q_tok0 : P.pos0;
        w.hole_lo = P.hole_lo; w.hole_hi = P.hole_hi; w.kv_step = 0; w.sub_blocks = 0; w.once = 0;
        w.part0 = tile * P.n_splits * Hkv + w.kv_head;
        w.eph_cnt[0] = w.eph_cnt[1] = 0; w.eph_blk[0] = w.eph_blk[1] = 0; w.eph_pos0[0] = w.eph_pos0[1] = 0;
    }
    const int slot0 = listed ? w.part : w.part0;          // (a listed part is not merged here)
    bool alone = false;                                   // see sk_attn_bf16_small
    for (;;) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                     // (opaque: see sk_attn_bf16_small)
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int c = lane & 15, g4 = (lane >> 4) * 4;
        const int head = w.kv_head, nrows = w.n_tok * G;
        const unsigned g_magic = P.g.g_magic;
        auto div_g = [&](const int row) __attribute__((always_inline)) { return (int)(((unsigned)row * g_magic) >> 16); };
        const int tok = div_g(c < nrows ? c : 0), hq = head * G + (c < nrows ? c - tok * G : 0);
        // a negative scale as its size and the other sign of the scores, so that the largest score is the largest weight and a
        // masked one has none
        const float c_scale = fabsf(P.g.scale_log2e);
        const uint32_t flip = P.g.scale_log2e < 0.f ? 0x80000000u : 0u;
        const bool causal = w.pos0 < SK_NO_CAUSAL;
        const int p_row = causal ? w.pos0 + tok : 0x7fffffff, p_first = causal ? w.pos0 : 0x7fffffff;
        int k_begin, k_end, o_begin = 0, o_end = 0;
        if (listed) { k_begin = w.kv_begin; k_end = w.kv_end; }
        else {
            const int pad = (P.kv_len + 15) & ~15;
            const int b = part * P.chunk, e = b + P.chunk > vis ? vis : b + P.chunk;
            k_begin = b; k_end = e < P.kv_len ? e : P.kv_len;
            o_begin = b > pad ? b - pad : 0; o_end = e - pad;
        }

        float4 q[NJ];
        {
            const float4* qp = (const float4*)((const float*)P.q + ((size_t)(w.q_tok0 + tok) * P.g.Hq + hq) * D + g4);
#pragma unroll
            for (int j = 0; j < NJ; ++j) q[j] = qp[j * 4];
        }
        sk_acc4 o[NH][4];
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int b = 0; b < 4; ++b) o[h][b] = sk_acc4{0.f, 0.f, 0.f, 0.f};
        float m_ref = SK_NEG_INF, l_run = 0.f;

#pragma unroll 1
        for (int s = 0; s < 4; ++s) {             // cached, own (raw), staged, staged
            int begin, end, pos_shift = 0, hole_lo = 0, hole_n = 0;
            sk_seg sg;
            if (s == 1) { begin = o_begin; end = o_end; pos_shift = P.pos0; if (!causal) pos_shift = 0; }
            else {
                sg = sk_make_seg(P, w, s == 0 ? 0 : s - 1);
                if (s == 0) { begin = k_begin; end = k_end; hole_lo = sg.hole_lo; hole_n = sg.hole_n; }
                else { begin = sg.begin; end = sg.end; pos_shift = sg.pos_shift; }
            }
            if (end <= begin) continue;
            const int n_tiles = (end - begin + 15) >> 4;
            const int rstride = s == 1 ? Hkv * ROWB : ROWB;
            auto row_base = [&](const int t, const unsigned char*& kp, const unsigned char*& vp) __attribute__((always_inline)) {
                const int t0 = begin + t * 16;
                if (s == 1) {
                    const size_t off = ((size_t)t0 * Hkv + head) * ROWB;
                    kp = (const unsigned char*)P.own_k + off; vp = (const unsigned char*)P.own_v + off;
                } else {
                    kp = sk_group_base(sg, t0) + (t0 & (sg.B - 1)) * ROWB;
                    vp = kp + sg.v_off;
                }
            };
            float4 kr[NJ], vr[4][NH];
            auto load_k = [&](const int t, const unsigned char* kp) __attribute__((always_inline)) {
                const int left = end - (begin + t * 16) - 1, row = c < left ? c : left;
                const float4* p = (const float4*)(kp + row * rstride) + (g4 >> 2);
#pragma unroll
                for (int j = 0; j < NJ; ++j) kr[j] = p[j * 4];
            };
            auto load_v = [&](const int t, const unsigned char* vp) __attribute__((always_inline)) {
                const int left = end - (begin + t * 16) - 1;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = g4 + i < left ? g4 + i : left;
#pragma unroll
                    for (int h = 0; h < NH; ++h) vr[i][h] = *((const float4*)(vp + row * rstride) + h * 16 + c);
                }
            };
            const unsigned char *kp = nullptr, *vp = nullptr;
            if (wave < n_tiles) { row_base(wave, kp, vp); load_k(wave, kp); load_v(wave, vp); }
#pragma unroll 1
            for (int t = wave; t < n_tiles; t += 4) {
                const bool more = t + 4 < n_tiles;
                if (more) row_base(t + 4, kp, vp);
                sk_acc4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j].x, q[j].x, sc, 0, 0, 0);
                    sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j].y, q[j].y, sc, 0, 0, 0);
                    sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j].z, q[j].z, sc, 0, 0, 0);
                    sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j].w, q[j].w, sc, 0, 0, 0);
                }
                if (more) load_k(t + 4, kp);
#pragma unroll
                for (int i = 0; i < 4; ++i) sc[i] = __uint_as_float(__float_as_uint(sc[i]) ^ flip);
                const int k0 = begin + t * 16;
                if (k0 + 16 > end || k0 + 15 + pos_shift > p_first || (k0 < hole_lo + hole_n && k0 + 16 > hole_lo)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = k0 + g4 + i;
                        const bool seen = key < end && key + pos_shift <= p_row && (unsigned)(key - hole_lo) >= (unsigned)hole_n;
                        sc[i] = seen ? sc[i] : SK_NEG_INF;
                    }
                }
                if (k0 + 16 > end) {              // rows behind the last key repeat it: their weight of 0 must not meet an infinity
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int h = 0; h < NH; ++h)
                            if (k0 + g4 + i >= end) vr[i][h] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
                const float mx = sk_max_over_groups(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]))) * c_scale;
                const bool raise = mx > m_ref + SK_RESCALE_SLACK;
                if (__any(raise)) {
                    const float alpha = raise ? sk_exp2(m_ref - mx) : 1.0f;
                    l_run *= alpha;
#pragma unroll
                    for (int h = 0; h < NH; ++h)
#pragma unroll
                        for (int b = 0; b < 4; ++b) o[h][b] *= alpha;
                    m_ref = raise ? mx : m_ref;
                }
                const float neg_m = m_ref == SK_NEG_INF ? 0.f : -m_ref;
                float p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = sk_exp2(fmaf(sc[i], c_scale, neg_m));
                l_run += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        o[h][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[i][h].x, p[i], o[h][0], 0, 0, 0);
                        o[h][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[i][h].y, p[i], o[h][1], 0, 0, 0);
                        o[h][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[i][h].z, p[i], o[h][2], 0, 0, 0);
                        o[h][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[i][h].w, p[i], o[h][3], 0, 0, 0);
                    }
                if (more) load_v(t + 4, vp);
            }
        }

        const float l_tot = sk_sum_over_groups(l_run);
        if (c < nrows) {
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    tr[wave][c][((h * 16 + g4 + i) ^ c) & (CPR - 1)] = make_float4(o[h][0][i], o[h][1][i], o[h][2][i], o[h][3][i]);
            if (g4 == 0) stat[wave][c] = make_float4(m_ref, l_tot, l_tot, 0.f);
        }
        if (sk_meet<D, 16>(P, tr, stat, &decision, tid, nrows, part, alone, slot0, n_parts, unit,
                           [&](const int row) __attribute__((always_inline)) {
                               const int t2 = div_g(row);
                               return (size_t)(w.q_tok0 + t2) * P.g.Hq + head * G + (row - t2 * G);
                           })) return;
        part = alone ? part + 1 : 0;
        alone = true;
    }
}

// ---------------------------------------------------------------------------------------------
// fp32-arithmetic attention kernel for bf16 pools (only on request, for comparison).  Tile of up to 16 query rows x 32 keys; every product and sum is an fp32 FMA.
// Thread (r = tid/16, c = tid%16): scores of row r for keys c and c+16; output
// dimensions c + 16 j of row r.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sk_attn_simple(const sk_launch P)
{
    constexpr int DMAX = 128;
    __shared__ float Qs[16][DMAX + 1];
    __shared__ float Ks[32][DMAX + 1];
    __shared__ float Vs[32][DMAX + 1];
    __shared__ float Ps[16][32 + 1];

    sk_touch_arguments<sizeof(sk_launch)>();
    sk_work w;
    if (!sk_decode_work(P, blockIdx.x, w)) return;
    const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
    const int d = P.g.d, G = P.g.G, Hq = P.g.Hq;
    const int nrows = w.n_tok * G;
    const bool row_valid = r < nrows;
    const int tok_local = row_valid ? r / G : 0;
    const int hq = w.kv_head * G + (row_valid ? r % G : 0);
    const bool causal = w.pos0 < SK_NO_CAUSAL;
    const int p_row = causal ? w.pos0 + tok_local : 0x7fffffff;
    const float c_scale = P.g.scale_log2e;
    const int nd = d >> 4;          // output dims per thread

    for (int idx = tid; idx < 16 * d; idx += 256) {
        int rr = idx / d, t = idx % d;
        float x = 0.f;
        if (rr < nrows) {
            size_t off = ((size_t)(w.q_tok0 + rr / G) * Hq + (w.kv_head * G + rr % G)) * d + t;
            x = bf16_bits_to_f32(((const uint16_t*)P.q)[off]);
        }
        Qs[rr][t] = x;
    }
    float o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = 0.f;
    float m_run = SK_NEG_INF, l_run = 0.f;

    for (int s = 0; s < 3; ++s) {
        sk_seg g = sk_make_seg(P, w, s);
        for (int t0 = g.begin; t0 < g.end; t0 += 32) {
            __syncthreads();
            // stage 32 keys and values as fp32, zero past the end
            for (int idx = tid; idx < 32 * d; idx += 256) {
                int tt = idx / d, t = idx % d;
                int tok = t0 + tt;
                float kx = 0.f, vx = 0.f;
                if (tok < g.end) {
                    const unsigned char* bb = sk_group_base(g, tok & ~15);
                    int slot = tok & (g.B - 1);
                    kx = bf16_bits_to_f32(((const uint16_t*)bb)[(size_t)slot * d + t]);
                    vx = bf16_bits_to_f32(((const uint16_t*)(bb + g.v_off))[((size_t)(slot >> 4) * d + t) * 16 + (slot & 15)]);
                }
                Ks[tt][t] = kx; Vs[tt][t] = vx;
            }
            __syncthreads();
            const int seg_last_pos = g.end - 1 + g.pos_shift;
            const int lim = p_row < seg_last_pos ? p_row : seg_last_pos;
            float sc[2];
            float mt_ = SK_NEG_INF;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int tt = c + 16 * j;
                float acc = 0.f;
                for (int t = 0; t < d; ++t) acc = fmaf(Qs[r][t], Ks[tt][t], acc);
                float x = acc * c_scale;
                x = (t0 + tt + g.pos_shift <= lim && (unsigned)(t0 + tt - g.hole_lo) >= (unsigned)g.hole_n) ? x : SK_NEG_INF;
                sc[j] = x;
                mt_ = fmaxf(mt_, x);
            }
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) mt_ = fmaxf(mt_, __shfl_xor(mt_, off, 64));
            const float m_new = fmaxf(m_run, mt_);
            const float m_use = (m_new == SK_NEG_INF) ? 0.f : m_new;
            const float alpha = (m_run == SK_NEG_INF) ? 0.f : sk_exp2(m_run - m_use);
            float psum = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float p = sk_exp2(sc[j] - m_use);
                Ps[r][c + 16 * j] = p;
                psum += p;
            }
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) psum += __shfl_xor(psum, off, 64);
            l_run = l_run * alpha + psum;
            m_run = m_new;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j < nd) {
                    float acc = o[j] * alpha;
                    const int t = c + 16 * j;
                    for (int tt = 0; tt < 32; ++tt) acc = fmaf(Ps[r][tt], Vs[tt][t], acc);
                    o[j] = acc;
                }
            }
        }
    }
    if (!row_valid) return;
    const size_t orow = ((size_t)(w.q_tok0 + tok_local) * Hq + hq);
    if (w.part < 0) {
        const float inv = 1.0f / l_run;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j < nd) {
                const int t = c + 16 * j;
                if (P.out_dtype == 0) ((float*)P.out)[orow * d + t] = o[j] * inv;
                else ((uint16_t*)P.out)[orow * d + t] = f32_to_bf16_bits(o[j] * inv);
            }
        }
        if (P.lse && c == 0) P.lse[orow] = (m_run + sk_log2(l_run)) * SK_LN2;
    } else {
        const size_t prow = (size_t)w.part * P.rows_per_slot + r;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < nd) P.part_o[prow * d + c + 16 * j] = o[j];
        if (c == 0) *((float4*)P.part_ml + prow) = make_float4(m_run, l_run, l_run, 0.f);
    }
}

// ---------------------------------------------------------------------------------------------
// Cross-split combine: one wave per output row.
//   M = max_s m_s ; L = sum_s l_s 2^(m_s - M) ; O = sum_s O_s 2^(m_s - M) / L
//   LSE = (M + log2 sum_s lx_s 2^(m_s - M)) ln 2       (lx: the row sums before bf16 rounding)
// A row tile and KV head's workgroups lie as many apart as there are of those, as the attention kernel's do: where that is a
// multiple of 8 both run on one XCD.  On another, the lines of the parts stay behind in its L2, and the next call's stores to the same slots
// wait for them to be taken back there (128 rows, 33 to 134 MB of keys loaded non-temporal, which do not push them out: 6 us
// a call, 24.5 -> 18.1 at 14,800 cached tokens, 34.8 -> 28.4 at 32,768).
// The parts of a round (R of them) are requested at once, beside the statistics: buffer loads return zeros behind the
// last part, so no branch stands between the loads.  R is the smallest of 8, 16 and 32 that takes the launch's parts in one
// round (kernels of few registers for launches of few parts: more rows in flight), 1 where a round would reach beyond
// 32-bit offsets.
// Bound: launch, two round trips (statistics and rows come in one), and the read of the parts for large calls (256 tokens of 32 heads in
// eight parts: 34 MB).  Against rounds of eight, each branch around its load and shuffles through LDS (us per call, whole): 23-token
// query at 14,800 cached 23.3 -> 21.6; 16 at 32,768 33.7 -> 31.8; 77-token append and 5-token query at 9,001 51.0 -> 48.3; 256-token
// append at 32,512 134.5 -> 132.2.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(2))) unsigned sk_u32x2;

// What the requests need comes in arguments of their own (the first 14 words of a kernel's arguments are in registers when a wave starts): where every tile has the same number of parts they
// go out before the argument block, which nobody has read yet, has arrived (0.7 us).
template <int D, int R>
__global__ __launch_bounds__(256) void sk_combine(const float* const part_ml, const float* const part_o, const uint32_t by_heads_mul, const int32_t by_heads_shift,
                                                  const int32_t Hkv, const int32_t rows_per_slot, const int32_t n_splits, const int32_t parts_all,
                                                  const int32_t tile_rows, const int32_t all_rows, const sk_launch P)
{
    const int item = blockIdx.x;                  // row tile and KV head
    const int row = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int n_parts = parts_all, part0, part_stride, q_tok0 = 0, kv_head;
    if (parts_all > 0) {
        const int tile = sk_divide(item, sk_div{by_heads_mul, by_heads_shift});
        kv_head = item - tile * Hkv;
        if (row >= tile_rows || row >= all_rows - tile * tile_rows) return;
        part0 = tile * n_splits * Hkv + kv_head; part_stride = Hkv;
        q_tok0 = tile;                            // (times the tile's tokens, below)
    } else {
        sk_touch_arguments<sizeof(sk_launch)>();
        sk_comb cb;
        if (P.mode == SK_MODE_LIST) cb = P.comb[item];
        else {
            const int tile = sk_divide(item, P.by_heads), head = item - tile * Hkv;
            int tok0 = tile * P.tok_per_tile;
            int ntok = P.n_tok - tok0; ntok = ntok < P.tok_per_tile ? ntok : P.tok_per_tile;
            int kv_vis;
            cb.n_parts = sk_tile_parts(P, tok0, ntok, &kv_vis);
            if (cb.n_parts == 1) return;              // written by the attention kernel
            cb.part0 = tile * P.n_splits * Hkv + head; cb.part_stride = Hkv;
            cb.q_tok0 = tok0; cb.n_tok = ntok; cb.kv_head = head;
        }
        if (row >= cb.n_tok * P.g.G) return;
        n_parts = cb.n_parts; part0 = cb.part0; part_stride = cb.part_stride; q_tok0 = cb.q_tok0; kv_head = cb.kv_head;
    }
    const size_t prow0 = (size_t)part0 * rows_per_slot + row, pstride = (size_t)part_stride * rows_per_slot;
    const float* ml = part_ml + prow0 * 4;
    const unsigned step = R > 1 ? (unsigned)(pstride * D * 4) : 0;
    float M = SK_NEG_INF, L = 0.f, Lx = 0.f, a0 = 0.f, a1 = 0.f;
    if (n_parts > 64) {              // rare: the maximum needs its own pass
        for (int s = lane; s < n_parts; s += 64) M = fmaxf(M, ml[(size_t)s * pstride * 4]);
        M = sk_wave_max(M);
    }
    for (int base = 0; base < n_parts; base += 64) {
        const int cnt = n_parts - base < 64 ? n_parts - base : 64;
        const float4 t = *(const float4*)(ml + (size_t)(base + (lane < cnt ? lane : cnt - 1)) * pstride * 4);
        float x0[R], x1[R];
        auto request = [&](const int j0) __attribute__((always_inline)) {
            const int left = cnt - j0 < R ? cnt - j0 : R;
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(part_o) + (prow0 + (size_t)(base + j0) * pstride) * D, 0,
                                                                                  (int)((unsigned)(left - 1) * step + D * 4), 0x00020000);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (D == 128) {
                    const sk_u32x2 x = __builtin_bit_cast(sk_u32x2, __builtin_amdgcn_raw_buffer_load_b64(rows, (unsigned)j * step + (unsigned)lane * 8, 0, 0));
                    x0[j] = __uint_as_float(x[0]); x1[j] = __uint_as_float(x[1]);
                } else {
                    x0[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (unsigned)j * step + (unsigned)lane * 4, 0, 0)); x1[j] = 0.f;
                }
            }
        };
        request(0);
        if (parts_all > 0 && base == 0) sk_touch_arguments<sizeof(sk_launch)>();
        const float m_s = lane < cnt ? t.x : SK_NEG_INF;
        if (n_parts <= 64) M = sk_wave_max(m_s);
        const float wgt = (m_s == SK_NEG_INF) ? 0.f : sk_exp2(m_s - M);
        L = fmaf(lane < cnt ? t.y : 0.f, wgt, L); Lx = fmaf(lane < cnt ? t.z : 0.f, wgt, Lx);
        for (int j0 = 0; j0 < cnt; j0 += R) {
            if (j0 > 0) request(j0);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const float wj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wgt), j0 + j));    // 0 for parts past the end
                a0 = fmaf(x0[j], wj, a0); a1 = fmaf(x1[j], wj, a1);
            }
        }
    }
    L = sk_wave_sum(L); Lx = sk_wave_sum(Lx);
    const float inv = 1.0f / L;
    if (parts_all > 0) q_tok0 *= P.tok_per_tile;
    const int tok = (int)(((unsigned)row * P.g.g_magic) >> 16);        // rows of a tile: below 256 (see sk_attn_bf16_body)
    const size_t orow = (size_t)(q_tok0 + tok) * P.g.Hq + kv_head * P.g.G + (row - tok * P.g.G);
    if (D == 128) {
        if (P.out_dtype == 0) *(float2*)((float*)P.out + orow * D + 2 * lane) = make_float2(a0 * inv, a1 * inv);
        else *(uint32_t*)((uint16_t*)P.out + orow * D + 2 * lane) = f32_to_bf16_bits(a0 * inv) | ((uint32_t)f32_to_bf16_bits(a1 * inv) << 16);
    } else {
        if (P.out_dtype == 0) ((float*)P.out)[orow * D + lane] = a0 * inv;
        else ((uint16_t*)P.out)[orow * D + lane] = f32_to_bf16_bits(a0 * inv);
    }
    if (P.lse && lane == 0) P.lse[orow] = (M + sk_log2(Lx)) * SK_LN2;
}

// ---------------------------------------------------------------------------------------------
// K/V commit.  One workgroup of 256 threads per (destination 16-token group, KV head); pure bit copies
// through integer lanes.
// ---------------------------------------------------------------------------------------------

// bf16, head_dim D: every thread takes one 16-byte chunk of a K row and of a V row; V goes through `vt` (16 rows
// of LDS, 16 * (D + 8) elements) to leave as [dim][16 tokens], in 16-byte pieces when the group starts at its first slot.
// Slots of the group behind the last committed token are zero-filled, so that a key the attention kernel masks
// out never multiplies 0 by leftover bits.
// Bound: one round trip to memory and the launch (128 groups of a 256-token chunk: 4.8 us; 1,304 of a 2,600-token one
// 8.2 -> 5.9 us against a loop over elements with divisions by run-time row lengths).
template <int D>
__device__ __forceinline__ void sk_commit_group(const sk_geom& g, const void* k, const void* v, const sk_scatter& it, const int head,
                                                int32_t* tables_rw, unsigned char* kv_rw, uint16_t* vt)
{
    constexpr int CPR = D / 8, LD = D + 8;                  // 16-byte chunks of a row; LDS row length
    const int tid = threadIdx.x, row = tid / CPR, cc = tid % CPR;
    unsigned char* dst = kv_rw + it.dst_off + (int64_t)head * (it.to_eph ? g.eph_head_stride : g.head_stride);
    if (it.tbl_index >= 0 && head == 0 && tid == 0) tables_rw[it.tbl_index] = it.block_id;
    if (row < it.count) {
        const size_t src = ((size_t)(it.src_tok0 + row) * g.Hkv + head) * (D * 2) + cc * 16;
        const uint4 x = *(const uint4*)((const unsigned char*)k + src), y = *(const uint4*)((const unsigned char*)v + src);
        *(uint4*)(dst + (it.dst_slot0 + row) * (D * 2) + cc * 16) = x;
        *(uint4*)(vt + row * LD + cc * 8) = y;
    }
    __syncthreads();
    if (tid >= 2 * D) return;
    const int first = it.dst_slot0 & 15;                    // position inside the 16-token group
    const int dim = tid >> 1, s0 = (tid & 1) * 8 - first;   // two threads per dimension, eight slots each; s0: token of the first
    uint16_t* vd = (uint16_t*)(dst + (it.to_eph ? g.eph_v_off : g.v_off)) + (size_t)(it.dst_slot0 >> 4) * D * 16 + dim * 16 + (tid & 1) * 8;
    uint32_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = (s0 + j >= 0 && s0 + j < it.count) ? vt[(s0 + j) * LD + dim] : 0u;
    if (first == 0) *(uint4*)vd = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (s0 + j >= 0) vd[j] = (uint16_t)e[j];
    }
}

// f32: rows as they are
__device__ __forceinline__ void sk_commit_group_f32(const sk_geom& g, const void* k, const void* v, const sk_scatter& it, const int head,
                                                    int32_t* tables_rw, unsigned char* base)
{
    unsigned char* dst = base + it.dst_off + (int64_t)head * (it.to_eph ? g.eph_head_stride : g.head_stride);
    const int v_off = it.to_eph ? g.eph_v_off : g.v_off, tid = threadIdx.x;
    if (it.tbl_index >= 0 && head == 0 && tid == 0) tables_rw[it.tbl_index] = it.block_id;
    const int log2_cpr = g.d == 128 ? 5 : 4;                // 16-byte chunks per row
    for (int c = tid; c < it.count << log2_cpr; c += 256) {
        const int row = c >> log2_cpr, cc = c & ((1 << log2_cpr) - 1);
        const size_t src = (((size_t)(it.src_tok0 + row) * g.Hkv + head) << (log2_cpr + 4)) + cc * 16;
        const size_t to = ((size_t)(it.dst_slot0 + row) << (log2_cpr + 4)) + cc * 16;
        const uint4 x = *(const uint4*)((const unsigned char*)k + src), y = *(const uint4*)((const unsigned char*)v + src);
        *(uint4*)(dst + to) = x;
        *(uint4*)(dst + v_off + to) = y;
    }
}

__device__ __forceinline__ void sk_scatter_item(const sk_geom& g, const void* k, const void* v, const sk_scatter& it,
                                                const int head, int32_t* tables_rw, unsigned char* kv_rw, unsigned char* eph_rw)
{
    __shared__ __attribute__((aligned(16))) uint16_t vt[16 * (128 + 8)];
    if (g.elem == 2) {
        unsigned char* base = it.to_eph ? eph_rw : kv_rw;
        if (g.d == 128) sk_commit_group<128>(g, k, v, it, head, tables_rw, base, vt);
        else sk_commit_group<64>(g, k, v, it, head, tables_rw, base, vt);
        return;
    }
    sk_commit_group_f32(g, k, v, it, head, tables_rw, it.to_eph ? eph_rw : kv_rw);
}

// Items read from a list in pinned host memory or in the workspace.  A batched call's list has items of another kind behind the others, which
// copy the lists that its other launches read from pinned memory to the workspace.
// Bound of those: the host link's latency, beside the commit.
__global__ __launch_bounds__(256) void sk_scatter_kernel(const sk_geom g, const sk_div by_heads, const void* k, const void* v,
                                                         const sk_scatter* items, int32_t* tables_rw,
                                                         unsigned char* kv_rw, unsigned char* eph_rw)
{
    const int i = sk_divide(blockIdx.x, by_heads), head = blockIdx.x - i * g.Hkv;
    const sk_scatter it = items[i];                          // at once: the list may lie in host memory
    if (it.to_eph == SK_COPY_LIST) {
        const int at = head * 256 + threadIdx.x;
        if (at < it.count) ((uint4*)(eph_rw + it.dst_off))[at] = ((const uint4*)items)[it.src_tok0 + at];
        return;
    }
    sk_scatter_item(g, k, v, it, head, tables_rw, kv_rw, eph_rw);
}
// ... or carried in the kernel arguments (single-session calls: no host-to-device copy in front)
__global__ __launch_bounds__(256) void sk_scatter_kernel_args(const sk_geom g, const sk_div by_heads, const void* k, const void* v,
                                                              const sk_scatter_list items, int32_t* tables_rw,
                                                              unsigned char* kv_rw, unsigned char* eph_rw)
{
    const int i = sk_divide(blockIdx.x, by_heads);
    sk_scatter_item(g, k, v, items.item[i], blockIdx.x - i * g.Hkv, tables_rw, kv_rw, eph_rw);
}


// Reads committed K/V back in token order (bit copy).  One thread per element pair is enough:
// this is a verification / export path.
__global__ __launch_bounds__(256) void sk_gather_kernel(const sk_geom g, int32_t tbl_off, int64_t first,
                                                        int64_t count, void* k_out, void* v_out)
{
    const int d = g.d;
    const int64_t total = count * g.Hkv * d;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(idx % d);
        const int head = (int)((idx / d) % g.Hkv);
        const int64_t tok = first + idx / ((int64_t)d * g.Hkv);
        const int blk = g.tables[tbl_off + (tok >> g.log2B)];
        const int slot = (int)(tok & (g.B - 1));
        const unsigned char* bb = g.kv + (int64_t)blk * g.blk_stride + (int64_t)head * g.head_stride;
        if (g.elem == 2) {
            ((uint16_t*)k_out)[idx] = ((const uint16_t*)bb)[(size_t)slot * d + t];
            ((uint16_t*)v_out)[idx] = ((const uint16_t*)(bb + g.v_off))[((size_t)(slot >> 4) * d + t) * 16 + (slot & 15)];
        } else {
            ((uint32_t*)k_out)[idx] = ((const uint32_t*)bb)[(size_t)slot * d + t];
            ((uint32_t*)v_out)[idx] = ((const uint32_t*)(bb + g.v_off))[(size_t)slot * d + t];
        }
    }
}

// Copies pool block `src` to block `dst`, all KV heads (the one block a fork or a copy-on-write
// duplicates).  Offsets are formed in 64 bits: a head's blocks lie head_stride bytes apart, which
// exceeds 2 GiB in large pools.
__global__ __launch_bounds__(256) void sk_copy_block_kernel(const sk_geom g, unsigned char* kv_rw, int32_t src, int32_t dst)
{
    const int head = blockIdx.y;
    const int64_t n16 = g.blk_stride >> 4;
    const uint4* s4 = (const uint4*)(kv_rw + (int64_t)head * g.head_stride + (int64_t)src * g.blk_stride);
    uint4* d4 = (uint4*)(kv_rw + (int64_t)head * g.head_stride + (int64_t)dst * g.blk_stride);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x) d4[i] = s4[i];
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------
int sk_launch_scatter(const sk_geom& g, const void* k, const void* v, const sk_scatter* items,
                      int32_t n_items, int32_t* tables_rw, unsigned char* kv_rw, unsigned char* eph_rw,
                      void* stream)
{
    if (n_items <= 0) return 0;
    hipLaunchKernelGGL(sk_scatter_kernel, dim3(n_items * g.Hkv), dim3(256), 0, (hipStream_t)stream,
                       g, sk_make_div((uint32_t)g.Hkv), k, v, items, tables_rw, kv_rw, eph_rw);
    return (int)hipGetLastError();
}

int sk_launch_scatter_args(const sk_geom& g, const void* k, const void* v, const sk_scatter_list& items,
                           int32_t n_items, int32_t* tables_rw, unsigned char* kv_rw, unsigned char* eph_rw,
                           void* stream)
{
    if (n_items <= 0) return 0;
    hipLaunchKernelGGL(sk_scatter_kernel_args, dim3(n_items * g.Hkv), dim3(256), 0, (hipStream_t)stream,
                       g, sk_make_div((uint32_t)g.Hkv), k, v, items, tables_rw, kv_rw, eph_rw);
    return (int)hipGetLastError();
}

// The two launchers below take an optional pair of events that the runtime fills with the
// dispatch's own start and end time stamps (the figures a profiler reports for the kernel), for
// sk_pool_set_profiling; without them they are plain launches.
#define SK_LAUNCH(kernel, grid, block)                                                                              \
    do {                                                                                                            \
        if (ev_start) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, (hipEvent_t)ev_start, (hipEvent_t)ev_stop, 0, L); \
        else hipLaunchKernelGGL(kernel, grid, block, 0, st, L);                                                     \
    } while (0)

int sk_launch_attention(const sk_launch& L, int variant, int32_t n_workgroups, void* stream, void* ev_start, void* ev_stop)
{
    if (n_workgroups <= 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    if (variant != SK_KV_SIMPLE && L.g.d != 128 && !(L.g.d == 64 && variant != SK_KV_MFMA128P)) return (int)hipErrorInvalidValue;
    const bool d64 = L.g.d == 64;
    switch (variant) {
    case SK_KV_MFMA256:
        if (d64) SK_LAUNCH((sk_attn_bf16_d64<8, 1, 4>), dim3(n_workgroups), dim3(512));
        else SK_LAUNCH((sk_attn_bf16_d128<8, 1, 4>), dim3(n_workgroups), dim3(512));
        break;
    case SK_KV_MFMA128:
        if (d64) SK_LAUNCH((sk_attn_bf16_d64<4, 1, 2>), dim3(n_workgroups), dim3(256));
        else SK_LAUNCH((sk_attn_bf16_d128<4, 1, 2>), dim3(n_workgroups), dim3(256));
        break;
    case SK_KV_MFMA64:
        if (d64) SK_LAUNCH((sk_attn_bf16_d64<2, 2, 2>), dim3(n_workgroups), dim3(256));
        else SK_LAUNCH((sk_attn_bf16_d128<2, 2, 2>), dim3(n_workgroups), dim3(256));
        break;
    case SK_KV_MFMA128P:     SK_LAUNCH((sk_attn_bf16_d128<4, 2, 2>), dim3(n_workgroups), dim3(512)); break;
    default:
        if (L.g.elem != 2) return (int)hipErrorInvalidValue;
        SK_LAUNCH(sk_attn_simple, dim3(n_workgroups), dim3(256));
    }
    return (int)hipGetLastError();
}

// The kernels that can read the call's own K/V in place and commit them: sk_attn_bf16_small, and sk_attn_f32 (every call
// of an fp32 pool; a batched one with own_mode none and nothing to commit).
int sk_launch_attention_small(const sk_launch& L, const sk_commit& C, int32_t n_workgroups, void* stream, void* ev_start, void* ev_stop)
{
    if (n_workgroups <= 0) return 0;
    hipStream_t st = (hipStream_t)stream;
#define SK_LAUNCH_SMALL(kernel, ...)                                                                                \
    do {                                                                                                            \
        if (ev_start) hipExtLaunchKernelGGL(kernel, dim3(n_workgroups), dim3(256), 0, st, (hipEvent_t)ev_start, (hipEvent_t)ev_stop, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(kernel, dim3(n_workgroups), dim3(256), 0, st, __VA_ARGS__);                         \
    } while (0)
    if (L.g.elem == 4) {
        if (L.g.d == 128) SK_LAUNCH_SMALL(sk_attn_f32<128>, L, C);
        else if (L.g.d == 64) SK_LAUNCH_SMALL(sk_attn_f32<64>, L, C);
        else return (int)hipErrorInvalidValue;
        return (int)hipGetLastError();
    }
    // G | log2B << 8 | shift of by_pad << 12 | padded << 17 | tokens << 18 | own tokens << 24 (at most 32 rows per KV head); a head's blocks
    // lie whole 4 KiB pages apart (a block holds K and V of at least 16 tokens of 64 dims)
    if (L.g.G < 1 || L.g.G > 255 || L.g.log2B > 15 || L.by_pad.shift > 31 || L.n_tok < 1 || L.n_tok * L.g.G > 32 || L.own_cnt < 0 || L.own_cnt > 32 ||
        (L.g.head_stride & 4095) || (L.g.head_stride >> 44) || (L.head_pad != L.g.Hkv && L.head_pad != ((L.g.Hkv + 7) & ~7)))
        return (int)hipErrorInvalidValue;          // would not fit its field, or the kernel's LDS
    const uint32_t shape = (uint32_t)L.g.G | (uint32_t)L.g.log2B << 8 | (uint32_t)L.by_pad.shift << 12 | (L.head_pad != L.g.Hkv ? 1u : 0u) << 17 |
                           (uint32_t)L.n_tok << 18 | (uint32_t)L.own_cnt << 24;
    const int32_t* table = L.g.tables + L.tbl_off;
    const unsigned char* q = (const unsigned char*)L.q;
    const uint32_t pages = (uint32_t)(L.g.head_stride >> 12);
    constexpr void (*kernel)(const int32_t*, const unsigned char*, const unsigned char*, uint32_t, int32_t, uint32_t, uint32_t, uint32_t, int32_t, int32_t,
                             int32_t, sk_launch, sk_commit) = sk_attn_bf16_small<128>;         // (a changed parameter list does not convert)
    static_assert(sk_argument_offset<11>(kernel) == offsetof(sk_small_args, P) && sk_argument_offset<12>(kernel) == offsetof(sk_small_args, C) &&
                  sk_argument_offset<6>(kernel) == offsetof(sk_small_args, pad_mul), "the kernel reads its arguments through sk_small_args");
#define SK_SMALL_ARGS table, q, L.g.kv, pages, L.g.Hkv, shape, L.by_pad.mul, L.g.g_magic, L.n_splits, L.chunk, L.kv_len, L, C
    if (L.g.d == 128) SK_LAUNCH_SMALL(sk_attn_bf16_small<128>, SK_SMALL_ARGS);
    else if (L.g.d == 64) SK_LAUNCH_SMALL(sk_attn_bf16_small<64>, SK_SMALL_ARGS);
    else return (int)hipErrorInvalidValue;
#undef SK_SMALL_ARGS
#undef SK_LAUNCH_SMALL
    return (int)hipGetLastError();
}

// max_parts: the most parts of a row tile of the launch; part_stride: slots from one part to the next.
int sk_launch_combine(const sk_launch& L, int32_t n_row_tiles, int32_t max_parts, int64_t part_stride, void* stream, void* ev_start, void* ev_stop)
{
    if (n_row_tiles <= 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid(n_row_tiles, L.rows_per_slot >> 2), block(256);
    const int64_t step = part_stride * L.rows_per_slot * L.g.d * 4;
    int round = max_parts <= 8 ? 8 : max_parts <= 16 ? 16 : 32;
    while (round > 1 && round * step >= (int64_t(1) << 32)) round = round > 8 ? round / 2 : 1;
    // Whether every tile has the same number of parts: by what the first tile and the last one see.
    int parts_all = 0;
    if (L.mode == SK_MODE_REGULAR && L.own_mode == SK_OWN_SMALL) parts_all = L.n_splits;
    else if (L.mode == SK_MODE_REGULAR && L.own_mode == SK_OWN_NONE) {
        const int first = L.n_tok < L.tok_per_tile ? L.n_tok : L.tok_per_tile;
        const int vis = L.pos0 < SK_NO_CAUSAL && L.pos0 + first < L.kv_len ? L.pos0 + first : L.kv_len;
        const int own = L.eph_cnt[0] > 0 || L.eph_cnt[1] > 0 ? 1 : 0;
        if ((vis + L.chunk - 1) / L.chunk + own == L.n_splits && L.n_splits > 1) parts_all = L.n_splits;
    }
    const sk_div by_heads = L.by_heads;
    const int32_t tile_rows = L.tok_per_tile * L.g.G, all_rows = L.n_tok * L.g.G;
#define SK_LAUNCH_COMBINE_R(D, R)                                                                                   \
    do {                                                                                                            \
        if (ev_start) hipExtLaunchKernelGGL((sk_combine<D, R>), grid, block, 0, st, (hipEvent_t)ev_start, (hipEvent_t)ev_stop, 0, L.part_ml, L.part_o, \
                                            by_heads.mul, by_heads.shift, L.g.Hkv, L.rows_per_slot, L.n_splits, parts_all, tile_rows, all_rows, L); \
        else hipLaunchKernelGGL((sk_combine<D, R>), grid, block, 0, st, L.part_ml, L.part_o,                        \
                                by_heads.mul, by_heads.shift, L.g.Hkv, L.rows_per_slot, L.n_splits, parts_all, tile_rows, all_rows, L); \
    } while (0)
#define SK_LAUNCH_COMBINE(D)                                                                                        \
    do {                                                                                                            \
        if (round == 32) SK_LAUNCH_COMBINE_R(D, 32);                                                                \
        else if (round == 16) SK_LAUNCH_COMBINE_R(D, 16);                                                           \
        else if (round == 8) SK_LAUNCH_COMBINE_R(D, 8);                                                             \
        else SK_LAUNCH_COMBINE_R(D, 1);                                                                             \
    } while (0)
    if (L.g.d == 128) SK_LAUNCH_COMBINE(128);
    else SK_LAUNCH_COMBINE(64);
#undef SK_LAUNCH_COMBINE
#undef SK_LAUNCH_COMBINE_R
    return (int)hipGetLastError();
}
#undef SK_LAUNCH

int sk_launch_gather(const sk_geom& g, int32_t tbl_off, int64_t first, int64_t count,
                     void* k_out, void* v_out, void* stream)
{
    if (count <= 0) return 0;
    int64_t total = count * g.Hkv * g.d;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    hipLaunchKernelGGL(sk_gather_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       g, tbl_off, first, count, k_out, v_out);
    return (int)hipGetLastError();
}

int sk_launch_copy_block(const sk_geom& g, unsigned char* kv_rw, int32_t src, int32_t dst, void* stream)
{
    const int64_t n16 = g.blk_stride >> 4;
    int64_t bx = (n16 + 255) / 256;
    if (bx > 64) bx = 64;
    hipLaunchKernelGGL(sk_copy_block_kernel, dim3((unsigned)bx, (unsigned)g.Hkv), dim3(256), 0, (hipStream_t)stream, g, kv_rw, src, dst);
    return (int)hipGetLastError();
}
