// CDNA4 (gfx950) kernels of the pipelined-sharding hot path: the dequantising matmuls of
// the decoder sub-layers with their fused RMSNorm / SwiGLU / residual steps, MoE routing and
// the expert combine, and attention over the KV cache.  Weight layout: see pack.cpp.  wave64 only.
//   matmuls by token count:  1 -> gemv_w4_kernel,  2..4 -> gemv_mt_kernel (whole scale groups),
//                            otherwise gemm_w4_kernel (+ splitk_epilogue* when K is split), or gemm_kslice_kernel
//                            (narrow matrices, more than 64 tokens; O from 49 tokens)
//   attention:  one query token -> attn_decode_kernel + attn_combine_kernel,
//               a chunk of query tokens -> attn_chunk_kernel, one walk over the cache and the chunk's own
//               rows; for a short chunk the walk is dealt out to several workgroups, whose records
//               attn_combine_chunk_kernel merges
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <cstdlib>

#include "kernels.h"

namespace ps {

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ h2_t as_h2(uint32_t v) { return __builtin_bit_cast(h2_t, v); }

// streaming 16-byte load: weights are read once per step, keep them out of the way of the caches
__device__ __forceinline__ uint4 load_stream(const uint4 *p) {
    const u4_t v = __builtin_nontemporal_load(reinterpret_cast<const u4_t *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 8 codes of one dword -> four fp16 pairs holding (q - 8), exact.  Codes sit in the
// mantissa of 1024 + q (low nibbles) or 1024 + 16 q (next nibbles).
// (v & mask) | magic in one VALU op: the mask rides the scalar operand slot, the magic a VGPR
__device__ __forceinline__ uint32_t and_or(uint32_t v, uint32_t mask, uint32_t magic) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(mask), "v"(magic));
    return r;
}

__device__ __forceinline__ void dequant8(uint32_t v, h2_t w[4]) {
    const h2_t k1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    const h2_t k16th = {(_Float16)0.0625f, (_Float16)0.0625f};
    const h2_t k72 = {(_Float16)72.0f, (_Float16)72.0f};
    const uint32_t v8 = v >> 8;
    w[0] = as_h2(and_or(v, 0x000F000Fu, 0x64006400u)) - k1032;
    w[1] = __builtin_elementwise_fma(as_h2(and_or(v, 0x00F000F0u, 0x64006400u)), k16th, -k72);
    w[2] = as_h2(and_or(v8, 0x000F000Fu, 0x64006400u)) - k1032;
    w[3] = __builtin_elementwise_fma(as_h2(and_or(v8, 0x00F000F0u, 0x64006400u)), k16th, -k72);
}

// Decode dot product of 8 codes with 8 activations WITHOUT removing the code offsets: the fp16
// patterns 1024 + q (codes 0, 1, 4, 5 of the dword) and 1024 + 16 q (codes 2, 3, 6, 7) go straight
// into the fp32 dot-product accumulators lo / hi.  With S_lo, S_hi the sums of the activations at
// those positions, sum((q - 8) x) = lo + hi / 16 - 1032 S_lo - 72 S_hi; the two S terms depend on
// the activations only and are shared by every row (see gemv_item).  Saves the four packed
// subtract / multiply-add operations per dword; the fp32 accumulators carry terms near 1024 |x|,
// which costs about 1e-4 of a block's sum in relative accuracy.
__device__ __forceinline__ void dot8_raw(uint32_t v, uint4 x, float &lo, float &hi) {
    const uint32_t v8 = v >> 8;
    lo = __builtin_amdgcn_fdot2(as_h2(and_or(v, 0x000F000Fu, 0x64006400u)), as_h2(x.x), lo, false);
    hi = __builtin_amdgcn_fdot2(as_h2(and_or(v, 0x00F000F0u, 0x64006400u)), as_h2(x.y), hi, false);
    lo = __builtin_amdgcn_fdot2(as_h2(and_or(v8, 0x000F000Fu, 0x64006400u)), as_h2(x.z), lo, false);
    hi = __builtin_amdgcn_fdot2(as_h2(and_or(v8, 0x00F000F0u, 0x64006400u)), as_h2(x.w), hi, false);
}

__device__ __forceinline__ float half_of(uint4 v, int s) {  // s-th fp16 of a 16-byte vector
    const uint32_t d = (s < 2) ? v.x : (s < 4) ? v.y : (s < 6) ? v.z : v.w;
    const uint16_t h = (s & 1) ? (uint16_t)(d >> 16) : (uint16_t)(d & 0xFFFFu);
    return (float)__builtin_bit_cast(_Float16, h);
}

__device__ __forceinline__ float sumsq8(uint4 v) {
    float s = 0.f;
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const h2_t p = as_h2(d[i]);
        s += (float)p.x * (float)p.x;
        s += (float)p.y * (float)p.y;
    }
    return s;
}

// sum over the wave, the same value in every lane: the 16 lanes of a row meet through DPP row
// operations, the four rows through four lane reads (no LDS permutes, whose six dependent round
// trips cost a wave several hundred cycles)
__device__ __forceinline__ float wave_sum(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));  // row_half_mirror
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));  // row_mirror
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)), r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)), r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return (r0 + r1) + (r2 + r3);
}

// Lanes l, l ^ 16, l ^ 32, l ^ 48 (one column of the wave's four rows) meet, the result in all four:
// (row 0 + row 1) + (row 2 + row 3), by the row-swap instructions of gfx950 (vector ALU, no LDS
// permute).  v_permlane16_swap exchanges the odd rows of its first operand with the even rows of its
// second, v_permlane32_swap the upper half of the first with the lower half of the second; with both
// operands the same value, the two results are the two partners of every lane (lane layout checked
// on the hardware with lane numbers as data).
template <bool MAX = false>
__device__ __forceinline__ float rows4_meet(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
    // written as instructions: the two operands are exchanged in place, so they are two registers
    // holding the same value (this compiler's builtin for the swap loses its second result when
    // the two results are combined, checked on the hardware); s_nop covers the write-to-swap
    // hazard the compiler would otherwise pad
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    float y = MAX ? __builtin_elementwise_maximum(a, b) : a + b, z = y;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(y), "+v"(z));
    return MAX ? __builtin_elementwise_maximum(y, z) : y + z;
#else
    return v;
#endif
}

// fp32 -> fp16 with the rounding kept as its own step: the value passes through an opaque
// register so the compiler cannot merge the producing multiply/add into a mixed-precision
// convert in one kernel and not in another (the decode paths must agree bit for bit)
__device__ __forceinline__ __half to_half(float v) {
    asm volatile("" : "+v"(v));
    return __float2half(v);
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// raw buffer descriptor over the whole 32-bit offset range from `base` (offsets are validated on the
// host); loads through it take a 32-bit lane offset plus a scalar offset
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)0xFFFFFFFFu, 0x00020000);
}
typedef __attribute__((address_space(3))) void lds_void;
// 16 bytes per lane from global memory straight into LDS: lane l of the wave lands at dst + 16 l
// (dst is wave-uniform), without passing through registers.  The host pass has no such builtin and
// only needs the kernel's signature.
__device__ __forceinline__ void load_to_lds16(__amdgpu_buffer_rsrc_t rsrc, lds_void *dst, uint32_t voff, uint32_t soff) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, voff, soff, 0, 0);
#endif
}
constexpr int kAuxNt = 2;   // non-temporal: streamed weights are not worth keeping in cache

// source column of logical input column k: identity, or the identity-on-V attention
// stand-in where query head h reads kv head h / group (head_dim 128)
__device__ __forceinline__ uint32_t gather_col(uint32_t k, uint32_t x_off, uint32_t group) {
    return x_off + ((k >> 7) / group) * 128u + (k & 127u);
}

// ------------------------------------------------------------------------------------
// MoE routing: per token the top_k largest fp32 logits (ties to the lower index, listed
// in descending order) and the softmax over the selected logits.  One wave per token.
// ------------------------------------------------------------------------------------
// Wave-wide maximum / minimum, the same value in every lane: the 16 lanes of a row meet through DPP
// row operations (no LDS traffic), the four rows through four lane reads.
__device__ __forceinline__ int dpp_i(int v, int ctrl) {
    switch (ctrl) {
        case 0: return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // quad_perm 1,0,3,2
        case 1: return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm 2,3,0,1
        case 2: return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror
        default: return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
    }
}
__device__ __forceinline__ float wave_max_all(float v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) v = fmaxf(v, __builtin_bit_cast(float, dpp_i(__builtin_bit_cast(int, v), c)));
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)), r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)), r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
__device__ __forceinline__ uint32_t wave_min_all(uint32_t v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) v = min(v, (uint32_t)dpp_i((int)v, c));
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return min(min(r0, r1), min(r2, r3));
}

template <int NR>   // 64 * NR >= E
__device__ __forceinline__ void route_tokens(const RouteArgs &ra, uint32_t block) {   // four tokens, one per wave
    const float *logits = ra.logits;
    const uint32_t M = ra.M, E = ra.E, top_k = ra.top_k;
    int32_t *idx = ra.idx;
    float *w = ra.w;
    const uint32_t m = block * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (m >= M) return;
    const float *l = logits + (size_t)m * E;
    float v[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint32_t e = r * 64 + lane;
        v[r] = e < E ? l[e] : -INFINITY;
    }
    uint32_t taken = 0;  // bit r: this lane's entry r already selected
    float sel = 0.f, lmax = 0.f;
    for (uint32_t j = 0; j < top_k; ++j) {
        float best = -INFINITY;
        uint32_t be = 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const uint32_t e = r * 64 + lane;
            if (e < E && !((taken >> r) & 1u) && (be == 0xFFFFFFFFu || v[r] > best)) { best = v[r]; be = e; }
        }
        // the largest value in the wave, then the lowest index among the lanes that hold it
        // (a lane with nothing left holds -inf and the index 0xFFFFFFFF, which never wins)
        const float top = wave_max_all(best);
        be = wave_min_all(best == top ? be : 0xFFFFFFFFu);
        best = top;
        if ((be & 63u) == (uint32_t)lane) taken |= 1u << (be >> 6);
        if (j == 0) lmax = best;
        if ((uint32_t)lane == j) sel = best;
        if (lane == 0) idx[(size_t)m * top_k + j] = (int32_t)be;
    }
    const float ex = (uint32_t)lane < top_k ? __expf(sel - lmax) : 0.f;
    const float den = wave_sum(ex);
    if ((uint32_t)lane < top_k) w[(size_t)m * top_k + lane] = ex / den;
}

// ------------------------------------------------------------------------------------
// Decode kernel, one token: fused 4-bit dequant GEMV.  A "unit" is one row-tile (16 outputs)
// or, for GATE_UP, a gate tile plus its up tile.  KSPLIT waves share a unit, wave kpart taking
// scale groups kpart, kpart + KSPLIT, ... of K; a workgroup holds NW / KSPLIT units.
// Each wave first issues all weight loads of its group (they do not depend on the
// activations), then fetches only the 1024 activations of that group and spreads them to its
// lanes through a wave-private LDS window (LDS operations of one wave execute in order, so no
// barrier is needed).  The RMSNorm sum of squares is accumulated from the same fetch.
// Partial sums of the KSPLIT waves meet in LDS in a fixed order behind the only barrier, so
// a row's result does not depend on which slab or slot it came from.
// ------------------------------------------------------------------------------------
template <int NT>
struct GemvBuf {
    uint4 sc[NT];
    uint4 wq[NT][8];
    uint4 xa, xb;
};

// weights of scale group g of a unit's NT tiles (independent of the activations).  unit, g and
// nsb_g are the same for the whole wave, so their share of the address is kept in scalar registers
// and the loads take (descriptor, lane offset, scalar offset): no per-lane address arithmetic.
template <int NT, bool FULLG = false>
__device__ __forceinline__ void gemv_issue_w(GemvBuf<NT> &b, const uint4 *W, uint32_t unit, uint32_t tile_u4,
                                             uint32_t g, uint32_t nsb_g, int lane) {
    const __amdgpu_buffer_rsrc_t wb = make_rsrc(W);
    const uint32_t tile_b = tile_u4 * 16u;
    const uint32_t base = __builtin_amdgcn_readfirstlane(unit * NT * tile_b + g * (9u * 1024u));
    // FULLG: every scale group has its 8 super-blocks, so the number of loads in flight is a
    // compile-time fact and the compiler can wait for exactly the load a dot product needs
    const uint32_t nsb_u = FULLG ? 8u : __builtin_amdgcn_readfirstlane(nsb_g);
    const uint32_t voff = (uint32_t)lane * 16u;
    // issue order = consumption order (loads return in order): scales, then super-block by
    // super-block across the tiles, so the dot products of a super-block can start while the later
    // ones are still in flight
#pragma unroll
    for (int t = 0; t < NT; ++t)
        b.sc[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wb, voff, base + t * tile_b + nsb_u * 1024u, kAuxNt));
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (FULLG || (uint32_t)s < nsb_u) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
                b.wq[t][s] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wb, voff, base + t * tile_b + s * 1024u, kAuxNt));
        }
    }
}

// activations of scale group g: 128 chunks of 8, lane takes chunks lane and lane + 64
template <int NT>
__device__ __forceinline__ void gemv_issue_x(GemvBuf<NT> &b, uint32_t g, uint32_t K, const __half *x,
                                             uint32_t x_off, uint32_t x_group, int lane) {
    const uint32_t k0 = g * 1024u + (uint32_t)lane * 8u, k1 = k0 + 512u;
    b.xa = make_uint4(0, 0, 0, 0);
    b.xb = make_uint4(0, 0, 0, 0);
    if (k0 < K) b.xa = *reinterpret_cast<const uint4 *>(x + gather_col(k0, x_off, x_group));
    if (k1 < K) b.xb = *reinterpret_cast<const uint4 *>(x + gather_col(k1, x_off, x_group));
}

// chunk q (0..127) of a group -> slot in the wave's LDS window: block b = q / 4, part p = q % 4,
// super-block sb = b / 4, c = b % 4; the four lanes groups c read distinct banks for a given p
__device__ __forceinline__ uint32_t xslot(uint32_t q) {
    const uint32_t b = q >> 2, p = q & 3u;
    return (b >> 2) * 16u + p * 4u + (b & 3u);
}

// LDS of one decode workgroup of NW waves: a 2 KB activation window per wave and the reduction
// scratch.  The scratch holds one
// partial sum per (unit, scale group): a row's result is the sum of its scale-group partials in
// ascending group order, whichever wave produced which partial -- so it depends neither on the
// K split nor on the workgroup shape, let alone on the slab or slot the weights came from.
constexpr int kMaxGroups = 16;   // K <= 16384
template <int NW>
struct GemvLds {
    uint4 x[NW][128];
    float red[(NW > 1 ? NW / 2 : 1) * kMaxGroups][2][16];   // K split >= 2: at most NW / 2 units per workgroup
    float red_ss[(NW > 1 ? NW / 2 : 1) * kMaxGroups];
    float corr[NW][32];   // per wave: code-offset corrections of the current scale group
};

// One work item of the decode GEMV: the NW waves of the workgroup cover NW / ks units, ks
// waves per unit.
// DBUF: a wave with several scale groups issues the next group's loads before computing the
// current one (costs a second register buffer; the one-tile modes can afford it).
template <int MODE, int NW, bool DBUF = false, bool FULLG = false>
__device__ __forceinline__ void gemv_item(const GemvArgs &a, const uint4 *W, const __half *x, __half *out,
                                          float *out_f32, uint32_t item, uint32_t ks, GemvLds<NW> &lds) {
    constexpr int NT = (MODE == GEMV_GATE_UP) ? 2 : 1;
    constexpr bool NORM = (MODE == GEMV_PLAIN || MODE == GEMV_GATE_UP);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, c = lane >> 4;
    const uint32_t units = NW / ks;
    const uint32_t unit = item * units + wave / ks;
    const uint32_t kpart = wave % ks;
    const bool active = unit < a.nunits;
    float acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = 0.f;
    float ss = 0.f;
    uint4 *win = lds.x[wave];
    const uint32_t row = a.out_row0 + unit * 16 + i;
    float resv = 0.f;   // residual of this lane's output row, fetched early (it only waits on the previous phase)
    const bool writer = active && kpart == 0 && c == 0;

    if (active && kpart < a.ngroups) {
        GemvBuf<NT> cur, nxt;
        uint32_t g = kpart;
        // activations first: they are ready (and cached), and nothing can be computed before them
        gemv_issue_x<NT>(cur, g, a.K, x, a.x_off, a.x_group, lane);
        gemv_issue_w<NT, FULLG>(cur, W, unit, a.tile_u4, g, min(8u, a.nsb - g * 8u), lane);
        if (MODE == GEMV_RESID && writer && a.res) resv = __half2float(a.res[row]);
        while (true) {
            const uint32_t nsb_g = FULLG ? 8u : min(8u, a.nsb - g * 8u);
            const uint32_t gn = g + ks;
            const bool more = gn < a.ngroups;
            if (DBUF && more) {
                gemv_issue_x<NT>(nxt, gn, a.K, x, a.x_off, a.x_group, lane);
                gemv_issue_w<NT, FULLG>(nxt, W, unit, a.tile_u4, gn, min(8u, a.nsb - gn * 8u), lane);
            }
            win[xslot(lane)] = cur.xa;
            win[xslot(lane + 64)] = cur.xb;
            // code-offset corrections (see dot8_raw): lane (c, i) sums the activations of super-block
            // i % 8, lane group c, that meet low-pattern and high-pattern codes; 1032 S_lo + 72 S_hi
            // goes through LDS and each lane picks up the term of its c per super-block
            {
                const uint32_t *wp = reinterpret_cast<const uint32_t *>(win) + ((i & 7) * 16 + c) * 4;
                const h2_t one = {(_Float16)1.0f, (_Float16)1.0f};
                float sl = 0.f, sh = 0.f;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const uint4 xq = *reinterpret_cast<const uint4 *>(wp + p * 16);
                    sl = __builtin_amdgcn_fdot2(as_h2(xq.x), one, sl, false);
                    sh = __builtin_amdgcn_fdot2(as_h2(xq.y), one, sh, false);
                    sl = __builtin_amdgcn_fdot2(as_h2(xq.z), one, sl, false);
                    sh = __builtin_amdgcn_fdot2(as_h2(xq.w), one, sh, false);
                }
                if (i < 8) lds.corr[wave][c * 8 + i] = fmaf(72.0f, sh, 1032.0f * sl);
            }
            const float *corr = &lds.corr[wave][c * 8];
            float gacc[NT];   // this scale group's partial sums
#pragma unroll
            for (int t = 0; t < NT; ++t) gacc[t] = 0.f;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (FULLG || (uint32_t)s < nsb_g) {
                    uint4 xv[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) xv[p] = win[s * 16 + p * 4 + c];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        float lo = 0.f, hi = 0.f;
                        dot8_raw(cur.wq[t][s].x, xv[0], lo, hi);
                        dot8_raw(cur.wq[t][s].y, xv[1], lo, hi);
                        dot8_raw(cur.wq[t][s].z, xv[2], lo, hi);
                        dot8_raw(cur.wq[t][s].w, xv[3], lo, hi);
                        const float part = fmaf(hi, 0.0625f, lo) - corr[s];
                        gacc[t] = fmaf(half_of(cur.sc[t], s), part, gacc[t]);
                    }
                }
            }
            // the 4 lanes of a row (c = 0..3) meet; then the group partial joins the others in group order
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                gacc[t] = rows4_meet<false>(gacc[t]);
            }
            float gss = 0.f;
            if (NORM) gss = wave_sum(sumsq8(cur.xa) + sumsq8(cur.xb));
            if (ks == 1) {   // this wave sees the groups in ascending order: add as it goes
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] += gacc[t];
                ss += gss;
            } else {
                const uint32_t slot = (wave / ks) * kMaxGroups + g;
                if (c == 0) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) lds.red[slot][t][i] = gacc[t];
                }
                if (NORM && lane == 0) lds.red_ss[slot] = gss;
            }
            if (!more) break;
            if (DBUF) {
                cur = nxt;
            } else {
                gemv_issue_x<NT>(cur, gn, a.K, x, a.x_off, a.x_group, lane);
                gemv_issue_w<NT, FULLG>(cur, W, unit, a.tile_u4, gn, min(8u, a.nsb - gn * 8u), lane);
            }
            g = gn;
        }
    }
    if (ks > 1) {
        __syncthreads();
        if (writer) {
            const uint32_t slot0 = (wave / ks) * kMaxGroups;
            for (uint32_t g = 0; g < a.ngroups; ++g) {
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] += lds.red[slot0 + g][t][i];
                if (NORM) ss += lds.red_ss[slot0 + g];
            }
        }
    }
    if (!writer) return;
    const float rinv = NORM ? rsqrtf(ss / (float)a.K + a.eps) : 1.f;
    if (MODE == GEMV_F32) {
        out_f32[row] = acc[0];
        return;
    }
    float v;
    if (MODE == GEMV_PLAIN) v = rinv * acc[0];
    else if (MODE == GEMV_RESID) v = resv + acc[0];
    else v = silu(rinv * acc[0]) * (rinv * acc[NT - 1]);
    out[row] = to_half(v);
}

// ROUTE: the workgroup behind the matrix's routes the token (a MoE layer's routing depends on nothing the layer computes, and
// as a launch of its own it costs 4 to 5 us between O and the experts; here it runs beside O).
template <int MODE, int NW, bool FULLG, bool ROUTE = false>
__global__ __launch_bounds__(NW * 64, 4) void gemv_w4_kernel(GemvArgs a, uint32_t ks, RouteArgs ra) {   // 4 waves per SIMD: at most 128 VGPRs
    if constexpr (ROUTE) {
        if (blockIdx.x == gridDim.x - 1) { route_tokens<4>(ra, 0); return; }
    }
    __shared__ GemvLds<NW> lds;
    const uint4 *W = a.W;
    const __half *x = a.x;
    __half *out = a.out;
    float *out_f32 = a.out_f32;
    if (a.tasks) {  // grouped launch: blockIdx.y selects the expert
        const DeviceTask t = a.tasks[blockIdx.y];
        const uint32_t pair = (uint32_t)a.pairs[t.pair0];
        if (MODE == GEMV_GATE_UP) {
            W = reinterpret_cast<const uint4 *>(t.w_gate_up);
            x = a.x + (size_t)(pair / a.top_k) * a.x_stride;
            out = a.out + (size_t)pair * a.out_stride;
        } else {
            W = reinterpret_cast<const uint4 *>(t.w_down);
            x = a.x + (size_t)pair * a.x_stride;
            out_f32 = a.out_f32 + (size_t)pair * a.out_stride;
        }
    }
    // second register buffer for the one-tile modes (the residual mode with ragged scale groups would
    // spill a register with it)
    constexpr bool DBUF = (MODE == GEMV_F32 || (MODE == GEMV_RESID && FULLG)) && NW < 16;
    gemv_item<MODE, NW, DBUF, FULLG>(a, W, x, out, out_f32, blockIdx.x, ks, lds);
}

// Few units of one or two waves: a workgroup each, so that every unit's weights come through a CU of their own instead of
// four units' through one (K = 1024, 176 gate/up units 4.3 -> 3.9 us; K = 512, QKV 64 units 3.3 -> 2.9, O 32 3.0 -> 2.75, gate/up 88
// 3.7 -> 3.2; K = 2048, O 128 units 4.1 -> 3.8).  Such steps are bound by the host where they are issued launch by launch, so it
// shows where they are replayed (three layers of K = 512 and a head, two steps 160.0 -> 153.1 us).  Beyond one unit per CU the
// larger workgroups are faster (K = 2048, 352 gate/up units 5.3 -> 6.2).
static bool gemv_unit_per_cu(uint32_t nunits, uint32_t ks, uint32_t ntasks) { return ks <= 2 && !ntasks && nunits <= 256; }

template <int MODE, bool FULLG, bool ROUTE = false>
static hipError_t launch_gemv_f(const GemvArgs &a, uint32_t ks, uint32_t ntasks, const RouteArgs &ra, hipStream_t st) {
    // waves per workgroup: at least the K split; two units per workgroup (8 waves) when that still
    // leaves about one workgroup per CU -- fewer, larger workgroups start sooner (measured on the
    // 8B shapes: QKV 6.6 -> 5.4 us, gate/up 13.4 -> 13.0 us; O, with 256 units, is best left at one
    // unit per workgroup).  The result does not depend on the shape.
    uint32_t nw = ks > 8 ? 16 : ks > 4 ? 8 : 4;
    if (ks == 4 && (a.nunits + 1) / 2 >= 192) nw = 8;   // (with one wave per unit, ks < 4, the larger workgroup measured slower)
    if (!ROUTE && gemv_unit_per_cu(a.nunits, ks, ntasks)) nw = ks;
    const uint32_t units = nw / ks;
    dim3 grid((a.nunits + units - 1) / units + (ROUTE ? 1 : 0), ntasks ? ntasks : 1);
    if constexpr (!ROUTE) {
        if (nw == 1) hipLaunchKernelGGL((gemv_w4_kernel<MODE, 1, FULLG>), grid, dim3(64), 0, st, a, ks, ra);
        if (nw == 2) hipLaunchKernelGGL((gemv_w4_kernel<MODE, 2, FULLG>), grid, dim3(128), 0, st, a, ks, ra);
        if (nw <= 2) return hipGetLastError();
    }
    if (nw == 16) hipLaunchKernelGGL((gemv_w4_kernel<MODE, 16, FULLG, ROUTE>), grid, dim3(1024), 0, st, a, ks, ra);
    else if (nw == 8) hipLaunchKernelGGL((gemv_w4_kernel<MODE, 8, FULLG, ROUTE>), grid, dim3(512), 0, st, a, ks, ra);
    else hipLaunchKernelGGL((gemv_w4_kernel<MODE, 4, FULLG, ROUTE>), grid, dim3(256), 0, st, a, ks, ra);
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_gemv_t(const GemvArgs &a, uint32_t ks, uint32_t ntasks, hipStream_t st) {
    return (a.nsb % 8 == 0) ? launch_gemv_f<MODE, true>(a, ks, ntasks, RouteArgs{}, st) : launch_gemv_f<MODE, false>(a, ks, ntasks, RouteArgs{}, st);
}

// The K split is a pure performance choice (results do not depend on it): it grows until the
// launch has about four waves per SIMD or every wave is down to one scale group.
uint32_t gemv_ksplit(uint32_t ngroups, uint32_t total_units) {
    uint32_t ks = 1;
    while (ks < 16 && ks < ngroups && total_units * ks < 4096) ks *= 2;
    return ks;
}

hipError_t launch_gemv(int mode, uint32_t ksplit, const GemvArgs &a, uint32_t ntasks, const RouteArgs *route, hipStream_t st) {
    if (ksplit != 1 && ksplit != 2 && ksplit != 4 && ksplit != 8 && ksplit != 16) return hipErrorInvalidValue;
    // weights are addressed as a uniform base plus 32-bit byte offsets
    if ((uint64_t)a.nunits * (mode == GEMV_GATE_UP ? 2u : 1u) * a.tile_u4 * 16u > 0xFFFFFFFFull) return hipErrorInvalidValue;
    if (route) {
        if (mode != GEMV_RESID || ntasks || route->M != 1 || !route_rides(*route)) return hipErrorInvalidValue;
        return (a.nsb % 8 == 0) ? launch_gemv_f<GEMV_RESID, true, true>(a, ksplit, 0, *route, st) : launch_gemv_f<GEMV_RESID, false, true>(a, ksplit, 0, *route, st);
    }
    switch (mode) {
        case GEMV_PLAIN: return launch_gemv_t<GEMV_PLAIN>(a, ksplit, ntasks, st);
        case GEMV_RESID: return launch_gemv_t<GEMV_RESID>(a, ksplit, ntasks, st);
        case GEMV_GATE_UP: return launch_gemv_t<GEMV_GATE_UP>(a, ksplit, ntasks, st);
        case GEMV_F32: return launch_gemv_t<GEMV_F32>(a, ksplit, ntasks, st);
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------
// Two to kGemvMtTokens tokens: the decode kernel's structure -- units, K split over the waves of a
// unit, a whole scale group of weights requested at once, wave-private activation windows, no
// barrier before the last reduction -- with the dot products on the matrix cores.  A wave's lanes
// hold a row-tile's weights exactly as the GEMM's do (lane (i, c): block 4 sb + c of row i, dword kk
// the A operand of MFMA step kk, the scale folded in); the B operand of a step is one 16-byte chunk
// of a token's window, MFMA column j serving token j % kGemvMtTokens.  Against the one-token kernel
// the weight stream is the same and the vector ALU does a third more per weight (the exact
// (q - 8) d instead of the raw patterns), whatever the token count; against the MFMA GEMM at these
// token counts there are no partial planes, no plane-sum launches and no separate RMS-factor
// launch (four launches per layer instead of seven).  K must be a multiple of 1024.
// The windows are filled from global memory straight into LDS; chunk q of token t sits in slot
// q ^ t, so the 16 lanes x 4 lane groups of an operand read touch 16 different slots.
// A row's result is the sum of its scale-group partials in ascending group order, as in the
// one-token kernel: it depends neither on the K split nor on the workgroup shape.
// ------------------------------------------------------------------------------------
template <int MODE, int NW>
__global__ __launch_bounds__(NW * 64, 4) void gemv_mt_kernel(GemvArgs a, uint32_t ks, uint32_t ntok) {
    extern __shared__ uint4 mt_lds[];
    // a wave holds ONE row-tile's weights of a scale group at a time (two tiles' do not fit the registers beside
    // the operands): of a gate/up unit it takes the gate tile first and, super-block by super-block as the gate
    // tile's registers are used up, requests the up tile's into them, so one window serves both tiles
    constexpr int NT = (MODE == GEMV_GATE_UP) ? 2 : 1;
    constexpr int TK = kGemvMtTokens;
    constexpr bool NORM = (MODE == GEMV_PLAIN || MODE == GEMV_GATE_UP);
    static_assert(MODE != GEMV_F32, "dense sub-layers only");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, c = lane >> 4;
    const uint32_t wpu = ks;                    // waves per unit
    const uint32_t units = NW / wpu;
    const uint32_t unit = blockIdx.x * units + wave / wpu;
    const uint32_t kpart = wave % ks;
    const bool active = unit < a.nunits;
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
    uint4 *win = mt_lds + wave_u * (TK * 128);                                   // [token][128 chunks of 8]
    float *red = reinterpret_cast<float *>(mt_lds + NW * (TK * 128));            // [(unit, group)][tile][token][16 rows]
    float *red_ss = red + units * a.ngroups * (NT * TK * 16);                    // [(unit, group)][token]
    const uint32_t tb = j & (TK - 1);                                            // the token this lane's MFMA column serves
    const __amdgpu_buffer_rsrc_t xbuf = make_rsrc(a.x);

    if (active && kpart < a.ngroups) {
        for (uint32_t g = kpart; g < a.ngroups; g += ks) {
            // activations of the group for every token first (they are needed first), then the weights
            // slot r * 64 + lane of token t's window holds chunk (r * 64 + lane) ^ t: the same 128-column
            // stretch (one input head) for every t, so the column map is worked out once per r
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const uint32_t col0 = gather_col(g * 1024u + (uint32_t)(r * 64 + (lane & 48)) * 8u, a.x_off, a.x_group);
#pragma unroll
                for (int t = 0; t < TK; ++t) {
                    const uint32_t tokc = min((uint32_t)t, ntok - 1);   // windows past the last token repeat it (never stored)
                    const uint32_t voff = (tokc * a.x_stride + col0 + (((uint32_t)lane & 15u) ^ (uint32_t)t) * 8u) * (uint32_t)sizeof(__half);
                    load_to_lds16(xbuf, (lds_void *)(win + t * 128 + r * 64), voff, 0);
                }
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            GemvBuf<1> cur;
            gemv_issue_w<1, true>(cur, a.W, unit * NT, a.tile_u4, g, 8u, lane);
            const __amdgpu_buffer_rsrc_t wrs = make_rsrc(a.W);
            const uint32_t up_base = __builtin_amdgcn_readfirstlane((unit * NT + 1) * a.tile_u4 * 16u + g * (9u * 1024u));
            uint4 sc_up = make_uint4(0, 0, 0, 0);
            if (NT == 2) sc_up = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, (uint32_t)lane * 16u, up_base + 8u * 1024u, kAuxNt));
            // the window fills are the oldest loads in flight: all but the weight loads behind them
            // (the compiler does not know of loads into LDS; later loads only make this wait stricter)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 + (NT - 1)) : "memory");
            const uint32_t slot = (wave / wpu) * a.ngroups + g;
            if (NORM) {
#pragma unroll
                for (int t = 0; t < TK; ++t) {
                    const uint4 xa = win[t * 128 + lane], xb = win[t * 128 + 64 + lane];
                    float sq = 0.f;
                    sq = __builtin_amdgcn_fdot2(as_h2(xa.x), as_h2(xa.x), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xa.y), as_h2(xa.y), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xa.z), as_h2(xa.z), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xa.w), as_h2(xa.w), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xb.x), as_h2(xb.x), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xb.y), as_h2(xb.y), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xb.z), as_h2(xb.z), sq, false);
                    sq = __builtin_amdgcn_fdot2(as_h2(xb.w), as_h2(xb.w), sq, false);
                    const float gss = wave_sum(sq);
                    if (lane == 0) red_ss[slot * TK + t] = gss;
                }
            }
            const uint4 *wb = win + tb * 128;
#pragma unroll
            for (int tile = 0; tile < NT; ++tile) {
                const uint4 sc = tile == 0 ? cur.sc[0] : sc_up;
                f4_t gacc = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const uint4 wq = cur.wq[0][s];
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        const h8_t B = __builtin_bit_cast(h8_t, wb[(uint32_t)(s * 16 + c * 4 + kk) ^ tb]);
                        const uint32_t q = kk == 0 ? wq.x : kk == 1 ? wq.y : kk == 2 ? wq.z : wq.w;
                        const uint32_t dw = (s < 2) ? sc.x : (s < 4) ? sc.y : (s < 6) ? sc.z : sc.w;
                        const _Float16 d = __builtin_bit_cast(_Float16, (uint16_t)((s & 1) ? (dw >> 16) : (dw & 0xFFFFu)));
                        const h2_t dd = {d, d};
                        h2_t w[4];
                        dequant8(q, w);
                        w[0] *= dd; w[1] *= dd; w[2] *= dd; w[3] *= dd;
                        const h8_t A = h8_t{w[0].x, w[0].y, w[1].x, w[1].y, w[2].x, w[2].y, w[3].x, w[3].y};
                        gacc = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, B, gacc, 0, 0, 0);
                    }
                    // this super-block's registers are free: the next tile's super-block sets out into them
                    if (tile + 1 < NT)
                        cur.wq[0][s] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, (uint32_t)lane * 16u, up_base + (uint32_t)s * 1024u, kAuxNt));
                }
                // lane (j, c) holds rows 4c .. 4c + 3 of token column j
                if (j < TK)
                    *reinterpret_cast<float4 *>(red + ((slot * NT + tile) * TK + j) * 16 + c * 4) = make_float4(gacc[0], gacc[1], gacc[2], gacc[3]);
            }
            asm volatile("" ::: "memory");   // the window's reads are behind us before the next group's fills are issued
        }
    }
    __syncthreads();
    if (!(active && kpart == 0 && (uint32_t)j < ntok)) return;
    const uint32_t slot0 = (wave / wpu) * a.ngroups;
    float acc[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = 0.f;
    float ss = 0.f;
    for (uint32_t g = 0; g < a.ngroups; ++g) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 v = *reinterpret_cast<const float4 *>(red + (((slot0 + g) * NT + t) * TK + j) * 16 + c * 4);
            acc[t][0] += v.x; acc[t][1] += v.y; acc[t][2] += v.z; acc[t][3] += v.w;
        }
        if (NORM) ss += red_ss[(slot0 + g) * TK + j];
    }
    const float rinv = NORM ? rsqrtf(ss / (float)a.K + a.eps) : 1.f;
    const size_t o = (size_t)j * a.out_stride + a.out_row0 + unit * 16 + c * 4;
    float v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (MODE == GEMV_PLAIN) v[r] = rinv * acc[0][r];
        else if (MODE == GEMV_RESID) v[r] = (a.res ? __half2float(a.res[o + r]) : 0.f) + acc[0][r];
        else v[r] = silu(rinv * acc[0][r]) * (rinv * acc[NT - 1][r]);
    }
    __half2 *dst = reinterpret_cast<__half2 *>(a.out + o);
    dst[0] = __halves2half2(to_half(v[0]), to_half(v[1]));
    dst[1] = __halves2half2(to_half(v[2]), to_half(v[3]));
}

size_t gemv_mt_lds_bytes(uint32_t nw, uint32_t units, uint32_t ngroups, uint32_t nt) {
    return (size_t)nw * kGemvMtTokens * 2048 + (size_t)units * ngroups * (nt * kGemvMtTokens * 64 + kGemvMtTokens * 4);
}

template <int MODE>
static hipError_t launch_gemv_mt_t(const GemvArgs &a, uint32_t ks, uint32_t ntok, hipStream_t st) {   // ks by value: adjusted below
    constexpr uint32_t NT = (MODE == GEMV_GATE_UP) ? 2 : 1;
    // workgroup shapes as for one token (launch_gemv_f)
    const uint32_t wpu = ks;
    uint32_t nw = wpu > 8 ? 16 : wpu > 4 ? 8 : 4;
    if (wpu == 4 && (a.nunits + 1) / 2 >= 192) nw = 8;
    if (gemv_unit_per_cu(a.nunits, ks, 0)) nw = ks;
    const uint32_t units = nw / wpu;
    const size_t lds = gemv_mt_lds_bytes(nw, units, a.ngroups, NT);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    dim3 grid((a.nunits + units - 1) / units);
    static const hipError_t attr16 = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemv_mt_kernel<MODE, 16>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    static const hipError_t attr8 = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemv_mt_kernel<MODE, 8>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr16 != hipSuccess) return attr16;
    if (attr8 != hipSuccess) return attr8;
    if (nw == 16) hipLaunchKernelGGL((gemv_mt_kernel<MODE, 16>), grid, dim3(1024), lds, st, a, ks, ntok);
    else if (nw == 8) hipLaunchKernelGGL((gemv_mt_kernel<MODE, 8>), grid, dim3(512), lds, st, a, ks, ntok);
    else if (nw == 4) hipLaunchKernelGGL((gemv_mt_kernel<MODE, 4>), grid, dim3(256), lds, st, a, ks, ntok);
    else if (nw == 2) hipLaunchKernelGGL((gemv_mt_kernel<MODE, 2>), grid, dim3(128), lds, st, a, ks, ntok);
    else hipLaunchKernelGGL((gemv_mt_kernel<MODE, 1>), grid, dim3(64), lds, st, a, ks, ntok);
    return hipGetLastError();
}

hipError_t launch_gemv_mt(int mode, uint32_t ksplit, const GemvArgs &a, uint32_t ntok, hipStream_t st) {
    if (ksplit != 1 && ksplit != 2 && ksplit != 4 && ksplit != 8 && ksplit != 16) return hipErrorInvalidValue;
    if (ntok < 1 || ntok > (uint32_t)kGemvMtTokens || a.nsb % 8 != 0 || a.tasks) return hipErrorInvalidValue;
    // weights and activations are addressed as a uniform base plus 32-bit byte offsets
    if ((uint64_t)a.nunits * (mode == GEMV_GATE_UP ? 2u : 1u) * a.tile_u4 * 16u > 0xFFFFFFFFull) return hipErrorInvalidValue;
    if ((uint64_t)ntok * a.x_stride * 2u > 0xFFFFFFFFull) return hipErrorInvalidValue;
    switch (mode) {
        case GEMV_PLAIN: return launch_gemv_mt_t<GEMV_PLAIN>(a, ksplit, ntok, st);
        case GEMV_RESID: return launch_gemv_mt_t<GEMV_RESID>(a, ksplit, ntok, st);
        case GEMV_GATE_UP: return launch_gemv_mt_t<GEMV_GATE_UP>(a, ksplit, ntok, st);
    }
    return hipErrorInvalidValue;
}

template <int NR>
__global__ __launch_bounds__(256) void route_kernel(RouteArgs ra) { route_tokens<NR>(ra, blockIdx.x); }

hipError_t launch_route(const RouteArgs &ra, hipStream_t st) {
    const uint32_t E = ra.E, blocks = (ra.M + 3) / 4;
    if (E > 1024 || ra.top_k == 0 || ra.top_k > 64 || ra.top_k > E) return hipErrorInvalidValue;
    if (E <= 128) hipLaunchKernelGGL(route_kernel<2>, dim3(blocks), dim3(256), 0, st, ra);
    else if (E <= 256) hipLaunchKernelGGL(route_kernel<4>, dim3(blocks), dim3(256), 0, st, ra);
    else hipLaunchKernelGGL(route_kernel<16>, dim3(blocks), dim3(256), 0, st, ra);
    return hipGetLastError();
}

bool route_rides(const RouteArgs &ra) { return ra.M && ra.E <= 256 && ra.top_k && ra.top_k <= 64 && ra.top_k <= ra.E; }

// ------------------------------------------------------------------------------------
// rinv[m] = 1 / sqrt(mean(x[m]^2) + eps), one workgroup per token (used when M > 1): thread t adds
// the 8-column chunks t, t + 256, ... in that order, the 64 lanes of a wave are summed by the
// butterfly, the four waves in order.  All of a thread's loads (up to four per round) are issued
// before the first is used; chunks past the row's end count as zeros.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ float factor_of_quarters(const RowQuarters &r, uint32_t m) {
    const float p0 = r.sq[m], p1 = r.sq[r.M + m], p2 = r.sq[2 * r.M + m], p3 = r.sq[3 * r.M + m];
    return rsqrtf((((p0 + p1) + p2) + p3) / (float)r.H + r.eps);
}

// The factor of one row, in thread 0 .. 255 alike (part: four floats of LDS)
__device__ __forceinline__ float row_factor(const __half *x, uint32_t H, float eps, float *part) {
    const uint4 *row = reinterpret_cast<const uint4 *>(x);
    const uint32_t nq = H / 8;
    float ss = 0.f;
    for (uint32_t q0 = 0; q0 < nq; q0 += 1024) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // (a chunk past the row's end re-reads the last one and counts as zeros: no branch around the load,
            // so the four requests go out together)
            const uint32_t q = q0 + u * 256 + threadIdx.x;
            const uint4 w = row[min(q, nq - 1)];
            v[u] = q < nq ? w : uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) ss += sumsq8(v[u]);
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    return rsqrtf((((part[0] + part[1]) + part[2]) + part[3]) / (float)H + eps);
}

// one unit of an upload
__device__ __forceinline__ void upload_unit(const UploadArgs &up, uint32_t unit) {
    if (unit >= up.n16) return;
    const uint32_t idx = unit < up.first16 ? unit : unit + up.skip16;
    reinterpret_cast<u4_t *>(up.dst)[idx] = __builtin_nontemporal_load(reinterpret_cast<const u4_t *>(up.src) + idx);
}

// NR > 0: the workgroups behind the first M route four tokens each (the MoE routing of a layer depends on nothing the
// layer computes here, and as a launch of its own it costs 4 to 5 us).  NR < 0: they take an upload.
template <int NR>
__global__ __launch_bounds__(256) void rinv_kernel(const __half *x, uint32_t M, uint32_t H, float eps, float *rinv, RouteArgs ra, UploadArgs up) {
    if constexpr (NR > 0) {
        if (blockIdx.x >= M) { route_tokens<NR>(ra, blockIdx.x - M); return; }
    } else if constexpr (NR < 0) {
        if (blockIdx.x >= M) { upload_unit(up, (blockIdx.x - M) * 256 + threadIdx.x); return; }
    }
    __shared__ float part[4];
    const uint32_t m = blockIdx.x;
    const float f = row_factor(x + (size_t)m * H, H, eps, part);
    if (threadIdx.x == 0) rinv[m] = f;
}

// Where a row's sum of squares over a run of columns stands: four runs of a row side by side, so a reader of many rows takes four
// of each by one request of whole lines
__device__ __forceinline__ size_t ssq_at(uint32_t run, uint32_t tok, uint32_t ntok) { return ((size_t)(run >> 2) * ntok + tok) * 4 + (run & 3); }

// v of another lane of the row
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// up to 16 runs' sums of squares, in pairs (runs from n on count as zeros)
__device__ __forceinline__ float sum_of_runs(const float *v, uint32_t n) {
    auto four = [&](uint32_t k) {
        return ((n > k ? v[k] : 0.f) + (n > k + 1 ? v[k + 1] : 0.f)) + ((n > k + 2 ? v[k + 2] : 0.f) + (n > k + 3 ? v[k + 3] : 0.f));
    };
    return (four(0) + four(4)) + (four(8) + four(12));
}

// The same factor with the sum taken the way the GEMM's residual epilogue and the matrices behind it take it (ssq_out /
// ssq_in of GemmArgs), bit for bit: runs of 128 columns, in each the four 32-column shares of a wave, in each share the
// four lanes of a token (4 columns of either row-tile).  H a multiple of 128.
__global__ __launch_bounds__(256) void rinv_runs_kernel(const __half *x, uint32_t H, float eps, float *rinv) {
    __shared__ float share[kMaxGroups * 8 * 4];      // K <= 16384: 128 runs
    const uint32_t m = blockIdx.x, runs = H / 128, w = (threadIdx.x >> 2) & 3, rg = threadIdx.x & 3;
    const __half *row = x + (size_t)m * H;
    for (uint32_t run = threadIdx.x >> 4; run < runs; run += 16) {
        uint2 v[2];
        float part[2] = {0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) v[t] = *reinterpret_cast<const uint2 *>(row + run * 128 + w * 32 + t * 16 + rg * 4);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const h2_t a01 = as_h2(v[t].x), a23 = as_h2(v[t].y);
            part[t] = fmaf((float)a01.x, (float)a01.x, part[t]); part[t] = fmaf((float)a01.y, (float)a01.y, part[t]);
            part[t] = fmaf((float)a23.x, (float)a23.x, part[t]); part[t] = fmaf((float)a23.y, (float)a23.y, part[t]);
        }
        float sq = part[0] + part[1];
        sq += dpp_of<0xB1>(sq);   // quad_perm 1,0,3,2
        sq += dpp_of<0x4E>(sq);   // quad_perm 2,3,0,1
        if (rg == 0) share[run * 4 + w] = sq;
    }
    __syncthreads();
    float mine = 0.f;      // run threadIdx.x
    if (threadIdx.x < runs) {
        const float *r4 = share + threadIdx.x * 4;
        mine = (r4[0] + r4[1]) + (r4[2] + r4[3]);
    }
    __syncthreads();
    if (threadIdx.x < kMaxGroups * 8) share[threadIdx.x] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.;
        for (uint32_t g = 0; g < runs; g += 16) s += sum_of_runs(share + g, runs - g);
        rinv[m] = rsqrtf((float)s / (float)H + eps);
    }
}

hipError_t launch_rinv_runs(const __half *x, uint32_t M, uint32_t H, float eps, float *rinv, hipStream_t st) {
    if (H % 128 || H > kMaxGroups * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rinv_runs_kernel, dim3(M), dim3(256), 0, st, x, H, eps, rinv);
    return hipGetLastError();
}

hipError_t launch_rinv(const __half *x, uint32_t M, uint32_t H, float eps, float *rinv, const RouteArgs *route, const UploadArgs &up, hipStream_t st) {
    if (route && up.n16) return hipErrorInvalidValue;
    if (up.n16) hipLaunchKernelGGL(rinv_kernel<-1>, dim3(M + (up.n16 + 255) / 256), dim3(256), 0, st, x, M, H, eps, rinv, RouteArgs{}, up);
    else if (!route) hipLaunchKernelGGL(rinv_kernel<0>, dim3(M), dim3(256), 0, st, x, M, H, eps, rinv, RouteArgs{}, up);
    else if (!route_rides(*route)) return hipErrorInvalidValue;
    else if (route->E <= 128) hipLaunchKernelGGL(rinv_kernel<2>, dim3(M + (route->M + 3) / 4), dim3(256), 0, st, x, M, H, eps, rinv, *route, up);
    else hipLaunchKernelGGL(rinv_kernel<4>, dim3(M + (route->M + 3) / 4), dim3(256), 0, st, x, M, H, eps, rinv, *route, up);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Decode attention over a KV cache (one new token; softmax(q.K / sqrt(d)) V, no positional
// encoding).  HBM-bound on the cache bytes: a workgroup streams 256 positions of one kv head
// (64 KB of K, then 64 KB of V) once for all G query heads that share it.
// 16 lanes hold one position (8 dims each), so a wave load covers 4 whole rows (1 KB contiguous).
// Pass 1: scores of the chunk -> LDS; chunk maximum per query head.  Pass 2: p = exp(s - max),
// sum of p and p-weighted V sums.  Chunks are merged by attn_combine_kernel in chunk order, so the
// result does not depend on where the cache shard lives.
// ------------------------------------------------------------------------------------
constexpr int kAttnWaves = 8;             // waves per workgroup (measured at a 16K context: 4 -> 1.716, 8 -> 1.680, 16 -> 1.744 ms per token)
constexpr int kAttnIts = 8;               // steps of 4 positions per wave
constexpr int kAttnPos = kAttnWaves * kAttnIts * 4;   // positions per workgroup (a multiple of kAttnChunk, which sizes the partials)
static_assert(kAttnPos % kAttnChunk == 0, "the workspace is sized for one partial per kAttnChunk positions");
// A operand of O^T += V^T P^T for a 32-position tile of staged V rows and a tile of 16 dims: lane (i, c) needs dim i
// of the 8 positions 8 c .. 8 c + 7, i.e. a COLUMN of the staged rows.  The LDS transpose read of gfx950
// (ds_read_b64_tr_b16) does that within each group of 16 lanes: lane L of a group names 8 bytes (4 numbers), lane m
// receives number m % 4 of lanes m / 4, m / 4 + 4, m / 4 + 8, m / 4 + 12 (checked on the hardware with index numbers
// as data).  With lane L naming row L / 4, dims 4 (L % 4) .. + 3 of the tile, lane i receives dim i of four
// consecutive positions; two reads, four rows apart, make the operand.
__device__ __forceinline__ h8_t v_operand(const unsigned char *p) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((__vector_size__(4 * sizeof(__fp16)))) __fp16 fp16x4_t;
    typedef __attribute__((address_space(3))) fp16x4_t lds_fp16x4_t;
    const fp16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_fp16x4_t *)(p));
    const fp16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_fp16x4_t *)(p + 4 * 256));
    const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
    return __builtin_bit_cast(h8_t, make_uint4(a.x, a.y, b.x, b.y));
#else
    return h8_t{};
#endif
}

// sum over each row of 16 lanes, result in every lane of the row (DPP: no LDS traffic)
__device__ __forceinline__ float row16_sum(float v) {
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));  // row_half_mirror
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));  // row_mirror
    return v;
}

template <int G>
__global__ __launch_bounds__(kAttnWaves * 64, 16 / kAttnWaves) void attn_decode_kernel(AttnArgs a) {
    __shared__ float red[kAttnWaves][G][128];
    __shared__ float redm[kAttnWaves][G], redl[kAttnWaves][G];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int dl = lane & 15, pg = lane >> 4;
    const uint32_t chunk = blockIdx.x, hk = blockIdx.y;               // kv head within this launch
    const uint32_t ctx = a.ctx_dev ? *a.ctx_dev : a.ctx;              // the same for the whole grid
    if (chunk * kAttnPos >= ctx) return;                              // (launches sized for the whole cache)
    const __half *K = reinterpret_cast<const __half *>(reinterpret_cast<const char *>(a.kv) + (size_t)hk * a.head_stride);
    const __half *V = K + (size_t)a.cap * 128;
    const uint32_t q0 = (a.head0 + hk) * G;                           // first query head of this kv head
    const float scale = 0.08838834764831845f;                         // 1 / sqrt(128)

    // the queries first (loads return in order: issued last they would arrive last, and the scores
    // could not start before every cache row had arrived)
    uint4 qv[G];
#pragma unroll
    for (int h = 0; h < G; ++h) qv[h] = *reinterpret_cast<const uint4 *>(a.q + (size_t)(q0 + h) * 128 + dl * 8);
    // all of the wave's cache rows are requested up front (K chunks, then V chunks):
    // the V rows stream in while the scores are computed
    // Buffer loads bounded to the ctx valid rows: a row past the end reads as zeros, so the loads
    // need no branch (a branch per load would also make the compiler wait for each load at once)
    const uint32_t base = chunk * kAttnPos + wave * (kAttnPos / kAttnWaves);
    const __amdgpu_buffer_rsrc_t kb = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(K), 0, (int)(ctx * 256u), 0x00020000);
    const __amdgpu_buffer_rsrc_t vb = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(V), 0, (int)(ctx * 256u), 0x00020000);
    const uint32_t voff = (uint32_t)pg * 256u + (uint32_t)dl * 16u;
    const uint32_t soff = __builtin_amdgcn_readfirstlane(base * 256u);
    uint4 kq[kAttnIts], vq[kAttnIts];
#pragma unroll
    for (int it = 0; it < kAttnIts; ++it)
        kq[it] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kb, voff, soff + it * 1024, kAuxNt));
#pragma unroll
    for (int it = 0; it < kAttnIts; ++it)
        vq[it] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(vb, voff, soff + it * 1024, kAuxNt));
    // A wave works alone until the very end (no workgroup barrier between the passes): scores of its
    // positions stay in registers (the 16 lanes of a position meet through DPP row operations and
    // all hold the score), its own maximum, its own weights and sums.
    float sc[kAttnIts][G], mx[G];
#pragma unroll
    for (int h = 0; h < G; ++h) mx[h] = -INFINITY;
#pragma unroll
    for (int it = 0; it < kAttnIts; ++it) {
        const uint32_t j = base + it * 4 + pg;
#pragma unroll
        for (int h = 0; h < G; ++h) {
            float d = 0.f;
            d = __builtin_amdgcn_fdot2(as_h2(qv[h].x), as_h2(kq[it].x), d, false);
            d = __builtin_amdgcn_fdot2(as_h2(qv[h].y), as_h2(kq[it].y), d, false);
            d = __builtin_amdgcn_fdot2(as_h2(qv[h].z), as_h2(kq[it].z), d, false);
            d = __builtin_amdgcn_fdot2(as_h2(qv[h].w), as_h2(kq[it].w), d, false);
            const float r = row16_sum(d) * scale;      // outside any branch: every lane takes part
            sc[it][h] = j < ctx ? r : -INFINITY;
            mx[h] = fmaxf(mx[h], sc[it][h]);
        }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {   // the wave's 4 position groups
        mx[h] = fmaxf(mx[h], __shfl_xor(mx[h], 16, 64));
        mx[h] = fmaxf(mx[h], __shfl_xor(mx[h], 32, 64));
    }
    // a wave whose positions all lie past the end has maximum -inf: its weights must be 0, not NaN
    float l[G], o[G][8];
#pragma unroll
    for (int h = 0; h < G; ++h) {
        l[h] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[h][e] = 0.f;
    }
#pragma unroll
    for (int it = 0; it < kAttnIts; ++it) {
        float vf[8];
        const uint32_t vd[4] = {vq[it].x, vq[it].y, vq[it].z, vq[it].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const h2_t pr = as_h2(vd[e]);
            vf[2 * e] = (float)pr.x;
            vf[2 * e + 1] = (float)pr.y;
        }
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const float p = sc[it][h] == -INFINITY ? 0.f : __expf(sc[it][h] - mx[h]);
            l[h] += p;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[h][e] = fmaf(p, vf[e], o[h][e]);
        }
    }
    // the 4 position groups of a wave meet (36 independent values: LDS permutes, which pipeline, measured
    // faster here than the in-register row swaps the one-token GEMV uses for its one or two values);
    // then the workgroup's waves through LDS, rescaled to the chunk maximum, in fixed order
#pragma unroll
    for (int h = 0; h < G; ++h) {
        l[h] += __shfl_xor(l[h], 16, 64);
        l[h] += __shfl_xor(l[h], 32, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            o[h][e] += __shfl_xor(o[h][e], 16, 64);
            o[h][e] += __shfl_xor(o[h][e], 32, 64);
        }
        if (pg == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) red[wave][h][dl * 8 + e] = o[h][e];
            if (dl == 0) { redl[wave][h] = l[h]; redm[wave][h] = mx[h]; }
        }
    }
    __syncthreads();
    for (int t = tid; t < G * 128; t += kAttnWaves * 64) {
        const int h = t >> 7, d = t & 127;
        // wave 0's first position is always valid in a launched chunk, so the chunk maximum is finite
        float m = redm[0][h];
#pragma unroll
        for (int k = 1; k < kAttnWaves; ++k) m = fmaxf(m, redm[k][h]);
        float od = 0.f, ld = 0.f;   // waves in ascending order
#pragma unroll
        for (int k = 0; k < kAttnWaves; ++k) {
            const float w = redm[k][h] == -INFINITY ? 0.f : __expf(redm[k][h] - m);
            od = fmaf(w, red[k][h][d], od);
            ld = fmaf(w, redl[k][h], ld);
        }
        float *dst = a.part + ((size_t)(q0 + h) * a.chunk_cap + chunk) * 130;
        dst[2 + d] = od;
        if (d == 0) {
            dst[0] = m;
            dst[1] = ld;
        }
    }
}

// ------------------------------------------------------------------------------------
// Attention for a CHUNK of new tokens (chunked prefill over the cache), on the matrix cores.  Score rows are
// (token, query head of the kv group) pairs; a workgroup of eight waves holds 64 rows of one kv head and walks
// ROUNDS of kAttnRound = 128 positions: the cache's, then the chunk's own K / V rows read in place from the QKV
// rows (base and row stride differ, nothing else), up to the last position any of its rows sees.  Wave
// (r2, pg) works on rows 32 r2 .. + 31 and positions 32 pg .. + 31 of every round:
//  scores, transposed: S^T = K Q^T, A = 16 positions x 32 dims of K, B = 16 query rows (registers, loaded once):
//   the accumulator then holds, in lane (row j, c), four positions of row j;
//  weights x values, transposed: O^T = V^T P^T, with B = the weights exactly as the score accumulators hold them
//   (the two 16-position tiles are numbered so that lane group c owns 8 consecutive positions: 4 from each) and
//   A = 16 dims x 32 positions of V by LDS transpose reads (v_operand);
// with a running maximum, weight sum and O^T per row and wave, which the four position groups of a row merge in
// LDS at the end, in order.
// What bounds it, per round and CU (64 rows): 64 KB of rows from the L2 (1024 cycles at 64 bytes per clock),
// 128 KB of operand reads from LDS, 2 x 32 MFMAs per SIMD (1024), about 1100 cycles of softmax arithmetic
// per SIMD (a third of them the exponentials).  So: rows go from memory straight into LDS, two rounds' worth of stages,
// the next round on its way while one is multiplied (one barrier per round); two row tiles per wave share every operand
// read; two waves per SIMD.  What the scores cost is kept to the least: a tile of 16 rows is rescaled (32 multiplications)
// only in rounds in which one of its rows rises by more than 2^8 above the maximum its weights are relative to, a round's place in
// memory goes into the fills' scalar base, and the stage is a compile-time number.  Each row decides by its own scores (512 tokens 64.8
// -> 59 us, 64 tokens 15.3 -> 15.0, against a rescaling in every round that raises a maximum): a rule by which the rows of a wave wait for
// each other is no faster, and a row's fp16 weights, and so its bits, then depend on the rows beside it.  Rows of one (kv
// head, round) are read by all row blocks: the head is the fastest grid index, so with 8 heads a head's blocks share an XCD's L2.
// SPLIT: the rounds are dealt out to `nsplit` workgroups per row block (short chunks leave most CUs idle
// otherwise) and each writes, per row, a record (maximum, weight sum, 128 weighted sums) that
// attn_combine_chunk_kernel merges in split order; without SPLIT the finished rows are written.  The deal goes by
// context, the plan's token count and the whole model's heads, never by the launch's, so the result does not
// depend on where a cache shard lives.
// FEW: fewer than 16 score rows, i.e. one row tile of the two.  Its softmax weights keep fp32's precision, as the
// one-token kernel's do: a weight (times 2^15, which leaves the remainders room and drops out in o / l) goes into the value
// product as three fp16 numbers, its rounding and what is left of it twice.  The remainders' sums are kept apart and
// added at the end.  One wave of each pair has rows, so the MFMAs are fewer than with full tiles, and the time is
// the fills' and the latencies'.  2 tokens over 4000 positions 8.3 us with the weights in fp16, 8.3 with three parts;
// 3 tokens over 1000 7.9 / 7.9.
// Measured, 32 query / 8 kv heads over 4096 cached positions: 512 tokens 59 us, over 15000 170; 64 tokens over 4000 15.0 (the launch that
// appended the rows, 5 us, is part of it).  A round takes more than its largest part (row fills alone 45 us, the rest without
// them 49), and these did not change that: every operand requested in front of the next round's fills, the next round's scores
// worked out beside this one's weights (+4 us), steps of 64 positions with three on their way (+6, twice the LDS reads), and four
// waves of 64 rows each, one per SIMD, with rows of their own and no barrier (fills alone 27 us, the rest 56, both 83: a lone wave
// waits out every fill instruction's issue).
// ------------------------------------------------------------------------------------
constexpr uint32_t kAttnRound = 128;                           // positions per round
constexpr uint32_t kAttnHalfStage = kAttnRound * 256;           // K or V rows of a round; in LDS: K of two rounds, V of two rounds
constexpr uint32_t kAttnOPitch = 132;                          // floats per row when the position groups meet
constexpr size_t kAttnRowsLds = 4 * 64 * kAttnOPitch * 4 + 2 * 4 * 64 * 4;   // the meeting's rows, maxima and sums (more than two stages)
static_assert(4 * kAttnHalfStage <= 4 * 64 * kAttnOPitch * 4 && kAttnRowsLds <= 160 * 1024, "LDS of the chunk attention");

// 16-byte piece u of a staged row lies in slot u ^ swizzle of the row.  K rows: an operand read takes, per lane
// group, piece u of the 16 rows 8 (i / 4) + i % 4: their swizzles are the 16 numbers i.  V rows: a transpose read
// takes 32 bytes (pieces 2 dt, 2 dt + 1) of the rows 8 c + i / 4: even swizzles keep the pair together, eight
// different ones spread the rows over all banks.
__device__ __forceinline__ uint32_t k_swz(uint32_t row) { return (row & 3u) | (((row >> 3) & 3u) << 2); }
__device__ __forceinline__ uint32_t v_swz(uint32_t row) { return ((row & 3u) | (((row >> 3) & 1u) << 2)) << 1; }

// largest of three numbers, without the quieting steps fmaxf puts around values the compiler did not compute itself
__device__ __forceinline__ float max3(float a, float b, float c) {
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

template <bool SPLIT, bool FEW>
__global__ __launch_bounds__(512, 2) void attn_chunk_kernel(AttnChunkArgs a) {
    constexpr int NT = FEW ? 1 : 2;      // row tiles of a wave that hold rows
    extern __shared__ uint4 at_lds[];
    unsigned char *lds = reinterpret_cast<unsigned char *>(at_lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t i = lane & 15, c = lane >> 4;
    const uint32_t r2 = wave & 1, pg = wave >> 1;
    const uint32_t hk = blockIdx.x, G = a.group;
    const uint32_t kv_head = a.head0 + hk, q0 = kv_head * G;
    const uint32_t R = a.ntok * G, row0 = blockIdx.y * 64;
    if (row0 >= R) return;
    // rounds of this workgroup: cache rounds first, then the chunk's own up to its rows' last token
    const uint32_t nr_cache = (a.ctx + kAttnRound - 1) / kAttnRound;
    const uint32_t last_tok = min(a.ntok - 1, (row0 + 63) / G);
    const uint32_t nr = nr_cache + last_tok / kAttnRound + 1;
    const uint32_t rd0 = SPLIT ? blockIdx.z * a.rounds_per_split : 0u;
    const uint32_t rd1 = SPLIT ? min(nr, rd0 + a.rounds_per_split) : nr;

    const __half *kc = reinterpret_cast<const __half *>(reinterpret_cast<const char *>(a.k_base) + (size_t)hk * a.head_stride);
    const __half *vc = kc + (size_t)a.cap * 128;
    const __half *ko = a.k_own + (size_t)kv_head * 128, *vo = a.v_own + (size_t)kv_head * 128;
    // a round's rows straight into LDS: wave w moves rows 16 w .. + 15 of K and of V, four rows per instruction;
    // positions past the end lie past the buffer's range, whose check returns zeros (their weights are zero, and an
    // infinite value in a row read in their place would make NaN of that).  The round's place in memory goes into the
    // buffer's base (scalar), so a lane's offsets stay as they are from round to round.
    uint32_t lk[2], lv[2];      // lane offsets of the first two instructions' rows and of the other two's (swizzles differ)
    auto lanes_of = [&](uint32_t row_b) {
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) {
            const uint32_t row = wave * 16 + u * 8 + c;
            lk[u] = (wave * 16 + c) * row_b + ((i ^ k_swz(row)) << 4);
            lv[u] = (wave * 16 + c) * row_b + ((i ^ v_swz(row)) << 4);
        }
    };
    lanes_of(rd0 >= nr_cache ? a.own_stride * 2u : 256u);
    auto stage = [&](uint32_t rd, uint32_t buf) {
        const bool own = rd >= nr_cache;
        if (rd == nr_cache) lanes_of(a.own_stride * 2u);
        const uint32_t row_b = own ? a.own_stride * 2u : 256u, npos = own ? a.ntok : a.ctx;
        const uint32_t P0 = (own ? rd - nr_cache : rd) * kAttnRound;
        const int range = (int)((npos - P0 - 1) * row_b + 256u);
        const size_t at = (size_t)P0 * row_b;
        const __amdgpu_buffer_rsrc_t kb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(own ? ko : kc) + at), 0, range, 0x00020000);
        const __amdgpu_buffer_rsrc_t vb = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(own ? vo : vc) + at), 0, range, 0x00020000);
        unsigned char *dk = lds + buf * kAttnHalfStage + wave * (16 * 256), *dv = dk + 2 * kAttnHalfStage;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
            load_to_lds16(kb, (lds_void *)(dk + t * 1024), lk[t >> 1] + t * 4 * row_b, 0);
            load_to_lds16(vb, (lds_void *)(dv + t * 1024), lv[t >> 1] + t * 4 * row_b, 0);
        }
    };
    if (rd0 < rd1) stage(rd0, 0);
    if (!SPLIT && a.home) {
        // The chunk's K and V rows go to the cache's home, positions ctx and up, which no row block reads: every block moves
        // the tokens whose first row it holds (as a launch of its own 5 us a layer, here inside the wait for the first round)
        const uint32_t t0 = (row0 + G - 1) / G, t1 = min(a.ntok, (row0 + 64 + G - 1) / G);
        unsigned char *const kh = reinterpret_cast<unsigned char *>(a.home[kv_head]);
        for (uint32_t u = tid; u < (t1 - t0) * 32; u += 512) {
            const uint32_t t = t0 + u / 32, e = u & 15;
            const bool v = u & 16;
            const uint4 piece = *reinterpret_cast<const uint4 *>((v ? vo : ko) + (size_t)t * a.own_stride + e * 8);
            *reinterpret_cast<uint4 *>(kh + ((size_t)(v ? a.cap : 0u) + a.ctx + t) * 256 + e * 16) = piece;
        }
    }

    // the wave's 32 query rows (B operands of the score MFMAs)
    uint32_t tok[NT], hq[NT];
    h8_t q[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint32_t rho = min(row0 + r2 * 32 + t * 16 + i, R - 1);
        tok[t] = rho / G; hq[t] = rho % G;
        const __half *qr = a.q + (size_t)tok[t] * a.q_stride + (size_t)(q0 + hq[t]) * 128 + c * 8;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) q[t][kk] = __builtin_bit_cast(h8_t, *reinterpret_cast<const uint4 *>(qr + kk * 32));
    }
    // weights are 2^(c2 s - c2 m) of the raw scores s = q.k: 1 / sqrt(128) and log2(e) in one factor
    constexpr float c2 = 0.08838834764831845f * 1.4426950408889634f;
    constexpr float up = FEW ? 32768.f : 1.f;  // weights are held as `up` times what they are
    // how far a row's scores may rise above the maximum its weights are relative to: 2^8 in its weights, which fp16 holds as exactly
    // as those below 1 (few rows: not at all, their factor leaves no room)
    constexpr float slack = FEW ? 0.f : 8.f / c2;
    float m_run[NT], l_run[NT];                // l_run: this lane's positions only
#pragma unroll
    for (int t = 0; t < NT; ++t) { m_run[t] = -INFINITY; l_run[t] = 0.f; }
    f4_t O[2][8];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) O[t][dt] = f4_t{0.f, 0.f, 0.f, 0.f};
    // LDS byte offsets of this lane's operand pieces in a stage
    uint32_t koff[4], voff[8];
#pragma unroll
    for (uint32_t kk = 0; kk < 4; ++kk) koff[kk] = (32 * pg + 8 * (i >> 2) + (i & 3)) * 256 + (((4 * kk + c) ^ i) << 4);
    {
        const uint32_t vrow = 32 * pg + 8 * c + (i >> 2);
#pragma unroll
        for (uint32_t dt = 0; dt < 8; ++dt)
            voff[dt] = 2 * kAttnHalfStage + vrow * 256 + (((2 * dt + ((i & 3) >> 1)) ^ v_swz(vrow)) << 4) + (i & 1) * 8;
    }
    auto round = [&](uint32_t rd, auto BUF) {      // (the stage is a compile-time number: LDS addresses are lane offset + constant)
        constexpr uint32_t buf = decltype(BUF)::value;
        // this wave's rows of the round have landed; behind the barrier everyone's have, and everyone has left
        // the other stage
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (rd + 1 < rd1) stage(rd + 1, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        const bool own = rd >= nr_cache;
        const uint32_t P0 = (own ? rd - nr_cache : rd) * kAttnRound + 32 * pg;    // the wave's first position
        // (uniform) the wave's positions all lie past what its rows see
        const uint32_t last_seen = own ? min(a.ntok - 1, (row0 + r2 * 32 + 31) / G) : a.ctx - 1;
        if (P0 > last_seen || (FEW && r2)) return;
        const unsigned char *st = lds + buf * kAttnHalfStage;
        f4_t S[NT][2];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int T = 0; T < 2; ++T) S[t][T] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const h8_t kr = __builtin_bit_cast(h8_t, *reinterpret_cast<const uint4 *>(st + koff[kk] + T * 1024));
#pragma unroll
                for (int t = 0; t < NT; ++t) S[t][T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kr, q[t][kk], S[t][T], 0, 0, 0);
            }
        // positions a row does not see: only the cache's last round and the own rounds can hold any (the empty statement
        // keeps this a branch: as selects it would be 32 vector instructions in every round)
        if (own || P0 + 32 > a.ctx) {
            asm volatile("");
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t limit = own ? tok[t] + 1 : a.ctx;
#pragma unroll
                for (int T = 0; T < 2; ++T)
#pragma unroll
                    for (int r = 0; r < 4; ++r) S[t][T][r] = P0 + 8 * c + 4 * T + r < limit ? S[t][T][r] : -INFINITY;
            }
        }
        float mx[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            mx[t] = max3(max3(S[t][0][0], S[t][0][1], S[t][0][2]), max3(S[t][0][3], S[t][1][0], S[t][1][1]), max3(S[t][1][2], S[t][1][3], S[t][1][3]));
            mx[t] = rows4_meet<true>(mx[t]);
        }
        // A row whose weights would pass 2^8 is rescaled to its new maximum, the tile's others by 1: each row by its own scores
        // alone, so what it becomes does not depend on its neighbours.  A row that has seen nothing holds zeros, and the
        // difference of two -inf is not a number.
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bool raise = mx[t] > m_run[t] + slack;
            if (__any(raise)) {
                mx[t] = raise ? mx[t] : m_run[t];
                const float resc = m_run[t] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run[t] - mx[t]) * c2);
                m_run[t] = mx[t];
                l_run[t] *= resc;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) {
                    O[t][dt] = O[t][dt] * resc;
                    if (FEW) O[1][dt] = O[1][dt] * resc;
                }
            }
        }
        h8_t P[FEW ? 3 : 2];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float ms = m_run[t] == -INFINITY ? 0.f : m_run[t] * c2;
            float pv[8];
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pv[4 * T + r] = __builtin_amdgcn_exp2f(fmaf(S[t][T][r], c2, -ms)) * up;
                    l_run[t] += pv[4 * T + r];
                }
            P[t] = h8_t{(_Float16)pv[0], (_Float16)pv[1], (_Float16)pv[2], (_Float16)pv[3],
                        (_Float16)pv[4], (_Float16)pv[5], (_Float16)pv[6], (_Float16)pv[7]};
            if (FEW) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float rest = pv[e] - (float)P[0][e];
                    P[1][e] = (_Float16)rest;
                    P[FEW ? 2 : 1][e] = (_Float16)(rest - (float)P[1][e]);
                }
            }
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            const h8_t vr = v_operand(st + voff[dt]);
#pragma unroll
            for (int t = 0; t < 2; ++t) O[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vr, P[t], O[t][dt], 0, 0, 0);
            if (FEW) O[1][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vr, P[FEW ? 2 : 1], O[1][dt], 0, 0, 0);
        }
    };
    for (uint32_t rd = rd0; rd < rd1; rd += 2) {
        round(rd, std::integral_constant<uint32_t, 0>{});
        if (rd + 1 < rd1) round(rd + 1, std::integral_constant<uint32_t, 1>{});
    }
    // the four position groups of a row meet: every wave leaves its rows, maxima and sums in LDS
    __syncthreads();     // the last stage's reads are behind everyone
    float *ob = reinterpret_cast<float *>(lds), *om = ob + 4 * 64 * kAttnOPitch, *ol = om + 4 * 64;
    if (FEW) {   // (an infinite value makes the remainders' sum NaN, where the weights' own has the infinity)
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r) O[0][dt][r] = fabsf(O[0][dt][r]) < INFINITY ? O[0][dt][r] + O[1][dt][r] : O[0][dt][r];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float l = rows4_meet<false>(l_run[t]);
        const uint32_t row = r2 * 32 + t * 16 + i;
        float *dst = ob + (pg * 64 + row) * kAttnOPitch + 4 * c;   // lane (row i, group c) holds dims 16 dt + 4 c + r
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<float4 *>(dst + 16 * dt) = make_float4(O[t][dt][0], O[t][dt][1], O[t][dt][2], O[t][dt][3]);
        if (c == 0) { om[pg * 64 + row] = m_run[t]; ol[pg * 64 + row] = l; }
    }
    __syncthreads();
    const uint32_t row = tid >> 3, d0 = (tid & 7) * 16, rho = row0 + row;
    if (rho >= R) return;
    float m = om[row];
#pragma unroll
    for (int g = 1; g < 4; ++g) m = fmaxf(m, om[g * 64 + row]);
    float l = 0.f, o[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float mg = om[g * 64 + row], w = mg == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mg - m) * c2);
        const float4 *src = reinterpret_cast<const float4 *>(ob + (g * 64 + row) * kAttnOPitch + d0);
        l = fmaf(w, ol[g * 64 + row], l);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float4 v = src[e];
            o[4 * e] = fmaf(w, v.x, o[4 * e]); o[4 * e + 1] = fmaf(w, v.y, o[4 * e + 1]);
            o[4 * e + 2] = fmaf(w, v.z, o[4 * e + 2]); o[4 * e + 3] = fmaf(w, v.w, o[4 * e + 3]);
        }
    }
    const uint32_t t = rho / G, h = q0 + rho % G;
    if (SPLIT) {
        float *dst = a.part + (((size_t)t * a.n_q + h) * a.nsplit + blockIdx.z) * 130;
        if (d0 == 0) *reinterpret_cast<float2 *>(dst) = make_float2(m * 0.08838834764831845f, l);
#pragma unroll
        for (int e = 0; e < 8; ++e) reinterpret_cast<float2 *>(dst + 2 + d0)[e] = make_float2(o[2 * e], o[2 * e + 1]);
    } else {
        const float inv = 1.0f / l;      // every row sees at least its own token
        uint32_t d[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            d[e] = (uint32_t)__builtin_bit_cast(uint16_t, to_half(o[2 * e] * inv)) | ((uint32_t)__builtin_bit_cast(uint16_t, to_half(o[2 * e + 1] * inv)) << 16);
        uint4 *dst = reinterpret_cast<uint4 *>(a.out + (size_t)t * a.out_stride + (size_t)h * 128 + d0);
        dst[0] = uint4{d[0], d[1], d[2], d[3]};
        dst[1] = uint4{d[4], d[5], d[6], d[7]};
    }
}

// How the positions of a chunk's attention are dealt out: plans of kAttnOnePassTokens tokens and more fill the
// CUs with row blocks (and their workspace holds no records); below, as many splits as bring the launch to
// about one workgroup per CU, in whole rounds.  One split means finished rows and no merge.
void attn_chunk_deal(uint32_t ctx, uint32_t plan_tokens, uint32_t group, uint32_t n_kv, uint32_t *nsplit, uint32_t *rounds_per_split) {
    const uint32_t rounds = (ctx + kAttnRound - 1) / kAttnRound + (plan_tokens + kAttnRound - 1) / kAttnRound;
    const uint32_t blocks = (plan_tokens * group + 63) / 64 * n_kv;
    uint32_t per = rounds;
    if (plan_tokens < kAttnOnePassTokens) {
        const uint32_t want = std::max(1u, std::min(rounds, 256u / std::max(1u, blocks)));
        per = (rounds + want - 1) / want;
    }
    *rounds_per_split = per;
    *nsplit = (rounds + per - 1) / per;
}

template <bool SPLIT, bool FEW>
static hipError_t launch_attn_chunk_k(const AttnChunkArgs &a, dim3 grid, hipStream_t st) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_chunk_kernel<SPLIT, FEW>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAttnRowsLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((attn_chunk_kernel<SPLIT, FEW>), grid, dim3(512), kAttnRowsLds, st, a);
    return hipGetLastError();
}

hipError_t launch_attn_chunk(const AttnChunkArgs &a, hipStream_t st) {
    if (a.nheads == 0 || a.ntok == 0) return hipSuccess;
    if (a.group == 0 || a.group > 16 || !a.k_own || !a.v_own || a.nsplit == 0) return hipErrorInvalidValue;
    if (a.few && a.ntok * a.group >= 16) return hipErrorInvalidValue;
    const uint32_t rounds = (a.ctx + kAttnRound - 1) / kAttnRound + (a.ntok + kAttnRound - 1) / kAttnRound;
    if ((uint64_t)a.nsplit * a.rounds_per_split < rounds || (a.nsplit > 1 ? !a.part : !a.out)) return hipErrorInvalidValue;
    if (a.home ? (uint64_t)a.ctx + a.ntok > a.cap : a.ctx > a.cap) return hipErrorInvalidValue;
    // 32-bit buffer offsets
    if (((uint64_t)a.ctx + kAttnRound) * 256u > 0x7FFFFFFFull || ((uint64_t)a.ntok + kAttnRound) * a.own_stride * 2u > 0x7FFFFFFFull) return hipErrorInvalidValue;
    dim3 grid(a.nheads, (a.ntok * a.group + 63) / 64, a.nsplit);
    return a.few ? a.nsplit > 1 ? launch_attn_chunk_k<true, true>(a, grid, st) : launch_attn_chunk_k<false, true>(a, grid, st)
                 : a.nsplit > 1 ? launch_attn_chunk_k<true, false>(a, grid, st) : launch_attn_chunk_k<false, false>(a, grid, st);
}

// One workgroup of 128 threads per (query head, token): thread d merges dimension d over the token's records
// in split order (a record of a split the token sees nothing of has maximum -inf), writes the attention output
// row (the O projection's input) and, for the first query head of each kv group, appends the token's K and V
// rows at position ctx + t of that head's cache home.
__global__ __launch_bounds__(128) void attn_combine_chunk_kernel(const float *part, uint32_t nsplit, uint32_t ctx, uint32_t cap,
                                                                 const __half *qkv, uint32_t qkv_w, uint32_t n_q, uint32_t n_kv,
                                                                 const uint64_t *home, __half *out, uint32_t out_stride) {
    const uint32_t h = blockIdx.x, t = blockIdx.y, d = threadIdx.x;
    const uint32_t group = n_q / n_kv, g = h / group;
    const float *ph = part + ((size_t)t * n_q + h) * nsplit * 130;
    // eight records at a time, every load of a round requested before the first is used (a record past the last
    // re-reads the last one and is left out); one walk with a running maximum, the sums in split order
    float mx = -INFINITY, L = 0.f, o = 0.f;
    for (uint32_t c0 = 0; c0 < nsplit; c0 += 8) {
        float mv[8], lv[8], ov[8], m8 = mx;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const float *pc = ph + (size_t)min(c0 + u, nsplit - 1) * 130;
            mv[u] = pc[0]; lv[u] = pc[1]; ov[u] = pc[2 + d];
        }
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) m8 = fmaxf(m8, mv[u]);
        // (no branch on a record's maximum: the loads would sink into it one by one)
        const float ms = m8 == -INFINITY ? 0.f : m8, resc = __expf(mx - ms);
        L *= resc;
        o *= resc;
        mx = m8;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const float w = __expf(mv[u] - ms);
            L = c0 + u < nsplit ? fmaf(w, lv[u], L) : L;   // (left out, not weighed with zero: a sum may be infinite)
            o = c0 + u < nsplit ? fmaf(w, ov[u], o) : o;
        }
    }
    out[(size_t)t * out_stride + (size_t)h * 128 + d] = to_half(o / L);
    if (h % group == 0) {
        __half *Kh = reinterpret_cast<__half *>(home[g]);
        Kh[((size_t)ctx + t) * 128 + d] = qkv[(size_t)t * qkv_w + (size_t)(n_q + g) * 128 + d];
        Kh[((size_t)cap + ctx + t) * 128 + d] = qkv[(size_t)t * qkv_w + (size_t)(n_q + n_kv + g) * 128 + d];
    }
}

hipError_t launch_attn_combine_chunk(const float *part, uint32_t nsplit, uint32_t ctx, uint32_t cap, const __half *qkv,
                                     uint32_t qkv_w, uint32_t n_q, uint32_t n_kv, uint32_t ntok, const uint64_t *home, __half *out,
                                     uint32_t out_stride, hipStream_t st) {
    if (ntok == 0) return hipSuccess;
    if (n_kv == 0 || n_q % n_kv || nsplit == 0 || (uint64_t)ctx + ntok > cap || ntok > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_combine_chunk_kernel, dim3(n_q, ntok), dim3(128), 0, st, part, nsplit, ctx, cap, qkv, qkv_w, n_q, n_kv, home,
                       out, out_stride);
    return hipGetLastError();
}

__global__ void set_u32_kernel(uint32_t *dst, uint32_t v) { *dst = v; }

hipError_t launch_set_u32(uint32_t *dst, uint32_t v, hipStream_t st) {
    hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(1), 0, st, dst, v);
    return hipGetLastError();
}

hipError_t launch_attn_decode(const AttnArgs &a, hipStream_t st) {
    if ((!a.ctx_dev && a.ctx == 0) || a.nheads == 0) return hipSuccess;
    // context read on the device: cover every chunk a cache of cap positions can hold (ctx < cap)
    const uint32_t span = a.ctx_dev ? a.cap - 1 : a.ctx;
    if (span == 0) return hipSuccess;
    dim3 grid((span + kAttnPos - 1) / kAttnPos, a.nheads);
    if (grid.x > a.chunk_cap) return hipErrorInvalidValue;
    switch (a.group) {
        case 1: hipLaunchKernelGGL(attn_decode_kernel<1>, grid, dim3(kAttnWaves * 64), 0, st, a); break;
        case 2: hipLaunchKernelGGL(attn_decode_kernel<2>, grid, dim3(kAttnWaves * 64), 0, st, a); break;
        case 4: hipLaunchKernelGGL(attn_decode_kernel<4>, grid, dim3(kAttnWaves * 64), 0, st, a); break;
        case 8: hipLaunchKernelGGL(attn_decode_kernel<8>, grid, dim3(kAttnWaves * 64), 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// One workgroup of eight waves per query head.  Thread t takes the maximum and weight sum of chunks t, t + 512, ...;
// wave w sums chunks [w per, (w + 1) per) of the weighted values, two dimensions per lane, and the eight sums meet in
// order.  It is a chain of latencies, nothing else (1 MB of records at a 16K context): everything that does not depend
// on a reduction -- the token's rows, the first maxima and sums, the first eight records of every wave -- is
// requested at once and without a branch (a chunk past the end re-reads the last one and is left out), the token's own
// score is worked out by every wave for itself, and three barriers remain.  At 63 chunks 7.4 -> 4.7 us (the former
// version's last, shorter quarter of the chunks was read one record at a time).
constexpr uint32_t kAttnMaxChunks = 8192;   // 1M positions

__global__ __launch_bounds__(512) void attn_combine_kernel(const float *part, uint32_t chunk_cap, uint32_t ctx_arg,
                                                           const uint32_t *ctx_dev, uint32_t cap, const __half *qkv,
                                                           uint32_t n_q, uint32_t n_kv, const uint64_t *home, __half *out) {
    const uint32_t ctx = ctx_dev ? *ctx_dev : ctx_arg;
    __shared__ float wmax[8], wsum[8];
    __shared__ float wbuf[kAttnMaxChunks];
    __shared__ float osum[8][128];
    const uint32_t h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t group = n_q / n_kv, g = h / group;
    const uint32_t nchunks = (ctx + kAttnPos - 1) / kAttnPos, last = nchunks ? nchunks - 1 : 0;
    const float *ph = part + (size_t)h * chunk_cap * 130;
    const uint32_t per = (nchunks + 7) / 8, c0 = wave * per, c1 = min(nchunks, c0 + per);
    const __half2 kn = *reinterpret_cast<const __half2 *>(qkv + (size_t)(n_q + g) * 128 + 2 * lane);
    const __half2 qd = *reinterpret_cast<const __half2 *>(qkv + (size_t)h * 128 + 2 * lane);
    float m0 = -INFINITY, l0 = 0.f;
    float2 v0[8];
    if (nchunks) {   // (uniform; with an empty cache no record has been written)
        const float *pm = ph + (size_t)min(tid, last) * 130;
        m0 = tid < nchunks ? pm[0] : -INFINITY;
        l0 = pm[1];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v0[u] = *reinterpret_cast<const float2 *>(ph + (size_t)min(c0 + u, last) * 130 + 2 + 2 * lane);
    }
    const float2 kf = __half22float2(kn), qf = __half22float2(qd);
    const float s_self = wave_sum(fmaf(qf.x, kf.x, qf.y * kf.y)) * 0.08838834764831845f;
    float mloc = fmaxf(s_self, m0);
    for (uint32_t cc = tid + 512; cc < nchunks; cc += 512) mloc = fmaxf(mloc, ph[(size_t)cc * 130]);
    mloc = wave_max_all(mloc);
    if (lane == 0) wmax[wave] = mloc;
    __syncthreads();
    float mx = wmax[0];
#pragma unroll
    for (int w = 1; w < 8; ++w) mx = fmaxf(mx, wmax[w]);
    float lloc = 0.f;
    if (tid < nchunks) {
        const float w = __expf(m0 - mx);
        wbuf[tid] = w;
        lloc = w * l0;
    }
    for (uint32_t cc = tid + 512; cc < nchunks; cc += 512) {
        const float w = __expf(ph[(size_t)cc * 130] - mx);
        wbuf[cc] = w;
        lloc = fmaf(w, ph[(size_t)cc * 130 + 1], lloc);
    }
    lloc = wave_sum(lloc);
    if (lane == 0) wsum[wave] = lloc;
    __syncthreads();
    float2 o = make_float2(0.f, 0.f);
    if (c0 < c1) {
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const float w = wbuf[min(c0 + u, last)];
            o.x = c0 + u < c1 ? fmaf(w, v0[u].x, o.x) : o.x;
            o.y = c0 + u < c1 ? fmaf(w, v0[u].y, o.y) : o.y;
        }
        for (uint32_t c = c0 + 8; c < c1; c += 8) {
            float2 v[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float2 *>(ph + (size_t)min(c + u, last) * 130 + 2 + 2 * lane);
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                const float w = wbuf[min(c + u, last)];
                o.x = c + u < c1 ? fmaf(w, v[u].x, o.x) : o.x;
                o.y = c + u < c1 ? fmaf(w, v[u].y, o.y) : o.y;
            }
        }
    }
    *reinterpret_cast<float2 *>(&osum[wave][2 * lane]) = o;
    __syncthreads();
    if (tid >= 128) return;
    const uint32_t d = tid;
    const float w_self = __expf(s_self - mx);
    float L = 0.f, od = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) { L += wsum[w]; od += osum[w][d]; }
    L += w_self;
    od = fmaf(w_self, __half2float(qkv[(size_t)(n_q + n_kv + g) * 128 + d]), od);
    out[(size_t)h * 128 + d] = to_half(od / L);
    if (h % group == 0) {   // append the token's rows to the cache home of kv head g
        __half *Kh = reinterpret_cast<__half *>(home[g]);
        Kh[(size_t)ctx * 128 + d] = qkv[(size_t)(n_q + g) * 128 + d];
        Kh[((size_t)cap + ctx) * 128 + d] = qkv[(size_t)(n_q + n_kv + g) * 128 + d];
    }
}

hipError_t launch_attn_combine(const float *part, uint32_t chunk_cap, uint32_t ctx, const uint32_t *ctx_dev, uint32_t cap,
                               const __half *qkv, uint32_t n_q, uint32_t n_kv, const uint64_t *home, __half *out, hipStream_t st) {
    // (with the context on the device the caller has checked it against cap; the chunk bound then goes by cap)
    const uint32_t span = ctx_dev ? cap - 1 : ctx;
    if (ctx >= cap || n_kv == 0 || n_q % n_kv || (span + kAttnPos - 1) / kAttnPos > kAttnMaxChunks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_combine_kernel, dim3(n_q), dim3(512), 0, st, part, chunk_cap, ctx, ctx_dev, cap, qkv, n_q, n_kv, home, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// MoE combine: out[m] = h[m] + sum_j w[m][j] * y[m*top_k + j], j in rank order.  Eight columns per thread and round
// (16-byte reads; four experts' rows requested before the first is added, a rank past the last re-reads the last one
// and is left out).  RINV: one workgroup per token, whose threads own the same chunks as in rinv_kernel, square the
// fp16 values they store and reduce in the same order, so rinv[m] has the bits of the separate launch (4 us), which is
// then left out; otherwise the chunks of a token are spread over blockIdx.y.
// ------------------------------------------------------------------------------------
template <bool RINV>
__global__ __launch_bounds__(256) void combine_kernel(const __half *h, const float *y, const float *w, uint32_t H,
                                                      uint32_t top_k, int residual, __half *out, float eps, float *rinv) {
    const uint32_t m = blockIdx.x, nq = H / 8;
    float ss = 0.f;
    for (uint32_t q = blockIdx.y * blockDim.x + threadIdx.x; q < nq; q += gridDim.y * blockDim.x) {
        const uint4 hv = residual ? *reinterpret_cast<const uint4 *>(h + (size_t)m * H + q * 8) : uint4{0u, 0u, 0u, 0u};
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (uint32_t j0 = 0; j0 < top_k; j0 += 4) {
            float wv[4];
            float4 yv[4][2];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const size_t pr = (size_t)m * top_k + min(j0 + u, top_k - 1);
                wv[u] = w[pr];
                const float4 *src = reinterpret_cast<const float4 *>(y + pr * H + q * 8);
                yv[u][0] = src[0];
                yv[u][1] = src[1];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (j0 + u < top_k) {
                    s[0] += wv[u] * yv[u][0].x; s[1] += wv[u] * yv[u][0].y; s[2] += wv[u] * yv[u][0].z; s[3] += wv[u] * yv[u][0].w;
                    s[4] += wv[u] * yv[u][1].x; s[5] += wv[u] * yv[u][1].y; s[6] += wv[u] * yv[u][1].z; s[7] += wv[u] * yv[u][1].w;
                }
            }
        }
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint16_t lo = __builtin_bit_cast(uint16_t, to_half((residual ? half_of(hv, 2 * e) : 0.f) + s[2 * e]));
            const uint16_t hi = __builtin_bit_cast(uint16_t, to_half((residual ? half_of(hv, 2 * e + 1) : 0.f) + s[2 * e + 1]));
            d[e] = (uint32_t)lo | ((uint32_t)hi << 16);
        }
        const uint4 o = uint4{d[0], d[1], d[2], d[3]};
        *reinterpret_cast<uint4 *>(out + (size_t)m * H + q * 8) = o;
        if (RINV) ss += sumsq8(o);
    }
    if constexpr (RINV) {
        __shared__ float part[4];
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
        __syncthreads();
        if (threadIdx.x == 0) rinv[m] = rsqrtf((((part[0] + part[1]) + part[2]) + part[3]) / (float)H + eps);
    }
}

hipError_t launch_combine(const __half *h, const float *y, const float *w, uint32_t M, uint32_t H, uint32_t top_k,
                          int residual, __half *out, float eps, float *rinv, hipStream_t st) {
    if (M == 0) return hipSuccess;
    if (H % 8 || top_k == 0) return hipErrorInvalidValue;
    if (rinv) hipLaunchKernelGGL(combine_kernel<true>, dim3(M), dim3(256), 0, st, h, y, w, H, top_k, residual, out, eps, rinv);
    else hipLaunchKernelGGL(combine_kernel<false>, dim3(M, (H / 8 + 63) / 64), dim3(64), 0, st, h, y, w, H, top_k, residual, out, eps, rinv);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Prefill / batched-decode kernel: 4-bit dequant GEMM on the matrix cores.
// v_mfma_f32_16x16x32_f16: A = weights (16 rows x 32 k), B = activations (32 k x 16 tokens).
// A lane's 16 weight bytes are four A operands as they sit in memory: lane (i, c) holds
// block 4*sb + c of row i, dword kk supplies k-slots c*8 .. c*8+7 of MFMA step kk, which
// this kernel maps to k = 32*(4*sb + c) + 8*kk + t; the B operand follows the same map.
// Scales are folded into the fp16 A operand ((q - 8) * d rounded to fp16).
// NW waves (4, or 8 for the many-token shape), each wave owns AT row-tiles and all MT tokens of
// the workgroup; the activation tile of one super-block (MT x 128 k) is staged in LDS, 16-byte
// chunks XOR-swizzled by token so that operand reads are conflict-free.
// ------------------------------------------------------------------------------------
// LDS column of activation chunk u (k = 8u .. 8u+7 of a super-block) within its token's 16-chunk
// row, before the XOR with the token index: MFMA step kk of lane group c consumes chunk 4c + kk,
// kept at column c + 4kk so that the four lane groups of one read touch adjacent columns (measured:
// the 4c + kk order costs 1.5x the LDS cycles of this one)
__device__ __forceinline__ uint32_t lds_col(uint32_t u) { return ((u & 3) << 2) | (u >> 2); }

// super-blocks of lookahead of the GEMM's prefetch ring (see the kernel): 2 for the few-token tiles;
// the 8-wave workgroup (one per CU, its activation stages shared by twice the row-tiles) has the
// LDS for 3, at 160 tokens for 2
constexpr int gemm_depth(int MT, int NW = 4, int KS = 1) { return NW / KS == 8 ? (MT <= 128 ? 3 : MT <= 160 ? 2 : 1) : MT <= 64 ? 2 : 1; }
// LDS of a workgroup: the activation stages (of each K part), then per wave two scale buffers of 1 KB per row-tile
constexpr size_t gemm_lds_bytes(int MT, int AT, int NW, int KS = 1) {
    return (size_t)KS * MT * 256 * (gemm_depth(MT, NW, KS) + 1) + (size_t)NW * 2 * AT * 1024;
}

// RMS factor of row tok of a launch's input: from the buffer of factors, or from the row's sums of squares, 16 runs at a time.
// Every workgroup reads all runs of its tokens, so their number and the requests they take are what it costs.  One 8B-shaped layer, us
// a forward: 130 tokens of a 1024-token plan (32 runs) 146 with four or one run to a request, 151 with 64 half runs, one to a
// request; 512 tokens of a 512-token plan (64 runs) 241.5 with four, 243.5 with one.  Two such layers, 330 tokens of a 512-token plan 382.5 with
// halves, 380.4 with whole runs, 16 rows of a 64-token plan 118.5 and 117.2.  32 runs to a round trip gained nothing.
__device__ __forceinline__ float row_rinv(const GemmArgs &a, uint32_t tok, uint32_t ntok) {
    if (!a.ssq_in) return a.rinv[tok];
    if (a.quarters) return factor_of_quarters(RowQuarters{a.ssq_in, ntok, a.quarters, a.eps}, tok);
    double s = 0.;
    float whole = 0.f;                                // of up to 16 runs of 128 columns: runs of 64 take two turns
    for (uint32_t g = 0; g < a.ssq_runs; g += 16) {   // (the buffer goes on for 64 nsb floats per token)
        const float4 *sq = reinterpret_cast<const float4 *>(a.ssq_in) + (size_t)(g / 4) * ntok + tok;
        float v[16];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float4 q = sq[(size_t)e * ntok];
            v[4 * e] = q.x; v[4 * e + 1] = q.y; v[4 * e + 2] = q.z; v[4 * e + 3] = q.w;
        }
        whole += sum_of_runs(v, a.ssq_runs - g);
        if (a.ssq_runs == a.nsb || (g & 16)) { s += whole; whole = 0.f; }
    }
    s += whole;
    return rsqrtf((float)s / (float)(a.nsb * 128) + a.eps);
}

// Super-blocks of K slice w of eight: four to each half of K, as even as they go, the longer ones first
struct KSlice { uint32_t begin, end; };
__device__ __forceinline__ KSlice k_slice(uint32_t nsb, uint32_t w) {
    const uint32_t half = nsb / 2, base = half / 4, more = half % 4, q = w & 3;
    const uint32_t begin = (w >> 2) * half + q * base + min(q, more);
    return {begin, begin + base + (q < more ? 1u : 0u)};
}

// KS: K parts inside the workgroup.  With 2, waves 0 .. NW / 2 - 1 multiply the first half of the super-blocks and
// the others, on the same rows and tokens, the second half, each half with activation stages of its own; the
// second half's accumulators then pass through LDS and are added to the first's.  SLICED: each part adds its four
// slices of K up one by one, as gemm_kslice_kernel does.
template <int MODE, int AT, int MT, bool GROUPED, int NW, int KS, bool SLICED>
__device__ __forceinline__ void gemm_w4_body(const GemmArgs &a, uint4 *lds) {   // lds: KS x (gemm_depth + 1) stages of MT x 16 chunks, then 2 AT KB of scales per wave
    constexpr int NMT = MT / 16;
    constexpr int NWR = NW / KS;                   // waves of one K part: each owns AT row-tiles
    constexpr int NFILL = MT / (4 * NWR);          // 16-byte chunks each thread moves per stage
    static_assert(MT % (4 * NWR) == 0, "a fill round covers 4 * NWR tokens");
    static_assert(KS == 1 || (KS == 2 && !GROUPED && NW == 8), "two K parts: one workgroup of eight waves");
    const int kpart = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / (NWR * 64));
    const int tid = KS == 1 ? threadIdx.x : threadIdx.x % (NWR * 64), lane = tid & 63, wave = tid >> 6;   // within the K part
    const int i = lane & 15, c = lane >> 4;

    const uint4 *W = a.W;
    uint32_t ntok = a.M;           // tokens this workgroup column may touch
    const int32_t *pairs = nullptr;
    if (GROUPED) {
        const DeviceTask t = a.tasks[blockIdx.z];
        W = reinterpret_cast<const uint4 *>(MODE == GEMM_GATE_UP ? t.w_gate_up : t.w_down);
        ntok = t.npairs;
        pairs = a.pairs + t.pair0;
    }
    const uint32_t m0 = blockIdx.y * MT;
    if (m0 >= ntok) return;

    // activation fill, global memory straight into LDS (buffer_load ... lds): round r of a wave
    // writes 64 consecutive 16-byte slots, i.e. thread tid fills slot tid & 15 of token
    // tok0 + 4 NWR r, tok0 = tid >> 4, and therefore fetches the chunk that belongs there,
    // u = lds_col(slot ^ (tok0 & 15)) (lds_col is its own inverse).
    // xoff: byte offset of that chunk in the token's row (grouped launches look the row up);
    // tokens past the end re-read the last valid row: their MFMA columns are never stored, and the
    // fill needs neither a branch nor zeros.  Addresses are a uniform base plus these 32-bit
    // offsets, so the loop does no 64-bit vector arithmetic.
    const uint32_t tok0 = tid >> 4, u = lds_col((tid & 15) ^ (tok0 & 15));
    // (the many-token tiles work the offsets out again at every fill, from the first round's and the last row's: their
    // accumulators leave no registers for one offset per round)
    constexpr bool XCALC = !GROUPED && MT > 160;
    uint32_t xoff[XCALC ? 1 : NFILL];
    const uint32_t xstep = 4 * NWR * a.x_stride * (uint32_t)sizeof(__half);
    const uint32_t xlast = ((ntok - 1) * a.x_stride + u * 8) * (uint32_t)sizeof(__half);
#pragma unroll
    for (int r = 0; r < (XCALC ? 1 : NFILL); ++r) {
        const uint32_t tok = min(m0 + tok0 + r * (4 * NWR), ntok - 1);
        size_t rowi = tok;
        if (GROUPED) rowi = (MODE == GEMM_GATE_UP) ? (size_t)(pairs[tok] / (int32_t)a.top_k) : (size_t)pairs[tok];
        xoff[r] = (uint32_t)((rowi * a.x_stride + u * 8) * sizeof(__half));
    }
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
    // weights: 32-bit byte offset of the lane's 16 bytes in its tiles' first super-block; tiles past
    // the slab read tile 0 (discarded)
    // (gate/up tiles come in pairs, so one offset serves both, the second tile a scalar offset further on)
    constexpr bool PAIRED = MODE == GEMM_GATE_UP && AT == 2;
    uint32_t woff[PAIRED ? 1 : AT];
#pragma unroll
    for (int t = 0; t < (PAIRED ? 1 : AT); ++t) {
        const uint32_t tile = (blockIdx.x * NWR + wave_u) * AT + t;
        woff[t] = ((tile < a.ntiles ? tile : 0) * a.tile_u4 + lane) * 16u;
    }
    const uint32_t tile_b = PAIRED ? a.tile_u4 * 16u : 0u;
    // buffer addressing: uniform part of an address in a scalar offset, lane part in xoff / woff
    const __amdgpu_buffer_rsrc_t xbuf = make_rsrc(a.x), wbuf = make_rsrc(W);

    f4_t acc[AT][NMT];
#pragma unroll
    for (int t = 0; t < AT; ++t)
#pragma unroll
        for (int n = 0; n < NMT; ++n) acc[t][n] = f4_t{0.f, 0.f, 0.f, 0.f};

    // Prefetch ring: DEPTH super-blocks are in flight ahead of the one being multiplied, in R =
    // DEPTH + 1 weight register sets and LDS stages.  With few tokens an iteration is shorter than
    // the memory latency, so one super-block of lookahead leaves the loop waiting on its loads.
    constexpr int DEPTH = gemm_depth(MT, NW, KS), R = DEPTH + 1;
    static_assert(AT <= 2, "the dequantisation is pipelined one MFMA step ahead; more tiles per wave do not fit the registers");
    constexpr int LPI = NFILL + AT;              // loads every prefetch issues per lane (scale fills, when it has them: AT more)
    // one super-block of weights of the wave's tiles: the lane's 16 code bytes
    struct Wset { uint4 q[AT]; };
    Wset wr[R];
    // The fp16 scales come once per scale group (8 super-blocks), not once per super-block: a lane's
    // 16 bytes of a group's scale area hold the scales of its block column for all 8 super-blocks,
    // and they go from global memory straight into a wave-private LDS window (two buffers per tile,
    // by group parity), from where each step picks the two bytes it needs.  (One 4-byte load per
    // super-block instead touched the same eight cache lines eight times over, between which the
    // activation fills had pushed them out of the vector cache: a timing probe without scale loads
    // ran the 64-token gate/up launch 14 % faster.)  Like the activation fills these loads are not
    // register writes the compiler could wait for; the counted waits below cover them.
    uint4 *const xs_lds = lds + kpart * (R * MT * 16);      // this K part's activation stages
    uint4 *const sc_lds = lds + KS * (R * MT * 16) + (kpart * NWR + wave_u) * (2 * AT * 64);
    auto fill_x = [&](uint32_t sb, uint32_t stage) {
        // (wave-uniform; said so explicitly, or the fill's scalar offset is taken in a lane loop)
        const uint32_t xs = __builtin_amdgcn_readfirstlane(gather_col(sb * 128, a.x_off, a.x_group) * (uint32_t)sizeof(__half));
#pragma unroll
        for (int r = 0; r < NFILL; ++r)
            load_to_lds16(xbuf, (lds_void *)(xs_lds + stage * (MT * 16) + r * (NWR * 64) + wave_u * 64), XCALC ? min(xoff[0] + r * xstep, xlast) : xoff[XCALC ? 0 : r], xs);
    };

    // scale group / slot of super-block sb, clamped to the last one (a prefetch past the end
    // re-reads the last super-block instead of branching; nothing consumes it)
    auto load_w = [&](uint32_t sbn, Wset &w) {
        sbn = min(sbn, a.nsb - 1);
        const uint32_t gn = sbn >> 3, sn = sbn & 7;
        const uint32_t gb = gn * (9 * 1024);
#pragma unroll
        for (int t = 0; t < AT; ++t)
            w.q[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, woff[PAIRED ? 0 : t], gb + sn * 1024 + t * tile_b, kAuxNt));
    };
    // scale area of group g of the wave's tiles -> the window's buffer of parity g & 1
    auto fill_scales = [&](uint32_t g) {
        const uint32_t so = g * (9 * 1024) + min(8u, a.nsb - g * 8u) * 1024;
#pragma unroll
        for (int t = 0; t < AT; ++t) load_to_lds16(wbuf, (lds_void *)(sc_lds + ((g & 1) * AT + t) * 64), woff[PAIRED ? 0 : t], so + t * tile_b);
    };
    // the scales the next dequantisation uses (dsc): the lane's fp16 number sbx & 7 of its group
    uint32_t dsc[AT];
    auto scales_of = [&](uint32_t sbx) {
        const uint32_t g = sbx >> 3, sn = sbx & 7;
#pragma unroll
        for (int t = 0; t < AT; ++t)
            dsc[t] = *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(sc_lds + ((g & 1) * AT + t) * 64) + lane * 16 + sn * 2);
    };
    // prefetched weights become visible to the compiler only where this is called, so nothing
    // derived from them is scheduled (and waited for) earlier
    auto arrive_w = [&](Wset &w) {
#pragma unroll
        for (int t = 0; t < AT; ++t) {
            // (an empty statement the compiler cannot see through: no instruction is issued)
            asm volatile("" : "+v"(w.q[t].x), "+v"(w.q[t].y), "+v"(w.q[t].z), "+v"(w.q[t].w));
        }
    };
    // A operands of MFMA step kk from raw dwords + scale: (q - 8) * d rounded to fp16
    auto dequant_t = [&](const Wset &ws, int kk, int t) -> h8_t {
        const uint32_t q = kk == 0 ? ws.q[t].x : kk == 1 ? ws.q[t].y : kk == 2 ? ws.q[t].z : ws.q[t].w;
        const _Float16 d = __builtin_bit_cast(_Float16, (uint16_t)dsc[t]);
        const h2_t dd = {d, d};
        h2_t w[4];
        dequant8(q, w);
        w[0] *= dd; w[1] *= dd; w[2] *= dd; w[3] *= dd;
        return h8_t{w[0].x, w[0].y, w[1].x, w[1].y, w[2].x, w[2].y, w[3].x, w[3].y};
    };
    auto dequant_a = [&](h8_t (&A)[AT], const Wset &ws, int kk) {
#pragma unroll
        for (int t = 0; t < AT; ++t) A[t] = dequant_t(ws, kk, t);
    };

    // One prefetch = the stage's NFILL LDS fills, THEN the 2 AT weight loads, in that order in the
    // instruction stream: the hand-counted waits below rely on it (loads complete in issue order, so
    // "all but the newest n" is a statement about which loads have landed).  The fence keeps the
    // compiler from moving the weight loads, which depend on nothing, above fills whose addresses do
    // (in grouped launches the fill offsets come from a load of the pair list).
    // Scale fills come first of all.  A group's scales travel with the prefetch of the super-block
    // BEFORE the group (the dequantisation of a step's first operands runs at the end of the step
    // before, ahead of the wait that covers the step's own prefetch), and with the walk's opening
    // prefetch (FIRST) for the group it starts in.  The buffer they overwrite was last read nine
    // steps earlier.
    auto prefetch = [&](uint32_t sb_fill, uint32_t stage, uint32_t sb_w, Wset &w, auto FIRST) {
        const uint32_t sbc = min(sb_w, a.nsb - 1);
        if constexpr (decltype(FIRST)::value) fill_scales(sbc >> 3);
        if ((sbc & 7) == 7 && sbc + 1 < a.nsb) fill_scales((sbc >> 3) + 1);
        fill_x(sb_fill, stage);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_w(sb_w, w);
    };

    // split-K: this workgroup covers super-blocks [sb_begin, sb_end) and writes an fp32 partial plane
    uint32_t sb_begin = 0, sb_end = a.nsb;
    if (!GROUPED && a.sb_per_part) {
        sb_begin = blockIdx.z * a.sb_per_part;
        sb_end = min(a.nsb, sb_begin + a.sb_per_part);
    }
    if (KS == 2) {   // (an even number of super-blocks: both halves take the same number of steps and barriers)
        sb_begin = kpart * (a.nsb / 2);
        sb_end = sb_begin + a.nsb / 2;
    }
    f4_t total[SLICED ? AT : 1][SLICED ? NMT : 1];      // of the K part's slices that are done
    if constexpr (SLICED) {
#pragma unroll
        for (int t = 0; t < AT; ++t)
#pragma unroll
            for (int n = 0; n < NMT; ++n) total[t][n] = f4_t{0.f, 0.f, 0.f, 0.f};
    }
    uint32_t slice = kpart * 4, slice_end = SLICED ? k_slice(a.nsb, slice).end : 0;
    prefetch(sb_begin, 0, sb_begin, wr[0], std::true_type{});
#pragma unroll
    for (int d = 1; d < DEPTH; ++d) prefetch(min(sb_begin + d, sb_end - 1), d, sb_begin + d, wr[d], std::false_type{});
    // (A launch of its own for the factors is 4 to 6 us and two dependent-launch gaps for a pass over data the matrix in
    // front had in registers: two layers of 300 tokens at H = 4096 351 -> 339 us, two trips of 512 tokens 1222 -> 1203 us;
    // at 2048 tokens, where the matrix kernels run at the card's power limit, no difference.  All of a token's runs in one row,
    // 16 bytes of 64 rows to a request, cost the 256-token tiles 7 us a launch and were slower there than the launch they replace.)
    // the RMS factor of token m0 + thread, from the buffer of factors or from the token's sums of squares (one per 128
    // columns of K or per 64): requested behind the opening prefetches, whose wait covers it, or, where the accumulators leave
    // it no register, after the walk
    constexpr bool FACTORS = !GROUPED && (MODE == GEMM_PLAIN || MODE == GEMM_GATE_UP), FACTORS_LATE = MT > 224;
    static_assert(!FACTORS || MT <= NW * 64, "one token per thread");
    float my_rinv = 0.f;
    auto factor_of = [&](uint32_t t) { my_rinv = row_rinv(a, min(m0 + t, ntok - 1), ntok); };
    if constexpr (FACTORS && !FACTORS_LATE) {
        if (threadIdx.x < MT) factor_of(threadIdx.x);
    }
    // the A operands of the next MFMA step are dequantised while this step's MFMAs run
    h8_t Acur[AT], Anxt[AT];
    arrive_w(wr[0]);
    // EARLY (three or more super-blocks of lookahead): a stage is required one step before it is
    // multiplied, so the barrier that ends step sb already covers the fills of stage sb + 2.  A wave
    // can then fetch the first B operands of step sb + 1 while step sb's last MFMAs run, instead
    // of every wave of the workgroup meeting the LDS latency together right after the barrier.
    constexpr bool EARLY = DEPTH >= 3;
    constexpr int kLand = EARLY ? DEPTH - 2 : DEPTH - 1;   // prefetches that may still be in flight at a barrier
    // a prefetch issues its LDS fills before its weight loads and loads return in order, so the
    // barrier of the EARLY shape needs only the fills of the stage it covers: that stage's weight
    // loads (from HBM, the slow ones; consumed a step later) may stay in flight as well
    // (counted without the scale fills that one prefetch in eight carries: with one of those among
    // the newest the wait asks for a little more than it needs, never for less)
    constexpr int kInFlight = kLand * LPI + (EARLY ? AT : 0);
    // Before the first step: everything issued so far has landed.  No count is assumed here, because
    // nothing orders the DEPTH opening prefetches among themselves: the compiler hoists the weight
    // loads of all of them above fills that wait for the pair list, and merges the scale loads of two
    // super-blocks that share a dword, so "all but the newest kInFlight" would not name the fills of
    // stage 0 (a build in which it happened not to gave wrong results now and then).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    scales_of(sb_begin);
    dequant_a(Acur, wr[0], 0);
    // RING: tiles whose operands of a whole MFMA step do not fit the registers twice beside the accumulators
    constexpr bool RING = MT > 160;
    h8_t Bc[NMT], Bn[NMT];
    if (EARLY) {
#pragma unroll
        for (int n = 0; n < NMT; ++n) Bc[n] = __builtin_bit_cast(h8_t, xs_lds[i * 16 + n * 256 + (c ^ i)]);
    }

    // one super-block: U = its position in the ring (compile-time, so every register set and LDS
    // stage below is addressed statically and nothing is copied when the ring turns)
    // TAIL: one of the at most R - 1 steps after the last whole turn of the ring.  What they would
    // prefetch lies past the end of the walk, so they issue nothing and wait for everything.
    auto step = [&](uint32_t sb, auto U, auto TAIL) {
        constexpr int u = decltype(U)::value;
        constexpr bool tail = decltype(TAIL)::value;
        constexpr int un = (u + 1) % R, up = (u + DEPTH) % R;   // next super-block's slot, the slot to refill
        // prefetch super-block sb + DEPTH: activations into the stage every wave left at the
        // barrier that ended the previous step, weights into the register set used then
        if (!tail) prefetch(min(sb + DEPTH, sb_end - 1), up, sb + DEPTH, wr[up], std::false_type{});
        __builtin_amdgcn_sched_barrier(0);   // keep the prefetch up here: its latency hides behind the MFMAs
        const uint4 *ls = xs_lds + u * (MT * 16) + i * 16;   // + n * 256: token n*16 + i
        const uint4 *lsn = xs_lds + un * (MT * 16) + i * 16;  // the next super-block's stage
        if constexpr (RING) {
            // the step's 4 NMT B operands in order (kk, token tile), in blocks of two through a ring of six: a block is
            // read while the two before it are multiplied.  The A operands of kk + 1 are dequantised, one row-tile
            // per block, in the first blocks of kk.
            constexpr int NF = 4 * NMT, NR = 6;
            h8_t Bb[NR], Ab[2][AT];
            // (c + 4 kk) ^ i = (c ^ i) ^ 4 kk: the four addresses of a step are made from one where they are used
            uint32_t lane_at = (uint32_t)(i * 16 + (c ^ i)) * 16u;
            asm volatile("" : "+v"(lane_at));
            const char *const stage_at = reinterpret_cast<const char *>(xs_lds + u * (MT * 16));
            auto read_b = [&](int f) {
                Bb[f % NR] = __builtin_bit_cast(h8_t, *reinterpret_cast<const uint4 *>(stage_at + (f % NMT) * 4096 + (lane_at ^ (uint32_t)(f / NMT) * 64u)));
            };
#pragma unroll
            for (int t = 0; t < AT; ++t) Ab[0][t] = Acur[t];
#pragma unroll
            for (int f = 0; f < NR - 2; ++f) read_b(f);
#pragma unroll
            for (int f0 = 0; f0 < NF; f0 += 2) {
                if (f0 + NR - 2 < NF) { read_b(f0 + NR - 2); read_b(f0 + NR - 1); }
                __builtin_amdgcn_sched_barrier(0);
                const int kk = f0 / NMT, t = (f0 % NMT) / 2;     // NMT is even: a block lies in one MFMA step
                if (t < AT) {
                    if (kk < 3) Ab[(kk + 1) & 1][t] = dequant_t(wr[u], kk + 1, t);
                    else {
                        if (t == 0) { arrive_w(wr[un]); scales_of(sb + 1); }
                        Ab[(kk + 1) & 1][t] = dequant_t(wr[un], 0, t);
                    }
                }
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int t2 = 0; t2 < AT; ++t2)
                        acc[t2][f0 % NMT + e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ab[kk & 1][t2], Bb[(f0 + e) % NR], acc[t2][f0 % NMT + e], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < AT; ++t) Acur[t] = Ab[0][t];
        } else {
        // B operands are read one MFMA step ahead, so the LDS latency hides behind a step's MFMAs
        if (!EARLY) {
#pragma unroll
            for (int n = 0; n < NMT; ++n) Bc[n] = __builtin_bit_cast(h8_t, ls[n * 256 + (c ^ i)]);
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            if (kk < 3) {
#pragma unroll
                for (int n = 0; n < NMT; ++n) Bn[n] = __builtin_bit_cast(h8_t, ls[n * 256 + ((c + (kk + 1) * 4) ^ i)]);
                __builtin_amdgcn_sched_barrier(0);   // or the scheduler sinks each read next to its MFMA
            } else if (EARLY) {
#pragma unroll
                for (int n = 0; n < NMT; ++n) Bn[n] = __builtin_bit_cast(h8_t, lsn[n * 256 + (c ^ i)]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (kk < 3) dequant_a(Anxt, wr[u], kk + 1);
            else {
                arrive_w(wr[un]);
                scales_of(sb + 1);
                dequant_a(Anxt, wr[un], 0);
            }
#pragma unroll
            for (int n = 0; n < NMT; ++n) {
#pragma unroll
                for (int t = 0; t < AT; ++t)
                    acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Acur[t], Bc[n], acc[t][n], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < AT; ++t) Acur[t] = Anxt[t];
            if (kk < 3 || EARLY) {
#pragma unroll
                for (int n = 0; n < NMT; ++n) Bc[n] = Bn[n];
            }
        }
        }
        // super-block sb + 1's activations have landed once all but the later prefetches are done.
        // A bare barrier: __syncthreads() carries a fence that makes the compiler wait for EVERY
        // LDS-direct load in flight, i.e. also for the deeper prefetches.  What must be ordered
        // here is ordered by hand: this wave's fill of the next stage is complete (vmcnt), and
        // its LDS reads of the current stage, which the next step's fill overwrites, have
        // returned (lgkmcnt).
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(tail ? 0 : kInFlight) : "memory");
        __builtin_amdgcn_s_barrier();
        if constexpr (SLICED) {
            if (sb + 1 == slice_end && sb + 1 < sb_end) {
#pragma unroll
                for (int t = 0; t < AT; ++t)
#pragma unroll
                    for (int n = 0; n < NMT; ++n) {
                        total[t][n] += acc[t][n];
                        acc[t][n] = f4_t{0.f, 0.f, 0.f, 0.f};
                    }
                slice_end = k_slice(a.nsb, ++slice).end;
            }
        }
    };
    // whole turns of the ring, then the remaining steps (no exit from inside a turn: the ring is back
    // in phase at the loop's back edge, so no register set is live across it in another slot)
    uint32_t sb = sb_begin;
    for (; sb + R <= sb_end; sb += R) {
        step(sb, std::integral_constant<int, 0>{}, std::false_type{});
        step(sb + 1, std::integral_constant<int, 1>{}, std::false_type{});
        if constexpr (R > 2) step(sb + 2, std::integral_constant<int, 2>{}, std::false_type{});
        if constexpr (R > 3) step(sb + 3, std::integral_constant<int, 3>{}, std::false_type{});
    }
    if (sb < sb_end) step(sb, std::integral_constant<int, 0>{}, std::true_type{});
    if constexpr (R > 2) {
        if (sb + 1 < sb_end) step(sb + 1, std::integral_constant<int, 1>{}, std::true_type{});
    }
    if constexpr (R > 3) {
        if (sb + 2 < sb_end) step(sb + 2, std::integral_constant<int, 2>{}, std::true_type{});
    }

    if constexpr (SLICED) {
#pragma unroll
        for (int t = 0; t < AT; ++t)
#pragma unroll
            for (int n = 0; n < NMT; ++n) acc[t][n] = total[t][n] + acc[t][n];
    }
    // (the lane, the thread and the wave's tiles are taken from scratch: nothing of them need live through the ring)
    uint32_t elane = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(elane));   // (volatile: computed here, not before the ring)
#endif
    const uint32_t etid = ((uint32_t)kpart * NWR + wave_u) * 64 + elane;
    // The last step's barrier is behind every wave, so no stage is read any more.  But where the walk ends in a whole turn
    // of the ring, its last step has issued a fill past the walk's end, into stage R - 2, and passed the barrier with it
    // in flight (up to one prefetch with DEPTH > 1).  Without K parts that harms nothing: what is written below lies in
    // stage 0.  The exchange of two K parts covers stages 0 and 1, written by the waves of part 1 while the fill belongs
    // to a wave of part 0: every wave lets its own land, then all meet.  (Gate/up of 28672
    // rows, 64 tokens: K = 4096 24.6 us without and with the wait; K = 3072, whose halves end in a whole turn, 19.8 us
    // with it.)
    if constexpr (KS == 2 && DEPTH > 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    float *const side = reinterpret_cast<float *>(lds) + (KS == 2 ? NWR * AT * NMT * 256 : 0);   // RMS factors of the tile's tokens / sums of squares
    if constexpr (FACTORS) {
        if (etid < MT) {
            if (FACTORS_LATE) factor_of(etid);
            side[etid] = my_rinv;
        }
    }
    // Two K parts: each finishes half of the token tiles and hands the other half's sums over, so all eight waves add,
    // round and store; the residual rows are requested before the parts meet.  (The first part alone finished everything
    // before, with the residual loads in the middle of it: 4096 columns, 512 tokens, O 25.0 -> 23.9 us, down 64.1 -> 62.3; 300
    // tokens 22.0 -> 20.9, 58.6 -> 57.0.  The other modes, which read nothing there, gain nothing measurable.)
    constexpr int NF = KS == 2 ? (NMT + 1) / 2 : NMT;     // token tiles this wave finishes, from n0 on
    const uint32_t n0 = KS == 2 && kpart ? NF : 0;
    const int j = elane & 15, rg = elane >> 4;
    const uint32_t tile_base = (blockIdx.x * NWR + wave_u) * AT;
    f4_t fin[AT][NF];
    constexpr bool RES_EARLY = KS == 2 && MODE == GEMM_RESID;
    uint2 res[RES_EARLY ? AT : 1][RES_EARLY ? NF : 1];
    if constexpr (RES_EARLY) {
        if (a.res) {
#pragma unroll
            for (int k = 0; k < NF; ++k)
#pragma unroll
                for (int t = 0; t < AT; ++t) {
                    const uint32_t tok = min(m0 + (n0 + k) * 16 + j, ntok - 1), tile = min(tile_base + t, a.ntiles - 1);
                    res[t][k] = *reinterpret_cast<const uint2 *>(a.res + (size_t)tok * a.out_stride + a.out_row0 + tile * 16 + rg * 4);
                }
        } else {
#pragma unroll
            for (int k = 0; k < NF; ++k)
#pragma unroll
                for (int t = 0; t < AT; ++t) res[t][k] = uint2{0u, 0u};
        }
    }
    if constexpr (KS == 2) {   // first half + second half
        f4_t *const xch = reinterpret_cast<f4_t *>(lds) + (size_t)wave_u * (AT * NMT * 64) + elane;
        if (kpart == 1) {
#pragma unroll
            for (int t = 0; t < AT; ++t)
#pragma unroll
                for (int n = 0; n < NF; ++n) xch[(t * NMT + n) * 64] = acc[t][n];
        } else {
#pragma unroll
            for (int t = 0; t < AT; ++t)
#pragma unroll
                for (int n = NF; n < NMT; ++n) xch[(t * NMT + n) * 64] = acc[t][n];
        }
        __syncthreads();
        if (kpart == 0) {
#pragma unroll
            for (int t = 0; t < AT; ++t)
#pragma unroll
                for (int n = 0; n < NF; ++n) fin[t][n] = acc[t][n] + xch[(t * NMT + n) * 64];
        } else {
#pragma unroll
            for (int t = 0; t < AT; ++t)
#pragma unroll
                for (int n = NF; n < NMT; ++n) fin[t][n - NF] = xch[(t * NMT + n) * 64] + acc[t][n];
        }
    } else {
#pragma unroll
        for (int t = 0; t < AT; ++t)
#pragma unroll
            for (int n = 0; n < NF; ++n) fin[t][n] = acc[t][n];
        if constexpr (FACTORS) __syncthreads();
    }

    // epilogue: lane holds token j = lane & 15 of each token tile and rows 4*(lane >> 4) + r
    constexpr bool SSQ_OUT = !GROUPED && MODE == GEMM_RESID;
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        const uint32_t n = n0 + k;
        if (NF * KS != NMT && n >= NMT) continue;      // (an odd number of token tiles)
        const uint32_t tok = m0 + n * 16 + j;
        float sq[AT] = {};   // RESID: squares of what this lane stores for its token
        if (MT > 224) asm volatile("" ::: "memory");   // (or every token's factor is read ahead, and there are no registers for them)
        if (tok < ntok) {
        size_t orow = tok;           // output row
        size_t xrow = tok;           // row of rinv / residual
        if (pairs) { orow = (size_t)pairs[tok]; xrow = orow / a.top_k; }
        if (MODE == GEMM_GATE_UP) {
            const float rinv = FACTORS ? side[n * 16 + j] : a.rinv[xrow];
#pragma unroll
            for (int t = 0; t < AT; t += 2) {
                if (tile_base + t >= a.ntiles) continue;
                const uint32_t col = a.out_row0 + ((tile_base + t) >> 1) * 16 + rg * 4;
                __half2 o01 = __floats2half2_rn(silu(rinv * fin[t][k][0]) * (rinv * fin[t + 1][k][0]),
                                               silu(rinv * fin[t][k][1]) * (rinv * fin[t + 1][k][1]));
                __half2 o23 = __floats2half2_rn(silu(rinv * fin[t][k][2]) * (rinv * fin[t + 1][k][2]),
                                               silu(rinv * fin[t][k][3]) * (rinv * fin[t + 1][k][3]));
                __half2 *dst = reinterpret_cast<__half2 *>(a.out + orow * a.out_stride + col);
                dst[0] = o01; dst[1] = o23;
            }
        } else {
#pragma unroll
            for (int t = 0; t < AT; ++t) {
                if (tile_base + t >= a.ntiles) continue;
                const uint32_t col = a.out_row0 + (tile_base + t) * 16 + rg * 4;
                if (MODE == GEMM_F32) {
                    float *plane = a.out_f32 + ((!GROUPED && a.sb_per_part) ? (size_t)blockIdx.z * a.part_stride : 0);
                    float4 *dst = reinterpret_cast<float4 *>(plane + orow * a.out_stride + col);
                    *dst = make_float4(fin[t][k][0], fin[t][k][1], fin[t][k][2], fin[t][k][3]);
                } else {
                    float v[4];
                    if (MODE == GEMM_PLAIN) {
                        const float rinv = side[n * 16 + j];
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = rinv * fin[t][k][r];
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = fin[t][k][r];
                        if constexpr (RES_EARLY) {
                            if (a.res) {
                                const float2 r01 = __half22float2(__builtin_bit_cast(__half2, res[t][k].x)), r23 = __half22float2(__builtin_bit_cast(__half2, res[t][k].y));
                                v[0] += r01.x; v[1] += r01.y; v[2] += r23.x; v[3] += r23.y;
                            }
                        } else if (a.res) {
                            const __half2 *rs = reinterpret_cast<const __half2 *>(a.res + orow * a.out_stride + col);
                            const float2 r01 = __half22float2(rs[0]), r23 = __half22float2(rs[1]);
                            v[0] += r01.x; v[1] += r01.y; v[2] += r23.x; v[3] += r23.y;
                        }
                    }
                    __half2 *dst = reinterpret_cast<__half2 *>(a.out + orow * a.out_stride + col);
                    const __half2 h01 = __floats2half2_rn(v[0], v[1]), h23 = __floats2half2_rn(v[2], v[3]);
                    dst[0] = h01;
                    dst[1] = h23;
                    if (SSQ_OUT) {
                        const float2 f01 = __half22float2(h01), f23 = __half22float2(h23);
                        sq[t] = fmaf(f01.x, f01.x, sq[t]); sq[t] = fmaf(f01.y, f01.y, sq[t]);
                        sq[t] = fmaf(f23.x, f23.x, sq[t]); sq[t] = fmaf(f23.y, f23.y, sq[t]);
                    }
                }
            }
        }
        }
        if constexpr (SSQ_OUT) {
            if (a.ssq_out) {      // the token's four lanes meet: the wave's 32 columns
                const float own = rows4_meet<false>(sq[0] + sq[AT - 1]);
                if (rg == 0) side[wave_u * MT + n * 16 + j] = own;
            }
        }
    }
    if constexpr (SSQ_OUT) {
        if (a.ssq_out) {      // four waves make a run of 128 columns
            static_assert(AT == 2 && NWR % 4 == 0 && NWR / 4 * MT <= NW * 64, "runs of 128 columns, one sum per thread");
            __syncthreads();
            const uint32_t run = etid / MT, tk = etid % MT, wrun = blockIdx.x * (NWR / 4) + run;
            if (run < NWR / 4 && m0 + tk < ntok && wrun * 8 < a.ntiles) {
                const float *r4 = side + run * 4 * MT + tk;
                a.ssq_out[ssq_at(a.out_row0 / 128 + wrun, m0 + tk, ntok)] = (r4[0] + r4[MT]) + (r4[2 * MT] + r4[3 * MT]);
            }
        }
    }
}

// The next smaller tiles that an expert's workgroups may take (0: none)
constexpr int gemm_lesser(int MT) { return MT == 32 ? 16 : MT == 48 ? 32 : MT == 64 ? 48 : MT == 96 ? 64 : MT == 128 ? 96 : 0; }

// Grouped: the launch's tile holds the busiest expert's tokens; the workgroups of an expert with fewer take the smallest of it
// and the two tiles below that holds theirs, since every column of a tile costs its fills, operand reads and MFMAs
// whether a token stands behind it or not.  128 experts of 1536 + 2048 rows, us: 4 tokens each on average and 13 at most (32-token
// tiles for all before) gate/up 54 -> 41, down 35 -> 28; 32 on average and 47 at most 64 -> 62, 48 -> 43.5.
template <int MODE, int AT, int MT, bool GROUPED, int NW = 4, int KS = 1, bool SLICED = false>
__global__ __launch_bounds__(NW * 64, NW == 8 ? 1 : 2) void gemm_w4_kernel(GemmArgs a) {
    extern __shared__ uint4 lds[];
    if constexpr (GROUPED && gemm_lesser(MT)) {
        constexpr int less = gemm_lesser(MT), least = gemm_lesser(less);
        const uint32_t ntok = a.tasks[blockIdx.z].npairs;
        if constexpr (least) {
            if (ntok <= least) { gemm_w4_body<MODE, AT, least, GROUPED, NW, KS, SLICED>(a, lds); return; }
        }
        if (ntok <= less) { gemm_w4_body<MODE, AT, less, GROUPED, NW, KS, SLICED>(a, lds); return; }
    }
    gemm_w4_body<MODE, AT, MT, GROUPED, NW, KS, SLICED>(a, lds);
}

// Partial planes of up to 64 tokens with an upload behind the grid's columns: a kernel of its own, since the question whether
// there is an upload costs every launch that asks it 0.4 us (four steps of two 2048-wide layers, 6 tokens: 345 -> 354 us, 48: 404 -> 414).
template <int MT>
__global__ __launch_bounds__(256, 2) void gemm_w4_upload_kernel(GemmArgs a, UploadArgs up, uint32_t columns) {
    extern __shared__ uint4 lds[];
    if (blockIdx.x >= columns) {
        if (blockIdx.y == 0 && blockIdx.z == 0) upload_unit(up, (blockIdx.x - columns) * 256 + threadIdx.x);
        return;
    }
    gemm_w4_body<GEMM_F32, 2, MT, false, 4, 1, false>(a, lds);
}

// ------------------------------------------------------------------------------------
// GEMM of a narrow matrix with K in eight slices, one to a wave (O, down and small QKV of plans above 64 tokens, O of some
// plans of 49 to 64).
//
// Such a matrix has to be cut into small tiles to give every CU one, and what a small tile of gemm_w4_kernel pays for is
// not its MFMAs: 128 rows x 48 tokens dequantise every weight seven times for 300 tokens and read each operand from LDS for
// two products only.  Here a workgroup of eight waves has 64 rows and 16 NMT tokens, and each wave multiplies ALL of them over
// its own eighth of K: a weight is dequantised once per 80 tokens instead of 48, an operand read serves four
// products, and no wave ever waits for another before the sums meet at the end: a wave's activations go through a ring of
// LDS slots of its own (one slot: a token tile's super-block), filled a whole super-block ahead, and all waits are counts.
// What bounds it: the fills.  300 tokens x 14336: 80 tokens' activations, 2.3 MB, and 0.5 MB of weights a CU, of which loads alone take 47
// us, everything but the loads 40, together 52.  Some 8 us of a round are its own (launch, first loads, the exchange), so the
// loads run at about 72 KB a microsecond and CU, where L2 to LDS alone reaches 68 to 100 by the shape of the requests; and two
// rounds lose to the two-K-part tiles.  4096 columns, us, against those, plans of as many tokens: O (K = 4096) 72 tokens 15.4 ->
// 11.3, 128: 15.8 -> 11.8, 192: 16.4 -> 13.5, 256: 17.4 -> 15.4, 300: 20.0 -> 19.1; down (K = 14336) 42.5 -> 28.0, 43 -> 29.5,
// 44.6 -> 38.0, 47.5 -> 43.9, 53.3 -> 51.6; 2048 columns, 200 tokens: O 9.9 -> 7.5, down (K = 5632) 19.4 -> 13.8, 512: 10.8 -> 10.1, 21.0 -> 20.2.
// Tried without gain: 128 rows with the slices in pairs on waves that share their fills (512 tokens 66 -> 75 us).
// ------------------------------------------------------------------------------------
constexpr int kSliceRows = 4;     // row-tiles of a workgroup
constexpr int kSliceWaves = 8;    // K slices
constexpr size_t kslice_ring_bytes(int NMT) { return (size_t)kSliceWaves * NMT * 4096; }
constexpr size_t kslice_sum_floats(int NMT) { return (size_t)kSliceWaves * kSliceRows * (NMT < 4 ? NMT : 4) * 256; }
constexpr size_t kslice_sum_bytes(int NMT) { return (kslice_sum_floats(NMT) + NMT * 2 * 16) * sizeof(float); }
constexpr size_t kslice_lds_bytes(int NMT) { return kslice_ring_bytes(NMT) > kslice_sum_bytes(NMT) ? kslice_ring_bytes(NMT) : kslice_sum_bytes(NMT); }

template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// A lane's four sums of a row-tile (columns tile * 16 + rg * 4 ..) for token tok, with the mode's epilogue; RESID: sq gets
// the sum of squares of what is stored
template <int MODE>
__device__ __forceinline__ void finish_rows(const GemmArgs &a, f4_t v, uint32_t tok, uint32_t tile, uint32_t rg, float rinv, uint2 res, float &sq) {
    if (tok >= a.M || tile >= a.ntiles) return;
    if (MODE == GEMM_PLAIN) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] *= rinv;
    } else if (a.res) {
        const float2 r01 = __half22float2(__builtin_bit_cast(__half2, res.x)), r23 = __half22float2(__builtin_bit_cast(__half2, res.y));
        v[0] += r01.x; v[1] += r01.y; v[2] += r23.x; v[3] += r23.y;
    }
    __half2 *dst = reinterpret_cast<__half2 *>(a.out + (size_t)tok * a.out_stride + a.out_row0 + tile * 16 + rg * 4);
    const __half2 h01 = __floats2half2_rn(v[0], v[1]), h23 = __floats2half2_rn(v[2], v[3]);
    dst[0] = h01;
    dst[1] = h23;
    if (MODE == GEMM_RESID) {
        const float2 f01 = __half22float2(h01), f23 = __half22float2(h23);
        sq = fmaf(f01.x, f01.x, sq); sq = fmaf(f01.y, f01.y, sq);
        sq = fmaf(f23.x, f23.x, sq); sq = fmaf(f23.y, f23.y, sq);
    }
}

template <int MODE, int NMT>
__device__ __forceinline__ void kslice_finish(const GemmArgs &a, const f4_t (&acc)[kSliceRows][NMT], uint4 *lds) {
    constexpr int RT = kSliceRows;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), m0 = blockIdx.y * (NMT * 16), M = a.M;
    // The slices meet, four token tiles at a time: every wave's sums go into LDS, then a wave adds up the eight of two
    // row-tiles of one token tile, a half of K after the other and each in order.  What is added to the rows is requested first.
    const uint32_t j = lane & 15, rg = lane >> 4, pair = wave >> 2, who = wave & 3;
    constexpr int NU = (NMT + 3) / 4;      // token tiles a wave finishes: who, who + 4, ..
    uint2 res[NU][2];
    if constexpr (MODE == GEMM_RESID) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t tok = min(m0 + (who + u * 4) * 16 + j, M - 1);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t tile = min(blockIdx.x * RT + pair * 2 + e, a.ntiles - 1);
                res[u][e] = a.res ? *reinterpret_cast<const uint2 *>(a.res + (size_t)tok * a.out_stride + a.out_row0 + tile * 16 + rg * 4) : uint2{0u, 0u};
            }
        }
    }
    float *const side = reinterpret_cast<float *>(lds) + kslice_sum_floats(NMT);
    f4_t *const sums = reinterpret_cast<f4_t *>(lds) + lane;      // [wave][token tile of the four][row-tile][lane]
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        constexpr int NB = NMT < 4 ? NMT : 4;
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            if (u * 4 + n >= NMT) break;
#pragma unroll
            for (int t = 0; t < RT; ++t) sums[((wave * NB + n) * RT + t) * 64] = acc[t][u * 4 + n];
        }
        if constexpr (MODE == GEMM_PLAIN) {
            if (u == 0 && threadIdx.x < NMT * 16) side[threadIdx.x] = row_rinv(a, min(m0 + threadIdx.x, M - 1), M);
        }
        __syncthreads();
        const uint32_t n = who + u * 4, tok = m0 + n * 16 + j;
        if (n >= NMT) continue;
        float sq[2] = {0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t tile = blockIdx.x * RT + pair * 2 + e;
            f4_t half[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f4_t *const s4 = sums + ((h * 4 * NB + who) * RT + pair * 2 + e) * 64;
                half[h] = ((s4[0] + s4[NB * RT * 64]) + s4[2 * NB * RT * 64]) + s4[3 * NB * RT * 64];
            }
            finish_rows<MODE>(a, half[0] + half[1], tok, tile, rg, MODE == GEMM_PLAIN ? side[n * 16 + j] : 0.f, res[u][e], sq[e]);
        }
        if (MODE == GEMM_RESID && a.ssq_out) {
            const float own = rows4_meet<false>(sq[0] + sq[1]);
            if (rg == 0) side[(n * 2 + pair) * 16 + j] = own;
        }
    }
    if (MODE == GEMM_RESID && a.ssq_out) {       // the workgroup's 64 columns are a run
        __syncthreads();
        const uint32_t n = threadIdx.x >> 4, jj = threadIdx.x & 15, tok = m0 + threadIdx.x;
        if (threadIdx.x < NMT * 16 && tok < M && blockIdx.x * RT < a.ntiles)
            a.ssq_out[ssq_at(a.out_row0 / 64 + blockIdx.x, tok, M)] = side[n * 32 + jj] + side[n * 32 + 16 + jj];
    }
}

template <int MODE, int NMT>
__global__ __launch_bounds__(kSliceWaves * 64, 1) void gemm_kslice_kernel(GemmArgs a) {
    extern __shared__ uint4 lds[];
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int RT = kSliceRows;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t i = lane & 15, c = lane >> 4;
    const uint32_t m0 = blockIdx.y * (NMT * 16);
    const KSlice slice = k_slice(a.nsb, wave);
    const uint32_t sb0 = slice.begin, nsb = slice.end - slice.begin;      // (at least two super-blocks: gemm_k_slices)

    f4_t acc[RT][NMT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int n = 0; n < NMT; ++n) acc[t][n] = f4_t{0.f, 0.f, 0.f, 0.f};

    const uint32_t row_b = a.x_stride * (uint32_t)sizeof(__half);
    const __amdgpu_buffer_rsrc_t wbuf = make_rsrc(a.W);
    // round r of a fill covers tokens 4 r .. 4 r + 3 of the tile: lane l puts chunk u0 ^ r of token 4 r + (l >> 4) into
    // column l & 15 of that token's row (the layout of gemm_w4_kernel's stages)
    const uint32_t u0 = lds_col((lane & 15) ^ (lane >> 4));
    uint32_t xoff[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) xoff[r] = (r * 4 + (lane >> 4)) * row_b + (u0 ^ r) * 16u;
    unsigned char *const ring = reinterpret_cast<unsigned char *>(lds) + wave * (NMT * 4096);
    uint32_t wbase[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const uint32_t tile = blockIdx.x * RT + t;
        wbase[t] = (tile < a.ntiles ? tile : 0) * a.tile_u4 * 16u;      // (tiles past the slab read tile 0: discarded)
    }
    // The workgroup's rows from super-block sb of the slice (clamped to the last) on, as a buffer that ends with the last row that is
    // there: a fill's rows past it are out of its range, i.e. zeros (never stored) and no access.  What names the row is a lane
    // offset, since a scalar offset takes no part in the range check.
    const char *const rows = reinterpret_cast<const char *>(a.x) + (size_t)m0 * row_b;
    const uint32_t rows_b = (a.M - m0) * row_b;
    auto columns = [&](uint32_t sb) {
        const uint32_t col = __builtin_amdgcn_readfirstlane(gather_col((sb0 + min(sb, nsb - 1)) * 128, a.x_off, a.x_group) * (uint32_t)sizeof(__half));
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(rows + col), 0, (int)(rows_b - col), 0x00020000);
    };
    auto fill = [&](__amdgpu_buffer_rsrc_t cols, int n) {
#pragma unroll
        for (int r = 0; r < 4; ++r) load_to_lds16(cols, (lds_void *)(ring + n * 4096 + r * 1024), xoff[r] + n * 16 * row_b, 0);
    };
    uint4 wq[RT], sc[RT];      // a super-block's codes; a scale group's scales
    auto load_w = [&](uint32_t sb) {
        const uint32_t sa = sb0 + sb, o = (sa >> 3) * (9 * 1024) + (sa & 7) * 1024;
#pragma unroll
        for (int t = 0; t < RT; ++t) wq[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, lane * 16, wbase[t] + o, kAuxNt));
    };
    auto load_sc = [&](uint32_t sb) {
        const uint32_t g = (sb0 + sb) >> 3, o = g * (9 * 1024) + min(8u, a.nsb - g * 8u) * 1024;
#pragma unroll
        for (int t = 0; t < RT; ++t) sc[t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wbuf, lane * 16, wbase[t] + o, kAuxNt));
    };
    // prefetched weights and scales become visible to the compiler only here: nothing derived from them is made (and waited for) earlier
    auto arrive = [&]() {
#pragma unroll
        for (int t = 0; t < RT; ++t)
            asm volatile("" : "+v"(wq[t].x), "+v"(wq[t].y), "+v"(wq[t].z), "+v"(wq[t].w), "+v"(sc[t].x), "+v"(sc[t].y), "+v"(sc[t].z), "+v"(sc[t].w));
    };
    h8_t A[4][RT];
    h2_t dd[RT];
    auto scales = [&](uint32_t sb) {
        const uint32_t sn = (sb0 + sb) & 7, sel = sn & 1 ? 0x03020302u : 0x01000100u;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const uint32_t lo = sn & 2 ? sc[t].y : sc[t].x, hi = sn & 2 ? sc[t].w : sc[t].z;
            dd[t] = as_h2(__builtin_amdgcn_perm(0, sn & 4 ? hi : lo, sel));
        }
    };
    auto dequant = [&](int kk) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const uint32_t q = kk == 0 ? wq[t].x : kk == 1 ? wq[t].y : kk == 2 ? wq[t].z : wq[t].w;
            h2_t w[4];
            dequant8(q, w);
            w[0] *= dd[t]; w[1] *= dd[t]; w[2] *= dd[t]; w[3] *= dd[t];
            A[kk][t] = h8_t{w[0].x, w[0].y, w[1].x, w[1].y, w[2].x, w[2].y, w[3].x, w[3].y};
        }
    };
    const uint32_t lane_at = (i * 16 + (c ^ i)) * 16u;
    h8_t Bc[4], Bn[4];
    auto read_b = [&](h8_t (&B)[4], int n) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) B[kk] = __builtin_bit_cast(h8_t, *reinterpret_cast<const uint4 *>(ring + n * 4096 + (lane_at ^ (kk * 64u))));
    };
    // One super-block, token tile by token tile.  REM: super-blocks behind it in the slice, 2 meaning two or more.
    auto step = [&](uint32_t sb, auto REM) {
        constexpr int rem = decltype(REM)::value;
        const __amdgpu_buffer_rsrc_t next = columns(sb + 1);
        auto tile = [&](auto N) {
            constexpr int n = decltype(N)::value;
            constexpr bool turn = n == NMT - 1;
            // the tile's operands have arrived in registers: its slot takes the next super-block's
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if constexpr (rem >= 1) fill(next, n);
            __builtin_amdgcn_sched_barrier(0);
            // Issued behind the next tile's fill: the fills of the other slots and, where that fill is of this super-block, the
            // weights of the next (loads return in order; scales on their way make the wait a little stricter)
            if constexpr (!turn) {
                wait_vm<(rem >= 1 ? (NMT - 1) * 4 + RT : (NMT - 2 - n) * 4)>();
                read_b(Bn, n + 1);
            } else if constexpr (rem >= 1) {
                wait_vm<(NMT - 1) * 4>();
                read_b(Bn, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // the next super-block's A operands are made beside the last tile's products, whose operands they replace
            if constexpr (turn && rem >= 1) { arrive(); scales(sb + 1); }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
                for (int t = 0; t < RT; ++t) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[kk][t], Bc[kk], acc[t][n], 0, 0, 0);
                if constexpr (turn && rem >= 1) dequant(kk);
            }
            if constexpr (turn && rem == 2) {
                __builtin_amdgcn_sched_barrier(0);
                if (((sb0 + sb + 2) & 7) == 0) load_sc(sb + 2);
                load_w(sb + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) Bc[kk] = Bn[kk];
        };
        tile(std::integral_constant<int, 0>{});
        tile(std::integral_constant<int, 1>{});
        if constexpr (NMT > 2) tile(std::integral_constant<int, 2>{});
        if constexpr (NMT > 3) tile(std::integral_constant<int, 3>{});
        if constexpr (NMT > 4) tile(std::integral_constant<int, 4>{});
        static_assert(NMT >= 2 && NMT <= 5, "token tiles of a workgroup");
    };
    load_sc(0);
    load_w(0);
    __builtin_amdgcn_sched_barrier(0);
    const __amdgpu_buffer_rsrc_t first = columns(0);
#pragma unroll
    for (int n = 0; n < NMT; ++n) fill(first, n);
    arrive();
    scales(0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) dequant(kk);
    __builtin_amdgcn_sched_barrier(0);
    if (((sb0 + 1) & 7) == 0) load_sc(1);
    load_w(1);
    wait_vm<0>();
    read_b(Bc, 0);
    uint32_t sb = 0;
    for (; sb + 2 < nsb; ++sb) step(sb, std::integral_constant<int, 2>{});
    step(sb, std::integral_constant<int, 1>{});
    step(sb + 1, std::integral_constant<int, 0>{});
    kslice_finish<MODE, NMT>(a, acc, lds);
#endif
}

template <int MODE, int NMT>
static hipError_t launch_gemm_kslice(const GemmArgs &a, hipStream_t st) {
    void (*const kernel)(GemmArgs) = gemm_kslice_kernel<MODE, NMT>;
    constexpr size_t ldsb = kslice_lds_bytes(NMT);
    static_assert(ldsb <= 160 * 1024, "LDS of a CU");
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)ldsb);
    if (attr != hipSuccess) return attr;
    const dim3 grid((a.ntiles + kSliceRows - 1) / kSliceRows, (a.M + NMT * 16 - 1) / (NMT * 16));
    hipLaunchKernelGGL(kernel, grid, dim3(kSliceWaves * 64), ldsb, st, a);
    return hipGetLastError();
}

template <int MODE, int AT, int MT, bool GROUPED, int NW, int KS, bool SLICED = false>
static hipError_t launch_gemm_k(const GemmArgs &a, uint32_t ntok, uint32_t gz, hipStream_t st) {
    constexpr size_t ldsb = gemm_lds_bytes(MT, AT, NW, KS);
    static_assert(ldsb <= 160 * 1024, "LDS of a CU");
    if (ldsb > 64 * 1024) {
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_w4_kernel<MODE, AT, MT, GROUPED, NW, KS, SLICED>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)ldsb);
        if (attr != hipSuccess) return attr;
    }
    constexpr uint32_t rows = NW / KS * AT;   // row-tiles of a workgroup
    dim3 grid((a.ntiles + rows - 1) / rows, (ntok + MT - 1) / MT, gz);
    hipLaunchKernelGGL((gemm_w4_kernel<MODE, AT, MT, GROUPED, NW, KS, SLICED>), grid, dim3(NW * 64), ldsb, st, a);
    return hipGetLastError();
}

// Two K parts inside the workgroup: for matrices whose 128-row workgroups at the plan's token count leave at most one
// per CU in tiles of up to 128 tokens.  Four waves of them are one wave per SIMD, which waits for its own operand reads
// and dequantisation; the second half of K on four more waves halves the steps.  Against the best shape without the
// parts: 128 tokens: QKV 25.6 -> 17.7 us, O 25.7 -> 17.1, down 73.6 -> 45.5; 512: QKV 39.2 -> 36.3, O 28.8 -> 25.5, down
// 85.8 -> 71.9; 1024: O 43.6 -> 40.9, down 139 -> 120, but QKV, 1.5 workgroups per CU, 61.7 -> 74.9.
static bool gemm_two_k_parts(const GemmArgs &a, uint32_t plan_tokens) {
    return a.nsb % 2 == 0 && (a.total_tiles + 7) / 8 * ((plan_tokens + 127) / 128) <= 256;
}

// Token tile of an unsplit launch of a.M rows: the one with the smallest product of rounds of workgroups (one
// eight-wave workgroup of 256 rows per CU, two four-wave ones of 128) and time per round.  A round costs a fixed
// part (a barrier, the first operand reads and the fills of every step) plus a part per token, so a large tile is
// cheap per token and few, full rounds matter most.  Measured on 4096-wide rows, us per round: 8 waves x 96 tokens 43,
// 128: 54, 160: 62, 192: 69, 224: 78, 256: 89; 4 waves x 64 tokens 26 alone on a CU, 43 with two.
// Gate/up, 28672 rows, launched alone, against the former 128-token tile: 300 tokens 111 -> 74 us (160), 512: 122 -> 105
// (256), 1024: 242 -> 209 (256), 1536: 380 -> 318 (256).  At 2048 tokens the rule says 256, by a hair over 192, and in the
// pass of a two-layer prefill, at the clock that holds under its load, the tiles are all alike: 256 438-446 us, 192
// 435-443, 160 434-444, 224 (a worse last round) 474; another time 256 466 on average and 441 at the least, the former tile
// 472-490 and 447.  QKV, 6144 rows, in that pass: 224 102-109, 160 135, 192 157, the former tile 115-120; O and down stay
// with 128: 69 and 207, 160 74 and 224, 192 86 and 267.
static uint32_t gemm_pick_tile(const GemmArgs &a, uint32_t widest) {
    const uint32_t g4 = (a.ntiles + 7) / 8, g8 = (a.ntiles + 15) / 16;
    uint32_t best = 0, best_cost = 0xFFFFFFFFu;
    for (uint32_t mt : {16u, 32u, 64u}) {
        if (mt < 64 && a.M > mt) continue;
        const uint32_t wg = g4 * ((a.M + mt - 1) / mt), one = mt == 64 ? 260 : mt == 32 ? 200 : 180, rest = wg % 512;
        const uint32_t cost = wg / 512 * (one * 5 / 3) + (rest == 0 ? 0 : rest <= 256 ? one : one * 5 / 3);
        if (cost < best_cost) { best_cost = cost; best = mt; }
    }
    for (uint32_t mt = 96; mt <= widest; mt += 32) {
        const uint32_t wg = g8 * ((a.M + mt - 1) / mt);
        const uint32_t cost = (wg + 255) / 256 * (185 + mt * 27 / 10);   // tenths of a microsecond
        if (cost < best_cost) { best_cost = cost; best = mt; }
    }
    return best;
}

// K in eight slices: for matrices of at least 16 super-blocks whose plan goes in one round of 64-token tiles of 128 rows.  Which of the
// kernels walks them goes by the rows that are there: gemm_kslice_kernel where its 64-row tiles of up to 80 tokens
// go in one round (a second round costs it more than it gains: 512 tokens of 4096 columns, O 24 -> 31 us, down 66 -> 87), else the two K
// parts, which then keep the slices' sums apart (SLICED) so that a row's bits do not depend on its company.  That costs them up to
// 1 us a launch (512 tokens: O 23.6 -> 24.3, down 67.8 -> 68.4; three additions of the accumulators and their zeroes, which no MFMA covers), against 4
// and 14 us gained at 128 tokens; plans that need larger tiles stay with plain K parts.  QKV of 6144 rows, 72 tokens: 15.9 -> 13.0 us, 128:
// 16.5 -> 15.7; 192 to 320, in two K parts, 0.8 slower.  Two layers, us a forward, against plain K parts in all plans: 4096 wide, plan of
// 512, 70 tokens 253 -> 217, 130: 266 -> 246, 200: 293 -> 290, 300: 340 -> 339, 384: 385 -> 390, 512: 474 -> 476; 2048 wide, plan of 512, 70: 127 ->
// 107, 200: 139 -> 123, 400: 156 -> 156, 512: 166 -> 166, plan of 1024, 500: 165 -> 164, 700: 197 -> 201, 1024: 245 -> 247.  So the rule gives
// up to 2 % of the long trips of such a plan for up to 15 % of its short ones.
static bool gemm_k_slices(uint32_t nsb, uint32_t total_tiles, uint32_t plan_tokens) {
    return plan_tokens > 64 && nsb % 2 == 0 && nsb >= 16 && (total_tiles + 7) / 8 * ((plan_tokens + 63) / 64) <= 256;
}
// (by the whole matrix, so that all its slabs leave the same sums of squares)
static bool gemm_slice_tiles(uint32_t total_tiles, uint32_t M) { return (total_tiles + kSliceRows - 1) / kSliceRows * ((M + 79) / 80) <= 256; }
bool gemm_leaves_halves(uint32_t nsb, uint32_t total_tiles, uint32_t plan_tokens, uint32_t M) {
    return gemm_k_slices(nsb, total_tiles, plan_tokens) && gemm_slice_tiles(total_tiles, M);
}

template <int MODE>
static hipError_t launch_gemm_m(const GemmArgs &a, uint32_t ntasks, uint32_t max_tok, hipStream_t st) {
    if (ntasks) {
        // grouped: one expert per blockIdx.z; the smallest tile that holds the busiest expert's tokens (128 experts of 1536 +
        // 2048 rows, 4 tokens each on average: gate/up 41 us with every expert in 16-token tiles, 45 in 32, 52 in 48, 65 in 64,
        // 83 in 96, 95 in 128; the kernel lets the others take smaller ones), since a second tile for a few busy experts
        // costs 14 to 16 us for the workgroups that find nothing to do (24 tokens on average, 40 at most: 32-token tiles 63 us,
        // 48-token tiles 56).  512 tokens through a layer, 48- instead of 64-token tiles: gate/up 69 -> 57 us, down 45 -> 40.
        if constexpr (MODE == GEMM_GATE_UP || MODE == GEMM_F32) {
            if (max_tok <= 16) return launch_gemm_k<MODE, 2, 16, true, 4, 1>(a, max_tok, ntasks, st);
            if (max_tok <= 32) return launch_gemm_k<MODE, 2, 32, true, 4, 1>(a, max_tok, ntasks, st);
            if (max_tok <= 48) return launch_gemm_k<MODE, 2, 48, true, 4, 1>(a, max_tok, ntasks, st);
            if (max_tok <= 64) return launch_gemm_k<MODE, 2, 64, true, 4, 1>(a, max_tok, ntasks, st);
            if (max_tok <= 96) return launch_gemm_k<MODE, 2, 96, true, 4, 1>(a, max_tok, ntasks, st);
            return launch_gemm_k<MODE, 2, 128, true, 4, 1>(a, max_tok, ntasks, st);
        }
        return hipErrorInvalidValue;   // experts: gate/up and the fp32 rows of down
    }
    const uint32_t parts = a.sb_per_part ? (a.nsb + a.sb_per_part - 1) / a.sb_per_part : 1;
    if constexpr (MODE == GEMM_RESID) {
        if (max_tok <= 64 && a.slices) {
            if (a.nsb % 2 || a.nsb < 16 || (a.ntiles + kSliceRows - 1) / kSliceRows * ((a.M + 31) / 32) > 256) return hipErrorInvalidValue;
            return launch_gemm_kslice<MODE, 2>(a, st);
        }
    }
    if (max_tok <= 64) {
        // batched decode: the smallest tile that holds the rows that are there (the tile never changes a bit of the
        // result).  A matrix that goes in one part has its two halves of K on eight waves: gate/up of the 8B shapes, 224
        // workgroups of four waves before, 16 tokens 19.7 -> 16.5 us, 32: 22.2 -> 18.7, 48: 27 -> 21.5, 64: 26.8 -> 23.9.
        // With partial planes (a few super-blocks per workgroup, one workgroup per CU already) the same gains nothing:
        // down 15.4 -> 16.6 at 64 tokens.
        if constexpr (MODE != GEMM_F32) {
            if (parts == 1 && gemm_two_k_parts(a, max_tok)) {
                if (a.M <= 16) return launch_gemm_k<MODE, 2, 16, false, 8, 2>(a, a.M, 1, st);
                if (a.M <= 32) return launch_gemm_k<MODE, 2, 32, false, 8, 2>(a, a.M, 1, st);
                if (a.M <= 48) return launch_gemm_k<MODE, 2, 48, false, 8, 2>(a, a.M, 1, st);
                return launch_gemm_k<MODE, 2, 64, false, 8, 2>(a, a.M, 1, st);
            }
        }
        if (a.M <= 16) return launch_gemm_k<MODE, 2, 16, false, 4, 1>(a, a.M, parts, st);
        if (a.M <= 32) return launch_gemm_k<MODE, 2, 32, false, 4, 1>(a, a.M, parts, st);
        if (a.M <= 48) return launch_gemm_k<MODE, 2, 48, false, 4, 1>(a, a.M, parts, st);
        return launch_gemm_k<MODE, 2, 64, false, 4, 1>(a, a.M, parts, st);
    }
    if constexpr (MODE == GEMM_F32) return hipErrorInvalidValue;   // partial planes: at most 64 tokens
    else {
        // Plans of more than 64 tokens.  The tile goes by the rows that are there (a.M) and never changes a bit of the
        // result; the K parts do, so they go by the whole matrix and the plan's token count.
        if constexpr (MODE != GEMM_GATE_UP) {
            if (gemm_k_slices(a.nsb, a.total_tiles, max_tok)) {
                const uint32_t groups = (a.ntiles + kSliceRows - 1) / kSliceRows;
                auto one_round = [&](uint32_t mt) { return groups * ((a.M + mt - 1) / mt) <= 256; };
                if (gemm_slice_tiles(a.total_tiles, a.M)) {
                    if (one_round(32)) return launch_gemm_kslice<MODE, 2>(a, st);
                    if (one_round(48)) return launch_gemm_kslice<MODE, 3>(a, st);
                    if (one_round(64)) return launch_gemm_kslice<MODE, 4>(a, st);
                    return launch_gemm_kslice<MODE, 5>(a, st);
                }
                if ((a.ntiles + 7) / 8 * ((a.M + 47) / 48) <= 256) return launch_gemm_k<MODE, 2, 48, false, 8, 2, true>(a, a.M, 1, st);
                return launch_gemm_k<MODE, 2, 64, false, 8, 2, true>(a, a.M, 1, st);
            }
        }
        if (gemm_two_k_parts(a, max_tok)) {
            // the smallest tile that still leaves at most one workgroup per CU (there is one: the rule saw to it).  What each
            // tile is worth where it is the one, against the next larger: O / down, us: 200 tokens 32: 19.1 / 52 against
            // 22.7 / 61; 300: 48: 22.2 / 62 against 22.9 / 64; 450: 64: 25.8 / 72 against 28.6 / 81; 600: 80: 30.8 / 87
            // against 32.7 / 93; 700: 96: 33.2 / 97 against 35.6 / 102; 850: 112: 37.4 / 107 against 40.5 / 115.  A tile
            // that is too small pays a second round (450 tokens in 48: 40 / 110).  QKV at 512 tokens 39.2 without the parts,
            // 36.3 in 112-token tiles; down at 768 122 without, 98.9 in 96
            const uint32_t groups = (a.ntiles + 7) / 8;
            auto one_round = [&](uint32_t mt) { return groups * ((a.M + mt - 1) / mt) <= 256; };
            if (one_round(32)) return launch_gemm_k<MODE, 2, 32, false, 8, 2>(a, a.M, 1, st);
            if (one_round(48)) return launch_gemm_k<MODE, 2, 48, false, 8, 2>(a, a.M, 1, st);
            if (one_round(64)) return launch_gemm_k<MODE, 2, 64, false, 8, 2>(a, a.M, 1, st);
            if (one_round(80)) return launch_gemm_k<MODE, 2, 80, false, 8, 2>(a, a.M, 1, st);
            if (one_round(96)) return launch_gemm_k<MODE, 2, 96, false, 8, 2>(a, a.M, 1, st);
            if (one_round(112)) return launch_gemm_k<MODE, 2, 112, false, 8, 2>(a, a.M, 1, st);
            return launch_gemm_k<MODE, 2, 128, false, 8, 2>(a, a.M, 1, st);
        }
        switch (gemm_pick_tile(a, MODE == GEMM_GATE_UP ? 256 : 224)) {   // (256 tokens spill in the other modes)
            case 16: return launch_gemm_k<MODE, 2, 16, false, 4, 1>(a, a.M, 1, st);
            case 32: return launch_gemm_k<MODE, 2, 32, false, 4, 1>(a, a.M, 1, st);
            case 64: return launch_gemm_k<MODE, 2, 64, false, 4, 1>(a, a.M, 1, st);
            case 96: return launch_gemm_k<MODE, 2, 96, false, 8, 1>(a, a.M, 1, st);
            case 128: return launch_gemm_k<MODE, 2, 128, false, 8, 1>(a, a.M, 1, st);
            case 160: return launch_gemm_k<MODE, 2, 160, false, 8, 1>(a, a.M, 1, st);
            case 192: return launch_gemm_k<MODE, 2, 192, false, 8, 1>(a, a.M, 1, st);
            case 224: return launch_gemm_k<MODE, 2, 224, false, 8, 1>(a, a.M, 1, st);
        }
        if constexpr (MODE == GEMM_GATE_UP) return launch_gemm_k<MODE, 2, 256, false, 8, 1>(a, a.M, 1, st);
        return hipErrorInvalidValue;
    }
}

template <int MT>
static hipError_t launch_gemm_upload_t(const GemmArgs &a, const UploadArgs &up, hipStream_t st) {
    constexpr size_t ldsb = gemm_lds_bytes(MT, 2, 4);
    static_assert(ldsb <= 64 * 1024, "LDS without an attribute");
    const uint32_t columns = (a.ntiles + 7) / 8, parts = a.sb_per_part ? (a.nsb + a.sb_per_part - 1) / a.sb_per_part : 1;
    hipLaunchKernelGGL(gemm_w4_upload_kernel<MT>, dim3(columns + kUploadWgs, (a.M + MT - 1) / MT, parts), dim3(256), ldsb, st, a, up, columns);
    return hipGetLastError();
}

// the kernel addresses weights and activations as a uniform base plus 32-bit byte offsets
static bool gemm_in_reach(const GemmArgs &a) {
    return (uint64_t)a.ntiles * a.tile_u4 * 16u <= 0xFFFFFFFFull && (uint64_t)a.M * (a.top_k ? a.top_k : 1u) * a.x_stride * 2u <= 0xFFFFFFFFull;
}

hipError_t launch_gemm_upload(const GemmArgs &a, uint32_t max_tok, const UploadArgs &up, hipStream_t st) {
    if (up.n16 > kUploadUnits || max_tok > 64 || !gemm_in_reach(a)) return hipErrorInvalidValue;
    if (a.M <= 16) return launch_gemm_upload_t<16>(a, up, st);
    if (a.M <= 32) return launch_gemm_upload_t<32>(a, up, st);
    if (a.M <= 48) return launch_gemm_upload_t<48>(a, up, st);
    return launch_gemm_upload_t<64>(a, up, st);
}

hipError_t launch_gemm(int mode, const GemmArgs &a, uint32_t ntasks, uint32_t max_tok, hipStream_t st) {
    if (!gemm_in_reach(a)) return hipErrorInvalidValue;
    switch (mode) {
        case GEMM_PLAIN: return launch_gemm_m<GEMM_PLAIN>(a, ntasks, max_tok, st);
        case GEMM_RESID: return launch_gemm_m<GEMM_RESID>(a, ntasks, max_tok, st);
        case GEMM_GATE_UP: return launch_gemm_m<GEMM_GATE_UP>(a, ntasks, max_tok, st);
        case GEMM_F32: return launch_gemm_m<GEMM_F32>(a, ntasks, max_tok, st);
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------
// Gathered host->device copy.  A fixed, small number of workgroups walks every shard of the list in
// turn, each taking its share of every shard in 16-byte units (a wave moves 1 KB contiguous per
// load), eight loads per thread in flight.
// ------------------------------------------------------------------------------------
constexpr uint32_t kGatherDescs = 128;   // descriptors staged in LDS at a time
constexpr uint32_t kGatherWgs = 16;
constexpr uint32_t kLdsPerCu = 160 * 1024;   // gfx950
__global__ __launch_bounds__(256) void h2d_gather_kernel(const CopyDesc *descs, uint32_t n) {
    __shared__ CopyDesc sd[kGatherDescs];
    // The rest of the CU's LDS is claimed and left unused: no workgroup that needs LDS (every matmul and
    // attention kernel and the plane sums of O, down and a first layer's QKV do) can then be placed on this CU, where its loads would
    // queue behind half a megabyte of PCIe reads on the CU's one vector-memory path (a one-token
    // matmul beside a gather: 45 us without the claim, 25 us with it, 13 us alone).
    __shared__ uint8_t rest[kLdsPerCu - sizeof(CopyDesc) * kGatherDescs];
    asm volatile("" ::"v"(&rest[threadIdx.x]));
    const uint32_t stride = gridDim.x * 256;
    for (uint32_t base = 0; base < n; base += kGatherDescs) {
        const uint32_t m = min(kGatherDescs, n - base);
        __syncthreads();
        // the list may sit in pinned host memory: one round trip over PCIe for the whole chunk
        if (threadIdx.x < m) sd[threadIdx.x] = descs[base + threadIdx.x];
        __syncthreads();
        for (uint32_t e = 0; e < m; ++e) {
            const u4_t *src = reinterpret_cast<const u4_t *>(sd[e].src);
            u4_t *dst = reinterpret_cast<u4_t *>(sd[e].dst);
            const uint32_t n16 = sd[e].n16;
            if (n16 == 0) continue;
            // past the end a load re-reads the last unit and its store is skipped, so the last pass
            // keeps eight loads in flight like the others
            for (uint32_t idx = blockIdx.x * 256 + threadIdx.x; idx < n16; idx += 8 * stride) {
                u4_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(src + min(idx + u * stride, n16 - 1));
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (idx + u * stride < n16) dst[idx + u * stride] = v[u];
            }
        }
    }
}

hipError_t launch_h2d_gather(const CopyDesc *descs, uint32_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    // 16 workgroups keep 512 KB of reads in flight, which fills the PCIe link; more only queue up
    // ahead of the compute stream's reads from HBM
    hipLaunchKernelGGL(h2d_gather_kernel, dim3(kGatherWgs), dim3(256), 0, st, descs, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// A forward's routing tables, pinned host memory -> workspace, in 16-byte units.  Tens of KB: the time is one round
// trip over PCIe (3 to 4 us for up to 30 KB, 8 us for 282 KB), and a kernel in the stream needs no hand-over to a copy
// engine and back (a 16-token step of two MoE layers 186 us by hipMemcpyAsync, 177 us this way).  Nothing reads them before
// the first layer's routing, so they ride, on workgroups of their own, in a launch in front of it: up to 32 KB
// in the first QKV GEMM where that leaves planes (two 16-token steps of two layers 334 -> 327 us), any number in the launch of its RMS factors where there is one
// (512 tokens: 3.3 us for the factors and 8.3 for the upload before, 9.5 together; in the GEMM's eight workgroups those 282 KB take 13 us longer than the GEMM).  This launch is for the rest.
// ------------------------------------------------------------------------------------
// Two runs in one launch: the tables' areas have room for every expert, and what is not in use stays where it is.
__global__ __launch_bounds__(256) void upload_tables_kernel(UploadArgs up) {
    upload_unit(up, blockIdx.x * 256 + threadIdx.x);
}

bool make_upload(const void *src, void *dst, uint64_t first, uint64_t second_at, uint64_t second, UploadArgs *up) {
    if ((uintptr_t)src % 16 || (uintptr_t)dst % 16 || first % 16 || second_at % 16 || second % 16 || second_at < first || (second_at + second) / 16 > 0x7FFFFFFFull)
        return false;
    *up = {static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), (uint32_t)(first / 16), (uint32_t)((second_at - first) / 16), (uint32_t)((first + second) / 16)};
    return true;
}

hipError_t launch_upload_tables(const UploadArgs &up, hipStream_t st) {
    if (up.n16 == 0) return hipSuccess;
    hipLaunchKernelGGL(upload_tables_kernel, dim3((up.n16 + 255) / 256), dim3(256), 0, st, up);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Rows computed on the host (experts run by the CPU back-end) land in one contiguous upload;
// this puts each where the combine step expects it: dst row idx[r] = src row r.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void scatter_rows_kernel(const float *src, const int32_t *idx, uint32_t H, float *dst) {
    const float4 *s4 = reinterpret_cast<const float4 *>(src + (size_t)blockIdx.x * H);
    float4 *d4 = reinterpret_cast<float4 *>(dst + (size_t)idx[blockIdx.x] * H);
    for (uint32_t j = threadIdx.x; j < H / 4; j += 256) d4[j] = s4[j];
}

hipError_t launch_scatter_rows(const float *src, const int32_t *idx, uint32_t n, uint32_t H, float *dst, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if (H % 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL(scatter_rows_kernel, dim3(n), dim3(256), 0, st, src, idx, H, dst);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Split-K epilogue (batched decode): out = epilogue(sum over parts, ascending, of the fp32
// partial planes).  One thread per output element; GATE_UP pairs a gate column with the up
// column 16 physical columns further on.
// ------------------------------------------------------------------------------------
template <int MODE>
__global__ __launch_bounds__(256) void splitk_epilogue_kernel(const float *partial, uint32_t parts, uint32_t part_stride,
                                                              uint32_t M, uint32_t ncols_phys, const float *rinv, RowQuarters sums,
                                                              const __half *res, __half *out, uint32_t out_stride,
                                                              uint32_t out_row0) {
    // one thread per four adjacent output columns (a 16-column tile is never straddled)
    const uint32_t ncols = MODE == GEMM_GATE_UP ? ncols_phys / 2 : ncols_phys;
    const uint32_t nq = ncols / 4;
    const size_t n = (size_t)M * nq;
    for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (size_t)gridDim.x * 256) {
        const uint32_t m = (uint32_t)(q / nq), j = (uint32_t)(q % nq) * 4;
        const uint32_t c0 = MODE == GEMM_GATE_UP ? (j >> 4) * 32 + (j & 15) : j;
        const float *p0 = partial + (size_t)m * ncols_phys + c0;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f), u = v;
        // all planes are requested before the first is added (a plane past the last re-reads the last one and
        // is left out of the sum): one round trip to memory instead of one per plane; the sum stays in plane order
        float4 pa[8], pb[8];
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            const size_t off = (size_t)min(p, parts - 1) * part_stride;
            pa[p] = *reinterpret_cast<const float4 *>(p0 + off);
            if (MODE == GEMM_GATE_UP) pb[p] = *reinterpret_cast<const float4 *>(p0 + off + 16);
        }
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            if (p < parts) {
                v.x += pa[p].x; v.y += pa[p].y; v.z += pa[p].z; v.w += pa[p].w;
                if (MODE == GEMM_GATE_UP) { u.x += pb[p].x; u.y += pb[p].y; u.z += pb[p].z; u.w += pb[p].w; }
            }
        }
        float r[4] = {v.x, v.y, v.z, v.w};
        if (MODE == GEMM_PLAIN) {
            const float ri = sums.sq ? factor_of_quarters(sums, m) : rinv[m];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = ri * r[e];
        } else if (MODE == GEMM_RESID) {
            if (res) {
                const __half2 *rs = reinterpret_cast<const __half2 *>(res + (size_t)m * out_stride + out_row0 + j);
                const float2 r01 = __half22float2(rs[0]), r23 = __half22float2(rs[1]);
                r[0] = r01.x + r[0]; r[1] = r01.y + r[1]; r[2] = r23.x + r[2]; r[3] = r23.y + r[3];
            }
        } else {
            const float ri = sums.sq ? factor_of_quarters(sums, m) : rinv[m];
            const float g[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = silu(ri * r[e]) * (ri * g[e]);
        }
        __half2 *d2 = reinterpret_cast<__half2 *>(out + (size_t)m * out_stride + out_row0 + j);
        d2[0] = __half2{to_half(r[0]), to_half(r[1])};
        d2[1] = __half2{to_half(r[2]), to_half(r[3])};
    }
}

hipError_t launch_splitk_epilogue(int mode, const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M,
                                  uint32_t ncols_phys, const float *rinv, const RowQuarters &sums, const __half *res, __half *out,
                                  uint32_t out_stride, uint32_t out_row0, hipStream_t st) {
    // four columns per thread: 16-byte plane reads, 8-byte stores (columns come in tiles of 16 and
    // out_row0 / out_stride are multiples of 16, so both stay aligned)
    if (ncols_phys % 16 || out_row0 % 4 || out_stride % 4 || part_stride % 4 || parts < 1 || parts > 8) return hipErrorInvalidValue;
    const size_t n = (size_t)M * (ncols_phys / 4);
    const uint32_t blocks = (uint32_t)std::min<size_t>((n + 255) / 256, 2048);
    switch (mode) {
        case GEMM_PLAIN:
            hipLaunchKernelGGL(splitk_epilogue_kernel<GEMM_PLAIN>, dim3(blocks), dim3(256), 0, st, partial, parts, part_stride, M, ncols_phys, rinv, sums, res, out, out_stride, out_row0);
            break;
        case GEMM_RESID:
            hipLaunchKernelGGL(splitk_epilogue_kernel<GEMM_RESID>, dim3(blocks), dim3(256), 0, st, partial, parts, part_stride, M, ncols_phys, rinv, sums, res, out, out_stride, out_row0);
            break;
        case GEMM_GATE_UP:
            hipLaunchKernelGGL(splitk_epilogue_kernel<GEMM_GATE_UP>, dim3(blocks), dim3(256), 0, st, partial, parts, part_stride, M, ncols_phys, rinv, sums, res, out, out_stride, out_row0);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Split-K epilogue of a matrix behind a norm (PLAIN) whose input rows' RMS factors nobody has left: the first layer's QKV.
// blockIdx.y is the token, blockIdx.x 1024 of its columns; every workgroup of a token works the factor out for itself, beside
// its planes' loads: thread t adds the chunks t, t + 256, ... of the input row, reduced as in rinv_kernel, so the factor has
// the bits of the launch (3 to 5 us, latency) that is left out.  64 tokens, 6144 columns of 4096: 4.5 us with or without.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void splitk_epilogue_norm_kernel(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t ncols,
                                                                   const __half *x, uint32_t H, float eps, __half *out,
                                                                   uint32_t out_stride, uint32_t out_row0) {
    __shared__ float part[4];
    const uint32_t m = blockIdx.y, j = (blockIdx.x * 256 + threadIdx.x) * 4, jc = min(j, ncols - 4);
    const float *p0 = partial + (size_t)m * ncols + jc;
    float4 pa[8];
#pragma unroll
    for (uint32_t p = 0; p < 8; ++p) pa[p] = *reinterpret_cast<const float4 *>(p0 + (size_t)min(p, parts - 1) * part_stride);
    const float ri = row_factor(x + (size_t)m * H, H, eps, part);
    if (j >= ncols) return;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (uint32_t p = 0; p < 8; ++p) {
        if (p < parts) { v.x += pa[p].x; v.y += pa[p].y; v.z += pa[p].z; v.w += pa[p].w; }
    }
    __half2 *d2 = reinterpret_cast<__half2 *>(out + (size_t)m * out_stride + out_row0 + j);
    d2[0] = __half2{to_half(ri * v.x), to_half(ri * v.y)};
    d2[1] = __half2{to_half(ri * v.z), to_half(ri * v.w)};
}

hipError_t launch_splitk_epilogue_norm(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M, uint32_t ncols, const __half *x,
                                       uint32_t H, float eps, __half *out, uint32_t out_stride, uint32_t out_row0, hipStream_t st) {
    if (M == 0) return hipSuccess;
    if (ncols % 16 || out_row0 % 4 || out_stride % 4 || part_stride % 4 || parts < 1 || parts > 8 || H % 8 || M > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(splitk_epilogue_norm_kernel, dim3((ncols + 1023) / 1024, M), dim3(256), 0, st, partial, parts, part_stride, ncols, x, H, eps,
                       out, out_stride, out_row0);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Split-K epilogue of a residual matrix whose launch covers whole rows of the hidden state
// (out = res + sum of the planes), with the RMS factor of the row it has just written: one
// workgroup per token.  Thread t owns the 8-column chunks t, t + 256, ... exactly as in
// rinv_kernel, squares the fp16 values it stores and reduces in the same order, so rinv[m] has the
// bits rinv_kernel would give on the stored row, and the separate launch can be left out.
// Planes past `parts` are not read (the load is redirected to the last plane and discarded by a
// select, so the loads carry no branch).
// ------------------------------------------------------------------------------------
template <int NR>   // > 0: the workgroups behind the first M route four tokens each, as in rinv_kernel
__global__ __launch_bounds__(256) void splitk_epilogue_resid_rinv_kernel(const float *partial, uint32_t parts,
                                                                         uint32_t part_stride, uint32_t M, uint32_t H,
                                                                         const __half *res, __half *out, float eps,
                                                                         float *rinv, RouteArgs ra) {
    if constexpr (NR > 0) {
        if (blockIdx.x >= M) { route_tokens<NR>(ra, blockIdx.x - M); return; }
    }
    __shared__ float part[4];
    const uint32_t m = blockIdx.x, nq = H / 8;
    const float *prow = partial + (size_t)m * H;
    float ss = 0.f;
    for (uint32_t q = threadIdx.x; q < nq; q += 256) {
        float4 a[8][2];
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            const float *src = prow + (size_t)(p < parts ? p : parts - 1) * part_stride + q * 8;
            a[p][0] = *reinterpret_cast<const float4 *>(src);
            a[p][1] = *reinterpret_cast<const float4 *>(src + 4);
        }
        uint4 rv = uint4{0u, 0u, 0u, 0u};
        if (res) rv = *reinterpret_cast<const uint4 *>(res + (size_t)m * H + q * 8);
        float r[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            const bool on = p < parts;   // adding +0 leaves a sum that started at +0 unchanged
            r[0] += on ? a[p][0].x : 0.f; r[1] += on ? a[p][0].y : 0.f;
            r[2] += on ? a[p][0].z : 0.f; r[3] += on ? a[p][0].w : 0.f;
            r[4] += on ? a[p][1].x : 0.f; r[5] += on ? a[p][1].y : 0.f;
            r[6] += on ? a[p][1].z : 0.f; r[7] += on ? a[p][1].w : 0.f;
        }
        if (res) {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = half_of(rv, e) + r[e];
        }
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint16_t lo = __builtin_bit_cast(uint16_t, to_half(r[2 * e]));
            const uint16_t hi = __builtin_bit_cast(uint16_t, to_half(r[2 * e + 1]));
            d[e] = (uint32_t)lo | ((uint32_t)hi << 16);
        }
        const uint4 o = uint4{d[0], d[1], d[2], d[3]};
        *reinterpret_cast<uint4 *>(out + (size_t)m * H + q * 8) = o;
        ss += sumsq8(o);
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) rinv[m] = rsqrtf((((part[0] + part[1]) + part[2]) + part[3]) / (float)H + eps);
}

hipError_t launch_splitk_epilogue_resid_rinv(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M,
                                             uint32_t H, const __half *res, __half *out, float eps, float *rinv,
                                             const RouteArgs *route, hipStream_t st) {
    if (M == 0) return hipSuccess;
    if (parts == 0 || parts > 8 || H % 8 || part_stride % 4 || !partial || !out || !rinv) return hipErrorInvalidValue;
    if (!route) hipLaunchKernelGGL(splitk_epilogue_resid_rinv_kernel<0>, dim3(M), dim3(256), 0, st, partial, parts, part_stride, M, H, res, out, eps, rinv, RouteArgs{});
    else if (!route_rides(*route)) return hipErrorInvalidValue;
    else if (route->E <= 128) hipLaunchKernelGGL(splitk_epilogue_resid_rinv_kernel<2>, dim3(M + (route->M + 3) / 4), dim3(256), 0, st, partial, parts, part_stride, M, H, res, out, eps, rinv, *route);
    else hipLaunchKernelGGL(splitk_epilogue_resid_rinv_kernel<4>, dim3(M + (route->M + 3) / 4), dim3(256), 0, st, partial, parts, part_stride, M, H, res, out, eps, rinv, *route);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// The same residual epilogue for dense layers, as four workgroups of one wave per token: wave w takes the chunks of the four-wave
// kernel's wave w, two per lane and round with every load requested before the first is used, and leaves its sum of squares
// for the readers to add up.  Bound by latency: a workgroup per token pulls 144 KB through each of 64 CUs in two rounds of
// loads that wait for each other, this form 36 KB through each of 256 in one; 64 tokens of 4096 columns from eight planes
// 4.3 -> 4.0 us in the kernel trace, 5 tokens 4.1 -> 3.4, 2 tokens of 2048 columns 3.4 -> 3.0, 2 of 512 2.7 -> 2.5 (about 2.5
// are a launch's own), so the form serves 2 tokens and up; four steps of two layers of 64 tokens 635 -> 613 us.
// SLICES: the planes are the eight K slices of a matrix that gemm_kslice_kernel finishes in one launch for more rows: the same
// sums in the same order, half of K after half, and the same sums of squares, a run of 128 columns being 16 lanes' here.
// ------------------------------------------------------------------------------------
template <bool SLICES>
__global__ __launch_bounds__(64) void splitk_epilogue_resid_quarters_kernel(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M,
                                                                            uint32_t H, const __half *res, __half *out, float *quarters) {
    // claimed and left unused: a workgroup that needs LDS is not placed on a CU whose LDS a gather copy holds, where its
    // loads would queue behind the reads over PCIe (beside a gather 31 us without the claim, 18 with it, 4 alone)
    __shared__ uint32_t claim[64];
    asm volatile("" ::"v"(&claim[threadIdx.x]));
    const uint32_t w = blockIdx.x, m = blockIdx.y, nq = H / 8;
    const float *prow = partial + (size_t)m * H;
    float ss = 0.f;
    for (uint32_t q0 = w * 64 + threadIdx.x; q0 < nq; q0 += 512) {
        float4 a[2][8][2];
        uint4 rv[2];
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) {
            const uint32_t q = q0 + u * 256 < nq ? q0 + u * 256 : q0;      // (past the row's end the first chunk again, not stored)
#pragma unroll
            for (uint32_t p = 0; p < 8; ++p) {
                const float *src = prow + (size_t)(p < parts ? p : parts - 1) * part_stride + q * 8;
                a[u][p][0] = *reinterpret_cast<const float4 *>(src);
                a[u][p][1] = *reinterpret_cast<const float4 *>(src + 4);
            }
            rv[u] = res ? *reinterpret_cast<const uint4 *>(res + (size_t)m * H + q * 8) : uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (uint32_t u = 0; u < 2; ++u) {
            if (q0 + u * 256 >= nq) break;
            float r[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, first[8];     // first: of the first half of K
#pragma unroll
            for (uint32_t p = 0; p < 8; ++p) {
                const bool on = p < parts;   // adding +0 leaves a sum that started at +0 unchanged
                r[0] += on ? a[u][p][0].x : 0.f; r[1] += on ? a[u][p][0].y : 0.f;
                r[2] += on ? a[u][p][0].z : 0.f; r[3] += on ? a[u][p][0].w : 0.f;
                r[4] += on ? a[u][p][1].x : 0.f; r[5] += on ? a[u][p][1].y : 0.f;
                r[6] += on ? a[u][p][1].z : 0.f; r[7] += on ? a[u][p][1].w : 0.f;
                if (SLICES && p == 3) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) { first[e] = r[e]; r[e] = 0.f; }
                }
            }
            if (SLICES) {
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] = first[e] + r[e];
            }
            if (res) {
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] = half_of(rv[u], e) + r[e];
            }
            uint32_t d[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint16_t lo = __builtin_bit_cast(uint16_t, to_half(r[2 * e]));
                const uint16_t hi = __builtin_bit_cast(uint16_t, to_half(r[2 * e + 1]));
                d[e] = (uint32_t)lo | ((uint32_t)hi << 16);
            }
            const uint4 o = uint4{d[0], d[1], d[2], d[3]};
            *reinterpret_cast<uint4 *>(out + (size_t)m * H + (q0 + u * 256) * 8) = o;
            if constexpr (SLICES) {
                // as four columns each of two row-tiles are added up there: lane and lane ^ 2 hold the same columns of either tile,
                // lane ^ 1 the tile's other half, the lane mirrored in its eight the other two tiles of 64 columns, the one mirrored in its
                // row the run's other half
                const h2_t h[4] = {as_h2(d[0]), as_h2(d[1]), as_h2(d[2]), as_h2(d[3])};
                float sq[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    float part = 0.f;
                    part = fmaf((float)h[2 * e].x, (float)h[2 * e].x, part); part = fmaf((float)h[2 * e].y, (float)h[2 * e].y, part);
                    part = fmaf((float)h[2 * e + 1].x, (float)h[2 * e + 1].x, part); part = fmaf((float)h[2 * e + 1].y, (float)h[2 * e + 1].y, part);
                    sq[e] = part + dpp_of<0x4E>(part);      // quad_perm 2,3,0,1
                }
                float run = sq[0] + sq[1];
                run += dpp_of<0xB1>(run);                   // quad_perm 1,0,3,2
                run += dpp_of<0x141>(run);                  // row_half_mirror
                run += dpp_of<0x140>(run);                  // row_mirror
                const uint32_t q = q0 + u * 256;
                if (q % 16 == 0) quarters[ssq_at(q / 16, m, M)] = run;
            } else {
                ss += sumsq8(o);
            }
        }
    }
    if constexpr (!SLICES) {
        ss = wave_sum(ss);
        if (threadIdx.x == 0) quarters[w * M + m] = ss;
    }
}

hipError_t launch_splitk_epilogue_resid_quarters(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M, uint32_t H,
                                                 const __half *res, __half *out, float *quarters, bool slices, hipStream_t st) {
    if (M == 0) return hipSuccess;
    if (parts == 0 || parts > 8 || H % 8 || part_stride % 4 || !partial || !out || !quarters || M > 65535 || (slices && (parts != 8 || H % 256))) return hipErrorInvalidValue;
    if (slices) hipLaunchKernelGGL(splitk_epilogue_resid_quarters_kernel<true>, dim3(4, M), dim3(64), 0, st, partial, parts, part_stride, M, H, res, out, quarters);
    else hipLaunchKernelGGL(splitk_epilogue_resid_quarters_kernel<false>, dim3(4, M), dim3(64), 0, st, partial, parts, part_stride, M, H, res, out, quarters);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Lane-layout probe for v_mfma_f32_16x16x32_f16 (in-bounds, integer-valued inputs):
// A[i][k] = 1 if (i, k) == (pi, pk) else 0, B[k][j] = 1 if (k, j) == (pk, pj): the single
// non-zero of C tells which lane/register holds C[pi][pj] under the layout assumed above.
// ------------------------------------------------------------------------------------
__global__ void mfma_probe_kernel(int pi, int pk, int pj, float *out /*[64][4]*/) {
    const int lane = threadIdx.x & 63, i = lane & 15, c = lane >> 4;
    h8_t A = {0, 0, 0, 0, 0, 0, 0, 0}, B = {0, 0, 0, 0, 0, 0, 0, 0};
    if (i == pi && c == pk / 8) A[pk % 8] = (_Float16)1.0f;
    if (i == pj && c == pk / 8) B[pk % 8] = (_Float16)1.0f;
    f4_t C = {0.f, 0.f, 0.f, 0.f};
    C = __builtin_amdgcn_mfma_f32_16x16x32_f16(A, B, C, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) out[lane * 4 + r] = C[r];
}

// LDS transpose read (ds_read_b64_tr_b16): LDS holds the 16-bit numbers 0 .. 2047 at their own index; lane l
// reads at byte address addr[l] (forced to a multiple of 8 inside the table) and stores its four results.
__global__ void lds_tr_probe_kernel(const uint32_t *addr, uint16_t *out /*[64][4]*/) {
    __shared__ __attribute__((aligned(16))) uint16_t tab[2048];
    const int lane = threadIdx.x & 63;
    for (int k = lane; k < 2048; k += 64) tab[k] = (uint16_t)k;
    __syncthreads();
    const uint32_t off = min(addr[lane] & ~7u, 4088u);
    typedef __attribute__((__vector_size__(4 * sizeof(__fp16)))) __fp16 fp16x4_t;
    typedef __attribute__((address_space(3))) fp16x4_t lds_fp16x4_t;
#if defined(__HIP_DEVICE_COMPILE__)
    const fp16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_fp16x4_t *)(reinterpret_cast<unsigned char *>(tab) + off));
    const uint2 bits = __builtin_bit_cast(uint2, v);
    out[lane * 4 + 0] = (uint16_t)(bits.x & 0xFFFFu);
    out[lane * 4 + 1] = (uint16_t)(bits.x >> 16);
    out[lane * 4 + 2] = (uint16_t)(bits.y & 0xFFFFu);
    out[lane * 4 + 3] = (uint16_t)(bits.y >> 16);
#endif
}

hipError_t launch_lds_tr_probe(const uint32_t *addr, uint16_t *out, hipStream_t st) {
    hipLaunchKernelGGL(lds_tr_probe_kernel, dim3(1), dim3(64), 0, st, addr, out);
    return hipGetLastError();
}

hipError_t launch_mfma_probe(int pi, int pk, int pj, float *out, hipStream_t st) {
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(1), dim3(64), 0, st, pi, pk, pj, out);
    return hipGetLastError();
}

}  // namespace ps
