// Launch interface between the executor (stack.hip) and the device kernels (kernels.hip).
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "ps_internal.h"

namespace ps {

enum { GEMV_PLAIN = 0, GEMV_RESID = 1, GEMV_GATE_UP = 2, GEMV_F32 = 3 };
enum { GEMM_PLAIN = 0, GEMM_RESID = 1, GEMM_GATE_UP = 2, GEMM_F32 = 3 };

// One token.  PLAIN: out = rinv * (W x) with rinv from x's RMS; RESID: out = res + W x;
// GATE_UP: out = silu(rinv * gate) * (rinv * up); F32: out_f32 = W x.
struct GemvArgs {
    const uint4 *W;       // first tile of the slab (ignored when tasks != null)
    uint32_t nunits;      // row-tiles (GATE_UP: tile pairs) in this launch
    uint32_t tile_u4;     // tile stride in 16-byte units
    uint32_t nsb, ngroups, K;
    const __half *x;      // input row
    uint32_t x_off, x_group;   // input column map (identity: 0, 1)
    uint32_t x_stride;    // grouped launches: elements between input rows
    float eps;
    const __half *res;    // RESID: residual row or null
    __half *out;
    float *out_f32;
    uint32_t out_row0;    // first output element of the slab
    uint32_t out_stride;  // grouped launches: elements between output rows
    uint32_t top_k;
    const DeviceTask *tasks;  // grouped (MoE) launch: one expert per blockIdx.y
    const int32_t *pairs;
};

// Two runs of 16-byte units from pinned host memory to the device, at the same places: units 0 .. first16 - 1, and n16 - first16 more
// from unit first16 + skip16 on
struct UploadArgs {
    const uint4 *src;
    uint4 *dst;
    uint32_t first16, skip16, n16;   // n16 0: nothing
};

// M tokens on the matrix cores.  Same modes; rinv comes from a buffer.
struct GemmArgs {
    const uint4 *W;
    uint32_t ntiles;      // row-tiles in this launch
    uint32_t total_tiles; // row-tiles of the whole matrix (picks the tile shape)
    uint32_t tile_u4, nsb;
    uint32_t M;
    const __half *x;
    uint32_t x_stride, x_off, x_group;
    const float *rinv;
    const __half *res;
    __half *out;
    float *out_f32;
    uint32_t out_stride, out_row0, top_k;
    uint32_t sb_per_part;  // split-K: super-blocks per blockIdx.z part (0 = whole K in one part)
    uint32_t part_stride;  // split-K: elements between the fp32 partial planes
    // Sums of squares instead of a buffer of RMS factors (plans of more than 64 tokens): RESID leaves, per token and run of 128
    // output columns (of 64 where a workgroup has no more: gemm_leaves_halves), the sum of squares of what it stored, four runs of a token side
    // by side: ssq_out[(run / 4 * M + token) * 4 + run % 4].  PLAIN and GATE_UP with ssq_in add a token's ssq_runs runs (nsb, or
    // twice as many of 64 columns; K columns), in pairs, so that both give the same sum, and take their RMS factors from them
    float *ssq_out;
    const float *ssq_in;
    uint32_t ssq_runs;
    uint32_t quarters;    // not 0: ssq_in holds four sums per token instead (ssq_in[w * M + token], see RowQuarters) of this many columns
    float eps;
    const DeviceTask *tasks;
    const int32_t *pairs;
    uint32_t slices;      // RESID, plans of up to 64 tokens: K in eight slices (o_in_slices)
};
constexpr uint32_t kUploadWgs = 8, kUploadUnits = kUploadWgs * 256;     // one unit a thread
// RMS factors of M rows as what the four waves of launch_rinv would add up: sq[w * M + row], H columns (sq null: no such sums)
struct RowQuarters {
    const float *sq;
    uint32_t M, H;
    float eps;
};

// one host->device copy of a gathered batch: n16 16-byte units from pinned host memory to VRAM
struct CopyDesc {
    uint64_t src, dst;
    uint32_t n16, pad0, pad1, pad2;
};
// one launch copies `n` shards (descs may live in pinned host memory): the GPU pulls them over
// PCIe itself, which avoids the per-call cost of many small hipMemcpyAsync
hipError_t launch_h2d_gather(const CopyDesc *descs, uint32_t n, hipStream_t st);
// small blocks of pinned host memory -> device, at the same places: bytes 0 .. first - 1 and second_at .. second_at + second - 1
// (everything a multiple of 16; false where it is not), and the launch that does it on its own
bool make_upload(const void *src, void *dst, uint64_t first, uint64_t second_at, uint64_t second, UploadArgs *up);
hipError_t launch_upload_tables(const UploadArgs &up, hipStream_t st);

// MoE routing of M tokens: the top_k largest fp32 logits (ties to the lower index, in descending order) and the
// softmax over them.  As a launch of its own, or riding in the launch that produces the layer's RMS factors or,
// for one token, in O's (`route` of these launches; route_rides says whether the sizes allow it)
struct RouteArgs {
    const float *logits;   // [M][E]
    uint32_t M, E, top_k;
    int32_t *idx;          // [M][top_k]
    float *w;
};
uint32_t gemv_ksplit(uint32_t ngroups, uint32_t total_units);
hipError_t launch_gemv(int mode, uint32_t ksplit, const GemvArgs &a, uint32_t ntasks, const RouteArgs *route, hipStream_t st);
hipError_t launch_gemm(int mode, const GemmArgs &a, uint32_t ntasks, uint32_t max_tok, hipStream_t st);
// the same for partial planes (F32, ungrouped) with an upload of at most kUploadUnits riding in it, on kUploadWgs workgroups of its own
hipError_t launch_gemm_upload(const GemmArgs &a, uint32_t max_tok, const UploadArgs &up, hipStream_t st);
// Two to kGemvMtTokens tokens of a dense sub-layer whose K is a multiple of 1024 (rows of x x_stride
// elements apart, rows of out and res out_stride apart): the one-token kernel's launch shape with the dot
// products on the matrix cores; PLAIN, RESID and GATE_UP, the RMS factors computed from the activations
constexpr int kGemvMtTokens = 4;
hipError_t launch_gemv_mt(int mode, uint32_t ksplit, const GemvArgs &a, uint32_t ntok, hipStream_t st);
// sums `parts` fp32 partial planes [M][ncols_phys] in ascending order and applies the mode's epilogue
hipError_t launch_splitk_epilogue(int mode, const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M,
                                  uint32_t ncols_phys, const float *rinv, const RowQuarters &sums, const __half *res, __half *out,
                                  uint32_t out_stride, uint32_t out_row0, hipStream_t st);
// the PLAIN epilogue with the RMS factors worked out from the matrix's input rows x [M][H], with launch_rinv's bits
hipError_t launch_splitk_epilogue_norm(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M, uint32_t ncols, const __half *x,
                                       uint32_t H, float eps, __half *out, uint32_t out_stride, uint32_t out_row0, hipStream_t st);
hipError_t launch_route(const RouteArgs &ra, hipStream_t st);
bool route_rides(const RouteArgs &ra);
// whether the launches of a matrix in plans of more than 64 tokens leave sums of squares (RESID) per 64 columns for M rows
bool gemm_leaves_halves(uint32_t nsb, uint32_t total_tiles, uint32_t plan_tokens, uint32_t M);
// the factors in the order of the GEMM's sums of squares (see GemmArgs), with their bits
hipError_t launch_rinv_runs(const __half *x, uint32_t M, uint32_t H, float eps, float *rinv, hipStream_t st);
// (up: an upload that rides in the launch, not together with route)
hipError_t launch_rinv(const __half *x, uint32_t M, uint32_t H, float eps, float *rinv, const RouteArgs *route, const UploadArgs &up, hipStream_t st);
// residual epilogue over whole rows of the hidden state (ncols == out_stride == H, first column 0,
// at most 8 planes) that also writes the RMS factor of each row it stores, bit-identical to
// launch_splitk_epilogue(GEMM_RESID, ...) followed by launch_rinv(out, ...)
hipError_t launch_splitk_epilogue_resid_rinv(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M,
                                             uint32_t H, const __half *res, __half *out, float eps, float *rinv,
                                             const RouteArgs *route, hipStream_t st);
// the same stores over four times the workgroups, with the sums of squares the factors come from instead of the factors
// (quarters[w * M + row]; whoever wants a factor adds a row's four): their bits once added up.  slices: eight planes are the slices of a
// matrix with K in slices, stores and sums of squares (per 128 columns) have the bits of the GEMM's in one launch; H a multiple of 256
hipError_t launch_splitk_epilogue_resid_quarters(const float *partial, uint32_t parts, uint32_t part_stride, uint32_t M, uint32_t H,
                                                 const __half *res, __half *out, float *quarters, bool slices, hipStream_t st);
// Decode attention over a KV cache, one new token.  A cache shard of one kv head is K rows
// [cap][128] followed by V rows [cap][128], fp16; `nheads` shards lie head_stride bytes apart from
// kv (kv heads head0 .. head0 + nheads - 1).  Each workgroup covers one kv head x one chunk of 256
// cached positions for the head's `group` query heads and writes, per query head and chunk, the
// chunk's score maximum, sum of weights and 128 weighted value sums (fp32) to
// part[(q_head * chunk_cap + chunk) * 130].  ctx = cached positions (nothing is launched for 0).
struct AttnArgs {
    const __half *kv;
    uint64_t head_stride;
    uint32_t cap, ctx, head0, nheads, group, chunk_cap;
    const __half *q;      // the token's QKV row: query head h at [h * 128]
    float *part;
    const uint32_t *ctx_dev;   // not null: the context length is read from here (device) instead of ctx, and
                               // the launch covers every chunk the cache can hold (a captured graph is
                               // replayed at any context); workgroups past the context leave at once
};
// Attention of a chunk of `ntok` new tokens (rows of q, q_stride elements apart): every token sees the ctx cached
// positions of its kv head (cache shards of kv heads head0 .. head0 + nheads - 1, k_base = the first one, head_stride
// bytes apart, K rows [cap][128] then V rows) and, causally, the chunk's own K / V rows, read in place from the
// tokens' QKV rows (k_own / v_own = kv head 0 of token 0, own_stride elements between tokens).  One launch per run of
// cache shards.  nsplit == 1: finished rows out[t][q_head * 128 ..], and the tokens' K / V rows appended at positions
// ctx .. ctx + ntok - 1 of home[kv head] (address of its K row 0; no home: not appended); > 1: records
// part[((t * n_q + q_head) * nsplit + split) * 130] (maximum, weight sum, 128 sums) for launch_attn_combine_chunk.
// nsplit and rounds_per_split come from attn_chunk_deal.  few: the weights in fp32's precision (fewer than 16 score rows).
struct AttnChunkArgs {
    const __half *k_base;
    uint64_t head_stride;
    uint32_t cap, ctx, head0, nheads, group, n_q;
    uint32_t ntok, q_stride, nsplit, rounds_per_split, few;
    const __half *k_own, *v_own;
    uint32_t own_stride;
    __half *out;
    uint32_t out_stride;
    const __half *q;
    float *part;
    const uint64_t *home;
};
// ctx and the plan's token count, query heads per kv head and kv heads of the model -> the deal of the positions
void attn_chunk_deal(uint32_t ctx, uint32_t plan_tokens, uint32_t group, uint32_t n_kv, uint32_t *nsplit, uint32_t *rounds_per_split);
hipError_t launch_attn_chunk(const AttnChunkArgs &a, hipStream_t st);
// merges every token's records in split order, writes the attention rows out[t][n_q * 128] (out_stride
// elements apart) and appends the tokens' K / V rows at positions ctx .. ctx + ntok - 1 of each kv head's cache home
hipError_t launch_attn_combine_chunk(const float *part, uint32_t nsplit, uint32_t ctx, uint32_t cap, const __half *qkv,
                                     uint32_t qkv_w, uint32_t n_q, uint32_t n_kv, uint32_t ntok, const uint64_t *home, __half *out,
                                     uint32_t out_stride, hipStream_t st);
// *dst = v (device word), in stream order
hipError_t launch_set_u32(uint32_t *dst, uint32_t v, hipStream_t st);
// dst[idx[r]][0..H) = src[r][0..H) for r < n (fp32 rows; H a multiple of 4; idx values are row numbers of dst)
hipError_t launch_scatter_rows(const float *src, const int32_t *idx, uint32_t n, uint32_t H, float *dst, hipStream_t st);
hipError_t launch_attn_decode(const AttnArgs &a, hipStream_t st);
// Merge the chunks of every query head in ascending order with the token's own position (score
// q.k_new / sqrt(128), value v_new), write the attention output (fp16 [n_q * 128]) and append the
// token's K and V rows at position ctx of each kv head's cache home (home[g] = address of that
// head's K row 0, device memory or device-visible pinned host memory).
hipError_t launch_attn_combine(const float *part, uint32_t chunk_cap, uint32_t ctx, const uint32_t *ctx_dev, uint32_t cap,
                               const __half *qkv, uint32_t n_q, uint32_t n_kv, const uint64_t *home, __half *out, hipStream_t st);
// out = h + the experts' rows weighted; rinv not null: also the RMS factor of every row stored, with launch_rinv's bits
hipError_t launch_combine(const __half *h, const float *y, const float *w, uint32_t M, uint32_t H, uint32_t top_k,
                          int residual, __half *out, float eps, float *rinv, hipStream_t st);
hipError_t launch_mfma_probe(int pi, int pk, int pj, float *out, hipStream_t st);
hipError_t launch_lds_tr_probe(const uint32_t *addr, uint16_t *out, hipStream_t st);

}  // namespace ps
