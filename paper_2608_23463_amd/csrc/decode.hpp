// Proxy-KV-cache decode (Eq. 19-21, Sec. 3.8): sizes, workspace layout and
// the launch sequences of the decode step and the cache append.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "../../include/proxyformer.h"

namespace pf {

struct DecodeDims {
  int B, d, nh, dh, M;
  int k[PF_MAX_LEVELS];
  int dl[PF_MAX_LEVELS + 1];  // d_0 = d_model ... d_M = d_model
  int64_t P;
  int esize;
  float eps;
  int append_rows;            // rows (sequence, block) compressed per append GEMM chunk
};

// Per-sequence positions, passed by value in kernel arguments: sequence b
// has n[b] cached rows and j[b] filled local slots; `write` marks the
// sequences whose rows a cache write stores (bit b). With ragged = 0 every
// sequence uses the scalar n and j.
struct DecodePos {
  int32_t n[PF_MAX_RAGGED_BATCH];
  int32_t j[PF_MAX_RAGGED_BATCH];
  uint64_t write;
  int32_t ragged;
};

constexpr size_t kStaticScratchBytes = (size_t)64 << 20;  // of the step without a workspace
constexpr int kDecodeMaxSplits = 256;   // cache-row slices per (sequence, head)
constexpr int kDecodeRowsPerSplit = 1024;  // most rows per slice (while kDecodeMaxSplits suffice)
constexpr int kDecodeSlices = 16;         // slices aimed at below that
constexpr int kAppendByRows = 64;         // largest batch whose one-block appends are planned by rows
constexpr int kAppendPlanBlocks = 8;      // and the batch they are planned as

struct DecodeWs {
  int splits_cap;                   // cache slices per (sequence, head) the partials hold
  int rows_cap;                     // (sequence, block) rows per append chunk
  size_t q, alpha, attn;            // [B, d], fp32 [B, h], [B, d]
  size_t part_m, part_l, part_acc;  // fp32 partial softmax states
  size_t z[PF_MAX_LEVELS];          // append: compression level outputs (j = 1..M)
  size_t gemm;
  size_t bytes;
  bool lean;                        // the plan with the least scratch (decode_step_ws)
};

int decode_dims(const pf_decode_config* c, DecodeDims* d, const char** why);
// Workspace of every decode call (steps and appends of any size).
DecodeWs decode_ws(const DecodeDims& d);
// Scratch of one decode step whose longest cache holds n_max rows: its own
// slice partials and the append of one block per sequence (smaller than
// decode_ws; the layout differs, the kernels are the same). Where that passes
// kStaticScratchBytes, the lean plan: slices of at least 1,024 rows, and an
// append without split-K partials (or, of a batch whose bits must not depend
// on it, in passes of as many blocks as fit).
DecodeWs decode_step_ws(const DecodeDims& d, int64_t n_max);
// The general workspace with the plan that decode_step_ws has for this step,
// so a step gives the same bits with a workspace and without. (Where the lean
// plan sets in, its slices are the faster ones: 512 sequences of 32 heads x
// 2,000 rows 1,684 us a step, 1,739 in slices of 128.) A step beyond that
// scratch on either plan takes the full one.
DecodeWs decode_ws_for_step(const DecodeDims& d, int64_t n_max);
// Rows per slice of a cache of n rows: the power of two from 128 (what a
// workgroup reads at once) to 1,024 that gives about kDecodeSlices slices, and
// beyond kDecodeMaxSplits * 1,024 rows what kDecodeMaxSplits slices take. It
// depends on the sequence's length alone, not on the batch, so a step gives a
// sequence the same bits alone and in any batch on the full plan. One sequence of 8 heads over
// 1,500 rows ran as 24 workgroups of eight dependent reads each in slices of
// 1,024: with the other changes of the step 26.2 us, 15.5 now; 32 sequences of
// 16 heads x 1,500, 4,000 and 9,000 rows are unchanged (55, 121, 224 us).
// `lean`: 1,024 rows at least, the fewest partials.
__host__ __device__ inline int slice_rows(int n, bool lean) {
  int c = lean ? kDecodeRowsPerSplit : 128;
  while (c < kDecodeRowsPerSplit && n > kDecodeSlices * c) c *= 2;
  if (n > kDecodeMaxSplits * c) c = (n - 1) / kDecodeMaxSplits + 1;
  return c;
}
// Cache slices the decode attention cuts n rows into, and their length.
void split_plan(int64_t n, bool lean, int* splits, int* chunk);

// Offset (elements) of 16-byte chunk c of row r in the projection kernels'
// staged A, [rows][d] with the chunks XOR-swizzled by row. The matrix tile has
// 32 rows whatever the batch: those past the `rows` staged ones (a power of
// two) repeat them, so no access leaves the staged block.
template <typename T>
__host__ __device__ constexpr int staged_offset(int r, int c, int rows, int d) {
  const int row = r & (rows - 1);
  return row * d + (c ^ (row & 7)) * (16 / (int)sizeof(T));
}
// LDS of a projection workgroup: the staged rows, four 32 x 33 partial tiles
// and a spare row of 32.
template <typename T>
constexpr size_t decode_small_gemm_lds(int d, int rows = 32) {
  return (size_t)rows * d * sizeof(T) + 4 * 32 * 33 * sizeof(float) + 32 * sizeof(float);
}

// `pos` carries the per-sequence positions when st.n_seq / st.j_seq are set;
// W is the scratch layout inside ws.
template <typename T>
hipError_t decode_step_run(const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                           const pf_decode_state& st, const DecodePos& pos, const void* x_t, void* y_t, char* ws,
                           hipStream_t stream);

// Prefill (parallel form of the generation block over a chunk of T tokens):
// buffers placed after the decode workspace, which the chunk's append uses.
struct PrefillWs {
  size_t u;      // [B*T, d] RMSNorm output, later the attention output A
  size_t q, k;   // [B, h, T, dh]
  size_t vt;     // values of the chunk: bf16 [B, h, T, dh]; fp32 [B, h, dh, ld_t] (token-contiguous)
  size_t alpha;  // fp32 [B*T, h]
  size_t vct;    // fp32 only: [B, h, dh, ld_c] cached values, row-contiguous (bf16: empty)
  size_t xc;     // [B, T/P*P, d] complete blocks, gathered when T % P != 0
  size_t gemm;   // split-K partials of the chunk's GEMMs
  size_t bytes;
  int64_t ld_t, ld_c;
};

// Limits of a prefill of T tokens with cache capacity n_cap (NULL: fits).
const char* prefill_limits(const DecodeDims& d, int64_t T, int64_t n_cap);
PrefillWs prefill_ws(const DecodeDims& d, int64_t T, int64_t n_cap);

template <typename T>
hipError_t prefill_run(const DecodeDims& d, const pf_decode_weights* w, const pf_decode_state& st, const void* x,
                       int64_t n_tok, void* y, char* ws, hipStream_t stream);

template <typename T>
hipError_t cache_append_run(const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                            const pf_decode_state& st, const DecodePos& pos, const void* x_blocks, int64_t nblk,
                            char* ws, hipStream_t stream);

}  // namespace pf
