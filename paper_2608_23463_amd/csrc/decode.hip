// Proxy-KV-cache decode step and block-triggered append (Eq. 19-21, Sec. 3.8).
//
// Step (one token per sequence, the batch in lockstep), four launches (three
// for up to 1,024 channels of the batch over few slices, which merge in the
// fourth):
//  1. decode_proj_kernel: u = RMSNorm(x) * gamma formed on the fly and
//     multiplied by W_q, W_k, W_v and W_alpha (one 32-column block of the
//     concatenated outputs per workgroup, MFMA over 32 batch rows): q to
//     scratch, k and v straight into slot j of the local block, alpha through
//     a sigmoid. It also stores x into block slot j.
//  2. decode_attn_kernel: the only HBM-heavy step. Cache rows of every
//     (sequence, head) are cut into slices; a workgroup streams one slice of
//     K and V with 16-byte loads (eight lanes per 64-channel row), keeps an
//     online softmax per row slot, and writes an unnormalised partial
//     (max, sum, weighted values). One extra slice per (sequence, head)
//     handles the current block's slots 0..j.
//  3. decode_combine_kernel: merges the cache slices in a fixed order (A_h),
//     normalises the local part (A_x) and forms A = A_x + alpha * A_h.
//  4. the projection kernel of step 1 in its second form:
//     y = x + A W_o^T + b_o.
// Append: compression GEMMs over whole blocks (the block is a zero-copy
// [rows, P*d] view), then the K/V proxy maps write straight into cache row n.
#include <algorithm>
#include <mutex>
#include <utility>
#include <vector>
#include <cmath>
#include <cstring>

#include "decode.hpp"
#include "epilogues.hpp"
#include "layer.hpp"
#include "runner.hpp"

namespace pf {

int decode_dims(const pf_decode_config* c, DecodeDims* d, const char** why) {
  *why = nullptr;
  memset(d, 0, sizeof(*d));  // the sizing memo compares whole structs
  if (!c) return *why = "config is NULL", PF_ERR_INVALID_ARG;
  if (c->dtype != PF_FP32 && c->dtype != PF_BF16) return *why = "dtype must be PF_FP32 or PF_BF16", PF_ERR_INVALID_ARG;
  if (c->batch < 1 || c->d_model < 1 || c->n_heads < 1 || c->head_dim < 1)
    return *why = "sizes must be >= 1", PF_ERR_INVALID_ARG;
  if ((int64_t)c->n_heads * c->head_dim != c->d_model) return *why = "n_heads * head_dim must equal d_model", PF_ERR_INVALID_ARG;
  if (c->n_levels < 1 || c->n_levels > PF_MAX_LEVELS) return *why = "n_levels must be in 1..4", PF_ERR_INVALID_ARG;
  if (!(c->rms_eps >= 0.0f)) return *why = "rms_eps must be >= 0", PF_ERR_INVALID_ARG;
  d->B = c->batch;
  d->d = c->d_model;
  d->nh = c->n_heads;
  d->dh = c->head_dim;
  d->M = c->n_levels;
  d->P = 1;
  for (int j = 0; j < d->M; ++j) {
    if (c->factors[j] < 1) return *why = "every factor k_j must be >= 1", PF_ERR_INVALID_ARG;
    d->k[j] = c->factors[j];
    d->P *= c->factors[j];
    if (d->P > (1 << 16)) return *why = "block size P too large", PF_ERR_INVALID_ARG;
  }
  d->dl[0] = d->d;
  for (int j = 1; j < d->M; ++j) d->dl[j] = c->level_dims[j - 1] > 0 ? c->level_dims[j - 1] : d->d;
  d->dl[d->M] = d->d;
  d->esize = c->dtype == PF_BF16 ? 2 : 4;
  d->eps = c->rms_eps;
  if (d->dh != 64 && d->dh != 128) return *why = "head_dim must be 64 or 128", PF_ERR_UNSUPPORTED;
  if ((int64_t)d->d * d->esize > 4096)
    return *why = "d_model * element size must be at most 4096 bytes (32 staged rows in LDS)", PF_ERR_UNSUPPORTED;
  for (int j = 0; j <= d->M; ++j)
    if (d->dl[j] % 8 != 0) return *why = "every channel width must be a multiple of 8", PF_ERR_UNSUPPORTED;
  // the append's compression GEMMs take rows of k_j * d_{j-1} elements (at
  // most 8 MiB: a GEMM tile's 256 rows share one 32-bit buffer range)
  for (int j = 0; j < d->M; ++j)
    if ((int64_t)d->k[j] * d->dl[j] * d->esize > kMaxGemmRowBytes)
      return *why = "a grouped row k_j * d_{j-1} * element size exceeds 8 MiB", PF_ERR_UNSUPPORTED;
  const int64_t lvl1_rows_per_block = d->P / d->k[0];
  d->append_rows = (int)std::max<int64_t>(1, std::min<int64_t>(4096, 65536 / lvl1_rows_per_block));
  return PF_OK;
}

// Offsets of every scratch buffer except the split-K partials: the slice
// partials of up to splits_cap cache slices per (sequence, head), and the
// append's level outputs for up to rows_cap (sequence, block) rows per chunk.
static DecodeWs decode_ws_layout(const DecodeDims& d, int splits_cap, int rows_cap) {
  DecodeWs w{};
  w.splits_cap = splits_cap;
  w.rows_cap = rows_cap;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align256(bytes);
    return o;
  };
  const size_t es = d.esize;
  w.q = take((size_t)d.B * d.d * es);
  w.alpha = take((size_t)d.B * d.nh * 4);
  w.attn = take((size_t)d.B * d.d * es);
  const size_t nparts = (size_t)d.B * d.nh * (splits_cap + 1);
  w.part_m = take(nparts * 4);
  w.part_l = take(nparts * 4);
  w.part_acc = take(nparts * d.dh * 4);
  int64_t per_block = d.P;  // rows of level j per block
  for (int j = 1; j <= d.M; ++j) {
    per_block /= d.k[j - 1];
    w.z[j] = take((size_t)rows_cap * per_block * d.dl[j] * es);
  }
  w.gemm = off;
  w.bytes = off;
  return w;
}

// ---- kernels ------------------------------------------------------------------

// ---- small-batch projections (steps 1 and 3) ------------------------------------
//
// out[b, c] for 32 rows b (blockIdx.y) and one block of 32 output columns
// (blockIdx.x) of A W^T, A = [B, d]: MFMA with the batch rows as the M side.
// The 32 rows of A are staged once in LDS (step 1: u = RMSNorm(x) * gamma,
// rounded to the activation type as a stored u would be), with 16-byte chunks
// XOR-swizzled by row so fragment reads are conflict-free. Each of the four
// waves takes a quarter of K; its weight fragments are requested eight
// k-steps ahead, and the four partial tiles are summed in LDS in a fixed order.
struct DecodeProjParams {
  const void* x;        // [B, d]: the token input (RMSNorm input; the residual of step 3)
  const void* a;        // [B, d]: step 3's A (attention output)
  const void* gamma;    // [d] RMSNorm scale (step 1)
  const void* w[4];     // step 1: W_q, W_k, W_v [d, d] and W_alpha [h, d]; step 3: W_o
  const void* bias[4];  // NULL = 0
  int width[4];         // output width of each matrix (d, d, d, h; step 3: d)
  int B, d, nh, dh;
  int64_t P;
  int j;                // local slot of the new token (lockstep)
  float eps;
  void* q;              // [B, d]
  void* k_loc;          // [B, h, P, dh]
  void* v_loc;
  float* alpha;         // [B, h]
  void* x_blk;          // [B, P, d]
  void* y;              // step 3: [B, d]
  DecodePos pos;        // per-sequence slots when pos.ragged
  __device__ __forceinline__ int slot(int b) const { return pos.ragged ? pos.j[b] : j; }
};

struct DecodeAttnParams {
  const void* q;       // [B, d]
  const void* kc;      // [B, h, n_cap, dh]
  const void* vc;
  const void* kl;      // [B, h, P, dh]
  const void* vl;
  float* part_m;       // [B*h, S+1]
  float* part_l;
  float* part_acc;     // [B*h, S+1, dh]
  const float* alpha;  // [B, h]
  void* attn;          // [B, d] output A
  int64_t n, n_cap, P;
  int j;               // local slots 0..j are valid
  int nh, splits, chunk;
  bool lean;
  float scale_log2;
  DecodePos pos;       // per-sequence n and j when pos.ragged
};

// out[u] = A[b, h, c0 + u * kStride] = A_x + alpha * A_h from the partials of
// one (sequence, head): cache slices merged in a fixed order with a running
// maximum (A_h, zero without cached rows), local slice normalised (A_x). The
// loads of up to kBatch slices, the local part and alpha go out together
// before any is used, so a step with up to kBatch slices waits for memory once.
// The multiply-adds are written out: every caller gets the same bits, so a
// sequence's result does not depend on the batch it is decoded in.
template <int DH, int kC, int kStride, int kBatch>
__device__ __forceinline__ void merge_partials(const DecodeAttnParams& p, int bh, int c0, float (&out)[kC]) {
  const int64_t base = (int64_t)bh * (p.splits + 1);
  const float al = p.alpha[bh];  // alpha is [B, h] as the partials are
  const float lx = p.part_l[base + p.splits];
  float ax[kC];
#pragma unroll
  for (int u = 0; u < kC; ++u) ax[u] = p.part_acc[(base + p.splits) * DH + c0 + kStride * u];
  float mrun = -INFINITY, lrun = 0.0f, arun[kC];
#pragma unroll
  for (int u = 0; u < kC; ++u) arun[u] = 0.0f;
  for (int s0 = 0; s0 < p.splits; s0 += kBatch) {
    float m[kBatch], l[kBatch], a[kBatch][kC];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int s = min(s0 + i, p.splits - 1);
      m[i] = p.part_m[base + s];
      l[i] = p.part_l[base + s];
#pragma unroll
      for (int u = 0; u < kC; ++u) a[i][u] = p.part_acc[(base + s) * DH + c0 + kStride * u];
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (s0 + i >= p.splits || m[i] == -INFINITY) continue;
      const float mn = fmaxf(mrun, m[i]);
      const float f0 = fast_exp2(mrun - mn), f1 = fast_exp2(m[i] - mn);
      lrun = fmaf(lrun, f0, l[i] * f1);
#pragma unroll
      for (int u = 0; u < kC; ++u) arun[u] = fmaf(arun[u], f0, a[i][u] * f1);
      mrun = mn;
    }
  }
#pragma unroll
  for (int u = 0; u < kC; ++u) out[u] = fmaf(al, mrun == -INFINITY ? 0.0f : arun[u] / lrun, ax[u] / lx);
}

// RPW: rows that each of the four waves stages, 8 for a full block of 32
// sequences, 4, 2 or 1 where the batch ends within 16, 8 or 4: the rows past them
// would be copies of the last, and their loads, norms and instructions are
// most of what precedes the first product (a step at d = 1024 over 500 rows: 8
// sequences 27.8 -> 22.2 us, 12 sequences 29.6 -> 25.7). A row's arithmetic is
// the same in all. The matrix tile keeps 32
// rows; those past the staged ones repeat them and are not stored.
//
// MERGE (the output map, head dimension MERGE): A is not read but merged here
// from the slice partials, rounded to the activation type as the stored A
// would be.
template <typename T, bool PROJ, int CPL, int RPW, int MERGE>
__global__ void __launch_bounds__(256) decode_small_gemm_kernel(const DecodeProjParams p, const DecodeAttnParams ap) {
  typedef Mma<T> MM;
  constexpr int kV = 16 / sizeof(T);  // elements per 16-byte chunk
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  T* a_s = reinterpret_cast<T*>(dyn);                                     // [4 RPW][d], swizzled chunks
  constexpr int kRowsA = 4 * RPW;
  float* red = reinterpret_cast<float*>(dyn + (size_t)kRowsA * p.d * sizeof(T));  // [4][32 * 33]
  float* inv_s = red + 4 * 32 * 33;                                       // [32]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, l32 = lane & 31;
  const int b0 = blockIdx.y * 32;
  const int cpr = p.d / kV;  // chunks per row
  // which matrix this column block belongs to (every width but the last is
  // a multiple of 32, so a block never straddles two matrices)
  int seg = 0, cs = blockIdx.x * 32;
  if constexpr (PROJ) {
    while (seg < 3 && cs >= p.width[seg]) {
      cs -= p.width[seg];
      ++seg;
    }
  }
  const int width = p.width[seg];
  const T* x = reinterpret_cast<const T*>(p.x);
  auto a_slot = [&](int r, int c) { return a_s + staged_offset<T>(r, c, kRowsA, p.d); };

  // weight fragments of this wave's quarter of K, eight k-steps at a time
  const int col = cs + l32;  // B column = weight row
  const bool col_ok = col < width;
  const T* wrow = reinterpret_cast<const T*>(p.w[seg]) + (int64_t)(col_ok ? col : 0) * p.d;
  // stage the rows of A: wave w takes rows RPW w .. RPW w + RPW - 1 (CPL 16-byte
  // chunks per lane and row), every load issued before any is used
  const T* src = PROJ ? x : reinterpret_cast<const T*>(p.a);
  u32x4 raw[RPW][CPL];
#pragma unroll
  for (int rr = 0; rr < RPW && MERGE == 0; ++rr)
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int b = min(b0 + wave * RPW + rr, p.B - 1), c = min(lane + 64 * i, cpr - 1);
      raw[rr][i] = ld16(src + (int64_t)b * p.d + c * kV);
    }
  // every other global read of the kernel goes out before the first use
  u32x4 graw[CPL];  // RMSNorm scale: the same chunks for every row
#pragma unroll
  for (int i = 0; i < CPL; ++i)
    graw[i] = PROJ ? ld16(reinterpret_cast<const T*>(p.gamma) + min(lane + 64 * i, cpr - 1) * kV)
                   : u32x4{0u, 0u, 0u, 0u};
  const int kq = p.d / 4, kbeg = wave * kq, nsteps = kq / 16;
  constexpr int kChunk = 16;  // k-steps of weight fragments requested at once
  typename MM::frag wf[kChunk];
  auto fetch_w = [&](int chunk) {  // unconditional (clamped) loads stay in flight together
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
      const int st = min(chunk * kChunk + i, nsteps - 1);
      wf[i] = MM::load(wrow + kbeg + st * 16 + g * 8);
    }
  };
  fetch_w(0);
  // the epilogue's reads (bias, residual) go out with the first requests too
  const T* bias = reinterpret_cast<const T*>(p.bias[seg]);
  float bv[4], xr[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int o = tid + u * 256, rr = o >> 5, cc = o & 31;
    const int b = min(b0 + rr, p.B - 1), c = min(cs + cc, width - 1);
    const float braw = to_f32((bias ? bias : x)[c]);  // unconditional read, no branch
    bv[u] = bias ? braw : 0.0f;
    xr[u] = PROJ ? 0.0f : to_f32(x[(int64_t)b * p.d + c]);
  }
  if constexpr (MERGE != 0) {
    // rows past the batch keep what the LDS held: their results are not stored
    for (int it = tid; it < p.B * (p.d / 2); it += 256) {
      const int r = it / (p.d / 2), c = 2 * (it - r * (p.d / 2));
      float v[2];
      merge_partials<MERGE, 2, 1, 16>(ap, r * ap.nh + c / MERGE, c % MERGE, v);
      T* slot = a_slot(r, c / kV) + c % kV;
      slot[0] = from_f32<T>(v[0]);
      slot[1] = from_f32<T>(v[1]);
    }
  } else {
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr) {
      const int r = wave * RPW + rr, b = b0 + r;
      float inv = 1.0f;
      if constexpr (PROJ) {
        float ss = 0.0f;
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
          const T* v = reinterpret_cast<const T*>(&raw[rr][i]);
          if (lane + 64 * i < cpr)
#pragma unroll
            for (int e = 0; e < kV; ++e) ss += to_f32(v[e]) * to_f32(v[e]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
        inv = 1.0f / sqrtf(ss / (float)p.d + p.eps);
      }
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const int c = lane + 64 * i;
        if (c >= cpr) continue;
        u32x4 v = raw[rr][i];
        if (b >= p.B) v = u32x4{0u, 0u, 0u, 0u};
        if constexpr (PROJ) {
          if (blockIdx.x == 0 && b < p.B)  // x into block slot j
            st16(reinterpret_cast<T*>(p.x_blk) + ((int64_t)b * p.P + p.slot(b)) * p.d + c * kV, v);
          const T* xv = reinterpret_cast<const T*>(&v);
          const T* gv = reinterpret_cast<const T*>(&graw[i]);
          T uv[kV];
#pragma unroll
          for (int e = 0; e < kV; ++e) uv[e] = from_f32<T>(to_f32(xv[e]) * inv * to_f32(gv[e]));
          v = *reinterpret_cast<const u32x4*>(uv);
        }
        st16(a_slot(r, c), v);
      }
    }
  }
  __syncthreads();

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  for (int chunk = 0; chunk * kChunk < nsteps; ++chunk) {
    if (chunk > 0) fetch_w(chunk);  // d > 1024 (bf16) only
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {  // fully unrolled: wf stays in registers
      const int st = chunk * kChunk + i;
      if (st >= nsteps) continue;
      const int k = kbeg + st * 16 + g * 8;
      typename MM::frag af;
      if constexpr (sizeof(T) == 2) {
        af = *reinterpret_cast<const typename MM::frag*>(a_slot(l32, k / kV));
      } else {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(a_slot(l32, k / kV));
        const f32x4 hi = *reinterpret_cast<const f32x4*>(a_slot(l32, k / kV + 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          af[e] = lo[e];
          af[e + 4] = hi[e];
        }
      }
      typename MM::frag bf = wf[i];
      if (!col_ok) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bf[e] = (T)0.0f;
      }
      acc = MM::mma(af, bf, acc);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave * 32 * 33 + acc_row(r, lane) * 33 + l32] = acc[r];
  __syncthreads();
  // four outputs per thread
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int o = tid + u * 256, rr = o >> 5, cc = o & 31;
    const int b = b0 + rr, c = cs + cc;
    if (b >= p.B || c >= width) continue;
    const int ri = rr * 33 + cc;
    const float v = ((red[ri] + red[32 * 33 + ri]) + red[2 * 32 * 33 + ri]) + red[3 * 32 * 33 + ri] + bv[u];
    if constexpr (PROJ) {
      if (seg == 0) {
        reinterpret_cast<T*>(p.q)[(int64_t)b * p.d + c] = from_f32<T>(v);
      } else if (seg < 3) {
        T* dst = reinterpret_cast<T*>(seg == 1 ? p.k_loc : p.v_loc);
        const int hd = c / p.dh, e = c - hd * p.dh;
        dst[(((int64_t)b * p.nh + hd) * p.P + p.slot(b)) * p.dh + e] = from_f32<T>(v);
      } else {
        p.alpha[(int64_t)b * p.nh + c] = sigmoidf(v);
      }
    } else {
      reinterpret_cast<T*>(p.y)[(int64_t)b * p.d + c] = from_f32<T>(xr[u] + v);
    }
  }
}

template <typename T, int DH>
__global__ void __launch_bounds__(256) decode_attn_kernel(const DecodeAttnParams p) {
  constexpr int kVec = 16 / sizeof(T);
  constexpr int LPR = DH / kVec;        // lanes per row
  constexpr int RPW = kWave / LPR;      // rows per wave per load
  constexpr int U = 4;                  // row groups in flight per lane
  const int s = blockIdx.x;
  const int bh = blockIdx.y;
  const int b = bh / p.nh, h = bh % p.nh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, rslot = lane / LPR;

  const T* base_k;
  const T* base_v;
  int64_t r0, r1;
  if (s < p.splits) {
    base_k = reinterpret_cast<const T*>(p.kc) + (int64_t)bh * p.n_cap * DH;
    base_v = reinterpret_cast<const T*>(p.vc) + (int64_t)bh * p.n_cap * DH;
    const int64_t n = p.pos.ragged ? p.pos.n[b] : p.n;
    const int chunk = p.pos.ragged ? slice_rows((int)n, p.lean) : p.chunk;
    r0 = (int64_t)s * chunk;
    r1 = std::min<int64_t>(n, r0 + chunk);  // empty slices leave m = -inf
  } else {
    base_k = reinterpret_cast<const T*>(p.kl) + (int64_t)bh * p.P * DH;
    base_v = reinterpret_cast<const T*>(p.vl) + (int64_t)bh * p.P * DH;
    r0 = 0;
    r1 = (p.pos.ragged ? p.pos.j[b] : p.j) + 1;
  }

  float qv[kVec];
  {
    const T* qp = reinterpret_cast<const T*>(p.q) + (int64_t)b * p.nh * DH + h * DH + sub * kVec;
#pragma unroll
    for (int i = 0; i < kVec; ++i) qv[i] = to_f32(qp[i]) * p.scale_log2;
  }
  float mrun = -INFINITY, lrun = 0.0f;
  float acc[kVec];
#pragma unroll
  for (int i = 0; i < kVec; ++i) acc[i] = 0.0f;

  const int64_t step = (int64_t)4 * U * RPW;
  for (int64_t rb = r0 + (int64_t)wave * U * RPW; rb < r1; rb += step) {
    u32x4 kraw[U], vraw[U];
    bool valid[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = rb + u * RPW + rslot;
      valid[u] = row < r1;
      u32x4 zero = {0u, 0u, 0u, 0u};
      kraw[u] = valid[u] ? ld16(base_k + row * DH + sub * kVec) : zero;
      vraw[u] = valid[u] ? ld16(base_v + row * DH + sub * kVec) : zero;
    }
    float sc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T* kt = reinterpret_cast<const T*>(&kraw[u]);
      float dot = 0.0f;
#pragma unroll
      for (int i = 0; i < kVec; ++i) dot += qv[i] * to_f32(kt[i]);
#pragma unroll
      for (int off = 1; off < LPR; off <<= 1) dot += __shfl_xor(dot, off);
      sc[u] = valid[u] ? dot : -INFINITY;
    }
    float mt = sc[0];
#pragma unroll
    for (int u = 1; u < U; ++u) mt = fmaxf(mt, sc[u]);
    const float mnew = fmaxf(mrun, mt);
    if (mnew == -INFINITY) continue;
    const float alpha = fast_exp2(mrun - mnew);
    mrun = mnew;
    lrun *= alpha;
#pragma unroll
    for (int i = 0; i < kVec; ++i) acc[i] *= alpha;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float pu = fast_exp2(sc[u] - mnew);
      lrun += pu;
      const T* vt = reinterpret_cast<const T*>(&vraw[u]);
#pragma unroll
      for (int i = 0; i < kVec; ++i) acc[i] += pu * to_f32(vt[i]);
    }
  }

  // Merge of the row slots (fixed order): a butterfly over the RPW slots of a
  // wave, then the four waves through LDS. (Through LDS alone, 4 * RPW slots
  // one after the other, the tail took longer than a 128-row slice's reads.)
#pragma unroll
  for (int off = LPR; off < kWave; off <<= 1) {
    const float mo = __shfl_xor(mrun, off), lo = __shfl_xor(lrun, off);
    const float mn = fmaxf(mrun, mo);
    const float f0 = mrun == -INFINITY ? 0.0f : fast_exp2(mrun - mn);
    const float f1 = mo == -INFINITY ? 0.0f : fast_exp2(mo - mn);
    lrun = lrun * f0 + lo * f1;
#pragma unroll
    for (int i = 0; i < kVec; ++i) acc[i] = acc[i] * f0 + __shfl_xor(acc[i], off) * f1;
    mrun = mn;
  }
  __shared__ float sm[4];
  __shared__ float sl[4];
  __shared__ float sacc[4][DH];
  if (lane == 0) {
    sm[wave] = mrun;
    sl[wave] = lrun;
  }
  if (rslot == 0) {
#pragma unroll
    for (int i = 0; i < kVec; ++i) sacc[wave][sub * kVec + i] = acc[i];
  }
  __syncthreads();
  if (tid < DH) {
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sm[i]);
    float l = 0.0f, a = 0.0f;
    if (mx != -INFINITY) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float f = fast_exp2(sm[i] - mx);
        l += sl[i] * f;
        a += sacc[i][tid] * f;
      }
    }
    const int64_t pidx = (int64_t)bh * (p.splits + 1) + s;
    p.part_acc[pidx * DH + tid] = a;
    if (tid == 0) {
      p.part_m[pidx] = mx;
      p.part_l[pidx] = l;
    }
  }
}

// Merge of the partials of every (sequence, head): one wave per (sequence,
// head), DH / 64 channels per lane; see merge_partials.
template <typename T, int DH>
__global__ void __launch_bounds__(256) decode_combine_kernel(const DecodeAttnParams p, int nbh) {
  const int bh = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (bh >= nbh) return;
  const int b = bh / p.nh, h = bh % p.nh, lane = threadIdx.x & 63;
  float v[DH / 64];
  merge_partials<DH, DH / 64, 64, 32>(p, bh, lane, v);
  T* out = reinterpret_cast<T*>(p.attn) + (int64_t)b * p.nh * DH + h * DH;
#pragma unroll
  for (int u = 0; u < DH / 64; ++u) out[lane + 64 * u] = from_f32<T>(v[u]);
}

// Proxy K/V rows into the cache: row rr = r0 + r is (sequence rr / nblk,
// block rr % nblk) and lands at cache row n0 + block (per-sequence n and a
// write mask with ragged positions).
template <typename T>
struct EpiCache {
  T* cache;
  const T* bias;
  int64_t n_cap, n0, nblk, r0;
  int nh, dh;
  DecodePos pos;
  // cache row of (sequence b, block i), or -1 when the sequence is not written
  __device__ __forceinline__ int64_t row_of(int64_t b, int64_t i) const {
    if (!pos.ragged) return n0 + i;
    return ((pos.write >> b) & 1) ? pos.n[b] + i : -1;
  }
  __device__ __forceinline__ void operator()(int r, int c, float v) const {
    if (bias) v += to_f32(bias[c]);
    const int64_t rr = r0 + r;
    const int64_t b = rr / nblk, i = rr - b * nblk;
    const int64_t row = row_of(b, i);
    if (row < 0) return;
    const int hd = c / dh, e = c - hd * dh;
    cache[(((int64_t)b * nh + hd) * n_cap + row) * dh + e] = from_f32<T>(v);
  }
  __device__ __forceinline__ void vec8(int r, int c, const float* v0) const {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v0[e] + (bias ? to_f32(bias[c + e]) : 0.0f);
    const int64_t rr = r0 + r;
    const int64_t b = rr / nblk, i = rr - b * nblk;
    const int64_t row = row_of(b, i);
    if (row < 0) return;
    const int hd = c / dh, e0 = c - hd * dh;
    store8(cache + (((int64_t)b * nh + hd) * n_cap + row) * dh + e0, v);
  }
};

template <typename T>
struct GemmGrouped<EpiCache<T>> : std::true_type {};
template <typename T>
struct EpiByRef<EpiCache<T>> : std::true_type {};

// ---- launch sequences ---------------------------------------------------------

// Blocks per pass of an append planned by rows: all of them while the split-K
// partials of a pass stay within 32 MiB.
template <typename T>
static int append_pass(const DecodeDims& d) {
  size_t most = 0;
  auto need = [&](const GemmProblem* prs, int count) {
    const GemmPlan pl = plan_gemm<T>(prs, count, Runner::kPlanCUsGemm);
    size_t sum = 0;
    for (int i = 0; i < count && pl.splits > 1; ++i) sum += plan_partials(prs[i], pl) * sizeof(float);
    most = std::max(most, sum);
  };
  int64_t rows = kAppendPlanBlocks * d.P;
  for (int j = 0; j < d.M; ++j) {
    rows /= d.k[j];
    GemmProblem pr{};
    pr.M = (int)rows;
    pr.N = d.dl[j + 1];
    pr.K = d.k[j] * d.dl[j];
    need(&pr, 1);
  }
  GemmProblem kv[2];
  for (GemmProblem& pr : kv) {
    pr.M = kAppendPlanBlocks;
    pr.N = pr.K = d.d;
  }
  need(kv, 2);
  int pass = kAppendByRows;
  while (pass > kAppendPlanBlocks && most * (pass / kAppendPlanBlocks) > ((size_t)32 << 20)) pass /= 2;
  return pass;
}

// One block of each of up to kAppendByRows sequences: K is cut as for
// kAppendPlanBlocks of them, so a block's proxy, and with it every later step
// that reads it, has the same bits in any such batch. (Cut by the batch, 12
// sequences of d = 1024 with 8 x 8 tokens per block summed 8 slices where one
// sequence sums 16.) More blocks are cut by their number: there the partials
// of a fixed cut would cost more than the products. A lean step does not cut
// those at all.
template <typename T>
static void append_impl(Runner& run, const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                        const pf_decode_state& st, const DecodePos& pos, const void* x_blocks, int64_t nblk, char* ws) {
  const int64_t total = (int64_t)d.B * nblk;   // (sequence, block) rows of the [B*nblk, P*d] view
  const int64_t row_elems = d.P * d.d;
  const bool by_rows = nblk == 1 && d.B <= kAppendByRows;
  const int pass = by_rows ? std::min(W.rows_cap, append_pass<T>(d)) : W.rows_cap;
  auto plan = [&](const GemmProblem* prs, int count, int64_t rows_per_block) {
    if (by_rows) return plan_gemm_rows<T>(prs, count, (int)(kAppendPlanBlocks * rows_per_block), Runner::kPlanCUsGemm);
    GemmPlan pl = plan_gemm<T>(prs, count, Runner::kPlanCUsGemm);
    if (W.lean) pl.splits = 1;
    return pl;
  };
  for (int64_t r0 = 0; r0 < total; r0 += pass) {
    const int rows = (int)std::min<int64_t>(pass, total - r0);
    const T* zin = reinterpret_cast<const T*>(x_blocks) + r0 * row_elems;
    int64_t lvl_rows = (int64_t)rows * d.P;
    for (int j = 0; j < d.M; ++j) {  // compression C (Eq. 7, 16)
      lvl_rows /= d.k[j];
      GemmProblem pr{};
      pr.a = zin;
      pr.lda = (int64_t)d.k[j] * d.dl[j];
      pr.b = w->compress[j].w;
      pr.ldb = pr.lda;
      pr.M = (int)lvl_rows;
      pr.N = d.dl[j + 1];
      pr.K = (int)pr.lda;
      T* out = reinterpret_cast<T*>(ws + W.z[j + 1]);
      EpiLinear<T> e{out, pr.N, reinterpret_cast<const T*>(w->compress[j].b), nullptr, 0, nullptr};
      const GemmPlan pl = plan(&pr, 1, lvl_rows / rows);
      run.gemm_group<T, LAYOUT_K, LAYOUT_K>("append_compress_gemm", &pr, &e, 1, &pl);
      zin = out;
    }
    const pf_linear* maps[2] = {&w->k_proxy, &w->v_proxy};
    void* caches[2] = {st.k_cache, st.v_cache};
    GemmProblem prs[2];
    EpiCache<T> epis[2];
    for (int i = 0; i < 2; ++i) {  // cached rows K_p, V_p (Eq. 21), one launch
      GemmProblem pr{};
      pr.a = zin;
      pr.lda = d.d;
      pr.b = maps[i]->w;
      pr.ldb = d.d;
      pr.M = rows;
      pr.N = d.d;
      pr.K = d.d;
      prs[i] = pr;
      epis[i] = EpiCache<T>{reinterpret_cast<T*>(caches[i]), reinterpret_cast<const T*>(maps[i]->b), st.n_cap, st.n,
                            nblk, r0, d.nh, d.dh, pos};
    }
    const GemmPlan pl = plan(prs, 2, 1);
    run.gemm_group<T, LAYOUT_K, LAYOUT_K>("append_kv_gemm", prs, epis, 2, &pl);
  }
}

void split_plan(int64_t n, bool lean, int* splits, int* chunk) {
  *chunk = slice_rows((int)n, lean);
  *splits = n <= 0 ? 0 : (int)((n + *chunk - 1) / *chunk);
}

// Lets a kernel use up to 160 KB of dynamic LDS, once per (kernel, device).
static hipError_t allow_lds(const void* kernel) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static std::vector<std::pair<const void*, int>> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  for (const auto& k : done)
    if (k.first == kernel && k.second == dev) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess && done.size() < 2 * kMaxDevices) done.emplace_back(kernel, dev);
  return e;
}

// Chunks per lane and row of the staged A: 1, 2 or 4 (d * sizeof(T) <= 4096);
// rows per wave by the batch (at most four sequences merge in the output map).
template <typename T, bool PROJ, int MERGE = 0>
static hipError_t launch_small_gemm(dim3 grid, const DecodeProjParams& pp, const DecodeAttnParams& ap,
                                    hipStream_t stream) {
  const int cpr = pp.d * (int)sizeof(T) / 16;
  auto go = [&](auto cpl, auto rpw) {
    auto kern = decode_small_gemm_kernel<T, PROJ, decltype(cpl)::value, decltype(rpw)::value, MERGE>;
    hipError_t e = allow_lds(reinterpret_cast<const void*>(kern));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(256), decode_small_gemm_lds<T>(pp.d, 4 * decltype(rpw)::value), stream, pp, ap);
    return hipGetLastError();
  };
  auto by_rows = [&](auto cpl) {
    if (MERGE != 0 || pp.B <= 4) return go(cpl, std::integral_constant<int, 1>{});
    if constexpr (MERGE == 0) {
      if (pp.B <= 8) return go(cpl, std::integral_constant<int, 2>{});
      if (pp.B <= 16) return go(cpl, std::integral_constant<int, 4>{});
    }
    return go(cpl, std::integral_constant<int, MERGE ? 1 : 8>{});
  };
  if (cpr <= 64) return by_rows(std::integral_constant<int, 1>{});
  if (cpr <= 128) return by_rows(std::integral_constant<int, 2>{});
  if constexpr (MERGE == 0 || sizeof(T) == 4) return by_rows(std::integral_constant<int, 4>{});
  return hipErrorInvalidValue;  // the merge takes at most kMergeInOutChannels: two chunks in bf16
}

// The merge joins the output map while a workgroup's copy of the partials is
// at most kMergeInOutBytes (16 heads of 64 channels over 16 slices and the
// block's) and its threads merge at most two channel pairs each, one after the
// other: every workgroup repeats the merge, so it pays only while that is
// shorter than a launch. us a step, merged and not: one sequence of 8 heads x
// 1,500, 30,000 (65 KB) and 60,000 rows (126 KB) 14.4 / 16.4, 26.7 / 27.5 and
// 37.2 / 37.1; of 16 heads x 16,384 (72 KB) and 24,000 rows (106 KB) 29.0 /
// 29.4 and 35.0 / 32.5; past the second bound 2 sequences of 16 heads x 1,500
// rows 23.4 / 19.1.
constexpr int64_t kMergeInOutBytes = 72 << 10;
constexpr int kMergeInOutChannels = 1024;

template <typename T>
static void step_impl(Runner& run, const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                      const pf_decode_state& st, const DecodePos& pos, const void* x_t, void* y_t, char* ws) {
  T* q = reinterpret_cast<T*>(ws + W.q);
  float* alpha = reinterpret_cast<float*>(ws + W.alpha);
  T* attn = reinterpret_cast<T*>(ws + W.attn);
  const int rblocks = (d.B + 31) / 32;

  DecodeProjParams pp{};
  pp.x = x_t;
  pp.gamma = w->rms_gamma;
  const pf_linear* lin[4] = {&w->q, &w->k, &w->v, &w->alpha};
  for (int i = 0; i < 4; ++i) {
    pp.w[i] = lin[i]->w;
    pp.bias[i] = lin[i]->b;
    pp.width[i] = i < 3 ? d.d : d.nh;
  }
  pp.B = d.B;
  pp.d = d.d;
  pp.nh = d.nh;
  pp.dh = d.dh;
  pp.P = d.P;
  pp.j = st.j;
  pp.eps = d.eps;
  pp.q = q;
  pp.k_loc = st.k_loc;
  pp.v_loc = st.v_loc;
  pp.alpha = alpha;
  pp.x_blk = st.x_blk;
  pp.pos = pos;
  static_assert(decode_small_gemm_lds<T>(2048 * 2 / sizeof(T)) <= 160 * 1024, "staged rows fit the LDS");
  run.launch("decode_proj", [&] {
    const dim3 grid(3 * d.d / 32 + (d.nh + 31) / 32, rblocks);
    return launch_small_gemm<T, true>(grid, pp, DecodeAttnParams{}, run.stream);
  });

  int splits = 0, chunk = 0;
  if (pos.ragged) {  // each sequence is cut by its own length
    for (int b = 0; b < d.B; ++b) {
      int sb;
      split_plan(pos.n[b], W.lean, &sb, &chunk);
      splits = std::max(splits, sb);
    }
  } else {
    split_plan(st.n, W.lean, &splits, &chunk);
  }
  DecodeAttnParams ap{};
  ap.q = q;
  ap.kc = st.k_cache;
  ap.vc = st.v_cache;
  ap.kl = st.k_loc;
  ap.vl = st.v_loc;
  ap.part_m = reinterpret_cast<float*>(ws + W.part_m);
  ap.part_l = reinterpret_cast<float*>(ws + W.part_l);
  ap.part_acc = reinterpret_cast<float*>(ws + W.part_acc);
  ap.alpha = alpha;
  ap.attn = attn;
  ap.n = st.n;
  ap.n_cap = st.n_cap;
  ap.P = d.P;
  ap.j = st.j;
  ap.nh = d.nh;
  ap.splits = splits;
  ap.chunk = chunk;
  ap.lean = W.lean;
  ap.scale_log2 = (float)(1.4426950408889634 / std::sqrt((double)d.dh));
  ap.pos = pos;
  run.launch("decode_attn", [&] {
    const dim3 grid(splits + 1, d.B * d.nh);
    if (d.dh == 64)
      hipLaunchKernelGGL((decode_attn_kernel<T, 64>), grid, dim3(256), 0, run.stream, ap);
    else
      hipLaunchKernelGGL((decode_attn_kernel<T, 128>), grid, dim3(256), 0, run.stream, ap);
    return hipGetLastError();
  });
  DecodeProjParams op{};
  op.x = x_t;
  op.a = attn;
  op.w[0] = w->o.w;
  op.bias[0] = w->o.b;
  op.width[0] = d.d;
  op.B = d.B;
  op.d = d.d;
  op.y = y_t;
  const int64_t part_bytes = (int64_t)d.B * d.nh * (splits + 1) * (d.dh + 2) * 4;
  if (part_bytes <= kMergeInOutBytes && d.B * d.d <= kMergeInOutChannels && d.B <= 4) {
    run.launch("decode_out", [&] {
      const dim3 grid(d.d / 32);
      return d.dh == 64 ? launch_small_gemm<T, false, 64>(grid, op, ap, run.stream)
                        : launch_small_gemm<T, false, 128>(grid, op, ap, run.stream);
    });
    return;
  }
  run.launch("decode_combine", [&] {
    const int nbh = d.B * d.nh;
    const dim3 grid((nbh + 3) / 4);
    if (d.dh == 64)
      hipLaunchKernelGGL((decode_combine_kernel<T, 64>), grid, dim3(256), 0, run.stream, ap, nbh);
    else
      hipLaunchKernelGGL((decode_combine_kernel<T, 128>), grid, dim3(256), 0, run.stream, ap, nbh);
    return hipGetLastError();
  });
  run.launch("decode_out", [&] {
    const dim3 grid(d.d / 32, rblocks);
    return launch_small_gemm<T, false>(grid, op, ap, run.stream);
  });
}

// Dry run of an append of nblk blocks per sequence.
static void dry_append(Runner& dry, const DecodeDims& d, const DecodeWs& W, int64_t nblk) {
  pf_decode_weights nw{};
  pf_decode_state ns{};
  ns.n_cap = 1;
  const DecodePos np{};
  if (d.esize == 2)
    append_impl<bf16>(dry, d, W, &nw, ns, np, nullptr, nblk, nullptr);
  else
    append_impl<float>(dry, d, W, &nw, ns, np, nullptr, nblk, nullptr);
}

// Split-K need (bytes) of the GEMMs of a config, which the appends issue.
struct DecodeNeed {
  size_t any;   // an append of any size, and any step's
  size_t step;  // one block per sequence on the full plan
};

static DecodeNeed decode_need_of(const DecodeDims& d) {
  DecodeWs w{};
  Runner any(true), step(true);
  for (int rows = 1; rows <= d.append_rows; ++rows) {
    // one append of `rows` blocks of a single sequence exercises every chunk
    // size; a last chunk of one block, two chunks of one
    DecodeDims d1 = d;
    d1.B = 1;
    w.rows_cap = rows;
    dry_append(any, d1, w, std::max(rows, 2));
  }
  w.rows_cap = d.append_rows;
  dry_append(step, d, w, 1);
  return {std::max(any.gemm_need, step.gemm_need), step.gemm_need};
}

// Memoised for the last few configs of the thread: the sweep plans every
// append size (about 0.25 ms) and its result is asked for on every call;
// sessions of several configs may take turns.
static DecodeNeed decode_need(const DecodeDims& d) {
  constexpr int kMemo = 8;
  static thread_local DecodeDims seen[kMemo];
  static thread_local DecodeNeed need[kMemo];
  static thread_local int count = 0, next = 0;
  for (int at = 0; at < count; ++at)
    if (memcmp(&seen[at], &d, sizeof(d)) == 0) return need[at];
  const DecodeNeed n = decode_need_of(d);
  seen[next] = d;
  need[next] = n;
  next = (next + 1) % kMemo;
  count = std::min(count + 1, kMemo);
  return n;
}

DecodeWs decode_ws(const DecodeDims& d) {
  DecodeWs w = decode_ws_layout(d, kDecodeMaxSplits, d.append_rows);
  w.bytes = w.gemm + align256(decode_need(d).any);
  return w;
}

// Slice partials a step over up to n_max rows writes: as many as any length
// up to n_max is cut into.
static int step_splits(int64_t n_max, bool lean) {
  int splits, chunk;
  split_plan(n_max, lean, &splits, &chunk);
  return lean ? splits : std::max<int>(splits, (int)std::min<int64_t>(kDecodeSlices, (n_max + 127) / 128));
}

static DecodeWs full_step_ws(const DecodeDims& d, int64_t n_max) {
  DecodeWs w = decode_ws_layout(d, step_splits(n_max, false), std::min(d.append_rows, d.B));
  w.bytes = w.gemm + align256(decode_need(d).step);
  return w;
}

DecodeWs decode_step_ws(const DecodeDims& d, int64_t n_max) {
  DecodeWs w = full_step_ws(d, n_max);
  for (int pass = w.rows_cap; w.bytes > kStaticScratchBytes; pass /= 2) {
    w = decode_ws_layout(d, step_splits(n_max, true), pass);
    w.lean = true;
    Runner dry(true);
    dry_append(dry, d, w, 1);
    w.bytes = w.gemm + align256(dry.gemm_need);
    if (pass == 1 || d.B > kAppendByRows) break;
  }
  return w;
}

DecodeWs decode_ws_for_step(const DecodeDims& d, int64_t n_max) {
  const DecodeWs step = decode_step_ws(d, n_max);
  DecodeWs w = decode_ws(d);
  w.lean = step.lean && step.bytes <= kStaticScratchBytes;
  return w;
}

template <typename T>
hipError_t decode_step_run(const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                           const pf_decode_state& st, const DecodePos& pos, const void* x_t, void* y_t, char* ws,
                           hipStream_t stream) {
  Runner run(false, stream, reinterpret_cast<float*>(ws + W.gemm));
  step_impl<T>(run, d, W, w, st, pos, x_t, y_t, ws);
  return run.err;
}

template <typename T>
hipError_t cache_append_run(const DecodeDims& d, const DecodeWs& W, const pf_decode_weights* w,
                            const pf_decode_state& st, const DecodePos& pos, const void* x_blocks, int64_t nblk,
                            char* ws, hipStream_t stream) {
  Runner run(false, stream, reinterpret_cast<float*>(ws + W.gemm));
  append_impl<T>(run, d, W, w, st, pos, x_blocks, nblk, ws);
  return run.err;
}

template hipError_t decode_step_run<bf16>(const DecodeDims&, const DecodeWs&, const pf_decode_weights*,
                                          const pf_decode_state&, const DecodePos&, const void*, void*, char*,
                                          hipStream_t);
template hipError_t decode_step_run<float>(const DecodeDims&, const DecodeWs&, const pf_decode_weights*,
                                           const pf_decode_state&, const DecodePos&, const void*, void*, char*,
                                           hipStream_t);
template hipError_t cache_append_run<bf16>(const DecodeDims&, const DecodeWs&, const pf_decode_weights*,
                                           const pf_decode_state&, const DecodePos&, const void*, int64_t, char*,
                                           hipStream_t);
template hipError_t cache_append_run<float>(const DecodeDims&, const DecodeWs&, const pf_decode_weights*,
                                            const pf_decode_state&, const DecodePos&, const void*, int64_t, char*,
                                            hipStream_t);

}  // namespace pf
