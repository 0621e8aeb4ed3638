// LSTM layer whose weight matrix W = [W_ih | W_hh] (4H x (I + H)) takes a
// tile-based pattern (Sec. III-B applied to the LSTM's matrix products,
// Sec. IV-C): only the kept tiles of W are read by the gate products and only
// they receive a weight gradient. Every hidden unit is kept.
//
// The batch is padded to Bp columns, a multiple of 4, in every buffer of the
// workspace, so that all products run on 16-byte loads whatever the batch; the
// padding columns of h, x and dz are zeros.
//
// XH[(I + H)][T Bp] holds [x_t; h_{t-1}] of every step side by side, dZ[4H][T Bp]
// the gate derivatives. Where the inputs are whole tiles (I a multiple of the
// tile), the input tiles' products run once over all T Bp columns (the
// projection Zx, and dX after the backward walk), and a step multiplies the
// recurrent tiles only, on its own column block of XH or dZ; else a step
// multiplies the whole stacked input. A pointwise kernel per step adds the
// bias and updates the cell (forward) or forms dz_t (backward). One tile
// weight-gradient call over all T Bp columns gives dW = M * (dZ XH^T).
// Forward and backward on MI355X, against steps over the whole stacked input on
// the batch as it is: T 33, batch 15, 448 -> 320, p = 0.5, 64 x 64 tiles 4790 ->
// 648 us; T 12, batch 12, 736 -> 896, 32 x 32 tiles 1935 -> 308 us; T 35, batch
// 64, 1024 -> 1024, 64 x 64 tiles 1482 -> 1460 us (1444 with one chain of sums in
// the products over all steps, whose error was up to 1.6 times the former one).

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "ard_internal.hpp"

namespace ard {
namespace {

__device__ __forceinline__ float sgm(float x) { return 1.0f / (1.0f + expf(-x)); }

struct TileLstm {
  int32_t T, B, Bp, I, H;
  int64_t TB;           // T * Bp: columns of XH and dZ
  float* XH;            // [(I + H)][T Bp]
  float* Zx;            // [4H][T Bp] projection of the inputs, or NULL (the step product holds it)
  float* z;             // [4H][Bp] step gate product
  float* G;             // [T][4H][Bp] activated gates i, f, g, o
  float* C;             // [T + 1][H][Bp] cell states, C[0] = c0
  float* dZ;            // [4H][T Bp]
  float* dxh;           // step input derivative: [H][Bp], or [(I + H)][Bp] without Zx
  float* dc;            // [H][Bp] cell derivative carry
  float* part;          // split partial sums of the step products
  float* xh;            // [(I + H)][Bp] and [4H][Bp]: contiguous copies of a step's columns
  float* dz;            // of XH and dZ where those rows are too long for the loads' offsets, or NULL
  int32_t zsplits;      // partial sums of z (1: z itself holds the product)
  int32_t dsplits;      // partial sums of dxh (1: dxh itself holds the product)
};

size_t al256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Rows of XH and dZ of this many columns and more are not read in place by the
// step products (a part's 32 rows must lie within 2^31 bytes).
constexpr int64_t kMaxRow = int64_t{1} << 23;

struct TileLayout {
  int64_t Bp;
  size_t XH, z, G, C, dZ, dxh, dc, part, xh, dz, total;
};

TileLayout tile_layout(int64_t T, int64_t B, int64_t I, int64_t H) {
  TileLayout L;
  size_t off = 0;
  const int64_t K = I + H, Bp = (B + 3) / 4 * 4;
  L.Bp = Bp;
  L.XH = off;  off += al256(4 * K * T * Bp);
  L.z = off;   off += al256(4 * 4 * H * Bp);
  L.G = off;   off += al256(4 * T * 4 * H * Bp);
  L.C = off;   off += al256(4 * (T + 1) * H * Bp);
  L.dZ = off;  off += al256(4 * 4 * H * T * Bp);
  L.dxh = off; off += al256(4 * K * Bp);
  L.dc = off;  off += al256(4 * H * Bp);
  // the splits of the larger step product (4H or I + H rows)
  const int64_t rows = 4 * H > K ? 4 * H : K;
  L.part = off; off += al256(4 * kTilePartSplits * rows * Bp);
  L.xh = L.dz = off;
  if (T * Bp >= kMaxRow) {
    L.xh = off; off += al256(4 * K * Bp);
    L.dz = off; off += al256(4 * 4 * H * Bp);
  }
  L.total = off;
  return L;
}

TileLstm tile_args(const TileLayout& L, char* w, const ard_lstm_tile_desc* d) {
  TileLstm s = {};
  s.T = d->seq_len;
  s.B = d->batch;
  s.Bp = static_cast<int32_t>(L.Bp);
  s.I = d->input_size;
  s.H = d->hidden_size;
  s.TB = s.T * L.Bp;
  auto at = [w](size_t off) { return reinterpret_cast<float*>(w + off); };
  s.XH = at(L.XH);
  s.z = at(L.z);
  s.G = at(L.G);
  s.C = at(L.C);
  s.dZ = at(L.dZ);
  s.dxh = at(L.dxh);
  s.dc = at(L.dc);
  s.part = at(L.part);
  if (s.TB >= kMaxRow) {
    s.xh = at(L.xh);
    s.dz = at(L.dz);
  } else if (s.I % d->weight_plan->tile == 0) {
    s.Zx = s.dZ;  // the forward's projection lives where the backward puts dZ
  }
  s.zsplits = s.dsplits = 1;
  return s;
}

// Element e of a step product: the product buffer itself, or the sum of its
// split partial sums (n elements each) in split order, the loads of up to
// eight splits issued together.
__device__ __forceinline__ float step_val(const float* direct, const float* part, int splits, int64_t n, int64_t e) {
  static_assert(kTilePartSplits <= 8, "one group of loads");
  if (splits <= 1) return direct[e];
  float t[8], v = 0.0f;
#pragma unroll
  for (int u = 0; u < 8; ++u) t[u] = u < splits ? part[u * n + e] : 0.0f;
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (u < splits) v += t[u];
  return v;
}

// Row j and column b of element e of rows of Bp: 32-bit division where e
// allows it (a 64-bit one is some hundred instructions).
__device__ __forceinline__ void row_col(int64_t e, int32_t Bp, int64_t& j, int32_t& b) {
  j = (e >> 32) == 0 ? static_cast<int64_t>(static_cast<uint32_t>(e) / static_cast<uint32_t>(Bp)) : e / Bp;
  b = static_cast<int32_t>(e - j * Bp);
}

// Before the first step: X into the input rows of XH for every t (blockIdx.y),
// h0 (or 0) into the recurrent rows of XH's first column block, c0 (or 0) into
// C[0]; zeros in the padding columns.
__global__ void __launch_bounds__(256) tile_lstm_init_kernel(TileLstm s, const float* __restrict__ X,
                                                             const float* __restrict__ h0,
                                                             const float* __restrict__ c0) {
  const int32_t t = blockIdx.y;
  const int64_t IB = static_cast<int64_t>(s.I) * s.Bp, HB = static_cast<int64_t>(s.H) * s.Bp;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  int64_t j;
  int32_t b;
  row_col(e, s.Bp, j, b);
  if (e < IB) {  // X[t][k][b] -> XH[k][t Bp + b]
    const float x = b < s.B ? X[(static_cast<int64_t>(t) * s.I + j) * s.B + b] : 0.0f;
    s.XH[j * s.TB + static_cast<int64_t>(t) * s.Bp + b] = x;
    if (s.xh && t == 0) s.xh[e] = x;
  }
  if (t == 0 && e < HB) {
    const bool in = b < s.B;
    const float h = in && h0 ? h0[j * s.B + b] : 0.0f;
    s.XH[(s.I + j) * s.TB + b] = h;
    if (s.xh) s.xh[IB + e] = h;
    s.C[e] = in && c0 ? c0[j * s.B + b] : 0.0f;
  }
}

// Step t: gates from z (+ Zx) + bias, cell and hidden state; h_t into Hs and
// the next step's block of XH; after the last step the final state into hT, cT.
__global__ void __launch_bounds__(256) tile_lstm_point_fwd_kernel(TileLstm s, int32_t t,
                                                                  const float* __restrict__ bias,
                                                                  const float* __restrict__ X, float* __restrict__ Hs,
                                                                  float* __restrict__ hT, float* __restrict__ cT) {
  const int64_t HB = static_cast<int64_t>(s.H) * s.Bp;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  int64_t j;
  int32_t b;
  row_col(e, s.Bp, j, b);
  if (e < HB) {
    float c = 0.0f, h = 0.0f;
    const bool in = b < s.B;
    if (in) {
      float zv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t r = static_cast<int64_t>(q) * s.H + j;
        zv[q] = step_val(s.z, s.part, s.zsplits, 4 * HB, r * s.Bp + b);
        if (s.Zx) zv[q] += s.Zx[r * s.TB + static_cast<int64_t>(t) * s.Bp + b];
        if (bias) zv[q] += bias[r];
      }
      const float ig = sgm(zv[0]), fg = sgm(zv[1]), gg = tanhf(zv[2]), og = sgm(zv[3]);
      const float cp = s.C[static_cast<int64_t>(t) * HB + e];
      c = fg * cp + ig * gg;
      h = og * tanhf(c);
      float* Gt = s.G + static_cast<int64_t>(t) * 4 * HB + e;
      Gt[0] = ig;
      Gt[HB] = fg;
      Gt[2 * HB] = gg;
      Gt[3 * HB] = og;
      const int64_t o = j * s.B + b;
      Hs[static_cast<int64_t>(t) * s.H * s.B + o] = h;
      if (t == s.T - 1) {
        if (hT) hT[o] = h;
        if (cT) cT[o] = c;
      }
    }
    s.C[static_cast<int64_t>(t + 1) * HB + e] = c;
    if (t + 1 < s.T) {
      s.XH[(s.I + j) * s.TB + static_cast<int64_t>(t + 1) * s.Bp + b] = h;
      if (s.xh) s.xh[static_cast<int64_t>(s.I) * s.Bp + e] = h;
    }
  }
  if (s.xh && t + 1 < s.T && e < static_cast<int64_t>(s.I) * s.Bp)
    s.xh[e] = b < s.B ? X[(static_cast<int64_t>(t + 1) * s.I + j) * s.B + b] : 0.0f;
}

// Step t backward: dh = dHs[t] + (recurrent rows of dxh from step t + 1, or
// dhT at the last step); dz_t into dZ's block t (zeros in the padding columns);
// dc carry. Without the hoisted projection dxh also holds d x_{t + 1}, which
// goes to dX.
__global__ void __launch_bounds__(256) tile_lstm_point_bwd_kernel(TileLstm s, int32_t t,
                                                                  const float* __restrict__ dHs,
                                                                  const float* __restrict__ dhT,
                                                                  const float* __restrict__ dcT,
                                                                  float* __restrict__ dX) {
  const int64_t HB = static_cast<int64_t>(s.H) * s.Bp, IB = s.Zx ? 0 : static_cast<int64_t>(s.I) * s.Bp;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  int64_t j;
  int32_t b;
  row_col(e, s.Bp, j, b);
  const bool last = t == s.T - 1, in = b < s.B;
  const int64_t n = IB + HB;  // elements of dxh
  if (!last && dX && e < IB && in)
    dX[(static_cast<int64_t>(t + 1) * s.I + j) * s.B + b] = step_val(s.dxh, s.part, s.dsplits, n, e);
  if (e >= HB) return;
  float dzq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (in) {
    const int64_t o = j * s.B + b;
    float dh = dHs[static_cast<int64_t>(t) * s.H * s.B + o];
    float dcin;
    if (last) {
      if (dhT) dh += dhT[o];
      dcin = dcT ? dcT[o] : 0.0f;
    } else {
      dh += step_val(s.dxh, s.part, s.dsplits, n, IB + e);
      dcin = s.dc[e];
    }
    const float* Gt = s.G + static_cast<int64_t>(t) * 4 * HB + e;
    const float ig = Gt[0], fg = Gt[HB];
    const float gg = Gt[2 * HB], og = Gt[3 * HB];
    const float c = s.C[static_cast<int64_t>(t + 1) * HB + e];
    const float cp = s.C[static_cast<int64_t>(t) * HB + e];
    const float tc = tanhf(c);
    const float d_o = dh * tc;
    const float dcv = dcin + dh * og * (1.0f - tc * tc);
    s.dc[e] = dcv * fg;
    dzq[0] = dcv * gg * ig * (1.0f - ig);
    dzq[1] = dcv * cp * fg * (1.0f - fg);
    dzq[2] = dcv * ig * (1.0f - gg * gg);
    dzq[3] = d_o * og * (1.0f - og);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s.dZ[(static_cast<int64_t>(q) * s.H + j) * s.TB + static_cast<int64_t>(t) * s.Bp + b] = dzq[q];
    if (s.dz) s.dz[q * HB + e] = dzq[q];
  }
}

// After the last backward step: dh0 and dc0 (and, without the hoisted
// projection, d x_0 into dX[0]).
__global__ void __launch_bounds__(256) tile_lstm_bwd_final_kernel(TileLstm s, float* __restrict__ dX,
                                                                  float* __restrict__ dh0, float* __restrict__ dc0) {
  const int64_t HB = static_cast<int64_t>(s.H) * s.Bp, IB = s.Zx ? 0 : static_cast<int64_t>(s.I) * s.Bp;
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  int64_t j;
  int32_t b;
  row_col(e, s.Bp, j, b);
  if (b >= s.B) return;
  const int64_t o = j * s.B + b, n = IB + HB;
  if (dX && e < IB) dX[o] = step_val(s.dxh, s.part, s.dsplits, n, e);
  if (e < HB) {
    if (dh0) dh0[o] = step_val(s.dxh, s.part, s.dsplits, n, IB + e);
    if (dc0) dc0[o] = s.dc[e];
  }
}

// dbias[r] = sum over the T B columns of dZ row r, one block per row in a
// fixed order (each thread strides the row, then a tree in LDS).
__global__ void __launch_bounds__(256) tile_lstm_dbias_kernel(const float* __restrict__ dZ, int64_t cols,
                                                              float* __restrict__ dbias) {
  __shared__ float part[256];
  const float* row = dZ + static_cast<int64_t>(blockIdx.x) * cols;
  float v = 0.0f;
  for (int64_t c = threadIdx.x; c < cols; c += 256) v += row[c];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) dbias[blockIdx.x] = part[0];
}

inline dim3 grid_of(int64_t n) { return dim3(static_cast<unsigned>((n + 255) / 256)); }

int check_tile_lstm(const ard_lstm_tile_desc* d) {
  if (!d) return fail(ARD_ERR_INVALID_ARG, "desc is NULL");
  if (d->dtype != ARD_F32) return fail(ARD_ERR_UNSUPPORTED, "the tile-pattern LSTM supports ARD_F32 only");
  if (d->seq_len < 1 || d->batch < 1 || d->input_size < 1 || d->hidden_size < 1)
    return fail(ARD_ERR_INVALID_ARG, "sizes must be >= 1");
  const ard_tile_plan* p = d->weight_plan;
  if (!p) return fail(ARD_ERR_INVALID_ARG, "weight_plan is NULL");
  if (p->n != 4 * d->hidden_size || p->k != d->input_size + d->hidden_size)
    return fail(ARD_ERR_INVALID_ARG, "weight_plan covers %d x %d, W is %d x %d", p->n, p->k, 4 * d->hidden_size,
                d->input_size + d->hidden_size);
  if (static_cast<int64_t>(d->seq_len) * d->batch >= (int64_t{1} << 31))
    return fail(ARD_ERR_INVALID_ARG, "seq_len * batch must be < 2^31");
  // the batch is padded to a multiple of 4 (the buffers of such a call exceed the GPU's memory)
  if (d->seq_len * ((static_cast<int64_t>(d->batch) + 3) / 4 * 4) >= (int64_t{1} << 31))
    return fail(ARD_ERR_UNSUPPORTED, "seq_len * padded batch must be < 2^31");
  return ARD_OK;
}

// A step's product over its column block: z_t (fwd) or dxh_t.
TilePart step_part(const TileLstm& s, const ard_tile_plan* p, const void* W, bool fwd, int32_t t) {
  const int32_t itiles = s.Zx ? s.I / p->tile : 0;  // hoisted input tiles
  TilePart q = {};
  const float* cols = (fwd ? s.XH + (s.Zx ? s.I * s.TB : 0) : s.dZ) + static_cast<int64_t>(t) * s.Bp;
  const float* copy = fwd ? s.xh : s.dz;
  q.act = copy ? copy : cols;
  q.lda = copy ? s.Bp : static_cast<int32_t>(s.TB);
  q.W = W;
  q.out = fwd ? s.z : s.dxh;
  q.own0 = fwd ? 0 : itiles;
  q.own_count = fwd ? p->tiles_n : p->tiles_k - itiles;
  q.lo = fwd ? itiles : 0;
  q.hi = fwd ? p->tiles_k : p->tiles_n;
  q.cols = q.ldo = q.nb = q.nv = s.Bp;
  q.partial = s.part;
  return q;
}

// Whether a product over all steps keeps the precision of lists split over four
// workgroups or more: where a step's `rows` tile rows and batch columns alone
// would leave most of the chip idle, on 64 x 64 tiles and batches that were never
// padded (the others ran in one chain).
bool split_chains(const TileLstm& s, const ard_tile_plan* p, int32_t rows) {
  const int64_t wgs = static_cast<int64_t>(rows) * (s.B <= 64 ? 1 : (s.B + 127) / 128);
  return p->tile == 64 && s.B == s.Bp && wgs <= 64;
}

}  // namespace
}  // namespace ard

using namespace ard;

extern "C" {

size_t ard_lstm_tile_workspace_bytes(const ard_lstm_tile_desc* desc) {
  if (check_tile_lstm(desc) != ARD_OK) return 0;
  return tile_layout(desc->seq_len, desc->batch, desc->input_size, desc->hidden_size).total;
}

int ard_lstm_tile_fwd(const ard_lstm_tile_desc* desc, const void* X, const void* W, const float* bias,
                      const void* h0, const void* c0, void* Hs, void* hT, void* cT, void* ws, size_t ws_bytes,
                      void* stream) {
  clear_error();
  int st = check_tile_lstm(desc);
  if (st != ARD_OK) return st;
  if (!X || !W || !Hs) return fail(ARD_ERR_INVALID_ARG, "X, W and Hs must not be NULL");
  const TileLayout L = tile_layout(desc->seq_len, desc->batch, desc->input_size, desc->hidden_size);
  if (!ws || ws_bytes < L.total)
    return fail(ARD_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", L.total, ws_bytes);
  if (!aligned16(ws)) return fail(ARD_ERR_INVALID_ARG, "workspace is not 16-byte aligned");
  const ard_tile_plan* p = desc->weight_plan;
  if ((st = tile_part_check(p, static_cast<int32_t>(L.Bp), W)) != ARD_OK) return st;
  hipStream_t sm = static_cast<hipStream_t>(stream);
  TileLstm s = tile_args(L, static_cast<char*>(ws), desc);
  const int64_t IB = static_cast<int64_t>(s.I) * s.Bp, HB = static_cast<int64_t>(s.H) * s.Bp;
  const float* Xf = static_cast<const float*>(X);
  // one grid row per step, in launches of at most 65535
  for (int32_t t0 = 0; t0 < s.T; t0 += 65535) {
    TileLstm q = s;
    q.XH += static_cast<int64_t>(t0) * s.Bp;
    dim3 grid = grid_of(IB > HB ? IB : HB);
    grid.y = static_cast<unsigned>(s.T - t0 < 65535 ? s.T - t0 : 65535);
    if (t0 > 0) q.H = 0, q.xh = nullptr;  // the initial state went with the first launch
    hipLaunchKernelGGL(tile_lstm_init_kernel, grid, dim3(256), 0, sm, q, Xf + t0 * static_cast<int64_t>(s.I) * s.B,
                       static_cast<const float*>(h0), static_cast<const float*>(c0));
    ARD_LAUNCH_CHECK();
  }
  if (s.Zx) {  // the input tiles' product over the columns of every step
    TilePart q = step_part(s, p, W, true, 0);
    q.act = s.XH;
    q.out = s.Zx;
    q.lo = 0;
    q.hi = s.I / p->tile;
    q.cols = q.ldo = q.nb = q.nv = static_cast<int32_t>(s.TB);
    q.partial = nullptr;
    q.chains = split_chains(s, p, p->tiles_n);
    if ((st = tile_part_f32(true, p, q, stream, nullptr)) != ARD_OK) return st;
  }
  for (int32_t t = 0; t < s.T; ++t) {
    if ((st = tile_part_f32(true, p, step_part(s, p, W, true, t), stream, &s.zsplits)) != ARD_OK) return st;
    hipLaunchKernelGGL(tile_lstm_point_fwd_kernel, grid_of(s.xh && IB > HB ? IB : HB), dim3(256), 0, sm, s, t, bias,
                       Xf, static_cast<float*>(Hs), static_cast<float*>(hT), static_cast<float*>(cT));
    ARD_LAUNCH_CHECK();
  }
  return ARD_OK;
}

int ard_lstm_tile_bwd(const ard_lstm_tile_desc* desc, const void* W, const void* dHs, const void* dhT,
                      const void* dcT, void* ws, size_t ws_bytes, void* dX, float* dW, float* dbias, void* dh0,
                      void* dc0, void* stream) {
  clear_error();
  int st = check_tile_lstm(desc);
  if (st != ARD_OK) return st;
  if (!W || !dHs) return fail(ARD_ERR_INVALID_ARG, "W and dHs must not be NULL");
  const TileLayout L = tile_layout(desc->seq_len, desc->batch, desc->input_size, desc->hidden_size);
  if (!ws || ws_bytes < L.total)
    return fail(ARD_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", L.total, ws_bytes);
  if (!aligned16(ws)) return fail(ARD_ERR_INVALID_ARG, "workspace is not 16-byte aligned");
  const ard_tile_plan* p = desc->weight_plan;
  if ((st = tile_part_check(p, static_cast<int32_t>(L.Bp), W)) != ARD_OK) return st;
  hipStream_t sm = static_cast<hipStream_t>(stream);
  TileLstm s = tile_args(L, static_cast<char*>(ws), desc);
  const int64_t IB = s.Zx ? 0 : static_cast<int64_t>(s.I) * s.Bp, HB = static_cast<int64_t>(s.H) * s.Bp;
  for (int32_t t = s.T - 1; t >= 0; --t) {
    hipLaunchKernelGGL(tile_lstm_point_bwd_kernel, grid_of(IB > HB ? IB : HB), dim3(256), 0, sm, s, t,
                       static_cast<const float*>(dHs), static_cast<const float*>(dhT),
                       static_cast<const float*>(dcT), static_cast<float*>(dX));
    ARD_LAUNCH_CHECK();
    if (t == 0 && s.Zx && !dh0) break;  // nothing reads the first step's recurrent derivative
    if ((st = tile_part_f32(false, p, step_part(s, p, W, false, t), stream, &s.dsplits)) != ARD_OK) return st;
  }
  if (dh0 || dc0 || (dX && !s.Zx)) {
    hipLaunchKernelGGL(tile_lstm_bwd_final_kernel, grid_of(IB > HB ? IB : HB), dim3(256), 0, sm, s,
                       static_cast<float*>(dX), static_cast<float*>(dh0), static_cast<float*>(dc0));
    ARD_LAUNCH_CHECK();
  }
  if (dX && s.Zx) {  // the input tiles' transposed product over the columns of every step
    TilePart q = step_part(s, p, W, false, 0);
    q.out = dX;
    q.own0 = 0;
    q.own_count = s.I / p->tile;
    q.cols = static_cast<int32_t>(s.TB);
    q.ldo = q.nv = s.B;
    q.nb = s.Bp;
    q.bstride = static_cast<int64_t>(s.I) * s.B;
    q.partial = nullptr;
    q.chains = split_chains(s, p, p->tiles_k);
    if ((st = tile_part_f32(false, p, q, stream, nullptr)) != ARD_OK) return st;
  }
  if (dW) {
    const ard_tile_desc tw = {ARD_F32, static_cast<int32_t>(s.TB), s.I + s.H, 4 * s.H, 1.0f, ARD_DROPPED_ZERO};
    if ((st = ard_tile_bwd_weight(&tw, p, s.XH, s.dZ, dW, stream)) != ARD_OK) return st;
  }
  if (dbias) {
    hipLaunchKernelGGL(tile_lstm_dbias_kernel, dim3(static_cast<unsigned>(4 * s.H)), dim3(256), 0, sm, s.dZ, s.TB,
                       dbias);
    ARD_LAUNCH_CHECK();
  }
  return ARD_OK;
}

}  // extern "C"
