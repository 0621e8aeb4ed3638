// Tile-layer kernels whose waves work alone (gfx950): products over lists of
// kept tiles (Sec. III-B) cut into 32-deep parts, for the shapes that the
// workgroup pipeline of ard_tile.hip does not take or does not fill the chip
// with: 32 x 32 tiles, batches whose rows are no multiple of 16 bytes, and the
// small products of a recurrent step.
//
// A workgroup owns 32 output rows and BN batch columns. Its waves take the
// parts of the row's list in turn (part u goes to wave u % NWV), each with LDS
// stages of its own, so no barrier runs inside the list walk: a wave waits for
// its own loads only, and a short or a long list keeps all waves equally busy.
// At the end the waves' sums are added through LDS in wave order.
//
// Why not one slab of the workgroup pipeline per tile: a 32 x 32 tile is 32 deep,
// a barrier and a load latency for a quarter of the work of a 64 x 64 tile's
// slab, and lists of different rows share no operand that a common slab could
// reuse. The waves' private stages keep NWV times STAGES - 1 parts in flight
// per compute unit instead.
//
// Measured on MI355X, a layer's plan, forward and backward at p = 0.5, against
// the register-staged one-buffer kernel these sizes ran on: fp32 2048 x 2048,
// batch 128, 32 x 32 tiles 172 -> 38 us (forward 69 -> 12); bf16 2816 x 384,
// batch 391, 64 x 64 tiles 296 -> 56 us.
#pragma once

#include "ard_gemm_fast.hpp"

namespace ard {

struct TileWaveArgs {
  const void* act;      // rows of the other side's tiles: Xt (fwd), dYt (bwd_data)
  const void* W;
  void* out;            // Yt or dXt
  const int32_t* ptr;   // row_ptr (fwd) or col_ptr (bwd_data)
  const int32_t* list;  // row_cols (fwd) or col_rows (bwd_data), ascending per row
  int32_t B, K, tile;   // columns of the product; row stride of W
  int32_t lda;          // row stride of act
  // output element (m, n): out[m * ldo + (n / nb) * bstride + n % nb], written
  // where n % nb < nv (a product over the columns of several steps at once;
  // nb is a multiple of 4, or B)
  int32_t ldo, nb, nv;
  int64_t bstride;
  int32_t nx, ny;       // grid: column blocks x 32-row blocks of the output
  int32_t own0;         // first output tile row (fwd) or column (bwd_data)
  int32_t lo, hi;       // list entries in [lo, hi) only; act row 0 belongs to entry lo
  float scale;
  // splits > 1: workgroup (tile, split) sums its share of the list into
  // partial[split][ny * 32][B], fp32 and unscaled
  int32_t splits;
  float* partial;
};

enum { WAVE_FWD = 0, WAVE_BWD_DATA = 1 };
constexpr int kAllTiles = 1 << 30;  // hi of an unrestricted list

template <typename T, int BN_, int NWV_, int STAGES_, int CHAINS_ = 1>
struct WaveCfg {
  using Cfg = FastCfg<T, 32, BN_, 32, STAGES_, 1, 1, 1, CHAINS_>;  // one wave's pipeline
  static constexpr int BN = BN_, NWV = NWV_, NT = 64 * NWV;
  static constexpr int ROW = BN * 4 + 32;                 // bytes of a reduction row (see fast_store)
  static constexpr int RED = NWV * 32 * ROW;
  static constexpr int STG = NWV * Cfg::LDS;
  static constexpr int ANYSTG = NWV * Cfg::STAGE;         // register loads need one stage
  static constexpr int LDS = RED > STG ? RED : STG;
  static constexpr int LDS_ANY = RED > ANYSTG ? RED : ANYSTG;
  static_assert(LDS <= 160 * 1024, "LDS of a compute unit");
};

// A wave's walk over its parts: next() gives the two operands' first
// elements of part u = first, first + step, ...; past the last part the last
// one again, so that every wave issues the same number of loads per stage.
// Entry e of the list sits in lane e - wbase of the window (see ListLoader).
struct PartWalk {
  const char* a0;
  const char* b0;
  int64_t a_tile, a_part, b_tile, b_part;
  const int32_t* list;
  int32_t n, parts, u, last, step, wbase, win, base;  // win: list[wbase + lane]

  __device__ __forceinline__ void refill() {
    const int lane = threadIdx.x & 63;
    const int32_t* p = list + (wbase + lane < n ? wbase + lane : n - 1);
    int32_t v;
    asm volatile("global_load_dword %0, %1, off\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
    win = v;
  }
  __device__ __forceinline__ void next(const char*& a, const char*& b) {
    const int e = parts == 1 ? u : u >> 1, part = parts == 1 ? 0 : u & 1;
    if (e - wbase >= 64) {
      wbase += (e - wbase) / 64 * 64;
      refill();
    }
    const int64_t t = __builtin_amdgcn_readlane(win, e - wbase);
    a = a0 + t * a_tile + part * a_part;
    b = b0 + (t - base) * b_tile + part * b_part;
    if (u + step <= last) u += step;
  }
};

// MFMAs of one 32-deep part held in the wave's LDS stage.
template <class Cfg, bool AMC, bool BMC>
__device__ __forceinline__ void wave_part(const char* st, AccChains<Cfg>& ch) {
  using Frags = StepFrags<Cfg, AMC, BMC>;
  constexpr int STEPS = Cfg::KW / Frags::KSTEP;
  Frags fr[2];
  fr[0].load(st, 0, 0, 0);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    if (s + 1 < STEPS) fr[(s + 1) & 1].load(st, 0, 0, (s + 1) * Frags::KSTEP);
    ch.mma(fr[s & 1], s);
  }
}

// Zeroes the k >= kv of a k-contiguous operand in a wave's stage; kv is a
// multiple of a 16-byte chunk.
template <class Cfg, int R>
__device__ __forceinline__ void wave_zero_tail_kc(char* region, int kv) {
  constexpr int CPR = Cfg::BK * Cfg::ES / 16, EPC = 16 / Cfg::ES;
  for (int e = threadIdx.x & 63; e < R * CPR; e += 64) {
    const int r = e / CPR, c = e % CPR;
    if (c * EPC >= kv) *reinterpret_cast<u32x4*>(region + kc_off<CPR>(r, c)) = u32x4{0u, 0u, 0u, 0u};
  }
}

// A wave's nu parts on direct loads. The next load goes into the stage that the
// previous part was read from: its LDS reads have returned (lgkmcnt 0), so no
// barrier is needed.
template <class Cfg, bool AMC, bool BMC, class Src, class SrcB, class Next>
__device__ __forceinline__ void wave_walk_dma(const Src& da, const SrcB& db, Next next, int nu,
                                              f32x16 (&acc)[Cfg::FM][Cfg::FN], char* smem) {
  if (nu <= 0) return;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));
  int is = 0, cs = 0;
  auto issue = [&]() {
    const char *a, *b;
    const int kv = next(a, b);
    da.issue(a, kv, lds0 + static_cast<uint32_t>(is * Cfg::STAGE), 0);
    db.issue(b, kv, lds0 + static_cast<uint32_t>(is * Cfg::STAGE) + Cfg::ABYTES, 0);
    is = is + 1 == Cfg::STAGES ? 0 : is + 1;
    return kv;
  };
  AccChains<Cfg> ch(acc);
  int kvs[Cfg::STAGES];  // valid k of the loaded parts, oldest first
#pragma unroll
  for (int s = 0; s < Cfg::STAGES - 1; ++s) kvs[s] = issue();
  for (int j = 0; j < nu; ++j) {
    if constexpr (Cfg::STAGES == 1) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      kvs[0] = issue();
      wait_vm<0>();
    } else {
      wait_vm<(Cfg::STAGES - 2) * Cfg::LPW>();
    }
    char* st = smem + cs * Cfg::STAGE;
    if constexpr (!AMC && !BMC) {
      if (kvs[0] < Cfg::BK) {
        wave_zero_tail_kc<Cfg, Cfg::BM>(st, kvs[0]);
        wave_zero_tail_kc<Cfg, Cfg::BN>(st + Cfg::ABYTES, kvs[0]);
      }
    }
    if constexpr (Cfg::STAGES > 1) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      kvs[Cfg::STAGES - 1] = issue();
#pragma unroll
      for (int s = 0; s + 1 < Cfg::STAGES; ++s) kvs[s] = kvs[s + 1];
    }
    wave_part<Cfg, AMC, BMC>(st, ch);
    cs = cs + 1 == Cfg::STAGES ? 0 : cs + 1;
  }
  ch.sum();
  wait_vm<0>();  // no direct load may still write LDS past this point
}

// The same on register loads (rows starting at any element): two parts in
// flight in registers, one LDS stage; a wave's LDS accesses execute in order.
template <class Cfg, bool AMC, bool BMC, class Src, class SrcB, class Next>
__device__ __forceinline__ void wave_walk_any(const Src& da, const SrcB& db, Next next, int nu,
                                              f32x16 (&acc)[Cfg::FM][Cfg::FN], char* smem) {
  if (nu <= 0) return;
  u32x4 ra[2][Src::PER_WAVE], rb[2][SrcB::PER_WAVE];
  auto load = [&](int i) {
    const char *a, *b;
    const int kv = next(a, b);
    da.load(a, kv, ra[i]);
    db.load(b, kv, rb[i]);
  };
  AccChains<Cfg> ch(acc);
  load(0);
  if (nu > 1) load(1);
  auto part = [&](int j, int i) {
    da.store(smem, 0, ra[i]);
    db.store(smem + Cfg::ABYTES, 0, rb[i]);
    if (j + 2 < nu) load(i);
    asm volatile("" ::: "memory");
    wave_part<Cfg, AMC, BMC>(smem, ch);
    asm volatile("" ::: "memory");
  };
  for (int j = 0; j < nu; j += 2) {
    part(j, 0);
    if (j + 1 < nu) part(j + 1, 1);
  }
  ch.sum();
}

// The waves' accumulators (32 x BN each) added in wave order; every thread then
// hands 4 consecutive columns of one row to put(row, column, values).
template <class WC, class Put>
__device__ __forceinline__ void wave_reduce(const f32x16 (&acc)[1][WC::BN / 32], char* smem, Put put) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  lds_barrier();  // every wave is done with its stages
  char* region = smem + wave * 32 * WC::ROW;
#pragma unroll
  for (int j = 0; j < WC::BN / 32; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      *reinterpret_cast<float*>(region + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * WC::ROW +
                                (32 * j + (lane & 31)) * 4) = acc[0][j][r];
  lds_barrier();
  constexpr int QPR = WC::BN / 4;
  for (int e = threadIdx.x; e < 32 * QPR; e += WC::NT) {
    const int row = e / QPR, q = e % QPR;
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < WC::NWV; ++w)
      v += *reinterpret_cast<const f32x4*>(smem + (w * 32 + row) * WC::ROW + q * 16);
    put(row, 4 * q, v);
  }
}

// Four consecutive outputs at p, of which the first n are inside.
template <typename OutT>
__device__ __forceinline__ void put4(OutT* p, const f32x4& v, float scale, int n, bool vec) {
  OutT w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = from_f32<OutT>(scale * v[i]);
  if (vec && n >= 4) {
    if constexpr (sizeof(OutT) == 2)
      *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(w);
    else
      *reinterpret_cast<f32x4*>(p) = *reinterpret_cast<const f32x4*>(w);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < n) p[i] = w[i];
  }
}

// fwd / bwd_data: 32 output rows x BN batch columns, position bid of the grid,
// split sp of the lists.
template <class WC, typename T, int PASS, bool ANY>
__device__ __forceinline__ void tile_wave_rows(const TileWaveArgs& a, int bid, int sp, char* smem) {
  using Cfg = typename WC::Cfg;
  constexpr bool AMC = PASS == WAVE_BWD_DATA;
  constexpr int ES = sizeof(T);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int blk, col;
  grouped_tile(bid, a.nx, a.ny, blk, col);
  const int splits = a.splits > 1 ? a.splits : 1;
  const int n0 = col * WC::BN;
  const int parts = a.tile / 32;
  const int own = a.own0 + blk / parts, sub = blk % parts;
  const int pa = __builtin_amdgcn_readfirstlane(a.ptr[own]);
  const int len = __builtin_amdgcn_readfirstlane(a.ptr[own + 1]) - pa;
  // the list's first window, and where the entries in [lo, hi) of the
  // ascending list begin and end in it
  const int first = len > 0 ? a.list[pa + (lane < len ? lane : len - 1)] : 0;
  int e0 = 0, e1 = len;
  if (a.lo > 0 || a.hi < kAllTiles) {
    int t = lane < len ? first : kAllTiles;
    e0 = __popcll(__ballot(t < a.lo));
    e1 = __popcll(__ballot(t < a.hi));
    for (int i = 64; i < len; i += 64) {
      t = i + lane < len ? a.list[pa + i + lane] : kAllTiles;
      e0 += __popcll(__ballot(t < a.lo));
      e1 += __popcll(__ballot(t < a.hi));
    }
  }
  const int units = (e1 - e0) * parts;
  const int u0 = units * sp / splits, u1 = units * (sp + 1) / splits;  // this split's parts
  const int nu = u1 - u0 > wave ? (u1 - u0 - wave + WC::NWV - 1) / WC::NWV : 0;

  f32x16 acc[1][Cfg::FN];
#pragma unroll
  for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.0f;

  const int64_t K = a.K, B = a.B, TT = a.tile;
  if (nu > 0) {
    PartWalk pw;
    const char* W = static_cast<const char*>(a.W);
    const int64_t row0 = own * TT + sub * 32;
    if constexpr (PASS == WAVE_FWD) {
      pw.a0 = W + row0 * K * ES;
      pw.a_tile = TT * ES;
      pw.a_part = 32 * ES;
    } else {
      pw.a0 = W + row0 * ES;
      pw.a_tile = TT * K * ES;
      pw.a_part = 32 * K * ES;
    }
    pw.b0 = static_cast<const char*>(a.act);
    pw.b_tile = TT * a.lda * ES;
    pw.b_part = static_cast<int64_t>(32) * a.lda * ES;
    pw.list = a.list + pa;
    pw.n = len;
    pw.parts = parts;
    pw.u = e0 * parts + u0 + wave;
    pw.last = e0 * parts + u1 - 1;
    pw.step = WC::NWV;
    pw.base = a.lo;
    pw.wbase = (pw.u / parts) / 64 * 64;
    pw.win = first;
    if (pw.wbase > 0) pw.refill();
    auto next = [&](const char*& pA, const char*& pB) {
      pw.next(pA, pB);
      return static_cast<int>(Cfg::BK);
    };
    if constexpr (ANY) {
      RegSrc<Cfg, 32, AMC> da;
      RegSrc<Cfg, WC::BN, true> db;
      da.init(K, 0, 32, 0);
      db.init(a.lda, n0, a.B, 0);
      wave_walk_any<Cfg, AMC, true>(da, db, next, nu, acc, smem + wave * Cfg::STAGE);
    } else {
      DmaSrc<Cfg, 32, AMC> da;
      DmaSrc<Cfg, WC::BN, true> db;
      da.init(K, 0, 32, 0);
      db.init(a.lda, n0, a.B, 0);
      wave_walk_dma<Cfg, AMC, true>(da, db, next, nu, acc, smem + wave * Cfg::LDS);
    }
  }
  if (splits > 1) {
    float* part = a.partial + (static_cast<int64_t>(sp) * a.ny + blk) * 32 * B;
    wave_reduce<WC>(acc, smem, [&](int row, int c, const f32x4& v) {
      if (n0 + c < a.B) put4<float>(part + row * B + n0 + c, v, 1.0f, a.B - n0 - c, a.B % 4 == 0);
    });
  } else {
    // pieces of 4 aligned elements: rows and blocks of whole pieces
    const bool vec = a.ldo % 4 == 0 && a.bstride % 4 == 0 && a.nb % 4 == 0 &&
                     reinterpret_cast<uintptr_t>(a.out) % (4 * sizeof(T)) == 0;
    T* out = static_cast<T*>(a.out) + static_cast<int64_t>(blk) * 32 * a.ldo;
    wave_reduce<WC>(acc, smem, [&](int row, int c, const f32x4& v) {
      if (n0 + c >= a.B) return;
      const int t = (n0 + c) / a.nb, b = n0 + c - t * a.nb;
      put4<T>(out + static_cast<int64_t>(row) * a.ldo + t * a.bstride + b, v, a.scale, a.nv - b, vec);
    });
  }
}

template <class WC, typename T, int PASS, bool ANY>
__global__ void __launch_bounds__(WC::NT) tile_wave_rows_kernel(TileWaveArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  tile_wave_rows<WC, T, PASS, ANY>(a, static_cast<int>(blockIdx.x), static_cast<int>(blockIdx.y), smem);
}

struct TileWaveDwArgs {
  const void* X;
  const void* dY;
  float* dW;
  const int32_t* chunks;  // weight-gradient group records
  int32_t B, K, tile;
  float scale;
};

constexpr int kWaveGroup = 4;  // tiles per group record

// bwd_weight: blocks of 32 rows x 128 columns of a group of up to four kept
// tiles of one tile row (all four 32 x 32 tiles, or one row half of two 64 x 64
// tiles), workgroup bid of nwg. The waves take the 32-deep parts of the batch
// in turn. A batch has few parts, so it is workgroups sharing a compute unit
// that hide the loads, the reduction and the stores (80 KB of LDS each), not a
// deep pipeline. Loading the fragments straight into registers instead was
// twice as slow (bf16 4096 x 4096, batch 512, 32 x 32 tiles: 97 us).
template <class WC, typename T, bool ANY>
__device__ __forceinline__ void tile_wave_dw(const TileWaveDwArgs& a, int bid, int nwg, char* smem) {
  using Cfg = typename WC::Cfg;
  constexpr int ES = sizeof(T);
  static_assert(WC::BN == 128, "four 32-wide or two 64-wide tiles");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int TT = a.tile, per = TT == 32 ? 1 : 4;  // blocks per group
  const int64_t B = a.B, K = a.K;
  const int total = __builtin_amdgcn_readfirstlane(a.chunks[0]) * per;
  const int nparts = (a.B + 31) / 32;
  for (int blk = bid; blk < total; blk += nwg) {
    const int32_t* rec = a.chunks + 4 + static_cast<int64_t>(blk / per) * (4 + kWaveGroup);
    const int half = per == 1 ? 0 : (blk >> 1) & 1;
    const int slot0 = per == 1 ? 0 : 2 * (blk & 1);  // first tile of the block
    const int tn = __builtin_amdgcn_readfirstlane(rec[0]);
    const int cnt = __builtin_amdgcn_readfirstlane(rec[2]);
    if (slot0 >= cnt) continue;  // the same for the whole workgroup
    const int64_t row0 = static_cast<int64_t>(tn) * TT + half * 32;
    f32x16 acc[1][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.0f;
    const int nu = nparts > wave ? (nparts - wave + WC::NWV - 1) / WC::NWV : 0;
    if (nu > 0) {
      int u = wave;
      const char* a0 = static_cast<const char*>(a.dY) + row0 * B * ES;
      const char* b0 = static_cast<const char*>(a.X);
      auto next = [&](const char*& pA, const char*& pB) {
        pA = a0 + static_cast<int64_t>(u) * 32 * ES;
        pB = b0 + static_cast<int64_t>(u) * 32 * ES;
        const int kv = a.B - u * 32;
        if (u + WC::NWV < nparts) u += WC::NWV;
        return kv;
      };
      // row r of the X side: row r % TT of the block's tile r / TT (the record pads short groups)
      auto xrow = [&](int r) { return rec[4 + slot0 + r / TT] * TT + r % TT; };
      if constexpr (ANY) {
        RegSrc<Cfg, 32, false> da;
        RegSrc<Cfg, 128, false> db;
        da.init(B, 0, 32, 0);
        db.init_rows(B, xrow, 0);
        wave_walk_any<Cfg, false, false>(da, db, next, nu, acc, smem + wave * Cfg::STAGE);
      } else {
        DmaSrc<Cfg, 32, false> da;
        DmaSrc<Cfg, 128, false> db;
        da.init(B, 0, 32, 0);
        db.init_rows(B, xrow, 0);
        wave_walk_dma<Cfg, false, false>(da, db, next, nu, acc, smem + wave * Cfg::LDS);
      }
    }
    wave_reduce<WC>(acc, smem, [&](int row, int c, const f32x4& v) {
      const int slot = slot0 + c / TT;
      if (slot < cnt)
        put4<float>(a.dW + (row0 + row) * K + static_cast<int64_t>(rec[4 + slot]) * TT + c % TT, v, a.scale, 4, true);
    });
    lds_barrier();  // the next block's loads overwrite the sums
  }
}

template <class WC, typename T, bool ANY>
__global__ void __launch_bounds__(WC::NT) tile_wave_dw_kernel(TileWaveDwArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  tile_wave_dw<WC, T, ANY>(a, static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), smem);
}

// The layer's backward in one launch: the bwd_data workgroups first, then the
// weight-gradient ones (the same device functions as the separate kernels: the
// results are theirs bit for bit).
template <class WCD, class WCW, typename T, bool ANY>
__global__ void __launch_bounds__(WCD::NT) tile_wave_bwd_kernel(TileWaveArgs d, TileWaveDwArgs w, int32_t nd) {
  static_assert(WCD::NT == WCW::NT, "one block size");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = static_cast<int>(blockIdx.x);
  if (b < nd)
    tile_wave_rows<WCD, T, WAVE_BWD_DATA, ANY>(d, b, 0, smem);
  else
    tile_wave_dw<WCW, T, ANY>(w, b - nd, static_cast<int>(gridDim.x) - nd, smem);
}

}  // namespace ard
