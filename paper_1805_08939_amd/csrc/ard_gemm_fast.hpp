// GEMM with direct global -> LDS loads and a deep K pipeline (gfx950).
//
// The same contraction as gemm_kernel (ard_gemm.hpp) for operand views that
// can be read in whole 16-byte chunks (row stride a multiple of 16 bytes,
// aligned base, no row or column gather, no load-time gate):
//
//  * global -> LDS without register staging: each lane issues
//    global_load_lds_dwordx4 for one 16-byte chunk of a tile;
//    a wave writes 64 consecutive LDS chunks, and the lane picks the global
//    chunk that belongs at its LDS position under an XOR swizzle that keeps the
//    MFMA fragment reads free of bank conflicts;
//  * k-contiguous operands live in LDS as [rows][BK] and are read as whole
//    fragments (ds_read_b128); m/n-contiguous operands (feature-major
//    activations, transposed weights) stay [BK][rows] exactly as in HBM: bf16
//    fragments come from ds_read_b64_tr_b16, whose 16-lane transpose delivers
//    4 consecutive k of one column per lane, fp32 fragments from one
//    ds_read_b32 per k (consecutive lanes read consecutive columns);
//  * STAGES LDS stages: the loads of the next STAGES - 1 slabs are in flight
//    while the waves run MFMA on the current one; a wave waits only for the
//    slab it is about to use (vmcnt counts the later slabs it has issued);
//  * optionally the waves of a workgroup split each slab's k between them and
//    reduce through LDS at the end (small output tiles that still fill the
//    chip);
//  * the last, partial K slab is cleaned in LDS (entries past the contraction
//    length set to 0) before use; rows past the output extents load a clamped
//    valid row and their results are discarded;
//  * operands are plain strided views (a row-based pattern's gather is folded
//    into base and row stride by the caller), so the main loop reads no index
//    lists: an index load would make the wave wait for every earlier direct load.
//
// The direct loads are issued as inline assembly and ordered only by the
// explicit vmcnt waits and LDS barriers of the main loop: the compiler, which
// cannot tell that an LDS read targets another stage than the loads in
// flight, would otherwise wait for all of them before such reads, and
// __syncthreads() waits for all outstanding vector memory operations.
#pragma once

#include <type_traits>

#include "ard_gemm.hpp"

namespace ard {

typedef short i16x4 __attribute__((ext_vector_type(4)));

// LD: how the operands are loaded.
enum FastLoad {
  LOAD_DMA = 0,   // direct loads
  LOAD_ANY = 1,   // rows starting at any element (register loads)
  LOAD_FLAT = 2   // direct loads of a flat contraction (FlatLoader)
};

template <typename T_, int BM_, int BN_, int BK_, int STAGES_, int WGM_, int WGN_, int KSPLIT_, int CHAINS_ = 1>
struct FastCfg {
  using T = T_;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_;
  static constexpr int WGM = WGM_, WGN = WGN_, KSPLIT = KSPLIT_;
  static constexpr int NW = WGM * WGN * KSPLIT, NT = 64 * NW;
  static constexpr int TM = BM / WGM, TN = BN / WGN;  // wave tile
  static constexpr int FM = TM / 32, FN = TN / 32;    // 32x32 MFMA blocks per wave
  static constexpr int KW = BK / KSPLIT;              // k per wave per slab
  static constexpr int CHAINS = CHAINS_;              // accumulators per output (AccChains)
  static constexpr int ES = sizeof(T);
  static constexpr int ABYTES = BM * BK * ES, BBYTES = BN * BK * ES;
  static constexpr int STAGE = ABYTES + BBYTES;
  static constexpr int LDS = STAGES * STAGE;
  // the k splits' accumulators and row sums, or the staging of the stores
  static constexpr int ENDS = KSPLIT > 1 ? KSPLIT * WGM * (WGN * FM * FN * 16 * 64 + FM * 32) * 4
                                         : NW * (32 * (TN * 4 + 32) + TM * 4);
  static constexpr int LDS_REG = ENDS > 2 * STAGE ? ENDS : 2 * STAGE;  // register loads keep two stages
  // 16-byte load instructions per wave per slab
  static constexpr int LPW = (ABYTES + BBYTES) / 16 / 64 / NW;
  static_assert(ABYTES % (1024 * NW) == 0 && BBYTES % (1024 * NW) == 0, "tile must split into wave loads");
  static_assert(KW % (ES == 2 ? 16 : 8) == 0, "per-wave k must hold whole MFMA steps");
};

// LDS layout. gfx950 LDS has 64 banks of 4 bytes: a wave's 16-byte reads are
// served 16 lanes per pass, its 8-byte reads 32 lanes per pass, and a pass is
// free of bank conflicts when its lanes touch 16 different 16-byte bank groups
// (byte address / 16 mod 16). Chunk c of row r goes to position
// r * CPR + (c ^ swizzle(r)); the swizzles make the fragment reads below
// conflict-free.
//
// k-contiguous tiles [R][BK] (CPR = BK*ES/16 chunks per row), read as 16 bytes
// per lane from 16 consecutive rows at one chunk: rows r and r + 16/CPR share
// bank groups unless the swizzle tells them apart.
template <int CPR>
__device__ __forceinline__ int kc_swz(int r) {
  constexpr int SH = CPR >= 16 ? 0 : CPR == 8 ? 1 : CPR == 4 ? 2 : 3;
  return (r >> SH) & (CPR - 1);
}
// m/n-contiguous tiles [BK][R] (CPR = R*ES/16 chunks per k-row). 16-bit data
// is read transposed: per 32 lanes, 4 consecutive k-rows x 4 consecutive
// chunks; 32-bit data per lane from k-rows k and k + 4, 8 chunks each.
template <int CPR, int ES>
__device__ __forceinline__ int mc_swz(int k) {
  if constexpr (ES == 2) {
    if constexpr (CPR >= 16)
      return (k & 3) << 2;
    else if constexpr (CPR == 8)
      return ((k >> 1) & 1) << 2;
    else
      return 0;
  } else {
    if constexpr (CPR >= 16)
      return ((k >> 2) & 1) << 3;
    else
      return 0;
  }
}

template <int CPR>
__device__ __forceinline__ int kc_off(int r, int c) {
  return (r * CPR + (c ^ kc_swz<CPR>(r))) * 16;
}
template <int CPR, int ES>
__device__ __forceinline__ int mc_off(int k, int c) {
  return (k * CPR + (c ^ mc_swz<CPR, ES>(k))) * 16;
}

// One direct load of 16 bytes per lane from sbase + voff into LDS at
// lds_base + 16 * lane. sbase (an SGPR pair) and lds_base are wave-uniform;
// lds_base travels in M0, which the compiler writes before the statement and
// which the load reads one wait state later at the earliest. The compiler's
// hazard tracking does not look into the statement: the first load of a group
// (FIRST) also waits the 5 states a vector memory instruction needs after a
// VALU write (v_readfirstlane) of an SGPR it reads; later loads of the group
// use the same base. No memory clobber: the load writes a stage that no LDS
// access between two loop barriers touches, and volatile statements keep
// their order relative to the barriers and waits.
template <bool FIRST>
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_base) {
  if constexpr (FIRST)
    asm volatile(
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(voff), "s"(sbase), "{m0}"(lds_base));
  else
    asm volatile(
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(voff), "s"(sbase), "{m0}"(lds_base));
}

// A wave-uniform pointer as such (SGPR pair): integer division and other VALU
// lowerings leave uniform values in VGPRs.
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// LDS address (byte offset in the workgroup's LDS) of a pointer into shared memory.
__device__ __forceinline__ uint32_t lds_addr(const char* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) char*)p));
}

// Workgroup barrier for the LDS hand-off: waits for this wave's own LDS
// operations only, not for its direct loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Per-lane sources of one operand's direct loads. Per slab a wave loads
// PER_WAVE blocks of 64 16-byte chunks; LDS chunk pos = blk * 64 + lane of the
// operand's region holds, for a k-contiguous tile [R][BK], row pos / CPR and
// the swizzled k chunk; for an m/n-contiguous tile [BK][R], k-row pos / CPR
// and the swizzled column chunk. A chunk is addressed as a 32-bit byte offset
// from the slab's first element (uniform, in SGPRs). Rows and columns past the
// extents are clamped once to a valid one (their results are discarded); a
// chunk past the contraction length of a partial slab loads the same row's
// (or column's) chunk at k 0 of the slab instead, and the slab's tail is
// zeroed in LDS before use.
template <class Cfg, int R, bool MC>
struct DmaSrc {
  static constexpr int ES = Cfg::ES, EPC = 16 / ES;  // EPC: elements per chunk
  static constexpr int CPR = MC ? R * ES / 16 : Cfg::BK * ES / 16;
  static constexpr int PER_WAVE = R * Cfg::BK * ES / 1024 / Cfg::NW;
  uint32_t off[PER_WAVE];   // byte offset of the lane's chunk from the slab base
  uint32_t off0[PER_WAVE];  // the same chunk at k (KC) or k-row (MC) 0 of the slab
  int k[PER_WAVE];          // the chunk's k (KC) or k-row (MC) within the slab

  // nblk > 0: m/n-contiguous with blocked columns (GemmArgs::nblk)
  __device__ __forceinline__ void init(int64_t ld, int r0, int rext, int wave, int nblk = 0, int64_t nstride = 0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int pos = (wave * PER_WAVE + i) * 64 + lane;
      if constexpr (!MC) {
        const int r = pos / CPR;
        const int c = (pos % CPR) ^ kc_swz<CPR>(r);
        const int row = r0 + r < rext ? r0 + r : rext - 1;
        off0[i] = static_cast<uint32_t>(row * ld * ES);
        off[i] = off0[i] + static_cast<uint32_t>(c * 16);
        k[i] = c * EPC;
      } else {
        const int kk = pos / CPR;
        const int c = (pos % CPR) ^ mc_swz<CPR, ES>(kk);
        int64_t col = r0 + c * EPC < rext ? r0 + c * EPC : 0;
        if (nblk > 0) {
          const int t = static_cast<int>(col) / nblk;
          col = t * nstride + (static_cast<int>(col) - t * nblk);
        }
        off0[i] = static_cast<uint32_t>(col * ES);
        off[i] = off0[i] + static_cast<uint32_t>(kk * ld * ES);
        k[i] = kk;
      }
    }
  }

  // A k-contiguous operand whose tile row r is row rowof(r) of the view: a
  // row gather folded into the lane offsets once, so the main loop reads no
  // index. Every rowof(r) must be a valid row.
  template <class F>
  __device__ __forceinline__ void init_rows(int64_t ld, F rowof, int wave) {
    static_assert(!MC, "row gather of a k-contiguous operand");
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int pos = (wave * PER_WAVE + i) * 64 + lane;
      const int r = pos / CPR;
      const int c = (pos % CPR) ^ kc_swz<CPR>(r);
      off0[i] = static_cast<uint32_t>(static_cast<int64_t>(rowof(r)) * ld * ES);
      off[i] = off0[i] + static_cast<uint32_t>(c * 16);
      k[i] = c * EPC;
    }
  }

  // Loads the slab whose first element is at sbase (uniform), of which the
  // first kv k (k-rows) are valid, into the LDS region at byte address region.
  __device__ __forceinline__ void issue(const char* sbase, int kv, uint32_t region, int wave) const {
    const char* b = uniform_ptr(sbase);
    const uint32_t r0 = region + static_cast<uint32_t>(wave * PER_WAVE * 1024);
    dma16<true>(b, k[0] < kv ? off[0] : off0[0], r0);
#pragma unroll
    for (int i = 1; i < PER_WAVE; ++i) dma16<false>(b, k[i] < kv ? off[i] : off0[i], r0 + static_cast<uint32_t>(i * 1024));
  }
};

// Zeroes the entries of a loaded slab whose k is >= kvalid (k from the slab start).
template <class Cfg, int R, bool MC>
__device__ __forceinline__ void fast_zero_tail(char* region, int kvalid) {
  constexpr int ES = Cfg::ES, EPC = 16 / ES;
  if constexpr (!MC) {
    constexpr int CPR = Cfg::BK * ES / 16;
    for (int e = threadIdx.x; e < R * Cfg::BK; e += Cfg::NT) {
      const int r = e / Cfg::BK, k = e % Cfg::BK;
      if (k >= kvalid) {
        char* p = region + kc_off<CPR>(r, k / EPC) + (k % EPC) * ES;
        if constexpr (ES == 2)
          *reinterpret_cast<uint16_t*>(p) = 0;
        else
          *reinterpret_cast<uint32_t*>(p) = 0;
      }
    }
  } else {
    constexpr int CPR = R * ES / 16;
    for (int e = threadIdx.x; e < Cfg::BK * CPR; e += Cfg::NT) {
      const int kk = e / CPR;
      if (kk >= kvalid) *reinterpret_cast<u32x4*>(region + e * 16) = u32x4{0u, 0u, 0u, 0u};
    }
  }
}

// bf16 MFMA operand fragment: 8 k (kk .. kk+15 split over the two lane halves)
// of the row/column rb + lane % 32.
template <class Cfg, int R, bool MC>
__device__ __forceinline__ bf16x8 frag_bf16(const char* region, int rb, int kk) {
  const int lane = threadIdx.x & 63;
  if constexpr (!MC) {
    constexpr int CPR = Cfg::BK * 2 / 16;
    return *reinterpret_cast<const bf16x8*>(region + kc_off<CPR>(rb + (lane & 31), (kk >> 3) + (lane >> 5)));
  } else {
    // 16-lane group g covers columns rb + 16 (g % 2) .. +15 and k kk + 8 (g / 2) .. +7,
    // read as two transposed 4-k halves
    constexpr int CPR = R * 2 / 16;
    const int g = lane >> 4, s = lane & 15;
    const int col = rb + 16 * (g & 1) + 4 * (s & 3);
    const int kr = kk + 8 * (g >> 1) + (s >> 2);
    const char* p0 = region + mc_off<CPR, 2>(kr, col >> 3) + (col & 7) * 2;
    const char* p1 = region + mc_off<CPR, 2>(kr + 4, col >> 3) + (col & 7) * 2;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p0));
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p1));
    bf16x8 out;
    const bf16* l4 = reinterpret_cast<const bf16*>(&lo);
    const bf16* h4 = reinterpret_cast<const bf16*>(&hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      out[e] = l4[e];
      out[e + 4] = h4[e];
    }
    return out;
  }
}

// fp32 MFMA operands: 4 k (kk + 4 * (lane / 32) + 0..3) of row/column rb + lane % 32.
template <class Cfg, int R, bool MC>
__device__ __forceinline__ f32x4 frag_f32(const char* region, int rb, int kk) {
  const int lane = threadIdx.x & 63;
  const int rc = rb + (lane & 31), k = kk + 4 * (lane >> 5);
  if constexpr (!MC) {
    constexpr int CPR = Cfg::BK * 4 / 16;
    return *reinterpret_cast<const f32x4*>(region + kc_off<CPR>(rc, k >> 2));
  } else {
    constexpr int CPR = R * 4 / 16;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = *reinterpret_cast<const float*>(region + mc_off<CPR, 4>(k + e, rc >> 2) + (rc & 3) * 4);
    return v;
  }
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  if constexpr (N == 0)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Fragments of one k step (16 bf16 or 8 fp32 k) of a wave's output tile, and
// the MFMAs that consume them.
template <class Cfg, bool AMC, bool BMC>
struct StepFrags {
  static constexpr int KSTEP = Cfg::ES == 2 ? 16 : 8;
  using FT = typename std::conditional<Cfg::ES == 2, bf16x8, f32x4>::type;
  FT a[Cfg::FM], b[Cfg::FN];

  __device__ __forceinline__ void load(const char* st, int wm, int wn, int kk) {
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) {
      if constexpr (Cfg::ES == 2)
        a[i] = frag_bf16<Cfg, Cfg::BM, AMC>(st, wm * Cfg::TM + 32 * i, kk);
      else
        a[i] = frag_f32<Cfg, Cfg::BM, AMC>(st, wm * Cfg::TM + 32 * i, kk);
    }
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j) {
      if constexpr (Cfg::ES == 2)
        b[j] = frag_bf16<Cfg, Cfg::BN, BMC>(st + Cfg::ABYTES, wn * Cfg::TN + 32 * j, kk);
      else
        b[j] = frag_f32<Cfg, Cfg::BN, BMC>(st + Cfg::ABYTES, wn * Cfg::TN + 32 * j, kk);
    }
  }

  // Adds the A values of this k step to per-lane row sums: with a
  // k-contiguous A, lane l holds k values of row rb + l % 32 only. bf16 pairs
  // go through v_dot2 against (1, 1), which needs no unpacked temporaries
  // (the 256x256 tile has no registers to spare).
  __device__ __forceinline__ void rowsum(float (&rs)[Cfg::FM]) const {
    static_assert(!AMC, "row sums need a k-contiguous A");
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) {
      if constexpr (Cfg::ES == 2) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 one = {static_cast<bf16>(1.0f), static_cast<bf16>(1.0f)};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pr = {a[i][2 * e], a[i][2 * e + 1]};
          rs[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, one, rs[i], false);
        }
      } else {
        rs[i] += (a[i][0] + a[i][1]) + (a[i][2] + a[i][3]);
      }
    }
  }

  // acc(m): the accumulators of MFMA m of this k step (one of 16 bf16 k, four of 2 fp32 k).
  template <class Accs>
  __device__ __forceinline__ void mma_to(Accs acc) const {
    if constexpr (Cfg::ES == 2) {
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
          acc(0)[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc(0)[i][j], 0, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
          for (int j = 0; j < Cfg::FN; ++j)
            acc(e)[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc(e)[i][j], 0, 0, 0);
    }
  }
  __device__ __forceinline__ void mma(f32x16 (&acc)[Cfg::FM][Cfg::FN]) const {
    mma_to([&](int) -> f32x16(&)[Cfg::FM][Cfg::FN] { return acc; });
  }
};

// A lane's sums of the A values that it reads (StepFrags::rowsum): a slab's in 32
// bits, those of the slabs in 64, for one lane adds an eighth or more of the
// whole contraction. A bias gradient over 1450 samples is then 6e-8 off its
// 64-bit value, 2.6e-7 with one chain in 32 bits. bf16 on direct loads keeps one
// chain in 32 bits: its values have 8 bits, its sums are 1e-8 off, and the 8192 x
// 8192 layer at batch 2048 takes 1% more time with a sum per slab.
template <class Cfg, int LD>
struct RowSums {
  static constexpr bool BY_SLAB = Cfg::ES == 4 || LD == LOAD_ANY;
  typename std::conditional<BY_SLAB, double, float>::type all[Cfg::FM];
  float slab[Cfg::FM];

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) all[i] = 0, slab[i] = 0.0f;
  }
  template <class Frags>
  __device__ __forceinline__ void add(const Frags& fr) {  // a k step's values
    if constexpr (BY_SLAB) fr.rowsum(slab);
    else fr.rowsum(all);
  }
  __device__ __forceinline__ void end_slab() {
    if constexpr (BY_SLAB) {
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) all[i] += slab[i], slab[i] = 0.0f;
    }
  }
};

// The accumulators of a wave. With CHAINS > 1 the MFMAs of a slab go to CHAINS
// sums in turn, added at the end: a fp32 sum's rounding error grows with the
// length of its chain of additions, and a tile that does not split its slab's
// k over waves would run one chain as long as the contraction.
template <class Cfg>
struct AccChains {
  using Acc = f32x16[Cfg::FM][Cfg::FN];
  Acc& first;
  f32x16 more[Cfg::CHAINS > 1 ? Cfg::CHAINS - 1 : 1][Cfg::FM][Cfg::FN];

  __device__ __forceinline__ explicit AccChains(Acc& acc) : first(acc) {
#pragma unroll
    for (int c = 0; c < Cfg::CHAINS - 1; ++c)
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) more[c][i][j][r] = 0.0f;
  }
  __device__ __forceinline__ Acc& of(int m) {  // MFMA m of the slab, a constant where it is used
    return m % Cfg::CHAINS == 0 ? first : more[m % Cfg::CHAINS - 1];
  }
  template <class Frags>
  __device__ __forceinline__ void mma(const Frags& fr, int s) {  // k step s of the slab
    constexpr int PER = Cfg::ES == 2 ? 1 : 4;                    // MFMAs of a k step per output block
    fr.mma_to([&](int e) -> Acc& { return of(PER * s + e); });
  }
  __device__ __forceinline__ void sum() {
    auto add = [](Acc& a, const Acc& b) {
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
        for (int j = 0; j < Cfg::FN; ++j) a[i][j] += b[i][j];
    };
    static_assert((Cfg::CHAINS & (Cfg::CHAINS - 1)) == 0, "pairwise sum");
#pragma unroll
    for (int w = 1; w < Cfg::CHAINS; w *= 2)
#pragma unroll
      for (int c = 0; c < Cfg::CHAINS; c += 2 * w) add(of(c), of(c + w));
  }
};

// The direct loads of one operand pair, slab after slab: wave-uniform
// pointers to the next slab's first element, its first k, its stage, and how
// many slabs of the split are still to come after it. Past the last slab the
// last one is loaded again (into a stage no longer read), so every wave issues
// the same number of loads per slab.
template <class Cfg, bool AMC, bool BMC>
struct SlabLoader {
  DmaSrc<Cfg, Cfg::BM, AMC> da;
  DmaSrc<Cfg, Cfg::BN, BMC> db;
  const char* na;
  const char* nb;
  int64_t a_step, b_step, a_wrap, b_wrap;
  int K, ik, is, left, wv;
  uint32_t lds0;

  // One slab's loads in two halves: A (issue_a), then B and the advance to
  // the next slab (issue_b); issue() does both.
  __device__ __forceinline__ void issue_a() {
    da.issue(na, K - ik, lds0 + static_cast<uint32_t>(is * Cfg::STAGE), wv);
  }
  __device__ __forceinline__ void issue_b() {
    db.issue(nb, K - ik, lds0 + static_cast<uint32_t>(is * Cfg::STAGE) + Cfg::ABYTES, wv);
    is = is + 1 == Cfg::STAGES ? 0 : is + 1;
    if (left > 0) {
      --left;
      na += a_step;
      nb += b_step;
      ik += Cfg::BK;
      if (ik >= K) ik = 0, na += a_wrap, nb += b_wrap;
    }
  }
  __device__ __forceinline__ void issue() {
    issue_a();
    issue_b();
  }
};

// The direct loads of a flat contraction (LOAD_FLAT): k = q * kb + r of a
// row lies at q * kbs + r, so a chunk's place in its row follows from k by one
// division (a multiply by 2^32 / kb, exact while k * kb < 2^32). Without it an
// LSTM's weight gradient, a sum over steps of products only a batch deep, runs
// every step's samples as a slab of its own, 20 of 32 or 64 k filled.
template <class Cfg, int R>
struct FlatSrc {
  static constexpr int ES = Cfg::ES, EPC = 16 / ES, CPR = Cfg::BK * ES / 16;
  static constexpr int PER_WAVE = R * Cfg::BK * ES / 1024 / Cfg::NW;
  uint32_t off[PER_WAVE];  // byte offset of the lane's row
  int k[PER_WAVE];         // the chunk's first k within the slab

  __device__ __forceinline__ void init(int64_t ld, int r0, int rext, int wave) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int pos = (wave * PER_WAVE + i) * 64 + lane;
      const int r = pos / CPR;
      off[i] = static_cast<uint32_t>((r0 + r < rext ? r0 + r : rext - 1) * ld * ES);
      k[i] = ((pos % CPR) ^ kc_swz<CPR>(r)) * EPC;
    }
  }
  // The chunks of the slab at k0 (past the contraction length: k 0, zeroed in LDS before use).
  __device__ __forceinline__ void issue(const char* base, int k0, int K, uint32_t kb, uint32_t magic, uint32_t kbs,
                                        uint32_t region, int wave) const {
    const char* b = uniform_ptr(base);
    const uint32_t r0 = region + static_cast<uint32_t>(wave * PER_WAVE * 1024);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const uint32_t kg = k0 + k[i] < K ? static_cast<uint32_t>(k0 + k[i]) : 0u;
      const uint32_t q = __umulhi(kg, magic);
      const uint32_t o = off[i] + (q * kbs + (kg - q * kb)) * ES;
      if (i == 0)
        dma16<true>(b, o, r0);
      else
        dma16<false>(b, o, r0 + static_cast<uint32_t>(i * 1024));
    }
  }
};

template <class Cfg>
struct FlatLoader {
  FlatSrc<Cfg, Cfg::BM> da;
  FlatSrc<Cfg, Cfg::BN> db;
  const char* na;
  const char* nb;
  uint32_t kb, magic, a_kbs, b_kbs;
  int K, ik, is, left, wv;
  uint32_t lds0;

  __device__ __forceinline__ void issue_a() {
    da.issue(na, ik, K, kb, magic, a_kbs, lds0 + static_cast<uint32_t>(is * Cfg::STAGE), wv);
  }
  __device__ __forceinline__ void issue_b() {
    db.issue(nb, ik, K, kb, magic, b_kbs, lds0 + static_cast<uint32_t>(is * Cfg::STAGE) + Cfg::ABYTES, wv);
    is = is + 1 == Cfg::STAGES ? 0 : is + 1;
    if (left > 0) --left, ik += Cfg::BK;
  }
  __device__ __forceinline__ void issue() {
    issue_a();
    issue_b();
  }
};

// Tile order. Workgroup i runs on XCD i % 8, each XCD with its own L2, so
// XCD x takes a contiguous run of positions t (xcd_position) in a grouped
// order: kGroupRows tile rows at a time, column by column within the group.
// The workgroups running together on one XCD then share a few A row panels
// and a few B column panels instead of each bringing its own. grouped_tile
// returns the tile row and column of workgroup bid in a grid of nx columns and
// ny rows.
__device__ __forceinline__ int xcd_position(int bid, int total) {
  const int xcd = bid % 8, per = total / 8, extra = total % 8;
  return xcd * per + (xcd < extra ? xcd : extra) + bid / 8;
}
// Tile row and column of position t of an nx x ny grid in the grouped order.
__device__ __forceinline__ void grouped_order(int t, int nx, int ny, int& row, int& col) {
  constexpr int kGroupRows = 8;
  const int first_row = (t / (kGroupRows * nx)) * kGroupRows;
  const int rows = ny - first_row < kGroupRows ? ny - first_row : kGroupRows;
  const int local = t % (kGroupRows * nx);
  col = local / rows;
  row = first_row + local % rows;
}
__device__ __forceinline__ void grouped_tile(int bid, int nx, int ny, int& row, int& col) {
  grouped_order(xcd_position(bid, nx * ny), nx, ny, row, col);
}

// The slab pipeline of one workgroup: nslab slabs that the loader issues one
// after the other into STAGES LDS stages. Each wave waits only for its own
// loads of the slab it is about to read (vmcnt: exactly (STAGES - 2) * LPW
// younger loads are allowed), then a barrier makes every wave's loads of that
// slab visible and certifies that all waves have finished reading the
// previous slab, whose stage takes the next load. Fragments are
// double-buffered in registers: the reads of the next k step (the first step
// of the next slab, behind the barrier) are issued before the MFMAs of the
// current one, so LDS latency and the barrier overlap MFMA execution. The
// loads issued at a barrier are split: the A half right behind it, the B half
// after the MFMAs of the slab's first k step, so that the waves do not all
// queue at the load unit at once while the matrix cores wait (measured on
// MI355X: 13% fewer cycles per slab for the 256x256 tile).
// With TAIL, ck is the first k of the first slab within a contraction of
// length K (slabs wrap to k 0 past K), and a slab with fewer than BK valid k
// is zeroed past them in LDS before use. With RSUM, rs also sums the A
// values the lane reads (RowSums). Returns with no direct load in
// flight.
template <class Cfg, bool AMC, bool BMC, bool TAIL, bool RSUM = false, class Loader>
__device__ __forceinline__ void run_slabs(Loader& ld, int nslab, int K, int ck, f32x16 (&acc)[Cfg::FM][Cfg::FN],
                                          int wm, int wn, int kw0, char* smem, RowSums<Cfg, LOAD_DMA>* rs = nullptr) {
  using Frags = StepFrags<Cfg, AMC, BMC>;
  constexpr int STEPS = Cfg::KW / Frags::KSTEP;
  static_assert(STEPS % 2 == 0, "a slab holds an even number of k steps");
  static_assert((Cfg::ES == 2 ? STEPS : 4 * STEPS) % Cfg::CHAINS == 0, "every chain takes as many MFMAs of a slab");
  AccChains<Cfg> ch(acc);
  int cs = 0;  // stage of the slab being computed
  Frags fr[2];
  char* st = smem;
  if (nslab > 0) {
#pragma unroll
    for (int s = 0; s < Cfg::STAGES - 1; ++s) ld.issue();
    wait_vm<(Cfg::STAGES - 2) * Cfg::LPW>();
    lds_barrier();
    if (TAIL && K - ck < Cfg::BK) {
      fast_zero_tail<Cfg, Cfg::BM, AMC>(st, K - ck);
      fast_zero_tail<Cfg, Cfg::BN, BMC>(st + Cfg::ABYTES, K - ck);
      lds_barrier();
    }
    ld.issue_a();  // B half after the first k step below
    fr[0].load(st, wm, wn, kw0);
  }
  // all slabs but the last one: the last k step crosses into the next slab
  for (int q = 0; q < nslab - 1; ++q) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) {
        fr[(s + 1) & 1].load(st, wm, wn, kw0 + (s + 1) * Frags::KSTEP);
      } else {
        cs = cs + 1 == Cfg::STAGES ? 0 : cs + 1;
        if (TAIL) {
          ck += Cfg::BK;
          if (ck >= K) ck = 0;
        }
        st = smem + cs * Cfg::STAGE;
        wait_vm<(Cfg::STAGES - 2) * Cfg::LPW>();
        lds_barrier();  // slab q + 1 visible; slab q read by no wave any more
        if (TAIL && K - ck < Cfg::BK) {
          fast_zero_tail<Cfg, Cfg::BM, AMC>(st, K - ck);
          fast_zero_tail<Cfg, Cfg::BN, BMC>(st + Cfg::ABYTES, K - ck);
          lds_barrier();
        }
        ld.issue_a();  // into the stage of slab q; B half after the next slab's first k step
        fr[(s + 1) & 1].load(st, wm, wn, kw0);
      }
      ch.mma(fr[s & 1], s);
      if constexpr (RSUM) {
        rs->add(fr[s & 1]);
        if (s + 1 == STEPS) rs->end_slab();
      }
      if (s == 0) ld.issue_b();
    }
  }
  if (nslab > 0) {  // the last slab (a separate copy keeps the loop body's LDS waits exact)
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) fr[(s + 1) & 1].load(st, wm, wn, kw0 + (s + 1) * Frags::KSTEP);
      ch.mma(fr[s & 1], s);
      if constexpr (RSUM) {
        rs->add(fr[s & 1]);
        if (s + 1 == STEPS) rs->end_slab();
      }
      if (s == 0) ld.issue_b();
    }
  }
  ch.sum();
  wait_vm<0>();  // no direct load may still write LDS past this point
}

// ------------------------------------------------------------------------
// The same GEMM for views whose rows start at any element (a batch or a row
// length that is no multiple of 16 bytes). A direct load moves whole 16-byte
// aligned chunks only, so here the slab passes through registers: every lane
// loads its chunks with 16-byte loads of element alignment (whole lines all
// the same: consecutive lanes read consecutive chunks) and writes them to the
// LDS position that the direct load would have filled. Two slabs are in
// flight in registers while a third is computed from LDS. A chunk that
// reaches past the extent is loaded element by element and padded with zeros:
// nothing past a row's last valid element is read, and no zeroing pass over a
// partial slab is needed.
// Bound by the latency of a slab's loads at small sizes, like the direct-load
// kernels. It replaced the general kernel's element loads (one load
// instruction per element instead of one per 4 fp32 or 8 bf16, with 64-bit
// address arithmetic in each). One layer's forward and backward on MI355X:
// bf16 batch 100, 1023 -> 1537: 63 -> 42 us; fp32 batch 330, 6566 -> 114:
// 126 -> 55 us; bf16 batch 860, 1586 -> 408: 83 -> 32 us.

// Sixteen bytes at an address aligned to ES bytes only.
template <int ES>
__device__ __forceinline__ u32x4 load16_any(const char* p) {
  typedef u32x4 u32x4_a2 __attribute__((aligned(2), may_alias));
  typedef u32x4 u32x4_a4 __attribute__((aligned(4), may_alias));
  if constexpr (ES == 2)
    return *reinterpret_cast<const u32x4_a2*>(p);
  else
    return *reinterpret_cast<const u32x4_a4*>(p);
}

// The first n (< 16 / ES) elements at p, zeros behind them.
template <int ES>
__device__ __forceinline__ u32x4 load16_part(const char* p, int n) {
  u32x4 x = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 16 / ES; ++e) {
    if (e < n) {
      if constexpr (ES == 4)
        x[e] = *reinterpret_cast<const uint32_t*>(p + 4 * e);
      else
        x[e / 2] |= static_cast<uint32_t>(*reinterpret_cast<const uint16_t*>(p + 2 * e)) << (16 * (e & 1));
    }
  }
  return x;
}

// DmaSrc's chunk-to-LDS assignment with loads into registers.
template <class Cfg, int R, bool MC>
struct RegSrc {
  static constexpr int ES = Cfg::ES, EPC = 16 / ES;
  static constexpr int CPR = MC ? R * ES / 16 : Cfg::BK * ES / 16;
  static constexpr int PER_WAVE = R * Cfg::BK * ES / 1024 / Cfg::NW;
  uint32_t off[PER_WAVE];  // byte offset of the lane's chunk from the slab base
  int k[PER_WAVE];         // the chunk's first k (KC) or its k-row (MC) within the slab
  int nv[PER_WAVE];        // MC: valid columns of the chunk, <= 0 none

  __device__ __forceinline__ void init(int64_t ld, int r0, int rext, int wave) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int pos = (wave * PER_WAVE + i) * 64 + lane;
      if constexpr (!MC) {
        const int r = pos / CPR;
        const int c = (pos % CPR) ^ kc_swz<CPR>(r);
        const int row = r0 + r < rext ? r0 + r : rext - 1;  // past the extent: a valid row, its results are discarded
        off[i] = static_cast<uint32_t>(row * ld * ES) + static_cast<uint32_t>(c * 16);
        k[i] = c * EPC;
      } else {
        const int kk = pos / CPR;
        const int c = (pos % CPR) ^ mc_swz<CPR, ES>(kk);
        const int col = r0 + c * EPC;
        off[i] = static_cast<uint32_t>(kk * ld * ES) + static_cast<uint32_t>(col * ES);
        k[i] = kk;
        nv[i] = rext - col;
      }
    }
  }

  // As DmaSrc::init_rows.
  template <class F>
  __device__ __forceinline__ void init_rows(int64_t ld, F rowof, int wave) {
    static_assert(!MC, "row gather of a k-contiguous operand");
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int pos = (wave * PER_WAVE + i) * 64 + lane;
      const int r = pos / CPR;
      const int c = (pos % CPR) ^ kc_swz<CPR>(r);
      off[i] = static_cast<uint32_t>(static_cast<int64_t>(rowof(r)) * ld * ES) + static_cast<uint32_t>(c * 16);
      k[i] = c * EPC;
    }
  }

  // The slab whose first element is at base, of which the first kv k (k-rows) are valid.
  __device__ __forceinline__ void load(const char* base, int kv, u32x4 (&v)[PER_WAVE]) const {
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int n = MC ? (k[i] < kv ? nv[i] : 0) : kv - k[i];
      if (n >= EPC)
        v[i] = load16_any<ES>(base + off[i]);
      else
        v[i] = load16_part<ES>(base + off[i], n);
    }
  }

  __device__ __forceinline__ void store(char* region, int wave, const u32x4 (&v)[PER_WAVE]) const {
    char* p = region + wave * PER_WAVE * 1024 + (threadIdx.x & 63) * 16;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) *reinterpret_cast<u32x4*>(p + i * 1024) = v[i];
  }
};

// SlabLoader's walk over the slabs with register loads.
template <class Cfg, bool AMC, bool BMC>
struct RegLoader {
  using SrcA = RegSrc<Cfg, Cfg::BM, AMC>;
  using SrcB = RegSrc<Cfg, Cfg::BN, BMC>;
  struct Regs {
    u32x4 a[SrcA::PER_WAVE], b[SrcB::PER_WAVE];
  };
  SrcA da;
  SrcB db;
  const char* na;
  const char* nb;
  int64_t a_step, b_step, a_wrap, b_wrap;
  int K, ik, wv;

  __device__ __forceinline__ void load(Regs& r) {  // the next slab, then the advance
    da.load(na, K - ik, r.a);
    db.load(nb, K - ik, r.b);
    na += a_step;
    nb += b_step;
    ik += Cfg::BK;
    if (ik >= K) ik = 0, na += a_wrap, nb += b_wrap;
  }
  __device__ __forceinline__ void store(char* stage, const Regs& r) const {
    da.store(stage, wv, r.a);
    db.store(stage + Cfg::ABYTES, wv, r.b);
  }
};

// The slab pipeline on register loads: slab q is computed from LDS stage
// q % 2 while slabs q + 1 and q + 2 are on their way in registers; one
// barrier per slab.
template <class Cfg, bool AMC, bool BMC, bool RSUM>
__device__ __forceinline__ void run_slabs_reg(RegLoader<Cfg, AMC, BMC>& ld, int nslab,
                                              f32x16 (&acc)[Cfg::FM][Cfg::FN], int wm, int wn, int kw0, char* smem,
                                              RowSums<Cfg, LOAD_ANY>* rs) {
  using Frags = StepFrags<Cfg, AMC, BMC>;
  constexpr int STEPS = Cfg::KW / Frags::KSTEP;
  static_assert(Cfg::STAGES >= 2, "two LDS stages");
  static_assert((Cfg::ES == 2 ? STEPS : 4 * STEPS) % Cfg::CHAINS == 0, "every chain takes as many MFMAs of a slab");
  if (nslab <= 0) return;
  AccChains<Cfg> ch(acc);
  typename RegLoader<Cfg, AMC, BMC>::Regs buf[2];
  ld.load(buf[0]);
  if (nslab > 1) ld.load(buf[1]);
  ld.store(smem, buf[0]);
  if (nslab > 2) ld.load(buf[0]);
  lds_barrier();
  auto slab = [&](int q, int par) {  // par = q % 2, a constant where it is used
    const char* st = smem + par * Cfg::STAGE;
    Frags fr[2];
    fr[0].load(st, wm, wn, kw0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) fr[(s + 1) & 1].load(st, wm, wn, kw0 + (s + 1) * Frags::KSTEP);
      ch.mma(fr[s & 1], s);
      if constexpr (RSUM) {
        rs->add(fr[s & 1]);
        if (s + 1 == STEPS) rs->end_slab();
      }
    }
    if (q + 1 < nslab) ld.store(smem + (par ^ 1) * Cfg::STAGE, buf[par ^ 1]);
    if (q + 3 < nslab) ld.load(buf[par ^ 1]);
    lds_barrier();  // slab q + 1 is in LDS; no wave reads slab q any more
  };
  for (int q = 0; q < nslab; q += 2) {
    slab(q, 0);
    if (q + 1 < nslab) slab(q + 1, 1);
  }
  ch.sum();
}

// Output of one wave's accumulator tile. Each block row of 32 rows passes
// through the wave's own LDS region in fp32 (epilogue applied on the way in),
// and every lane then writes 4 consecutive values of one output row (16 bytes
// fp32, 8 bytes bf16): a store instruction covers whole 128-byte lines instead
// of one element per lane. The ReLU gate of the layer below is read the same
// way. Falls back to element stores when the output rows are not contiguous
// or not aligned for those pieces. Called by all waves (it holds a barrier).
template <typename OutT, class Cfg, int EPI>
__device__ __forceinline__ void fast_store(const GemmArgs& g, f32x16 (&acc)[Cfg::FM][Cfg::FN], int m0, int n0,
                                           int wm, int wn, int64_t bz, int split, char* smem) {
  const bool part = g.splits > 1;
  const int64_t es = part ? 4 : static_cast<int64_t>(sizeof(OutT));
  const int64_t ld = part ? g.N : g.c.ld;
  char* base = part ? reinterpret_cast<char*>(g.partial + (bz * g.splits + split) * static_cast<int64_t>(g.M) * g.N)
                    : reinterpret_cast<char*>(static_cast<OutT*>(g.c.p) + bz * g.c.bstride);
  const char* gate = (!part && EPI != EPI_STORE && g.c.gate)
                         ? reinterpret_cast<const char*>(static_cast<const OutT*>(g.c.gate) + bz * g.c.bstride)
                         : nullptr;
  const int64_t piece = 4 * es;
  const bool vec = (part || (g.c.cidx == nullptr && g.c.col_stride <= 1 && g.c.ridx == nullptr)) &&
                   (EPI != EPI_COLS || (g.c_nstride % 4 == 0 && g.nvalid % 4 == 0)) && (ld * es) % piece == 0 &&
                   reinterpret_cast<uintptr_t>(base) % piece == 0 &&
                   reinterpret_cast<uintptr_t>(gate) % piece == 0;
  if (!vec) {
    store_tile<OutT, Cfg, EPI>(g, acc, m0, n0, wm, wn, bz, split);
    return;
  }
  // fp32 rows of TN values plus 32 bytes: the two half-waves' writes (rows r
  // and r + 4) then fall on disjoint banks
  constexpr int ROW = Cfg::TN * 4 + 32;
  constexpr int CPRW = Cfg::TN / 4;  // 16-byte pieces per row
  constexpr int RPI = 64 / CPRW;     // rows per read instruction
  // the bias of the wave's TM rows sits behind the staging regions
  static_assert(Cfg::NW * (32 * ROW + Cfg::TM * 4) <= Cfg::LDS, "epilogue staging exceeds LDS");
  static_assert(Cfg::KSPLIT > 1 || Cfg::NW * (32 * ROW + Cfg::TM * 4) == Cfg::ENDS, "epilogue staging");
  lds_barrier();  // every wave is done with the stages
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lr = lane & 31, lh = lane >> 5;
  char* region = smem + wave * 32 * ROW;
  const int m0w = m0 + wm * Cfg::TM, n0w = n0 + wn * Cfg::TN;
  // The bias entries of the wave's rows, loaded once with every load in
  // flight together (a load per accumulator row, each waited for before its
  // row's values are staged, cost ~4 us per call of a small product), then
  // read from LDS: the wave reads only what it wrote itself.
  const bool has_bias = !part && EPI != EPI_STORE && g.c.bias;
  float* bias_lds = reinterpret_cast<float*>(smem + Cfg::NW * 32 * ROW) + wave * Cfg::TM;
  if (has_bias) {
    float bv[(Cfg::TM + 63) / 64];
#pragma unroll
    for (int e = 0; e * 64 < Cfg::TM; ++e) {
      const int m = m0w + e * 64 + lane;
      bv[e] = (e * 64 + lane < Cfg::TM && m < g.M) ? g.c.bias[bias_row(g.c, m)] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e * 64 < Cfg::TM; ++e)
      if (e * 64 + lane < Cfg::TM) bias_lds[e * 64 + lane] = bv[e];
  }
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = 8 * (r >> 2) + 4 * lh + (r & 3);
      const float bias = has_bias ? bias_lds[32 * i + rl] : 0.0f;
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j) {
        float v = acc[i][j][r];
        if (!part) v = epilogue<EPI>(g.c, v, bias);
        *reinterpret_cast<float*>(region + rl * ROW + (32 * j + lr) * 4) = v;
      }
    }
    // the ReLU gate of the rows this lane writes, every load issued before
    // the first store (the stores may alias the gate as far as the compiler
    // knows, so loads between them would each wait for the one before)
    typedef typename std::conditional<sizeof(OutT) == 2, uint2, f32x4>::type GateT;
    GateT gpre[32 / RPI];
    if (gate) {
#pragma unroll
      for (int t = 0; t < 32 / RPI; ++t) {
        const int rl = lane / CPRW + RPI * t, ch = lane % CPRW;
        const int m = m0w + 32 * i + rl, n = n0w + 4 * ch;
        if (m < g.M && n + 3 < g.N)
          gpre[t] = *reinterpret_cast<const GateT*>(reinterpret_cast<const OutT*>(gate) +
                                                    static_cast<int64_t>(m) * ld + n);
      }
    }
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) {
      const int rl = lane / CPRW + RPI * t, ch = lane % CPRW;
      const f32x4 v = *reinterpret_cast<const f32x4*>(region + rl * ROW + ch * 16);
      const int m = m0w + 32 * i + rl, n = n0w + 4 * ch;
      if (m >= g.M) continue;
      if (EPI == EPI_COLS && !part && !col_in<EPI>(g, n)) continue;
      const int64_t o = static_cast<int64_t>(m) * ld + (EPI == EPI_COLS && !part ? out_col<EPI>(g, n) : n);
      if (part) {
        float* out = reinterpret_cast<float*>(base) + o;
        if (n + 3 < g.N) {
          *reinterpret_cast<f32x4*>(out) = v;
        } else {
          for (int e = 0; e < 4; ++e)
            if (n + e < g.N) out[e] = v[e];
        }
        continue;
      }
      OutT* out = reinterpret_cast<OutT*>(base) + o;
      const OutT* gt = gate ? reinterpret_cast<const OutT*>(gate) + o : nullptr;
      if (n + 3 < g.N) {
        OutT w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = from_f32<OutT>(v[e]);
        if (gt) {
          OutT gv[4];
          *reinterpret_cast<GateT*>(gv) = gpre[t];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!(to_f32(gv[e]) > 0.0f)) w[e] = from_f32<OutT>(0.0f);
        }
        if constexpr (sizeof(OutT) == 2)
          *reinterpret_cast<uint2*>(out) = *reinterpret_cast<const uint2*>(w);
        else
          *reinterpret_cast<f32x4*>(out) = *reinterpret_cast<const f32x4*>(w);
      } else {
        for (int e = 0; e < 4; ++e) {
          if (n + e >= g.N) break;
          float x = v[e];
          if (gt && !(to_f32(gt[e]) > 0.0f)) x = 0.0f;
          out[e] = from_f32<OutT>(x);
        }
      }
    }
  }
}

// Row sums of A (RSUM, see GemmArgs::rsum) for the tile row of a workgroup
// in tile column 0: lanes l and l + 32 of a wave hold the two k halves of
// row 32 i + l % 32, the waves of a k split are added in LDS in split order.
// One workgroup's output tile: position bid of an nx x ny tile grid in the
// grouped order, batch-and-split index bzs.
template <class Cfg, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM = false, int LD = LOAD_DMA>
__device__ __forceinline__ void fast_gemm_tile(const GemmArgs& g, int tile_row, int tile_col, int bzs, char* smem) {
  using T = typename Cfg::T;
  const int n0 = tile_col * Cfg::BN;
  const int m0 = tile_row * Cfg::BM;
  const int splits = g.splits > 1 ? g.splits : 1;
  const int64_t bz = splits > 1 ? bzs / splits : bzs;
  const int split = splits > 1 ? bzs % splits : 0;
  const int wave = threadIdx.x >> 6;
  const int ks = wave / (Cfg::WGM * Cfg::WGN);
  const int wmn = wave % (Cfg::WGM * Cfg::WGN);
  const int wm = wmn / Cfg::WGN, wn = wmn % Cfg::WGN;

  const T* abase = static_cast<const T*>(g.a.p) + bz * g.a.bstride;
  const T* bbase = static_cast<const T*>(g.b.p) + bz * g.b.bstride;

  f32x16 acc[Cfg::FM][Cfg::FN];
#pragma unroll
  for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  const int kbatch = g.kbatch > 0 ? g.kbatch : 1;
  const int klen = LD == LOAD_FLAT ? kbatch * g.K : g.K;  // length of one run of slabs
  const int nks = (klen + Cfg::BK - 1) / Cfg::BK;
  const int nslab = LD == LOAD_FLAT ? nks : kbatch * nks;
  // slabs of this split (32-bit divisions: nslab * splits < 2^31; none without a split)
  int q0 = 0, q1 = nslab;
  if (splits > 1) {
    q0 = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(nslab * split) / splits));
    q1 = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(nslab * (split + 1)) / splits));
  }

  // slabs q0 .. q1 - 1 of this split
  static_assert(DmaSrc<Cfg, Cfg::BM, AMC>::PER_WAVE + DmaSrc<Cfg, Cfg::BN, BMC>::PER_WAVE == Cfg::LPW, "load count");
  constexpr int ES = Cfg::ES;
  RowSums<Cfg, LD == LOAD_ANY ? LOAD_ANY : LOAD_DMA> rs;
  rs.clear();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (LD == LOAD_FLAT) {
    static_assert(!AMC && !BMC, "k-contiguous operands");
    FlatLoader<Cfg> ld;
    ld.wv = wv;
    ld.lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));
    if (q0 < q1) {
      ld.da.init(g.a.ld, m0, g.M, wv);
      ld.db.init(g.b.ld, n0, g.N, wv);
    }
    ld.kb = static_cast<uint32_t>(g.K);
    ld.magic = static_cast<uint32_t>(((uint64_t{1} << 32) + ld.kb - 1) / ld.kb);
    ld.a_kbs = static_cast<uint32_t>(g.a.kbstride);
    ld.b_kbs = static_cast<uint32_t>(g.b.kbstride);
    ld.na = uniform_ptr(reinterpret_cast<const char*>(abase));
    ld.nb = uniform_ptr(reinterpret_cast<const char*>(bbase));
    ld.K = klen;
    ld.ik = q0 * Cfg::BK;
    ld.is = 0;
    ld.left = q1 - q0 - 1;
    run_slabs<Cfg, AMC, BMC, true, RSUM>(ld, q1 - q0, klen, ld.ik, acc, wm, wn, ks * Cfg::KW, smem, &rs);
  } else {
    using Loader = typename std::conditional<LD == LOAD_ANY, RegLoader<Cfg, AMC, BMC>, SlabLoader<Cfg, AMC, BMC>>::type;
    Loader ld;
    ld.wv = wv;
    if (q0 < q1) {
      ld.da.init(g.a.ld, m0, g.M, ld.wv);
      if constexpr (EPI == EPI_COLS && LD == LOAD_DMA)
        ld.db.init(g.b.ld, n0, g.N, ld.wv, g.nblk, g.b_nstride);
      else
        ld.db.init(g.b.ld, n0, g.N, ld.wv);
    }
    ld.K = g.K;
    ld.a_step = (AMC ? g.a.ld : 1) * Cfg::BK * ES;
    ld.b_step = (BMC ? g.b.ld : 1) * Cfg::BK * ES;
    ld.a_wrap = g.a.kbstride * ES - nks * ld.a_step;
    ld.b_wrap = g.b.kbstride * ES - nks * ld.b_step;
    const int ib = q0 == 0 ? 0 : q0 / (nks > 0 ? nks : 1);
    ld.ik = (q0 - ib * nks) * Cfg::BK;
    ld.na = uniform_ptr(reinterpret_cast<const char*>(abase) + (ib * g.a.kbstride) * ES + ld.ik / Cfg::BK * ld.a_step);
    ld.nb = uniform_ptr(reinterpret_cast<const char*>(bbase) + (ib * g.b.kbstride) * ES + ld.ik / Cfg::BK * ld.b_step);
    if constexpr (LD == LOAD_ANY) {
      run_slabs_reg<Cfg, AMC, BMC, RSUM>(ld, q1 - q0, acc, wm, wn, ks * Cfg::KW, smem, &rs);
    } else {
      ld.lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));
      ld.is = 0;
      ld.left = q1 - q0 - 1;
      run_slabs<Cfg, AMC, BMC, true, RSUM>(ld, q1 - q0, g.K, ld.ik, acc, wm, wn, ks * Cfg::KW, smem, &rs);
    }
  }
  const int rlane = threadIdx.x & 63;
  if constexpr (RSUM) {
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i) rs.all[i] += __shfl_xor(rs.all[i], 32);
  }
  const bool rs_out = RSUM && splits == 1 && tile_col == 0 && wn == 0 && rlane < 32;
  auto put_rsum = [&](int i, float v) {
    const int m = m0 + wm * Cfg::TM + 32 * i + rlane;
    if (m < g.M) g.rsum[bz * g.rsum_bstride + static_cast<int64_t>(m) * g.rsum_ld] = g.c.scale * v;
  };
  if constexpr (Cfg::KSPLIT == 1) {
    if (rs_out) {
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) put_rsum(i, static_cast<float>(rs.all[i]));
    }
    fast_store<OutT, Cfg, EPI>(g, acc, m0, n0, wm, wn, bz, split, smem);
  } else {
    // the KSPLIT waves of one output tile reduce through LDS; wave ks finishes
    // the accumulator registers t (flattened over i, j, r) with t % KSPLIT == ks
    constexpr int NREG = Cfg::FM * Cfg::FN * 16;
    static_assert((Cfg::KSPLIT * Cfg::WGM * Cfg::WGN * NREG * 64 + Cfg::KSPLIT * Cfg::WGM * Cfg::FM * 32) * 4 <=
                      Cfg::ENDS,
                  "reduction buffer");
    static_assert((RSUM ? Cfg::ENDS : Cfg::KSPLIT * Cfg::WGM * Cfg::WGN * NREG * 64 * 4) <= Cfg::LDS,
                  "reduction buffer exceeds LDS");
    float* red = reinterpret_cast<float*>(smem);
    const int lane = threadIdx.x & 63;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Cfg::FM; ++i)
#pragma unroll
      for (int j = 0; j < Cfg::FN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          red[((ks * Cfg::WGM * Cfg::WGN + wmn) * NREG + (i * Cfg::FN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    // row sums of the k splits after the accumulators: [KSPLIT][WGM][FM][32]
    float* rred = red + Cfg::KSPLIT * Cfg::WGM * Cfg::WGN * NREG * 64;
    if constexpr (RSUM) {
      if (wn == 0 && lane < 32) {
#pragma unroll
        for (int i = 0; i < Cfg::FM; ++i)
          rred[((ks * Cfg::WGM + wm) * Cfg::FM + i) * 32 + lane] = static_cast<float>(rs.all[i]);
      }
    }
    __syncthreads();
    if (rs_out && ks == 0) {
#pragma unroll
      for (int i = 0; i < Cfg::FM; ++i) {
        float v = 0.0f;
#pragma unroll
        for (int u = 0; u < Cfg::KSPLIT; ++u) v += rred[((u * Cfg::WGM + wm) * Cfg::FM + i) * 32 + lane];
        put_rsum(i, v);
      }
    }
    const int lr = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int t = ks; t < NREG; t += Cfg::KSPLIT) {
      const int i = t / (Cfg::FN * 16), j = (t / 16) % Cfg::FN, r = t % 16;
      float v = 0.0f;
#pragma unroll
      for (int u = 0; u < Cfg::KSPLIT; ++u) v += red[((u * Cfg::WGM * Cfg::WGN + wmn) * NREG + t) * 64 + lane];
      const int m = m0 + wm * Cfg::TM + 32 * i + 8 * (r >> 2) + 4 * lh + (r & 3);
      const int n = n0 + wn * Cfg::TN + 32 * j + lr;
      if (m >= g.M || n >= g.N || !col_in<EPI>(g, n)) continue;
      if (splits > 1) {
        g.partial[(bz * splits + split) * static_cast<int64_t>(g.M) * g.N + static_cast<int64_t>(m) * g.N + n] = v;
        continue;
      }
      const int64_t orow = gather(g.c.ridx, m);
      const float bias = (EPI != EPI_STORE && g.c.bias) ? g.c.bias[bias_row(g.c, m)] : 0.0f;
      const int64_t o = orow * g.c.ld + out_col<EPI>(g, n);
      v = epilogue<EPI>(g.c, v, bias);
      if (EPI != EPI_STORE && g.c.gate && !(to_f32(static_cast<const OutT*>(g.c.gate)[bz * g.c.bstride + o]) > 0.0f))
        v = 0.0f;
      (static_cast<OutT*>(g.c.p) + bz * g.c.bstride)[o] = from_f32<OutT>(v);
    }
  }
}

// The grid is nx x ny output tiles times nz (batch entries times k splits).
// When every z-slice reads its own operands (a split contraction, or a batch
// with no operand shared between entries), XCD positions run over the whole
// grid, z-major: a z-slice goes to as few XCDs as possible, so that the
// workgroups on one XCD share the A and B panels of one slice (split z on
// XCD z when the tiles of a slice are a multiple of 8) instead of each XCD
// holding a few tiles of every slice. When an operand is shared by the batch
// entries (batch stride 0), positions run within each slice: XCD x then holds
// the same tiles of every entry and the shared panels stay in its L2.
template <class Cfg, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM = false, int LD = LOAD_DMA>
__global__ void __launch_bounds__(Cfg::NT) fast_gemm_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nx = gridDim.x, ny = gridDim.y, nxy = nx * ny;
  int tile_row, tile_col, z;
  if (gridDim.z > 1 && g.splits <= 1 && (g.a.bstride == 0 || g.b.bstride == 0)) {
    grouped_tile(blockIdx.y * nx + blockIdx.x, nx, ny, tile_row, tile_col);
    z = blockIdx.z;
  } else {
    const int bid = (blockIdx.z * ny + blockIdx.y) * nx + blockIdx.x;
    const int t = xcd_position(bid, nxy * gridDim.z);
    grouped_order(t % nxy, nx, ny, tile_row, tile_col);
    z = t / nxy;
  }
  fast_gemm_tile<Cfg, AMC, BMC, OutT, EPI, RSUM, LD>(g, tile_row, tile_col, z, smem);
}

// Two independent GEMMs of one configuration in one launch (no batch, no k
// split): the first workgroups take the tiles of g1, the rest those of g2.
// One launch instead of two saves a kernel's fixed start and drain time, and
// two problems too small to fill the chip alone run side by side.
template <class Cfg, bool AMC1, bool BMC1, typename OutT1, int EPI1, bool RSUM1, bool AMC2, bool BMC2,
          typename OutT2, int EPI2, bool RSUM2, int LD = LOAD_DMA>
__global__ void __launch_bounds__(Cfg::NT) fast_gemm_pair_kernel(GemmArgs g1, GemmArgs g2) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nx1 = (g1.N + Cfg::BN - 1) / Cfg::BN, ny1 = (g1.M + Cfg::BM - 1) / Cfg::BM;
  const int b = static_cast<int>(blockIdx.x);
  int row, col;
  if (b < nx1 * ny1) {
    grouped_tile(b, nx1, ny1, row, col);
    fast_gemm_tile<Cfg, AMC1, BMC1, OutT1, EPI1, RSUM1, LD>(g1, row, col, 0, smem);
  } else {
    const int nx2 = (g2.N + Cfg::BN - 1) / Cfg::BN, ny2 = (g2.M + Cfg::BM - 1) / Cfg::BM;
    grouped_tile(b - nx1 * ny1, nx2, ny2, row, col);
    fast_gemm_tile<Cfg, AMC2, BMC2, OutT2, EPI2, RSUM2, LD>(g2, row, col, 0, smem);
  }
}

// Whether a problem can run on fast_gemm_kernel with operand A m-contiguous
// (AMC) or not, B n-contiguous (BMC) or not: every operand is a plain strided
// view read in whole 16-byte chunks, and every chunk of a slab lies less than
// 2^31 bytes past the slab's first element (the lanes' 32-bit load offsets;
// the slab base itself is a 64-bit pointer). A slab of a k-contiguous operand
// spans rows 0 .. ext - 1 of ld elements, BK <= 256 k each; one of an
// m/n-contiguous operand spans at most 256 k-rows of ld elements and columns
// 0 .. ext - 1.
template <bool AMC, bool BMC>
inline bool fast_ok(const GemmArgs& g, size_t esize) {
  const int64_t epc = static_cast<int64_t>(16 / esize);
  auto ok = [epc, esize](const GemmOperand& o, int ext, bool mc) {
    const int64_t e = ext > 0 ? ext : 1;
    const int64_t span = mc ? e + 256 * o.ld : (e - 1) * o.ld + 256;
    return o.ridx == nullptr && o.cidx == nullptr && o.y == nullptr && o.ld % epc == 0 && o.bstride % epc == 0 &&
           o.kbstride % epc == 0 && (reinterpret_cast<uintptr_t>(o.p) & 15u) == 0 && o.ld >= 0 &&
           span * static_cast<int64_t>(esize) < (int64_t{1} << 31);
  };
  return ok(g.a, g.M, AMC) && ok(g.b, g.N, BMC);
}

// Whether a problem can run on the register-load variant: plain strided views
// (no gather, no load-time gate) with the same bound on a slab's span, rows
// starting at any element.
template <bool AMC, bool BMC>
inline bool any_ok(const GemmArgs& g, size_t esize) {
  auto ok = [esize](const GemmOperand& o, int ext, bool mc) {
    const int64_t e = ext > 0 ? ext : 1;
    const int64_t span = mc ? e + 256 * o.ld : (e - 1) * o.ld + 256;
    return o.ridx == nullptr && o.cidx == nullptr && o.y == nullptr && o.ld >= 0 &&
           span * static_cast<int64_t>(esize) < (int64_t{1} << 31);
  };
  return ok(g.a, g.M, AMC) && ok(g.b, g.N, BMC);
}

// Configurations: large tiles for large grids, 32x32 tiles with the k of each
// slab split over the waves (4 for bf16, 8 for fp32) for small grids.
template <typename T>
struct FastCfgs;
template <>
struct FastCfgs<bf16> {
  using Huge = FastCfg<bf16, 256, 256, 64, 2, 2, 4, 1>;   // 128 KB LDS, 8 waves (2 per SIMD)
  using Wide = FastCfg<bf16, 128, 256, 32, 4, 2, 4, 1>;   // 96 KB, 8 waves
  using Tall = FastCfg<bf16, 256, 128, 32, 4, 4, 2, 1>;   // 96 KB, 8 waves
  using Big = FastCfg<bf16, 128, 128, 64, 3, 2, 2, 1>;    // 96 KB
  using Small = FastCfg<bf16, 32, 32, 128, 4, 1, 1, 4>;   // 64 KB
};
template <>
struct FastCfgs<float> {
  // Mid, Duo and Huge leave room for two or three workgroups on a compute unit:
  // one's MFMAs run while another waits for its first slabs or stores. Big and
  // Small are for grids of at most one. Measured on MI355X over 1236 products, the
  // time over the best of all: without Big 1.0002 (but up to 1.07), without Duo
  // 1.0010, without Mid 1.027, without Huge 1.0024. Huge with four stages is no
  // faster with one workgroup on a unit (1.006 of two stages) and 7% slower with
  // more; Big takes 0.92 to 1.04 of Duo with one, and its eight chains per output
  // are what products off the Small tile must keep (least_plan_f32).
  // Their last parameter is the number of accumulators per output (AccChains):
  // with one, the 1500 -> 8800 layer at batch 700 (forward and backward) is
  // 8.4e-7 off the 64-bit result and takes 301 us, with these 4.2e-7 and 302 us;
  // an LSTM 1024 -> 1024, T 35, batch 64: 8.2e-7, 916 us and 4.7e-7, 916 us. Big
  // has as many chains per output as the 32 x 32 tile (8).
  using Huge = FastCfg<float, 128, 128, 32, 2, 2, 4, 1, 2>;  // 64 KB, 8 waves
  using Wide = Huge;
  using Tall = Huge;
  using Big = FastCfg<float, 64, 64, 64, 3, 2, 2, 2, 4>;     // 96 KB, 8 waves on 32-deep k shares
  using Duo = FastCfg<float, 64, 64, 64, 2, 2, 2, 2, 2>;     // 64 KB, as Big with half the accumulators
  using Mid = FastCfg<float, 64, 64, 32, 3, 2, 2, 1, 4>;     // 48 KB, 4 waves
  using Narrow = FastCfg<float, 128, 32, 32, 4, 2, 1, 2>; // 80 KB, 4 waves on 16-deep k shares
  using Small = FastCfg<float, 32, 32, 128, 4, 1, 1, 8>;  // 128 KB, 8 waves on 16-deep k shares
};

enum FastKind { FAST_HUGE, FAST_WIDE, FAST_TALL, FAST_BIG, FAST_SMALL, FAST_NARROW, FAST_MID, FAST_DUO };

struct FastPlan {
  int kind;    // FastKind
  int splits;  // workgroups per output tile along K (partials reduced by a second kernel)
  double us;   // modelled time (fp32)
};

// Split count s for a tile count: the largest power of two that keeps the grid
// within one round of the chip and every split at least kMinSlabsPerSplit slabs.
inline int fast_splits(int64_t tiles, int64_t slabs) {
  int s = 1;
  while (tiles * s * 2 <= kTargetBlocks && slabs / (s * 2) >= kMinSlabsPerSplit && s * 2 <= kMaxSplits) s *= 2;
  return s;
}

// The plan that sized workspaces before the cost model below: the largest tile
// whose grid covers 5/8 of the chip, splits on long contractions only, in at
// most cap floats. It gives the room that a call must be given (a call with
// more room may split further, one with this much is never refused), and the
// precision that a plan must keep: its tiles had no further accumulators.
inline FastPlan least_plan_f32(int M, int N, int K, int kbatch, int batch, int64_t cap) {
  using C = FastCfgs<float>;
  auto tiles_of = [&](int bm, int bn) {
    return static_cast<int64_t>((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch;
  };
  const int64_t kb = kbatch > 0 ? kbatch : 1;
  auto slabs_of = [&](int bk) { return kb * ((K + bk - 1) / bk); };
  constexpr int64_t kFill = kTargetBlocks * 5 / 8;
  FastPlan p = {};
  int64_t tiles;
  int bk;
  if (N <= C::Narrow::BN && tiles_of(C::Narrow::BM, C::Narrow::BN) >= kFill) {
    p.kind = FAST_NARROW, tiles = tiles_of(C::Narrow::BM, C::Narrow::BN), bk = C::Narrow::BK;
  } else if (M > 64 && N > 64 && tiles_of(128, 128) >= kFill) {
    p.kind = FAST_HUGE, tiles = tiles_of(128, 128), bk = C::Huge::BK;
  } else if (tiles_of(64, 64) >= kFill) {
    p.kind = FAST_BIG, tiles = tiles_of(64, 64), bk = C::Big::BK;
  } else {
    p.kind = FAST_SMALL, tiles = tiles_of(32, 32), bk = C::Small::BK;
  }
  const int64_t slabs = slabs_of(bk);
  p.splits = 1;
  if (p.kind == FAST_SMALL) {
    double best_t = 0.9 * static_cast<double>(slabs);
    for (int s = 2; s <= kMaxSplits && tiles * s <= kTargetBlocks && slabs >= s; s *= 2) {
      const double t = 0.9 * static_cast<double>((slabs + s - 1) / s) + 3.0;
      if (t < best_t) best_t = t, p.splits = s;
    }
  } else if (kb * K >= 8192) {
    p.splits = fast_splits(tiles, slabs);
  }
  while (p.splits > 1 && static_cast<int64_t>(p.splits) * M * N * batch > cap) p.splits /= 2;
  return p;
}

// MFMAs (of 2 k each) in the longest chain of additions behind one output: its
// rounding error grows with it. Measured over 120 products of 1 to 3 M outputs, a
// plan whose chains are no longer than another's is at most 5% (splits by 16)
// and on average less far from the 64-bit result.
inline int64_t chain_f32(int bk, int ksplit, int chains, int K, int64_t kb, int splits) {
  const int64_t slabs = kb * ((K + bk - 1) / bk), q = (slabs + splits - 1) / splits;
  const int64_t share = bk / ksplit;
  int64_t last = share;  // k of the first wave in the last slab
  if (kb == 1 && splits == 1 && K - (slabs - 1) * bk < share) last = K - (slabs - 1) * bk;
  return ((q - 1) * share + last + 2 * chains - 1) / (2 * chains);
}
template <class Cfg>
inline int64_t chain_f32(int chains, int K, int64_t kb, int splits) {
  return chain_f32(Cfg::BK, Cfg::KSPLIT, chains, K, kb, splits);
}
inline int64_t least_chain_f32(const FastPlan& p, int K, int64_t kb) {
  using C = FastCfgs<float>;
  return p.kind == FAST_HUGE     ? chain_f32<C::Huge>(1, K, kb, p.splits)
         : p.kind == FAST_NARROW ? chain_f32<C::Narrow>(1, K, kb, p.splits)
         : p.kind == FAST_BIG    ? chain_f32<C::Big>(1, K, kb, p.splits)
                                 : chain_f32<C::Small>(1, K, kb, p.splits);
}

// Modelled time of a fp32 product, in us, of one tile configuration: the fixed
// time of a launch, its first slabs and its stores; the matrix-core time of the
// n tiles on the fullest compute unit (614 GFLOP/s) times a factor for what their
// waits leave idle with one, two or more of them; a further start per round; the
// loaded and the stored bytes at 5 TB/s; for a split its reduction launch and
// partial sums.
struct CostF32 {
  int kind;
  double fixed, one, two, many, round, load, store, split, sums;
};

// Fitted to 22000 times of 2178 products on MI355X (forward, dX and dW of random
// layers, batch 16 to 2048, 64 to 8192 wide, and of larger ones up to 400
// GFLOP), within 2% of them in the mean square. The configuration and split that
// it picks is 0.1% slower than the best one in the mean over them and 17% at the
// most; the constants before, from eleven products, were 3.2% and 83%, and left
// one layer in ten slower than the fill rule that they had replaced (batch 32,
// 1952 -> 2604 forward 13.4 -> 19.2 us; batch 1652, 80 -> 3252 backward 35 -> 56).
// Mid has 0.4 us more than fitted: with operands out of the caches, as between a
// network's layers, its 32-deep slabs wait longer than Duo's (the 784-2048-2048-10
// network's step at batch 128 88.7 us without, 86.7 with; the pick 0.2% over the best).
constexpr CostF32 kCostF32[5] = {
    {FAST_HUGE, 6.98, 1.11, 1.06, 1.03, 1.84, 0.083, 1.06, 3.07, 1.45},
    {FAST_MID, 6.20, 1.46, 1.19, 1.13, 0.95, 0.056, 0.63, 2.45, 1.78},
    {FAST_BIG, 6.17, 1.26, 1.23, 1.20, 3.71, 0.052, 1.07, 1.96, 1.30},
    {FAST_DUO, 5.96, 1.29, 1.10, 1.09, 1.78, 0.051, 0.89, 1.88, 1.55},
    {FAST_SMALL, 4.85, 1.45, 1.42, 1.34, 2.80, 0.059, 1.19, 2.43, 2.07},
};

// The same with register loads (LOAD_ANY) by the operands' contiguous sides: A
// along k and B along n (forward), both across k (dX), both along k (dW). Fitted
// to 13000 times of 1152 products with rows off 16 bytes on MI355X, within 5%;
// the picks are 0.7% slower than the best ones in the mean and 20% at the most
// (one table for all three forms: 1.3% and 27%).
constexpr CostF32 kCostRegF32[3][5] = {
    {{FAST_HUGE, 6.78, 1.52, 1.52, 1.44, 1.88, 0.229, 1.49, 0.92, 1.70},
     {FAST_MID, 5.70, 2.73, 1.92, 1.68, 0.50, 0.169, 0.61, 1.21, 1.80},
     {FAST_BIG, 5.59, 1.89, 1.93, 1.95, 2.37, 0.268, 0.17, 2.02, 0.76},
     {FAST_DUO, 5.42, 1.90, 1.47, 1.55, 1.34, 0.205, 0.47, 2.03, 1.32},
     {FAST_SMALL, 4.22, 2.74, 1.97, 1.98, 0.92, 0.112, 0.54, 2.52, 2.66}},
    {{FAST_HUGE, 7.23, 1.60, 1.30, 1.27, 0.22, 0.163, 1.44, 0.41, 1.92},
     {FAST_MID, 5.00, 3.34, 2.13, 1.83, 1.04, 0.141, 0.40, 1.50, 1.65},
     {FAST_BIG, 5.08, 2.21, 2.11, 2.13, 2.23, 0.187, 0.51, 2.20, 0.82},
     {FAST_DUO, 5.14, 2.18, 1.68, 1.76, 0.89, 0.165, 0.48, 2.13, 1.25},
     {FAST_SMALL, 3.93, 3.15, 2.26, 2.30, 0.78, 0.054, 0.95, 2.67, 3.23}},
    {{FAST_HUGE, 7.11, 1.41, 1.45, 1.42, 1.33, 0.345, 1.46, 1.01, 1.60},
     {FAST_MID, 6.06, 2.32, 1.78, 1.68, 0.23, 0.100, 1.23, 1.09, 2.11},
     {FAST_BIG, 6.22, 1.61, 1.77, 1.83, 2.93, 0.277, 0.54, 1.74, 0.31},
     {FAST_DUO, 6.07, 1.67, 1.40, 1.62, 1.46, 0.125, 0.70, 1.74, 1.28},
     {FAST_SMALL, 4.80, 2.33, 1.79, 2.10, 1.08, 0.050, 1.06, 2.33, 1.56}},
};
constexpr int reg_form(bool amc, bool bmc) { return amc ? 1 : bmc ? 0 : 2; }

// What the planner needs to know of a configuration.
struct TileF32 {
  int bm, bn, bk, ksplit, chains;
};
inline TileF32 tile_f32(int kind) {
  auto of = [](auto cfg) {
    using C = decltype(cfg);
    return TileF32{C::BM, C::BN, C::BK, C::KSPLIT, C::CHAINS};
  };
  using C = FastCfgs<float>;
  return kind == FAST_HUGE  ? of(C::Huge{})
         : kind == FAST_MID ? of(C::Mid{})
         : kind == FAST_DUO ? of(C::Duo{})
         : kind == FAST_BIG ? of(C::Big{})
                            : of(C::Small{});
}

inline double time_f32(const CostF32& c, const TileF32& t, int M, int N, int K, int64_t kb, int batch, int splits) {
  const int64_t tiles = static_cast<int64_t>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * batch * splits;
  const int64_t q = (kb * ((K + t.bk - 1) / t.bk) + splits - 1) / splits;
  const double n = static_cast<double>((tiles + kTargetBlocks - 1) / kTargetBlocks);
  const double work = 2.0 * t.bm * t.bn * t.bk * q / 614e3, out = 4.0 * M * N * batch / 5e6;
  double us = c.fixed + n * work * (n > 2 ? c.many : n > 1 ? c.two : c.one) + c.round * (n - 1) +
              c.load * 4.0 * tiles * q * (t.bm + t.bn) * t.bk / 5e6 + c.store * out;
  if (splits > 1) us += c.split + c.sums * splits * out;
  return us;
}

// What a split weight gradient adds: the bias gradient, which an unsplit one
// takes from the rows that it reads, is then a launch of its own over the M x K
// operand (measured: 4 us and 1 us per 5 MB).
inline double rowsums_us(int M, int K) { return 4.0 + 4.0 * M * K / 5e6; }

// fp32: the (configuration, split) pair with the smallest modelled time whose
// partial sums fit cap floats. rowsums: see rowsums_us; costs: of the loads that
// will run. A plan with longer chains of additions than
// least_plan_f32's is not taken: without that line one product in fifty (all
// with K below 1100) was up to 1.4 times further off its 64-bit value.
inline FastPlan plan_fast_f32(int M, int N, int K, int kbatch, int batch, int64_t cap, bool rowsums = false,
                              const CostF32 (&costs)[5] = kCostF32) {
  using C = FastCfgs<float>;
  const int64_t kb = kbatch > 0 ? kbatch : 1;
  auto tiles_of = [&](int bm, int bn) {
    return static_cast<int64_t>((M + bm - 1) / bm) * ((N + bn - 1) / bn) * batch;
  };
  // at most 32 columns (an LSTM's per-step products at a small batch): 128 x
  // 32 tiles, so that most of each tile is not zero padding of the columns
  if (N <= C::Narrow::BN && tiles_of(C::Narrow::BM, C::Narrow::BN) >= kTargetBlocks * 5 / 8) {
    const int64_t tiles = tiles_of(C::Narrow::BM, C::Narrow::BN);
    int64_t s = kb * K >= 8192 ? fast_splits(tiles, kb * ((K + C::Narrow::BK - 1) / C::Narrow::BK)) : 1;
    while (s > 1 && s * M * N * batch > cap) s /= 2;
    return {FAST_NARROW, static_cast<int>(s), 0.0};
  }
  const int64_t longest = least_chain_f32(least_plan_f32(M, N, K, kbatch, batch, cap), K, kb);
  FastPlan best = {FAST_SMALL, 1, 1e300};
  for (const CostF32& c : costs) {
    const TileF32 t = tile_f32(c.kind);
    const int64_t tiles = tiles_of(t.bm, t.bn), slabs = kb * ((K + t.bk - 1) / t.bk);
    for (int s = 1; s <= kMaxSplits; s *= 2) {
      if (s > 1 && (slabs < s || tiles * s > 4 * kTargetBlocks ||
                    static_cast<int64_t>(s) * M * N * batch > cap))
        break;
      if (chain_f32(t.bk, t.ksplit, t.chains, K, kb, s) > longest) continue;
      double us = time_f32(c, t, M, N, K, kb, batch, s);
      if (s > 1 && rowsums) us += rowsums_us(M, K);
      if (us < best.us) best = {c.kind, s, us};
    }
  }
  return best;
}

// bf16: the (configuration, split) pair with the smallest modelled time. A
// workgroup's time is its MFMA work (whole tiles and slabs) over the rate one
// workgroup of that configuration reaches with the chip full (measured on
// MI355X), somewhat faster when fewer workgroups than compute units share the
// chip; workgroups beyond the first 256 run in further rounds; a split adds
// the partial-sum round trip and its reduction launch.
inline FastPlan plan_fast_bf16(int M, int N, int K, int kbatch, int batch) {
  using C = FastCfgs<bf16>;
  struct Cand {
    int kind, bm, bn, bk;
    double rate;  // flop/s per workgroup with 256 workgroups resident
  };
  static const Cand cands[] = {
      {FAST_HUGE, C::Huge::BM, C::Huge::BN, C::Huge::BK, 4.2e12},
      {FAST_WIDE, C::Wide::BM, C::Wide::BN, C::Wide::BK, 3.5e12},
      {FAST_TALL, C::Tall::BM, C::Tall::BN, C::Tall::BK, 3.4e12},
      {FAST_BIG, C::Big::BM, C::Big::BN, C::Big::BK, 2.7e12},
      {FAST_SMALL, C::Small::BM, C::Small::BN, C::Small::BK, 0.5e12},
  };
  const int64_t kb = kbatch > 0 ? kbatch : 1;
  FastPlan best = {FAST_SMALL, 1};
  double best_t = 1e300;
  for (const Cand& c : cands) {
    const int64_t tiles = static_cast<int64_t>((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * batch;
    const int64_t slabs = kb * ((K + c.bk - 1) / c.bk);
    for (int s = 1; s <= kMaxSplits; s *= 2) {
      if (s > 1 && (slabs / s < kMinSlabsPerSplit || tiles * s > 2 * kTargetBlocks)) break;
      const int64_t wgs = tiles * s;
      const int64_t rounds = (wgs + kTargetBlocks - 1) / kTargetBlocks;
      const double occ = wgs < kTargetBlocks ? static_cast<double>(wgs) / kTargetBlocks : 1.0;
      const double rate = c.rate * (1.0 + 0.3 * (1.0 - occ));
      const double work = 2.0 * c.bm * c.bn * c.bk * ((slabs + s - 1) / s);
      double t = rounds * work / rate;
      if (s > 1) t += 4.0 * M * N * batch * (s + 1) / 5e12 + 3e-6;
      if (t < best_t) {
        best_t = t;
        best = {c.kind, s};
      }
    }
  }
  return best;
}

// cap: floats of partial sums that the caller has room for (fp32; the bf16 plan
// is the one that sizes them).
template <typename T>
inline FastPlan plan_fast(int M, int N, int K, int kbatch, int batch, int64_t cap, bool rowsums = false) {
  if constexpr (sizeof(T) == 2)
    return plan_fast_bf16(M, N, K, kbatch, batch);
  else
    return plan_fast_f32(M, N, K, kbatch, batch, cap, rowsums);
}

constexpr int64_t kAnyRoom = int64_t{1} << 60;

// Floats of split-K partials of a product: what a call must be given room for
// (required), and what it makes use of if it has room floats.
template <typename T>
inline size_t fast_partial_floats(int M, int N, int K, bool required, bool rowsums, int64_t room) {
  int64_t s;
  if constexpr (sizeof(T) == 4) {
    if (required) {
      s = least_plan_f32(M, N, K, 1, 1, kAnyRoom).splits;
    } else {  // on whichever loads
      s = plan_fast_f32(M, N, K, 1, 1, room, rowsums).splits;
      for (const auto& costs : kCostRegF32) {
        const int r = plan_fast_f32(M, N, K, 1, 1, room, rowsums, costs).splits;
        if (r > s) s = r;
      }
    }
  } else
    s = plan_fast_bf16(M, N, K, 1, 1).splits;
  return s > 1 ? static_cast<size_t>(s) * M * N : 0;
}

template <class Cfg, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM = false, int LD = LOAD_DMA>
inline hipError_t launch_fast(const GemmArgs& g, int batch, hipStream_t stream) {
  const int splits = g.splits > 1 ? g.splits : 1;
  auto kern = fast_gemm_kernel<Cfg, AMC, BMC, OutT, EPI, RSUM, LD>;
  constexpr int LDS = LD == LOAD_ANY ? Cfg::LDS_REG : Cfg::LDS;
  // per instantiation, once (thread-safe static initialisation): allow more than 64 KB of dynamic LDS
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  if (attr != hipSuccess) return attr;
  dim3 grid((g.N + Cfg::BN - 1) / Cfg::BN, (g.M + Cfg::BM - 1) / Cfg::BM, batch * splits);
  hipLaunchKernelGGL(kern, grid, dim3(Cfg::NT), LDS, stream, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  const int64_t mn = static_cast<int64_t>(g.M) * g.N;
  if (reduce4_ok<OutT>(g)) {
    hipLaunchKernelGGL((splitk_reduce4_kernel<OutT, EPI>), dim3(static_cast<unsigned>((mn / 4 + 255) / 256), batch),
                       dim3(256), 0, stream, g);
  } else {
    hipLaunchKernelGGL((splitk_reduce_kernel<OutT, EPI>), dim3(static_cast<unsigned>((mn + 255) / 256), batch),
                       dim3(256), 0, stream, g);
  }
  return hipGetLastError();
}

// Launches g1 and g2 (both fast_ok, or both any_ok with LOAD_ANY; splits 1, no
// batch) as one grid of fast_gemm_pair_kernel on the 32x32 configuration of T.
template <typename T, bool AMC1, bool BMC1, typename OutT1, int EPI1, bool RSUM1, bool AMC2, bool BMC2,
          typename OutT2, int EPI2, bool RSUM2, int LD = LOAD_DMA>
inline hipError_t launch_fast_pair(GemmArgs g1, GemmArgs g2, hipStream_t stream) {
  using Cfg = typename FastCfgs<T>::Small;
  auto kern = fast_gemm_pair_kernel<Cfg, AMC1, BMC1, OutT1, EPI1, RSUM1, AMC2, BMC2, OutT2, EPI2, RSUM2, LD>;
  constexpr int LDS = LD == LOAD_ANY ? Cfg::LDS_REG : Cfg::LDS;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  if (attr != hipSuccess) return attr;
  g1.splits = g2.splits = 1;
  if (!RSUM1) g1.rsum = nullptr;
  if (!RSUM2) g2.rsum = nullptr;
  const int64_t n1 = static_cast<int64_t>((g1.N + Cfg::BN - 1) / Cfg::BN) * ((g1.M + Cfg::BM - 1) / Cfg::BM);
  const int64_t n2 = static_cast<int64_t>((g2.N + Cfg::BN - 1) / Cfg::BN) * ((g2.M + Cfg::BM - 1) / Cfg::BM);
  if (n1 + n2 == 0) return hipSuccess;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(n1 + n2)), dim3(Cfg::NT), LDS, stream, g1, g2);
  return hipGetLastError();
}

// Modelled time of fast_gemm_pair_kernel on fp32 operands, in us: its fixed
// time, the longest tile or the tiles shared out over the chip, further rounds,
// the loaded and the stored bytes (fitted to 152 layers on direct and 297 on
// register loads on MI355X, within 8%).
inline double pair_us_f32(const GemmArgs& g1, const GemmArgs& g2, bool reg) {
  using C = FastCfgs<float>::Small;
  auto tiles = [](const GemmArgs& g) {
    return static_cast<double>((g.M + C::BM - 1) / C::BM) * ((g.N + C::BN - 1) / C::BN);
  };
  auto slabs = [](const GemmArgs& g) { return static_cast<double>((g.K + C::BK - 1) / C::BK); };
  const double t1 = tiles(g1), t2 = tiles(g2), q1 = slabs(g1), q2 = slabs(g2);
  const double work = 2.0 * C::BM * C::BN * C::BK / 614e3, longest = q1 > q2 ? q1 : q2;
  const double share = (t1 * q1 + t2 * q2) / kTargetBlocks;
  const double rounds = static_cast<double>((static_cast<int64_t>(t1 + t2) + kTargetBlocks - 1) / kTargetBlocks);
  const double loads = 4.0 * (t1 * q1 + t2 * q2) * (C::BM + C::BN) * C::BK / 5e6;
  const double outs = 4.0 * (static_cast<double>(g1.M) * g1.N + static_cast<double>(g2.M) * g2.N) / 5e6;
  const double mma = (longest > share ? longest : share) * work;
  return reg ? 4.0 + 2.73 * mma + 0.70 * (rounds - 1) + 0.084 * loads + 0.64 * outs
             : 4.9 + 1.14 * mma + 2.42 * (rounds - 1) + 0.22 * loads;
}

// Whether bwd_data (g1) and bwd_weight (g2, with row sums) run as one
// fast_gemm_pair_kernel launch of 32x32 tiles without a k split. bf16: where both
// plans take those. fp32: also where those tiles are least_plan_f32's of both and
// one launch is modelled faster than the two planned ones. Without that line the
// cost model, which plans each product alone, sent one in fourteen of the layers
// that had run as one launch to two (batch 184, 364 -> 832: 10.5 -> 18.1 us; batch
// 704, 512 -> 688: 22.7 -> 32.2).
template <typename T>
inline bool pair_ok(const GemmArgs& g1, const FastPlan& p1, const GemmArgs& g2, const FastPlan& p2, int64_t cap,
                    bool reg) {
  if (g1.M <= 0 || g1.N <= 0 || g2.M <= 0 || g2.N <= 0) return false;
  if (p1.kind == FAST_SMALL && p2.kind == FAST_SMALL && p1.splits == 1 && p2.splits == 1) return true;
  if constexpr (sizeof(T) == 2) {
    return false;
  } else {
    auto small = [cap](const GemmArgs& g) {
      const FastPlan l = least_plan_f32(g.M, g.N, g.K, 1, 1, cap);
      return l.kind == FAST_SMALL && l.splits == 1;
    };
    return p1.us > 0.0 && p2.us > 0.0 && small(g1) && small(g2) && pair_us_f32(g1, g2, reg) < p1.us + p2.us;
  }
}
template <typename T>
inline bool fast_pair_ok(const GemmArgs& g1, const GemmArgs& g2, int64_t cap) {
  return pair_ok<T>(g1, plan_fast<T>(g1.M, g1.N, g1.K, 1, 1, cap), g2,
                    plan_fast<T>(g2.M, g2.N, g2.K, 1, 1, cap, true), cap, false);
}

template <typename T, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM, int LD = LOAD_DMA>
inline hipError_t launch_planned(const GemmArgs& g, int kind, int batch, hipStream_t stream) {
  using C = FastCfgs<T>;
  switch (kind) {
    case FAST_HUGE:
      // the bf16 256x256 tile has no registers left for row sums (it spills)
      if constexpr (RSUM && sizeof(T) == 2) return hipErrorNotSupported;
      else return launch_fast<typename C::Huge, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
    case FAST_WIDE:
      return launch_fast<typename C::Wide, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
    case FAST_TALL:
      return launch_fast<typename C::Tall, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
    case FAST_BIG:
      return launch_fast<typename C::Big, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
    case FAST_MID:  // fp32 only
      if constexpr (sizeof(T) == 4) return launch_fast<typename C::Mid, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
      else return hipErrorNotSupported;
    case FAST_DUO:  // fp32 only
      if constexpr (sizeof(T) == 4) return launch_fast<typename C::Duo, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
      else return hipErrorNotSupported;
    case FAST_NARROW:  // fp32 only
      if constexpr (sizeof(T) == 4) return launch_fast<typename C::Narrow, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
      else return hipErrorNotSupported;
    default:
      return launch_fast<typename C::Small, AMC, BMC, OutT, EPI, RSUM, LD>(g, batch, stream);
  }
}

// Runs a GEMM on the fast kernel; the caller has checked fast_ok(). With
// RSUM, g.rsum receives the row sums of A when the plan has no k split and is
// not the bf16 256x256 tile, and *rsum_done says whether it did (else the
// caller computes them itself). smallest: 32x32 tiles without a split (one half
// of a pair run on its own).
template <typename T, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM = false>
inline hipError_t run_fast_gemm(GemmArgs g, int batch, hipStream_t stream, float* partial, int64_t cap,
                                bool* rsum_done = nullptr, bool smallest = false) {
  if (rsum_done) *rsum_done = false;
  if (g.M <= 0 || g.N <= 0 || batch <= 0) return hipSuccess;
  FastPlan p = {FAST_SMALL, 1, 0.0};
  if (!smallest) p = plan_fast<T>(g.M, g.N, g.K, g.kbatch, batch, partial ? cap : 0, RSUM);
  // the kernel splits the slabs with 32-bit arithmetic
  const int64_t kb = g.kbatch > 0 ? g.kbatch : 1;
  if (!partial || kb * (g.K / 32 + 1) * p.splits >= int64_t{1} << 31) p.splits = 1;
  g.splits = p.splits;
  g.partial = partial;
  if (RSUM && g.rsum && p.splits == 1 && !(sizeof(T) == 2 && p.kind == FAST_HUGE)) {
    if (rsum_done) *rsum_done = true;
    return launch_planned<T, AMC, BMC, OutT, EPI, RSUM>(g, p.kind, batch, stream);
  }
  g.rsum = nullptr;
  return launch_planned<T, AMC, BMC, OutT, EPI, false>(g, p.kind, batch, stream);
}

// Plan of the register-load variant. fp32: the cost model with this variant's
// times. bf16 has two tile sizes here: its 256-wide tiles leave no registers for
// two slabs in flight; its split count never exceeds what the workspace of the
// problem was sized for (the direct-load or the general kernel's plan).
template <typename T>
inline FastPlan plan_any(int form, int M, int N, int K, int kbatch, int batch, int64_t cap, bool rowsums = false) {
  if constexpr (sizeof(T) == 4) {
    return plan_fast_f32(M, N, K, kbatch, batch, cap, rowsums, kCostRegF32[form]);
  } else {
    using C = FastCfgs<bf16>;
    FastPlan p = plan_fast_bf16(M, N, K, kbatch, batch);
    const int gs = plan_gemm<T>(M, N, K, kbatch, batch).splits;
    const int most = p.splits > gs ? p.splits : gs;
    const int64_t kb = kbatch > 0 ? kbatch : 1;
    auto tiles_of = [&](int b) { return static_cast<int64_t>((M + b - 1) / b) * ((N + b - 1) / b) * batch; };
    p.kind = tiles_of(C::Big::BM) >= kTargetBlocks / 2 ? FAST_BIG : FAST_SMALL;
    const int b = p.kind == FAST_BIG ? C::Big::BM : C::Small::BM, bk = p.kind == FAST_BIG ? C::Big::BK : C::Small::BK;
    p.splits = fast_splits(tiles_of(b), kb * ((K + bk - 1) / bk));
    if (p.splits > most) p.splits = most;
    return p;
  }
}

// Whether a product on rows off 16 bytes is too short for the register loads,
// whose pipeline and 128- or 64-deep slabs a contraction of at most 64 does not
// fill: the general kernel (ard_gemm.hpp) then takes less time. Measured on
// MI355X, general over register loads: fp32, up to 64 / 65 to 128 tiles of 64 x
// 64, K up to 48: 0.98 / 0.90 (911 x 260 x 34: 5.7 / 7.1 us), up to 64: 1.05 /
// 0.90, up to 96: 1.25 / 1.15, more tiles: 1.1 to 2; bf16 on 128 x 128 tiles whose
// output rows hold no whole 4-element pieces, K below 64: 0.79 (2169 x 2797 x 17:
// 23 / 36 us), with whole pieces, which only the register-load kernel stores at
// once, 1.5 (4612 x 596 x 64: 22.7 / 12.4), K up to 128: 1.3, on 32 x 32 tiles: 1.2.
// Not for products with row sums, which the general kernel does not take.
template <typename T>
inline bool short_contraction(int M, int N, int K) {
  auto tiles_of = [&](int b) { return static_cast<int64_t>((M + b - 1) / b) * ((N + b - 1) / b); };
  if constexpr (sizeof(T) == 4)
    return K <= (tiles_of(64) > kTargetBlocks / 4 ? 64 : 48) && tiles_of(64) <= kTargetBlocks * 5 / 8;
  else
    return K < 64 && N % 4 != 0 && tiles_of(FastCfgs<bf16>::Big::BM) >= kTargetBlocks / 2;
}
// Whether run_strided_gemm takes the product.
template <typename T, bool AMC, bool BMC>
inline bool strided_ok(const GemmArgs& g, bool rowsums = false) {
  return fast_ok<AMC, BMC>(g, sizeof(T)) ||
         (any_ok<AMC, BMC>(g, sizeof(T)) && (rowsums || !short_contraction<T>(g.M, g.N, g.K)));
}

// Runs a GEMM whose operands are plain strided views (strided_ok): on the direct
// loads where the rows start on 16 bytes (fast_ok), else on register loads.
template <typename T, bool AMC, bool BMC, typename OutT, int EPI, bool RSUM = false>
inline hipError_t run_strided_gemm(GemmArgs g, int batch, hipStream_t stream, float* partial, int64_t cap,
                                   bool* rsum_done = nullptr, bool smallest = false) {
  if (fast_ok<AMC, BMC>(g, sizeof(T)))
    return run_fast_gemm<T, AMC, BMC, OutT, EPI, RSUM>(g, batch, stream, partial, cap, rsum_done, smallest);
  if (rsum_done) *rsum_done = false;
  if (g.M <= 0 || g.N <= 0 || batch <= 0) return hipSuccess;
  FastPlan p = {FAST_SMALL, 1, 0.0};
  if (!smallest) p = plan_any<T>(reg_form(AMC, BMC), g.M, g.N, g.K, g.kbatch, batch, partial ? cap : 0, RSUM);
  const int64_t kb = g.kbatch > 0 ? g.kbatch : 1;
  if (!partial || kb * (g.K / 32 + 1) * p.splits >= int64_t{1} << 31) p.splits = 1;
  g.splits = p.splits;
  g.partial = partial;
  using C = FastCfgs<T>;
  const bool rs = RSUM && g.rsum && p.splits == 1;
  if (!rs) g.rsum = nullptr;
  if (rsum_done) *rsum_done = rs;
  auto go = [&](auto cfg) {
    using Cfg = decltype(cfg);
    if constexpr (RSUM) {
      if (rs) return launch_fast<Cfg, AMC, BMC, OutT, EPI, true, LOAD_ANY>(g, batch, stream);
    }
    return launch_fast<Cfg, AMC, BMC, OutT, EPI, false, LOAD_ANY>(g, batch, stream);
  };
  if (p.kind == FAST_SMALL) return go(typename C::Small{});
  if constexpr (sizeof(T) == 4) {
    if (p.kind == FAST_HUGE) return go(typename C::Huge{});
    if (p.kind == FAST_NARROW) return go(typename C::Narrow{});
    if (p.kind == FAST_MID) return go(typename C::Mid{});
    if (p.kind == FAST_DUO) return go(typename C::Duo{});
  }
  return go(typename C::Big{});
}

// Whether the pair runs as one launch of the register-load 32x32 tiles.
template <typename T>
inline bool any_pair_ok(const GemmArgs& g1, const GemmArgs& g2, int64_t cap) {
  return pair_ok<T>(g1, plan_any<T>(reg_form(true, true), g1.M, g1.N, g1.K, 1, 1, cap), g2,
                    plan_any<T>(reg_form(false, false), g2.M, g2.N, g2.K, 1, 1, cap, true), cap, true);
}

// A fp32 product over the columns of several steps at once (EPI_COLS): B's and
// C's columns in blocks. cols_ok: fast_ok, blocks of whole chunks, and a slab's
// span below 2^31 bytes with the blocks' strides.
template <bool AMC>
inline bool cols_ok(const GemmArgs& g) {
  if (!fast_ok<AMC, true>(g, 4) || g.nblk <= 0 || g.nblk % 4 || g.b_nstride % 4) return false;
  return ((static_cast<int64_t>(g.N) / g.nblk + 1) * g.b_nstride + 256 * g.b.ld) * 4 < (int64_t{1} << 31);
}
template <bool AMC>
inline hipError_t run_cols_gemm(GemmArgs g, hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const FastPlan p = plan_fast_f32(g.M, g.N, g.K, 1, 1, 0);
  g.splits = 1;
  g.partial = nullptr;
  g.rsum = nullptr;
  return launch_planned<float, AMC, true, float, EPI_COLS, false>(g, p.kind, 1, stream);
}

// A fp32 product with both operands k-contiguous over a flat contraction
// (LOAD_FLAT); see FlatLoader. rsum is always taken when set.
inline bool flat_ok(const GemmArgs& g) {
  const int64_t kb = g.kbatch > 0 ? g.kbatch : 1, k = kb * g.K;
  auto span = [&](const GemmOperand& o, int ext) {
    return (static_cast<int64_t>(ext - 1) * o.ld + (kb - 1) * o.kbstride + g.K) * 4 < (int64_t{1} << 31);
  };
  return fast_ok<false, false>(g, 4) && g.K % 4 == 0 && k * g.K < (int64_t{1} << 32) && k < (int64_t{1} << 30) &&
         g.M > 0 && g.N > 0 && span(g.a, g.M) && span(g.b, g.N);
}
template <bool RSUM>
inline hipError_t run_flat_gemm(GemmArgs g, int batch, hipStream_t stream) {
  const FastPlan p = plan_fast_f32(g.M, g.N, (g.kbatch > 0 ? g.kbatch : 1) * g.K, 1, batch, 0);
  g.splits = 1;
  g.partial = nullptr;
  if (!RSUM) g.rsum = nullptr;
  return launch_planned<float, false, false, float, EPI_FWD, RSUM, LOAD_FLAT>(g, p.kind, batch, stream);
}

}  // namespace ard
