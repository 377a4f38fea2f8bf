// fp16 MFMA GEMM for the projection and feed-forward matrices of a decoder layer
// (paper Sec. 2.1: self-attention module + feed-forward network; these four
// products are the bulk of a chunk step's arithmetic).
//
//   out[t, f] = sum_k X[t, k] * W[f, k]      X: activations, W: weights [out, in]
//
// Both operands are in the P32 layout (hat_layout.h).  The kernel computes the
// transposed product C^T = W * X^T with v_mfma_f32_16x16x32_f16: MFMA rows are
// output features, MFMA columns are tokens.  In the accumulator a lane then owns
// one token and runs of 4 consecutive features, which is exactly an 8-byte piece
// of the P32 layout of the *next* operand, so every epilogue stores coalesced.
//
// Data movement: global -> LDS with direct-to-LDS loads (global_load_lds_dwordx4),
// no register staging, into a ring of k-tiles.  In the tiles of the largest batches the
// multiplying waves load too, the refill spread thinly between the MFMAs, as a load holds
// the issuing wave while it waits for its turn; the tile shape (bytes moved per flop)
// decides the rest.  Because the P32 panel slab of a k-tile is contiguous in memory and is kept contiguous in
// LDS, each wave instruction moves one 1 KB run, and an MFMA operand is one
// ds_read_b128 at lane*16 + immediate, conflict-free without a swizzle.
// Loader waves.  The tiles of batches up to a few hundred rows (G > 0) have waves that load and do nothing else, with scalar addresses, so that they
// neither hold an MFMA wave while a load issues nor wait behind the matrix pipe for an address (a 64-bit vector address next to 32x32x16 MFMAs: one 1 KB load in 141
// clocks a wave instead of 70).  That alone gains nothing (gate/up of 256 rows, 7B shape, 61 us both): what bounds these products is that a CU's loads return in order and
// that about 32 KB of them can be on their way (a CU by itself streams weights at 54 B/ns with any number of loads issued: 32 KB in 0.6 us), so that X, which comes from
// L2, waits behind W, which comes from HBM.  Loads alone of the 96 x 256 tile, W and X of each k-tile in turn: 46 us; W of two k-tiles, then X of the two:
// 36.  So W is loaded G k-tiles at a time, into a ring of its own that is twice that long, and X in a shorter one; W that one token tile alone reads
// is loaded non-temporally (W alone 31.7 -> 27.5 us).  Gate/up of 256 rows 61.2 -> 51.5 us, of 77 44.1 -> 39, QKV 43 -> 38, O 20.3 -> 19.1, down 36.9 -> 34.8.
// The MFMA waves and the loader waves share the registers of a SIMD three ways (168 each).  The accumulators of tiles of 192 and 256 features with 160 and more token rows, and of 192 x 128
// with the halves of K on different waves, do not leave that many.  192 x 128 on 2 x 4 waves and 256 x 128 would (117 and 137 registers, 144 and 160 KB of LDS); they have not been measured.
// LDS reads are issued from inline asm so that the compiler does not serialise
// them behind the outstanding direct-to-LDS loads; the waits are explicit:
// vmcnt for "my loads of this k-tile have landed", a barrier for "everyone's
// have", lgkmcnt for the operand reads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "hat_device_util.h"
#include "hat_kernels.h"
#include "hat_layout.h"

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef kv_t kvx4 __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }
// fp32 -> fp16, round to nearest even, saturating instead of overflowing to infinity
__device__ __forceinline__ _Float16 to_act(float x) { return (_Float16)__builtin_amdgcn_fmed3f(x, -65504.f, 65504.f); }

template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { hat_static_for<N>(f); }
template <int OFF>
__device__ __forceinline__ f16x8 lds_read(uint32_t addr) { return hat_lds_read<OFF>(addr); }
template <int N>
__device__ __forceinline__ void wait_vmcnt() { hat_wait_vmcnt<N>(); }
template <int N>
__device__ __forceinline__ void wait_operands(f16x8 (&v)[N]) { hat_wait_operands(v); }

// The QKV result on its way out.  A thread has rows i0 .. i0+3 (lo; i0 < 16) and i0+16 .. i0+19 (hi) of a panel of W, which are features
// f .. f+3 and f+hd/2 .. of a head (hat_launch_retile).  q and k are rotated in fp32 and rounded once; k and v go to the
// token's cache slot.
struct QkvPart {   // where a panel's features belong (uniform)
  int which, head, f0;   // 0 q, 1 k, 2 v; its first feature, below hd/2
};
__device__ __forceinline__ QkvPart qkv_part(const HatQkvOut& o, int panel) {
  const int ppd = o.hd >> 5, head3 = panel / ppd;   // panels per head
  const int which = head3 / o.H;
  return {which, head3 - which * o.H, (panel - head3 * ppd) * 16};
}
struct QkvAngles { f32x4 c01, c23; };   // (cos, sin) of four pairs
__device__ __forceinline__ QkvAngles qkv_angles(const HatQkvOut& o, int tok, int f) {
  const float2* t = o.table + (size_t)tok * (o.hd >> 1) + f;
  return {*(const f32x4*)t, *(const f32x4*)(t + 2)};
}
// q, k and v saturate at the fp16 range before anything else happens to them
__device__ __forceinline__ f32x4 saturate(f32x4 x) {
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_fmed3f(x[e], -65504.f, 65504.f);
  return x;
}
__device__ __forceinline__ void rotate(const QkvAngles& ang, f32x4& lo, f32x4& hi) {
  const float c[4] = {ang.c01[0], ang.c01[2], ang.c23[0], ang.c23[2]}, s[4] = {ang.c01[1], ang.c01[3], ang.c23[1], ang.c23[3]};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a = lo[e], b = hi[e];
    // (which product is rounded first is written out: left to the compiler it is another one with each form of the code around it)
    lo[e] = __builtin_fmaf(a, c[e], -(b * s[e]));
    hi[e] = __builtin_fmaf(b, c[e], a * s[e]);
  }
}
__device__ __forceinline__ f16x4 to_act4(f32x4 x) { return __builtin_convertvector(saturate(x), f16x4); }
__device__ __forceinline__ kvx4 to_kv4(f32x4 x, int kv_f16) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  if (kv_f16) return __builtin_bit_cast(kvx4, to_act4(x));
  return __builtin_bit_cast(kvx4, __builtin_convertvector(x, bf16x4));
}
// Where the four features from `i0` of a panel on go for one token, apart from what is the same for all tokens: offsets of q in its
// P32 row (from the workgroup's first row on: 32 bits do not hold an offset in a step of more than 2^31 / Nout rows), of k in its tile, of v in its tile
// (relative to the head's pages).  A thread computes them once for all panels.
struct QkvToken {
  int q;
  size_t k, v;
};
__device__ __forceinline__ QkvToken qkv_token(const HatGemm& g, int row0, int tok, int dst, int i0) {
  const size_t page = (size_t)(dst >> 4) * kv_head_elems(g.qkv.hd);
  const int slot = dst & 15;
  return {(int)p32_index(tok - row0, i0, g.Nout), page + ktile_index(slot, i0), page + 16 * g.qkv.hd + vtile_index(slot, i0)};
}
// lo: rows i0 .. i0+3 of the panel, hi: rows i0+16 .. (their partners).  row0: the workgroup's first token, a multiple of 32
__device__ __forceinline__ void store_qkv(const HatGemm& g, int row0, const QkvPart& part, const QkvToken& t, const QkvAngles& ang, f32x4 lo, f32x4 hi) {
  const HatQkvOut& o = g.qkv;
  const int half = o.hd >> 1;
  lo = saturate(lo);
  hi = saturate(hi);
  if (part.which < 2) rotate(ang, lo, hi);
  if (part.which == 0) {
    act_t* q = g.outP + p32_index(row0, part.head * o.hd + part.f0, g.Nout) + t.q;
    *(f16x4*)q = to_act4(lo);
    *(f16x4*)(q + (half >> 3) * 256) = to_act4(hi);
    return;
  }
  const kvx4 a = to_kv4(lo, o.kv_f16), b = to_kv4(hi, o.kv_f16);
  kv_t* head = o.pool + (size_t)part.head * o.n_pages * kv_head_elems(o.hd);
  if (part.which == 1) {
    kv_t* k = head + ktile_index(0, part.f0) + t.k;
    *(kvx4*)k = a;
    *(kvx4*)(k + ktile_index(0, half)) = b;
  } else {   // a V tile is feature-major: two-byte stores
    kv_t* v = head + vtile_index(0, part.f0) + t.v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[8 * e] = a[e];
      v[vtile_index(0, half) + 8 * e] = b[e];
    }
  }
}

template <int BF, int BT, int WF, int WT, int WK, int BKT, int NSTAGE, int G>
struct Tile {
  static constexpr int NW = WF * WT * WK;           // waves that multiply
  static constexpr int NL = G > 0 ? BKT / 16 : 0;   // loader waves: each brings one of the 1 KB chunks of every slab
  static constexpr int MI = BF / WF / 16;   // 16-row feature blocks per wave
  static constexpr int NJ = BT / WT / 16;   // 16-row token blocks per wave
  static constexpr int PF = BF / 32, PT = BT / 32;
  static constexpr int SLAB = (BKT / 8) * 512;  // bytes of one panel's k-slab
  static constexpr int CPS = SLAB / 1024;       // 1 KB wave-chunks per slab
  static constexpr int NCH = (PF + PT) * CPS;
  static constexpr int LPW = (NCH + NW - 1) / NW;  // direct-to-LDS loads per wave per stage (the last waves: one less, where they don't divide)
  static constexpr int STAGE = (PF + PT) * SLAB;
  static constexpr int KS = BKT / 32 / WK;      // k-steps of one wave per stage
  static constexpr int WR = 2 * G;              // G > 0: k-tiles in the ring of W
  static constexpr int LDS_BYTES = G > 0 ? (WR * PF + NSTAGE * PT) * SLAB : NSTAGE * STAGE;
  static_assert(BF % (WF * 32) == 0 && BT % (WT * 16) == 0 && (WT == 1 || WT % 2 == 0), "whole 32-row panels of features, 16-row blocks of tokens");
  static_assert(KS >= 1 && BKT % (32 * WK) == 0 && (WK == 1 || WK == 2), "whole k-steps");
  static_assert(G > 0 || (NSTAGE >= 2 && NSTAGE <= 4 && (NSTAGE - 1) * LPW <= 63), "wait_pending covers up to 3 pending tiles; vmcnt is 6 bits");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS per workgroup");
  // registers of a lane: accumulators, two sets of operands, and what addresses and counters take
  static constexpr int REGS = MI * NJ * 4 + 2 * (MI + NJ) * 4 + 32;
  static_assert(REGS <= 512 / ((NW + NL + 3) / 4), "the waves of a SIMD share its registers");
  static_assert(G == 0 || (NSTAGE >= 2 && NSTAGE <= G + 1 && (NSTAGE - 2) * PT + G * PF <= 63), "a tile of X is never before its tile of W");
  static_assert(WK == 1 || WF * WT * MI * NJ * 1024 <= LDS_BYTES, "the two halves of K meet in the ring");
};

// Matrix instruction: v_mfma_f32_16x16x32_f16.  Random operands drive the matrix pipes into the chip's power limit, and this
// shape takes less power than 32x32x16: a loop of nothing but MFMAs runs at 1920 .. 1980 TFLOP/s against 1640 .. 1715 (2420 both on
// zeros), gate/up of 4096 rows (13B shape) at 1290 against 1155.  It needs two waves on a SIMD: with one, its 16 clocks do not hide
// the issue of the next operand reads and loads (256 x 192 on four waves: 359 -> 437 us), so every large tile has eight
// waves.  Where eight wave tiles would read too much LDS per product (192 x 128: 48 rows each), WK = 2 gives the two waves of a
// SIMD the same output block and each half of a stage's k; they meet in LDS at the end.
// Against the 32x32x16 loop on four waves, in steps (weights from HBM), QKV, gate/up and down: 13B shape at 512 rows 79 -> 73 us, 129 -> 115, 76 -> 72, at 4096 533 ->
// 474, 948 -> 837, 504 -> 440; at 256 rows of the 7B shape, where the weight stream decides, level (39.0 -> 40.1, 61.2 -> 60.7, 36.4 -> 36.2).
template <int BF, int BT, int WF, int WT, int WK, int BKT, int NSTAGE, int G, int EPI>
__global__ __launch_bounds__((Tile<BF, BT, WF, WT, WK, BKT, NSTAGE, G>::NW + Tile<BF, BT, WF, WT, WK, BKT, NSTAGE, G>::NL) * 64) void gemm_kernel(HatGemm g, int ksplit, int full) {
  using TL = Tile<BF, BT, WF, WT, WK, BKT, NSTAGE, G>;
  constexpr int MI = TL::MI, NJ = TL::NJ, PF = TL::PF, PT = TL::PT, SLAB = TL::SLAB, CPS = TL::CPS;
  constexpr int LPW = TL::LPW, STAGE = TL::STAGE, KS = TL::KS;

  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave / (WF * WT), wq = wave % (WF * WT);
  const int wf = wq / WT, wt = wq % WT;

  // workgroup -> tile.  Consecutive hardware ids go round-robin over the 8 XCDs;
  // give each XCD a contiguous run of tiles so that tiles sharing a weight panel
  // meet in one L2.
  const int nF = (g.Nw + BF - 1) / BF;
  int nT = (g.T + BT - 1) / BT;
  int b = blockIdx.x, kz = blockIdx.z, tt0 = 0;
  if (EPI == HAT_EPI_RESID && full > 0) {   // whole tiles first, then the split ones (one-dimensional grid)
    if (b < full * nF) {
      nT = full;
      ksplit = 1;
    } else {
      b -= full * nF;
      tt0 = full;
      nT -= full;
      kz = b / (nT * nF);
      b -= kz * nT * nF;
    }
  }
  const int nblk = nT * nF;
  {
    const int per = nblk / 8, rem = nblk % 8;
    const int x = b % 8, i = b / 8;
    b = x * per + (x < rem ? x : rem) + i;
  }
  // within an XCD's run, walk groups of 4 feature tiles across the token tiles: the ~32
  // workgroups resident on an XCD then form a 4 x 8 patch of tiles (12 distinct operand
  // slabs per k-tile instead of 16+) and more of their loads hit in L2
  int ft, tt;
  {
    constexpr int GF = 4;
    const int grp = b / (GF * nT);
    const int f0 = grp * GF;
    const int gf = (nF - f0) < GF ? (nF - f0) : GF;
    const int r = b - grp * GF * nT;
    ft = f0 + r % gf;
    tt = tt0 + r / gf;
  }
  const int Tpanels = (g.T + 31) >> 5;

  const int KT = g.K / BKT;
  const int kt0 = (int)((long)kz * KT / ksplit);
  const int kt1 = (int)((long)(kz + 1) * KT / ksplit);
  const int nkt = G > 0 ? __builtin_amdgcn_readfirstlane(kt1 - kt0) : kt1 - kt0;

  if constexpr (G > 0) {
    constexpr int WR = TL::WR;
    if (wave >= TL::NW) {   // a loader wave: the same barriers as the others
      const int lw = wave - TL::NW, lane16 = lane * 16;
      const size_t krow = (size_t)(g.K >> 3) * 256;
      const size_t k0 = (size_t)kt0 * (BKT / 8) * 256 + lw * 512;
      const int fp = __builtin_amdgcn_readfirstlane(ft) * PF, tp = __builtin_amdgcn_readfirstlane(tt) * PT;
      const void* wbase = hat_uniform(g.W + (size_t)fp * krow + k0);
      const void* xbase = hat_uniform(g.X + (size_t)tp * krow + k0);
      int w[PF], x[PT];   // bytes from there to each panel (beyond the last: that one again)
#pragma unroll
      for (int q = 0; q < PF; ++q) w[q] = min(q, (g.Nw >> 5) - 1 - fp) * (int)krow * 2;
#pragma unroll
      for (int q = 0; q < PT; ++q) x[q] = min(q, Tpanels - 1 - tp) * (int)krow * 2;
      auto run = [&](auto auxc) {
        int ws = 0, xs = 0;   // ring slots of the next tiles
        auto load_w = [&](int t) {
#pragma unroll
          for (int q = 0; q < PF; ++q) hat_load_lds<decltype(auxc)::value>(wbase, lds + (ws * PF + q) * SLAB + lw * 1024, lane16, w[q] + t * SLAB);
          ws = ws + 1 == WR ? 0 : ws + 1;
        };
        auto load_x = [&](int t) {
#pragma unroll
          for (int q = 0; q < PT; ++q) hat_load_lds<0>(xbase, lds + (WR * PF + xs * PT + q) * SLAB + lw * 1024, lane16, x[q] + t * SLAB);
          xs = xs + 1 == NSTAGE ? 0 : xs + 1;
        };
        for (int t = 0; t < G && t < nkt; ++t) load_w(t);
        for (int t = 0; t < NSTAGE - 1 && t < nkt; ++t) load_x(t);
        int i = 0;
        for (; i + 2 * G <= nkt; i += G)   // every tile that is to be loaded exists
          static_for<G>([&](auto pc) {
            constexpr int p = decltype(pc)::value;
            // behind X of tile i + p: X of the NSTAGE - 2 tiles after it, and a group of W if one was issued among them
            constexpr int groups = p >= 1 && p <= NSTAGE - 2 ? 1 : 0;
            wait_vmcnt<(NSTAGE - 2) * PT + groups * G * PF>();
            __builtin_amdgcn_s_barrier();
            if constexpr (p == 0)
              for (int t = 0; t < G; ++t) load_w(i + G + t);
            load_x(i + p + NSTAGE - 1);
          });
        for (const int i0 = i; i < nkt; ++i) {   // the last tiles: only X is counted
          const int behind = min(NSTAGE - 2, nkt - 1 - i);
          static_for<NSTAGE - 1>([&](auto b) {
            if (behind == b) wait_vmcnt<decltype(b)::value * PT>();
          });
          __builtin_amdgcn_s_barrier();
          if (i == i0)
            for (int t = i + G; t < nkt; ++t) load_w(t);
          if (i + NSTAGE - 1 < nkt) load_x(i + NSTAGE - 1);
        }
      };
      if (nT == 1) run(std::integral_constant<int, 2>{});
      else run(std::integral_constant<int, 0>{});
      wait_vmcnt<0>();
      if constexpr (WK == 2) {
        __syncthreads();
        __syncthreads();
      }
      return;
    }
  }

  // per-wave chunk sources (per-lane address); destinations are wave-uniform
  constexpr int EXTRA = TL::NCH % TL::NW;            // that many waves bring LPW chunks, the others one less (0: all bring LPW)
  const bool more = EXTRA == 0 || wave < EXTRA;
  const int ch0 = more ? wave * LPW : EXTRA * LPW + (wave - EXTRA) * (LPW - 1);
  const act_t* src[LPW];
  const size_t krow = (size_t)(g.K >> 3) * 256;  // elements per panel
#pragma unroll
  for (int c = 0; c < LPW; ++c) {
    const int ch = c + 1 < LPW || more ? ch0 + c : ch0;
    const int q = ch / CPS, sub = ch % CPS;
    const act_t* base;
    if (q < PF) {
      int pnl = ft * PF + q;
      pnl = pnl < (g.Nw >> 5) ? pnl : (g.Nw >> 5) - 1;  // ragged last feature tile: same
      base = g.W + (size_t)pnl * krow;
    } else {
      int pnl = tt * PT + (q - PF);
      pnl = pnl < Tpanels ? pnl : Tpanels - 1;  // ragged last tile: re-read a real panel
      base = g.X + (size_t)pnl * krow;
    }
    src[c] = base + (size_t)kt0 * (BKT / 8) * 256 + sub * 512 + lane * 8;
  }
  auto issue_chunk = [&](int i, int c) {  // chunk c of k-tile i (relative to kt0)
    if (EXTRA != 0 && c + 1 == LPW && !more) return;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(src[c] + (size_t)i * (BKT / 8) * 256),
        (__attribute__((address_space(3))) void*)(lds + (i % NSTAGE) * STAGE + (ch0 + c) * 1024), 16, 0, 0);
  };
  auto wait_tiles = [&](auto tc) {  // at most tc k-tiles of my loads still in flight
    constexpr int t = decltype(tc)::value < NSTAGE ? decltype(tc)::value : NSTAGE - 1;
    if (more) wait_vmcnt<t * LPW>();
    else wait_vmcnt<t * (LPW - 1)>();
  };
  auto wait_pending = [&](int tiles) {
    switch (tiles) {
      case 0: wait_tiles(std::integral_constant<int, 0>{}); break;
      case 1: wait_tiles(std::integral_constant<int, 1>{}); break;
      case 2: wait_tiles(std::integral_constant<int, 2>{}); break;
      default: wait_tiles(std::integral_constant<int, 3>{}); break;
    }
  };

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  if constexpr (G == 0) {
#pragma unroll
    for (int s = 0; s < NSTAGE; ++s)
      if (s < nkt) {
#pragma unroll
        for (int c = 0; c < LPW; ++c) issue_chunk(s, c);
      }
  }

  // An operand is 16 rows x 32 k: lane l holds row l%16, k-octet l/16.  A wave's feature blocks are consecutive; its token
  // blocks are every WT-th of the tile, so that any number of them keeps the same distance in LDS for every wave.
  const uint32_t lane_off = lds_base + (lane >> 4) * 512 + (lane & 15) * 16 + wk * (KS * 2048);
  const uint32_t offW = lane_off + (wf * MI / 2) * SLAB;
  const uint32_t offX = lane_off + (G > 0 ? TL::WR * PF : PF) * SLAB + (wt >> 1) * SLAB + (wt & 1) * 256;
  f16x8 a[2][MI], bb[2][NJ];
  constexpr int NMFMA = MI * NJ;
  int wo = 0, xo = 0;   // (G > 0) the current tile's places in the rings
  auto read_operands = [&](auto setc, auto ksc, int i) {
    constexpr int set = decltype(setc)::value, ks = decltype(ksc)::value;
    uint32_t aW, aX;
    if constexpr (G > 0) {
      aW = offW + wo;
      aX = offX + xo;
    } else {
      aW = offW + (i % NSTAGE) * STAGE;
      aX = offX + (i % NSTAGE) * STAGE;
    }
    static_for<MI>([&](auto ii) { a[set][ii] = lds_read<(ii / 2) * SLAB + (ii % 2) * 256 + ks * 2048>(aW); });
    static_for<NJ>([&](auto jj) {
      constexpr int off = WT == 1 ? (jj / 2) * SLAB + (jj % 2) * 256 : jj * (WT / 2) * SLAB;
      bb[set][jj] = lds_read<off + ks * 2048>(aX);
    });
  };
  // One continuous pipeline over k-steps of 32.  The operands of the next k-step are read from LDS
  // while the MFMAs of this one run, also across k-tile boundaries: at the last k-step of
  // tile i a wave first makes sure tile i+1 has landed (its own loads: vmcnt; everyone's:
  // barrier -- which also says everyone is done reading tile i), reads tile i+1's first
  // operands, and only then issues tile i's last MFMAs.  The direct-to-LDS loads of tile
  // i+NSTAGE (into the buffer tile i just vacated) are slotted between the MFMAs of the
  // following KS k-steps, in KS parts: part 0 right after that boundary, parts 1.. over the next tile's k-steps 0..KS-2.
  // They are spread thinly because a direct-to-LDS load holds the issuing wave for on the order of a hundred cycles.
  // `steady`: tile i + NSTAGE exists, so nothing has to be asked (one k-step per tile only: see the loops below).
  auto kstep = [&](auto curc, auto ksc, int i, auto steadyc) {
    constexpr int cur = decltype(curc)::value, ks = decltype(ksc)::value;
    constexpr bool steady = decltype(steadyc)::value;
    constexpr std::integral_constant<int, cur ^ 1> next{};
    wait_operands(a[cur]);
    wait_operands(bb[cur]);
    if constexpr (ks + 1 < KS) {
      read_operands(next, std::integral_constant<int, ks + 1>{}, i);
    } else if (steady || i + 1 < nkt) {
      if constexpr (G == 0) {
        const int after = nkt - 2 - i;  // tiles issued behind tile i+1
        if (steady || after >= NSTAGE - 2) wait_tiles(std::integral_constant<int, NSTAGE - 2>{});
        else wait_pending(after);
      } else {
        wo = wo + PF * SLAB == TL::WR * PF * SLAB ? 0 : wo + PF * SLAB;
        xo = xo + PT * SLAB == NSTAGE * PT * SLAB ? 0 : xo + PT * SLAB;
      }
      __builtin_amdgcn_s_barrier();
      read_operands(next, std::integral_constant<int, 0>{}, i + 1);
    }
    constexpr int part = (ks + 1) % KS, CPP = (LPW + KS - 1) / KS;
    const int rtile = (ks + 1 == KS) ? i + NSTAGE : i - 1 + NSTAGE;
    const bool refill = rtile < nkt && ((ks + 1 == KS) ? (i + 1 < nkt) : (i >= 1));
    // keep the operand reads ahead of this k-step's MFMAs (the scheduler would otherwise
    // sink them behind the MFMAs and expose the LDS latency)
    __builtin_amdgcn_sched_barrier(0);
    static_for<NMFMA>([&](auto n) {
      // back and forth along the token blocks: each MFMA shares an operand with the one before it
      constexpr int ii = n / NJ, jj = (ii & 1) ? NJ - 1 - n % NJ : n % NJ;
      acc[ii][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[cur][ii], bb[cur][jj], acc[ii][jj], 0, 0, 0);
      static_for<CPP>([&](auto q) {
        constexpr int slot = q * NMFMA / CPP + NMFMA / CPP / 2;
        constexpr int c = part * CPP + q;
        if constexpr (G == 0 && slot == n && c < LPW) {
          if (steady || refill) issue_chunk(rtile, c);
        }
      });
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  auto ktile = [&](auto curc, int i, auto steadyc) {
    static_for<KS>([&](auto ks) { kstep(std::integral_constant<int, (decltype(curc)::value + ks) & 1>{}, ks, i, steadyc); });
  };
  constexpr std::integral_constant<int, 0> set0{};
  constexpr std::integral_constant<int, KS & 1> set1{};   // the register set on which an odd tile starts
  if (nkt > 0) {
    if constexpr (G == 0) wait_pending(nkt - 1 < NSTAGE - 1 ? nkt - 1 : NSTAGE - 1);
    __builtin_amdgcn_s_barrier();
    read_operands(set0, std::integral_constant<int, 0>{}, 0);
  }
  int i = 0;
  if constexpr (KS == 1) {
    for (; i + 1 + NSTAGE < nkt; i += 2) {
      ktile(set0, i, std::true_type{});
      ktile(set1, i + 1, std::true_type{});
    }
  }
  for (; i < nkt; i += 2) {
    ktile(set0, i, std::false_type{});
    if (i + 1 < nkt) ktile(set1, i + 1, std::false_type{});
  }

  // the two halves of K: a wave hands its partner one half of the token blocks and finishes the other
  constexpr int NJO = WK == 1 ? NJ : (NJ + 1) / 2;
  int j0 = 0, jn = NJ;
  if constexpr (WK == 2) {
    __syncthreads();   // everyone is done with the ring
    f32x4* red = (f32x4*)lds + wq * (MI * NJ * 64) + lane;
#pragma unroll
    for (int ii = 0; ii < MI; ++ii)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if ((j < NJO) == (wk == 1)) red[(ii * NJ + j) * 64] = acc[ii][j];
    __syncthreads();
    j0 = wk * NJO;
    jn = wk == 0 ? NJO : NJ - NJO;
#pragma unroll
    for (int ii = 0; ii < MI; ++ii)
#pragma unroll
      for (int j = 0; j < NJO; ++j) {
        if (wk == 1 && j + NJO < NJ) acc[ii][j] = acc[ii][j + NJO < NJ ? j + NJO : j];
        if (j < jn) acc[ii][j] += red[(ii * NJ + j0 + j) * 64];
      }
  }

  // ---- epilogue.  lane: token = 16 * (token block) + lane%16 ; feature = f0 + 16i + 4*(lane/16) + r
  const int h4 = (lane >> 4) * 4, n = lane & 15;
  const int f_base = ft * BF + wf * MI * 16;
  auto token = [&](int j) { return tt * BT + (wt + WT * (j0 + j)) * 16 + n; };
  if constexpr (EPI == HAT_EPI_RESID) {
    // fp32 result: added into the residual when K is not split, else stored as this
    // split's partial sum (the next consumer of the residual folds the partials in)
    const int row0 = tt0 * BT;   // first row of the partial sums
    if (f_base >= g.Nout) return;
    if (ksplit > 1) {
      float* base = g.part + (size_t)((long)kz * (g.T - row0) - row0) * g.Nout + f_base + h4;
#pragma unroll
      for (int j = 0; j < NJO; ++j) {
        if (token(j) >= g.T || j >= jn) continue;
        float* p = base + (size_t)token(j) * g.Nout;
#pragma unroll
        for (int i = 0; i < MI; ++i)
          if (f_base + i * 16 < g.Nout) *(f32x4*)(p + i * 16) = acc[i][j];
      }
      return;
    }
    // A thread's pieces of the residual (those beyond its end: a piece that is there) are read together, or in two halves where they do not fit the
    // registers, before the first is written back.  One at a time, each read waits out a memory round trip and the store before it, as the two may
    // alias: O and down of 2788 rows (7B shape) 98.4 -> 94.3 and 218.1 -> 212.5 us, of 4096 rows (13B shape) 195.9 -> 190.2 and 449.1 -> 444.6.  What is left of the
    // update is its traffic, 92 MB that all workgroups of a single round move at the same time.
    constexpr int H = MI * NJO <= 24 ? NJO : (NJO + 1) / 2;   // token blocks read together
#pragma unroll
    for (int jh = 0; jh < NJO; jh += H) {
      f32x4 r[MI][H];
#pragma unroll
      for (int j = jh; j < jh + H && j < NJO; ++j) {
        const float* p = g.resid + (size_t)min(token(j), g.T - 1) * g.Nout + f_base + h4;
#pragma unroll
        for (int i = 0; i < MI; ++i) r[i][j - jh] = *(const f32x4*)(p + (f_base + i * 16 < g.Nout ? i * 16 : 0));
      }
      // (one wait for all of them: left to the compiler there is one for each token block, under its branch, and each waits for the stores before it too)
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
#pragma unroll
      for (int j = jh; j < jh + H && j < NJO; ++j) {
        if (token(j) >= g.T || j >= jn) continue;
        float* p = g.resid + (size_t)token(j) * g.Nout + f_base + h4;
#pragma unroll
        for (int i = 0; i < MI; ++i)
          if (f_base + i * 16 < g.Nout) *(f32x4*)(p + i * 16) = r[i][j - jh] + acc[i][j];
      }
    }
    return;
  }
  if constexpr (EPI == HAT_EPI_QKV) {
    // All loads of a panel before its first store: behind a store that may alias, each would wait out a memory round trip of its own.
    int row0 = tt * BT;
    asm volatile("" : "+s"(row0));   // (or the offsets of q, the same in every workgroup, are computed before the loop and take registers through it)
    QkvToken t[NJO];
#pragma unroll
    for (int j = 0; j < NJO; ++j) t[j] = qkv_token(g, row0, token(j), g.qkv.kv_dst[min(token(j), g.T - 1)], h4);
#pragma unroll
    for (int i = 0; i < MI; i += 2) {
      const int fb = f_base + i * 16;
      if (fb >= g.Nout) continue;
      const QkvPart part = qkv_part(g.qkv, fb >> 5);
      QkvAngles ang[NJO];
      if (part.which < 2) {
#pragma unroll
        for (int j = 0; j < NJO; ++j) ang[j] = qkv_angles(g.qkv, min(token(j), g.T - 1), part.f0 + h4);
      }
#pragma unroll
      for (int j = 0; j < NJO; ++j)
        if (token(j) < g.T && j < jn) store_qkv(g, row0, part, t[j], ang[j], acc[i][j], acc[i + 1][j]);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < NJO; ++j) {
    const int tok = token(j);
    if (tok >= g.T || j >= jn) continue;
    if constexpr (EPI == HAT_EPI_P32) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int fb = f_base + i * 16;
        if (fb >= g.Nout) continue;
        // the feature of W's row fb (hat_launch_retile)
        const int ppd = g.qkv.hd >> 5, panel = fb >> 5, head3 = panel / ppd;
        const int f = head3 * g.qkv.hd + (panel - head3 * ppd) * 16 + (i & 1) * (g.qkv.hd >> 1);
        f16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = to_act(acc[i][j][e]);
        *(f16x4*)(g.outP + p32_index(tok, f + h4, g.Nout)) = v;
      }
    } else if constexpr (EPI == HAT_EPI_SWIGLU) {
      // a 32-row block of W holds 16 gate rows then the 16 up rows of the same features
#pragma unroll
      for (int i = 0; i < MI; i += 2) {
        const int fb = (f_base + i * 16) / 2;  // output feature block (16 wide)
        if (fb >= g.Nout) continue;
        f16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = to_act(silu_f(acc[i][j][e]) * acc[i + 1][j][e]);
        *(f16x4*)(g.outP + p32_index(tok, fb + h4, g.Nout)) = v;
      }
    }
  }
}

template <int NP, int NT>
struct StreamDepth {   // k-steps in flight per wave: what the register file holds next to the accumulators
  static constexpr int value = NP + NT <= 4 ? 8 : NP == 1 ? 6 : 4;
};
// ---- few token rows: weights streamed into operand registers -------------------------------
// At most a few dozen rows make the product a read of W and nothing else, so this kernel is built
// for the HBM stream and not for the matrix pipe.  A workgroup owns 32 NP features x 32 NT tokens and
// its 8 waves split K: each wave loads its own 1 KB operand pieces of W (non-temporal: one reader, or two where 65 .. 96
// rows make two token tiles)
// and of X straight into MFMA operand registers, kept D k-steps ahead by a register ring, with no LDS and no
// barrier until the 8 partial tiles meet in LDS at the end.  32-feature tiles give QKV and gate/up of the 7B shape 384 and
// 688 workgroups (two of them resident on a CU) where the LDS tiles above have 96 and 172, and the split of K
// inside the workgroup needs no partial sums in memory.  Lanes of token columns beyond T repeat
// the last row's address, so that a 5-row batch fetches 5 rows of X and not 32.
// Bound by the HBM stream: QKV of the 7B shape (100 MB) at 5 rows 31.0 -> 22.0 us (3.2 -> 4.6 TB/s, launch and
// drain included), gate/up (180 MB) 36.9 -> 33.5 us (5.4 TB/s); QKV at 96 rows 35.8 -> 31.5 us.
template <int NP, int NT, int EPI>
__global__ __launch_bounds__(512, NP* NT <= 1 ? 4 : 2) void gemm_stream_kernel(HatGemm g, int ksplit) {
  constexpr int NW = 8;
  constexpr int D = StreamDepth<NP, NT>::value;
  constexpr int TILES = NP * NT;
  constexpr int GRP = TILES < 2 ? TILES : 2;   // 32 x 32 tiles summed per LDS round
  static_assert(TILES % GRP == 0, "a round is whole");
  __shared__ __attribute__((aligned(16))) f32x4 red[NW][GRP][4][64];
  // accumulators and ring, with 40 registers for addresses; two workgroups of the smallest tile on a CU, one of the others
  static_assert(TILES * 16 + D * (NP + NT) * 4 + 40 <= (TILES <= 1 ? 128 : 256), "a lane's registers");
  static_assert(sizeof(red) * (TILES <= 1 ? 2 : 1) <= 160 * 1024, "the LDS of a CU");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int nF = (EPI == HAT_EPI_QKV ? g.Nout : g.Nw) / (32 * NP);
  const int ft = blockIdx.x % nF, tt = blockIdx.x / nF;
  // A QKV workgroup's two panels are hd/64 apart, with its neighbour's between them: side by side they measured 24.0 -> 25.0 us at
  // 32 rows of the 7B shape (fp16 cache), 30.0 -> 30.4 at 77.
  const int pstep = EPI == HAT_EPI_QKV && NP == 2 ? g.qkv.hd >> 6 : 1;
  const int panel0 = ft / pstep * (NP * pstep) + ft % pstep;
  const int KS = g.K >> 4;                     // k-steps of 16
  const int part = blockIdx.z * NW + wave, parts = ksplit * NW;
  const int s0 = (int)((long)part * KS / parts), s1 = (int)((long)(part + 1) * KS / parts);
  const int cnt = s1 - s0;

  const size_t krow = (size_t)(g.K >> 3) * 256;
  const act_t* wsrc[NP];
  const act_t* xsrc[NT];
#pragma unroll
  for (int i = 0; i < NP; ++i) wsrc[i] = g.W + (size_t)(panel0 + i * pstep) * krow + (size_t)s0 * 512 + h * 256 + n * 8;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    int row = (tt * NT + j) * 32 + n;
    row = row < g.T ? row : g.T - 1;
    xsrc[j] = g.X + (size_t)(row >> 5) * krow + (size_t)s0 * 512 + h * 256 + (row & 31) * 8;
  }
  f32x16 acc[NP][NT];
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  f16x8 a[D][NP], b[D][NT];
  auto load = [&](auto dc, int s) {
    constexpr int d = decltype(dc)::value;
#pragma unroll
    for (int i = 0; i < NP; ++i) a[d][i] = __builtin_nontemporal_load((const f16x8*)(wsrc[i] + (size_t)s * 512));
#pragma unroll
    for (int j = 0; j < NT; ++j) b[d][j] = *(const f16x8*)(xsrc[j] + (size_t)s * 512);
  };
  auto mma = [&](auto dc) {
    constexpr int d = decltype(dc)::value;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[d][i], b[d][j], acc[i][j], 0, 0, 0);
  };
  // the main loop's loads are unconditional (a load under a branch would make every wait behind it a
  // wait for all loads); the last D .. 2D-1 k-steps, or a K share shorter than D, take the guarded tail
  int s = 0;
  if (cnt >= D) {
    static_for<D>([&](auto d) { load(d, d); });
    for (; s + 2 * D <= cnt; s += D)
      static_for<D>([&](auto d) {
        mma(d);
        load(d, s + D + d);
        __builtin_amdgcn_sched_barrier(0);
      });
  } else {
    static_for<D>([&](auto d) {
      if (d < cnt) load(d, d);
    });
  }
  const int rem = cnt - s;   // below 2D; the first min(rem, D) of them are in registers
  static_for<D>([&](auto d) {
    if (d < rem) mma(d);
    if (D + d < rem) load(d, s + D + d);
  });
  static_for<D>([&](auto d) {
    if (D + d < rem) mma(d);
  });

  // ---- sum of the 8 waves' tiles and epilogue: thread = 4 consecutive features of one token
#pragma unroll
  for (int t0 = 0; t0 < TILES; t0 += GRP) {
    if (t0 > 0) __syncthreads();
#pragma unroll
    for (int u = 0; u < GRP; ++u) {
      const f32x16& v = acc[(t0 + u) % NP][(t0 + u) / NP];
#pragma unroll
      for (int q = 0; q < 4; ++q) red[wave][u][q][lane] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    }
    __syncthreads();
    auto total = [&](int u, int q) {
      f32x4 v = red[0][u][q][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += red[w][u][q][lane];
      return v;
    };
    if constexpr (EPI == HAT_EPI_QKV) {
      const int u = wave >> 1, q = wave & 1;   // rows 8 q .. of tile u of the round, and their partners 16 rows further
      const int tok = (tt * NT + (t0 + u) / NP) * 32 + n;
      if (u < GRP && tok < g.T) {
        const QkvPart part = qkv_part(g.qkv, panel0 + (t0 + u) % NP * pstep);
        const int i0 = 8 * q + 4 * h;
        const QkvToken t = qkv_token(g, tt * NT * 32, tok, g.qkv.kv_dst[tok], i0);
        const QkvAngles ang = part.which < 2 ? qkv_angles(g.qkv, tok, part.f0 + i0) : QkvAngles{};
        store_qkv(g, tt * NT * 32, part, t, ang, total(u, q), total(u, q + 2));
      }
    } else {
      const int u = threadIdx.x >> 8, q = (threadIdx.x >> 6) & 3;
      const int tok = (tt * NT + (t0 + u) / NP) * 32 + n;
      const int fb = (ft * NP + (t0 + u) % NP) * (EPI == HAT_EPI_SWIGLU ? 16 : 32);
      if (u < GRP && (EPI != HAT_EPI_SWIGLU || q < 2) && tok < g.T && fb < g.Nout) {
        const int f = fb + 8 * q + 4 * h;
        const f32x4 v = total(u, q);
        if constexpr (EPI == HAT_EPI_RESID) {
          float* p = (ksplit == 1 ? g.resid : g.part + (size_t)blockIdx.z * g.T * g.Nout) + (size_t)tok * g.Nout + f;
          *(f32x4*)p = ksplit == 1 ? *(const f32x4*)p + v : v;
        } else {
          const f32x4 up = total(u, q + 2);
          f16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = to_act(silu_f(v[e]) * up[e]);
          *(f16x4*)(g.outP + p32_index(tok, f, g.Nout)) = o;
        }
      }
    }
  }
}

// tile table: id, features x tokens, waves along features x tokens, halves of K, k per stage, stages (of X, where W has a ring of its own), k-tiles of W
// that are loaded together (0: no loader waves).  G and the stages of X are what 160 KB of LDS hold; k-tiles of 32 there measured 4 .. 6 us behind (barriers).
// Heights of 64, 96 and 192 rows exist so that the tile count can match the 256 CUs where
// 128 / 256 leave a quarter or a third of them idle (7B-shaped QKV and gate/up at T <= 256).
// Without one of them the products of a layer lose, on average over seven widths and 22 batch sizes of 33 .. 3556 rows (at the most): 64 x 64 0.6 % (6.6), 64 x 128 0.5 (4.9), 96 x 256
// 0.5 (6.0), 128 x 128 0.4 (6.2), 128 x 256 0.4 (7.4), 96 x 128 0.4 (4.3), 256 x 128 0.3 (6.3), 96 x 64 and 128 x 160 0.1 (4.0), 64 x 256 0.1 (2.0), 256 x 64 0.06 (4.6).
// Tiles 20-22 take 224, 192 and 160 token rows: for batches whose row count leaves the last 256-row tile mostly empty
// or the tile count just above a multiple of the 256 CUs.  Tile 23
// (128 x 160) is for batches of 129 .. 160 rows, e.g. 30 devices x 5 draft rows: one token tile
// instead of a full and a nearly empty one.
// Waves: 64 x 128 and the like each, 12 operand reads for 32 MFMAs, where that makes eight wave tiles of whole 32-row panels; two
// halves of K otherwise (192 x 128 on gate/up of the 7B shape with the weights in the caches, 256 rows: 96 x 64 in halves of K 48.2 us, 96 x 32
// 53.7; from HBM the two are within 4 % of each other either way), unless the weight stream decides (weights from HBM, 128 x 160 at 150 rows: O 15.1 us against 16.4 in halves of K, down 25.7 against 27.0; 128 x 64 at 56 rows: 12.8
// against 13.2 and 22.2 against 22.5).
// Stages of 32 k let a wave hold both register sets and still have four stages; fewer, longer ones measured level (128-row
// tiles) or behind (256 x 256 at 4096 rows: 900 us with 4 x 32, 967 with 2 x 64, 919 with 5 x 32).
// Neither regime offers tiles 0, 1, 6, 8 and 16.  1 is the product whose rotation and append are a launch of their own, which the others are compared with; the others are taken by
// their number only (hat_mid_debug_force_gemm).
#define HAT_FOR_TILES(X, EPI)          \
  X(0, 256, 256, 2, 4, 1, 32, 4, 0, EPI)  \
  X(1, 192, 128, 2, 4, 1, 32, 4, 0, EPI)  \
  X(2, 128, 256, 2, 4, 1, 64, 3, 2, EPI)  \
  X(3, 256, 128, 4, 2, 1, 64, 3, 0, EPI)  \
  X(4, 128, 128, 2, 4, 1, 64, 4, 3, EPI)  \
  X(5, 256, 64, 4, 1, 2, 64, 3, 2, EPI)   \
  X(6, 256, 32, 4, 1, 2, 64, 3, 2, EPI)   \
  X(7, 128, 64, 2, 4, 1, 64, 4, 4, EPI)   \
  X(8, 128, 32, 2, 1, 2, 64, 4, 4, EPI)   \
  X(9, 64, 256, 1, 8, 1, 64, 3, 3, EPI)   \
  X(10, 128, 64, 2, 4, 1, 64, 4, 0, EPI)  \
  X(11, 64, 64, 1, 2, 2, 64, 4, 6, EPI) \
  X(12, 64, 128, 1, 4, 2, 64, 4, 6, EPI)  \
  X(13, 192, 128, 2, 2, 2, 64, 3, 0, EPI) \
  X(14, 96, 128, 1, 8, 1, 64, 4, 4, EPI)  \
  X(15, 96, 256, 1, 8, 1, 64, 3, 2, EPI)  \
  X(16, 192, 64, 2, 2, 2, 64, 3, 2, EPI)  \
  X(17, 192, 256, 2, 4, 1, 32, 4, 0, EPI) \
  X(18, 96, 64, 1, 2, 2, 64, 4, 4, EPI)   \
  X(19, 256, 256, 4, 2, 1, 32, 4, 0, EPI) \
  X(20, 256, 224, 4, 2, 1, 32, 4, 0, EPI) \
  X(21, 256, 192, 4, 2, 1, 32, 4, 0, EPI) \
  X(22, 256, 160, 4, 2, 1, 32, 4, 0, EPI) \
  X(23, 128, 160, 4, 2, 1, 64, 3, 3, EPI)
constexpr int kNumLdsTiles = 24;
// The QKV product without rotation and append is built for one tile, as the form that the others are compared with.
constexpr bool lds_built(int id, int epi) { return epi != HAT_EPI_P32 || id == HAT_APART_TILE; }
// the streaming kernel's tiles (32 NP features x 32 NT tokens): id, NP, NT.  Four waves instead of eight, 32 x 64 and
// 32 x 96 measured level with or behind these at every size; 64 x 32 is for the QKV product of 17 .. 32 rows (see hat_gemm_plan).
#define HAT_FOR_STREAM(X, EPI) \
  X(24, 1, 1, EPI)             \
  X(25, 2, 2, EPI)             \
  X(26, 2, 3, EPI)             \
  X(27, 2, 1, EPI)
// Which of them exist for an epilogue: those that stream_plan gives it.
constexpr bool stream_built(int id, int epi) {
  return epi == HAT_EPI_QKV ? id >= 24 && id <= 27 : epi == HAT_EPI_SWIGLU ? id >= 24 && id <= 26 : epi == HAT_EPI_RESID ? id == 24 || id == 26 : false;
}
constexpr int kStream32 = 24, kStream64 = 25, kStream96 = 26, kStream64x32 = 27;
constexpr int kNumTiles = 28;

struct TileInfo { int bf, bt, waves, bkt, nstage; float eff; int loaders, lds; };   // (waves that multiply, waves that load)
// How fast a tile's k-loop is taken to be where it is not load-bound, against the matrix peak, and with it the constants of the large regime below: weights for the
// choice, found by random search for the least loss against the best tile and K split and not fitted to the times (0: not offered).  All loops were the multiplying waves' own
// then, with 128 x 64 in the form that is tile 10 now.  Measured with those tiles, K splits and
// split tails of the four products, norms included, at 36 batch sizes of 390 .. 4096 rows and seven widths (1024 x 2816 .. 8192 x 28672; the search had seen 9 sizes up to 2048
// rows of three of them): the four choices of a layer lost 0.24 % of it on average at 20 of the sizes and 0.31 % at the other 16.  Searched again on the 20 sizes of all widths, with a cost of its own for
// the rotating epilogue, the constants came to 0.20 .. 0.23 % there and 0.32 .. 0.38 % at the other 16: what is left is the model's form (it counts whole
// rounds of workgroups, where large products go by their padded work).
// Of the tiles with loader waves four are offered here.  Over 20 sizes of 1101 .. 4096 rows and eight widths they take, of the time of those earlier loops, 128 x 256 0.90 .. 0.99, 128 x 128 0.89 .. 1.02,
// 96 x 128 0.90 .. 1.00 and 128 x 160 0.89 .. 1.04 (the higher ones at 256 and 1024 columns), so their weights are on the low side: the present choices lose 0.4 .. 1.4 % of a
// layer at 1024 .. 5120 and 8192 columns and 2.6 % at 6144.  128 x 64 with loader waves (7) takes 0.98 .. 1.09 times as long
// as without (10), 1.03 .. 1.07 for O and down of 256 and 1024 columns, which take this tile (all these with events around each launch); whole steps of 256 .. 1792 columns take 1 .. 3 % less with 10
// (1101 rows of 256 columns 39.2 -> 37.8 us a layer, 2000 of 1024 103.0 -> 102.0).
constexpr float kEff[kNumLdsTiles] = {0.f, 0.f, 0.537f, 0.533f, 0.744f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.679f, 0.f, 0.f, 0.527f, 0.570f, 0.f, 0.f, 0.535f, 0.f, 0.645f, 0.584f, 0.542f, 0.534f, 0.531f};
constexpr int kSmallT = 384;
// Up to kMidT rows: us that a k-tile of 64 is taken to cost each tile (0: not offered), and what else the model counts (hat_gemm_plan).
// Weights for the choice like kEff, searched on all tiles, one to eight pieces of K and the norms at 30 batch sizes of 33 .. 1100 rows and seven widths (1024 x 2816 .. 8192 x 28672): the choices
// lose 0.24 % of a layer's products on average; searched on two thirds of the sizes 0.23 .. 0.30 % there and 0.30 .. 0.45 % on the others.  The constants before, with these
// tiles, lost 2 .. 9 % (192 rows 8.1, 420 8.8, 256 6.3, 1024 3.0).
// 128 x 64 without loader waves (10) starts and ends sooner than its loader form (7), which takes less for a k-tile whose panel of W nobody else reads: a round of its own, searched at eleven widths from
// 256 x 704 to 7168 x 18944.  It is offered from 257 rows on, where its panels of W are read by five and more token tiles, which then find them in L2.  Whole steps, us a layer, without it | with it: 512 rows of 256 columns 36.6 | 34.5,
// of 512 columns 46.6 | 43.4, 441 rows of 1024 55.6 | 54.9, 320 of 1280 58.5 | 57.9; at 236 sizes of 257 .. 1100 rows and thirteen widths up to 7 % less, nowhere more than 0.5 % more.
// Below it loses as often as it gains (33 .. 128 rows 0.6 .. 2.4 % of a layer at 1024 and 2560 .. 4608 columns).  Times of single launches with events around them show it ahead there: such launches favour the tiles without loader waves by
// about 1 us, so choices are compared in whole steps that are not profiled.
constexpr int kMidT = 1100;
constexpr float kTau[kNumLdsTiles] = {0.f, 0.f, 0.725f, 0.866f, 0.474f, 0.844f, 0.f, 0.405f, 0.f, 0.491f, 0.360f, 0.238f, 0.328f, 0.684f, 0.403f, 0.606f, 0.f, 1.046f, 0.338f, 1.306f, 1.204f, 1.045f, 0.951f, 0.590f};
struct MidCosts { double round, round_plain, fraction, shared, part, tbs, stream, resid; };
constexpr MidCosts kMid = {7.79, 7.1, 0.192, 0.0730, 0.460, 6.01, 13.79, 0.506};
constexpr TileInfo kTiles[kNumTiles] = {
#define HAT_INFO(id, bf, bt, wf, wt, wk, bkt, ns, g_, epi) {bf, bt, (wf) * (wt) * (wk), bkt, ns, kEff[id], Tile<bf, bt, wf, wt, wk, bkt, ns, g_>::NL, Tile<bf, bt, wf, wt, wk, bkt, ns, g_>::LDS_BYTES},
    HAT_FOR_TILES(HAT_INFO, 0)
#undef HAT_INFO
// "stages" of a streaming tile: its register ring counted in 32-k pieces
#define HAT_INFO(id, np, nt, epi) {32 * (np), 32 * (nt), 8, 32, StreamDepth<np, nt>::value / 2, 0.f, 0, 8 * ((np) * (nt) < 2 ? 1 : 2) * 4096},
    HAT_FOR_STREAM(HAT_INFO, 0)
#undef HAT_INFO
};

template <int EPI>
hipError_t launch_epi(const HatGemm& g, const HatGemmPlan& p, hipStream_t st) {
#define HAT_TRY(id, bf, bt, wf, wt, wk, bkt, ns, g_, epi)                   \
  if constexpr (lds_built(id, epi)) if (p.tile == id) {                 \
    using TL = Tile<bf, bt, wf, wt, wk, bkt, ns, g_>;                       \
    const int nT = (g.T + bt - 1) / bt, nF = (g.Nw + bf - 1) / bf;      \
    dim3 grid(nT * nF, 1, p.ksplit);                                    \
    if (p.full > 0) grid = dim3(p.full * nF + (nT - p.full) * nF * p.ksplit); \
    auto kern = gemm_kernel<bf, bt, wf, wt, wk, bkt, ns, g_, epi>;          \
    kern<<<grid, dim3((TL::NW + TL::NL) * 64), TL::LDS_BYTES, st>>>(g, p.ksplit, p.full); \
    return hipGetLastError();                                           \
  }
  HAT_FOR_TILES(HAT_TRY, EPI)
#undef HAT_TRY
#define HAT_TRY(id, np, nt, epi)                                                     \
  if constexpr (stream_built(id, epi)) {                                             \
    if (p.tile == id) {                                                              \
      const int nF = (epi == HAT_EPI_QKV ? g.Nout : g.Nw) / (32 * (np));             \
      dim3 grid(((g.T + 32 * (nt) - 1) / (32 * (nt))) * nF, 1, p.ksplit);            \
      gemm_stream_kernel<np, nt, epi><<<grid, dim3(512), 0, st>>>(g, p.ksplit);      \
      return hipGetLastError();                                                      \
    }                                                                                \
  }
  HAT_FOR_STREAM(HAT_TRY, EPI)
#undef HAT_TRY
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t attr_epi() {
  hipError_t e;
#define HAT_ATTR(id, bf, bt, wf, wt, wk, bkt, ns, g_, epi)                                                    \
  if constexpr (lds_built(id, epi)) {                                                                     \
    e = hipFuncSetAttribute((const void*)gemm_kernel<bf, bt, wf, wt, wk, bkt, ns, g_, epi>,                   \
                            hipFuncAttributeMaxDynamicSharedMemorySize, Tile<bf, bt, wf, wt, wk, bkt, ns, g_>::LDS_BYTES); \
    if (e != hipSuccess) return e;                                                                        \
  }
  HAT_FOR_TILES(HAT_ATTR, EPI)
#undef HAT_ATTR
  return hipSuccess;
}

}  // namespace

int hat_gemm_tile_count() { return kNumTiles; }
bool hat_gemm_tile_info(int id, int* bf, int* bt, int* waves, int* bkt, int* nstage) {
  if (id < 0 || id >= kNumTiles) return false;
  const TileInfo& q = kTiles[id];
  if (bf) *bf = q.bf;
  if (bt) *bt = q.bt;
  if (waves) *waves = q.waves;
  if (bkt) *bkt = q.bkt;
  if (nstage) *nstage = q.nstage;
  return true;
}

bool hat_gemm_tile_resources(int id, int* loaders, int* lds) {
  if (id < 0 || id >= kNumTiles) return false;
  if (loaders) *loaders = kTiles[id].loaders;
  if (lds) *lds = kTiles[id].lds;
  return true;
}

hipError_t hat_gemm_init() {
  hipError_t e;
  if ((e = attr_epi<HAT_EPI_P32>()) != hipSuccess) return e;
  if ((e = attr_epi<HAT_EPI_SWIGLU>()) != hipSuccess) return e;
  if ((e = attr_epi<HAT_EPI_RESID>()) != hipSuccess) return e;
  if ((e = attr_epi<HAT_EPI_QKV>()) != hipSuccess) return e;
  return hat_attn_init();
}

// Where the streaming kernel is the faster one.  Swept over the 7B-, 13B- and hd-64-shaped layers at 5 .. 128 rows; times
// in us against the best LDS tile:
//  - no split of K in memory (QKV, gate/up), up to 32 rows: QKV 31.0 -> 22.0 (7B, 5 rows), 32.4 -> 24.7 (32 rows), 38.7 -> 26.8
//    (13B), 17.3 -> 8.7 (hd 64).  Beyond 16 rows the X operand's traffic shows once there are more than three
//    workgroups per CU: gate/up at 32 rows 36.6 -> 35.8 with 688 workgroups (7B), but 51.3 -> 56.1 with 864 (13B).
//  - 33 .. 96 rows: 64-feature tiles, two or three token panels per workgroup, as long as every workgroup has a CU of
//    its own (256 registers): QKV 33.5 -> 27.6 (7B, 64 rows), 35.8 -> 31.5 (96 rows), 42.8 -> 34.1 (13B, 64); gate/up 18.9 ->
//    16.9 (hd 64, 176 workgroups), but 37.9 -> 52 with 344 (7B).  Three panels only where that leaves half the CUs busy.
//  - O and down: K split until the workgroups fill the CUs once; the gain is the few partial sums (RMSNorm 8.2 -> 6.7),
//    the products themselves are level (O 10.9 -> 10.3, down 20.3 -> 20.0 at 5 rows; 14.8 -> 14.2 and 26.1 -> 25.5 at 77).
//    With the 160 panels of the 13B shape the CUs are not filled: up to 16 rows still 23.9 -> 20.4 with the norm, at
//    32 rows 24.2 -> 25.8; at 33 .. 64 rows down loses more (22.9 -> 25.4) than the norm gains.  Nor are they with the 32 panels of
//    1024 x 2816 in four pieces each, whose products are short: a layer of 17 rows 37.7 -> 35.2 with O streamed, 34.9 with down (32 rows:
//    38.7 -> 36.4, 35.8).
// Whole layers with and without it, weights out of reach of the caches, at eight widths from 1024 x 2816 to 8192 x 28672:
//   rows          16                 32                 64                 96
//   1024    47.2 ->  29.4      48.2 ->  37.5      46.8 ->  43.4      47.1 ->  43.2
//   2048    65.7 ->  44.5      66.6 ->  48.5      68.8 ->  61.4      71.1 ->  65.6
//   3072    91.5 ->  69.2      93.0 ->  73.4      95.7 ->  87.7     106.1 ->  97.4
//   4096   118.5 ->  97.6     120.8 -> 103.6     127.8 -> 119.9     145.7 -> 136.0
//   5120   154.3 -> 133.5     159.0 -> 143.4     170.0 -> 156.7     196.7 -> 187.1
//   6144   203.4 -> 173.8     203.5 -> 202.7     214.3 -> 214.1     246.0 -> 250.2
//   8192   370.2 -> 321.8     375.0 -> 361.0     389.6 -> 389.7     425.3 -> 419.8
// (one product lost more than the runs differ: down of 6144 x 16384 at 96 rows, 2 us of 250).
static bool stream_plan(const HatGemm& g, HatGemmPlan* p) {
  if (g.T > 96 || g.epilogue == HAT_EPI_P32) return false;
  p->ksplit = 1;
  if (g.epilogue != HAT_EPI_RESID) {
    if (g.T <= 32) {
      p->tile = kStream32;
      return g.T <= 16 || g.Nw / 32 <= 768;
    }
    p->tile = g.T > 64 && g.Nw / 64 >= 128 ? kStream96 : kStream64;
    const int bt = p->tile == kStream96 ? 96 : 64;
    return (g.T + bt - 1) / bt * (g.Nw / 64) <= 256;
  }
  if (g.T > 32 && g.T <= 64) return false;
  p->tile = g.T <= 32 ? kStream32 : kStream96;
  const int tiles = g.Nw / (g.T <= 32 ? 32 : 64);
  if (g.T <= 32 && (long)g.Nw * g.K <= 1 << 18) return true;   // nothing to stream: the K split among a workgroup's waves is the gain
  while (p->ksplit < 4 && tiles * p->ksplit * 2 <= 256 && g.part && (long)p->ksplit * 2 * g.T <= g.part_rows) p->ksplit *= 2;
  return tiles * p->ksplit >= (g.T <= 16 || p->ksplit == 4 ? 128 : 192);
}

HatGemmPlan hat_gemm_plan(const HatGemm& g) {
  // Estimated time of a candidate = rounds of 256 workgroups x the larger of the
  // MFMA time and the L2->LDS streaming time of one workgroup; split-K (only where
  // the result is accumulated in fp32) adds the traffic of its partial sums.
  HatGemmPlan best{0, 1};
  if (g.epilogue == HAT_EPI_QKV) {
    // wherever the product streams: the epilogue costs less than the rotary and append kernel it replaces (5 us).
    // 64-feature tiles from 17 rows on: 24.4 against 27.0 us at 32 rows of the 7B shape (half the reads of X and
    // whole panels of W), but 22.3 against 21.0 at 5 rows (192 workgroups instead of 384).  One such workgroup fits a CU:
    // above 256 of them (d_model 5504 and up) a second round costs more than it saves, and the 32-feature tile is ahead of the LDS
    // tiles up to 24 rows only (layer of 6144 x 4096 at 17 / 24 / 32 rows: LDS 121.7 / 115.1 / 120.3 us, 32-feature tile 115.9 / 112.2 /
    // 121.4, 64-feature tile 118.2 / 115.9 / 122.3).
    if (g.force_tile >= 0) {
      best.tile = stream_built(g.force_tile, HAT_EPI_QKV) ? g.force_tile : -1;
      return best;
    }
    if (!stream_plan(g, &best)) best.tile = -1;
    if (best.tile == kStream32 && g.T > 16) best.tile = g.Nout / 64 <= 256 ? kStream64x32 : g.T <= 24 ? kStream32 : -1;
    return best;
  }
  if (g.force_tile >= 0 && (g.force_tile < kNumLdsTiles || stream_built(g.force_tile, g.epilogue))) {
    best.tile = g.force_tile;
    best.ksplit = g.force_ksplit > 0 ? g.force_ksplit : 1;
    if (g.epilogue != HAT_EPI_RESID || !g.part) best.ksplit = 1;
    while (best.ksplit > 1 && ((long)best.ksplit * g.T > g.part_rows || g.K / 64 / best.ksplit < 1)) --best.ksplit;
    return best;
  }
  HatGemmPlan stream{};
  if (stream_plan(g, &stream)) return stream;
  // Two regimes, each a small cost model whose constants are searched for the least loss against the best measured tile and K split.
  // Up to kMidT rows (kTau): a k-tile costs what it costs the tile, more where a panel of W is read by several token tiles; a round of workgroups costs
  // its prologue and drain; the last round counts for less than a whole one; the partial sums of a K split, written here and read by the consumer of the
  // residual, and the update of the fp32 residual cost by their rows; and the weight stream cannot be beaten.
  // Above that (kEff) a k-tile costs the larger of its MFMA time at the tile's own
  // weight and its load time at 23.7 B/clk, a round of workgroups costs ~4.3 us of
  // prologue and drain, and the epilogue's traffic is not hidden: 14 B/clk per CU for the
  // fp16 stores (the rotating epilogue of QKV, which costs more, is taken for one: its choices lose 0.03 % of a layer),
  // 7.65 for the read-modify-write of the fp32 residual, 6.7 for split-K partial
  // sums (written here, read back by the consumer of the residual).
  double best_cost = 1e300, tail_cost = 1e300;
  HatGemmPlan tail{0, 1};
  const int KT = g.K / 64;
  const bool large = g.T > kMidT;
  for (int c = 0; c < kNumLdsTiles; ++c) {
    const TileInfo& q = kTiles[c];
    // (0: tiles that are never the best there; beyond kSmallT rows nor are 64-row token tiles with loader waves)
    if (large ? q.eff == 0.f : kTau[c] == 0.f || (c == 10 ? g.T <= 256 : g.T > kSmallT && q.bt < 128)) continue;
    // 160/192/224-row token tiles: not up to 256 rows, except the 128 x 160 tile (23), which exists for batches
    // of 129 .. 160 rows (a second, mostly empty 128-row token tile costs them 15-20 %) and competes with the others there: most O, gate/up and down products from 4096 columns on take it, but not O of 4096 columns
    // (64 x 256: a step of 150 rows 150.9 -> 149.8 us a layer) nor gate/up of 7168, where its 296 workgroups go round twice (192 x 256: 129 rows 355.5 -> 343.3).  Gate/up of the 7B shape at 150 rows takes it, 50.3 us,
    // where 96 x 256, which pads 256 rows, would take 47.9.  Above 256 rows a third
    // 128-row token tile or a second 256-row one is as empty: the four products and the norms of a layer at 257 and 320 rows 219 -> 193 and 229 -> 202 us (7B shape),
    // 282 -> 257 and 301 -> 267 (13B) when these tiles were offered there; at 384 rows, three whole 128-row
    // tiles but also two of 192, steps take 318 -> 304 us a layer (13B), 431 -> 393 (6144 columns) and 883 -> 766 (8192).
    const bool tall = g.T > 256 || (c == 23 && g.T > 128 && g.T <= 160);
    if ((q.bt & (q.bt - 1)) != 0 && !tall) continue;
    const int nT = (g.T + q.bt - 1) / q.bt, nF = (g.Nw + q.bf - 1) / q.bf;
    const int max_split = (g.epilogue == HAT_EPI_RESID && g.part) ? 16 : 1;
    for (int ks = 1; ks <= max_split; ++ks) {
      if (ks > 1 && (KT / ks < 4 || (long)ks * g.T > g.part_rows)) break;
      const double blocks = (double)nT * nF * ks;
      const double rounds = std::ceil(blocks / 256.0);
      const double kt = std::ceil((double)KT / ks) + 2.0;                     // + pipeline fill
      const double rows = (double)g.T * g.Nout / 256.0;                       // output elements per CU
      double cost;
      if (large) {
        const double mfma_cyc = 2.0 * q.bf * q.bt * 64 / (4 * 1017.0 * q.eff);  // per k-tile, 4 SIMDs
        const double load_cyc = (q.bf + q.bt) * 64 * 2 / 23.7;
        const double tile_cyc = std::max(mfma_cyc, load_cyc) + 0.068 * std::min(mfma_cyc, load_cyc);
        double cyc = rounds * kt * tile_cyc + rounds * 10300.0;
        if (g.epilogue != HAT_EPI_RESID) cyc += rows * 2.0 / 14.0;
        else if (ks == 1) cyc += rows * 8.0 / 7.65;
        else cyc += rows * 8.0 * ks / 6.73;
        const double hbm_cyc = 2.0 * g.Nw * g.K / 5.5e12 * 2.4e9 + 7000.0;
        cost = std::max(cyc, hbm_cyc) + 1e-3 * cyc;                             // tie-break below the HBM floor
      } else {
        const double r = (1 - kMid.fraction) * rounds + kMid.fraction * std::max(1.0, blocks / 256.0);
        double us = r * (kt * kTau[c] * (nT > 1 ? 1 + kMid.shared : 1) + (c == 10 ? kMid.round_plain : kMid.round));
        if (g.epilogue == HAT_EPI_RESID) us += 1e-3 * rows * (ks > 1 ? ks * kMid.part : kMid.resid);
        cost = std::max(us, 2e-6 * g.Nw * g.K / kMid.tbs + kMid.stream) + 0.02 * us;
      }
      if (cost < best_cost) { best_cost = cost; best.tile = c; best.ksplit = ks; }
    }
    // A last round that leaves most CUs idle: the token tiles that fill whole rounds stay whole, the rest is split
    // along K until its pieces fill about a round.  320 tiles on 256 CUs (4096 rows of the 13B shape) take 1.35 rounds
    // instead of 2.  The matrix pipes draw the chip's power limit in a step of this size (clock 1.6 GHz in a
    // full round), so the idle CUs are not all loss.  Only where it is predicted to win by 4.5 %, and in at most 8 pieces.  O and down with their norms, whole against
    // split in us: at the sizes of kEff the rule takes it 47 times, all at 5120, 6144 and 8192 columns.  Down gains each time, 10 .. 171 us (13B shape 4096 rows 544 -> 490,
    // 3300 rows 465 -> 410; 6144 x 16384 2788 rows 558 -> 480; 8192 x 28672 2300 rows 1061 -> 890); O gains 1 .. 27 in 16 of 19 (3300 rows of 5120 218 -> 200) and
    // loses 2 and twice 7 (3840 and 3450 rows of 6144, 3072 of 8192 392 -> 399).  Predicted below 4.5 % it gains 0 .. 6 at four sizes.  In 13 .. 16 pieces
    // (2065 rows of 3072 x 8192, predicted 5 %) a layer lost 594 -> 598.
    if (!large || max_split == 1) continue;
    const int whole = nT * nF / 256, full = whole * 256 / nF;
    if (full < 1 || full >= nT) continue;
    for (int ks = 2; ks <= 8 && KT / ks >= 4 && (long)ks * (g.T - full * q.bt) <= g.part_rows; ++ks) {
      const double pieces = (double)(nT - full) * nF * ks - (256.0 * whole - (double)full * nF);   // idle CUs take some early
      const double mfma_cyc = 2.0 * q.bf * q.bt * 64 / (4 * 1017.0 * q.eff), load_cyc = (q.bf + q.bt) * 64 * 2 / 23.7;
      const double tile_cyc = std::max(mfma_cyc, load_cyc) + 0.068 * std::min(mfma_cyc, load_cyc);
      const double part_rounds = std::ceil(pieces / 256.0);
      double cyc = whole * ((KT + 2.0) * tile_cyc + 10300.0) + part_rounds * ((std::ceil((double)KT / ks) + 2.0) * tile_cyc + 10300.0);
      cyc += full * q.bt * (double)g.Nout / 256.0 * 8.0 / 7.65 + (g.T - full * q.bt) * (double)g.Nout / 256.0 * 8.0 * ks / 6.73;
      cyc += 12000.0;   // the norm that follows takes two launches
      if (cyc * 1.001 < tail_cost) { tail_cost = cyc * 1.001; tail.tile = c; tail.ksplit = ks; tail.full = full; }
    }
  }
  return tail_cost < 0.955 * best_cost ? tail : best;
}

hipError_t hat_launch_gemm(const HatGemm& g, const HatGemmPlan& p, hipStream_t st) {
  if (g.T <= 0) return hipSuccess;
  if (g.K % 64 != 0 || g.Nw % 256 != 0) return hipErrorInvalidValue;
  if (p.ksplit > 1 && (g.epilogue != HAT_EPI_RESID || !g.part)) return hipErrorInvalidValue;
  switch (g.epilogue) {
    case HAT_EPI_P32: return launch_epi<HAT_EPI_P32>(g, p, st);
    case HAT_EPI_SWIGLU: return launch_epi<HAT_EPI_SWIGLU>(g, p, st);
    case HAT_EPI_RESID: return launch_epi<HAT_EPI_RESID>(g, p, st);
    case HAT_EPI_QKV: return launch_epi<HAT_EPI_QKV>(g, p, st);
  }
  return hipErrorInvalidValue;
}
