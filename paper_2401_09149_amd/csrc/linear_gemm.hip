// Linear modules without bias, forward and backward (include/ie_linear.h; Sec. 2.1; Sec. 4.2
// "Computation Profiler": the input of dimension (b, S/s_sp, H) applied to a Linear module):
//   y = x w^T,   dx = dy w,   dw = dy^T x        x [M,K], w [N,K], y, dy [M,N], all bf16 row-major.
// All three are C[I,J] = sum_r A(i,r) B(j,r) with each operand stored either with r contiguous
// ("direct": x and w in the forward, dy in dx) or with its output index contiguous ("transposed":
// w in dx, dy and x in dw), so kernel templates with two flags serve them.
//
// Three kernels share the tile order, the copies and the fragment layouts.  linear_pp_kernel computes 256 x 256 tiles of C
// and is the faster one per product; linear_ring_kernel computes smaller ones, down to 32 x 32, for outputs that
// do not fill the chip with large tiles (pick_tile in dispatch.hpp chooses); linear_own_kernel serves the forward product over few
// tokens (pick_own).  In the first two a workgroup is 8 wavefronts (two per SIMD),
// one workgroup per CU, each walking its share of the tiles; operands reach LDS by asynchronous copies that run ahead
// of the products across tile boundaries.  Tiles sit in LDS row-major with swizzled 16-byte chunks; a direct operand's
// fragment is one 16-byte LDS read, a transposed operand's two transpose loads.  The products are formed transposed,
// C^T = B A^T (B's rows as the MFMA's row operand), so that a lane ends up holding one row i of C with consecutive j.
#include "../../include/ie_linear.h"

#include <hip/hip_runtime.h>

#include <type_traits>

#include "attn_common.hpp"
#include "dispatch.hpp"
#include "launch.hpp"

namespace ie {
namespace {

constexpr int kWaves = 8;
constexpr int kPanel = 8;                          // i-tiles that share a j-tile back to back

struct GemmParams {
  const char* a;   // the operand indexed by (i, r)
  const char* b;   // the operand indexed by (j, r)
  __bf16* c;       // [I][J]
  int64_t I, J, R;
  int64_t a_pitch, b_pitch;  // bytes between rows of a / b as stored
  int64_t c_pitch;           // elements
  int tiles_i, tiles_j, tiles;
};

// Swizzle of a direct tile (rows of 128 bytes): the 16-byte chunk c of row r sits at chunk position
// c ^ dswz(r).  A 16-byte LDS read is served 16 lanes at a time across 256 bytes of banks, i.e. two rows
// of this tile side by side, so the 16 consecutive rows of a fragment read must put the requested
// chunk at 8 different positions for the even rows and 8 for the odd ones.  (The attention tiles'
// swizzle, made for 256-byte rows and for transpose loads as well, gives only 4: measured, half of all
// LDS cycles of the forward product were bank conflicts with it.)
__device__ __forceinline__ uint32_t dswz(uint32_t r) { return (r >> 1) & 7u; }

// One wave's share of the copy of SUB consecutive 64-deep tiles of one operand, `EXT` = tile extent along the output index.
// A lane's offsets are worked out once per output tile (set_tile), so that a step's copies are a base address and nothing
// else, whole tile or not.  (Worked out in every step, with a path of its own for whole tiles, they were some 180
// instructions ahead of a step's LDS reads: dw 8192 tokens 3200 x 3200 209 -> 168 us and 12288 x 4096 668 -> 633, dx 4096
// tokens 17152 x 3200 426 -> 355, forward 2048 tokens 9600 x 3200 139 -> 123, all with 256 x 256 tiles; dw 6144 tokens
// 512 x 1344, 64 x 64 tiles, 37 -> 29.)  Instruction t of wave w is piece w + WAVES t of the
// SUB * EXT / 8 pieces of 1 KiB, in LDS order.
template <bool T, int EXT, int SUB, int WAVES = kWaves>
struct TileCopy {
  static constexpr uint32_t PIECES = EXT / 8;         // 1 KiB pieces of one 64-deep tile
  static constexpr int NI = SUB * PIECES / WAVES;
  static constexpr uint32_t CPR = T ? EXT / 8 : 8;    // 16-byte chunks per row
  static constexpr uint32_t RPP = 64 / CPR;           // rows per piece
  static constexpr int NV = SUB > 1 ? 1 : NI;         // (SUB > 1: a lane's instructions differ in the 64-deep tile only)
  static_assert(SUB == 1 || WAVES % PIECES == 0, "");
  uint32_t wave;
  uint32_t voff[NV];     // byte offset of this lane's 16 bytes of instruction t
  __device__ __forceinline__ void init(int tid) { wave = WAVES == 1 ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6); }
  // `valid`: rows (direct) or 16-byte chunks (transposed) that exist along the output index; what lies past them repeats
  // the last.  `first`: the tile starts at that row or chunk.
  __device__ __forceinline__ void set_tile(int tid, uint32_t pitch, int valid, uint32_t first = 0) {
    const uint32_t lane = tid & 63, last = (uint32_t)valid - 1;
    auto clamp = [&](uint32_t x) __attribute__((always_inline)) { return x + first < last ? x + first : last; };
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const uint32_t r = lane / CPR + (wave + WAVES * t) % PIECES * RPP;
      const uint32_t chunk = lane % CPR ^ (T ? (uint32_t)swz<EXT>((int)r) : dswz(r));
      voff[t] = T ? r * pitch + (clamp(chunk) << 4) : clamp(r) * pitch + (chunk << 4);
    }
  }
  // `g`: first byte of the step; `subs` of its SUB tiles exist (the others repeat the last one and are not used);
  // `sub_step`: bytes between them.
  __device__ __forceinline__ void issue(uint32_t lds, const char* g, int64_t sub_step = 0, int subs = 1) const {
#pragma unroll
    for (int t = 0; t < NI; ++t) issue_piece(t, lds, g, sub_step, subs);
  }
  __device__ __forceinline__ void issue_piece(int t, uint32_t lds, const char* g, int64_t sub_step = 0, int subs = 1) const {
    const uint32_t piece = wave + WAVES * t;
    const char* src = g;
    if constexpr (SUB > 1) {
      const uint32_t sub = piece / PIECES;
      src += (int64_t)(sub < (uint32_t)subs ? sub : (uint32_t)subs - 1) * sub_step;
    }
    async_copy16(voff[NV == 1 ? 0 : t], src, lds + piece * 1024);
  }
};

// Operand of v_mfma_f32_32x32x16_bf16: output indices o .. o+31, 16-deep slice ks of one 64-deep tile of extent EXT
// (pitch 128 bytes, or 2 EXT if transposed).
template <bool T, int EXT>
__device__ __forceinline__ bf16x8 ring_frag(const char* tile, int lane, int o, int ks) {
  const int n = lane & 31, h = lane >> 5;
  if (!T) return lds_read8(tile, (o + n) * 128 + (((2 * ks + h) ^ (int)dswz((uint32_t)(o + n))) << 4));
  const int c0 = o + 16 * ((lane >> 4) & 1), r0 = 16 * ks + 8 * h;
  return cat4(lds_read_tr4(tile + tr_off<EXT>(lane, r0, c0)), lds_read_tr4(tile + tr_off<EXT>(lane, r0 + 4, c0)));
}

// Operand of v_mfma_f32_16x16x32_bf16 (lane l: row l % 16, contraction indices 8 (l / 16) .. +7): output indices
// o .. o+15, 32-deep slice ks.
template <bool T, int EXT>
__device__ __forceinline__ bf16x8 frag16(const char* tile, int lane, int o, int ks) {
  const int n = lane & 15, g = lane >> 4;
  if (!T) return lds_read8(tile, (o + n) * 128 + (((4 * ks + g) ^ (int)dswz((uint32_t)(o + n))) << 4));
  const int r0 = 32 * ks + 8 * g;
  return cat4(lds_read_tr4(tile + tr_off<EXT>(lane, r0, o)), lds_read_tr4(tile + tr_off<EXT>(lane, r0 + 4, o)));
}

// One lane's share of a 32 x 32 accumulator block: row i of C, 32 consecutive j, of which the
// first `cols` (a multiple of 8) exist.  Same exchange as store_block32_bf16.
__device__ __forceinline__ void store_block(__bf16* dst, const f32x16& acc, int h, bool ok, int cols) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  uint32_t w[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x2_t pr;
      pr[0] = (__bf16)acc[4 * q + 2 * j];
      pr[1] = (__bf16)acc[4 * q + 2 * j + 1];
      w[q][j] = __builtin_bit_cast(uint32_t, pr);
    }
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    uint32_t lo[2], hi[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      auto r = __builtin_amdgcn_permlane32_swap(w[2 * g][j], w[2 * g + 1][j], false, false);
      lo[j] = r[0];
      hi[j] = r[1];
    }
    u32x4 out = {lo[0], lo[1], hi[0], hi[1]};
    if (ok && 16 * g + 8 * h < cols) *reinterpret_cast<u32x4*>(dst + 16 * g + 8 * h) = out;
  }
}

// Tile sequence.  The hardware deals consecutive workgroups round-robin to the 8 XCDs; XCD x
// (= workgroup index % 8) works through a contiguous eighth of the sequence, and the sequence
// walks panels of 8 i-tiles, all 8 against one j-tile before the next j-tile, so that the
// workgroups that run together on an XCD share a few A and B panels in its L2.  `l` numbers the
// tiles of one XCD's eighth.
struct GemmTile {
  const char* ga;  // first byte of the A tile of contraction step 0 (the copies' position moves it on step by step)
  const char* gb;
  int64_t i0, j0;
  int i_valid, j_valid, a_valid, b_valid;
  bool valid;
};
template <bool A_T, bool B_T, int TI, int TJ>
__device__ __forceinline__ GemmTile decode_gemm_tile(const GemmParams& p, int l) {
  GemmTile g;
  const int per = (p.tiles + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + l;
  g.valid = l < per && t < p.tiles;
  if (!g.valid) return g;
  const int panel_tiles = kPanel * p.tiles_j;
  const int panel = t / panel_tiles, in_panel = t % panel_tiles;
  const int rows_in_panel = p.tiles_i - panel * kPanel < kPanel ? p.tiles_i - panel * kPanel : kPanel;
  const int tj = in_panel / rows_in_panel;
  const int ti = panel * kPanel + in_panel % rows_in_panel;
  g.i0 = (int64_t)ti * TI;
  g.j0 = (int64_t)tj * TJ;
  g.i_valid = (int)(p.I - g.i0 < TI ? p.I - g.i0 : TI);
  g.j_valid = (int)(p.J - g.j0 < TJ ? p.J - g.j0 : TJ);
  g.ga = p.a + (A_T ? g.i0 * 2 : g.i0 * p.a_pitch);
  g.gb = p.b + (B_T ? g.j0 * 2 : g.j0 * p.b_pitch);
  g.a_valid = A_T ? g.i_valid / 8 : g.i_valid;
  g.b_valid = B_T ? g.j_valid / 8 : g.j_valid;
  return g;
}

// ---- 256 x 256 tiles ------------------------------------------------------------------------------
// Bound: the matrix pipeline at the clock that power management grants.  What an MFMA costs in power is why this
// kernel is built on the 16x16x32 form (half the accumulator traffic per product of the 32x32x16 one): with the same
// schedule the 32x32x16 form took 2-7 % longer at 8192 tokens x 4096, at a lower clock.
// Wave (wi, wj) owns rows 64 wi .. +63 of both 128-row halves A0, A1 of the tile and columns 32 wj .. +31 of both
// 128-column halves B0, B1 (128 accumulator registers).  The two waves of a SIMD (w and w + 4) alternate: while one
// runs a cluster of 32 MFMAs, the other reads its next operands and issues copies; one workgroup barrier separates the
// turns, waves 4-7 are one turn late.  A 64-deep step is two turns: read A0, B0, B1, products A0 B0 and A0 B1; read A1,
// products A1 B1 and A1 B0.  A half that has been read is copied over at once with the step after next's, so a copy
// has a whole step to arrive in two LDS stages of 64 KiB.  (Four turns of 16 MFMAs per step, copies behind the MFMAs
// instead of behind the reads, 32-deep steps in a ring of four or five, and one turn of 64 per step were 3-4 %, 15-20 %,
// 10-15 % and 40 % slower: every turn pays an LDS latency, and a copy that waits for the memory pipeline in a cluster
// holds the MFMAs behind it.)
// 8192 tokens, the twelve products of hidden 4096 / MLP 11008: 0.47-0.62 of the 2.5 PFLOP/s peak, the matrix pipeline busy
// 83 % (forward), 76 % (dx) and 64 % (dw) of the time (eight waves in step at one barrier per 64-deep step: QKV 664, 649,
// 688 us; these turns: 571, 578, 668; with the copies' offsets worked out once per tile: 543, 563, 633).
constexpr int TI = 256, TJ = 256;
constexpr int P_HALF_BYTES = 128 * 128;              // half an operand tile: 128 output indices x 64 deep
constexpr int P_STAGE_BYTES = 4 * P_HALF_BYTES;      // A0 | A1 | B0 | B1
constexpr int P_SMEM_BYTES = 2 * P_STAGE_BYTES;
template <bool A_T, bool B_T>
__global__ __launch_bounds__(kWaves * 64, 1) void linear_pp_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g4 = lane >> 4;
  const int wi = wv & 1, wj = (wv >> 1) & 3;
  const bool late = wv >= 4;
  const int lstep = (int)(gridDim.x >> 3);
  const int nkt = (int)(p.R / 64);
  const int64_t a_step = A_T ? 64 * p.a_pitch : 128, b_step = B_T ? 64 * p.b_pitch : 128;
  TileCopy<A_T, 128, 1> ca[2];   // the two halves of the operand tile
  TileCopy<B_T, 128, 1> cb[2];
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) { ca[hf].init(tid); cb[hf].init(tid); }
  const uint32_t lds0 = lds_address(smem);

  int cl = (int)(blockIdx.x >> 3), ckt = 0, cslot = 0;
  GemmTile ctile = decode_gemm_tile<A_T, B_T, TI, TJ>(p, cl);
  if (!ctile.valid) return;
  GemmTile cur = ctile;
  int l = cl;
  auto set_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      ca[hf].set_tile(tid, (uint32_t)p.a_pitch, ctile.a_valid, hf * (A_T ? 16 : 128));
      cb[hf].set_tile(tid, (uint32_t)p.b_pitch, ctile.b_valid, hf * (B_T ? 16 : 128));
    }
  };
  // A step's copies: A0, B0 and B1 first, A1 a turn later, which then moves on to the next step.
  auto copy_first = [&]() __attribute__((always_inline)) {
    const uint32_t base = lds0 + cslot * P_STAGE_BYTES;
    ca[0].issue(base, ctile.ga);
    cb[0].issue(base + 2 * P_HALF_BYTES, ctile.gb);
    cb[1].issue(base + 3 * P_HALF_BYTES, ctile.gb);
  };
  auto copy_last = [&]() __attribute__((always_inline)) {
    ca[1].issue(lds0 + cslot * P_STAGE_BYTES + P_HALF_BYTES, ctile.ga);
    cslot ^= 1;
    ctile.ga += a_step;
    ctile.gb += b_step;
    if (++ckt == nkt) {
      ckt = 0;
      cl += lstep;
      ctile = decode_gemm_tile<A_T, B_T, TI, TJ>(p, cl);
      if (ctile.valid) set_tile();
    }
  };
  set_tile();
  copy_first();
  copy_last();
  bool pend = ctile.valid;   // the step at the copies' position lacks its A1
  if (pend) copy_first();
  async_wait_all();
  __syncthreads();
  auto bar = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto reads_done = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if (late) bar();
  int slot = 0;
  for (;;) {
    f32x4 acc[2][2][4][2];   // [A half][B half][ib][jb]
#pragma unroll
    for (int x = 0; x < 32; ++x) acc[x >> 4][(x >> 3) & 1][(x >> 1) & 3][x & 1] = f32x4{0, 0, 0, 0};
    bf16x8 fa[4][2], fb[2][2][2];
    for (int kt = 0; kt < nkt; ++kt) {
      const char* st = smem + slot * P_STAGE_BYTES;
      auto read_a = [&](int hf) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int ib = 0; ib < 4; ++ib) fa[ib][ks] = frag16<A_T, 128>(st + hf * P_HALF_BYTES, lane, wi * 64 + ib * 16, ks);
      };
      auto read_b = [&](int hf) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int jb = 0; jb < 2; ++jb) fb[hf][jb][ks] = frag16<B_T, 128>(st + (2 + hf) * P_HALF_BYTES, lane, wj * 32 + jb * 16, ks);
      };
      auto products = [&](int ha, int hb) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int ib = 0; ib < 4; ++ib)
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) acc[ha][hb][ib][jb] = mfma16(fb[hb][jb][ks], fa[ib][ks], acc[ha][hb][ib][jb]);
        __builtin_amdgcn_s_setprio(0);
      };
      read_b(0);
      read_a(0);
      read_b(1);
      // A1 of the next step goes where every wave has read this slot's predecessor in the previous turn but one.  What
      // must have landed behind this turn is this step's A1: all but the eight youngest copies, six of the next
      // step's first three halves and the two issued here (the epilogue's stores are younger and only tighten the wait).
      if (pend) {
        copy_last();
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      reads_done();
      products(0, 0);
      products(0, 1);
      bar();
      read_a(1);
      // The step after next's A0, B0 and B1 go where this step's have been read; the next step's must have landed.
      pend = ctile.valid;
      if (pend) {
        copy_first();
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      reads_done();
      products(1, 1);
      products(1, 0);
      bar();
      slot ^= 1;
    }
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) {
        const int il = ha * 128 + wi * 64 + ib * 16 + n;
        const bool ok = il < cur.i_valid;
        __bf16* crow = p.c + (cur.i0 + (ok ? il : 0)) * p.c_pitch + cur.j0;
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          const u32x4 out = exchange_pair16(acc[ha][hb][ib][0], acc[ha][hb][ib][1]);   // eight consecutive columns per lane
          const int j = hb * 128 + wj * 32 + 16 * (g4 & 1) + 8 * (g4 >> 1);
          if (ok && j < cur.j_valid) *reinterpret_cast<u32x4*>(crow + j) = out;
        }
      }
    l += lstep;
    cur = decode_gemm_tile<A_T, B_T, TI, TJ>(p, l);
    if (!cur.valid) break;
  }
  if (!late) bar();
}

// ---- smaller tiles ----------------------------------------------------------------------------------
// The same products where 256 x 256 tiles would leave most of the chip idle (few tokens, small layers) or where the
// time is the weights' way from HBM: tiles of CI x CJ, contraction steps of 64 SUB through a ring of NS LDS stages
// with NS - 1 of them in flight, and WK groups of waves that each take every WK-th 16-deep slice of a step for the
// whole tile (their partial sums are added through LDS at the tile's end, in fp32 and in a fixed order).
// Bound: at one step in flight a step took 1.25 us however little it did, the latency of a cold copy, so the ring holds
// as many bytes in flight as fit (80-120 KiB); what is left is HBM for a handful of tokens (one token, 22016 x 4096:
// 34 us = 5.3 TB/s) and LDS bandwidth and the barrier per step for the wider tiles.
template <int CI_, int CJ_, int WI_, int WJ_, int WK_, int SUB_, int NS_>
struct RingCfg {
  static constexpr int CI = CI_, CJ = CJ_, WI = WI_, WJ = WJ_, WK = WK_, SUB = SUB_, NS = NS_;
  static constexpr int NIB = CI / WI / 32, NJB = CJ / WJ / 32;   // 32 x 32 blocks of a wave
  static constexpr int A_BYTES = CI * 128, B_BYTES = CJ * 128;   // one 64-deep tile of each operand
  static constexpr int STAGE_BYTES = SUB * (A_BYTES + B_BYTES);
  static constexpr int RED_BYTES = WK > 1 ? CI * CJ * 4 * WK : 0;
  static constexpr int SMEM_BYTES = NS * STAGE_BYTES + RED_BYTES;
  static constexpr int COPIES = STAGE_BYTES / 1024 / kWaves;     // copy instructions of a wave per stage
  static_assert(WI * WJ * WK == kWaves && SMEM_BYTES <= 160 * 1024 && STAGE_BYTES % (1024 * kWaves) == 0, "");
};

template <bool A_T, bool B_T, typename C>
__global__ __launch_bounds__(kWaves * 64, 1) void linear_ring_kernel(GemmParams p) {
  constexpr int CI = C::CI, CJ = C::CJ, SUB = C::SUB, NS = C::NS, WK = C::WK, NIB = C::NIB, NJB = C::NJB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int wi = wv % C::WI, wj = (wv / C::WI) % C::WJ, wk = wv / (C::WI * C::WJ);
  const int lstep = (int)(gridDim.x >> 3);
  const int nr = (int)(p.R / 64);                 // 64-deep tiles of the contraction
  const int nkt = (nr + SUB - 1) / SUB;           // steps
  const int64_t a_step = A_T ? 64 * p.a_pitch : 128, b_step = B_T ? 64 * p.b_pitch : 128;

  TileCopy<A_T, CI, SUB> ca;
  TileCopy<B_T, CJ, SUB> cb;
  ca.init(tid);
  cb.init(tid);
  const uint32_t lds0 = lds_address(smem);

  // The copies run ahead of the products by NS - 1 steps, across tile boundaries: (ctile, ckt) is the next step to copy.
  int cl = (int)(blockIdx.x >> 3), ckt = 0, cslot = 0;
  GemmTile ctile = decode_gemm_tile<A_T, B_T, CI, CJ>(p, cl);
  if (!ctile.valid) return;
  GemmTile cur = ctile;
  int l = cl;
  ca.set_tile(tid, (uint32_t)p.a_pitch, ctile.a_valid);
  cb.set_tile(tid, (uint32_t)p.b_pitch, ctile.b_valid);
  auto copy_next = [&]() __attribute__((always_inline)) {
    const uint32_t base = lds0 + cslot * C::STAGE_BYTES;
    const int subs = nr - ckt * SUB;
    ca.issue(base, ctile.ga, a_step, subs);
    cb.issue(base + SUB * C::A_BYTES, ctile.gb, b_step, subs);
    ctile.ga += SUB * a_step;
    ctile.gb += SUB * b_step;
    cslot = cslot + 1 == NS ? 0 : cslot + 1;
    if (++ckt == nkt) {
      ckt = 0;
      cl += lstep;
      ctile = decode_gemm_tile<A_T, B_T, CI, CJ>(p, cl);
      if (ctile.valid) {
        ca.set_tile(tid, (uint32_t)p.a_pitch, ctile.a_valid);
        cb.set_tile(tid, (uint32_t)p.b_pitch, ctile.b_valid);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (ctile.valid) copy_next();

  int slot = 0;
  for (;;) {
    f32x16 acc[NIB][NJB];
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ib][jb][r] = 0.0f;
    for (int kt = 0; kt < nkt; ++kt) {
      // This wave's copies of the step have landed (the younger steps' may be open while there are any to come; the
      // epilogue's stores are younger than the copies they leave open, so the count is safe with them too) and its LDS
      // reads of the previous step are done; behind the barrier the same holds for all waves.
      if (ctile.valid) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(C::COPIES * (NS - 2)) : "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (ctile.valid) copy_next();   // into the stage everyone has just left
      const char* st = smem + slot * C::STAGE_BYTES;
      auto slice = [&](int ks) __attribute__((always_inline)) {
        const char* ta = st + (SUB > 1 ? (ks >> 2) * C::A_BYTES : 0);
        const char* tb = st + SUB * C::A_BYTES + (SUB > 1 ? (ks >> 2) * C::B_BYTES : 0);
        bf16x8 fi[NIB], fj[NJB];
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib) fi[ib] = ring_frag<A_T, CI>(ta, lane, (wi * NIB + ib) * 32, ks & 3);
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) fj[jb] = ring_frag<B_T, CJ>(tb, lane, (wj * NJB + jb) * 32, ks & 3);
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
          for (int jb = 0; jb < NJB; ++jb) acc[ib][jb] = mfma32(fj[jb], fi[ib], acc[ib][jb]);
      };
      const int left = (nr - kt * SUB) * 4;   // 16-deep slices that exist from here on
      if (SUB == 1 || left >= SUB * 4) {
#pragma unroll
        for (int s = 0; s < SUB * 4 / WK; ++s) slice(wk + WK * s);
      } else {
        for (int ks = wk; ks < left; ks += WK) slice(ks);
      }
      slot = slot + 1 == NS ? 0 : slot + 1;
    }

    if constexpr (WK == 1) {
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        const int il = (wi * NIB + ib) * 32 + n;
        const bool ok = il < cur.i_valid;
        __bf16* crow = p.c + (cur.i0 + (ok ? il : 0)) * p.c_pitch + cur.j0;
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) {
          const int jl = (wj * NJB + jb) * 32;
          store_block(crow + jl, acc[ib][jb], h, ok, cur.j_valid - jl);
        }
      }
    } else {
      // Partial sums through LDS, [wj wi group][block][quad q][wk][lane] x 16 bytes: quad q of a block is four
      // consecutive columns 8 q + 4 h of row n.  Reader wk adds the quads q = wk, wk + WK, ... of its group's blocks.
      constexpr int NB = NIB * NJB;
      float* red = reinterpret_cast<float*>(smem + NS * C::STAGE_BYTES) + (wj * C::WI + wi) * NB * 4 * WK * 256;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x16& a = acc[ib][jb];
            f32x4 v = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
            *reinterpret_cast<f32x4*>(red + (((ib * NJB + jb) * 4 + q) * WK + wk) * 256 + lane * 4) = v;
          }
      // (the reads below are done before this wave reaches the next step's barrier, hence before the area is written again)
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        const int il = (wi * NIB + ib) * 32 + n;
        const bool ok = il < cur.i_valid;
        __bf16* crow = p.c + (cur.i0 + (ok ? il : 0)) * p.c_pitch + cur.j0;
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb)
          for (int q = wk; q < 4; q += WK) {
            const float* src = red + ((ib * NJB + jb) * 4 + q) * WK * 256 + lane * 4;
            f32x4 sum = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
            for (int k = 1; k < WK; ++k) sum += *reinterpret_cast<const f32x4*>(src + k * 256);
            const int j = (wj * NJB + jb) * 32 + 8 * q + 4 * h;
            bf16x4 out = {(__bf16)sum[0], (__bf16)sum[1], (__bf16)sum[2], (__bf16)sum[3]};
            if (ok && j < cur.j_valid) *reinterpret_cast<bf16x4*>(crow + j) = out;
          }
      }
    }
    l += lstep;
    cur = decode_gemm_tile<A_T, B_T, CI, CJ>(p, l);
    if (!cur.valid) break;
  }
}

// ---- forward product over few tokens: waves that share nothing ----------------------------------------
// A small tile's step in the ring kernel is a chain of barrier, copies, LDS reads and products that eight waves walk
// together, 0.23-0.28 us for 16 KiB.  Here each of four waves, one per SIMD, computes the whole tile over every fourth 64-deep
// step, with a ring in LDS of its own: no barrier until the four partial sums are added (in fp32, in the order of the waves,
// through the slots that each wave has read last), every byte is read from LDS once, and a step's fragments go to registers
// in one go, so that its slots are filled again behind its own first products.
// Bound: the loaded latency of the copies (2 us) over the 112-160 KiB that LDS has room for in flight, 55-65 GB/s per CU.  (L2 alone
// delivers 105.  Fragments loaded from memory straight to registers take half the rate, whatever their number in flight; lines of
// the weights touched 4 to 32 steps ahead make every tile slower.)  200 tokens, the ring kernel -> this one, weights in
// the caches and from memory: 4096 x 4096 17.6 -> 14.4, 17.8 -> 16.9 us, 4096 x 11008 39.8 -> 33.9, 42.2 -> 42.1 (64 x 64), 12288 x
// 4096 39.2 -> 29.7, 41.0 -> 35.4 (128 x 96).
template <int CI_, int CJ_, int NA_, int NB_>
struct OwnCfg {
  static constexpr int CI = CI_, CJ = CJ_, NA = NA_, NB = NB_, WAVES = 4;   // NA, NB: 64-deep steps of each operand in a wave's ring
  static constexpr int NIB = CI / 32, NJB = CJ / 32, BLOCKS = NIB * NJB;
  static constexpr int A_BYTES = CI * 128, B_BYTES = CJ * 128;              // one step of each operand
  static constexpr int RING_BYTES = NA * A_BYTES + NB * B_BYTES, SMEM_BYTES = WAVES * RING_BYTES;
  static constexpr int CA = CI / 8, CB = CJ / 8;                            // copy instructions of a step
  // Copies younger than those of the step that comes next, A's or B's, whichever are the fewer.
  static constexpr int YOUNGER = CB + (NA - 1) * (CA + CB) < (NB - 1) * (CA + CB) ? CB + (NA - 1) * (CA + CB) : (NB - 1) * (CA + CB);
  // Blocks of partial sums that fit the two slots a wave has read last.
  static constexpr int ROUNDS = (BLOCKS + NIB + NJB - 1) / (NIB + NJB), PER_ROUND = (BLOCKS + ROUNDS - 1) / ROUNDS;
  static_assert(SMEM_BYTES <= 160 * 1024 && YOUNGER < 64 && NA <= NB, "");
};

template <typename C>
__global__ __launch_bounds__(C::WAVES * 64, 1) void linear_own_kernel(GemmParams p) {
  constexpr int CI = C::CI, CJ = C::CJ, NA = C::NA, NB = C::NB, NIB = C::NIB, NJB = C::NJB, W = C::WAVES;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int lstep = (int)(gridDim.x >> 3);
  const int nr = (int)(p.R / 64);
  const int mine = (nr - wv + W - 1) / W;   // steps of this wave per tile: wv, wv + 4, ...; NB at least

  TileCopy<false, CI, 1, 1> ca;
  TileCopy<false, CJ, 1, 1> cb;
  ca.init(tid);
  cb.init(tid);
  char* const ring = smem + wv * C::RING_BYTES;
  const uint32_t lds_a = lds_address(ring), lds_b = lds_a + NA * C::A_BYTES;

  int l = (int)(blockIdx.x >> 3);
  GemmTile cur = decode_gemm_tile<false, false, CI, CJ>(p, l);
  if (!cur.valid) return;
  const char* ga = cur.ga + wv * 128;   // the next steps to copy
  const char* gb = cur.gb + wv * 128;
  ca.set_tile(lane, (uint32_t)p.a_pitch, cur.a_valid);
  cb.set_tile(lane, (uint32_t)p.b_pitch, cur.b_valid);
  auto copy_a = [&](int slot) __attribute__((always_inline)) { ca.issue(lds_a + slot * C::A_BYTES, ga); ga += W * 128; };
  auto copy_b = [&](int slot) __attribute__((always_inline)) { cb.issue(lds_b + slot * C::B_BYTES, gb); gb += W * 128; };
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    if (s >= NB - NA) copy_a(s - (NB - NA));
    copy_b(s);
  }

  int sa = 0, sb = 0;   // slots of the step that comes next
  for (int done = 1;; ++done) {   // `done`: tiles up to and with this one
    f32x16 acc[NIB][NJB];
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ib][jb][r] = 0.0f;
    // One step: its copies have landed (stores of an epilogue in between only tighten the wait), its fragments go to
    // registers, and behind the first products its slots are filled again.
    auto step = [&](auto with_copies) __attribute__((always_inline)) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::YOUNGER) : "memory");
      const char* ta = ring + sa * C::A_BYTES;
      const char* tb = ring + NA * C::A_BYTES + sb * C::B_BYTES;
      bf16x8 fi[NIB][4], fj[NJB][4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int ib = 0; ib < NIB; ++ib) fi[ib][ks] = ring_frag<false, CI>(ta, lane, ib * 32, ks);
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) fj[jb][ks] = ring_frag<false, CJ>(tb, lane, jb * 32, ks);
      }
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      const uint32_t base_a = lds_a + sa * C::A_BYTES, base_b = lds_b + sb * C::B_BYTES;
      constexpr int MF = 4 * NIB * NJB;
      static_assert(MF >= C::CA + C::CB, "a copy behind each of the first products");
#pragma unroll
      for (int x = 0; x < MF; ++x) {
        const int ks = x / (NIB * NJB), ib = x / NJB % NIB, jb = x % NJB;
        acc[ib][jb] = mfma32(fj[jb][ks], fi[ib][ks], acc[ib][jb]);
        if (with_copies) {
          if (x < C::CA) ca.issue_piece(x, base_a, ga);
          else if (x < C::CA + C::CB) cb.issue_piece(x - C::CA, base_b, gb);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (with_copies) {
        ga += W * 128;
        gb += W * 128;
        sa = sa + 1 == NA ? 0 : sa + 1;
        sb = sb + 1 == NB ? 0 : sb + 1;
      }
    };
    for (int kt = NB; kt < mine; ++kt) step(std::true_type{});
    // The copies of B are at the next tile now.  There is none: they repeat this one's last step, which nothing reads.
    l += lstep;
    const GemmTile next = decode_gemm_tile<false, false, CI, CJ>(p, l);
    if (next.valid) {
      cb.set_tile(lane, (uint32_t)p.b_pitch, next.b_valid);
      gb = next.gb + wv * 128;
    } else {
      gb -= W * 128;
    }
#pragma unroll
    for (int s = 0; s < NB; ++s) {
      if (s == NB - NA) {   // and those of A
        if (next.valid) {
          ca.set_tile(lane, (uint32_t)p.a_pitch, next.a_valid);
          ga = next.ga + wv * 128;
        } else {
          ga -= W * 128;
        }
      }
      if (s == NB - 1) {
        step(std::false_type{});
      } else {
        step(std::true_type{});
        if (!next.valid) {
          gb -= W * 128;
          if (s >= NB - NA) ga -= W * 128;
        }
      }
    }

    // Partial sums through the slots that each wave has read last: [block of the round][quad q][lane] x 16 bytes, quad q of a
    // block four consecutive columns 8 q + 4 h of row n; wave w adds the quads q = w, in the order of the waves.
    auto block_at = [&](int k, int b) __attribute__((always_inline)) {   // block b of wave k
      const int last = done * ((nr - k + W - 1) / W) - 1;
      char* r = smem + k * C::RING_BYTES;
      return reinterpret_cast<float*>(b < NIB ? r + last % NA * C::A_BYTES + b * 4096
                                              : r + NA * C::A_BYTES + last % NB * C::B_BYTES + (b - NIB) * 4096) + lane * 4;
    };
#pragma unroll
    for (int r0 = 0; r0 < C::BLOCKS; r0 += C::PER_ROUND) {
#pragma unroll
      for (int b = r0; b < r0 + C::PER_ROUND && b < C::BLOCKS; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& a = acc[b / NJB][b % NJB];
          f32x4 v = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
          *reinterpret_cast<f32x4*>(block_at(wv, b - r0) + q * 256) = v;
        }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int b = r0; b < r0 + C::PER_ROUND && b < C::BLOCKS; ++b) {
        f32x4 sum = *reinterpret_cast<const f32x4*>(block_at(0, b - r0) + wv * 256);
#pragma unroll
        for (int k = 1; k < W; ++k) sum += *reinterpret_cast<const f32x4*>(block_at(k, b - r0) + wv * 256);
        const int il = b / NJB * 32 + n, j = b % NJB * 32 + 8 * wv + 4 * h;
        bf16x4 out = {(__bf16)sum[0], (__bf16)sum[1], (__bf16)sum[2], (__bf16)sum[3]};
        if (il < cur.i_valid && j < cur.j_valid) *reinterpret_cast<bf16x4*>(p.c + (cur.i0 + il) * p.c_pitch + cur.j0 + j) = out;
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // read by all: the next round, or the next copies
    }
    if (!next.valid) break;
    copy_a(sa);
    copy_b(sb);
    sa = sa + 1 == NA ? 0 : sa + 1;
    sb = sb + 1 == NB ? 0 : sb + 1;
    cur = next;
  }
  async_wait_all();
}

constexpr int64_t kMaxDim = (int64_t)1 << 22;   // rows stay below 8 MiB: 256 rows of byte offsets fit 32 bits

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

int check_dims(int64_t M, int64_t N, int64_t K) {
  if (M <= 0 || N <= 0 || K <= 0) return IE_ERR_SHAPE;
  if (M >= kMaxDim * 64 || N >= kMaxDim || K >= kMaxDim) return IE_ERR_SHAPE;
  return IE_OK;
}

// Tiles, grid and launch of one kernel: one workgroup per CU at most, the tiles dealt to the XCDs in eighths.
template <typename K>
int launch_tiles(K kernel, GemmParams p, int ti, int tj, int smem, hipStream_t st, int waves = kWaves) {
  int rc = set_smem(kernel, smem);
  if (rc) return rc;
  p.tiles_i = (int)ceil_div(p.I, ti);
  p.tiles_j = (int)ceil_div(p.J, tj);
  const int64_t tiles = (int64_t)p.tiles_i * p.tiles_j;
  if (tiles >= ((int64_t)1 << 28)) return IE_ERR_SHAPE;
  p.tiles = (int)tiles;
  hipError_t e;
  const int cus = cu_count(&e);
  if (e != hipSuccess) return hip_fail(e);
  const int per = (p.tiles + 7) / 8;                      // tiles of one XCD's share
  const int per_xcd_wgs = cus / 8 < per ? cus / 8 : per;  // one workgroup per CU
  const unsigned grid = 8u * (unsigned)(per_xcd_wgs < 1 ? 1 : per_xcd_wgs);
  kernel<<<dim3(grid), dim3(waves * 64), smem, st>>>(p);
  e = hipGetLastError();
  return e == hipSuccess ? IE_OK : hip_fail(e);
}

using Ring256x128 = RingCfg<256, 128, 4, 2, 1, 1, 3>;
using Ring128x256 = RingCfg<128, 256, 2, 4, 1, 1, 3>;
using Ring128 = RingCfg<128, 128, 2, 4, 1, 1, 4>;
using Ring64x128 = RingCfg<64, 128, 2, 4, 1, 1, 6>;
using Ring64 = RingCfg<64, 64, 1, 2, 4, 1, 6>;
using Ring32 = RingCfg<32, 32, 1, 1, 8, 4, 4>;

template <bool A_T, bool B_T, typename C>
int launch_ring(const GemmParams& p, hipStream_t st) {
  return launch_tiles(linear_ring_kernel<A_T, B_T, C>, p, C::CI, C::CJ, C::SMEM_BYTES, st);
}

template <typename C>
int launch_own(const GemmParams& p, hipStream_t st) {
  return launch_tiles(linear_own_kernel<C>, p, C::CI, C::CJ, C::SMEM_BYTES, st, C::WAVES);
}

template <bool A_T, bool B_T>
int launch_gemm(const GemmParams& p, hipStream_t st) {
  hipError_t e;
  const int cus = cu_count(&e);
  if (e != hipSuccess) return hip_fail(e);
  float us;
  const Tile tile = pick_tile(p.I, p.J, p.R, A_T ? 2 : B_T ? 1 : 0, cus, &us);
  if constexpr (!A_T && !B_T) {
    switch (pick_own(p.I, p.J, p.R, cus, us, kCost[tile].ti)) {
      case kOwn64: return launch_own<OwnCfg<64, 64, 2, 2>>(p, st);
      case kOwn64x96: return launch_own<OwnCfg<64, 96, 2, 2>>(p, st);
      case kOwn128x96: return launch_own<OwnCfg<128, 96, 1, 2>>(p, st);
      default: break;
    }
  }
  switch (tile) {
    case kRing256x128: return launch_ring<A_T, B_T, Ring256x128>(p, st);
    case kRing128x256: return launch_ring<A_T, B_T, Ring128x256>(p, st);
    case kRing128: return launch_ring<A_T, B_T, Ring128>(p, st);
    case kRing64x128: return launch_ring<A_T, B_T, Ring64x128>(p, st);
    case kRing64: return launch_ring<A_T, B_T, Ring64>(p, st);
    case kRing32:
      if constexpr (!A_T && !B_T) return launch_ring<A_T, B_T, Ring32>(p, st);
      [[fallthrough]];
    default: return launch_tiles(linear_pp_kernel<A_T, B_T>, p, TI, TJ, P_SMEM_BYTES, st);
  }
}

}  // namespace
}  // namespace ie

extern "C" {

int ie_linear_fwd(const void* x, const void* w, void* y, int64_t M, int64_t N, int64_t K, void* stream) {
  if (!x || !w || !y) return IE_ERR_NULL;
  if (int rc = ie::check_dims(M, N, K)) return rc;
  if (K % 64 != 0 || N % 8 != 0) return IE_ERR_UNSUPPORTED;   // contraction over K; rows of y are written 16 bytes at a time
  if (!ie::aligned16(x) || !ie::aligned16(w) || !ie::aligned16(y)) return IE_ERR_ALIGN;
  ie::GemmParams p{};
  p.a = static_cast<const char*>(x); p.b = static_cast<const char*>(w); p.c = static_cast<__bf16*>(y);
  p.I = M; p.J = N; p.R = K;
  p.a_pitch = K * 2; p.b_pitch = K * 2; p.c_pitch = N;
  return ie::launch_gemm<false, false>(p, static_cast<hipStream_t>(stream));
}

int ie_linear_bwd_input(const void* dy, const void* w, void* dx, int64_t M, int64_t N, int64_t K, void* stream) {
  if (!dy || !w || !dx) return IE_ERR_NULL;
  if (int rc = ie::check_dims(M, N, K)) return rc;
  if (N % 64 != 0 || K % 8 != 0) return IE_ERR_UNSUPPORTED;   // contraction over N
  if (!ie::aligned16(dy) || !ie::aligned16(w) || !ie::aligned16(dx)) return IE_ERR_ALIGN;
  ie::GemmParams p{};
  p.a = static_cast<const char*>(dy); p.b = static_cast<const char*>(w); p.c = static_cast<__bf16*>(dx);
  p.I = M; p.J = K; p.R = N;
  p.a_pitch = N * 2; p.b_pitch = K * 2; p.c_pitch = K;
  return ie::launch_gemm<false, true>(p, static_cast<hipStream_t>(stream));
}

int ie_linear_bwd_weight(const void* dy, const void* x, void* dw, int64_t M, int64_t N, int64_t K, void* stream) {
  if (!dy || !x || !dw) return IE_ERR_NULL;
  if (int rc = ie::check_dims(M, N, K)) return rc;
  if (M % 64 != 0 || N % 8 != 0 || K % 8 != 0) return IE_ERR_UNSUPPORTED;   // contraction over M
  if (!ie::aligned16(dy) || !ie::aligned16(x) || !ie::aligned16(dw)) return IE_ERR_ALIGN;
  ie::GemmParams p{};
  p.a = static_cast<const char*>(dy); p.b = static_cast<const char*>(x); p.c = static_cast<__bf16*>(dw);
  p.I = N; p.J = K; p.R = M;
  p.a_pitch = N * 2; p.b_pitch = K * 2; p.c_pitch = K;
  return ie::launch_gemm<true, true>(p, static_cast<hipStream_t>(stream));
}

}  // extern "C"
