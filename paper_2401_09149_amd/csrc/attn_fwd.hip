// Forward kernel: O = softmax(scale * Q K^T + mask) V and the per-row log-sum-exp, one
// workgroup per (batch, head, 128-query tile), streaming 64-key tiles of K and V through
// double-buffered LDS (fused attention of Sec. 2.1 / Sec. 4.2, recast for CDNA4).
//
// Each of the 4 wavefronts owns 32 query rows and keeps its Q fragments in registers.
// Scores are produced TRANSPOSED, S^T = K Q^T, so that one lane holds one query column:
// the row maximum and row sum are then reductions over the lane's own registers plus
// one half-wave swap, and the exponentiated scores are already in the B-operand layout
// of the second product O^T = V^T P^T, whose A operand (V^T) is gathered from the
// row-major V tile by LDS transpose loads.
#include <type_traits>

#include "attn_common.hpp"
#include "dispatch.hpp"
#include "launch.hpp"
#include "mfma_asm.hpp"
#include "tile_queue.hpp"

namespace ie {

// FLIP: items flip_lo .. flip_hi - 1 run in the opposite order, eight at a time (AttnParams; a kernel of its own, because the
// order costs a small launch 0.4 us, 4 %, before its first copy).
// LAZY (head dimension 64): unmasked blocks after a row's first look for no maximum (below).  It is held to 128 registers, for four
// workgroups to a CU; since tile coordinates and copy addresses are scalars it takes 125 and the other form 128 without being
// told to.  Both together, against three workgroups: 4 x 2000 x 16, 1024 items, 82.7 -> 77.0 us bidirectional, 49.7 -> 43.3 causal,
// 4 x 8192 x 16 1156 -> 1089 and 588 -> 554.
template <int D, bool FLIP, bool LAZY>
__global__ __launch_bounds__(kThreads, LAZY ? 4 : 2) void attn_fwd_kernel(AttnParams p) {
  constexpr int BM = 128, BN = 64;
  constexpr int NKS = D / 16;  // k-steps of the QK^T product
  constexpr int NDB = D / 32;  // 32-wide blocks of the head dimension in O^T
  constexpr int TILE_BYTES = BN * D * 2;
  constexpr int STAGE_BYTES = 2 * TILE_BYTES;  // K tile, then V tile
  constexpr int ROW_BYTES = D * 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];  // 2 stages
  __shared__ int scratch[8];

  const int tid = threadIdx.x, lane = tid & 63, wv = (int)uniform((uint32_t)tid >> 6);
  const int n = lane & 31, h = lane >> 5, grp = lane >> 4;

  int item = (int)blockIdx.x;
  if (FLIP && item >= p.flip_lo && item < p.flip_hi) item = p.flip_lo + (((p.flip_hi - p.flip_lo) >> 3) - 1 - ((item - p.flip_lo) >> 3)) * 8 + (item & 7);
  TileCoord tc = decode_tile<BM, kThreads, true>(p, p.Hq, true, scratch, item, tid);
  if (!tc.valid) return;
  const int g = tc.h / (p.Hq / p.Hkv);
  // Tile coordinates come through LDS where documents are packed, so the compiler takes them for per-lane values: as scalars
  // they leave the loop's copies no vector arithmetic (282 of 1902 VALU instructions of the kernel at head dimension 128; 2 x
  // 4096 x 32 282 -> 273 us, 3001 x 32, 4 per group, 85.2 -> 82.5, packed 16384 x 8 in 40 documents 64.8 -> 61.7).
  const int64_t q0 = uniform(tc.t0), doc_end = uniform(tc.doc_end);
  const int64_t q_end = (q0 + BM < doc_end) ? q0 + BM : doc_end;  // one past the tile's last row
  const int64_t k_begin = uniform(tc.doc_begin);
  const int64_t k_end = p.causal ? q_end : doc_end;
  const int nk = (int)(k_end - k_begin);  // visible keys of the tile (before the per-row causal cut)
  const int nkt = (nk + BN - 1) / BN;     // key tiles
  const int nfull = nk / BN;              // of which complete

  const int64_t q_stride = (int64_t)p.Hq * D;
  const int64_t kv_pitch = (int64_t)p.Hkv * D * 2;  // bytes between consecutive tokens of one kv head
  const char* qbase = reinterpret_cast<const char*>(p.q + tc.h * D) + tc.b * p.q_bstride;
  const char* kbase = uniform(reinterpret_cast<const char*>(p.k + g * D) + tc.b * p.kv_bstride);   // key tile kt starts at token k_begin + kt * BN
  const char* vbase = uniform(reinterpret_cast<const char*>(p.v + g * D) + tc.b * p.kv_bstride);
  auto key_tile_off = [&](const int kt) __attribute__((always_inline)) { return tok_off(p, k_begin + (int64_t)kt * BN, kv_pitch); };

  const uint32_t lds0 = lds_address(smem);
  AsyncTile<D> ld;
  ld.init(tid, kv_pitch);
  ld.load(lds0, kbase + key_tile_off(0), nk);
  ld.load(lds0 + TILE_BYTES, vbase + key_tile_off(0), nk);

  // This lane's query row (clamped into the tile so that out-of-range lanes repeat the last row).
  const int rows_rel_end = (int)(q_end - k_begin), wave_row_min = (int)(q0 - k_begin) + wv * 32;
  int row_rel = wave_row_min + n;  // position of the row among the document's keys
  if (row_rel >= rows_rel_end) row_rel = rows_rel_end - 1;
  const int lim0 = (p.causal ? row_rel : nk - 1) - 4 * h;  // last visible key relative to the lane's first key of tile 0

  // Q fragments: B operand of S^T = K Q^T, column n = query, k = head-dim index.
  bf16x8 qf[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8*>(qbase + tok_off(p, k_begin + row_rel, q_stride * 2) + (ks * 16 + h * 8) * 2);

  // Per-lane LDS addresses inside stage 0; stage, tile and row-block offsets are immediates.
  const char* k_ptr[NKS];  // K tile, A operand: row = key n (+32 for the second block), chunk = 2ks + h
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) k_ptr[ks] = smem + tile_off<D>(n, 2 * ks + h);
  // V tile, transpose loads: rows 4h..4h+3 (v_ptr0) and 8+4h.. (v_ptr8) of each 16-key group
  const char* v_ptr0[NDB];
  const char* v_ptr8[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    v_ptr0[db] = smem + TILE_BYTES + tr_off<D>(lane, 4 * (grp >> 1), 32 * db + 16 * (grp & 1));
    v_ptr8[db] = smem + TILE_BYTES + tr_off<D>(lane, 8 + 4 * (grp >> 1), 32 * db + 16 * (grp & 1));
  }

  const float c = p.scale_log2;
  // The running reference m only moves when a row maximum exceeds it by more than kSlack (in
  // log2 units): exponentials then stay below 2^kSlack, the final normalisation by l is exact
  // either way, and the accumulator is rescaled only a handful of times per row.
  constexpr float kSlack = 8.0f;
  const float slack_raw = kSlack / c;
  // At head dimension 64, where a block has half the MFMAs for the same elementwise work, unmasked blocks after a row's
  // first look for no maximum: their exponentials are taken against the reference as it is, and a block in which one lane's
  // 16 of them sum to more than this is done again with the true one.  Probabilities of up to 2^24 are as exact as others,
  // in fp32 and in bf16.  12 of 70 VALU instructions per block less: 8192 x 16 170 -> 161 us, 4 x 8192 x 16 bidirectional
  // 1212 -> 1165 (at head dimension 128 within 1 %).  The products then wait for the whole block's sum, which only other
  // waves hide: fwd64_is_lazy in dispatch.hpp says where there are enough of them.
  constexpr float kRedo = 16777216.0f;
  float m = -INFINITY;  // reference maximum, raw (unscaled) score units
  float l = 0.f;        // this lane's share of the row sum (its half of the keys)
  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;

  // One 64-key LDS tile is consumed as two 32-key blocks, each with its own softmax update.
  // `stage` is the byte offset of the stage holding tile kt; FULL_NEXT says that tile kt+1
  // exists and is complete (the common case, no per-lane address arithmetic).
  auto tile_step = [&](const int kt, const int stage, auto full_next) __attribute__((always_inline)) {
    const int kb = kt * BN;  // first key of the tile, relative to k_begin
    const uint32_t next_lds = lds0 + (STAGE_BYTES - stage);
    if (full_next) {
      ld.load_full(next_lds, kbase + key_tile_off(kt + 1));
      ld.load_full(next_lds + TILE_BYTES, vbase + key_tile_off(kt + 1));
    } else if (kt + 1 < nkt) {
      ld.load(next_lds, kbase + key_tile_off(kt + 1), nk - kb - BN);
      ld.load(next_lds + TILE_BYTES, vbase + key_tile_off(kt + 1), nk - kb - BN);
    }
    // Mask: only tiles that reach past the wave's first row (causal) or past the last key.
    const bool need_mask = (p.causal && kb + BN - 1 > wave_row_min) || (kb + BN > nk);
    const int lim = lim0 - kb;

#pragma unroll
    for (int j = 0; j < 2; ++j) {
      // S^T block: rows = keys kb + 32j .. +31, column = this lane's query
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        s = mfma32(lds_read8(k_ptr[ks], stage + 32 * j * ROW_BYTES), qf[ks], s);
      }
      // (the compiler counts the wait states behind a chain along one of the ways through the branches below, not the shortest)
      if (LAZY) asm volatile("s_nop 1" : "+v"(s));

      // V^T fragments of this block: requested now, consumed after the exponentials
      bf16x8 vfrag[2][NDB];
#pragma unroll
      for (int sblk = 0; sblk < 2; ++sblk)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          const int off = stage + (32 * j + 16 * sblk) * ROW_BYTES;
          vfrag[sblk][db] = cat4(lds_read_tr4(v_ptr0[db] + off), lds_read_tr4(v_ptr8[db] + off));
        }

      // The row maxima, and the reference where one outgrew it.
      auto move_reference = [&](const float limit) __attribute__((always_inline)) {
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        mx = halfwave_max(mx);
        if (__builtin_amdgcn_ballot_w64(mx > limit) == 0) return;
        const float m_new = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
      };
      bf16x8 pf[2];
      float block_sum = 0.f;
      float& sum = LAZY ? block_sum : l;
      auto exponentials = [&]() __attribute__((always_inline)) {
        const float mc = m * c;
        if (LAZY) sum = 0.f;
#pragma unroll
        for (int sblk = 0; sblk < 2; ++sblk) {
          bf16x2 pr[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * sblk + 2 * t], c, -mc));
            const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * sblk + 2 * t + 1], c, -mc));
            pr[t] = pack_bf16(e0, e1);
            sum += e0 + e1;  // fp32 sum of the unrounded exponentials: lse needs more than bf16 precision
          }
          pf[sblk] = cat_pairs(pr[0], pr[1], pr[2], pr[3]);
        }
      };
      if (need_mask) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * j + 8 * (r >> 2) + (r & 3) > lim) s[r] = -INFINITY;
      }
      const bool search = !LAZY || need_mask || (j == 0 && kt == 0);
      if (search) move_reference(m + slack_raw);
      exponentials();
      if (!search && __builtin_amdgcn_ballot_w64(!(sum <= kRedo)) != 0) {
        move_reference(m);
        exponentials();
      }
      if (LAZY) l += sum;
      // O^T += V^T P^T
#pragma unroll
      for (int sblk = 0; sblk < 2; ++sblk)
#pragma unroll
        for (int db = 0; db < NDB; ++db) oacc[db] = mfma32(vfrag[sblk][db], pf[sblk], oacc[db]);
    }
    async_wait_all();  // the copies of the next stage have landed ...
    __syncthreads();   // ... for every wave, and every wave is done reading this stage
  };

#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) consume(qf[ks]);
  async_wait_all();
  __syncthreads();
  int kt = 0;
  // steady state: two tiles per trip so that the stage offsets are compile-time constants
  for (; kt + 2 < nfull; kt += 2) {
    tile_step(kt, 0, std::true_type{});
    tile_step(kt + 1, STAGE_BYTES, std::true_type{});
  }
  for (; kt < nkt; ++kt) tile_step(kt, (kt & 1) * STAGE_BYTES, std::false_type{});

  // Epilogue: normalise, write O (bf16) and LSE (natural log).  (The lane is asked for again, so that neither its parts nor
  // its row stay in registers through the loop.)
  const int lane_e = lane_id(), h_e = lane_e >> 5;
  row_rel = wave_row_min + (lane_e & 31);
  const bool row_ok = row_rel < rows_rel_end;
  if (!row_ok) row_rel = rows_rel_end - 1;
  const int64_t row = k_begin + row_rel;
  const float l_full = halfwave_sum(l);
  const float inv_l = 1.0f / l_full;
  __bf16* orow = p.o_out + ((int64_t)tc.b * p.S * p.Hq + tc.h) * D + row * q_stride;
#pragma unroll
  for (int db = 0; db < NDB; ++db) store_block32_bf16(orow + 32 * db, oacc[db], inv_l, h_e, row_ok);
  if (row_ok && h_e == 0) p.lse_out[((int64_t)tc.b * p.Hq + tc.h) * p.S + row] = (m * c + __builtin_amdgcn_logf(l_full)) * kLn2;
}

// The same item (128 query rows, head dimension 128) for launches of a few items per CU, where a workgroup has its CU to
// itself for most of the time: one wave per SIMD, so MFMAs and everything else are interleaved instruction by instruction
// (mfma_asm.hpp).  Per 32-key block b a phase runs S(b + 1) and PV(b - 1), one MFMA of each at a time, and behind each MFMA
// one element of the softmax of block b; K rows of block b + 2 and V^T fragments of block b land in the registers that
// their predecessors have just left.  No running maximum: as in attn_fwd_wide.hip a block is done again, against its true
// maximum, when its sum outgrows 2^24.  64-key K/V tiles in a ring of four stages, one barrier per tile.
// Bound: the wave's one instruction stream; of all SIMDs' cycles at 8192 x 8, where the CUs are at work nine tenths of the time,
// MFMAs take 39 % and VALU issue 32 %, the rest goes to 1.5 LDS reads per MFMA, copies and waits.  Against the compiler-scheduled kernel with two workgroups to a CU: 8192 x 1 (no
// CU has two items) 144 -> 118 us, 8192 x 8 179 -> 154, 6000 x 8 116 -> 94, 2500 x 20 54 -> 46; with more than two items per CU
// their ways in and out, 8 us each, stand alone and it falls behind (3001 x 32 87 : 98; fwd128_route in dispatch.hpp).
struct FwdSeqCfg {
  static constexpr int D = 128, BM = 128, BN = 64, STAGES = 4;
  static constexpr int TILE_BYTES = BN * D * 2, STAGE_BYTES = 2 * TILE_BYTES;   // K tile, then V tile
  static constexpr int SMEM_BYTES = STAGES * STAGE_BYTES;
};
__global__ __launch_bounds__(kThreads, 1) void attn_fwd_seq_kernel(AttnParams p) {
  using C = FwdSeqCfg;
  constexpr int D = C::D, BM = C::BM, BN = C::BN, TILE_BYTES = C::TILE_BYTES, STAGE_BYTES = C::STAGE_BYTES, ROW_BYTES = D * 2;
  constexpr int NKS = D / 16, NDB = D / 32;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int scratch[8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 31, h = lane >> 5, grp = lane >> 4;

  TileCoord tc = decode_tile<BM>(p, p.Hq, true, scratch, blockIdx.x, tid);
  if (!tc.valid) return;
  const int g = tc.h / (p.Hq / p.Hkv);
  const int64_t q0 = uniform(tc.t0), doc_end = uniform(tc.doc_end);
  const int64_t q_end = (q0 + BM < doc_end) ? q0 + BM : doc_end;
  const int64_t k_begin = uniform(tc.doc_begin);
  const int64_t k_end = p.causal ? q_end : doc_end;
  const int nk = (int)(k_end - k_begin);
  const int nkt = (nk + BN - 1) / BN;

  const int64_t q_stride = (int64_t)p.Hq * D;
  const int64_t kv_pitch = (int64_t)p.Hkv * D * 2;
  const char* qbase = reinterpret_cast<const char*>(p.q + tc.h * D) + tc.b * p.q_bstride;
  const char* kbase = uniform(reinterpret_cast<const char*>(p.k + g * D) + tc.b * p.kv_bstride);
  const char* vbase = uniform(reinterpret_cast<const char*>(p.v + g * D) + tc.b * p.kv_bstride);
  const uint32_t lds0 = lds_address(smem);
  AsyncTile<D> ld;
  ld.init(tid, kv_pitch);
  // Tile T's copy: eight instructions per wave, all at once (any number of valid rows) or one by one (a whole tile).
  static_assert(2 * AsyncTile<D>::NI == NKS, "one piece per slot of a phase");
  struct Copy { const char* k; const char* v; uint32_t lds; };
  auto describe = [&](const int T) __attribute__((always_inline)) {
    const int64_t off = tok_off(p, k_begin + (int64_t)T * BN, kv_pitch);
    return Copy{kbase + off, vbase + off, lds0 + (uint32_t)(T % C::STAGES) * STAGE_BYTES};
  };
  auto copy_all = [&](const int T) __attribute__((always_inline)) {
    const Copy c = describe(T);
    ld.load(c.lds, c.k, nk - T * BN);
    ld.load(c.lds + TILE_BYTES, c.v, nk - T * BN);
  };
  for (int T = 0; T < C::STAGES - 1 && T < nkt; ++T) copy_all(T);

  const int rows_rel_end = (int)(q_end - k_begin);
  const int row_rel_raw = (int)(q0 - k_begin) + wv * 32 + n;
  const int row_rel = row_rel_raw < rows_rel_end ? row_rel_raw : rows_rel_end - 1;
  const int64_t row = k_begin + row_rel;
  bf16x8 qf[NKS];   // live in AGPRs
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) qf[ks] = global_load_to_agpr(qbase + tok_off(p, row, q_stride * 2) + (ks * 16 + h * 8) * 2);

  const char* k_ptr[NKS];   // row n of a K tile, chunk 2ks + h
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) k_ptr[ks] = smem + tile_off<D>(n, 2 * ks + h);
  const char* v_ptr0[NDB];  // transpose loads on the V tile
  const char* v_ptr8[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    v_ptr0[db] = smem + TILE_BYTES + tr_off<D>(lane, 4 * (grp >> 1), 32 * db + 16 * (grp & 1));
    v_ptr8[db] = smem + TILE_BYTES + tr_off<D>(lane, 8 + 4 * (grp >> 1), 32 * db + 16 * (grp & 1));
  }
  const float c = p.scale_log2;
  constexpr float kRedo = 16777216.0f;
  float m = -INFINITY, negmc = INFINITY, l = 0.f;   // reference maximum (raw units), -m * c, this lane's share of the row sum
  f32x16 o[NDB];   // live in AGPRs
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  bf16x8 kf[NKS];        // rows of the block whose scores come next
  bf16x8 vt[2][NDB];     // V^T fragments of the block whose PV product comes next (zeros: there is none yet)
  bf16x8 pf[2];          // its probabilities
  f32x16 s[2];           // by block parity
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int t = 0; t < 8; ++t) pf[i][t] = (__bf16)0.f;
    // (opaque: known to be zeros, they would be written in front of the MFMAs that read them, without the wait states)
    asm volatile("" : "+v"(pf[i]));
#pragma unroll
    for (int db = 0; db < NDB; ++db) { vt[i][db] = pf[i]; asm volatile("" : "+v"(vt[i][db])); }
  }
  agpr_loads_wait();   // Q and the first tiles
  __syncthreads();

  // A block is done again: its true maximum becomes the reference, what has been summed so far is rescaled.
  auto redo = [&](f32x16& sx, uint32_t (&pw)[8], float& lsum, const bool masked, const int lim) __attribute__((always_inline)) {
    if (masked) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) > lim) sx[r] = -INFINITY;
    }
    float mx = sx[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sx[r]);
    mx = halfwave_max(mx);
    mfma_result_fence();
    const float m_new = fmaxf(m, mx);
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
    m = m_new;
    negmc = -m_new * c;
    l *= alpha;
    // (element by element through one VGPR, in assembly: left to the compiler, the accumulators leave the AGPRs)
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float tmp;
        asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\ts_nop 0\n\tv_accvgpr_write_b32 %0, %1"
                     : "+a"(o[db][r]), "=&v"(tmp)
                     : "v"(alpha));
      }
    mfma_result_fence();
    lsum = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sx[2 * t], c, negmc));
      const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sx[2 * t + 1], c, negmc));
      pw[t] = __builtin_bit_cast(uint32_t, pack_bf16(e0, e1));
      lsum += e0 + e1;
    }
  };
  // One phase: block `PAR` of the current tile, at LDS byte offset `cur`; `next`: the following tile's.
  auto phase = [&](auto par_c, auto masked_c, auto last_c, const int cur, const int next, const bool copying, const Copy& cp,
                   const int lim) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par_c)::value;
    constexpr bool MASKED = decltype(masked_c)::value, LAST = decltype(last_c)::value;
    constexpr bool HAS_S = !(LAST && PAR == 1);
    constexpr int BLK = 32 * ROW_BYTES;
    uint32_t pw[8];
    float pr[16], lsum = 0.f;
    auto elem = [&](int e) __attribute__((always_inline)) {
      if (MASKED) {
        softmax_elem_masked(pr[e], s[PAR][e], c, negmc, 8 * (e >> 2) + (e & 3), lim);
        if (e >= 3 && (e & 1)) sum_pack_pair(lsum, pw[e / 2 - 1], pr[e - 3], pr[e - 2]);
      }
      else if (e < 2) exp_elem(pr[e], s[PAR][e], c, negmc);
      else if (e == 2) exp_elem_first_sum(pr[2], s[PAR][2], c, negmc, lsum, pr[0], pr[1], pw[0]);
      else if (e & 1) exp_elem_add(pr[e], s[PAR][e], c, negmc, lsum, pr[e - 1]);
      else exp_elem_add_pack(pr[e], s[PAR][e], c, negmc, lsum, pr[e - 1], pw[e / 2 - 1], pr[e - 2]);
    };
    if (MASKED) asm volatile("" : "+v"(lsum));   // (opaque, as above)
#pragma unroll
    for (int mm = 0; mm < NKS; ++mm) {
      if (HAS_S) {
        if (mm == 0) mfma_first_b_agpr(s[PAR ^ 1], kf[0], qf[0]);
        else mfma_next_b_agpr(s[PAR ^ 1], kf[mm], qf[mm]);
      }
      if (!LAST) kf[mm] = lds_read8(k_ptr[mm] + next, PAR * BLK);
      elem(2 * mm);
      asm_fence();
      mfma_acc_agpr(o[mm % NDB], vt[mm / NDB][mm % NDB], pf[mm / NDB]);
      {
        const int off = PAR * BLK + 16 * (mm / NDB) * ROW_BYTES;
        vt[mm / NDB][mm % NDB] = cat4(lds_read_tr4(v_ptr0[mm % NDB] + cur + off), lds_read_tr4(v_ptr8[mm % NDB] + cur + off));
      }
      elem(2 * mm + 1);
      if (PAR == 0 && copying) {
        constexpr int NI = AsyncTile<D>::NI;
        ld.load_full_piece(cp.lds + (mm / NI) * TILE_BYTES, mm / NI ? cp.v : cp.k, mm % NI);
      }
      asm_fence();
    }
    asm volatile("s_nop 0");   // (element 15's exponential is the previous instruction but for copies)
    if (MASKED) sum_pack_pair(lsum, pw[7], pr[14], pr[15]);
    else add_pack(lsum, pr[15], pw[7], pr[14]);
    if (__builtin_amdgcn_ballot_w64(sum_beyond(lsum, kRedo)) != 0) redo(s[PAR], pw, lsum, MASKED, lim);
    l += lsum;
    pf[0] = frag_from_words(pw[0], pw[1], pw[2], pw[3]);
    pf[1] = frag_from_words(pw[4], pw[5], pw[6], pw[7]);
    asm_fence();
  };
  auto tile = [&](const int T, auto masked_c, auto last_c) __attribute__((always_inline)) {
    if (T > 0) {
      // Tile T + 1 has landed (all but the eight copies of tile T + 2), and everyone has read what tile T + 3 replaces.
      if (T + 2 < nkt) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    const int T3 = T + C::STAGES - 1;
    const bool spread = (T3 + 1) * BN <= nk;
    Copy cp{};
    if (spread) cp = describe(T3);
    else if (T3 < nkt) copy_all(T3);
    const int cur = (T % C::STAGES) * STAGE_BYTES, next = ((T + 1) % C::STAGES) * STAGE_BYTES;
    const int lim = (p.causal ? row_rel : nk - 1) - T * BN - 4 * h;   // last visible key relative to the lane's first key
    phase(std::integral_constant<int, 0>{}, masked_c, last_c, cur, next, spread, cp, lim);
    phase(std::integral_constant<int, 1>{}, masked_c, last_c, cur, next, false, cp, lim - 32);
  };

  // S(0), with the rows of block 1 read behind it
#pragma unroll
  for (int mm = 0; mm < NKS; ++mm) kf[mm] = lds_read8(k_ptr[mm], 0);
  asm_fence();
#pragma unroll
  for (int mm = 0; mm < NKS; ++mm) {
    if (mm == 0) mfma_first_b_agpr(s[0], kf[0], qf[0]);
    else mfma_next_b_agpr(s[0], kf[mm], qf[mm]);
    kf[mm] = lds_read8(k_ptr[mm], 32 * ROW_BYTES);
    asm_fence();
  }
  mfma_result_fence();
  int T = 0;
  const int first_masked = p.causal ? (int)(q0 - k_begin) / BN : nk / BN;   // tiles before it are visible to all rows
  for (; T < first_masked && T + 1 < nkt; ++T) tile(T, std::false_type{}, std::false_type{});
  for (; T + 1 < nkt; ++T) tile(T, std::true_type{}, std::false_type{});
  tile(T, std::true_type{}, std::true_type{});
#pragma unroll
  for (int mm = 0; mm < NKS; ++mm) mfma_acc_agpr(o[mm % NDB], vt[mm / NDB][mm % NDB], pf[mm / NDB]);
  mfma_results_ready(o);

  // Epilogue: normalise, write O (bf16) and LSE (natural log).
  const bool row_ok = row_rel_raw < rows_rel_end;
  const float l_full = halfwave_sum(l);
  const float inv_l = 1.0f / l_full;
  __bf16* orow = p.o_out + ((int64_t)tc.b * p.S * p.Hq + tc.h) * D + (k_begin + row_rel) * q_stride;
#pragma unroll
  for (int db = 0; db < NDB; ++db) store_block32_bf16(orow + 32 * db, o[db], inv_l, h, row_ok);
  if (row_ok && h == 0) p.lse_out[((int64_t)tc.b * p.Hq + tc.h) * p.S + k_begin + row_rel] = (m * c + __builtin_amdgcn_logf(l_full)) * kLn2;
}

template <int D, bool SEQ, bool FLIP, bool LAZY>
static int launch_fwd_d(AttnParams p, int cus, hipStream_t st) {
  constexpr int smem = SEQ ? FwdSeqCfg::SMEM_BYTES : 2 * 2 * 64 * D * 2;   // (two stages of a K and a V tile)
  const int64_t tiles = tiles_per_head(p.S, 128, p.cu, p.num_docs);
  const int64_t grid = tiles * p.B * p.Hq;
  if (grid >= ((int64_t)1 << 31)) return kErrShape;
  p.tiles = (int32_t)tiles;
  p.q_heavy = fwd_head_by_head(tiles, grid, p.causal != 0, p.cu != nullptr, D == 64, cus, p.B * p.Hq % 8 != 0, p.Hq / p.Hkv,
                               (int64_t)p.B * p.S * p.Hkv * D * 4, p.S - (tiles - 1) * 128);
  static KernelSetup setup;
  int per_cu = 1;
  if constexpr (SEQ) {
    int rc = kernel_setup(setup, attn_fwd_seq_kernel, smem, &per_cu);
    if (rc) return rc;
    attn_fwd_seq_kernel<<<dim3((unsigned)grid), dim3(kThreads), smem, st>>>(p);
  } else {
    int rc = kernel_setup(setup, attn_fwd_kernel<D, FLIP, LAZY>, smem, &per_cu);
    if (rc) return rc;
    // The second item on each CU goes by the opposite order (fwd_flips in dispatch.hpp).
    if (FLIP) {
      p.flip_lo = cus & ~7;
      p.flip_hi = (int32_t)(grid < 2 * p.flip_lo ? grid & ~(int64_t)7 : 2 * p.flip_lo);
    }
    attn_fwd_kernel<D, FLIP, LAZY><<<dim3((unsigned)grid), dim3(kThreads), smem, st>>>(p);
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : hip_fail(e);
}

template <int D>
static int launch_fwd_narrow(AttnParams p, int cus, hipStream_t st) {
  const int64_t tiles = tiles_per_head(p.S, 128, p.cu, p.num_docs), items = tiles * p.B * p.Hq;
  const bool flip = fwd_flips(items, tiles, p.causal != 0, p.cu != nullptr, cus);
  if constexpr (D == 64) {
    if (fwd64_is_lazy(items, p.causal != 0, p.cu != nullptr, cus, p.cu ? p.S / 128 / (p.num_docs > 0 ? p.num_docs : 1) : tiles))
      return flip ? launch_fwd_d<D, false, true, true>(p, cus, st) : launch_fwd_d<D, false, false, true>(p, cus, st);
  }
  return flip ? launch_fwd_d<D, false, true, false>(p, cus, st) : launch_fwd_d<D, false, false, false>(p, cus, st);
}

int launch_fwd(AttnParams p, int D, hipStream_t st) {
  hipError_t e;
  const int cus = cu_count(&e);
  if (e != hipSuccess) return hip_fail(e);
  if (D == 64) return launch_fwd_narrow<64>(p, cus, st);
  const bool narrow = fwd_prefers_128_rows(ceil_div(p.S, 256) * p.B * p.Hq, p.S, p.cu != nullptr);
  Fwd128 route = narrow ? Fwd128::kNarrow : Fwd128::kWide;
  if (tile_rows_setting.load(std::memory_order_relaxed) == 0)   // (not the caller's choice)
    route = fwd128_route(p.B, p.S, p.Hq, p.causal != 0, p.num_docs, cus, narrow);
  if (route == Fwd128::kWide) {
    const int rc = launch_fwd_wide(p, st);
    if (rc != kErrBusy || !narrow) return rc;   // (what sizes alone give to 128-row items runs without a queue if none is free)
    route = Fwd128::kNarrow;
  }
  return route == Fwd128::kSeq ? launch_fwd_d<128, true, false, false>(p, cus, st) : launch_fwd_narrow<128>(p, cus, st);
}

}  // namespace ie
