// gfx950 (MI355X, CDNA4) kernels for the gradients of tile-sparse 3D attention.
//
// What is computed: the forward pass (Sec. 3.3 of Efficient-vDiT) gives query
// token s the output out_s = sum_t P_st v_t, P_st = softmax over the keys t of the
// frames its frame keeps of scale * <q_s, k_t>. With the upstream gradient dO, the
// forward's row log-sum-exp lse_s and delta_s = <dO_s, out_s>, the chain rule
// through the softmax gives, over kept (s, t) pairs only:
//   P_st = exp(scale <q_s, k_t> - lse_s),  dP_st = <dO_s, v_t>,
//   dS_st = P_st (dP_st - delta_s),
//   dq_s = scale sum_t dS_st k_t,  dk_t = scale sum_s dS_st q_s,  dv_t = sum_s P_st dO_s.
// Stage 3 of the method (Sec. 3.4) trains the sparse model through this; dropped
// tiles are never read here either.
//
// Passes (all on the caller's stream)
//   prep  lse in base 2 and -delta per query row (both gradient kernels start
//         their dP accumulations at -delta, so dP - delta takes no vector op).
//   dq    one workgroup per 128 query rows of a query frame (or of the text with a
//         prefix, see Layout), over the kept key
//         tiles (the forward's work list): S^T = K Q^T, dP^T = V dO^T,
//         dQ^T += K^T dS^T. Each lane owns one query of its wave's 32-query
//         column block, so lse and -delta are per-lane constants.
//   dkdv  one workgroup per 128 key rows of a key frame, over the query tiles of
//         the frames that keep it (the work list of the transposed mask):
//         S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS. Each lane owns
//         one key of its wave's 32-key column block.
//         At d = 128 large calls of long units run it with one wave per SIMD
//         (dkdv_roll_unit).
//   sum   adds the fp32 partials of frames the work plan split into pieces.
// Small calls run dq and dk/dv in one launch (bwd_all_kernel).
// dq is recomputed in its own pass instead of being accumulated from the key side:
// fp32 atomics from every (key block, query block) pair would move several TB/s
// through L2 at this shape, more than recomputing S and dP costs on the matrix cores.
//
// Both gradient kernels keep one operand of every product in registers (the
// wave's 32 queries or 32 keys) and stream the other through LDS (see kRowsPerWg
// below for why not 64 as in the forward kernel).
//
// LDS layout: every staged tile is read both row-wise (16 bytes per lane, 16
// consecutive rows per access) and transposed (ds_read_b64_tr_b16: 4 consecutive
// rows x 64 bytes per half-wave access), so one XOR swizzle dsw(r) of the 16-byte
// pieces serves both: over 16 consecutive rows it spreads one piece column over
// all 64 banks, and over 4 consecutive rows (starting at a multiple of 4) it puts
// the rows' 64-byte quads in different bank groups.
#include <hip/hip_runtime.h>

#include <type_traits>

#include <float.h>
#include <stdint.h>

#include <algorithm>

#include "launch.h"
#include "tile_common.h"
#include "unit_order.h"

namespace ta {
namespace {

constexpr int kBwdWaves = 4;
constexpr int kBwdThreads = 64 * kBwdWaves;
// Each wave owns one 32-row column block (32 queries in the dq pass, 32 keys in
// the dk/dv pass). That keeps every operand, accumulator and score in 256 VGPRs,
// so two workgroups share a CU and one wave's softmax-gradient arithmetic overlaps
// the other's matrix instructions. Measured at the 93-frame shape this beats 64
// rows per wave at one workgroup per CU (which halves the LDS fragment reads per
// MFMA but puts the accumulators in AGPRs, copies the scores out of them and
// serialises the vector work) by 17% (dq) and 12% (dk/dv). Both passes at d = 128 as well
// own 32 rows per wave; large calls of long units run the dk/dv pass with one wave per
// SIMD there.
constexpr int kRowsPerWg = kBwdWaves * 32;

// What one pass of the key side produces. At d = 128 dK and dV together do not fit 256
// VGPRs (their accumulators, K and V operands alone take 192): in the shared launch of
// small calls, whose kernel runs at two workgroups per CU, the key side is two passes
// there (dV: S and P only; dK: S, dP and dS) that form S twice; larger calls
// of long units (kMinRollBlocks) run dkdv_roll_unit.
enum KeyPass { kDkDv = 0, kDvOnly = 1, kDkOnly = 2 };
template <int D>
constexpr bool split_key_pass() { return D == 128; }

// Calls of at most this many rounds of resident workgroups run every pass in one launch
// (see bwd_all_kernel). At d = 128 the shared launch forms S twice on the key side, which
// the kernel of its own does not (see dkdv_roll_unit): they meet at 3 to 4 rounds (H = 4,
// 10 x 700 tokens, col g = 1, 2 rounds: 104 us in one launch, 118 in two; H = 8, g = 2:
// 235 and 233; H = 16: 447 and 430; H = 24, 12 x 900, sym: 2.11 and 1.87 ms).
template <int D>
constexpr uint32_t merge_rounds() { return D == 128 ? 3 : 48; }

// Calls at d = 128 whose key-side units walk fewer 32-query blocks than this on average stay in
// the shared launch however many rounds they are: dkdv_roll_unit, alone on its compute unit,
// hides nothing of a unit's start (five blocks loaded ahead) and end. Measured (shared launch
// and dkdv_roll_unit, same process): 2 x 37 heads of 47 x 37, col, 3, 9 and 17 blocks: 210
// and 257 us, 317 and 380, 447 and 513; 2 x 20 heads of 40 x 128, 15 and 31: 343 and 378, 497
// and 498; 40 x 100, 35: 476 and 477; 24 heads of 24 x 512, 31 and 46: 677 and 678, 929 and 877;
// 12 heads of 40 x 200, 34: 300 and 286.
constexpr int kMinRollBlocks = 32;

template <int D>
struct BShape {
  static constexpr int kChunks = D / 16;
  static constexpr int kDBlocks = D / 32;
  static constexpr int kPieces = D / 8;
  static constexpr int kTileElems = kBlockK * D;
  static constexpr int kLoadsPerWave = kBlockK * kPieces / 64 / kBwdWaves;
  static_assert(kBlockK * kPieces == 64 * kBwdWaves * kLoadsPerWave, "whole loads per wave");
};

template <int D>
__device__ __forceinline__ int dsw(int r) {
  if constexpr (D == 64) return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
  else if constexpr (D == 96) return (r >> 2) & 3;
  else return ((r & 3) << 2) | ((r >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int d_slot(int r, int p) { return (r * (D / 8) + (p ^ dsw<D>(r))) * 8; }

// Direct global -> LDS loads of one 64-row tile in the dsw layout (see the
// forward kernel's TileLoader: the XOR only permutes pieces inside a row, and one
// load covers whole rows or aligned quads, so it reads contiguous memory).
template <int D>
struct DualLoader {
  int off[BShape<D>::kLoadsPerWave];
  __device__ __forceinline__ void init(int wave, int lane) {
#pragma unroll
    for (int j = 0; j < BShape<D>::kLoadsPerWave; ++j) {
      const int q = 64 * (wave + kBwdWaves * j) + lane;
      const int r = q / BShape<D>::kPieces, ps = q % BShape<D>::kPieces;
      off[j] = (r * D + 8 * (ps ^ dsw<D>(r))) * 2;
    }
  }
  __device__ __forceinline__ void load(const uint16_t* Xh, size_t row0, int nvalid,
                                       const uint16_t* lds, int wave) const {
    const i32x4 rs = buffer_words(Xh + row0 * D, (uint32_t)(nvalid * D * 2));
    const uint32_t base = lds_addr(lds);
#pragma unroll
    for (int j = 0; j < BShape<D>::kLoadsPerWave; ++j)
      load_to_lds(rs, __builtin_amdgcn_readfirstlane(base + 1024u * (uint32_t)(wave + kBwdWaves * j)),
                  off[j]);
  }
};

// Row-wise fragment offsets (A operand, rows = tile rows): lane (n, h) reads row
// n of a 32-row block, piece 2 cc + h of chunk cc. Row block rb adds rb * 32 * D
// (the swizzle depends only on the low 4 bits of the row).
template <int D>
struct RowAddr {
  // At d = 96 the swizzle only permutes the low two bits of the piece index, so
  // chunks cc and cc + 2 sit 4 pieces apart.
  static constexpr int kN = D == 96 ? 2 : D / 16;
  int at[kN];
  __device__ __forceinline__ void init(int n, int hf) {
#pragma unroll
    for (int cc = 0; cc < kN; ++cc) at[cc] = d_slot<D>(n, 2 * cc + hf);
  }
  __device__ __forceinline__ int get(int cc) const {
    if constexpr (D == 96) return at[cc & 1] + 32 * (cc >> 1);
    else return at[cc];
  }
};

// Transposed fragment offsets (A operand, rows = d, contraction over tile rows):
// lane l (group g = l/16, j = l%16) reads row 4(g/2) + j/4 (lo) and that row + 8
// (hi), d = 32 mb + 16(g%2) + 4(j%4) .. +3. Chunk ch (16 rows) adds 16 ch * D.
template <int D>
struct TrAddr {
  // At d = 96 the swizzle leaves the quad index 4 mb of a piece alone: d-block mb
  // sits 32 mb elements further.
  static constexpr int kN = D == 96 ? 1 : D / 32;
  int lo[kN], hi[kN];
  __device__ __forceinline__ void init(int lane) {
    const int g = lane >> 4, j = lane & 15;
    const int r = 4 * (g >> 1) + (j >> 2);
#pragma unroll
    for (int mb = 0; mb < kN; ++mb) {
      const int p = 4 * mb + 2 * (g & 1) + ((j >> 1) & 1);
      lo[mb] = d_slot<D>(r, p) + 4 * (j & 1);
      hi[mb] = d_slot<D>(r + 8, p) + 4 * (j & 1);
    }
  }
  __device__ __forceinline__ int get_lo(int mb) const { return D == 96 ? lo[0] + 32 * mb : lo[mb]; }
  __device__ __forceinline__ int get_hi(int mb) const { return D == 96 ? hi[0] + 32 * mb : hi[mb]; }
};

template <int D>
__device__ __forceinline__ bf16x8 row_frag(const uint16_t* tile, const RowAddr<D>& ra, int rb, int cc) {
  return as_bf16x8(load16(tile + rb * 32 * D + ra.get(cc)));
}

// 32 d-rows x 16 tile rows: the contraction index k of lane half h maps to tile
// rows 16 ch + 4h + (0..3) and 16 ch + 8 + 4h + (0..3), the order in which a C
// fragment's entries 8c2 .. 8c2+7 hold their rows.
template <int D>
__device__ __forceinline__ bf16x8 tr_frag(const uint16_t* tile, const TrAddr<D>& ta, int mb, int ch) {
  const uint16_t* p = tile + 16 * ch * D;
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + ta.get_lo(mb)));
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + ta.get_hi(mb)));
  const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
  return as_bf16x8(u32x4{a[0], a[1], b[0], b[1]});
}

// B-operand slices of this lane's row (query or key) of a tensor: d = 16 cc + 8h .. +7.
template <int D>
__device__ __forceinline__ void load_row_operand(const uint16_t* row, bool valid, uint32_t keep,
                                                 uint32_t flip, int hf, bf16x8 (&x)[D / 16]) {
#pragma unroll
  for (int cc = 0; cc < D / 16; ++cc) {
    u32x4 w = {0u, 0u, 0u, 0u};
    if (valid) w = (load16(row + 16 * cc + 8 * hf) & keep) ^ flip;
    x[cc] = as_bf16x8(w);
  }
}

// Stores 16 d-values of this lane's row from a transposed accumulator block
// (entry 4i + j holds d = 32 mb + 8i + 4h + j), times s, as bf16 or fp32.
template <int D>
__device__ __forceinline__ void store_row_bf16(uint16_t* row, const f32x16 (&acc)[D / 32], float s, int hf) {
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 x = {acc[mb][4 * i] * s, acc[mb][4 * i + 1] * s, acc[mb][4 * i + 2] * s,
                       acc[mb][4 * i + 3] * s};
      const bf16x4 y = __builtin_convertvector(x, bf16x4);
      *reinterpret_cast<u32x2*>(row + 32 * mb + 8 * i + 4 * hf) = __builtin_bit_cast(u32x2, y);
    }
}
template <int D>
__device__ __forceinline__ void store_row_f32(float* row, const f32x16 (&acc)[D / 32], float s, int hf) {
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 x = {acc[mb][4 * i] * s, acc[mb][4 * i + 1] * s, acc[mb][4 * i + 2] * s,
                       acc[mb][4 * i + 3] * s};
      *reinterpret_cast<f32x4*>(row + 32 * mb + 8 * i + 4 * hf) = x;
    }
}

// ---------------------------------------------------------------------------
// prep: lse2 = lse * log2(e), ndelta = -<dO, out> (fp32 sum of bf16 products).
// One workgroup per 64 rows: the 256 threads read the rows' 16-byte pieces
// contiguously (coalesced), leave per-piece partial dots in LDS, and 64 threads
// add up one row each.
constexpr int kPrepRows = 64;

template <int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const uint16_t* __restrict__ out,
                                                       const uint16_t* __restrict__ dout,
                                                       const float* __restrict__ lse,
                                                       float* __restrict__ lse2,
                                                       float* __restrict__ ndelta, int64_t rows) {
  constexpr int kPieces = D / 8;
  constexpr int kPerThread = kPrepRows * kPieces / 256;
  static_assert(kPrepRows * kPieces == 256 * kPerThread, "whole pieces per thread");
  __shared__ float part[kPrepRows * kPieces];
  const int64_t row0 = (int64_t)blockIdx.x * kPrepRows;
  const int64_t n_rows = rows - row0 < kPrepRows ? rows - row0 : kPrepRows;
  const int64_t base = row0 * D;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int piece = threadIdx.x + 256 * j;  // piece / kPieces = row within the block
    float acc = 0.f;
    if (piece < n_rows * kPieces) {
      const bf16x8 x = as_bf16x8(load16(out + base + 8 * piece));
      const bf16x8 y = as_bf16x8(load16(dout + base + 8 * piece));
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = __builtin_fmaf((float)x[e], (float)y[e], acc);
    }
    part[piece] = acc;
  }
  __syncthreads();
  if (threadIdx.x < n_rows) {
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < kPieces; ++c) acc += part[threadIdx.x * kPieces + c];
    const int64_t r = row0 + threadIdx.x;
    ndelta[r] = -acc;
    lse2[r] = lse[r] * 1.4426950408889634f;
  }
}

// ---------------------------------------------------------------------------
// P = exp2(c s - lse2) clamped to [0, 1] (the clamp folds into the exponential's
// output modifier). For kept keys the exponent is <= 0 up to rounding, so the clamp
// changes nothing but rounding; it keeps P finite for the rows and keys past a
// tile's valid range, whose zero-filled operands then contribute exactly nothing
// (see the kernels), so no tile needs a mask.
__device__ __forceinline__ float prob(float s, float c, float lse2) {
  return __builtin_amdgcn_fmed3f(fast_exp2(__builtin_fmaf(s, c, -lse2)), 0.f, 1.f);
}

// fn(integral_constant<int, i>) for i = 0 .. N-1, in order.
template <int N, int I = 0, typename Fn>
__device__ __forceinline__ void static_for(Fn&& fn) {
  if constexpr (I < N) {
    fn(std::integral_constant<int, I>{});
    static_for<N, I + 1>(static_cast<Fn&&>(fn));
  }
}

// ---------------------------------------------------------------------------
// dq pass.
//
// dS^T of one 32-key block for one column block, as the B operand of
// dQ^T += K^T dS^T: entries 8c2 .. 8c2+7 of the C fragment. dp already holds
// dP - delta (its accumulation started at -delta).
__device__ __forceinline__ void dq_scores(const f32x16& s, const f32x16& dp, float c, float lse2,
                                          bf16x8 (&ds)[2]) {
#pragma unroll
  for (int c2 = 0; c2 < 2; ++c2) {
    f32x8 x;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p = prob(s[8 * c2 + e], c, lse2);
      x[e] = p * dp[8 * c2 + e];
    }
    ds[c2] = __builtin_convertvector(x, bf16x8);
  }
}

// The query-side pass over one work unit (b, item, query block).
template <int D, bool PREFIX>
__device__ __forceinline__ void dq_unit(const BwdArgs& a, int nqb, uint32_t work,
                                        uint16_t (&sK)[2][BShape<D>::kTileElems],
                                        uint16_t (&sV)[2][BShape<D>::kTileElems]) {
  using Sh = BShape<D>;
  const uint32_t per_b = (uint32_t)a.n_items_q * (uint32_t)nqb;
  const uint32_t b = work / per_b;
  const uint32_t rem = work - b * per_b;
  const int32_t* item = a.items_q + 5 * (rem / nqb);
  const uint32_t bh = b * (uint32_t)a.H + (uint32_t)item[0];
  const int frame = item[1], kbeg = item[2], n_kept = item[3], slot = item[4];
  const int qb = (int)(rem % nqb);
  const int T = a.T;
  const Layout<PREFIX> lay{a.F, T, a.P};
  const int seg0 = lay.start(frame), seg_len = lay.len(frame);
  // With a prefix the text segment is shorter than the grid's query blocks assume.
  if (PREFIX && qb * kRowsPerWg >= seg_len) return;

  const size_t head_rows = (size_t)a.P * PREFIX + (size_t)a.F * T;
  const uint16_t* Kh = a.k + bh * head_rows * D;
  const uint16_t* Vh = a.v + bh * head_rows * D;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 31, hf = lane >> 5;
  const int qrow = qb * kRowsPerWg + wave * 32 + n;
  const bool wave_active = qb * kRowsPerWg + wave * 32 < seg_len;

  // This lane's query: Q^T and dO^T B-operand slices, its lse (base 2) and -delta,
  // the start of every dP^T accumulation.
  bf16x8 qf[Sh::kChunks], gf[Sh::kChunks];
  const bool valid = qrow < seg_len;
  const size_t qr = (size_t)bh * head_rows + seg0 + qrow;
  load_row_operand<D>(a.q + qr * D, valid, a.keep, a.flip, hf, qf);
  load_row_operand<D>(a.dout + qr * D, valid, ~0u, 0u, hf, gf);
  const float lse2 = valid ? a.lse2[qr] : 0.f;
  const float ndlt = valid ? a.ndelta[qr] : 0.f;
  f32x16 dp_start;
#pragma unroll
  for (int e = 0; e < 16; ++e) dp_start[e] = ndlt;

  f32x16 acc[Sh::kDBlocks];
#pragma unroll
  for (int mb = 0; mb < Sh::kDBlocks; ++mb) acc[mb] = f32x16{};

  const int tpf = (T + kBlockK - 1) / kBlockK;
  int n_tiles = n_kept * tpf;
  if constexpr (PREFIX) {
    // the text segment (index F) sorts last in a kept list
    if (n_kept > 0 && a.cols_q[kbeg + n_kept - 1] == a.F) n_tiles += (a.P + kBlockK - 1) / kBlockK - tpf;
  }
  if (n_tiles > 0) {
    DualLoader<D> ld;
    ld.init(wave, lane);
    RowAddr<D> ra;
    ra.init(n, hf);
    TrAddr<D> ta;
    ta.init(lane);
    SegmentCursor<PREFIX> cur, nxt;
    cur.start(a.cols_q + kbeg, lay);
    ld.load(Kh, cur.key0(), cur.nvalid(), sK[0], wave);
    ld.load(Vh, cur.key0(), cur.nvalid(), sV[0], wave);
    nxt = cur;
    nxt.advance(n_kept);
    wait_tile_loads();
    __syncthreads();

    // S^T and dP^T - delta of 32-key block kb (raw logits; keys past the tile's valid
    // rows read zero rows).
    auto scores = [&](const uint16_t* tk, const uint16_t* tv, int kb, f32x16& sc, f32x16& dp) {
      sc = f32x16{};
      dp = dp_start;
#pragma unroll
      for (int cc = 0; cc < Sh::kChunks; ++cc) {
        sc = mfma32(row_frag<D>(tk, ra, kb, cc), qf[cc], sc);
        dp = mfma32(row_frag<D>(tv, ra, kb, cc), gf[cc], dp);
      }
    };
    // dQ^T += K^T dS^T over block kb.
    auto accumulate = [&](const uint16_t* tk, int kb, const bf16x8 (&ds)[2]) {
#pragma unroll
      for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
        for (int mb = 0; mb < Sh::kDBlocks; ++mb)
          acc[mb] = mfma32(tr_frag<D>(tk, ta, mb, 2 * kb + c2), ds[c2], acc[mb]);
    };

    // One tile; the buffer index is a compile-time constant (tiles run in pairs), so
    // every LDS address is a per-lane base plus an immediate offset.
    auto tile_step = [&](auto bufc, int t) {
      constexpr int buf = decltype(bufc)::value;
      if (t + 1 < n_tiles) {
        ld.load(Kh, nxt.key0(), nxt.nvalid(), sK[buf ^ 1], wave);
        ld.load(Vh, nxt.key0(), nxt.nvalid(), sV[buf ^ 1], wave);
      }
      if (wave_active) {
        // Block 1's S/dP run on the matrix cores while block 0's dS forms on the
        // vector ALUs, then block 0's dQ update while block 1's dS forms. The
        // scheduling fences keep each phase's fragments and scores from being
        // hoisted into the previous one (5% faster than leaving the order free).
        if constexpr (D != 96) {
        f32x16 s0, dp0, s1, dp1;
        bf16x8 ds0[2], ds1[2];
        scores(sK[buf], sV[buf], 0, s0, dp0);
        __builtin_amdgcn_sched_barrier(0);
        scores(sK[buf], sV[buf], 1, s1, dp1);
        dq_scores(s0, dp0, a.c, lse2, ds0);
        __builtin_amdgcn_sched_barrier(0);
        accumulate(sK[buf], 0, ds0);
        dq_scores(s1, dp1, a.c, lse2, ds1);
        __builtin_amdgcn_sched_barrier(0);
        accumulate(sK[buf], 1, ds1);
        } else {
          // At d = 96 the same phases as one stream of fenced packets of one MFMA, its
          // fragment read two packets ahead and an even share of the vector steps (see the
          // dk/dv pass): 204 registers instead of 226, 93-frame gradients 16.20 -> 16.15 ms,
          // 29-frame sym 7.57 -> 7.53 ms. Not at d = 64 (the text form 0.5% slower), nor
          // at d = 128, where it does not fit 256 registers.
          constexpr int kC = Sh::kChunks, kMb = Sh::kDBlocks, kAhead = 2;
          constexpr int kHalf = 2 * kC, kAcc = 2 * kMb, kN = 2 * kHalf + 2 * kAcc;
          f32x16 sc[2], dp[2];
          bf16x8 ds[2][2];
          float t0, t1, y0, y1;
          auto frag = [&](auto ic) -> bf16x8 {
            constexpr int i = decltype(ic)::value;
            if constexpr (i < 2 * kHalf) {
              constexpr int h = i / kHalf, r = i % kHalf;
              return row_frag<D>(r % 2 ? sV[buf] : sK[buf], ra, h, r / 2);
            } else {
              constexpr int j = i - 2 * kHalf, h = j / kAcc, r = j % kAcc;
              return tr_frag<D>(sK[buf], ta, r % kMb, 2 * h + r / kMb);
            }
          };
          bf16x8 fr[kAhead + 1];
          static_for<kAhead>([&](auto jc) { fr[decltype(jc)::value] = frag(jc); });
          __builtin_amdgcn_sched_barrier(0);
          static_for<kN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i + kAhead < kN)
              fr[(i + kAhead) % (kAhead + 1)] = frag(std::integral_constant<int, i + kAhead>{});
            const bf16x8& f = fr[i % (kAhead + 1)];
            if constexpr (i < 2 * kHalf) {
              constexpr int h = i / kHalf, r = i % kHalf;
              if constexpr (r % 2 == 0) sc[h] = mfma32(f, qf[r / 2], r == 0 ? f32x16{} : sc[h]);
              else dp[h] = mfma32(f, gf[r / 2], r == 1 ? dp_start : dp[h]);
            } else {
              constexpr int j = i - 2 * kHalf, h = j / kAcc, r = j % kAcc;
              acc[r % kMb] = mfma32(f, ds[h][r / kMb], acc[r % kMb]);
            }
            constexpr int h = i < kHalf ? -1 : (i < 2 * kHalf ? 0 : (i < 2 * kHalf + kAcc ? 1 : -1));
            if constexpr (h >= 0) {
              constexpr int k = h == 0 ? i - kHalf : i - 2 * kHalf, kPk = h == 0 ? kHalf : kAcc;
#pragma unroll
              for (int m = k * 72 / kPk; m < (k + 1) * 72 / kPk; ++m) {
                const int op = m % 9, e = 2 * (m / 9), c2 = e / 8;
                if (op == 0) t0 = __builtin_fmaf(sc[h][e], a.c, -lse2);
                if (op == 1) t1 = __builtin_fmaf(sc[h][e + 1], a.c, -lse2);
                if (op == 2) t0 = __builtin_amdgcn_fmed3f(fast_exp2(t0), 0.f, 1.f);
                if (op == 4) t1 = __builtin_amdgcn_fmed3f(fast_exp2(t1), 0.f, 1.f);
                if (op == 6) y0 = t0 * dp[h][e];
                if (op == 7) y1 = t1 * dp[h][e + 1];
                if (op == 8) {
                  const f32x2 dd = {y0, y1};
                  u32x4 dw = __builtin_bit_cast(u32x4, ds[h][c2]);
                  dw[(e % 8) / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(dd, bf16x2));
                  ds[h][c2] = __builtin_bit_cast(bf16x8, dw);
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        }
      }
      cur = nxt;
      nxt.advance(n_kept);
      wait_tile_loads();
      __syncthreads();
    };
    for (int t = 0; t < n_tiles; t += 2) {
      tile_step(std::integral_constant<int, 0>{}, t);
      if (t + 1 < n_tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    }
  }

  if (qrow < seg_len) {
    if (slot < 0) {
      store_row_bf16<D>(a.dq + qr * D, acc, a.scale, hf);
    } else {
      const int slot_rows = PREFIX ? max(T, a.P) : T;
      const size_t prow = ((size_t)slot * a.B + b) * slot_rows + qrow;
      store_row_f32<D>(a.ws_dq + prow * D, acc, a.scale, hf);
    }
  }
}

// ---------------------------------------------------------------------------
// dk/dv pass.
// The key-side pass over one work unit (b, item of the transposed plan, key block).
template <int D, bool PREFIX, int MODE>
__device__ __forceinline__ void dkdv_unit(const BwdArgs& a, int nkb, uint32_t work,
                                          uint16_t (&sQ)[2][BShape<D>::kTileElems],
                                          uint16_t (&sG)[2][BShape<D>::kTileElems],
                                          float (&sL)[2][kBlockK], float (&sD)[2][kBlockK]) {
  constexpr bool kWantDv = MODE != kDkOnly, kWantDk = MODE != kDvOnly;
  using Sh = BShape<D>;
  const uint32_t per_b = (uint32_t)a.n_items_k * (uint32_t)nkb;
  const uint32_t b = work / per_b;
  const uint32_t rem = work - b * per_b;
  const int32_t* item = a.items_k + 5 * (rem / nkb);
  const uint32_t bh = b * (uint32_t)a.H + (uint32_t)item[0];
  const int frame = item[1], qbeg = item[2], n_keep = item[3], slot = item[4];
  const int kblk = (int)(rem % nkb);
  const int T = a.T;
  const Layout<PREFIX> lay{a.F, T, a.P};
  const int seg0 = lay.start(frame), seg_len = lay.len(frame);
  if (PREFIX && kblk * kRowsPerWg >= seg_len) return;

  const size_t head_rows = (size_t)a.P * PREFIX + (size_t)a.F * T;
  const uint16_t* Qh = a.q + bh * head_rows * D;
  const uint16_t* Gh = a.dout + bh * head_rows * D;
  const float* Lh = a.lse2 + bh * head_rows;
  const float* Dh = a.ndelta + bh * head_rows;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 31, hf = lane >> 5;
  const int krow = kblk * kRowsPerWg + wave * 32 + n;
  const bool wave_active = kblk * kRowsPerWg + wave * 32 < seg_len;

  // This lane's key as B operand of S = Q K^T and dP = dO V^T.
  bf16x8 kf[Sh::kChunks], vf[kWantDk ? Sh::kChunks : 1];
  const bool valid = krow < seg_len;
  const size_t kr = (size_t)bh * head_rows + seg0 + krow;
  load_row_operand<D>(a.k + kr * D, valid, a.keep, a.flip, hf, kf);
  if constexpr (kWantDk) load_row_operand<D>(a.v + kr * D, valid, ~0u, 0u, hf, vf);

  f32x16 dk[kWantDk ? Sh::kDBlocks : 1], dv[kWantDv ? Sh::kDBlocks : 1];
#pragma unroll
  for (int mb = 0; mb < Sh::kDBlocks; ++mb) {
    if constexpr (kWantDk) dk[mb] = f32x16{};
    if constexpr (kWantDv) dv[mb] = f32x16{};
  }

  const int tpf = (T + kBlockK - 1) / kBlockK;
  int n_tiles = n_keep * tpf;
  if constexpr (PREFIX) {
    if (n_keep > 0 && a.cols_k[qbeg + n_keep - 1] == a.F) n_tiles += (a.P + kBlockK - 1) / kBlockK - tpf;
  }
  if (n_tiles > 0) {
    DualLoader<D> ld;
    ld.init(wave, lane);
    RowAddr<D> ra;
    ra.init(n, hf);
    TrAddr<D> ta;
    ta.init(lane);
    // Q, dO, lse2 and -delta of one 64-query tile; rows past the valid range read
    // as zeros, so they add exactly nothing below (zero Q and dO rows, P <= 1).
    auto load_tile = [&](const SegmentCursor<PREFIX>& tc, int bi) {
      const size_t row0 = tc.key0();
      const int nv = tc.nvalid();
      ld.load(Qh, row0, nv, sQ[bi], wave);
      ld.load(Gh, row0, nv, sG[bi], wave);
      if (wave == 0) {
        load_dword_to_lds(buffer_words(Lh + row0, (uint32_t)(nv * 4)), lds_addr((const uint16_t*)sL[bi]),
                          4 * lane);
        if constexpr (kWantDk)
          load_dword_to_lds(buffer_words(Dh + row0, (uint32_t)(nv * 4)), lds_addr((const uint16_t*)sD[bi]),
                            4 * lane);
      }
    };
    SegmentCursor<PREFIX> cur, nxt;
    cur.start(a.cols_k + qbeg, lay);
    load_tile(cur, 0);
    nxt = cur;
    nxt.advance(n_keep);
    wait_tile_loads();
    __syncthreads();

    // dP - delta of 32-query half qc of the tile: the accumulation starts at the rows' -delta
    // (entry 8 c2 + 4u + j holds query row 32 qc + 16 c2 + 8u + 4h + j), read at the
    // half's first packet.
    auto dp_start = [&](int buf, int qc, f32x16& dp) {
#pragma unroll
      for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(&sD[buf][32 * qc + 16 * c2 + 8 * u + 4 * hf]);
#pragma unroll
          for (int j = 0; j < 4; ++j) dp[8 * c2 + 4 * u + j] = d4[j];
        }
    };
    // One tile; the buffer index is a compile-time constant (the loop below runs tiles
    // in pairs), so every LDS address is a per-lane base plus an immediate offset.
    auto tile_step = [&](auto bufc, int t) {
      constexpr int buf = decltype(bufc)::value;
      if (t + 1 < n_tiles) load_tile(nxt, buf ^ 1);
      if (wave_active) {
        // One stream of MFMAs (8 D/16 per tile for dV and dK together), each in a
        // fenced packet with its share of the vector work; the operand fragment of
        // MFMA i is read from LDS at packet i - 2 into one of three rotating
        // registers (i - 1 and two registers in the dK pass of d = 128), so no MFMA
        // waits on a read issued just before it (3.5% faster than leaving the order to
        // the compiler, measured at the 93-frame shape). Stream: S (and dP) of half 0, S
        // (and dP) of half 1 with half 0's P (and dS) forming, the dV/dK update of
        // half 0 with half 1's P (and dS) forming, the update of half 1. The passes of
        // d = 128 run the same stream: the dV pass (S, P, dV) without dP, dS and dK,
        // the dK pass (S, dP, dS, dK) without P and dV and with each fragment read one
        // packet ahead into two registers (two ahead would need more registers than it
        // has; the stream is 4.5% faster than the compiler's order there).
        constexpr int kC = Sh::kChunks, kMb = Sh::kDBlocks;
        constexpr int kAhead = MODE == kDkOnly ? 1 : 2;  // packets between a read and its use
        constexpr int kHalf = (kWantDk ? 2 : 1) * kC;                   // S (+ dP) MFMAs of a half
        constexpr int kAcc = ((int)kWantDv + (int)kWantDk) * 2 * kMb;  // update MFMAs of a half
        constexpr int kN = 2 * kHalf + 2 * kAcc;                        // the whole stream
        constexpr int kPerC2 = kAcc / 2;                                 // update MFMAs per chunk
        f32x16 sc[2], dp[kWantDk ? 2 : 1];
        bf16x8 pb[kWantDv ? 2 : 1][2], db[kWantDk ? 2 : 1][2];
        f32x4 l4[2][4];  // lse2 of this lane's 16 queries of each half, 4 at a time
        float t0, t1, y0, y1;
        // Update MFMA r of a half: chunk c2, d-block mb, dK (else dV).
        auto upd = [](int r, int& c2, int& mb, bool& is_dk) {
          c2 = r / kPerC2;
          const int q = r % kPerC2;
          if (kWantDv && kWantDk) {
            mb = q / 2;
            is_dk = q % 2;
          } else {
            mb = q;
            is_dk = kWantDk;
          }
        };
        auto frag = [&](auto ic) -> bf16x8 {
          constexpr int i = decltype(ic)::value;
          if constexpr (i < 2 * kHalf) {
            constexpr int h = i / kHalf, r = i % kHalf;
            if constexpr (r < kC) return row_frag<D>(sQ[buf], ra, h, r);
            else return row_frag<D>(sG[buf], ra, h, r - kC);
          } else {
            constexpr int j = i - 2 * kHalf, h = j / kAcc, r = j % kAcc;
            int c2, mb;
            bool is_dk;
            upd(r, c2, mb, is_dk);
            return tr_frag<D>(is_dk ? sQ[buf] : sG[buf], ta, mb, 2 * h + c2);
          }
        };
        auto mfma = [&](auto ic, const bf16x8& f) {
          constexpr int i = decltype(ic)::value;
          if constexpr (i < 2 * kHalf) {
            constexpr int h = i / kHalf, r = i % kHalf;
            if constexpr (r < kC) sc[h] = mfma32(f, kf[r], r == 0 ? f32x16{} : sc[h]);
            else if constexpr (kWantDk) dp[h] = mfma32(f, vf[r - kC], dp[h]);
          } else {
            constexpr int j = i - 2 * kHalf, h = j / kAcc, r = j % kAcc;
            int c2, mb;
            bool is_dk;
            upd(r, c2, mb, is_dk);
            if constexpr (kWantDk && kWantDv) {
              if (is_dk) dk[mb] = mfma32(f, db[h][c2], dk[mb]);
              else dv[mb] = mfma32(f, pb[h][c2], dv[mb]);
            } else if constexpr (kWantDk) {
              dk[mb] = mfma32(f, db[h][c2], dk[mb]);
            } else {
              dv[mb] = mfma32(f, pb[h][c2], dv[mb]);
            }
          }
        };
        // Vector work of packet i: LDS reads of -delta (dP starts) and lse2 ahead of
        // their use, and P (and dS) of half 0 over the second half's S/dP packets, of
        // half 1 over half 0's update packets.
        auto side = [&](auto ic) {
          constexpr int i = decltype(ic)::value;
          if constexpr (kWantDk && (i == 0 || i == kHalf)) dp_start(buf, i / kHalf, dp[i / kHalf]);
          // lse2 of queries 4 q4 .. 4 q4 + 3 (entries 4 q4 ..) of half hh, read one packet
          // before the first one whose share of the steps below needs them (in that packet
          // itself for half 0 of the d = 128 dK pass). A packet earlier measured 0 to 0.3%
          // slower at d = 96 (93-frame gradients 15.97 -> 16.02 ms), 0.7% at d = 64 (24 heads
          // of 24 x 1200: 1.518 -> 1.529 ms) and the same at d = 128.
          static_for<8>([&](auto qc) {
            constexpr int hh = decltype(qc)::value / 4, q4 = decltype(qc)::value % 4;
            constexpr int st = hh == 0 ? kHalf : 2 * kHalf, pk = hh == 0 ? kHalf : kAcc;
            constexpr int at = st + ((2 * q4 + 1) * pk + 7) / 8 - 1 - kAhead;
            if constexpr (at == i)
              l4[hh][q4] = *reinterpret_cast<const f32x4*>(&sL[buf][32 * hh + 16 * (q4 / 2) + 8 * (q4 % 2) + 4 * hf]);
          });
          constexpr int h = i < kHalf ? -1 : (i < 2 * kHalf ? 0 : (i < 2 * kHalf + kAcc ? 1 : -1));
          if constexpr (h >= 0) {
            constexpr int k = h == 0 ? i - kHalf : i - 2 * kHalf;  // packet within the share
            constexpr int kPk = h == 0 ? kHalf : kAcc;
            // Ten steps per pair, an exponential counting two, dealt out evenly: the pairs
            // as lumps made some packets longer than their MFMA (0.3-0.6% slower).
#pragma unroll
            for (int m = k * 80 / kPk; m < (k + 1) * 80 / kPk; ++m) {
              // pair m / 10 of the half's queries (entries e, e + 1 = 8 c2 + 4 uu + j)
              const int op = m % 10, e = 2 * (m / 10), c2 = e / 8, uu = (e % 8) / 4, j = e % 4;
              if (op == 0) t0 = __builtin_fmaf(sc[h][e], a.c, -l4[h][2 * c2 + uu][j]);
              if (op == 1) t1 = __builtin_fmaf(sc[h][e + 1], a.c, -l4[h][2 * c2 + uu][j + 1]);
              if (op == 2) t0 = __builtin_amdgcn_fmed3f(fast_exp2(t0), 0.f, 1.f);
              if (op == 4) t1 = __builtin_amdgcn_fmed3f(fast_exp2(t1), 0.f, 1.f);
              if constexpr (kWantDk) {
                if (op == 6) y0 = t0 * dp[h][e];
                if (op == 7) y1 = t1 * dp[h][e + 1];
              }
              if constexpr (kWantDv) {
                if (op == 8) {
                  const f32x2 pp = {t0, t1};
                  u32x4 pw = __builtin_bit_cast(u32x4, pb[h][c2]);
                  pw[(e % 8) / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
                  pb[h][c2] = __builtin_bit_cast(bf16x8, pw);
                }
              }
              if constexpr (kWantDk) {
                if (op == 9) {
                  const f32x2 dd = {y0, y1};
                  u32x4 dw = __builtin_bit_cast(u32x4, db[h][c2]);
                  dw[(e % 8) / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(dd, bf16x2));
                  db[h][c2] = __builtin_bit_cast(bf16x8, dw);
                }
              }
            }
          }
        };
        bf16x8 fr[kAhead + 1];
        static_for<kAhead>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          fr[j] = frag(std::integral_constant<int, j>{});
        });
        __builtin_amdgcn_sched_barrier(0);
        static_for<kN>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          if constexpr (i + kAhead < kN)
            fr[(i + kAhead) % (kAhead + 1)] = frag(std::integral_constant<int, i + kAhead>{});
          mfma(ic, fr[i % (kAhead + 1)]);
          side(ic);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      cur = nxt;
      nxt.advance(n_keep);
      wait_tile_loads();
      __syncthreads();
    };
    for (int t = 0; t < n_tiles; t += 2) {
      tile_step(std::integral_constant<int, 0>{}, t);
      if (t + 1 < n_tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    }
  }

  // dK uses the unflipped q of the LDS tiles, so scale (with its sign) applies.
  if (krow < seg_len) {
    if (slot < 0) {
      if constexpr (kWantDk) store_row_bf16<D>(a.dk + kr * D, dk, a.scale, hf);
      if constexpr (kWantDv) store_row_bf16<D>(a.dv + kr * D, dv, 1.f, hf);
    } else {
      const int slot_rows = PREFIX ? max(T, a.P) : T;
      const size_t prow = ((size_t)slot * a.B + b) * slot_rows + krow;
      if constexpr (kWantDk) store_row_f32<D>(a.ws_dk + prow * D, dk, a.scale, hf);
      if constexpr (kWantDv) store_row_f32<D>(a.ws_dv + prow * D, dv, 1.f, hf);
    }
  }
}

// ---------------------------------------------------------------------------
// dk/dv pass at d = 128, one wave per SIMD.
//
// dK, dV (128 registers), the K and V operands (64) and the scores of a 32-key block do not
// fit 256 VGPRs together, and as two passes (dV, dK) S is formed twice. This kernel
// runs one 4-wave workgroup per compute unit with 512 registers per wave: the accumulators
// stay in AGPRs, everything the vector ALU touches in VGPRs, and S is formed once (four
// products instead of five). With one wave per SIMD nothing else hides a stall, so each
// wave runs one unbroken stream of matrix instructions over 32-query blocks:
//   body h:  S, dP of block h          | P, dS of block h - 1, second half of its queries
//            dV, dK update of h - 1    | P, dS of block h, first half
// with the vector work dealt out a few instructions per MFMA, every operand fragment read
// kAhead packets ahead across the phases, and the blocks in a ring of kRing LDS slots, five
// blocks loaded ahead, so that one barrier per two blocks suffices and never waits for the
// block it is about to use. (MFMA 47% busy at 1.99 GHz as a plain tile loop, 60% at
// 1.84 GHz as this stream.) Measured at the 93-frame shape, H = 18, col g = 1, the dk/dv
// pass 12.55 -> 9.81 ms.

// This lane's id, read where it is called (an asm statement the compiler cannot hoist):
// the epilogues derive their rows from it, so no row address is held in vector registers
// across a tile loop.
__device__ __forceinline__ int fresh_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

// acc += a b with the accumulator kept in AGPRs. The compiler does not track the hazards of
// an asm MFMA; here none can arise: a comes from LDS (its wait counts asm operands), b was
// written by the vector ALU at least one MFMA earlier, and acc is read by nothing but these
// MFMAs, the next on the same accumulator 2 D/32 - 1 others later, until the drain after the
// loop.
__device__ __forceinline__ void mfma_acc(bf16x8 a, bf16x8 b, f32x16& acc) {
  asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

constexpr int kRing = 8;
// Elements of a ring slot: the 32-row Q and dO blocks, lse2 and -delta (64 floats each, the
// first 32 used).
template <int D>
constexpr int roll_slot() { return 2 * 32 * D + 256; }

template <int D, bool PREFIX>
__device__ __forceinline__ void dkdv_roll_unit(const BwdArgs& a, int nkb, uint32_t work, uint16_t* ring) {
  using Sh = BShape<D>;
  constexpr int kC = Sh::kChunks, kMb = Sh::kDBlocks;
  constexpr int kBlk = 32 * D;              // elements of a 32-row block of one tensor
  constexpr int kSlot = roll_slot<D>();
  constexpr int kLd = kBlk * 2 / 2048;      // tile loads per wave and block (two waves per tensor)
  constexpr int kAhead = 3;
  const uint32_t per_b = (uint32_t)a.n_items_k * (uint32_t)nkb;
  const uint32_t b = work / per_b;
  const uint32_t rem = work - b * per_b;
  const int32_t* item = a.items_k + 5 * (rem / nkb);
  const uint32_t bh = b * (uint32_t)a.H + (uint32_t)item[0];
  const int frame = item[1], qbeg = item[2], n_keep = item[3], slot = item[4];
  const int kblk = (int)(rem % nkb);
  const int T = a.T;
  const Layout<PREFIX> lay{a.F, T, a.P};
  const int seg0 = lay.start(frame), seg_len = lay.len(frame);
  if (PREFIX && kblk * kRowsPerWg >= seg_len) return;

  const size_t head_rows = (size_t)a.P * PREFIX + (size_t)a.F * T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = kblk * kRowsPerWg + wave * 32;  // this wave's first key of the segment

  // This lane's key as B operand of S = Q K^T and dP = dO V^T.
  bf16x8 kf[kC], vf[kC];
  f32x16 dk[kMb], dv[kMb];
  {
    const int lane = fresh_lane(), krow = row0 + (lane & 31);
    const size_t kr = (size_t)bh * head_rows + seg0 + krow;
    load_row_operand<D>(a.k + kr * D, krow < seg_len, a.keep, a.flip, lane >> 5, kf);
    load_row_operand<D>(a.v + kr * D, krow < seg_len, ~0u, 0u, lane >> 5, vf);
  }
#pragma unroll
  for (int mb = 0; mb < kMb; ++mb) dk[mb] = dv[mb] = f32x16{};

  const int bpf = (T + 31) / 32;
  int nb = n_keep * bpf;  // 32-query blocks
  if constexpr (PREFIX) {
    if (n_keep > 0 && a.cols_k[qbeg + n_keep - 1] == a.F) nb += (a.P + 31) / 32 - bpf;
  }
  if (nb > 0) {
    const int lane = fresh_lane();
    const int hf = lane >> 5;
    RowAddr<D> ra;
    ra.init(lane & 31, hf);
    TrAddr<D> ta;
    ta.init(lane);
    // Waves 0 and 1 load the Q blocks (half a block each) and lse2, waves 2 and 3 dO and
    // -delta. Both waves of a tensor load the same row values, so that every wave has the
    // same number of loads in flight.
    const bool second = wave >= 2;
    const uint16_t* src = (second ? a.dout : a.q) + bh * head_rows * D;
    const float* lsrc = (second ? a.ndelta : a.lse2) + bh * head_rows;
    int off[kLd];
#pragma unroll
    for (int j = 0; j < kLd; ++j) {
      const int q = 64 * ((wave & 1) * kLd + j) + lane;
      const int r = q / Sh::kPieces, ps = q % Sh::kPieces;
      off[j] = (r * D + 8 * (ps ^ dsw<D>(r))) * 2;
    }
    const uint32_t lds_dst = lds_addr(ring) + (second ? kBlk * 2 : 0) + (wave & 1) * kLd * 1024;
    const uint32_t lds_row_dst = lds_addr(ring) + 4 * kBlk + (second ? 256 : 0);
    // The block to load next: its rows start at src / lsrc, `left` rows of its segment
    // remain (0 past the last block: those loads write zeros), at ring byte offset ld_off.
    // The kept list is read with scalar loads.
    using ColsPtr = const __attribute__((address_space(4))) int32_t*;
    const ColsPtr cols = (ColsPtr)(a.cols_k + qbeg);
    int ld_e = 0, left = lay.len(cols[0]);
    uint32_t ld_off = 0;
    {
      const int64_t r0 = lay.start(cols[0]);
      src += r0 * D;
      lsrc += r0;
    }
    // (buffer_words without its readfirstlanes: everything here is scalar already)
    auto words = [](const void* p, uint32_t bytes) {
      const uint64_t x = reinterpret_cast<uint64_t>(p);
      return i32x4{(int)(uint32_t)x, (int)(uint32_t)(x >> 32), (int)bytes, 0x00020000};
    };
    auto load_part = [&](int j) {
      load_to_lds(words(src, (uint32_t)(min(left, 32) * D * 2)), lds_dst + ld_off + 1024u * j, off[j]);
    };
    auto load_rows = [&]() {
      load_dword_to_lds(words(lsrc, (uint32_t)(min(left, 32) * 4)), lds_row_dst + ld_off, 4 * lane);
    };
    auto load_advance = [&]() {
      ld_off = ld_off == (kRing - 1) * kSlot * 2 ? 0 : ld_off + kSlot * 2;
      src += 32 * D;
      lsrc += 32;
      left -= 32;
      if (left <= 0) {
        left = 0;
        if (++ld_e < n_keep) {
          const int j = cols[ld_e];
          const size_t r0 = (size_t)bh * head_rows + lay.start(j);
          src = (second ? a.dout : a.q) + r0 * D;
          lsrc = (second ? a.ndelta : a.lse2) + r0;
          left = lay.len(j);
        }
      }
    };
    // Zeros in the last slot: the block that the body before block 0's update runs over.
    // (Weights of zero times block 0's own rows would turn an infinite dO into NaN.) Then
    // blocks 0 .. 4 in flight, the zeros and block 0 visible.
    const int left0 = left;
    left = 0;
    ld_off = (kRing - 1) * kSlot * 2;
#pragma unroll
    for (int i = 0; i < kLd; ++i) load_part(i);
    load_rows();
    left = left0;
    ld_off = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      if (j > 0) load_advance();
#pragma unroll
      for (int i = 0; i < kLd; ++i) load_part(i);
      load_rows();
    }
    wait_loads<4 * (kLd + 1)>();
    __syncthreads();

    // By block parity: S and dP - delta, P and dS of the first 16 query entries (queries
    // 16 c2 + 8u + 4 hf + j are entries 8 c2 + 4u + j); p1, d1 of the second.
    f32x16 sc[2], dp[2];
    bf16x8 p0[2], d0[2], p1, d1;
    auto row_values = [&](const uint16_t* at, int first, f32x4& lo, f32x4& hi) {
      const float* L = reinterpret_cast<const float*>(at + 2 * kBlk) + first + 4 * hf;
      lo = *reinterpret_cast<const f32x4*>(L);
      hi = *reinterpret_cast<const f32x4*>(L + 8);
    };
    // P and dS of entries 8 c2 .. 8 c2 + 7, as a list of 10 steps per pair of entries (an
    // exponential counts two) dealt out evenly to n packets; packet i's share.
    float t0, t1, y0, y1;
    auto vec_share = [&](auto parc, auto c2c, auto ic, auto nc, const f32x4(&l4)[2]) {
      constexpr int par = decltype(parc)::value, c2 = decltype(c2c)::value, i = decltype(ic)::value,
                    n = decltype(nc)::value;
      if constexpr (i >= 0) {
#pragma unroll
        for (int m = i * 40 / n; m < (i + 1) * 40 / n; ++m) {
          const int op = m % 10, e = 8 * c2 + 2 * (m / 10), w = (e % 8) / 2;
          if (op == 0) t0 = __builtin_fmaf(sc[par][e], a.c, -l4[(e % 8) / 4][e % 4]);
          if (op == 1) t1 = __builtin_fmaf(sc[par][e + 1], a.c, -l4[(e % 8) / 4][e % 4 + 1]);
          if (op == 2) t0 = __builtin_amdgcn_fmed3f(fast_exp2(t0), 0.f, 1.f);  // as prob()
          if (op == 4) t1 = __builtin_amdgcn_fmed3f(fast_exp2(t1), 0.f, 1.f);
          if (op == 6) y0 = t0 * dp[par][e];
          if (op == 7) y1 = t1 * dp[par][e + 1];
          if (op >= 8) {
            const f32x2 v = op == 8 ? f32x2{t0, t1} : f32x2{y0, y1};
            bf16x8& dst = op == 8 ? (c2 ? p1 : p0[par]) : (c2 ? d1 : d0[par]);
            u32x4 x = __builtin_bit_cast(u32x4, dst);
            x[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
            dst = __builtin_bit_cast(bf16x8, x);
          }
        }
      }
    };
    constexpr int kNA = 2 * kC, kNU = 4 * kMb;  // fragments (= MFMAs) of the two phases
    auto frag_a = [&](const uint16_t* at, auto ic) -> bf16x8 {
      constexpr int i = decltype(ic)::value;
      return as_bf16x8(load16(at + (i < kC ? ra.get(i) : kBlk + ra.get(i - kC))));
    };
    auto frag_u = [&](const uint16_t* at, auto ic) -> bf16x8 {
      constexpr int i = decltype(ic)::value, c2 = i / (2 * kMb), q = i % (2 * kMb);
      return tr_frag<D>(at + (q % 2 ? 0 : kBlk), ta, q / 2, c2);
    };
    bf16x8 pf[kAhead];        // the first fragments of the next phase
    uint32_t at_c = 0, at_p = (kRing - 1) * kSlot;  // ring offsets (elements) of blocks h and h - 1
    auto body = [&](auto parc) {
      constexpr int par = decltype(parc)::value;
      const uint32_t at_n = at_c == (kRing - 1) * kSlot ? 0 : at_c + kSlot;
      const uint16_t *tc = ring + at_c, *tp = ring + at_p, *tn = ring + at_n;
      f32x4 l4[2];
      bf16x8 fr[kAhead + 1];
      using ParC = std::integral_constant<int, par>;
      using ParP = std::integral_constant<int, par ^ 1>;
      row_values(tp, 16, l4[0], l4[1]);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) fr[j] = pf[j];
      __builtin_amdgcn_sched_barrier(0);
      static_for<kNA>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i + kAhead < kNA) fr[(i + kAhead) % (kAhead + 1)] = frag_a(tc, std::integral_constant<int, i + kAhead>{});
        else pf[i + kAhead - kNA] = frag_u(tp, std::integral_constant<int, i + kAhead - kNA>{});
        if constexpr (i == kC - 2) {  // dP starts at the rows' -delta
          f32x4 d4[4];
          row_values(tc, 64, d4[0], d4[1]);
          row_values(tc, 80, d4[2], d4[3]);
#pragma unroll
          for (int e = 0; e < 16; ++e) dp[par][e] = d4[e / 4][e % 4];
        }
        const bf16x8& f = fr[i % (kAhead + 1)];
        if constexpr (i < kC) sc[par] = mfma32(f, kf[i], i == 0 ? f32x16{} : sc[par]);
        else dp[par] = mfma32(f, vf[i - kC], dp[par]);
        vec_share(ParP{}, std::integral_constant<int, 1>{}, std::integral_constant<int, i - 1>{},
                  std::integral_constant<int, kNA - 1>{}, l4);
        __builtin_amdgcn_sched_barrier(0);
      });
      // The asm statement keeps the compiler from sinking the packets' vector work past
      // the branch in load_advance, to the first use of p1 and d1.
      asm volatile("" : "+v"(p1), "+v"(d1));
      load_advance();
      if constexpr (par == 0) {
        // Blocks h + 1 and h + 2 have landed (those of h + 3 and h + 4 may be in flight),
        // for every wave once all are here; every wave is also done with block h - 2, so
        // the slots of blocks h - 3 and h - 2 can take blocks h + 5 and h + 6.
        wait_loads<2 * (kLd + 1)>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      row_values(tc, 0, l4[0], l4[1]);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) fr[j] = pf[j];
      __builtin_amdgcn_sched_barrier(0);
      static_for<kNU>([&](auto ic) {
        constexpr int i = decltype(ic)::value, c2 = i / (2 * kMb), q = i % (2 * kMb), mb = q / 2;
        if constexpr (i + kAhead < kNU) fr[(i + kAhead) % (kAhead + 1)] = frag_u(tp, std::integral_constant<int, i + kAhead>{});
        else pf[i + kAhead - kNU] = frag_a(tn, std::integral_constant<int, i + kAhead - kNU>{});
        if constexpr (i >= 1 && i <= kLd) load_part(i - 1);
        if constexpr (i == kLd + 1) load_rows();
        const bf16x8& f = fr[i % (kAhead + 1)];
        if constexpr (q % 2) mfma_acc(f, c2 ? d1 : d0[par ^ 1], dk[mb]);
        else mfma_acc(f, c2 ? p1 : p0[par ^ 1], dv[mb]);
        vec_share(ParC{}, std::integral_constant<int, 0>{}, std::integral_constant<int, i - 2>{},
                  std::integral_constant<int, kNU - 2>{}, l4);
        __builtin_amdgcn_sched_barrier(0);
      });
      asm volatile("" : "+v"(p0[par]), "+v"(d0[par]));
      at_p = at_c;
      at_c = at_n;
    };
    // Before block 0 there is nothing to update: P, dS (exp2(-inf)) and rows are zero. Blocks
    // nb and nb + 1 are zeros, so the bodies past the last block add exactly nothing.
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      sc[1][e] = -INFINITY;
      dp[1][e] = 0.f;
    }
    p0[1] = d0[1] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
    static_for<kAhead>([&](auto jc) { pf[decltype(jc)::value] = frag_a(ring, jc); });
    for (int h = 0; h <= nb; h += 2) {
      body(std::integral_constant<int, 0>{});
      body(std::integral_constant<int, 1>{});
    }
    wait_tile_loads();
  }

  // The last MFMAs are done before the accumulators are read (16 passes at most).
#pragma unroll
  for (int mb = 0; mb < kMb; ++mb) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(dk[mb]), "+a"(dv[mb]));
  // dK uses the unflipped q of the LDS blocks, so scale (with its sign) applies.
  const int lane = fresh_lane(), hf = lane >> 5, row = row0 + (lane & 31);
  if (row < seg_len) {
    if (slot < 0) {
      const size_t at = ((size_t)bh * head_rows + seg0 + row) * D;
      store_row_bf16<D>(a.dk + at, dk, a.scale, hf);
      store_row_bf16<D>(a.dv + at, dv, 1.f, hf);
    } else {
      const int slot_rows = PREFIX ? max(T, a.P) : T;
      const size_t at = (((size_t)slot * a.B + b) * slot_rows + row) * D;
      store_row_f32<D>(a.ws_dk + at, dk, a.scale, hf);
      store_row_f32<D>(a.ws_dv + at, dv, 1.f, hf);
    }
  }
}

template <int D, bool PREFIX>
__global__ __launch_bounds__(kBwdThreads, 1) void bwd_dkdv_roll_kernel(const BwdArgs a, int nblk) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kRing * roll_slot<D>()];
  const uint32_t x = blockIdx.x % 8, u = a.share_k[x] + blockIdx.x / 8;
  if (u < a.share_k[x + 1]) dkdv_roll_unit<D, PREFIX>(a, nblk, u, ring);
}

// One pass per launch: each XCD (the workgroups with blockIdx % 8 == x) runs a contiguous
// share of the pass's units.
template <int D, bool PREFIX>
__global__ __launch_bounds__(kBwdThreads, 2) void bwd_dq_kernel(const BwdArgs a, int nblk) {
  using Sh = BShape<D>;
  __shared__ __attribute__((aligned(1024))) uint16_t sK[2][Sh::kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t sV[2][Sh::kTileElems];
  const uint32_t x = blockIdx.x % 8, u = a.share_q[x] + blockIdx.x / 8;
  if (u < a.share_q[x + 1]) dq_unit<D, PREFIX>(a, nblk, u, sK, sV);
}

template <int D, bool PREFIX>
__global__ __launch_bounds__(kBwdThreads, 2) void bwd_dkdv_kernel(const BwdArgs a, int nblk) {
  using Sh = BShape<D>;
  __shared__ __attribute__((aligned(1024))) uint16_t sQ[2][Sh::kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t sG[2][Sh::kTileElems];
  __shared__ __attribute__((aligned(256))) float sL[2][kBlockK];
  __shared__ __attribute__((aligned(256))) float sD[2][kBlockK];
  const uint32_t x = blockIdx.x % 8, u = a.share_k[x] + blockIdx.x / 8;
  if (u < a.share_k[x + 1]) dkdv_unit<D, PREFIX, kDkDv>(a, nblk, u, sQ, sG, sL, sD);
}

// All passes in one launch, for calls of few rounds of workgroups: XCD x runs its share of
// the key side's units, then of the query side's (at d = 128 the dK pass, dq, then the dV
// pass), in each head the longest items first. As launches of their own each pass ends on a ragged round
// with most slots empty, and a small call takes the sum of the passes' latencies. Measured
// (launches of their own -> one launch, same process): B = 2, H = 4, 5 x 257 tokens at
// d = 96, col g = 1 47.7 -> 38.1 us; H = 8, 10 x 700 at d = 64 137 -> 121 us; H = 6,
// 24 x 3600 at d = 96, sym (25 rounds) 6.53 -> 6.40 ms; H = 12 col (40 rounds) 8.51 ->
// 8.43 ms (d = 128: merge_rounds). Over many rounds the seam is nothing and the
// shared kernel costs (H = 24 col, 80 rounds: 16.58 -> 16.68 ms), so longer calls keep a
// launch per pass (merge_rounds; kMinRollBlocks).
template <int D, bool PREFIX>
__global__ __launch_bounds__(kBwdThreads, 2) void bwd_all_kernel(const BwdArgs a, int nblk) {
  using Sh = BShape<D>;
  __shared__ __attribute__((aligned(1024))) uint16_t s0[2][Sh::kTileElems];
  __shared__ __attribute__((aligned(1024))) uint16_t s1[2][Sh::kTileElems];
  __shared__ __attribute__((aligned(256))) float sL[2][kBlockK];
  __shared__ __attribute__((aligned(256))) float sD[2][kBlockK];
  const uint32_t x = blockIdx.x % 8;
  const uint32_t k0 = a.share_k[x], nk = a.share_k[x + 1] - k0;
  const uint32_t q0 = a.share_q[x], nq = a.share_q[x + 1] - q0;
  uint32_t pos = blockIdx.x / 8;
  if (pos < nk) {
    dkdv_unit<D, PREFIX, split_key_pass<D>() ? kDkOnly : kDkDv>(a, nblk, k0 + pos, s0, s1, sL, sD);
    return;
  }
  pos -= nk;
  if (pos < nq) {
    dq_unit<D, PREFIX>(a, nblk, q0 + pos, s0, s1);
    return;
  }
  if constexpr (split_key_pass<D>()) {
    pos -= nq;
    if (pos < nk) dkdv_unit<D, PREFIX, kDvOnly>(a, nblk, k0 + pos, s0, s1, sL, sD);
  }
}

// ---------------------------------------------------------------------------
// Sum of the partials of split segments, of dq, dk and dv in one launch (grid y picks the
// tensor): one thread per (split segment, batch entry, row, 8 consecutive d), rounded to
// bf16 (RNE). Partials are laid out [slot][batch][L][d] with L = max(T, P) rows per slot
// (T without a prefix).
template <int D>
__global__ __launch_bounds__(256) void sum_partials_kernel(const SumArgs a) {
  constexpr int kGroups = D / 8;
  const SumJob& job = a.job[blockIdx.y];
  const int F = a.F, T = a.T, P = a.P, L = max(T, P);
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t per_seg = (size_t)a.B * L * kGroups;
  if (idx >= per_seg * (size_t)job.n_heavy) return;
  const int hv = (int)(idx / per_seg);
  const size_t r = idx - (size_t)hv * per_seg;
  const int grp = (int)(r % kGroups);
  const size_t row = r / kGroups;  // b * L + t
  const size_t b = row / L, t = row - b * L;
  const int head = job.heavy[4 * hv], frame = job.heavy[4 * hv + 1];
  const int slot0 = job.heavy[4 * hv + 2], np = job.heavy[4 * hv + 3];
  const int seg0 = frame < F ? P + frame * T : 0, seg_len = frame < F ? T : P;
  if ((int)t >= seg_len) return;
  const size_t slot_stride = (size_t)a.B * L;
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < np; ++p) {
    const f32x4* src =
        reinterpret_cast<const f32x4*>(job.ws + ((size_t)(slot0 + p) * slot_stride + row) * D + 8 * grp);
    a0 += src[0];
    a1 += src[1];
  }
  const size_t orow = (b * a.H + head) * ((size_t)P + (size_t)F * T) + seg0 + t;
  const f32x8 x = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
  *reinterpret_cast<bf16x8*>(job.out + orow * D + 8 * grp) = __builtin_convertvector(x, bf16x8);
}

template <int D>
hipError_t prep_d(const PrepArgs& a, hipStream_t stream) {
  const int64_t blocks = (a.rows + kPrepRows - 1) / kPrepRows;
  hipLaunchKernelGGL(bwd_prep_kernel<D>, dim3((uint32_t)blocks), dim3(256), 0, stream, a.out, a.dout,
                     a.lse, a.lse2, a.ndelta, a.rows);
  return hipGetLastError();
}

template <int D, bool PREFIX>
void bwd_launches(const BwdArgs& a, int nblk, hipStream_t stream) {
  const dim3 threads(kBwdThreads);
  const uint32_t passes_k = split_key_pass<D>() ? 2 : 1;
  const uint32_t units = passes_k * a.n_wg_k + a.n_wg_q;
  uint32_t nk[8], nq[8], all[8];  // positions of each XCD
  for (int x = 0; x < 8; ++x) {
    nk[x] = a.share_k[x + 1] - a.share_k[x];
    nq[x] = a.share_q[x + 1] - a.share_q[x];
    all[x] = passes_k * nk[x] + nq[x];
  }
  const bool few = units <= merge_rounds<D>() * 8u * (uint32_t)a.slots_per_xcd;
  const bool fits = (uint64_t)grid_of(all) * kBwdThreads <= UINT32_MAX;
  if (few || (split_key_pass<D>() && a.key_blocks < kMinRollBlocks && fits)) {
    hipLaunchKernelGGL((bwd_all_kernel<D, PREFIX>), dim3(grid_of(all)), threads, 0, stream, a, nblk);
    return;
  }
  hipLaunchKernelGGL((bwd_dq_kernel<D, PREFIX>), dim3(grid_of(nq)), threads, 0, stream, a, nblk);
  if constexpr (split_key_pass<D>()) {
    hipLaunchKernelGGL((bwd_dkdv_roll_kernel<D, PREFIX>), dim3(grid_of(nk)), threads, 0, stream, a, nblk);
  } else {
    hipLaunchKernelGGL((bwd_dkdv_kernel<D, PREFIX>), dim3(grid_of(nk)), threads, 0, stream, a, nblk);
  }
}

template <int D>
hipError_t bwd_d(const BwdArgs& a, hipStream_t stream) {
  const int nblk = (std::max(a.T, a.P) + kRowsPerWg - 1) / kRowsPerWg;
  if (a.P > 0) bwd_launches<D, true>(a, nblk, stream);
  else bwd_launches<D, false>(a, nblk, stream);
  return hipGetLastError();
}

template <int D>
hipError_t sum_d(const SumArgs& a, hipStream_t stream) {
  int n_heavy = 0;
  for (int j = 0; j < a.n_jobs; ++j) n_heavy = std::max(n_heavy, a.job[j].n_heavy);
  const size_t threads = (size_t)n_heavy * a.B * std::max(a.T, a.P) * (D / 8);
  const size_t blocks = (threads + 255) / 256;
  hipLaunchKernelGGL(sum_partials_kernel<D>, dim3((uint32_t)blocks, (uint32_t)a.n_jobs), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

int bwd_queries_per_workgroup(int) { return kRowsPerWg; }

int bwd_keys_per_workgroup(int) { return kRowsPerWg; }

#define TA_DISPATCH_D(fn, a, stream)          \
  switch ((a).d) {                            \
    case 64: return fn<64>(a, stream);        \
    case 96: return fn<96>(a, stream);        \
    case 128: return fn<128>(a, stream);      \
    default: return hipErrorInvalidValue;     \
  }

hipError_t launch_bwd_prep(const PrepArgs& a, hipStream_t stream) { TA_DISPATCH_D(prep_d, a, stream) }
hipError_t launch_bwd(const BwdArgs& a, hipStream_t stream) { TA_DISPATCH_D(bwd_d, a, stream) }
hipError_t launch_sum_partials(const SumArgs& a, hipStream_t stream) { TA_DISPATCH_D(sum_d, a, stream) }

#undef TA_DISPATCH_D

}  // namespace ta
