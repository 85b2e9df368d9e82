// Output layer of the sparse MLP (Sec. 5.1): Z = H1 W2^T + b2 over L labels,
// softmax + multi-label cross-entropy, its gradient and the SGD update of W2
// and b2 (Sec. 2.1), and top-k prediction.  Logits are never stored.
//
// Forward (k_out_fwd_train): workgroup = (label split, block of rows).  For
// every 32-label tile: Z^T = W2_tile H1^T on the matrix cores; a single-pass
// online max / sum of exponentials per row; and, with the same
// probabilities, O^T += W2_tile^T P^T.  O/s is sum_l softmax(Z)_l W2[l], the
// dense part of dH1 = (P - T) W2 / B, so the backward never needs a second
// pass over W2 for dH1.  Rows are the N dimension of both products, so all
// per-row state (running max, rescale factor) is per lane.
// Per row, after the forward: k_out_lse_targets merges the splits' (max, sum)
// pairs (log-sum-exp) and forms the target terms and the loss; k_out_dA1
// merges the splits' O (dH1 = (O/s - mean_{y in Y_i} W2[y]) / B,
// dA1 = dH1 * [A1 > 0]); one launch does both when they share a stream.
// The backward with the W2 / b2 update is in k_out_bwd.hip.
#include <algorithm>

#include <float.h>
#include <math.h>

#include <hip/hip_ext.h>

#include "asgd_dev.h"
#include "asgd_kernels.h"
#include "aux_dev.h"
#include "out_tile.h"

namespace asgd {

// Number of workgroup b of n in XCD-major order.  Workgroups are dealt to the 8
// XCDs in turn (b to XCD b mod 8), each with its own L2; numbered this way, those
// of one XCD are consecutive, so neighbours (the row blocks of a split, which read
// the same W2 tiles; rows that share the cache lines of the per-split arrays) are
// served by one L2 instead of each fetching from memory.
__device__ __forceinline__ int xcd_order(int b, int n) {
  const int x = b & 7;
  return x * (n >> 3) + min(x, n & 7) + (b >> 3);
}

int out_rows_per_block(bool use_bf16) { return use_bf16 ? FwdShape<true>::RB : FwdShape<false>::RB; }

// ---------------------------------------------------------------------------
// Forward, training: per (split, row) partial max, sum of exponentials and O.
// ---------------------------------------------------------------------------
// LDS ring of W2 tiles: one workgroup barrier per FwdRing::P tiles.  Between
// two barriers the waves read tiles t .. t+P and store t+P+1 .. t+2P, so a ring
// of 2P+1 tiles keeps what is read and what is written apart.  The bf16 tile
// (10 KB) allows P = 2; the fp32 operands (two 17-18 KB layouts per tile) keep
// P = 1.
template <bool BF16>
struct FwdRing {
  static constexpr int P = BF16 ? 2 : 1;
  static constexpr int N = 2 * P + 1;
};

// With a label job, workgroup n_fwd of the launch (dispatched last, on a CU
// the forward leaves free) groups the batch's labels for the backward: it
// depends only on the gather and finishes long before the forward, so the
// backward needs no event from another stream.  Its counters live in the
// launch's dynamic LDS (or in global memory when they do not fit).  With a
// sort job, the workgroups after it run the feature sort's first pass.
template <bool BF16>
__global__ __launch_bounds__(FWD_THREADS) void k_out_fwd_train(
    const float* __restrict__ W2, const float* __restrict__ b2, int L,
    const typename Mma<BF16>::elem* __restrict__ H1, int B, int tiles_per_split, int n_tiles,
    float* __restrict__ m_part, float* __restrict__ s_part, float* __restrict__ o_part,
    int ld_part, int s_eff, int n_fwd, LabelJob lj, SortJob sj) {
  using M = Mma<BF16>;
  using E = typename M::elem;
  using Fr = typename M::frag;
  constexpr int RB = FwdShape<BF16>::RB;
  constexpr int NCH = 32 / M::KC;
  static_assert(FwdShape<BF16>::NB == 1, "one 32-row block per wave");
  constexpr int P = FwdRing<BF16>::P, NRING = FwdRing<BF16>::N;
  __shared__ __attribute__((aligned(16))) E wr[NRING][tile_elems<BF16>()];
  __shared__ __attribute__((aligned(16))) E wt[NRING][tileT_elems<BF16>()];
  __shared__ __attribute__((aligned(16))) float bt[NRING][OUT_TILE];

  extern __shared__ __attribute__((aligned(16))) int32_t job_lds[];
  if ((int)blockIdx.x > n_fwd) {  // the feature sort's first pass
    wg_sort_pass<FWD_THREADS>(sj, (int)blockIdx.x - n_fwd - 1, job_lds);
    return;
  }
  if ((int)blockIdx.x == n_fwd) {
    if (lj.in_lds)
      wg_label_blocks<FWD_THREADS, true>(lj.lkeys, lj.m, L, lj.lrow, lj.lbeg, lj.lpair, job_lds,
                                         job_lds + ((L + 31) >> 5));
    else
      wg_label_blocks<FWD_THREADS, false>(lj.lkeys, lj.m, L, lj.lrow, lj.lbeg, lj.lpair, lj.lcnt, job_lds);
    return;
  }
  const int lane = threadIdx.x & 63, g = lane >> 5, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroup -> (split, row block).  Workgroups are dealt to the 8 XCDs in
  // turn (workgroup b to XCD b mod 8), each with its own L2, so the row blocks
  // of one split (which read the same W2 tiles) get consecutive numbers in
  // XCD-major order v: they share an XCD, and its L2 serves the tiles once.
  const int nrb = n_fwd / s_eff;
  const int b = (int)blockIdx.x;
  const int v = xcd_order(b, n_fwd);
  const int split = v / nrb;
  const int t_begin = split * tiles_per_split;
  const int t_end = min(n_tiles, t_begin + tiles_per_split);
  const int t_last = t_end - 1;
  // Rows past B (up to the 256-row padding, zero in H1) are computed like the
  // others and never written out, so the loop has no row-dependent branch.
  const int row0 = (v % nrb) * RB + wave * 32;
  const W2Src src = w2_src(W2, b2, L);
  const int rbase[2] = {tw_row_base(n, g, 0), tw_row_base(n, g, 1)};
  const int cbase[2] = {tw_col_base(lane, 0), tw_col_base(lane, 1)};

  // H1^T as the B operand (K = hidden, N = rows), resident for the whole split.
  Fr hf[4][NCH];
  const E* hrow = H1 + (size_t)(row0 + n) * HID;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int c = 0; c < NCH; ++c) hf[kb][c] = h1_frag<BF16>(hrow, kb, c, g);
  // Redefine the fragments once they have arrived (empty asm), so the loop below
  // never waits on these loads again and its wait counters track only the W2
  // prefetch.
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(hf[kb][c]));

  // Z^T tile from LDS buffer `buf`: A = W2 rows (M = labels, K = hidden),
  // B = H1^T; the accumulator starts at the labels' biases (-inf past L).
  auto z_tile = [&](int buf) {
    const float4* bq = reinterpret_cast<const float4*>(bt[buf]);
    f32x16 z;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = bq[2 * q + g];
      z[4 * q + 0] = b.x; z[4 * q + 1] = b.y; z[4 * q + 2] = b.z; z[4 * q + 3] = b.w;
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) z = M::mma(tile_frag_w<BF16>(wr[buf], rbase, n, kb, c, g), hf[kb][c], z);
    return z;
  };

  // (from -FLT_MAX and not -inf: on a tile of nothing but labels of bias -inf, which leaves
  // the reference where it is, -inf would make each numerator 2^(-inf + inf))
  float m_run = -FLT_MAX, s_run = 0.0f;
  f32x16 acc_o[4];
#pragma unroll
  for (int hb = 0; hb < 4; ++hb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[hb][r] = 0.0f;

  // Software pipeline over a ring of LDS tiles and two register tiles.  In the
  // iteration of tile t: the logits of tile t+1 go to the matrix cores while
  // the softmax numerators of tile t are formed; then O^T += W2_t^T P_t^T
  // while tile t+P+1 (loaded into registers two iterations earlier) is
  // converted into the ring and tile t+P+3 is loaded in its place; a barrier
  // closes every P-th iteration.  Tile u lives in ring slot (u - t_begin) mod
  // NRING.  Tile indices are clamped to the split's last tile, so every load,
  // store and product is unconditional (a clamped copy is never consumed).
  // Every split has at least one tile.
  TileRegs tr0, tr1;
  auto slot = [&](int u) { return (u - t_begin) % NRING; };
#pragma unroll
  for (int u = 0; u <= P; ++u) {
    const int tu = min(t_begin + u, t_last);
    tile_load(src, tu, tr0);
    tile_store<BF16, true>(tr0, L, tu, wr[u], wt[u], bt[u]);
  }
  tile_load(src, min(t_begin + P + 1, t_last), tr0);
  tile_load(src, min(t_begin + P + 2, t_last), tr1);
  __syncthreads();
  f32x16 z = z_tile(0);

  // Online softmax in base 2 with lazy rescaling: p = 2^(z log2e - m2) where m2
  // is a per-row reference that is raised only when a tile's maximum exceeds it
  // by more than LAZY (so p <= 2^LAZY); the final normalisation uses the same
  // reference, so the result is exact up to rounding.
  constexpr float LAZY = 8.0f, LAZY_SUM = 256.0f;  // LAZY_SUM = 2^LAZY
  auto iteration = [&](int t, TileRegs& tr) {
    const int b0 = slot(t), b1 = slot(t + 1), bst = slot(t + P + 1);
    // Operands of this iteration's two products, read from LDS first so that
    // their latency is covered by the max / rescale work below: A of the next
    // tile's logits (W2 rows, with the biases as the accumulator's start) and
    // A of this tile's O (W2^T rows).
    // (fp32 operands take 16 chunks per 32-wide block: those are read at use,
    // as holding them all would not fit the register file.)
    constexpr int PRE = BF16 ? NCH : 1;
    Fr za[4][PRE], oa[4][PRE];
    if constexpr (BF16) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int c = 0; c < NCH; ++c) za[kb][c] = tile_frag_w<BF16>(wr[b1], rbase, n, kb, c, g);
    }
    f32x16 zn;
    {
      const float4* bq = reinterpret_cast<const float4*>(bt[b1]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 b = bq[2 * q + g];
        zn[4 * q + 0] = b.x; zn[4 * q + 1] = b.y; zn[4 * q + 2] = b.z; zn[4 * q + 3] = b.w;
      }
    }
    if constexpr (BF16) {
#pragma unroll
      for (int hb = 0; hb < 4; ++hb)
#pragma unroll
        for (int c = 0; c < NCH; ++c) oa[hb][c] = tile_frag_wt<BF16>(wr[b0], wt[b0], cbase, hb, c, lane);
    }

    // The next tile's logits go to the matrix cores first; this tile's
    // numerators are formed on the vector units while they run, against the
    // current reference, and formed again in the rare iteration that raises
    // it, so every p that is used is computed against the reference the row
    // ends with at that point.
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        zn = M::mma(BF16 ? za[kb][c % PRE] : tile_frag_w<BF16>(wr[b1], rbase, n, kb, c, g), hf[kb][c], zn);
    // The tile's maximum is only formed when some lane's numerators sum past
    // 2^LAZY (or are not finite, as on a row's first tile, whose reference is
    // -FLT_MAX): no numerator exceeds its lane's sum, so every other tile keeps
    // p <= 2^LAZY against the current reference.
    float p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(z[r], LOG2E, -m_run));
    float ps = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) ps += p[r];
    if (__any(!(ps <= LAZY_SUM))) {
      // running maximum of this tile (rows are lanes: one max per lane pair)
      float tmax = z[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, z[r]);
      tmax = half_swap_max(tmax);
      const float m2c = tmax * LOG2E;
      const float m2n = m2c > m_run + LAZY ? m2c : m_run;
      const float scale = __builtin_amdgcn_exp2f(m_run - m2n);
      s_run *= scale;
#pragma unroll
      for (int hb = 0; hb < 4; ++hb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[hb][r] *= scale;
      m_run = m2n;
      ps = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = __builtin_amdgcn_exp2f(fmaf(z[r], LOG2E, -m_run));
        ps += p[r];
      }
    }
    s_run += ps;
    Fr pf[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) pf[c] = frag_acc<BF16>(p, c);
    // O^T += W2_t^T P^T : A = W2^T rows (M = hidden, K = labels).
#pragma unroll
    for (int hb = 0; hb < 4; ++hb)
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        acc_o[hb] = M::mma(BF16 ? oa[hb][c % PRE] : tile_frag_wt<BF16>(wr[b0], wt[b0], cbase, hb, c, lane),
                           pf[c], acc_o[hb]);
    tile_store<BF16, true>(tr, L, min(t + P + 1, t_last), wr[bst], wt[bst], bt[bst]);
    tile_load(src, min(t + P + 3, t_last), tr);
    if ((t - t_begin) % P == P - 1) __syncthreads();
    z = zn;
  };
  for (int t = t_begin; t < t_end; t += 2) {
    iteration(t, tr0);
    if (t + 1 >= t_end) break;
    iteration(t + 1, tr1);
  }

  const int row = row0 + n;
  const float stot = s_run + __shfl_xor(s_run, 32);
  if (row < B) {
    if (g == 0) {
      m_part[(size_t)split * ld_part + row] = m_run * LN2;
      s_part[(size_t)split * ld_part + row] = stot;
    }
    float* o = o_part + ((size_t)split * ld_part + row) * HID;
#pragma unroll
    for (int hb = 0; hb < 4; ++hb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(o + 32 * hb + 8 * q + 4 * g) =
            make_float4(acc_o[hb][4 * q], acc_o[hb][4 * q + 1], acc_o[hb][4 * q + 2],
                        acc_o[hb][4 * q + 3]);
  }
}

// ---------------------------------------------------------------------------
// The same for short splits (k_out_fwd_short).  Workgroup = (label split, 32 rows), its 8 waves on
// tiles of their own (t = wave, wave + 8, ... of the split): no tile is shared, so
// nothing in the loop waits for another wave, and the waves' partials merge in LDS,
// so a split is 8 waves' tiles long and there are few of them (at least 32 splits
// where there are the tiles, see fwd_plan).  The partials are
// what a short label space pays for above: every split writes, and the per-row pass
// reads back, 512 bytes per row, 32 MB at 240 splits and 256 rows, where W2 of
// 30,000 labels is 15 MB.  Batches of few rows also have no padding rows here (above,
// a workgroup computes 256 rows).  The price is that every 32 rows read all of W2
// (from the L2 that a split's row blocks share) and convert it: fwd_is_short says up
// to where it is worth that.  30,000 labels, 256 rows: the kernel 17 -> 14 us and the
// per-row pass after it 16 -> 9.
// ---------------------------------------------------------------------------
template <bool BF16>
struct ShortTile {
  static constexpr int ELEMS = tile_elems<BF16>();
  static constexpr int BYTES = ELEMS * (int)sizeof(typename Mma<BF16>::elem);
};
constexpr int SHORT_LD = HID + 4;  // row stride of a wave's merged O (floats)
// LDS: the waves' tiles during the loop, their O afterwards; biases, maxima and sums
template <bool BF16>
constexpr int short_lds() {
  constexpr int tiles = 8 * ShortTile<BF16>::BYTES, merged = 8 * 32 * SHORT_LD * 4;
  return (tiles > merged ? tiles : merged) + 3 * 8 * 32 * 4;
}

template <bool BF16>
__global__ __launch_bounds__(FWD_THREADS) void k_out_fwd_short(
    const float* __restrict__ W2, const float* __restrict__ b2, int L,
    const typename Mma<BF16>::elem* __restrict__ H1, int B, int tiles_per_split, int n_tiles,
    float* __restrict__ m_part, float* __restrict__ s_part, float* __restrict__ o_part,
    int ld_part, int s_eff, int n_fwd, LabelJob lj, SortJob sj) {
  using M = Mma<BF16>;
  using E = typename M::elem;
  using Fr = typename M::frag;
  constexpr int NCH = 32 / M::KC;
  constexpr int WAVES = FwdShape<BF16>::WAVES;
  extern __shared__ __attribute__((aligned(16))) char short_smem[];
  if ((int)blockIdx.x >= n_fwd) {
    int32_t* job_lds = reinterpret_cast<int32_t*>(short_smem);
    if ((int)blockIdx.x > n_fwd)
      wg_sort_pass<FWD_THREADS>(sj, (int)blockIdx.x - n_fwd - 1, job_lds);
    else if (lj.in_lds)
      wg_label_blocks<FWD_THREADS, true>(lj.lkeys, lj.m, L, lj.lrow, lj.lbeg, lj.lpair, job_lds,
                                         job_lds + ((L + 31) >> 5));
    else
      wg_label_blocks<FWD_THREADS, false>(lj.lkeys, lj.m, L, lj.lrow, lj.lbeg, lj.lpair, lj.lcnt, job_lds);
    return;
  }
  const int lane = threadIdx.x & 63, g = lane >> 5, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int AREA = short_lds<BF16>() - 3 * WAVES * 32 * 4;
  E* const tile = reinterpret_cast<E*>(short_smem) + wave * ShortTile<BF16>::ELEMS;
  float* const bt = reinterpret_cast<float*>(short_smem + AREA) + wave * 32;
  float* const red_m = reinterpret_cast<float*>(short_smem + AREA) + WAVES * 32;      // [WAVES][32]
  float* const red_s = reinterpret_cast<float*>(short_smem + AREA) + 2 * WAVES * 32;  // [WAVES][32]
  // the row blocks of a split on one XCD, as in k_out_fwd_train
  const int nrb = n_fwd / s_eff, wg = (int)blockIdx.x;
  const int v = xcd_order(wg, n_fwd);
  const int split = v / nrb;
  const int t_begin = split * tiles_per_split;
  const int t_end = min(n_tiles, t_begin + tiles_per_split);
  const int row0 = (v % nrb) * 32;
  const int rbase[2] = {tw_row_base(n, g, 0), tw_row_base(n, g, 1)};
  const int cbase[2] = {tw_col_base(lane, 0), tw_col_base(lane, 1)};

  // a tile's 32 rows as whole 512-byte rows, two per load (past L: zeros)
  const __amdgpu_buffer_rsrc_t w2r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W2), (short)0, L * HID * 4, BUF_RSRC_WORD3);
  const __amdgpu_buffer_rsrc_t b2r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(b2), (short)0, L * 4, BUF_RSRC_WORD3);
  const int r_lo = lane >> 5, col = 4 * (lane & 31);
  const int voff = (r_lo * HID + col) * 4;
  float4 nv[16];
  float nb;
  auto load = [&](int t) {
#pragma unroll
    for (int k = 0; k < 16; ++k)
      nv[k] = __builtin_bit_cast(
          float4, __builtin_amdgcn_raw_buffer_load_b128(w2r, voff + k * 2 * HID * 4,
                                                        (int)((unsigned)t * (unsigned)(OUT_TILE * HID * 4)), 0));
    nb = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b2r, n * 4, t * OUT_TILE * 4, 0));
  };
  int t = t_begin + wave;
  const bool any = t < t_end;  // (a short last split may leave waves without a tile)
  if (any) load(t);
  Fr hf[4][NCH];
  const E* hrow = H1 + (size_t)(row0 + n) * HID;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int c = 0; c < NCH; ++c) hf[kb][c] = h1_frag<BF16>(hrow, kb, c, g);

  float m_run = -FLT_MAX, s_run = 0.0f;  // as in k_out_fwd_train
  f32x16 acc_o[4];
#pragma unroll
  for (int hb = 0; hb < 4; ++hb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[hb][r] = 0.0f;
  constexpr float LAZY = 8.0f, LAZY_SUM = 256.0f;  // as in k_out_fwd_train
#pragma unroll 1
  for (; t < t_end; t += WAVES) {
    // the loaded tile into the wave's LDS tile, and the next one requested
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int r = 2 * k + r_lo;
      if constexpr (BF16) {
        bf16x4 p;
        p[0] = (bf16)nv[k].x; p[1] = (bf16)nv[k].y; p[2] = (bf16)nv[k].z; p[3] = (bf16)nv[k].w;
        *reinterpret_cast<bf16x4*>(tile + tw_off(r, col)) = p;
      } else {
        *reinterpret_cast<float4*>(tile + r * FwdShape<false>::WR + col) = nv[k];
      }
    }
    bt[n] = t * OUT_TILE + n < L ? nb : -INFINITY;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (t + WAVES < t_end) load(t + WAVES);
    // Z^T = W2_tile H1^T from the biases
    f32x16 z;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = *reinterpret_cast<const float4*>(bt + 8 * q + 4 * g);
      z[4 * q + 0] = b.x; z[4 * q + 1] = b.y; z[4 * q + 2] = b.z; z[4 * q + 3] = b.w;
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) z = M::mma(tile_frag_w<BF16>(tile, rbase, n, kb, c, g), hf[kb][c], z);
    float p[16], ps = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = __builtin_amdgcn_exp2f(fmaf(z[r], LOG2E, -m_run));
      ps += p[r];
    }
    if (__any(!(ps <= LAZY_SUM))) {
      float tmax = z[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, z[r]);
      tmax = half_swap_max(tmax);
      const float m2c = tmax * LOG2E;
      const float m2n = m2c > m_run + LAZY ? m2c : m_run;
      const float scale = __builtin_amdgcn_exp2f(m_run - m2n);
      s_run *= scale;
#pragma unroll
      for (int hb = 0; hb < 4; ++hb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[hb][r] *= scale;
      m_run = m2n;
      ps = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = __builtin_amdgcn_exp2f(fmaf(z[r], LOG2E, -m_run));
        ps += p[r];
      }
    }
    s_run += ps;
    // O^T += W2_t^T P^T.  fp32: the W2^T operand (lane = hidden unit) is read straight
    // from the row-major tile, 32 consecutive floats per half wavefront.
    Fr pf[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) pf[c] = frag_acc<BF16>(p, c);
#pragma unroll
    for (int hb = 0; hb < 4; ++hb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        if constexpr (BF16)
          acc_o[hb] = M::mma(tile_frag_wt<BF16>(tile, nullptr, cbase, hb, c, lane), pf[c], acc_o[hb]);
        else
          acc_o[hb] = M::mma(tile[kofs<false>(c, g, 0) * FwdShape<false>::WR + 32 * hb + n], pf[c], acc_o[hb]);
      }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }

  // Merge: every wave rescales to the rows' common maximum (a wave without a tile
  // holds m = -FLT_MAX and contributes zeros), then the sums are added in wave order.
  const float stot = s_run + __shfl_xor(s_run, 32);
  if (g == 0) red_m[wave * 32 + n] = m_run;
  __syncthreads();  // (and every wave is done with its tile)
  float mx = red_m[n];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, red_m[w * 32 + n]);
  const float sc = any ? __builtin_amdgcn_exp2f(m_run - mx) : 0.0f;
  if (g == 0) red_s[wave * 32 + n] = any ? stot * sc : 0.0f;
  float* const om = reinterpret_cast<float*>(short_smem) + (wave * 32 + n) * SHORT_LD;
#pragma unroll
  for (int hb = 0; hb < 4; ++hb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(om + 32 * hb + 8 * q + 4 * g) =
          make_float4(acc_o[hb][4 * q] * sc, acc_o[hb][4 * q + 1] * sc, acc_o[hb][4 * q + 2] * sc,
                      acc_o[hb][4 * q + 3] * sc);
  __syncthreads();
  // thread: 8 hidden units of row threadIdx.x / 16
  const int orow = threadIdx.x >> 4, h8 = (threadIdx.x & 15) * 8;
  const int row = row0 + orow;
  if (row >= B) return;
  const float* src = reinterpret_cast<const float*>(short_smem) + orow * SHORT_LD + h8;
  float4 o0 = *reinterpret_cast<const float4*>(src), o1 = *reinterpret_cast<const float4*>(src + 4);
#pragma unroll
  for (int w = 1; w < WAVES; ++w) {
    const float4 a = *reinterpret_cast<const float4*>(src + w * 32 * SHORT_LD);
    const float4 b = *reinterpret_cast<const float4*>(src + w * 32 * SHORT_LD + 4);
    o0.x += a.x; o0.y += a.y; o0.z += a.z; o0.w += a.w;
    o1.x += b.x; o1.y += b.y; o1.z += b.z; o1.w += b.w;
  }
  const size_t at = (size_t)split * ld_part + row;
  *reinterpret_cast<float4*>(o_part + at * HID + h8) = o0;
  *reinterpret_cast<float4*>(o_part + at * HID + h8 + 4) = o1;
  if (h8 == 0) {
    float M2 = red_m[orow], S = red_s[orow];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      M2 = fmaxf(M2, red_m[w * 32 + orow]);
      S += red_s[w * 32 + orow];
    }
    m_part[at] = M2 * LN2;
    s_part[at] = S;
  }
}

// Where the forward runs k_out_fwd_short.  Measured, us per step with it | without:
//   L = 1,000, B = 128 (fp32): 53 | 60    L = 30,000, B = 256: 64 | 73    L = 120,000, B = 256: 100 | 106
//   L = 670,091, B = 32: 247 | 253        L = 670,091, B = 64: 236 | 254  L = 670,091, B = 128: 253 | 251
//   L = 205,443, B = 256: 132 | 133       L = 30,000, B = 600: 111 | 112  L = 60,000, B = 600: 126 | 122
static bool fwd_is_short(int n_tiles, int B) {
  return B <= 64 || n_tiles * ((B + 31) / 32) <= 32768;  // (tile, 32-row block) products
}

// Splits of the forward and whether it runs k_out_fwd_short.
FwdPlan fwd_plan(bool use_bf16, int L, int B, int wgs) {
  const int n_tiles = (L + OUT_TILE - 1) / OUT_TILE;
  FwdPlan p;
  p.is_short = fwd_is_short(n_tiles, B);
  const int rb = p.is_short ? 32 : out_rows_per_block(use_bf16);
  p.nrb = (B + rb - 1) / rb;
  int s = p.is_short ? wgs / p.nrb : (wgs + p.nrb - 1) / p.nrb;
  // Short: a tile for each wave, or up to 32 splits of fewer tiles.  A step of so few labels
  // is one tile's chain per wave, and two waves of a SIMD share its matrix cores (128 fp32
  // products of a tile: 3.4 us), so the tiles go to more CUs until the per-row pass pays for
  // the splits.  us per step, 8 tiles per split | up to 32 splits | 60 splits:
  //   fp32, B = 128: L = 1,000 41.7 | 37.0 | -    L = 4,000 42.3 | 39.1 | 39.3   L = 10,000 55.7 | 55.7 | 56.3
  //   bf16, B = 128: L = 1,000 34.4 | 33.4 | -    L = 4,000 34.7 | 34.4 | 34.6   L = 10,000 37.2 | 37.2 | 37.4
  constexpr int WAVES = FwdShape<true>::WAVES, SPREAD = 32;
  const int most = p.is_short ? std::max((n_tiles + WAVES - 1) / WAVES, std::min(n_tiles, SPREAD)) : n_tiles;
  if (s > most) s = most;
  if (s < 1) s = 1;
  p.tps = (n_tiles + s - 1) / s;
  p.splits = (n_tiles + p.tps - 1) / p.tps;
  return p;
}

LabelJobPlan label_job_plan_for(const void* fn, int nthreads, int L) {
  LabelJobPlan p{};
  hipFuncAttributes fa{};
  int dev = 0, lds_max = 0;
  if (hipFuncGetAttributes(&fa, fn) != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return p;
  // what the kernel's own arrays leave of a workgroup's LDS (160 KB on gfx950)
  const int budget = lds_max - (int)fa.sharedSizeBytes;
  p.lds_budget = budget;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, budget) != hipSuccess) return p;
  const int ints = (L + 31) / 32 + nthreads / 64;
  p.in_lds = ints * 4 <= budget;
  p.lds_bytes = 4 * (p.in_lds ? ints : nthreads / 64);
  p.ok = p.lds_bytes <= budget;
  return p;
}

LabelJobPlan label_job_plan(bool use_bf16, int L) {
  const void* fn = use_bf16 ? (const void*)k_out_fwd_short<true> : (const void*)k_out_fwd_short<false>;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return {};
  return label_job_plan_for(use_bf16 ? (const void*)k_out_fwd_train<true> : (const void*)k_out_fwd_train<false>,
                            FWD_THREADS, L);
}

hipError_t launch_out_fwd_train(bool use_bf16, const float* W2, const float* b2, int L, const void* H1,
                                int B, const FwdPlan& fp, float* m_part, float* s_part, float* o_part,
                                int ld_part, const LabelJob* job, const LabelJobPlan* plan, const SortJob* sort,
                                int n_cu, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  const int n_tiles = (L + OUT_TILE - 1) / OUT_TILE;
  const int n_fwd = fp.splits * fp.nrb;
  LabelJob lj{};
  int lds = 0, n_job = 0;
  if (job) {
    if (!plan || !plan->ok) return hipErrorInvalidValue;
    lj = *job;
    lj.in_lds = plan->in_lds;
    lds = plan->lds_bytes;
    n_job = 1;
  }
  SortJob sj{};
  if (sort && sort->n > 0) {
    if (!job || sort->n > SORT_RIDE_MAX) return hipErrorInvalidValue;  // (its workgroups follow the label job's)
    sj = *sort;
    const int need = sort_pass_lds(sj.nbits, FWD_THREADS);
    if (need > plan->lds_budget) return hipErrorInvalidValue;
    if (need > lds) lds = need;
    // on the CUs that the forward's own workgroups and the label job leave free: more
    // workgroups than those would run one after the other
    n_job += sort_spread(&sj, FWD_THREADS, n_cu - n_fwd % n_cu - 1);
  }
  const dim3 grid(n_fwd + n_job), block(FWD_THREADS);
  auto go = [&](auto kern, auto* h1) {
    hipExtLaunchKernelGGL(kern, grid, block, lds, st, t0, t1, 0, W2, b2, L, h1, B, fp.tps, n_tiles, m_part, s_part,
                          o_part, ld_part, fp.splits, n_fwd, lj, sj);
    return hipGetLastError();
  };
  if (fp.is_short) {  // (all of its LDS is dynamic; label counters that fit the other kernel's fit here too)
    const int own = use_bf16 ? short_lds<true>() : short_lds<false>();
    if (own > lds) lds = own;
    return use_bf16 ? go(k_out_fwd_short<true>, (const bf16*)H1) : go(k_out_fwd_short<false>, (const float*)H1);
  }
  return use_bf16 ? go(k_out_fwd_train<true>, (const bf16*)H1) : go(k_out_fwd_train<false>, (const float*)H1);
}

// ---------------------------------------------------------------------------
// Per row, in two kernels so that only the small one sits between the forward
// and the backward:
//   k_out_lse_targets  lse from the splits' (max, sum) pairs, and the row's
//                      target terms: the mean of W2[y] over y in Y_i (the
//                      pre-update W2, before the backward writes it), the
//                      target logits and the loss;
//   k_out_dA1          the splits' O merged against the same maxima,
//                      dH1 = (O/s - mean_{y in Y_i} W2[y]) / B, dA1 = dH1 [A1 > 0]
//                      (runs beside the backward: it reads no W2).
// A step that forms dA1 on the model's stream anyway runs both in one launch
// (k_out_lse_targets<., true>).
// k_out_lse_targets: 512 threads, one (max, sum) pair per thread merged by
// wavefront reductions, 8 wavefronts x the row's labels for the target terms.
// k_out_dA1: 8 split groups x 32 threads x 4 hidden units (256 threads, 4 KB of LDS,
// so that it fits on a CU beside the backward); each group merges its splits online
// against its own running maximum, then the groups are rescaled to the row's maximum.
// Every partial is combined in a fixed order, so the results do not depend on
// scheduling.
// ---------------------------------------------------------------------------
constexpr int CMB_THREADS = 512;
constexpr int CMB_WAVES = CMB_THREADS / 64;   // 8
constexpr int DA_GROUPS = 8;        // k_out_dA1
constexpr int DA_GROUPS_WIDE = 16;  // k_out_lse_targets<., true>

// (m, s) <- the merge of two (maximum, sum of 2^(x - maximum)) pairs, base 2 or
// natural alike through exp_fast (natural logarithms here)
__device__ __forceinline__ void ms_merge_ln(float& m, float& s, float m2, float s2) {
  const float mm = fmaxf(m, m2);
  if (mm == -INFINITY) return;
  s = (m == -INFINITY ? 0.0f : s * exp_fast(m - mm)) + (m2 == -INFINITY ? 0.0f : s2 * exp_fast(m2 - mm));
  m = mm;
}

// DA: the row's dA1 as well, in the same workgroup (16 split groups), for a
// step that runs it on the model's stream anyway: one launch instead of two;
// the launch's first workgroups then run a pass of the feature sort, which takes as
// long as the rows do (as the last ones they started late: mid step 54.2 | 53.7 us).
// The launch is a chain of memory round trips (label range, label ids, their W2
// rows).  A group's first DA_PRE splits load before that chain and merge after it,
// and the log-sum-exp comes from the groups' merge, so the partials add no round
// trip, barrier or reduction of their own: tiny step 37.3 -> 35.9 us (mid and
// wide-feature, where the sort's pass bounds the launch, within 0.3 us).
template <bool BF16, bool DA>
__global__ __launch_bounds__(CMB_THREADS) void k_out_lse_targets(
    int splits, const float* __restrict__ m_part, const float* __restrict__ s_part, int ld_part,
    const float* __restrict__ W2, const float* __restrict__ b2, int L,
    const typename Mma<BF16>::elem* __restrict__ H1, CsrDev y, int has_y, float* __restrict__ lse_out,
    float* __restrict__ loss_rows, float* __restrict__ tw_out, const float* __restrict__ o_part,
    const float* __restrict__ A1, int B, float invB, float* __restrict__ dA1, DenseBwd dn, SortJob sj) {
  static_assert(!DA || CMB_THREADS == 32 * DA_GROUPS_WIDE, "dA1 takes the workgroup as 16 split groups");
  __shared__ float red_s[CMB_WAVES];
  __shared__ float red_m[CMB_WAVES];
  __shared__ float red_t[CMB_WAVES][HID];
  __shared__ float red_z[CMB_WAVES];
  const int n_sort = DA ? (int)gridDim.x - B : 0;
  if constexpr (DA) {
    extern __shared__ __attribute__((aligned(16))) int32_t job_lds[];
    if ((int)blockIdx.x < n_sort) {  // the feature sort's second pass: it takes longest, so first
      wg_sort_pass<CMB_THREADS>(sj, (int)blockIdx.x, job_lds);
      return;
    }
  }
  const int i = xcd_order((int)blockIdx.x - n_sort, B), t = threadIdx.x, lane = t & 63, w = t >> 6;
  constexpr int DA_PRE = DA ? 4 : 1;
  const int grp = t >> 5, h4 = (t & 31) * 4;
  float pm[DA_PRE], ps[DA_PRE], a1 = 0.0f;
  float4 po[DA_PRE];
  auto load_splits = [&](int k0) {  // (past the last split: the last, left out below)
#pragma unroll
    for (int u = 0; u < DA_PRE; ++u) {
      const size_t r = (size_t)min(k0 + DA_GROUPS_WIDE * u, splits - 1) * ld_part + i;
      pm[u] = m_part[r];
      ps[u] = s_part[r];
      po[u] = *reinterpret_cast<const float4*>(o_part + r * HID + h4);
    }
  };
  if constexpr (DA) {
    load_splits(grp);
    a1 = A1[(size_t)i * HID + (t & (HID - 1))];
  } else {
    float mg = -INFINITY, St = 0.0f;
    for (int k = t; k < splits; k += CMB_THREADS)
      ms_merge_ln(mg, St, m_part[(size_t)k * ld_part + i], s_part[(size_t)k * ld_part + i]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ms_merge_ln(mg, St, __shfl_xor(mg, o), __shfl_xor(St, o));
    if (lane == 0) {
      red_s[w] = St;
      red_m[w] = mg;
    }
  }
  // target terms: wave w takes labels q = w, w + 8, ... of row i, in that
  // order; lane owns hidden 2l, 2l+1.  The row's label ids are read
  // lane-parallel (every wave counts the valid ones), and a wave's W2 rows load
  // TGT_BATCH at a time ahead of their reductions.
  constexpr int TGT_BATCH = 4;
  float tw0 = 0.0f, tw1 = 0.0f, zw = 0.0f;
  int cnt = 0;
  if (has_y) {
    const int ybase = y.indptr[0];
    int ys = y.indptr[i], ye = y.indptr[i + 1];
    ys = max(ys, ybase);
    ye = min(ye, ybase + y.nnz);
    if (ye < ys) ye = ys;
    const float h0 = (float)H1[(size_t)i * HID + 2 * lane];
    const float h1v = (float)H1[(size_t)i * HID + 2 * lane + 1];
    for (int q0 = ys; q0 < ye; q0 += 64) {
      const int q = q0 + lane;
      const int lab = q < ye ? y.indices[q] : -1;
      cnt += __popcll(__ballot(lab >= 0 && lab < L));
    }
    // this wave's labels: the k-th is q = ys + w + 8k, k < mine; 64 per pass
    const int mine = (ye - ys - w + CMB_WAVES - 1) / CMB_WAVES;
    for (int k0 = 0; k0 < mine; k0 += 64) {
      const int qk = ys + w + CMB_WAVES * (k0 + lane);
      const int labv = k0 + lane < mine ? y.indices[qk] : -1;
      const int nk = min(64, mine - k0);
      for (int u0 = 0; u0 < nk; u0 += TGT_BATCH) {
        float2 wv[TGT_BATCH];
        float bv[TGT_BATCH];
        bool ok[TGT_BATCH];
#pragma unroll
        for (int u = 0; u < TGT_BATCH; ++u) {
          const int lab = __builtin_amdgcn_readlane(labv, min(u0 + u, nk - 1));
          ok[u] = u0 + u < nk && lab >= 0 && lab < L;
          const int lb = ok[u] ? lab : 0;
          wv[u] = *reinterpret_cast<const float2*>(W2 + (size_t)lb * HID + 2 * lane);
          bv[u] = b2[lb];
        }
#pragma unroll
        for (int u = 0; u < TGT_BATCH; ++u) {
          if (!ok[u]) continue;
          tw0 += wv[u].x;
          tw1 += wv[u].y;
          float o0 = wv[u].x, o1 = wv[u].y;
          if constexpr (BF16) {
            o0 = (float)(bf16)wv[u].x;
            o1 = (float)(bf16)wv[u].y;
          }
          zw += wave_sum(fmaf(h0, o0, h1v * o1)) + bv[u];
        }
      }
    }
    red_t[w][2 * lane] = tw0;
    red_t[w][2 * lane + 1] = tw1;
    if (lane == 0) red_z[w] = zw;
  }
  __shared__ float red_o[DA ? DA_GROUPS_WIDE : 1][HID];
  __shared__ float red_s2[DA_GROUPS_WIDE];
  __shared__ float red_m2[DA_GROUPS_WIDE];
  if constexpr (DA) {
    // from -FLT_MAX, and no split holds -inf (see k_out_dA1): no inf - inf
    float mg = -FLT_MAX, St = 0.0f;
    float4 O = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int k0 = grp;;) {
#pragma unroll
      for (int u = 0; u < DA_PRE; ++u) {
        // (opaque to the compiler, which otherwise moves the loads down here, into a branch each)
        asm volatile("" : "+v"(pm[u]), "+v"(ps[u]), "+v"(po[u].x), "+v"(po[u].y), "+v"(po[u].z), "+v"(po[u].w));
        const bool in = k0 + DA_GROUPS_WIDE * u < splits;
        const float mn = in ? fmaxf(mg, pm[u]) : mg;
        const float a = exp_fast(mg - mn), e = exp_fast(pm[u] - mn);
        St = in ? fmaf(e, ps[u], St * a) : St;
        O.x = in ? fmaf(e, po[u].x, O.x * a) : O.x;
        O.y = in ? fmaf(e, po[u].y, O.y * a) : O.y;
        O.z = in ? fmaf(e, po[u].z, O.z * a) : O.z;
        O.w = in ? fmaf(e, po[u].w, O.w * a) : O.w;
        mg = mn;
      }
      k0 += DA_GROUPS_WIDE * DA_PRE;
      if (k0 >= splits) break;
      load_splits(k0);
    }
    asm volatile("" : "+v"(a1));
    *reinterpret_cast<float4*>(&red_o[grp][h4]) = O;
    if ((t & 31) == 0) {
      red_s2[grp] = St;
      red_m2[grp] = mg;
    }
  }
  __syncthreads();
  float my_d = 0.0f;
  if (t < HID) {
    float M, Stot, Ot = 0.0f;
    if constexpr (DA) {
      M = red_m2[0];
#pragma unroll
      for (int k = 1; k < DA_GROUPS_WIDE; ++k) M = fmaxf(M, red_m2[k]);
      Stot = 0.0f;
#pragma unroll
      for (int k = 0; k < DA_GROUPS_WIDE; ++k) {
        const float e = exp_fast(red_m2[k] - M);
        Ot = fmaf(e, red_o[k][t], Ot);
        Stot = fmaf(e, red_s2[k], Stot);
      }
    } else {
      M = red_m[0], Stot = red_s[0];
#pragma unroll
      for (int k = 1; k < CMB_WAVES; ++k) ms_merge_ln(M, Stot, red_m[k], red_s[k]);
    }
    const float lse = M + logf(Stot);
    if (t == 0) lse_out[i] = lse;
    if (has_y) {
      float tw = red_t[0][t], zs = red_z[0];
#pragma unroll
      for (int k = 1; k < CMB_WAVES; ++k) {
        tw += red_t[k][t];
        zs += red_z[k];
      }
      const float inv_cnt = cnt > 0 ? 1.0f / (float)cnt : 0.0f;
      float mean;
      {
#pragma clang fp contract(off)  // (rounded by itself, as k_out_dA1 reads it)
        mean = tw * inv_cnt;
      }
      if constexpr (DA) {
        my_d = a1 > 0.0f ? (Ot / Stot - mean) * invB : 0.0f;
        dA1[(size_t)i * HID + t] = my_d;
      } else {
        tw_out[(size_t)i * HID + t] = mean;
      }
      if (t == 0) loss_rows[i] = lse - zs * inv_cnt;
    }
  }
  if constexpr (DA) {
    if (dn.Wh) {
      // my_d is the row's dA2: the first layer's dA1 = (dA2 Wh) * [A1 > 0], 4 groups of 128
      // threads over 32 units of the second layer each, added in group order
      __shared__ float d2[HID];
      if (t < HID) d2[t] = my_d;
      __syncthreads();
      const int k = t & (HID - 1), q = t / HID;
      float acc = 0.0f;
#pragma unroll
      for (int o = 0; o < HID / 4; ++o)
        acc = fmaf(d2[q * (HID / 4) + o], dn.Wh[(size_t)(q * (HID / 4) + o) * HID + k], acc);
      red_o[q][k] = acc;  // (read by everyone before the barrier above)
      __syncthreads();
      if (t < HID) {
        const float s = ((red_o[0][t] + red_o[1][t]) + red_o[2][t]) + red_o[3][t];
        dn.dA1[(size_t)i * HID + t] = dn.A1[(size_t)i * HID + t] > 0.0f ? s : 0.0f;
      }
    }
  }
}

// dA1 of one row: each group merges its splits' O online against its own running maximum,
// then the groups are rescaled to the row's maximum; thread t < HID writes hidden unit t.
__global__ __launch_bounds__(32 * DA_GROUPS) void k_out_dA1(int splits, const float* __restrict__ m_part,
                                                           const float* __restrict__ s_part,
                                                           const float* __restrict__ o_part, int ld_part,
                                                           const float* __restrict__ tw, const float* __restrict__ A1,
                                                           float invB, float* __restrict__ dA1) {
  __shared__ float red_o[DA_GROUPS][HID];
  __shared__ float red_s[DA_GROUPS];
  __shared__ float red_m[DA_GROUPS];
  const int i = xcd_order((int)blockIdx.x, (int)gridDim.x), t = threadIdx.x;
  const float tw_t = t < HID ? tw[(size_t)i * HID + t] : 0.0f;
  const int grp = t >> 5, h4 = (t & 31) * 4;
  float mg = -INFINITY, St = 0.0f;
  float4 O = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 8
  for (int s = grp; s < splits; s += DA_GROUPS) {
    const size_t r = (size_t)s * ld_part + i;
    const float ms = m_part[r];
    const float ss = s_part[r];
    const float4 o = *reinterpret_cast<const float4*>(o_part + r * HID + h4);
    // (no split has -inf: one of nothing but labels of bias -inf holds -FLT_MAX ln 2 and s = 0)
    const float mn = fmaxf(mg, ms);
    const float a = exp_fast(mg - mn), e = exp_fast(ms - mn);
    St = fmaf(e, ss, St * a);
    O.x = fmaf(e, o.x, O.x * a);
    O.y = fmaf(e, o.y, O.y * a);
    O.z = fmaf(e, o.z, O.z * a);
    O.w = fmaf(e, o.w, O.w * a);
    mg = mn;
  }
  *reinterpret_cast<float4*>(&red_o[grp][h4]) = O;
  if ((t & 31) == 0) {
    red_s[grp] = St;
    red_m[grp] = mg;
  }
  __syncthreads();
  if (t < HID) {
    float M = red_m[0];
#pragma unroll
    for (int k = 1; k < DA_GROUPS; ++k) M = fmaxf(M, red_m[k]);
    float Ot = 0.0f, Stot = 0.0f;
#pragma unroll
    for (int k = 0; k < DA_GROUPS; ++k) {
      const float e = red_m[k] == -INFINITY ? 0.0f : exp_fast(red_m[k] - M);
      Ot = fmaf(e, red_o[k][t], Ot);
      Stot = fmaf(e, red_s[k], Stot);
    }
    const float dh = (Ot / Stot - tw_t) * invB;
    dA1[(size_t)i * HID + t] = A1[(size_t)i * HID + t] > 0.0f ? dh : 0.0f;
  }
}

int lse_sort_threads() { return CMB_THREADS; }

hipError_t launch_out_lse_targets(bool use_bf16, int B, int splits, const float* m_part, const float* s_part,
                                  int ld_part, const float* W2, const float* b2, int L, const void* H1,
                                  const CsrDev* y, float* lse, float* loss_rows, float* tw, const float* o_part,
                                  const float* A1, float* dA1, const DenseBwd* dense, const SortJob* sort,
                                  hipStream_t st, hipEvent_t done) {
  CsrDev yy = y ? *y : CsrDev{0, 0, 0, nullptr, nullptr, nullptr};
  const bool da = y && dA1;
  const float invB = 1.0f / (float)B;
  if (dense && !da) return hipErrorInvalidValue;
  const DenseBwd dn = dense ? *dense : DenseBwd{};
  SortJob sj{};
  int lds = 0, n_sort = 0;
  if (sort && sort->n > 0) {
    if (!da || sort->n > SORT_RIDE_MAX) return hipErrorInvalidValue;
    sj = *sort;
    lds = sort_pass_lds(sj.nbits, CMB_THREADS);
    const int chunk = CMB_THREADS * sj.per_thread;  // (spread by sort_plan_ride)
    n_sort = (sj.n + chunk - 1) / chunk;
  }
  const dim3 grid(B + n_sort), block(CMB_THREADS);
  auto go = [&](auto kern, auto* h1) {
    if (done)
      hipExtLaunchKernelGGL(kern, grid, block, lds, st, nullptr, done, 0, splits, m_part, s_part, ld_part, W2, b2, L,
                            h1, yy, (int)(y != nullptr), lse, loss_rows, tw, o_part, A1, B, invB, dA1, dn, sj);
    else
      hipLaunchKernelGGL(kern, grid, block, lds, st, splits, m_part, s_part, ld_part, W2, b2, L, h1, yy,
                         y != nullptr, lse, loss_rows, tw, o_part, A1, B, invB, dA1, dn, sj);
  };
  if (use_bf16) {
    if (da)
      go(k_out_lse_targets<true, true>, (const bf16*)H1);
    else
      go(k_out_lse_targets<true, false>, (const bf16*)H1);
  } else {
    if (da)
      go(k_out_lse_targets<false, true>, (const float*)H1);
    else
      go(k_out_lse_targets<false, false>, (const float*)H1);
  }
  return hipGetLastError();
}

hipError_t launch_out_dA1(int B, int splits, const float* m_part, const float* s_part, const float* o_part,
                          int ld_part, const float* tw, const float* A1, float* dA1, hipStream_t st) {
  hipLaunchKernelGGL(k_out_dA1, dim3(B), dim3(32 * DA_GROUPS), 0, st, splits, m_part, s_part, o_part, ld_part, tw, A1,
                     1.0f / (float)B, dA1);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Prediction: per (split, row) top-k lists of (score, label), ties -> smaller id.
//
// Workgroup = (label split, 8 waves x 32 NB rows), W2 tiles through the LDS ring
// of the training forward.  A wave issues the next tile's logits to the matrix
// cores and meanwhile compares this tile's best score per row with the row's k-th
// best so far.  With 64 rows per wave (NB = 2) every W2 fragment read from LDS
// feeds two products: at 32 rows per wave the reads alone (64 KB per tile and CU)
// take as long as the products.
// A row is a lane pair (n, n + 32) whose list lives in registers, the same on both
// lanes, as KR = 1, 8 or 32 sorted double keys (below): an entry enters by a chain of
// max / min pairs, and only the accumulator registers with a score that reaches the
// list are looked at.  (Sorted lists of scores and ids in LDS took 4 us per tile
// while they filled: 50 of 70 us for 50 rows of 30,000 labels.)
// ---------------------------------------------------------------------------
// A (score, label) pair as a double that orders by score, then by smaller label: the
// score's value with the label (22 bits) below its last bit, complemented for positive
// scores.  Infinite scores become +-2^128 (so that the label bits make no NaN); NaN
// scores and labels past L become the empty key, below every other.
constexpr int TOPK_REG_K = 8;  // longer lists: 32 entries, 32 rows per wave
constexpr double TOPK_INF = 0x1p128, TOPK_EMPTY = -0x1p200, TOPK_FENCE = 0x1p300;
constexpr unsigned TOPK_ID_MASK = (1u << 22) - 1;
constexpr int TOPK_NONE = 0x7fffffff;  // the id where a row has fewer than k ranked labels (NaN logits are not)

__device__ __forceinline__ double max_key(double a, double b) {
  double d;
  // (asm: no canonicalising moves, as no key is NaN.  The compiler's hazard pass does not see
  // that it writes registers, so no matrix product may be in flight that still reads them as its
  // C.  Only a row block's first product of a tile can read another C than its own result, and
  // the others of its tile follow it in one chain, at least seven of 8 passes (32 rows per wave
  // with bf16 operands; 14 with 64 rows, 63 with fp32 operands), each waiting for the one
  // before: over 200 cycles, where the read of C ends within 20.  Keys are formed in a later
  // basic block than the tile's products, which none of them moves past.)
  asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double min_key(double a, double b) {
  double d;
  asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double topk_key(float sc, int id, int L) {
  sc += 0.0f;  // -0 ranks with +0
  const double d = min_key(max_key((double)sc, -TOPK_INF), TOPK_INF);
  const unsigned flip = ~(unsigned)(__builtin_bit_cast(int, sc) >> 31) & TOPK_ID_MASK;
  const uint64_t u = __builtin_bit_cast(uint64_t, d) | ((unsigned)id ^ flip);
  return sc == sc && id < L ? __builtin_bit_cast(double, u) : TOPK_EMPTY;
}
__device__ __forceinline__ float topk_score(double key) { return (float)key; }  // the label bits round away
__device__ __forceinline__ int topk_id(double key) {
  const uint64_t u = __builtin_bit_cast(uint64_t, key);
  return (int)(((unsigned)u ^ ((u >> 63) ? 0u : TOPK_ID_MASK)) & TOPK_ID_MASK);
}

template <bool BF16, int NB, int KR>
__global__ __launch_bounds__(FWD_THREADS) void k_out_fwd_topk(
    const float* __restrict__ W2, const float* __restrict__ b2, int L,
    const typename Mma<BF16>::elem* __restrict__ H1, int B, int tiles_per_split, int n_tiles,
    int s_eff, int k, double* __restrict__ part) {
  using M = Mma<BF16>;
  using E = typename M::elem;
  using Fr = typename M::frag;
  constexpr int WAVES = FwdShape<BF16>::WAVES;
  constexpr int WROWS = 32 * NB;
  constexpr int RB = WAVES * WROWS;
  constexpr int NCH = 32 / M::KC;
  constexpr int P = FwdRing<BF16>::P, NRING = FwdRing<BF16>::N;
  __shared__ __attribute__((aligned(16))) E wr[NRING][tile_elems<BF16>()];
  __shared__ __attribute__((aligned(16))) float bt[NRING][OUT_TILE];

  const int lane = threadIdx.x & 63, g = lane >> 5, n = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup -> (split, row block): the row blocks of a split share an XCD (see k_out_fwd_train)
  const int n_wg = (int)gridDim.x, nrb = n_wg / s_eff, wg = (int)blockIdx.x;
  const int v = xcd_order(wg, n_wg);
  const int split = v / nrb;
  const int t_begin = split * tiles_per_split;
  const int t_end = min(n_tiles, t_begin + tiles_per_split);
  const int t_last = t_end - 1;
  const int row0 = (v % nrb) * RB + wave * WROWS;
  const bool active = row0 < B;  // (waves past the batch only move W2 tiles)
  const W2Src src = w2_src(W2, b2, L);
  const int rbase[2] = {tw_row_base(n, g, 0), tw_row_base(n, g, 1)};

  // the rows' lists, best first; the first KR - k entries hold a key that nothing
  // displaces, so the k-th best is always the last entry
  double keys[NB][KR];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int j = 0; j < KR; ++j) keys[nb][j] = j < KR - k ? TOPK_FENCE : TOPK_EMPTY;
  Fr hf[NB][4][NCH];
  float thr[NB];  // the row's k-th best score so far (+inf: no such row, nothing reaches it)
  bool rvalid[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    // (rows past round_up(B, 32) of the buffer are not read)
    const int row = row0 + nb * 32 + n;
    rvalid[nb] = row < B;
    thr[nb] = rvalid[nb] ? -INFINITY : INFINITY;
    const E* hrow = H1 + (size_t)(row0 + nb * 32 < B ? row : n) * HID;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) hf[nb][kb][c] = h1_frag<BF16>(hrow, kb, c, g);
  }
  // the first P + 3 tiles, requested together
  TileRegs pre[P + 1], tr0, tr1;
#pragma unroll
  for (int u = 0; u <= P; ++u) tile_load(src, min(t_begin + u, t_last), pre[u]);
  tile_load(src, min(t_begin + P + 1, t_last), tr0);
  tile_load(src, min(t_begin + P + 2, t_last), tr1);
  // (the loop's wait counters then track only the W2 prefetch)
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(hf[nb][kb][c]));

  auto z_tile = [&](int buf, f32x16 (&z)[NB]) {
    const float4* bq = reinterpret_cast<const float4*>(bt[buf]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = bq[2 * q + g];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        z[nb][4 * q + 0] = b.x; z[nb][4 * q + 1] = b.y; z[nb][4 * q + 2] = b.z; z[nb][4 * q + 3] = b.w;
      }
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const Fr a = tile_frag_w<BF16>(wr[buf], rbase, n, kb, c, g);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) z[nb] = M::mma(a, hf[nb][kb][c], z[nb]);
      }
  };
  // Scores of tile t into the lists.  Most tiles hold none that reaches its row's
  // k-th: one maximum per row and a vote.
  auto rank = [&](int t, const f32x16 (&z)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float m = z[nb][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) m = fmaxf(m, z[nb][r]);  // (ignores NaN: those are never ranked)
      if (!__any(m >= thr[nb])) continue;
      unsigned hits = 0;  // registers with a score that reaches some row's list
#pragma unroll
      for (int r = 0; r < 16; ++r) hits |= __any(z[nb][r] >= thr[nb]) ? 1u << r : 0u;
#pragma unroll 1
      while (hits) {
        const int r = __builtin_ctz(hits);
        hits &= hits - 1;
        // the keys of the row's two lanes, on both (through integers, see half_swap_max)
        const uint64_t u = __builtin_bit_cast(
            uint64_t, topk_key(z[nb][r], t * OUT_TILE + 8 * (r >> 2) + 4 * g + (r & 3), L));
        const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
        const unsigned l0 = lo[0], l1 = lo[1], h0 = hi[0], h1 = hi[1];
        double c0 = __builtin_bit_cast(double, (uint64_t)h0 << 32 | l0);
        double c1 = __builtin_bit_cast(double, (uint64_t)h1 << 32 | l1);
#pragma unroll
        for (int j = 0; j < KR; ++j) {
          const double k0 = max_key(keys[nb][j], c0);
          c0 = min_key(keys[nb][j], c0);
          keys[nb][j] = max_key(k0, c1);
          c1 = min_key(k0, c1);
        }
        if (rvalid[nb]) thr[nb] = topk_score(keys[nb][KR - 1]);
      }
    }
  };

  // The pipeline of k_out_fwd_train: tile u lives in ring slot (u - t_begin) mod
  // NRING; the iteration of tile t issues the logits of t+1, ranks those of t,
  // stores tile t+P+1 (loaded two iterations earlier) and loads t+P+3; a barrier
  // closes every P-th iteration.  Indices are clamped to the split's last tile.
  auto slot = [&](int u) { return (u - t_begin) % NRING; };
#pragma unroll
  for (int u = 0; u <= P; ++u)
    tile_store<BF16, false>(pre[u], L, min(t_begin + u, t_last), wr[u], nullptr, bt[u]);
  __syncthreads();
  f32x16 z[NB], zn[NB];
  if (active) z_tile(0, z);
  auto iteration = [&](int t, TileRegs& tr, const f32x16 (&zc)[NB], f32x16 (&zx)[NB]) {
    const int bst = slot(t + P + 1);
    if (active) {
      z_tile(slot(t + 1), zx);
      rank(t, zc);
    }
    tile_store<BF16, false>(tr, L, min(t + P + 1, t_last), wr[bst], nullptr, bt[bst]);
    tile_load(src, min(t + P + 3, t_last), tr);
    if ((t - t_begin) % P == P - 1) __syncthreads();
  };
  for (int t = t_begin; t < t_end; t += 2) {
    iteration(t, tr0, z, zn);
    if (t + 1 >= t_end) break;
    iteration(t + 1, tr1, zn, z);
  }
  // row-major lists: the combine reads a row's candidates as one run
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if (!rvalid[nb] || g) continue;
    double* o = part + ((size_t)(row0 + nb * 32 + n) * s_eff + split) * k;
#pragma unroll
    for (int j = 0; j < KR; ++j)
      if (j >= KR - k) o[j - (KR - k)] = keys[nb][j];
  }
}

// Rows per wave and label splits of a prediction: one workgroup per CU over all
// row blocks (a small batch needs every CU to read W2: 50 rows of 30,000 labels
// took 110 us on 64 workgroups, and 16,384 rows of 670,091 labels 4.8 ms at 32
// rows per wave).
TopkShape topk_shape(bool use_bf16, int B, int k, int n_tiles, int n_cu) {
  TopkShape p;
  p.nb = use_bf16 && B > 256 && k <= TOPK_REG_K ? 2 : 1;
  const int rb = FwdShape<true>::WAVES * 32 * p.nb;
  p.nrb = (B + rb - 1) / rb;
  int s = (n_cu + p.nrb - 1) / p.nrb;
  if (s > n_tiles) s = n_tiles;
  p.tps = (n_tiles + s - 1) / s;
  p.splits = (n_tiles + p.tps - 1) / p.tps;
  return p;
}

hipError_t launch_out_fwd_topk(bool use_bf16, const float* W2, const float* b2, int L, const void* H1,
                               int B, const TopkShape& sh, int k, double* part, hipStream_t st) {
  const int n_tiles = (L + OUT_TILE - 1) / OUT_TILE;
  const dim3 grid(sh.splits * sh.nrb), block(FWD_THREADS);
  auto go = [&](auto kern, auto* h1) {
    hipLaunchKernelGGL(kern, grid, block, 0, st, W2, b2, L, h1, B, sh.tps, n_tiles, sh.splits, k, part);
    return hipGetLastError();
  };
  if (!use_bf16) {
    const float* h = (const float*)H1;
    if (k == 1) return go(k_out_fwd_topk<false, 1, 1>, h);
    return k <= TOPK_REG_K ? go(k_out_fwd_topk<false, 1, TOPK_REG_K>, h) : go(k_out_fwd_topk<false, 1, 32>, h);
  }
  const bf16* h = (const bf16*)H1;
  if (sh.nb == 2) return k == 1 ? go(k_out_fwd_topk<true, 2, 1>, h) : go(k_out_fwd_topk<true, 2, TOPK_REG_K>, h);
  if (k == 1) return go(k_out_fwd_topk<true, 1, 1>, h);
  return k <= TOPK_REG_K ? go(k_out_fwd_topk<true, 1, TOPK_REG_K>, h) : go(k_out_fwd_topk<true, 1, 32>, h);
}

// Final top-k of a row from its splits' sorted lists, by one wavefront: the
// row's keys come into LDS as one run, lane l keeps the heads of lists l, l + 64,
// ..., and each of the k rounds takes the best head and advances its list.
constexpr int TOPK_LISTS = 6;  // lists per lane: up to 384 splits

__global__ __launch_bounds__(64) void k_topk_combine(int splits, int k, const double* __restrict__ part,
                                                     int32_t* __restrict__ ids, float* __restrict__ scores) {
  extern __shared__ double ck[];
  const int i = blockIdx.x, lane = threadIdx.x;
  const int nc = splits * k;
  const double* pr = part + (size_t)i * nc;
  constexpr int BATCH = 8;  // keys in flight per lane (one latency per 512 of them)
  for (int e0 = lane; e0 < nc; e0 += 64 * BATCH) {
    double v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) v[j] = pr[min(e0 + 64 * j, nc - 1)];
#pragma unroll
    for (int j = 0; j < BATCH; ++j)
      if (e0 + 64 * j < nc) ck[e0 + 64 * j] = v[j];
  }
  __syncthreads();
  double head[TOPK_LISTS];
  int pos[TOPK_LISTS];
#pragma unroll
  for (int j = 0; j < TOPK_LISTS; ++j) {
    const int l = lane + 64 * j;
    pos[j] = 0;
    head[j] = l < splits ? ck[l * k] : TOPK_EMPTY;
  }
  for (int out = 0; out < k; ++out) {
    double best = head[0];
#pragma unroll
    for (int j = 1; j < TOPK_LISTS; ++j) best = max_key(best, head[j]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) best = max_key(best, __shfl_xor(best, o));
    const bool none = best == TOPK_EMPTY;  // other keys are unique: the winner's list is the one with this head
#pragma unroll
    for (int j = 0; j < TOPK_LISTS; ++j)
      if (!none && head[j] == best) head[j] = ++pos[j] < k ? ck[(lane + 64 * j) * k + pos[j]] : TOPK_EMPTY;
    if (lane == 0) {
      ids[(size_t)i * k + out] = none ? TOPK_NONE : topk_id(best);
      if (scores) scores[(size_t)i * k + out] = none ? -INFINITY : topk_score(best);
    }
  }
}

hipError_t launch_topk_combine(int B, int splits, int k, const double* part, int32_t* ids, float* scores,
                               hipStream_t st) {
  if (splits > 64 * TOPK_LISTS) return hipErrorInvalidValue;
  const size_t shm = (size_t)splits * k * sizeof(double);
  if (shm > 64 * 1024) {  // (above the default limit of a launch: 256 splits of more than 32 entries)
    const hipError_t e =
        hipFuncSetAttribute((const void*)k_topk_combine, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_topk_combine, dim3(B), dim3(64), shm, st, splits, k, part, ids, scores);
  return hipGetLastError();
}

}  // namespace asgd
