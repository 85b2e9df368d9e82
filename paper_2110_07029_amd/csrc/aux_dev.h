// Device bodies of the index work of a training step, written for workgroups
// that can ride along inside a larger launch instead of needing launches, and a
// cross-stream event, of their own: the label grouping (one workgroup of the
// output-layer forward's launch) and a pass of the feature sort (workgroups of
// the forward's and of the per-row launch after it).
#pragma once

#include "asgd_dev.h"

namespace asgd {

// Exclusive scan of one int per thread over the workgroup (NT threads), plus
// the total; wsum: NT/64 ints of LDS.  Ends with a barrier, so wsum can be
// reused right after.
template <int NT>
__device__ __forceinline__ int wg_exclusive_scan(int x, int* wsum, int* total) {
  constexpr int W = NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const int v = wsum[k];
    before += k < w ? v : 0;
    all += v;
  }
  __syncthreads();
  *total = all;
  return before + inc - x;
}

// (row, label) pairs grouped by 32-label block by one workgroup of NT
// threads: a counter per block (cnt: LDS when LDS, else global memory of
// ceil(L/32) ints), an exclusive scan into lbeg, then every valid pair is
// placed in its block's range.  lbeg[b] .. lbeg[b+1] (b < ceil(L/32)) is
// block b's range of lpair, each entry (row << 5) | (label % 32); invalid
// labels (key L) are dropped.  The order of the pairs inside a block is not
// fixed: the backward only ORs them into a bit mask, whose value does not
// depend on it.  wsum: NT/64 ints of LDS.
template <bool LDS>
__device__ __forceinline__ int lb_load(const int32_t* p) {
  if constexpr (LDS)
    return *p;
  else  // counters updated by atomics at L2: read past the L1
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool LDS>
__device__ __forceinline__ void lb_sync() {
  if constexpr (!LDS) __threadfence();
  __syncthreads();
}

template <int NT, bool LDS>
__device__ void wg_label_blocks(const int32_t* __restrict__ lkeys, int m, int L,
                                const int32_t* __restrict__ lrow, int32_t* __restrict__ lbeg,
                                int32_t* __restrict__ lpair, int32_t* cnt, int32_t* wsum) {
  const int nb = (L + 31) >> 5;
  const int t = threadIdx.x;
  for (int b = t; b < nb; b += NT) cnt[b] = 0;
  lb_sync<LDS>();
  for (int q = t; q < m; q += NT) {
    const int lab = lkeys[q];
    if (lab >= 0 && lab < L) atomicAdd(&cnt[lab >> 5], 1);
  }
  lb_sync<LDS>();
  // thread t owns the contiguous blocks [t*per, t*per + per)
  const int per = (nb + NT - 1) / NT;
  const int b0 = min(nb, t * per), b1 = min(nb, b0 + per);
  int local = 0;
  for (int b = b0; b < b1; ++b) local += lb_load<LDS>(cnt + b);
  int total;
  int run = wg_exclusive_scan<NT>(local, wsum, &total);
  for (int b = b0; b < b1; ++b) {
    const int c = lb_load<LDS>(cnt + b);
    lbeg[b] = run;
    cnt[b] = run;  // becomes the block's fill cursor
    run += c;
  }
  if (t == 0) lbeg[nb] = total;
  lb_sync<LDS>();
  for (int q = t; q < m; q += NT) {
    const int lab = lkeys[q];
    if (lab >= 0 && lab < L) {
      const int pos = atomicAdd(&cnt[lab >> 5], 1);
      lpair[pos] = (lrow[q] << 5) | (lab & 31);
    }
  }
}

// One pass of the stable radix sort over digit d = (key >> shift) & (2^nbits - 1),
// for chunk c of NT * per_thread keys, without any launch or exchange between
// workgroups: the workgroup itself counts all n < 2^16 keys by digit (every digit's
// total and its count before the chunk, as the halves of one LDS counter), scans the
// totals, ranks its own keys by 64-lane ballots and running counts per wave, and
// scatters them.  Every workgroup counts all the keys (LDS atomics, about one per clock
// and CU), so this is for small batches: 18,600 keys take about as long as a short
// output layer, beside which they cost nothing; 79,000 take several times a pass of
// k_sort.hip.  Beside the shorter per-row launch the counting decided (10.4 us for 18,600
// keys, 6.7 without the sort), so pass 0 adds up pass 1's counts per chunk in memory as
// its keys land, and pass 1 reads those.
// lds: sort_pass_lds(nbits, NT) bytes, 16-byte aligned.
template <int NT>
__device__ void wg_sort_pass(const SortJob& j, int c, int32_t* lds) {
  constexpr int W = NT / 64;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int nd = 1 << j.nbits, mask = nd - 1, n = j.n;
  unsigned* cnt = reinterpret_cast<unsigned*>(lds);                    // [nd]: total | before the chunk << 16
  unsigned short* wcnt = reinterpret_cast<unsigned short*>(cnt + nd);  // [W][nd]: this chunk's, by wave
  int* wsum = reinterpret_cast<int*>(wcnt + W * nd);                   // [W]
  const int32_t* __restrict__ keys = j.keys_in;
  const int c0 = c * NT * j.per_thread;
  const int p0 = c0 + w * 64 * j.per_thread + lane;  // a wave's keys are consecutive
  for (int d = t; d < nd; d += NT) cnt[d] = 0;  // (before the barrier; the counts come after it)
  for (int d = t; d < W * nd / 2; d += NT) reinterpret_cast<unsigned*>(wcnt)[d] = 0;
  __syncthreads();
  if (j.hist && j.next_chunk == 0) {
    // pass 1: pass 0 has left the counts of every chunk
    const int nc = (n + NT * j.per_thread - 1) / (NT * j.per_thread);
    for (int d = t; d < nd; d += NT) {
      unsigned tot = 0, bef = 0;
      constexpr int BATCH = 16;  // counts in flight
      for (int b0 = 0; b0 < nc; b0 += BATCH) {
        int v[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) v[u] = j.hist[min(b0 + u, nc - 1) * nd + d];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          tot += b0 + u < nc ? v[u] : 0;
          bef += b0 + u < c ? v[u] : 0;
        }
      }
      cnt[d] = tot | bef << 16;
    }
  } else {
    // four keys per 16-byte load, BATCH loads in flight
    constexpr int BATCH = 8;
    const int n4 = n >> 2;
    auto count = [&](int k, int q) {
      atomicAdd(&cnt[(k >> j.shift) & mask], q < c0 ? 0x10001u : 1u);
    };
    for (int q0 = t; q0 < n4; q0 += NT * BATCH) {
      int4 v[BATCH];
  #pragma unroll
      for (int u = 0; u < BATCH; ++u) v[u] = reinterpret_cast<const int4*>(keys)[min(q0 + u * NT, n4 - 1)];
  #pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int q = q0 + u * NT;
        if (q < n4) {  // (a chunk starts at a multiple of four keys: all four lie on one side of it)
          count(v[u].x, 4 * q);
          count(v[u].y, 4 * q);
          count(v[u].z, 4 * q);
          count(v[u].w, 4 * q);
        }
      }
    }
    if (4 * n4 + t < n) count(keys[4 * n4 + t], 4 * n4 + t);
  }
  // lanes of the wave with the same digit
  auto peers_of = [&](int d, bool valid) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < j.nbits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    return peers;
  };
  const uint64_t below = (1ull << lane) - 1ull;
  for (int it = 0; it < j.per_thread; ++it) {
    const int p = p0 + 64 * it;
    const bool valid = p < n;
    const int d = ((valid ? keys[p] : 0) >> j.shift) & mask;
    const uint64_t peers = peers_of(d, valid);
    if (valid && (peers & below) == 0) wcnt[w * nd + d] += (unsigned short)__popcll(peers);
  }
  __syncthreads();
  // exclusive scan of the totals, over contiguous digits per thread
  const int per = (nd + NT - 1) / NT;
  const int d0 = min(nd, t * per), d1 = min(nd, d0 + per);
  int local = 0;
  for (int x = d0; x < d1; ++x) local += (int)(cnt[x] & 0xffffu);
  int total;
  int run = wg_exclusive_scan<NT>(local, wsum, &total);
  for (int x = d0; x < d1; ++x) {
    const unsigned v = cnt[x];
    cnt[x] = (unsigned)run + (v >> 16);  // the chunk's first position of digit x
    run += (int)(v & 0xffffu);
    int sum = 0;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      const int m = wcnt[ww * nd + x];
      wcnt[ww * nd + x] = (unsigned short)sum;
      sum += m;
    }
  }
  __syncthreads();
  for (int it = 0; it < j.per_thread; ++it) {
    const int p = p0 + 64 * it;
    const bool valid = p < n;
    const int key = valid ? keys[p] : 0;
    const int val = valid ? (j.vals_in ? j.vals_in[p] : p) : 0;
    const int d = (key >> j.shift) & mask;
    const uint64_t peers = peers_of(d, valid);
    const int before = __popcll(peers & below);
    const int c = wcnt[w * nd + d];  // every peer reads the count before the leader updates it
    if (valid && before == 0) wcnt[w * nd + d] = (unsigned short)(c + __popcll(peers));
    if (valid) {
      const int pos = (int)cnt[d] + c + before;
      j.keys_out[pos] = key;
      j.vals_out[pos] = val;
      if (j.next_chunk > 0)
        atomicAdd(&j.hist[(pos / j.next_chunk << j.next_nbits) | (key >> j.next_shift & ((1 << j.next_nbits) - 1))], 1);
    }
  }
}

// ---- joining the sparse update's segments that cross windows ----------------------
// (k_sparse.hip; also workgroups of the backward's launch)
constexpr int SPU_WIN = 32;      // sorted entries per window
constexpr int JOIN_BATCH = 16;   // continuing pieces loaded together
constexpr int JOIN_WINDOWS = 8;  // windows per wavefront beside the backward (their joins run one after the other)

// Windows [first, first + COUNT) by one wavefront: a window whose last entry's
// segment starts in it and runs past its end adds the segment's pieces (its own
// part[2w + 1], then part[2v] of the windows v after it, in order) and applies the sum
// to W1.  One lane looks at each window; the heads found are joined in turn.
template <int COUNT>
__device__ __forceinline__ void wave_join_windows(const JoinJob& j, int first) {
  const int lane = threadIdx.x & 63;
  const int32_t* __restrict__ skeys = j.skeys;
  const int n_keys = j.n_keys, F = j.F;
  const int w0 = (first + lane) * SPU_WIN;
  int f = F;
  if (lane < COUNT && w0 + SPU_WIN < n_keys) {
    const int last = skeys[w0 + SPU_WIN - 1], next = skeys[w0 + SPU_WIN];
    const int head = skeys[w0], before = w0 > 0 ? skeys[w0 - 1] : -1;
    // (a segment that continues from the window before is joined by an earlier one)
    if (last < F && next == last && !(head == last && before == last)) f = last;
  }
  uint64_t heads = __ballot(f < F);
  while (heads) {
    const int src = __builtin_ctzll(heads);
    heads &= heads - 1;
    const int fw = __builtin_amdgcn_readlane(f, src), win = first + src;
    const float2* P = reinterpret_cast<const float2*>(j.part) + lane;
    float2* wp = reinterpret_cast<float2*>(j.W1 + (size_t)fw * HID) + lane;
    const float2 w = *wp;
    float2 acc = P[(size_t)(2 * win + 1) * (HID / 2)];
    // windows win+1 .. win+m hold the rest: window v is followed by another piece when it
    // is all fw and the next window starts with fw (one lane per window)
    int m = 0;
    for (;;) {
      const int v1 = (win + 2 + m + lane) * SPU_WIN;  // first entry after window win+1+m+lane
      const bool more = v1 < n_keys && skeys[v1] == fw && skeys[v1 - 1] == fw;
      const uint64_t stop = __ballot(!more);
      if (stop) {
        m += __builtin_ctzll(stop) + 1;
        break;
      }
      m += 64;
    }
    for (int v0 = 0; v0 < m; v0 += JOIN_BATCH) {
      float2 c[JOIN_BATCH];
#pragma unroll
      for (int k = 0; k < JOIN_BATCH; ++k) c[k] = P[(size_t)(2 * (win + 1 + min(v0 + k, m - 1))) * (HID / 2)];
#pragma unroll
      for (int k = 0; k < JOIN_BATCH; ++k)
        if (v0 + k < m) {
          acc.x += c[k].x;
          acc.y += c[k].y;
        }
    }
    *wp = make_float2(fmaf(-j.lr, acc.x, w.x), fmaf(-j.lr, acc.y, w.y));
  }
}

// ---- the second hidden layer, one row in the workgroup that has it ------------------
// A2 = relu(A1) Wh^T + bh for one row, by 256 threads of the workgroup (t < 256 work, the
// others only pass): thread (o, half) sums 64 inputs of unit o.  h_s: relu(A1) in LDS,
// written before a barrier.  Returns the unit's A2 on both halves.
__device__ __forceinline__ float dense_row_unit(const float* __restrict__ Wh, const float* __restrict__ bh,
                                                const float* h_s, int t) {
  const int o = t >> 1, k0 = (t & 1) * (HID / 2);
  const float4* w = reinterpret_cast<const float4*>(Wh + (size_t)o * HID + k0);
  float acc = t & 1 ? 0.0f : bh[o];
#pragma unroll
  for (int k = 0; k < HID / 8; ++k) {
    const float4 v = w[k];
    const float4 h = *reinterpret_cast<const float4*>(h_s + k0 + 4 * k);
    acc = fmaf(v.x, h.x, acc);
    acc = fmaf(v.y, h.y, acc);
    acc = fmaf(v.z, h.z, acc);
    acc = fmaf(v.w, h.w, acc);
  }
  return acc + __shfl_xor(acc, 1);
}

// dWh[o][k] = sum_r dA2[r][o] relu(A1[r][k]) and dbh[o] = sum_r dA2[r][o], in row order;
// then the update in place.  One workgroup of 256 threads: output units 2 bid and 2 bid + 1
// x 128 input units; the rows come through LDS in chunks of 64, the next chunk's loads in
// flight while one is summed (a chunk's load latency is longer than its sums).
constexpr int WGRAD_WGS = HID / 2;
__device__ inline void dense_wgrad_wg(const DenseWgrad& wg, int B, float lr, int bid) {
  constexpr int CHUNK = 64, NT = 2 * HID, LD = CHUNK * HID / 4 / NT;  // 8 float4 per thread
  __shared__ float hs[CHUNK][HID];
  __shared__ float ds[CHUNK][2];
  const int tid = threadIdx.x;
  const int k = tid % HID, half = tid / HID;
  const int o = bid * 2 + half;
  typedef float v4 __attribute__((ext_vector_type(4)));
  v4 a[LD];
  float d = 0.0f;
  auto load = [&](int c0) {  // (rows past B: the last one, multiplied by a zero dA2)
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      const int e = tid + u * NT, r = min(c0 + e / (HID / 4), B - 1);
      a[u] = *reinterpret_cast<const v4*>(wg.A1 + (size_t)r * HID + 4 * (e % (HID / 4)));
    }
    const int r = c0 + tid / 2;
    d = tid < 2 * CHUNK && r < B ? wg.dA2[(size_t)r * HID + bid * 2 + tid % 2] : 0.0f;
  };
  load(0);
  const float w_old = wg.Wh[o * HID + k], b_old = wg.bh[o];
  float acc = 0.0f, db = 0.0f;
  for (int c0 = 0; c0 < B; c0 += CHUNK) {
    __syncthreads();  // the previous chunk is consumed
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      float* p = &hs[0][0] + 4 * (tid + u * NT);
      p[0] = fmaxf(a[u].x, 0.0f); p[1] = fmaxf(a[u].y, 0.0f); p[2] = fmaxf(a[u].z, 0.0f); p[3] = fmaxf(a[u].w, 0.0f);
    }
    if (tid < 2 * CHUNK) ds[tid / 2][tid % 2] = d;
    __syncthreads();
    if (c0 + CHUNK < B) load(c0 + CHUNK);
#pragma unroll 8
    for (int r = 0; r < CHUNK; ++r) {
      const float dv = ds[r][half];
      acc = fmaf(dv, hs[r][k], acc);
      db += dv;
    }
  }
  wg.Wh[o * HID + k] = fmaf(-lr, acc, w_old);
  if (k == 0) wg.bh[o] = fmaf(-lr, db, b_old);
}

}  // namespace asgd
