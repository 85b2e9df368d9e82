// Stable LSD radix sort of int32 keys with their original positions as the
// payload.  It orders the batch's feature entries so that the sparse W1
// gradient becomes a segmented reduction over equal feature ids (no contended
// atomics, fixed summation order).
//
// One pass over a digit of up to 11 bits:
//   hist    : per-workgroup digit counts of a 1024-key chunk (LDS counters),
//             stored block-major: hist[block][digit]
//   scatter : every workgroup sums the digits' counts (all chunks' and those before
//             its own) and scans them into its scatter offsets; stable ranks inside
//             the chunk from 64-lane ballots (lanes with the same digit in one wave),
//             per-wave running counts, then a prefix over the four waves; keys land
//             at offset + rank.
// Every workgroup that sums reads all chunks' counts (up to 4 KB per chunk), which beside the
// output layer's launches, on the few CUs and registers these leave, costs more than it saves
// from about SORT_SCAN_COUNTS on: from there a launch of its own (scan, one workgroup) forms the
// offsets.  us per step, summing in the scatter | in a launch, one model by itself and three in
// turn: 79,000 keys of 20 bits (10-bit digits, 79,000 counts) L = 100,000 128 | 132, 113 | 110;
// 120,000 keys of 20 bits L = 100,000 190 | 136, 142 | 138, L = 30,000 142 | 126, 100 | 99;
// 87,000 keys of 17 bits (44,000 counts) 99 | 101, 88 | 91; 72,000 keys of 15 bits (18,000
// counts) three in turn 113 | 116; 46,000 keys of 20 bits (46,000 counts) 109 | 110.
// hist and scatter size their LDS by the pass's digit width (dynamic LDS, 4 << bits
// and 12 << bits bytes), not by the widest digit: a narrow pass then fits on a CU
// beside the output-layer kernels of the other stream.
#include "asgd_dev.h"
#include "asgd_kernels.h"

namespace asgd {

constexpr int SORT_THREADS = 256;
constexpr int SORT_WAVES = SORT_THREADS / 64;
constexpr int SORT_PER_WAVE = SORT_CHUNK / SORT_WAVES;  // 256
constexpr int SORT_ITERS = SORT_PER_WAVE / 64;         // 4

int sort_blocks(int n) { return (n + SORT_CHUNK - 1) / SORT_CHUNK; }

__global__ __launch_bounds__(SORT_THREADS) void k_sort_hist(const int32_t* __restrict__ keys, int n,
                                                            int shift, int nbits, int nblk,
                                                            int32_t* __restrict__ hist) {
  extern __shared__ int cnt[];  // 1 << nbits counters
  const int nd = 1 << nbits;
  for (int d = threadIdx.x; d < nd; d += SORT_THREADS) cnt[d] = 0;
  __syncthreads();
  const int b0 = blockIdx.x * SORT_CHUNK;
  for (int t = threadIdx.x; t < SORT_CHUNK; t += SORT_THREADS) {
    const int p = b0 + t;
    if (p < n) atomicAdd(&cnt[(keys[p] >> shift) & (nd - 1)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < nd; d += SORT_THREADS) hist[blockIdx.x * nd + d] = cnt[d];
}

// Scatter offsets offs[b * ndig + d] = (keys with a smaller digit) + (keys with
// digit d in earlier chunks), by one workgroup: thread t owns digits t and
// t + SCAN_THREADS; per chunk b, the threads read consecutive digits (one
// coalesced row of hist), and one block-wide exclusive scan of the per-digit
// totals gives every digit's base.
constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_DPT = (1 << SORT_MAX_BITS) / SCAN_THREADS;  // digits per thread
constexpr int SCAN_BATCH = 16;  // chunk counts loaded together

__global__ __launch_bounds__(SCAN_THREADS) void k_sort_scan(const int32_t* __restrict__ hist,
                                                            int nblk, int ndig,
                                                            int32_t* __restrict__ offs) {
  __shared__ int wsum[SCAN_THREADS / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // (the chunks' counts are read SCAN_BATCH at a time, all loads in flight
  // before the first sum)
  int tot[SCAN_DPT];
#pragma unroll
  for (int k = 0; k < SCAN_DPT; ++k) tot[k] = 0;
#pragma unroll
  for (int k = 0; k < SCAN_DPT; ++k) {
    const int d = t + k * SCAN_THREADS;
    if (d >= ndig) continue;
    for (int b0 = 0; b0 < nblk; b0 += SCAN_BATCH) {
      int c[SCAN_BATCH];
#pragma unroll
      for (int j = 0; j < SCAN_BATCH; ++j) c[j] = b0 + j < nblk ? hist[(size_t)(b0 + j) * ndig + d] : 0;
#pragma unroll
      for (int j = 0; j < SCAN_BATCH; ++j) tot[k] += c[j];
    }
  }
  // digits in order d = t + k * SCAN_THREADS: scan the block once per k
  int carry = 0;
#pragma unroll
  for (int k = 0; k < SCAN_DPT; ++k) {
    int x = tot[k];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    if (w == 0) {
      int v = lane < SCAN_THREADS / 64 ? wsum[lane] : 0;
#pragma unroll
      for (int o = 1; o < SCAN_THREADS / 64; o <<= 1) {
        const int y = __shfl_up(v, o);
        if (lane >= o) v += y;
      }
      if (lane < SCAN_THREADS / 64) wsum[lane] = v;
    }
    __syncthreads();
    const int base = carry + (w > 0 ? wsum[w - 1] : 0) + x - tot[k];
    carry += wsum[SCAN_THREADS / 64 - 1];
    __syncthreads();
    tot[k] = base;  // becomes the running offset of digit t + k * SCAN_THREADS
  }
#pragma unroll
  for (int k = 0; k < SCAN_DPT; ++k) {
    const int d = t + k * SCAN_THREADS;
    if (d >= ndig) continue;
    for (int b0 = 0; b0 < nblk; b0 += SCAN_BATCH) {
      int c[SCAN_BATCH];
#pragma unroll
      for (int j = 0; j < SCAN_BATCH; ++j) c[j] = b0 + j < nblk ? hist[(size_t)(b0 + j) * ndig + d] : 0;
#pragma unroll
      for (int j = 0; j < SCAN_BATCH; ++j)
        if (b0 + j < nblk) {
          offs[(size_t)(b0 + j) * ndig + d] = tot[k];
          tot[k] += c[j];
        }
    }
  }
}

constexpr int SORT_SCAN_COUNTS = 48 << 10;  // (chunk, digit) counts

// offs: the scan's offsets, or null: this workgroup forms its own from hist.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(SortJob j, int nblk, const int32_t* __restrict__ hist,
                                                               const int32_t* __restrict__ offs) {
  extern __shared__ int lds_sc[];
  const int nd = 1 << j.nbits, mask = nd - 1, n = j.n;
  int* base = lds_sc;  // [nd]: the chunk's first position of every digit
  unsigned short* wcnt_lds = reinterpret_cast<unsigned short*>(base + nd);  // [SORT_WAVES][nd]
  __shared__ int wsum[SORT_WAVES];
  auto wcnt = [&](int ww, int d) -> unsigned short& { return wcnt_lds[ww * nd + d]; };
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, blk = blockIdx.x;
  const int p0 = blk * SORT_CHUNK + w * SORT_PER_WAVE;
  int key[SORT_ITERS], val[SORT_ITERS], rank[SORT_ITERS];
#pragma unroll
  for (int it = 0; it < SORT_ITERS; ++it) {
    const int p = p0 + it * 64 + lane;
    key[it] = p < n ? j.keys_in[p] : 0;
    val[it] = p < n ? (j.vals_in ? j.vals_in[p] : p) : 0;
  }
  for (int d = lane; d < nd; d += 64) wcnt(w, d) = 0;
  if (offs) {
    for (int d = t; d < nd; d += SORT_THREADS) base[d] = offs[(size_t)blk * nd + d];
  } else {
    int carry = 0;
    for (int d0 = 0; d0 < nd; d0 += SORT_THREADS) {
      const int d = d0 + t;
      int tot = 0, bef = 0;
      constexpr int BATCH = 16;  // chunk counts in flight
      for (int b0 = 0; b0 < nblk; b0 += BATCH) {
        int c[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) c[k] = d < nd ? hist[(size_t)min(b0 + k, nblk - 1) * nd + d] : 0;
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
          tot += b0 + k < nblk ? c[k] : 0;
          bef += b0 + k < blk ? c[k] : 0;
        }
      }
      // exclusive scan of the totals over the workgroup's digits
      int inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
      }
      if (lane == 63) wsum[w] = inc;
      __syncthreads();
      int before = carry;
#pragma unroll
      for (int k = 0; k < SORT_WAVES; ++k) {
        before += k < w ? wsum[k] : 0;
        carry += wsum[k];
      }
      if (d < nd) base[d] = before + inc - tot + bef;
      __syncthreads();
    }
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int it = 0; it < SORT_ITERS; ++it) {
    const bool valid = p0 + it * 64 + lane < n;
    const int d = (key[it] >> j.shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < j.nbits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const int before = __popcll(peers & below);
    const int c = wcnt(w, d);  // every peer reads the count before the leader updates it
    rank[it] = c + before;
    if (valid && before == 0) wcnt(w, d) = (unsigned short)(c + __popcll(peers));
  }
  __syncthreads();
  for (int d = t; d < nd; d += SORT_THREADS) {
    int run = 0;
#pragma unroll
    for (int ww = 0; ww < SORT_WAVES; ++ww) {
      const int c = wcnt(ww, d);
      wcnt(ww, d) = (unsigned short)run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < SORT_ITERS; ++it) {
    if (p0 + it * 64 + lane < n) {
      const int d = (key[it] >> j.shift) & mask;
      const int pos = base[d] + wcnt(w, d) + rank[it];
      j.keys_out[pos] = key[it];
      j.vals_out[pos] = val[it];
    }
  }
}

int sort_spread(SortJob* job, int nthreads, int wgs) {
  const int keys = nthreads * (wgs > 1 ? wgs : 1);
  job->per_thread = (job->n + keys - 1) / keys;
  if (job->per_thread > 127) job->per_thread = 127;  // what the 16-bit counters hold
  const int chunk = nthreads * job->per_thread;
  return (job->n + chunk - 1) / chunk;
}

int sort_plan_ride(SortPlan* plan, int nthreads1, int wgs1, int32_t* hist) {
  if (plan->passes < 2) return 0;
  SortJob &p0 = plan->pass[0], &p1 = plan->pass[1];
  sort_spread(&p1, nthreads1, wgs1);
  // Few keys are counted faster than the counts are cleared, added up and read: us per step
  // with them | without, at 2,500 keys 43.0 | 42.3, 15,200 52.9 | 52.9, 18,600 53.9 | 55.4,
  // 44,300 128.2 | 132.3.
  if (p1.n < 16384) return 0;
  // chunks of at least two keys per thread (SORT_CHUNK): their counts then fit hist
  const int most = p1.n / (2 * nthreads1);
  sort_spread(&p1, nthreads1, wgs1 < most ? wgs1 : most);
  const int chunk = nthreads1 * p1.per_thread;
  p0.hist = p1.hist = hist;
  p0.next_chunk = chunk;
  p0.next_shift = p1.shift;
  p0.next_nbits = p1.nbits;
  return ((p1.n + chunk - 1) / chunk) << p1.nbits;
}

int sort_pass_lds(int nbits, int nthreads) {
  const int nd = 1 << nbits, w = nthreads / 64;
  return nd * 4 + w * nd * 2 + w * 4;
}

SortPlan sort_plan(const int32_t* keys_in, int n, int key_bits, int32_t* keys_a, int32_t* vals_a, int32_t* keys_b,
                   int32_t* vals_b) {
  SortPlan p{};
  p.keys_out = keys_a;
  p.vals_out = vals_a;
  if (n <= 0) return p;
  if (key_bits < 1) key_bits = 1;
  p.passes = key_bits > SORT_MAX_BITS ? 2 : 1;  // (key_bits <= 2 * SORT_MAX_BITS)
  const int bits = (key_bits + p.passes - 1) / p.passes;
  p.pass[0] = SortJob{keys_in, nullptr, n, 0, bits, keys_a, vals_a, 1, nullptr, 0, 0, 0};
  if (p.passes == 2) {
    p.pass[1] = SortJob{keys_a, vals_a, n, bits, key_bits - bits, keys_b, vals_b, 1, nullptr, 0, 0, 0};
    p.keys_out = keys_b;
    p.vals_out = vals_b;
  }
  return p;
}

hipError_t launch_sort(const SortPlan& plan, int32_t* hist, hipStream_t st) {
  for (int k = 0; k < plan.passes; ++k) {
    const SortJob& j = plan.pass[k];
    const int nblk = sort_blocks(j.n);
    const int32_t* offs = nullptr;
    hipLaunchKernelGGL(k_sort_hist, dim3(nblk), dim3(SORT_THREADS), (size_t)4 << j.nbits, st, j.keys_in, j.n, j.shift,
                       j.nbits, nblk, hist);
    if (nblk << j.nbits >= SORT_SCAN_COUNTS) {
      int32_t* o = hist + ((size_t)nblk << SORT_MAX_BITS);
      hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(SCAN_THREADS), 0, st, hist, nblk, 1 << j.nbits, o);
      offs = o;
    }
    // (nd offsets of 4 bytes and SORT_WAVES x nd counters of 2)
    hipLaunchKernelGGL(k_sort_scatter, dim3(nblk), dim3(SORT_THREADS), (size_t)(4 + 2 * SORT_WAVES) << j.nbits, st, j,
                       nblk, (const int32_t*)hist, offs);
  }
  return hipGetLastError();
}

}  // namespace asgd
