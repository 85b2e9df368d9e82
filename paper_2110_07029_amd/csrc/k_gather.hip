// First layer: CSR batch times W1 as coalesced row gathers (sparse input layer
// of the paper's MLP, Sec. 5.1), plus the per-entry sort keys used by the
// backward pass and the model initialisation.
#include <hip/hip_ext.h>

#include <type_traits>

#include "asgd_dev.h"
#include "asgd_kernels.h"
#include "aux_dev.h"

namespace asgd {

// ---------------------------------------------------------------------------
// Xavier-uniform init from the counter-based splitmix64 stream.
// ---------------------------------------------------------------------------
__global__ void k_init_uniform(float* __restrict__ w, int64_t count, uint64_t key, float bound) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += stride) {
    uint64_t z = (uint64_t)e ^ key;
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    const float u = (float)(uint32_t)(z >> 40) * 0x1p-24f;  // exact: 24-bit grid
    const float t = 2.0f * u - 1.0f;                          // exact in float32
    w[e] = t * bound;                                         // the only rounding
  }
}

hipError_t launch_init_uniform(float* w, int64_t count, uint64_t key, float bound, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_init_uniform, dim3((unsigned)blocks), dim3(256), 0, st, w, count, key, bound);
  return hipGetLastError();
}

__global__ void k_fill_int(int32_t* p, int32_t v, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) p[e] = v;
}

hipError_t launch_fill_int(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_int, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A1[i] = b1 + sum_{(f, v) in row i} v * W1[f];  H1 = max(A1, 0).
// One workgroup per sample row; for batches whose rows average
// GATHER_LONG_ROW entries or more, GATHER_SPLIT workgroups per row, each
// writing its partial sum, and a second launch adds them (the step time
// follows the longest row, which then spreads over several CUs).  Lane l owns
// hidden units 2l and 2l+1, so every W1 row is one coalesced 512-byte access.
// The row's entries are split into one contiguous range per wavefront; a wavefront
// loads up to 64 (id, value) pairs at once (one per lane, also writing their
// sort keys), broadcasts them with readlane and issues 16 W1 row loads before
// the first is used.  Lanes past the range carry id -1, so a partial group of
// 16 costs one round trip like a full one (the step time follows the longest
// row of the batch, and nnz per row is heavy-tailed).  The partial sums are
// added in wavefront order (then in workgroup order), then b1.
// ---------------------------------------------------------------------------
// Beside the backward of a pipelined step: four wavefronts (one per SIMD), so that
// the workgroup can start on a CU where the output-layer backward leaves room for
// only one more wavefront per SIMD.  Alone on the model's stream, up to
// GATHER_WIDE_ROWS rows: eight, as the longest row decides (15.3 -> 10.5 us for 256
// rows of 75 entries on average, 10.7 -> 8.6 for 50; 2,000 rows: equal; 16,384 rows,
// which fill the GPU: 78 -> 107; sixteen: slower from 600 rows on).  Long rows split
// over workgroups: eight.
constexpr int GATHER_WIDE_ROWS = 2048;
constexpr int GATHER_UNROLL = 16;
static_assert(64 % GATHER_UNROLL == 0, "readlane indices stay below 64");

// Unit t / 2 of row i's second hidden layer, by thread t of 256 (h_s: relu(A1) in LDS).
template <bool BF16>
__device__ __forceinline__ void dense_row_store(const DenseFwd& dn, const float* h_s, int i, int t,
                                                typename Mma<BF16>::elem* H1, typename Mma<BF16>::elem* H1T,
                                                int ld_t) {
  const float a2 = dense_row_unit(dn.Wh, dn.bh, h_s, t);
  if (t & 1) return;
  const int o = t >> 1;
  dn.A2[(size_t)i * HID + o] = a2;
  const float h = fmaxf(a2, 0.0f);
  H1[(size_t)i * HID + o] = (typename Mma<BF16>::elem)h;
  if constexpr (!BF16) H1T[(size_t)o * ld_t + i] = h;
}

// DENSE: the workgroup that has a row's A1 also forms the row's second hidden layer
// (A2 = relu(A1) Wh^T + bh; Wh comes from L2) and writes relu(A2) as the operand.
template <bool BF16, int SPLIT, int WAVES, bool DENSE>
__global__ __launch_bounds__(64 * WAVES) void k_gather_fwd(
    CsrDev x, CsrDev y, int has_y, const float* __restrict__ W1, const float* __restrict__ b1,
    int F, int L, float* __restrict__ A1, typename Mma<BF16>::elem* __restrict__ H1,
    typename Mma<BF16>::elem* __restrict__ H1T, int rows_pad, int ld_t, int32_t* __restrict__ keys,
    int32_t* __restrict__ row_of, int32_t* __restrict__ lkeys, int32_t* __restrict__ lrow,
    float* __restrict__ rw,
    int32_t* __restrict__ err, int validate, float* __restrict__ gpart, DenseFwd dn,
    int32_t* __restrict__ zero, int n_zero) {
  static_assert(!DENSE || SPLIT == 1, "split rows: k_gather_finish");
  using E = typename Mma<BF16>::elem;
  __shared__ float2 part[WAVES][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = (int)blockIdx.x / SPLIT, piece = (int)blockIdx.x % SPLIT;
  const int h0 = 2 * lane;
  for (int e = (int)blockIdx.x * (64 * WAVES) + (int)threadIdx.x; e < n_zero; e += (int)gridDim.x * (64 * WAVES))
    zero[e] = 0;
  if (i >= x.n_rows) {  // padding rows of the output-layer operands are zero
    if (wave == 0 && piece == 0) {
      H1[(size_t)i * HID + h0] = (E)0.0f;
      H1[(size_t)i * HID + h0 + 1] = (E)0.0f;
      if constexpr (!BF16) {  // the transposed copy is read only by the fp32 backward
        H1T[(size_t)h0 * ld_t + i] = (E)0.0f;
        H1T[(size_t)(h0 + 1) * ld_t + i] = (E)0.0f;
      }
    }
    return;
  }
  int bad = 0;
  const int base = x.indptr[0];
  int s = x.indptr[i], e = x.indptr[i + 1];
  if (s < base || e > base + x.nnz || e < s) {
    bad |= ERR_INDPTR;
    s = max(s, base);
    e = min(e, base + x.nnz);
    if (e < s) e = s;
  }
  // wavefront gw of the row's SPLIT * WAVES takes the gw-th contiguous range
  const int gw = piece * WAVES + wave;
  const int per = (e - s + SPLIT * WAVES - 1) / (SPLIT * WAVES);
  const int ws = min(e, s + gw * per), we = min(e, ws + per);
  float2 acc = make_float2(0.0f, 0.0f);
  for (int p0 = ws; p0 < we; p0 += 64) {
    const int p = p0 + lane;
    int f = -1;
    float v = 0.0f;
    if (p < we) {
      f = x.indices[p];
      v = x.values[p];
      int key = f;
      if (f < 0 || f >= F) {
        bad |= ERR_FEATURE_ID;
        key = F;  // sorts after every feature; the W1 update skips it
        f = -1;
      } else if (validate && p > s && x.indices[p - 1] >= f) {
        bad |= ERR_DUPLICATE;
      }
      keys[p - base] = key;
      row_of[p - base] = i;
    }
    const int cnt = min(64, we - p0);
    for (int j = 0; j < cnt; j += GATHER_UNROLL) {
      int fj[GATHER_UNROLL];
      float vj[GATHER_UNROLL];
      float2 wv[GATHER_UNROLL];
#pragma unroll
      for (int u = 0; u < GATHER_UNROLL; ++u) {
        fj[u] = __builtin_amdgcn_readlane(f, j + u);
        vj[u] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), j + u));
      }
#pragma unroll
      for (int u = 0; u < GATHER_UNROLL; ++u)  // id -1 (padding, invalid) reads row 0, discarded below
        wv[u] = *reinterpret_cast<const float2*>(W1 + (size_t)max(fj[u], 0) * HID + h0);
#pragma unroll
      for (int u = 0; u < GATHER_UNROLL; ++u) {
        if (fj[u] >= 0) {
          acc.x = fmaf(vj[u], wv[u].x, acc.x);
          acc.y = fmaf(vj[u], wv[u].y, acc.y);
        }
      }
    }
  }
  part[wave][lane] = acc;

  if (has_y && piece == 0 && wave == WAVES - 1) {
    const int ybase = y.indptr[0];
    int ys = y.indptr[i], ye = y.indptr[i + 1];
    if (ys < ybase || ye > ybase + y.nnz || ye < ys) {
      bad |= ERR_INDPTR;
      ys = max(ys, ybase);
      ye = min(ye, ybase + y.nnz);
      if (ye < ys) ye = ys;
    }
    if (ye == ys) bad |= ERR_EMPTY_LABELS;
    if (lane == 0) rw[i] = ye > ys ? 1.0f / (float)(ye - ys) : 0.0f;
    for (int q = ys + lane; q < ye; q += 64) {
      const int lab = y.indices[q];
      int key = lab;
      if (lab < 0 || lab >= L) {
        bad |= ERR_LABEL_ID;
        key = L;  // dropped when the pairs are grouped by label block
      } else if (validate && q > ys && y.indices[q - 1] >= lab) {
        bad |= ERR_DUPLICATE;
      }
      lkeys[q - ybase] = key;
      lrow[q - ybase] = i;
    }
  }
  if (bad) atomicOr(err, bad);
  __syncthreads();
  if (wave == 0) {
    float2 a = part[0][lane];
#pragma unroll
    for (int k = 1; k < WAVES; ++k) {
      a.x += part[k][lane].x;
      a.y += part[k][lane].y;
    }
    if constexpr (SPLIT > 1) {
      *reinterpret_cast<float2*>(gpart + ((size_t)piece * ld_t + i) * HID + h0) = a;
      return;
    }
    const float2 bb = *reinterpret_cast<const float2*>(b1 + h0);
    a.x = bb.x + a.x;
    a.y = bb.y + a.y;
    *reinterpret_cast<float2*>(A1 + (size_t)i * HID + h0) = a;
    const float r0 = fmaxf(a.x, 0.0f), r1 = fmaxf(a.y, 0.0f);
    if constexpr (DENSE) {
      part[0][lane] = make_float2(r0, r1);  // (wave 0 has read every part)
    } else {
      H1[(size_t)i * HID + h0] = (E)r0;
      H1[(size_t)i * HID + h0 + 1] = (E)r1;
      if constexpr (!BF16) {
        H1T[(size_t)h0 * ld_t + i] = (E)r0;
        H1T[(size_t)(h0 + 1) * ld_t + i] = (E)r1;
      }
    }
  }
  if constexpr (DENSE) {
    __syncthreads();
    if (threadIdx.x < 2 * HID)
      dense_row_store<BF16>(dn, reinterpret_cast<const float*>(part[0]), i, (int)threadIdx.x, H1, H1T, ld_t);
  }
}

// Rows split over GATHER_SPLIT workgroups: A1 = b1 + the pieces' sums in
// piece order, then H1 (and H1^T for fp32 operands) as above.
template <bool BF16, bool DENSE>
__global__ __launch_bounds__(DENSE ? 2 * HID : 64) void k_gather_finish(
    int n_rows, const float* __restrict__ gpart, int ld_t, const float* __restrict__ b1, float* __restrict__ A1,
    typename Mma<BF16>::elem* __restrict__ H1, typename Mma<BF16>::elem* __restrict__ H1T, DenseFwd dn) {
  using E = typename Mma<BF16>::elem;
  __shared__ float2 h_s[64];
  const int i = blockIdx.x, h0 = 2 * threadIdx.x;
  if (i >= n_rows) return;
  if (threadIdx.x < 64) {
    float2 a = *reinterpret_cast<const float2*>(gpart + (size_t)i * HID + h0);
#pragma unroll
    for (int k = 1; k < GATHER_SPLIT; ++k) {
      const float2 v = *reinterpret_cast<const float2*>(gpart + ((size_t)k * ld_t + i) * HID + h0);
      a.x += v.x;
      a.y += v.y;
    }
    const float2 bb = *reinterpret_cast<const float2*>(b1 + h0);
    a.x = bb.x + a.x;
    a.y = bb.y + a.y;
    *reinterpret_cast<float2*>(A1 + (size_t)i * HID + h0) = a;
    const float r0 = fmaxf(a.x, 0.0f), r1 = fmaxf(a.y, 0.0f);
    if constexpr (DENSE) {
      h_s[threadIdx.x] = make_float2(r0, r1);
    } else {
      H1[(size_t)i * HID + h0] = (E)r0;
      H1[(size_t)i * HID + h0 + 1] = (E)r1;
      if constexpr (!BF16) {
        H1T[(size_t)h0 * ld_t + i] = (E)r0;
        H1T[(size_t)(h0 + 1) * ld_t + i] = (E)r1;
      }
    }
  }
  if constexpr (DENSE) {
    __syncthreads();
    dense_row_store<BF16>(dn, reinterpret_cast<const float*>(h_s), i, (int)threadIdx.x, H1, H1T, ld_t);
  }
}

hipError_t launch_gather_fwd(bool use_bf16, const CsrDev& x, const CsrDev* y, const float* W1,
                             const float* b1, int F, int L, float* A1, void* H1, void* H1T,
                             int rows_pad, int ld_t, int32_t* keys, int32_t* row_of,
                             int32_t* lkeys, int32_t* lrow, float* rw, int32_t* err, int validate,
                             float* gpart, bool alone, const DenseFwd* dense, int32_t* zero, int n_zero,
                             hipStream_t st, hipEvent_t done) {
  CsrDev yy = y ? *y : CsrDev{0, 0, 0, nullptr, nullptr, nullptr};
  const DenseFwd dn = dense ? *dense : DenseFwd{};
  const bool wide = alone && x.n_rows <= GATHER_WIDE_ROWS;
  const bool split = gpart && gather_splits_rows(x.n_rows, x.nnz);
  // the last launch completes `done`
  auto go = [&](auto kern, int pieces, int waves, auto* h1, auto* h1t, hipEvent_t ev) {
    const dim3 grid(rows_pad * pieces), block(64 * waves);
    const int has_y = y != nullptr;
    if (ev)
      hipExtLaunchKernelGGL(kern, grid, block, 0, st, nullptr, ev, 0, x, yy, has_y, W1, b1, F, L, A1, h1, h1t,
                            rows_pad, ld_t, keys, row_of, lkeys, lrow, rw, err, validate, gpart, dn, zero, n_zero);
    else
      hipLaunchKernelGGL(kern, grid, block, 0, st, x, yy, has_y, W1, b1, F, L, A1, h1, h1t, rows_pad, ld_t, keys,
                         row_of, lkeys, lrow, rw, err, validate, gpart, dn, zero, n_zero);
  };
  auto finish = [&](auto kern, int threads, auto* h1, auto* h1t) {
    if (done)
      hipExtLaunchKernelGGL(kern, dim3(x.n_rows), dim3(threads), 0, st, nullptr, done, 0, x.n_rows,
                            (const float*)gpart, ld_t, b1, A1, h1, h1t, dn);
    else
      hipLaunchKernelGGL(kern, dim3(x.n_rows), dim3(threads), 0, st, x.n_rows, (const float*)gpart, ld_t, b1, A1,
                         h1, h1t, dn);
  };
  auto all = [&](auto bf, auto* h1, auto* h1t) {
    constexpr bool BF = decltype(bf)::value;
    if (split) {
      go(k_gather_fwd<BF, GATHER_SPLIT, 8, false>, GATHER_SPLIT, 8, h1, h1t, nullptr);
      if (dense)
        finish(k_gather_finish<BF, true>, 2 * HID, h1, h1t);
      else
        finish(k_gather_finish<BF, false>, 64, h1, h1t);
    } else if (dense) {
      go(k_gather_fwd<BF, 1, 8, true>, 1, 8, h1, h1t, done);
    } else if (wide) {
      go(k_gather_fwd<BF, 1, 8, false>, 1, 8, h1, h1t, done);
    } else {
      go(k_gather_fwd<BF, 1, 4, false>, 1, 4, h1, h1t, done);
    }
  };
  if (use_bf16)
    all(std::true_type{}, (bf16*)H1, (bf16*)H1T);
  else
    all(std::false_type{}, (float*)H1, (float*)H1T);
  return hipGetLastError();
}

}  // namespace asgd
