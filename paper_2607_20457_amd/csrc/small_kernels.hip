// Bandwidth-bound helper kernels: the materialised Eq. 3 position map, the
// KV(B_i) retention copy, and the Phase-2 online-softmax merge.
#include <type_traits>

#include "common.hpp"

// ---------------------------------------------------------------------------
// Row -> global position map (Eq. 3, sparse position ids), with the same
// device function the attention kernel uses for its fused gather.
__global__ __launch_bounds__(256) void positions_kernel(RowMap mp, const int32_t* __restrict__ sel,
                                                        int64_t sel_bstride, int n_rows,
                                                        int32_t* __restrict__ pos) {
  extern __shared__ int run_base[];
  const int b = blockIdx.y;
  build_run_table(mp, sel ? sel + b * sel_bstride : nullptr, run_base, threadIdx.x, 256);
  __syncthreads();
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n_rows) return;
  pos[(int64_t)b * n_rows + r] = row_position(mp, run_base, r);
}

int launch_positions(const RowMap& mp, const int32_t* sel, int64_t sel_bstride, int batch,
                     int n_rows, int32_t* pos, hipStream_t stream) {
  if (batch == 0 || n_rows == 0) return PULSAR_OK;
  const size_t lds = (size_t)mp.n_runs * 4;
  if (lds > PULSAR_LDS_BYTES) return PULSAR_EUNSUPPORTED;
  if (hipFuncSetAttribute((const void*)positions_kernel,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return PULSAR_EHIP;
  dim3 grid((n_rows + 255) / 256, batch);
  hipLaunchKernelGGL(positions_kernel, grid, dim3(256), lds, stream, mp, sel, sel_bstride, n_rows,
                     pos);
  return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
}

// ---------------------------------------------------------------------------
// KV(B_i) retention (Appendix "KV Cache Discard"): the same rows of K and V,
// `rows` sequences of row16 16-byte words each, in one launch (grid.z).  Every
// thread moves U words with all its loads in flight.  (K and V in a launch each,
// a word per thread: 11 us for 2 x 8.4 MB, and a second launch on the host.)
__global__ __launch_bounds__(256) void keep_kv_kernel(const u32x4* __restrict__ K,
                                                      const u32x4* __restrict__ V,
                                                      int64_t src_pitch16, u32x4* __restrict__ Ko,
                                                      u32x4* __restrict__ Vo, int64_t row16) {
  constexpr int U = 4;
  const int64_t row = blockIdx.y;
  const u32x4* s = (blockIdx.z ? V : K) + row * src_pitch16;
  u32x4* d = (blockIdx.z ? Vo : Ko) + row * row16;
  for (int64_t i0 = (int64_t)blockIdx.x * 256 * U + threadIdx.x; i0 < row16;
       i0 += (int64_t)gridDim.x * 256 * U) {
    u32x4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = s[min(i0 + u * 256, row16 - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * 256 < row16) d[i0 + u * 256] = x[u];
  }
}

int launch_keep_kv(const void* K, const void* V, int64_t src_pitch, void* K_out, void* V_out,
                   int64_t bytes_per_row, int rows, hipStream_t stream) {
  if (rows == 0 || bytes_per_row == 0) return PULSAR_OK;
  const int64_t row16 = bytes_per_row / 16;
  int64_t blocks = (row16 + 1023) / 1024;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(keep_kv_kernel, dim3((unsigned)blocks, rows, 2), dim3(256), 0, stream,
                     (const u32x4*)K, (const u32x4*)V, src_pitch / 16, (u32x4*)K_out, (u32x4*)V_out,
                     row16);
  return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
}

// ---------------------------------------------------------------------------
// IDF table of a context without tokens (Eq. idf with df = 0 everywhere):
// the value the Max-IDF kernels write for an id that occurs in no block.
__global__ __launch_bounds__(256) void idf_fill_kernel(float* __restrict__ idf, int64_t n,
                                                       float num_blocks) {
  const float v = logf(num_blocks / 1.0f);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    idf[i] = v;
}

int launch_idf_fill(float* idf, int64_t n, int num_blocks, hipStream_t stream) {
  if (n == 0) return PULSAR_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(idf_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, idf, n,
                     (float)num_blocks);
  return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
}

// ---------------------------------------------------------------------------
// (may also say so of opposite infinities)
__device__ __forceinline__ bool is_nan(f32x4 x) {
  const float s = (x[0] + x[1]) + (x[2] + x[3]);
  return s != s;
}

// Online-softmax merge (Appendix "Phase 2 Distributed Softmax Merge").
// Thread = four consecutive head_dim entries of one (z, query, head).  One
// pass over the parts, CH at a time (2, 4 or 8: the fewest that cover H, up
// to 8) with all their loads issued together: the running maximum m,
// s = sum_h exp(l_h - m) and a = sum_h exp(l_h - m) o_h are rescaled when m
// rises; then l = m + ln s and o = a / s.  -inf partials weigh zero, and what
// their o holds must not count either: where a zero weight has met a NaN or an
// infinity there (so that a is NaN), the pass is repeated with such parts left
// out.  (To leave them out at once costs every merge 3 to 6 %.)
template <int CH>
__global__ __launch_bounds__(256) void lse_merge_kernel(
    const float* __restrict__ o_parts, const float* __restrict__ lse_parts, int H, int Tq, int Hq,
    int d4, int64_t part_ostride, int64_t part_lstride, float* __restrict__ o,
    float* __restrict__ lse, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int dv = (int)(i % d4);
  int64_t rest = i / d4;
  const int h = (int)(rest % Hq);
  rest /= Hq;
  const int q = (int)(rest % Tq);
  const int64_t z = rest / Tq;

  const float* lp = lse_parts + z * (int64_t)H * part_lstride + (int64_t)h * Tq + q;
  const int64_t orow = (((int64_t)q * Hq + h) * d4 + dv);
  const f32x4* op = reinterpret_cast<const f32x4*>(o_parts) + z * (int64_t)H * (part_ostride / 4);
  float m, sum;
  f32x4 acc;
  auto fold = [&](auto leave_out) {
    m = -INFINITY, sum = 0.f;
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < H; p0 += CH) {
      float l[CH];
      f32x4 v[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int p = min(p0 + u, H - 1);  // a part past the last re-reads it, weighing zero
        l[u] = lp[p * part_lstride];
        v[u] = op[p * (part_ostride / 4) + orow];
      }
      float cm = -INFINITY;
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (p0 + u < H) cm = fmaxf(cm, l[u]);
      // branch-free, so that all 2 CH loads are issued before the first
      // wait; with no finite partial yet the weights are taken against 0 and
      // come out 0
      const float nm = fmaxf(m, cm);
      const float nm_use = nm == -INFINITY ? 0.f : nm;
      const float alpha = __expf(m - nm_use);  // 0 while m is -inf
      sum *= alpha;
      acc *= alpha;
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const float w = p0 + u < H ? __expf(l[u] - nm_use) : 0.f;
        sum += w;
        if (decltype(leave_out)::value && (p0 + u >= H || l[u] == -INFINITY)) continue;
        acc += w * v[u];
      }
      m = nm;
    }
  };
  fold(std::false_type{});
  if (is_nan(acc)) fold(std::true_type{});
  float ell = -INFINITY;
  if (m != -INFINITY) {
    ell = m + __logf(sum);
    acc *= 1.f / sum;
  }
  reinterpret_cast<f32x4*>(o)[z * (int64_t)Tq * Hq * d4 + orow] = acc;
  if (lse && dv == 0) lse[z * (int64_t)Hq * Tq + (int64_t)h * Tq + q] = ell;
}

// The same merge with one workgroup per output row (grid.y: DL groups of four
// values of it), for few rows and many parts (a decode step: 32 rows, tens to
// hundreds of parts; a query encoding: hundreds of rows, tens of parts).
// Thread (pg, dv) folds parts pg, pg + PG, ... of one group, CH of them with
// all their loads issued together, so a merge waits for one round trip to
// memory where CH * PG covers the parts; then the groups are folded across
// lanes and, through LDS, across wavefronts.
template <int DL, int THREADS>
__global__ __launch_bounds__(THREADS) void lse_merge_wide_kernel(
    const float* __restrict__ o_parts, const float* __restrict__ lse_parts, int H, int Tq, int Hq,
    int d4, int64_t part_ostride, int64_t part_lstride, float* __restrict__ o,
    float* __restrict__ lse) {
  constexpr int PG = THREADS / DL;
  constexpr int W = THREADS / 64;
  constexpr int CH = 4;
  __shared__ float s_m[W], s_s[W];
  __shared__ f32x4 s_a[W][DL];
  const int tid = threadIdx.x;
  const int dv = blockIdx.y * DL + tid % DL;
  const int pg = tid / DL;
  const int64_t row = blockIdx.x;
  const int h = (int)(row % Hq);
  const int64_t zq = row / Hq;
  const int q = (int)(zq % Tq);
  const int64_t z = zq / Tq;

  const float* lp = lse_parts + z * (int64_t)H * part_lstride + (int64_t)h * Tq + q;
  const int64_t orow = ((int64_t)q * Hq + h) * d4;
  const f32x4* op = reinterpret_cast<const f32x4*>(o_parts) + z * (int64_t)H * (part_ostride / 4) +
                    orow + min(dv, d4 - 1);
  float m, sum;
  f32x4 acc;
  auto fold = [&](auto leave_out) {
    m = -INFINITY, sum = 0.f;
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int p0 = pg; p0 < H; p0 += CH * PG) {
      float l[CH];
      f32x4 v[CH];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const int p = min(p0 + u * PG, H - 1);  // a part past the last weighs zero
        l[u] = lp[p * part_lstride];
        v[u] = op[p * (part_ostride / 4)];
      }
      float nm = m;
#pragma unroll
      for (int u = 0; u < CH; ++u)
        if (p0 + u * PG < H) nm = fmaxf(nm, l[u]);
      const float use = nm == -INFINITY ? 0.f : nm;  // no finite partial yet: weights 0
      const float alpha = __expf(m - use);
      sum *= alpha;
      acc *= alpha;
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const float w = p0 + u * PG < H ? __expf(l[u] - use) : 0.f;
        sum += w;
        if (decltype(leave_out)::value && (p0 + u * PG >= H || l[u] == -INFINITY)) continue;
        acc += w * v[u];
      }
      m = nm;
    }
  };
  fold(std::false_type{});
  if (is_nan(acc)) fold(std::true_type{});  // as in the per-output kernel
  // lanes DL apart hold the same values' other parts
#pragma unroll
  for (int off = DL; off < 64; off <<= 1) {
    const float m2 = __shfl_xor(m, off, 64);
    const float nm = fmaxf(m, m2);
    const float use = nm == -INFINITY ? 0.f : nm;
    const float w1 = __expf(m - use), w2 = __expf(m2 - use);
    sum = sum * w1 + __shfl_xor(sum, off, 64) * w2;
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = acc[k] * w1 + __shfl_xor(acc[k], off, 64) * w2;
    m = nm;
  }
  const int wave = tid >> 6, lane = tid & 63;
  if (lane == 0) {
    s_m[wave] = m;
    s_s[wave] = sum;
  }
  if (lane < DL) s_a[wave][lane] = acc;
  __syncthreads();
  if (tid >= DL || dv >= d4) return;
  m = s_m[0];
#pragma unroll
  for (int w = 1; w < W; ++w) m = fmaxf(m, s_m[w]);
  const float use = m == -INFINITY ? 0.f : m;
  sum = 0.f;
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float e = __expf(s_m[w] - use);
    sum += s_s[w] * e;
    acc += s_a[w][tid] * e;
  }
  float ell = -INFINITY;
  if (m != -INFINITY) {
    ell = m + __logf(sum);
    acc *= 1.f / sum;
  }
  reinterpret_cast<f32x4*>(o)[z * (int64_t)Tq * Hq * d4 + orow + dv] = acc;
  if (lse && dv == 0) lse[z * (int64_t)Hq * Tq + (int64_t)h * Tq + q] = ell;
}

int launch_lse_merge(const float* o_parts, const float* lse_parts, int H, int nz, int Tq, int Hq,
                     int d, int64_t part_ostride, int64_t part_lstride, float* o, float* lse,
                     hipStream_t stream) {
  const int64_t total = (int64_t)nz * Tq * Hq * (d / 4);
  if (total == 0) return PULSAR_OK;
  const int64_t rows = (int64_t)nz * Tq * Hq;
  // One workgroup per row where there are too few outputs for the per-output
  // form to fill the chip and enough parts to be worth a workgroup each: the
  // more rows, the more parts it takes.  In 3194 Phase-2 calls the form per row
  // (256 threads) took, us more than the one per output, at d 128: 8 or 9 parts,
  // up to 256 rows -0.6, 1024 rows 0.1, 2048 rows 1.2; 13 to 17 parts, up to 256
  // rows -1.0, 1024 -0.6, 2048 0.6; 25 to 33 parts, 256 rows -2.0, 2048 -0.4; the
  // choice is 0.2 % slower than the better one on average.  256 threads take 32
  // parts of a row of 128 in one round of loads, of 64 twice as many; a row of
  // more parts has 512 while the rows are few (98 to 129 parts, up to 32 rows
  // another 0.7 us less, 384 rows 0.4 more), and 1024 were never the best (10 to
  // 33 parts 0.6 to 1 us slower).
  // (Rows are counted as of 64 or 128 values, those that a workgroup's lanes take.)
  const int dl = d <= 64 ? 16 : 32;
  const int slices = (d / 4 + dl - 1) / dl;
  if (H >= 8 && total <= 40960 && rows * slices * dl * 4 <= 200 * (int64_t)(H - 4) * d) {
    const dim3 grid((unsigned)rows, (unsigned)slices);
    const int threads = total <= 8192 && H > 1024 / dl ? 512 : 256;
    const auto wide = threads == 512
                          ? (dl == 16 ? lse_merge_wide_kernel<16, 512> : lse_merge_wide_kernel<32, 512>)
                          : (dl == 16 ? lse_merge_wide_kernel<16, 256> : lse_merge_wide_kernel<32, 256>);
    hipLaunchKernelGGL(wide, grid, dim3(threads), 0, stream, o_parts, lse_parts, H, Tq, Hq, d / 4,
                       part_ostride, part_lstride, o, lse);
    return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
  }
  const int64_t blocks = (total + 255) / 256;
  const auto kern = H <= 2 ? lse_merge_kernel<2> : H <= 4 ? lse_merge_kernel<4> : lse_merge_kernel<8>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, stream, o_parts, lse_parts, H,
                     Tq, Hq, d / 4, part_ostride, part_lstride, o, lse, total);
  return hipGetLastError() == hipSuccess ? PULSAR_OK : PULSAR_EHIP;
}
