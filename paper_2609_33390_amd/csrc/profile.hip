// Acceptance-profile statistics of verified blocks (Section 3.2, Eq.
// nonuniform_tpf and Eq. brisk_weighting; Appendix "Brisk Backbone", Eq.
// idlm_tpf_instantiation).
//
// From the accepted-prefix lengths L_b in [0, M] of many verified blocks:
// a_i = 1 - rejected_i / reached_i (block b reaches positions 1..L_b + 1 and
// is rejected at L_b + 1 when L_b < M), survival A_k = prod_{j<=k} a_j, the
// ISD tokens per forward TPF = (2 + sum_{k=1}^{M-1} A_k) / (2 - A_M) and
// FPT = 1 / TPF, the position sensitivities w_raw_i = -dFPT/dz_i under the
// log-odds z_i = log(a_i / (1 - a_i)), and the mean-one weights
// w_i = M w_raw_i / (sum_j w_raw_j + eps).
//
// Two launches: workgroups histogram disjoint slices of the lengths into
// partial histograms (no atomics on global memory, so the counts do not depend
// on scheduling), then one workgroup adds the partials and evaluates the
// closed forms in fp64, one position per thread, with scans for the products
// and sums.  Both are bound by latency, so what counts is the number of
// dependent steps: at 2^20 lengths, M = 32, the pair took 15.6 + 11.8 us with
// a barrier pair per bin in the first and serial loops over the positions in
// the second, and takes 6.2 + 6.6 us.
#include "device_common.h"
#include "kernels.h"

namespace brisk {

namespace {

constexpr int kHistThreads = 256;
constexpr int kMaxHistGroups = 256;
constexpr int kBlocksPerGroup = 4096;

int hist_groups(int n_blocks) {
  const int g = (n_blocks + kBlocksPerGroup - 1) / kBlocksPerGroup;
  return g < 1 ? 1 : (g > kMaxHistGroups ? kMaxHistGroups : g);
}

// Columns of counters per bin, and the LDS they take: one per thread while 64
// KiB hold them, fewer for larger M (threads of one column then add in turn).
constexpr int hist_cols(int M) { return M < 64 ? 256 : M < 256 ? 64 : M < 512 ? 16 : 8; }

// Partial histogram of this workgroup's slice: part[j * groups + workgroup].
template <int COLS>
__global__ __launch_bounds__(kHistThreads) void accept_hist_kernel(const int32_t* __restrict__ len,
                                                                   int n_blocks, int M,
                                                                   uint32_t* __restrict__ part) {
  extern __shared__ __align__(16) uint32_t h[];  // [M + 1][COLS]
  const int tid = threadIdx.x;
  const int per = (n_blocks + gridDim.x - 1) / gridDim.x;
  const int b0 = blockIdx.x * per;
  const int b1 = min(b0 + per, n_blocks);
  // a slice of 4096 lengths is one batch: all its loads in flight at once
  constexpr int BATCH = 16;
  int Ls[BATCH];
  auto load = [&](int bb) {
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int b = bb + q * kHistThreads + tid;
      Ls[q] = b < b1 ? len[b] : 0;
    }
  };
  load(b0);
  for (int j = tid; j < (M + 1) * (COLS / 4); j += kHistThreads)
    reinterpret_cast<uint4*>(h)[j] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  for (int bb = b0; bb < b1; bb += kHistThreads * BATCH) {
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int L = Ls[q] < 0 ? 0 : (Ls[q] > M ? M : Ls[q]);
      // additions without a result do not wait for each other
      if (bb + q * kHistThreads + tid < b1) atomicAdd(&h[L * COLS + tid % COLS], 1u);
    }
    if (bb + kHistThreads * BATCH < b1) load(bb + kHistThreads * BATCH);
  }
  __syncthreads();
  // four counters a lane, COLS / 4 lanes a bin
  constexpr int LPB = COLS / 4, BPI = kHistThreads / LPB;
  for (int j0 = 0; j0 <= M; j0 += BPI) {
    const int j = j0 + tid / LPB;
    uint32_t v = 0;
    if (j <= M) {
      const uint4 c = reinterpret_cast<const uint4*>(h)[j * LPB + tid % LPB];
      v = (c.x + c.y) + (c.z + c.w);
    }
#pragma unroll
    for (int off = 1; off < LPB; off <<= 1) v += __shfl_xor(v, off, kWave);
    if (j <= M && tid % LPB == 0) part[static_cast<size_t>(j) * gridDim.x + blockIdx.x] = v;
  }
}

constexpr int kProfThreads = 1024, kProfWaves = kProfThreads / kWave;
static_assert(kProfThreads >= 1024, "one position per thread");

// Inclusive scan over the threads of the workgroup, towards higher threads
// (UP) or lower ones: the wave's own scan, then the totals of the waves
// before it, in order.  `ident` is op's neutral element; s holds kProfWaves
// values, and the caller puts a barrier between two uses of it.
template <bool UP, class T, class Op>
__device__ __forceinline__ T block_scan(T v, T ident, Op op, T* s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const T o = UP ? __shfl_up(v, off, kWave) : __shfl_down(v, off, kWave);
    if (UP ? lane >= off : lane + off < kWave) v = op(v, o);
  }
  if (lane == (UP ? kWave - 1 : 0)) s[wave] = v;
  __syncthreads();
  T before = ident;
  for (int w = 0; w < kProfWaves; ++w)
    if (UP ? w < wave : w > wave) before = op(before, s[w]);
  return op(v, before);
}

__global__ __launch_bounds__(kProfThreads) void accept_profile_kernel(const uint32_t* __restrict__ part,
                                                                      int groups, int n_blocks, int M, double eps,
                                                                      double* __restrict__ a_out,
                                                                      double* __restrict__ raw_out,
                                                                      double* __restrict__ w_out,
                                                                      double* __restrict__ tpf_fpt) {
  __shared__ uint32_t cnt[1025];  // blocks per accepted length
  __shared__ uint32_t s_u[kProfWaves];
  __shared__ double s_a[kProfWaves], s_b[kProfWaves], s_c[kProfWaves], s_end[2];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // a wavefront adds the partials of two bins at a time, their loads together
  static_assert(kMaxHistGroups <= 4 * kWave, "four partials a lane");
  for (int j0 = wave; j0 <= M; j0 += 2 * kProfWaves) {
    uint32_t v[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = j0 + i * kProfWaves, g = lane + q * kWave;
        v[i][q] = j <= M && g < groups ? part[static_cast<size_t>(j) * groups + g] : 0u;
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint32_t c = (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) c += __shfl_xor(c, off, kWave);
      if (lane == 0 && j0 + i * kProfWaves <= M) cnt[j0 + i * kProfWaves] = c;
    }
  }
  __syncthreads();
  // position i = t + 1: reached_i = #{L >= i - 1}, rejected_i = #{L = i - 1}
  const bool on = t < M;
  const uint32_t rej = on ? cnt[t] : 0u;
  const auto add = [](auto x, auto y) { return x + y; };
  const uint32_t upto = block_scan<true>(rej, 0u, add, s_u);  // #{L <= i - 1}
  const double reach = static_cast<double>(static_cast<uint32_t>(n_blocks) - (upto - rej));
  const double a = on && reach > 0.0 ? 1.0 - static_cast<double>(rej) / reach : 1.0;
  const double A = block_scan<true>(a, 1.0, [](double x, double y) { return x * y; }, s_a);  // A_i
  // S_i = sum_{k=i}^{M-1} A_k
  const double S = block_scan<false>(t < M - 1 ? A : 0.0, 0.0, add, s_b);
  if (t == 0) s_end[0] = S;
  if (t == M - 1) s_end[1] = A;
  __syncthreads();
  const double num = 2.0 + s_end[0], den = 2.0 - s_end[1];
  const double R = on ? (1.0 - a) * (s_end[1] * num + den * S) / (num * num) : 0.0;
  const double sum_from = block_scan<false>(R, 0.0, add, s_c);
  if (t == 0) {
    s_end[0] = sum_from;  // read above, before block_scan's barrier
    tpf_fpt[0] = num / den;
    tpf_fpt[1] = den / num;
  }
  __syncthreads();
  if (on) {
    a_out[t] = a;
    raw_out[t] = R;
    w_out[t] = M * R / (s_end[0] + eps);
  }
}

}  // namespace

size_t accept_profile_workspace_bytes(int n_blocks, int M) {
  return static_cast<size_t>(hist_groups(n_blocks)) * (M + 1) * sizeof(uint32_t);
}

void launch_accept_profile(const int32_t* accept_len, int n_blocks, int M, double eps, double* a,
                           double* w_raw, double* w, double* tpf_fpt, void* ws, hipStream_t s) {
  const int groups = hist_groups(n_blocks);
  uint32_t* part = static_cast<uint32_t*>(ws);
  const size_t hist_lds = static_cast<size_t>(M + 1) * hist_cols(M) * sizeof(uint32_t);
  const dim3 g(groups), b(kHistThreads);
  switch (hist_cols(M)) {
    case 256: hipLaunchKernelGGL(accept_hist_kernel<256>, g, b, hist_lds, s, accept_len, n_blocks, M, part); break;
    case 64: hipLaunchKernelGGL(accept_hist_kernel<64>, g, b, hist_lds, s, accept_len, n_blocks, M, part); break;
    case 16: hipLaunchKernelGGL(accept_hist_kernel<16>, g, b, hist_lds, s, accept_len, n_blocks, M, part); break;
    default: hipLaunchKernelGGL(accept_hist_kernel<8>, g, b, hist_lds, s, accept_len, n_blocks, M, part); break;
  }
  hipLaunchKernelGGL(accept_profile_kernel, dim3(1), dim3(kProfThreads), 0, s, part, groups, n_blocks, M, eps, a,
                     w_raw, w, tpf_fpt);
}

}  // namespace brisk
