// Corrector training loss, forward (Appendix "Candidate-Refinement Head
// Details", Eq. head_training_loss; Algorithm 1(a), corrector training).
//
// At position j of a block with candidate set S_j: p_S = the verifier
// distribution restricted to S_j and renormalised, q_S = the base proposal
// distribution restricted to S_j, r = softmax of the refined logits;
// l_j = CE(p_S, r) + beta KL(q_S || r).  Only the positions whose
// verification is reached count: the accepted prefix and the first rejected
// position (every position of a fully accepted block).  The loss is the mean
// of l_j over those positions.
//
// One workgroup per position: its four wavefronts take the verifier logits
// <E_out[v_k], h_j> of the candidates (dot products over d), then wavefront 0
// holds candidate k in lane k for the three log-softmaxes.  A second launch
// adds the per-position losses in a fixed order.
//
// The first launch is bound by the gathered lm_head rows, so a wavefront has
// two of them and the hidden row in flight at once; the second by latency, so
// a thread has a batch of its positions in flight.  At 256 x 16 positions (38%
// reached), d = 4096, K = 8: 26 + 9.4 us with one chunk of a row and one
// position at a time, 24.4 + 4.0 us now.
#include "device_common.h"
#include "kernels.h"

namespace brisk {

namespace {

__device__ __forceinline__ bool reached(const int32_t* accept_len, int r, int L) {
  const int b = r / L, j = r % L;
  return j <= accept_len[b];
}

__global__ __launch_bounds__(256) void loss_pos_kernel(const uint16_t* __restrict__ Hv,
                                                       const uint16_t* __restrict__ W,
                                                       const int32_t* __restrict__ cand_id,
                                                       const float* __restrict__ cand_logit,
                                                       const float* __restrict__ refined,
                                                       const int32_t* __restrict__ accept_len, int L,
                                                       int K, int d, int V, float beta,
                                                       float* __restrict__ loss_pos,
                                                       float* __restrict__ ce_out,
                                                       float* __restrict__ kl_out) {
  __shared__ float s_lp[64];
  const int r = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (!reached(accept_len, r, L)) {
    if (threadIdx.x == 0) {
      loss_pos[r] = 0.f;
      if (ce_out) ce_out[r] = 0.f;
      if (kl_out) kl_out[r] = 0.f;
    }
    return;
  }
  const uint16_t* h = Hv + static_cast<size_t>(r) * d;
  auto row_of = [&](int k) {
    return W + static_cast<size_t>(clamp_id(cand_id[static_cast<size_t>(r) * K + min(k, K - 1)], V)) * d;
  };
  auto dot8 = [](float& s, uint4 a, uint4 b) {
    s += bf16_lo(a.x) * bf16_lo(b.x) + bf16_hi(a.x) * bf16_hi(b.x);
    s += bf16_lo(a.y) * bf16_lo(b.y) + bf16_hi(a.y) * bf16_hi(b.y);
    s += bf16_lo(a.z) * bf16_lo(b.z) + bf16_hi(a.z) * bf16_hi(b.z);
    s += bf16_lo(a.w) * bf16_lo(b.w) + bf16_hi(a.w) * bf16_hi(b.w);
  };
  // candidates k and k + 4 together, CH 512-element chunks of each row in
  // flight (a 4096-long row at once)
  constexpr int CH = 8;
  for (int k = wave; k < K; k += 8) {
    const bool two = k + 4 < K;  // wave-uniform
    const uint16_t *w0 = row_of(k), *w1 = row_of(k + 4);
    float s0 = 0.f, s1 = 0.f;
    for (int c0 = lane * 8; c0 < d; c0 += CH * 512) {
      uint4 hv[CH], a0[CH], a1[CH];
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        const int c = c0 + i * 512;
        hv[i] = c < d ? *reinterpret_cast<const uint4*>(h + c) : make_uint4(0, 0, 0, 0);
        a0[i] = c < d ? *reinterpret_cast<const uint4*>(w0 + c) : make_uint4(0, 0, 0, 0);
        a1[i] = c < d && two ? *reinterpret_cast<const uint4*>(w1 + c) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        if (c0 + i * 512 < d) {
          dot8(s0, a0[i], hv[i]);
          dot8(s1, a1[i], hv[i]);
        }
      }
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if (lane == 0) {
      s_lp[k] = s0;
      if (two) s_lp[k + 4] = s1;
    }
  }
  __syncthreads();
  if (wave != 0) return;
  const bool on = lane < K;
  const float lp = on ? s_lp[lane] : -INFINITY;
  const float lq = on ? cand_logit[static_cast<size_t>(r) * K + lane] : -INFINITY;
  const float lr = on ? refined[static_cast<size_t>(r) * K + lane] : -INFINITY;
  // log-softmax over the K lanes of each of the three logit vectors
  const float mp = wave_allmax(lp), mq = wave_allmax(lq), mr = wave_allmax(lr);
  const float zp = wave_allsum(on ? __expf(lp - mp) : 0.f);
  const float zq = wave_allsum(on ? __expf(lq - mq) : 0.f);
  const float zr = wave_allsum(on ? __expf(lr - mr) : 0.f);
  const float log_p = lp - mp - __logf(zp), log_q = lq - mq - __logf(zq), log_r = lr - mr - __logf(zr);
  const float ce = wave_allsum(on ? -__expf(log_p) * log_r : 0.f);
  const float kl = wave_allsum(on ? __expf(log_q) * (log_q - log_r) : 0.f);
  if (lane == 0) {
    loss_pos[r] = ce + beta * kl;
    if (ce_out) ce_out[r] = ce;
    if (kl_out) kl_out[r] = kl;
  }
}

// mean over the reached positions: per-thread strided partial sums, then a
// fixed-order tree, so the result does not depend on scheduling
constexpr int kMeanThreads = 1024;
__global__ __launch_bounds__(kMeanThreads) void loss_mean_kernel(const float* __restrict__ loss_pos,
                                                                 const int32_t* __restrict__ accept_len,
                                                                 int rows, int L, float* __restrict__ out) {
  constexpr int NW = kMeanThreads / kWave, BATCH = 4;
  __shared__ double s_sum[NW];
  __shared__ int s_cnt[NW];
  double sum = 0.0;
  int cnt = 0;
  for (int r0 = threadIdx.x; r0 < rows; r0 += kMeanThreads * BATCH) {
    float v[BATCH];
    int acc[BATCH];
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int r = min(r0 + q * kMeanThreads, rows - 1);
      v[q] = loss_pos[r];
      acc[q] = accept_len[r / L];
    }
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int r = r0 + q * kMeanThreads;
      if (r < rows && r % L <= acc[q]) {
        sum += v[q];
        ++cnt;
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    sum += __shfl_xor(sum, off, kWave);
    cnt += __shfl_xor(cnt, off, kWave);
  }
  if ((threadIdx.x & 63) == 0) {
    s_sum[threadIdx.x >> 6] = sum;
    s_cnt[threadIdx.x >> 6] = cnt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sum = 0.0;
    cnt = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      sum += s_sum[w];
      cnt += s_cnt[w];
    }
    out[0] = cnt > 0 ? static_cast<float>(sum / cnt) : 0.f;
    out[1] = static_cast<float>(cnt);
  }
}

}  // namespace

void launch_corrector_loss(const uint16_t* ver_hidden, const uint16_t* lm_head, const int32_t* cand_id,
                           const float* cand_logit, const float* refined, const int32_t* accept_len,
                           int B, int L, int K, int d, int V, float beta, float* loss_pos, float* ce,
                           float* kl, float* loss_mean, hipStream_t s) {
  const int rows = B * L;
  hipLaunchKernelGGL(loss_pos_kernel, dim3(rows), dim3(256), 0, s, ver_hidden, lm_head, cand_id,
                     cand_logit, refined, accept_len, L, K, d, V, beta, loss_pos, ce, kl);
  hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(kMeanThreads), 0, s, loss_pos, accept_len, rows, L,
                     loss_mean);
}

}  // namespace brisk
