// Re-anchor selection on the device (sec. 3.1 Eq. 4, sec. 3.2 Eq. 5,
// sec. 3.3 (ii)) and the device node offsets of the candidate trees it
// produces, so that a verify step needs no host round-trip.
//
// r(i) = (c_1 c_2 ... c_i)(1 - c_{i+1}), i = 0..B-2, is the probability that
// exactly i drafts of the block are accepted when position k is accepted
// independently with probability c_k. It is evaluated in float64 with one
// fixed operation order (product from c_1 upward, then the factor 1 - c_{i+1},
// no contraction), so the selection is reproducible bit for bit. The K largest
// r(i) are kept, equal values going to the smaller i; prefix length i becomes
// the re-anchor block position p = i + 1.
#include "launchers.h"

namespace d2sd {

namespace {

constexpr int kSelectThreads = 64;    // one wave per request: B - 1 <= 63 prefix lengths
constexpr int kIndptrThreads = 256;

// The same value of lane `src` (uniform over the wave).
__device__ __forceinline__ float lane_of(float x, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src));
}

// Latency-bound: one wave per request and a chain of n products. Each lane
// holds one confidence and one posterior; the chain reaches the confidences by
// lane reads, the ranking the posteriors in LDS (whose reads run ahead of the
// comparisons). With a load per step of the chain 64 requests of 15
// confidences took 3.5 us, now 3.0; of 63, 7.7 and 6.1; 4096 of 63, 10.5 and
// 9.5 (11.0 with the posteriors by lane reads, four vector instructions each).
#pragma clang fp contract(off)
__global__ __launch_bounds__(kSelectThreads) void select_reanchor_kernel(
    int B, int Kmax, const float* __restrict__ conf, const int* __restrict__ K, int* __restrict__ p_out,
    double* __restrict__ r_out) {
  const int b = blockIdx.x;
  const int i = threadIdx.x;           // prefix length
  const int n = B - 1;                 // number of prefix lengths 0..B-2
  const float c = i < n ? conf[(size_t)b * n + i] : 0.0f;
  const int Kb = clampi(K[b], 0, min(Kmax, n));
  double prod = 1.0;                    // c_1 ... c_i, from c_1 upward
  for (int k = 0; k + 1 < n; ++k) {
    const double next = prod * (double)lane_of(c, k);
    prod = k < i ? next : prod;
  }
  const double r = prod * (1.0 - (double)c);
  // Ranking key: a NaN posterior (from confidences outside [0, 1] or NaN)
  // ranks below every number, so the order stays total and exactly Kb
  // prefix lengths are kept.
  const double key = __builtin_isnan(r) ? -INFINITY : r;
  __shared__ double s_key[kSelectThreads];
  s_key[i] = key;
  __syncthreads();
  int rank = 0;                         // prefix lengths ordered before i
  for (int j = 0; j < n; ++j) {
    const double rj = s_key[j];
    rank += (rj > key) || (rj == key && j < i);
  }
  const bool keep = i < n && rank < Kb;
  if (r_out && i < n) r_out[(size_t)b * n + i] = r;
  // kept prefix lengths in ascending order: slot = kept lanes below this one
  const uint64_t kept = __ballot(keep);
  if (keep) {
    const int slot = __popcll(kept & ((1ull << i) - 1ull));
    if (slot < Kb) p_out[(size_t)b * Kmax + slot] = i + 1;
  }
  for (int k = Kb + i; k < Kmax; k += kSelectThreads) p_out[(size_t)b * Kmax + k] = -1;
}

// node_indptr[b+1] - node_indptr[b] = B + sum_k (B - p_k), with K and p
// clamped exactly as the tree builder clamps them.
//
// Latency-bound: one workgroup, kIndptrThreads requests at a time. A row of p
// is loaded whole (its first B - 1 entries: rows may be longer), eight entries at a time, beside K (not up to K once K is
// there), and the sums are scanned in registers with one barrier instead of
// sixteen. 64 requests of up to 8 positions: 2.9 -> 1.8 us; with rows of 2048
// entries 3.3 -> 2.6 (94 while all of a row was read).
__global__ __launch_bounds__(kIndptrThreads) void tree_indptr_kernel(int batch, int B, int Kmax,
                                                                     const int* __restrict__ K,
                                                                     const int* __restrict__ p,
                                                                     int* __restrict__ node_indptr) {
  constexpr int WAVES = kIndptrThreads / kWave;
  __shared__ int s_sum[2][WAVES];
  const int t = threadIdx.x;
  const int lane = t % kWave, wave = t / kWave;
  if (t == 0) node_indptr[0] = 0;
  int carry = 0;
  for (int b0 = 0, odd = 0; b0 < batch; b0 += kIndptrThreads, odd ^= 1) {
    const int b = b0 + t;
    int nb = 0;
    if (b < batch) {
      const int k_raw = K[b];
      const int* row = p + (size_t)b * Kmax;
      nb = B;
      const int cols = min(Kmax, B - 1);   // entries that can count
      for (int k0 = 0; k0 < cols; k0 += 8) {
        int v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row[min(k0 + j, cols - 1)];
        const int Kb = clampi(k_raw, 0, min(Kmax, B - 1));
#pragma unroll
        for (int j = 0; j < 8; ++j) nb += k0 + j < Kb ? B - clampi(v[j], 1, B - 1) : 0;
      }
    }
    int sum = wave_scan<false>(nb);
    if (lane == kWave - 1) s_sum[odd][wave] = sum;
    __syncthreads();                    // s_sum[odd] is written again two chunks, so one barrier, later
    sum += carry;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      if (w < wave) sum += s_sum[odd][w];
      carry += s_sum[odd][w];
    }
    if (b < batch) node_indptr[b + 1] = sum;
  }
}

}  // namespace

hipError_t launch_select_reanchor(int batch, int B, int Kmax, const float* conf, const int* K, int* p_out,
                                  double* r_out, hipStream_t stream) {
  hipLaunchKernelGGL(select_reanchor_kernel, dim3(batch), dim3(kSelectThreads), 0, stream, B, Kmax, conf, K,
                     p_out, r_out);
  return hipGetLastError();
}

hipError_t launch_tree_indptr(int batch, int B, int Kmax, const int* K, const int* p, int* node_indptr,
                              hipStream_t stream) {
  hipLaunchKernelGGL(tree_indptr_kernel, dim3(1), dim3(kIndptrThreads), 0, stream, batch, B, Kmax, K, p,
                     node_indptr);
  return hipGetLastError();
}

}  // namespace d2sd
