// Candidate-tree build (sec. 3.2 branch construction; sec. 3.3 (ii)-(iii)).
//
// One workgroup per request. The tree is produced in closed form: with the
// re-anchor positions sorted ascending and branch k (0-based rank) starting at
// node off_k = B + sum_{k' < k} (B - p_k'), the node n >= B of branch k sits at
// block position p_k + (n - off_k), and its ancestor-or-self set is the main
// prefix {0 .. p_k - 1} plus the branch run {off_k .. n}. A main node j sees
// {0 .. j}. Every mask word is therefore the union of two bit ranges, which is
// computed directly instead of walking parent pointers.
//
// The build is latency-bound. Positions and branch starts are ranked, summed
// and counted by lane reads, with one barrier; ranked in LDS, with the starts
// summed by one thread and searched by every node, the build of
// 64 trees of 40-110 nodes took 4.15 us, now 3.9.
#include "launchers.h"

namespace d2sd {

namespace {

constexpr int kTreeThreads = 256;
constexpr int kMaxNodes = D2SD_MAX_B + D2SD_MAX_B * (D2SD_MAX_B - 1) / 2;  // 2080
// A node's branch is counted among up to kCounted starts by lane reads, and
// searched among more in LDS: 64 trees of 63 branches 98.0 -> 82.6 us, 4096 of
// 15 13.5 -> 12.5; 64 of 8 are counted in 3.4 (searched linearly in LDS: 3.6).
constexpr int kCounted = 12;

__global__ __launch_bounds__(kTreeThreads) void tree_build_kernel(
    int B, int Kmax, const int* __restrict__ K, const int* __restrict__ p,
    const int* __restrict__ node_indptr, int total_nodes, int mask_words, int* __restrict__ parent,
    int* __restrict__ depth, int* __restrict__ path_id, uint32_t* __restrict__ anc_mask,
    int* __restrict__ path_leaf) {
  __shared__ int s_p[D2SD_MAX_B];      // positions sorted ascending
  __shared__ int s_off[D2SD_MAX_B];    // first nodes of their branches
  const int b = blockIdx.x;
  const int t = threadIdx.x;
  const int lane = t % kWave;
  // All global inputs in one batch of independent loads: the row of p is
  // read whole (it is Kmax entries long whatever K[b] is).
  const int k_raw = K[b];
  const int ip0 = node_indptr[b], ip1 = node_indptr[b + 1];
  const int raw = lane < min(Kmax, B - 1) ? p[(size_t)b * Kmax + lane] : 0;
  const int Kb = clampi(k_raw, 0, min(Kmax, B - 1));
  const int pt = clampi(raw, 1, B - 1);

  // Every wave ranks the positions in its lanes (K <= B - 1 <= 63): the rank
  // is the number of smaller ones (equal ones by index), and the branch starts
  // after the nodes of theirs. The waves write the same values.
  int rank = 0, off = B, end = B;
  for (int j = 0; j < Kb; ++j) {
    const int pj = lane_of(pt, j);
    const bool before = pj < pt || (pj == pt && j < lane);
    rank += before;
    off += before ? B - pj : 0;
    end += B - pj;
  }
  if (lane < Kb) {
    s_p[rank] = pt;
    s_off[rank] = off;
  }
  __syncthreads();

  const int base = clampi(ip0, 0, total_nodes);
  const int Nb = clampi(min(end, ip1 - base), 0, total_nodes - base);
  for (int n0 = 0; n0 < Nb; n0 += kTreeThreads) {   // all lanes: `off` is read from the ones of other nodes
    const int n = n0 + t;
    int k = -1;                                     // branch: starts at or before n, less one
    if (Kb <= kCounted)
      for (int j = 0; j < Kb; ++j) k += lane_of(off, j) <= n;
    else
      for (int step = 32; step > 0; step /= 2)
        if (k + step < Kb && s_off[k + step] <= n) k += step;
    if (n >= Nb) break;
    int pos, path, par, main_hi, br_lo, br_hi;
    if (n < B) {
      pos = n; path = 0; par = n - 1;
      main_hi = n + 1; br_lo = 0; br_hi = 0;
    } else {
      const int pk = s_p[k];
      pos = pk + (n - s_off[k]);
      path = k + 1;
      par = (n == s_off[k]) ? pk - 1 : n - 1;
      main_hi = pk; br_lo = s_off[k]; br_hi = n + 1;
    }
    const size_t g = (size_t)base + n;
    parent[g] = par;
    depth[g] = pos;
    path_id[g] = path;
    uint32_t* row = anc_mask + g * mask_words;
    for (int w = 0; w < mask_words; ++w) row[w] = range_bits(0, main_hi, w) | range_bits(br_lo, br_hi, w);
  }
  for (int k = t; k <= Kmax; k += kTreeThreads) {
    int leaf = -1;
    if (k == 0) leaf = B - 1;
    else if (k <= Kb) leaf = s_off[k - 1] + (B - s_p[k - 1]) - 1;
    path_leaf[(size_t)b * (Kmax + 1) + k] = leaf;
  }
}

// Trees given as parent arrays (node 0 the root, parent[n] < n): the
// third-level cascade and resampled chains. Node n walks its parent links,
// setting one mask bit per ancestor-or-self and counting the depth; a parent
// outside [0, n) makes n a root of its own. path_id[n] counts the nodes m in
// 1..n whose parent is not m - 1 (path starts).
//
// Latency-bound: a walk is as long as the node's depth. The links are staged
// in LDS, and as they only lead to smaller indexes, the mask words are filled
// from the highest down in a register and stored once each. The path starts
// are counted by ballot, kTreeThreads nodes at a time, with one barrier.
// 16 requests of 48-80 nodes: 6.0 us with links and masks walked in memory,
// 5.5 us now; one request: 5.4 -> 3.4 us.
__global__ __launch_bounds__(kTreeThreads) void tree_from_parents_kernel(
    const int* __restrict__ node_indptr, int total_nodes, int max_nodes, int mask_words,
    const int* __restrict__ parent, int* __restrict__ depth, int* __restrict__ path_id,
    uint32_t* __restrict__ anc_mask) {
  __shared__ short s_par[kMaxNodes];
  __shared__ int s_starts[2][kTreeThreads / kWave];
  const int b = blockIdx.x;
  const int t = threadIdx.x;
  const int lane = t % kWave, wave = t / kWave;
  const int base = clampi(node_indptr[b], 0, total_nodes);
  const int Nb = clampi(node_indptr[b + 1] - base, 0, min(max_nodes, total_nodes - base));
  int carry = 0;
  for (int n0 = 0, odd = 0; n0 < Nb; n0 += kTreeThreads, odd ^= 1) {
    const int n = n0 + t;
    const int q = n < Nb ? parent[base + n] : -1;
    if (n < Nb) s_par[n] = (short)(q >= 0 && q < n ? q : -1);
    const unsigned long long starts = __ballot(n > 0 && n < Nb && q != n - 1);
    if (lane == 0) s_starts[odd][wave] = __popcll(starts);
    __syncthreads();
    int id = carry + __popcll(starts & (~0ull >> (kWave - 1 - lane)));
#pragma unroll
    for (int w = 0; w < kTreeThreads / kWave; ++w) {
      if (w < wave) id += s_starts[odd][w];
      carry += s_starts[odd][w];
    }
    if (n < Nb) path_id[base + n] = id;
  }
  // every link is in LDS: the last chunk's barrier
  for (int n = t; n < Nb; n += kTreeThreads) {
    uint32_t* row = anc_mask + (size_t)(base + n) * mask_words;
    int d = -1, a = n;
    for (int w = mask_words - 1; w >= 0; --w) {
      uint32_t bits = 0u;
      for (; a >= 32 * w; a = s_par[a]) {
        bits |= 1u << (a & 31);
        ++d;
      }
      row[w] = bits;
    }
    depth[base + n] = d;
  }
}

}  // namespace

hipError_t launch_tree_from_parents(int batch, const int* node_indptr, int total_nodes, int max_nodes,
                                    int mask_words, const int* parent, int* depth, int* path_id,
                                    uint32_t* anc_mask, hipStream_t stream) {
  hipLaunchKernelGGL(tree_from_parents_kernel, dim3(batch), dim3(kTreeThreads), 0, stream, node_indptr,
                     total_nodes, max_nodes, mask_words, parent, depth, path_id, anc_mask);
  return hipGetLastError();
}

hipError_t launch_tree_build(int batch, int B, int Kmax, const int* K, const int* p,
                             const int* node_indptr, int total_nodes, int mask_words, int* parent,
                             int* depth, int* path_id, uint32_t* anc_mask, int* path_leaf,
                             hipStream_t stream) {
  hipLaunchKernelGGL(tree_build_kernel, dim3(batch), dim3(kTreeThreads), 0, stream, B, Kmax, K, p,
                     node_indptr, total_nodes, mask_words, parent, depth, path_id, anc_mask,
                     path_leaf);
  return hipGetLastError();
}

}  // namespace d2sd
