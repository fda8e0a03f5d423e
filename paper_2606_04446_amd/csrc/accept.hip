// Greedy longest-accepted-path selection and bonus token (sec. 2 "DFlash"
// prefix matching; sec. 3.3 (iv) longest accepted prefix across branches).
//
// One workgroup per request. Acceptance of a node is the AND of the match
// flags on its root path. It is computed for all nodes at once by pointer
// jumping (a parallel prefix scan along parent links): after round r every
// node holds the AND over its nearest 2^r path nodes and a pointer to its
// 2^r-th ancestor, so ceil(log2(B)) rounds cover any root path. The accepted
// length and the chosen node come from one max-reduction over the key
// (depth, -index), which implements "deepest accepted node, lowest canonical
// index on ties".
//
// The kernel is latency-bound (a few hundred nodes per request): every global
// input of a node is read in one batch of independent loads at the start and
// staged in LDS, so the match flags, the scan and the walk up the chosen path
// never wait on global memory again. The ancestor tables of the jumping rounds
// are kept, so that the chosen path's nodes are found by all depths at once.
// On 1 / 8 / 16 requests of 48-80 nodes, from launch to end: 3.7 / 5.5 / 5.4 us
// when one lane walked the path, 3.2 / 4.9 / 5.0 us now; what is left is the
// launch and the two dependent loads. The tables hold the match flags too:
// 52 KB keep three workgroups on a CU. With flags of their own and a level that
// nothing reads, 60 KB and two, 4096 requests took 17.6 us, now 11.7 (15.1 when
// one lane walked the path).
#include "launchers.h"

namespace d2sd {

namespace {

constexpr int kAcceptThreads = 256;
constexpr int kMaxNodes = D2SD_MAX_B + D2SD_MAX_B * (D2SD_MAX_B - 1) / 2;  // 2080
constexpr int kLevels = 6;             // 2^0 .. 2^5 add up to every distance below D2SD_MAX_B
// An entry of the ancestor tables: the ancestor's index + 1 (0: none), and
// whether all links up to it match.
constexpr int kOk = 1 << 12;
static_assert(kMaxNodes < kOk, "index bits");
static_assert(3 * (kMaxNodes * (2 * kLevels + 1 + 3 * 4) + 256) <= 160 * 1024, "three workgroups on a CU");

__global__ __launch_bounds__(kAcceptThreads) void accept_path_kernel(
    int B, const int* __restrict__ node_indptr, int total_nodes, const int* __restrict__ parent,
    const int* __restrict__ depth, const int* __restrict__ path_id, const int* __restrict__ draft,
    const int* __restrict__ argmax, int* __restrict__ accept_len, int* __restrict__ best_path,
    int* __restrict__ accept_node, int* __restrict__ path_nodes, int* __restrict__ out_tokens) {
  __shared__ uint16_t s_up[kLevels][kMaxNodes];   // of the 2^r-th ancestor
  __shared__ uint8_t s_dep[kMaxNodes];
  __shared__ int s_tok[kMaxNodes];
  __shared__ int s_arg[kMaxNodes];
  __shared__ int s_pid[kMaxNodes];
  __shared__ int s_best[kAcceptThreads / kWave];

  const int b = blockIdx.x;
  const int t = threadIdx.x;
  const int base = clampi(node_indptr[b], 0, total_nodes);
  const int Nb = clampi(node_indptr[b + 1] - base, 0, min(kMaxNodes, total_nodes - base));

  for (int c = t; c < Nb; c += kAcceptThreads) {
    int par = parent[base + c];
    if (par < 0 || par >= c) par = -1;   // canonical order puts parents first
    s_up[0][c] = (uint16_t)(par + 1);
    s_tok[c] = draft[base + c];
    s_arg[c] = argmax[base + c];
    s_pid[c] = path_id[base + c];
    s_dep[c] = (uint8_t)clampi(depth[base + c], 0, B - 1);
  }
  __syncthreads();
  for (int c = t; c < Nb; c += kAcceptThreads) {
    const int up = s_up[0][c];
    if (up == 0 || s_tok[c] == s_arg[up - 1]) s_up[0][c] = (uint16_t)(up | kOk);
  }
  __syncthreads();
  // An entry joined with its ancestor's reaches twice as far.
  auto joined = [&](int level, int c) {
    const int e = s_up[level][c];
    const int up = e & (kOk - 1);
    return up == 0 ? e : s_up[level][up - 1] & (e | (kOk - 1));
  };
  int level = 0;
  for (; 2 << level < B; ++level) {
    for (int c = t; c < Nb; c += kAcceptThreads) s_up[level + 1][c] = (uint16_t)joined(level, c);
    __syncthreads();
  }

  // key = depth * 65536 + (65535 - index) over accepted nodes; the root is
  // always accepted, so the maximum exists whenever Nb > 0.
  int best = -1;
  for (int c = t; c < Nb; c += kAcceptThreads)
    if (joined(level, c) & kOk) best = max(best, (int)s_dep[c] * 65536 + (65535 - c));
  // every key but "none" is >= 0; the scan's last lane holds the maximum
  const int top = lane_of(wave_scan<true>(best + 1), kWave - 1) - 1;
  if ((t % kWave) == 0) s_best[t / kWave] = top;
  __syncthreads();
  if (t >= kWave) return;                      // B <= 64: one wave writes the path
  best = top;
#pragma unroll
  for (int w = 1; w < kAcceptThreads / kWave; ++w) best = max(best, s_best[w]);
  const int L = best < 0 ? 0 : best / 65536;
  const int chosen = best < 0 ? -1 : 65535 - best % 65536;
  // Lane d: the ancestor of the chosen node at distance L - d, by its binary
  // digits; all depths at once instead of a walk of L dependent reads.
  int node = t <= L ? chosen : -1;
  for (int r = 0, steps = L - t; r < kLevels && (1 << r) <= L; ++r)
    if (node >= 0 && ((steps >> r) & 1)) node = (s_up[r][node] & (kOk - 1)) - 1;
  const int next = __shfl_down(node, 1);       // the path's node at depth d + 1
  if (t < B) {
    int tok = -1;
    if (t < L && next >= 0) tok = s_tok[next];
    if (t == L && chosen >= 0) tok = s_arg[chosen];
    path_nodes[(size_t)b * B + t] = node;
    out_tokens[(size_t)b * B + t] = tok;
  }
  if (t == 0) {
    accept_len[b] = L;
    best_path[b] = chosen >= 0 ? s_pid[chosen] : 0;
    accept_node[b] = chosen;
  }
}

}  // namespace

hipError_t launch_accept_path(int batch, int B, const int* node_indptr, int total_nodes,
                              const int* parent, const int* depth, const int* path_id,
                              const int* draft, const int* argmax, int* accept_len, int* best_path,
                              int* accept_node, int* path_nodes, int* out_tokens,
                              hipStream_t stream) {
  hipLaunchKernelGGL(accept_path_kernel, dim3(batch), dim3(kAcceptThreads), 0, stream, B,
                     node_indptr, total_nodes, parent, depth, path_id, draft, argmax, accept_len,
                     best_path, accept_node, path_nodes, out_tokens);
  return hipGetLastError();
}

}  // namespace d2sd
