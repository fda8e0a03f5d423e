// Verify attention over an even division of the batch's key tiles: the shape
// of grids that one work item per (request, KV head, row group, fixed split)
// would fill badly (few requests, ragged contexts).
//
// A stream is one (request b, KV head h, row group): up to twelve 32-row query
// tiles and the request's key tiles of 32 keys, context first, tree keys last.
// All streams, in (b, h, row group) order, form one line of costs; workgroup i
// of the grid (one per CU) takes the i-th equal share of it, so every CU gets
// the same amount of work whatever the context lengths are. The context
// lengths are known to the device only: each workgroup reads them (and the
// node offsets), scans the costs and finds its own share. A share holds the
// end of one stream, whole streams, the start of another; each part is a
// piece. A stream that is one piece is finalised in place; otherwise every
// piece writes a partial state, and the number of pieces and the workgroup of
// the first go to the workspace for the split merge. A workgroup has at most
// one piece that continues a stream and one that a later workgroup continues,
// so two slots per workgroup hold all partial states. Their outputs are fp32: rounded to
// bf16 a piece costs as much accuracy as the rounding of the result, however
// many there are.
//
// Twelve waves, one query tile each. The key tiles go through a ring of LDS
// slots filled by LDS DMA, several steps deep: a piece is a short stream whose
// copies have to be in flight early, and at few rows per key the kernel is
// bound by HBM, which takes tens of KB in flight per CU. A bf16 step is two
// key tiles, whose score chains run interleaved and whose softmax is one. An
// fp32 step is bound by the matrix pipes, which a stream of few query tiles
// would fill unevenly: there the waves form KG = min(2, 12 / T) key groups,
// each taking every KG-th key tile, merged through LDS at the end of a piece.
//
// The scheduling is integer code with divisions; one wave does it and hands
// the pieces to the others through LDS (done by all twelve it took 5 us of a
// 20 us call: three waves share a SIMD's issue slots).
//
// Inside a slot the 16-byte chunks are placed so that every read of a tile is
// one per-lane address plus an immediate: K in blocks of 8 rows x 8 chunks,
// chunk-major (the 32 rows of one chunk, read as the MFMA A operand, fall on
// all banks because octets of rows are 128 bytes apart modulo 256), V in
// blocks of 8 rows x 64 bytes (bf16, one transposing read each) or row-major
// (fp32). Each 1 KB block is one DMA instruction that reads whole 128-byte
// lines. A lane's addresses take two registers instead of twelve, which
// leaves room for K fragments in flight.
// A pass, fixed splits before: attention of 1 request of 32k tokens 73.7 -> 53.0
// us (of which the kernel moves its 134 MB in 46); a verify step of 8 of 1k-8k
// 98.7 -> 76.9; of 16 of 0-8k without host offsets 190 -> 131; fp32 attention, 4
// of 300-3000, 216 -> 91 (58 TFLOP/s over the whole pass).
// A call on little work is bound by its start: about 3 us until a workgroup
// has its piece, 2 until the query rows and page ids are there, 4 until the
// first tiles of all CUs have arrived, 2 for the stores.
#include "attention_device.h"

namespace d2sd {

namespace {

namespace bal {
constexpr int COPY_WAVES = 8;
constexpr int MAX_BATCH = kBalancedMaxBatch;
constexpr int PER_LANE = MAX_BATCH / kWave;   // requests per lane of the scheduling wave
constexpr int CHUNK_TILES = 1024;             // key tiles whose page ids are staged at a time
constexpr int KT = 32;                        // keys per tile
constexpr int WAVES = kBalWaves;
constexpr int THREADS = WAVES * kWave;
constexpr int FIRST_COPY = WAVES - COPY_WAVES;   // the copying waves are the last ones: few query tiles leave them idle
}  // namespace bal

template <typename T>
struct BalTile;
template <>
struct BalTile<__bf16> {
  static constexpr int ROW_BYTES = kD * 2;
  static constexpr int OCT_STRIDE = 8 * ROW_BYTES + 128;       // K: octet of rows, padded
  static constexpr int K_BYTES = 4 * OCT_STRIDE;
  static constexpr int SLOT = K_BYTES + bal::KT * ROW_BYTES;
  static constexpr int SLOTS = 8;
  static constexpr int MAX_KG = 1;
  static constexpr int STEP = 2;                               // key tiles per step and key group
  static constexpr int COPIES = 1;                             // 1 KB K (and V) blocks per copy wave and tile
  // What a key tile costs beside `tiles` query tiles, in units of 0.056 us
  // (0.064 from HBM). Measured per key tile and CU, of 8 and 16 requests from
  // the Infinity Cache and from HBM, in us: 1-4 query tiles 0.57 / 0.71 (the
  // arrival of its 16 KB), 5 0.80 / 0.93, 6 0.81 / 1.00, 7 0.87 / 1.08,
  // 8 0.95 / 1.15, 9 1.18 / 1.34, 10 1.25 / 1.36, 12 1.35 / 1.55: a step for
  // each query tile that a SIMD's waves take in turn, and less for each tile.
  // Counted as whole rounds (8, 8, 12 for up to 4, 8 and 12 tiles), CUs whose
  // requests had few tiles waited for the others: 16 requests of 0-8k tokens
  // and 40-110 nodes took 123.1 us (mean of eight batches), now 119.6.
  __device__ static __forceinline__ int cost(int tiles, int) { return max(MIN_COST, tiles + 3 * ((tiles + 3) >> 2) + 3); }
  static constexpr int MIN_COST = kBalMinCostBf16;
  static constexpr int OVERHEAD = kBalOverheadBf16;            // start and end of a stream, about 9 us (96: 5% slower, 144-256 level)
};
template <>
struct BalTile<float> {
  static constexpr int ROW_BYTES = kD * 4;
  static constexpr int OCT_STRIDE = 8 * ROW_BYTES + 128;
  static constexpr int K_BYTES = 4 * OCT_STRIDE;
  static constexpr int SLOT = K_BYTES + bal::KT * ROW_BYTES;
  static constexpr int SLOTS = 4;
  static constexpr int MAX_KG = 2;
  static constexpr int STEP = 1;
  static constexpr int COPIES = 2;
  // fp32 is MFMA bound: a quarter of a round of one query tile per SIMD.
  __device__ static __forceinline__ int cost(int tiles, int kg) {
    return max(MIN_COST, kg == 1 ? (tiles + 3) & ~3 : 2 * ((tiles + 1) >> 1));
  }
  static constexpr int MIN_COST = kBalMinCostF32;
  static constexpr int OVERHEAD = kBalOverheadF32;             // against 8: 4 requests of 300-3000 tokens 93.7 -> 92.0 us
};

// Sizes of one request and what they cost.
struct BalReq {
  int node_base, Nb, C;
  int T, rg, tpg;       // query tiles, row groups, tiles per row group
  int kg;               // key groups
  int n_ctx, n_tiles;   // context key tiles, all key tiles
  int cost;             // per key tile
  int work;             // per stream, without its start: max(n_tiles, 1) * cost
  int streams;          // hkv * rg (0: no rows)
};

// a / b for a >= 0, b > 0 and a quotient below 2^20, whose float estimate is
// off by one at most (an integer division is 20 instructions).
__device__ __forceinline__ int quick_div(int a, int b) {
  int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
  const int r = a - q * b;
  q += r >= b;
  q -= r < 0;
  return q;
}

template <typename T>
__device__ __forceinline__ BalReq bal_request(const Params& p, int node_base, int Nb, int C) {
  using BT = BalTile<T>;
  BalReq r;
  r.node_base = node_base;
  r.Nb = Nb;
  r.C = C;
  r.T = ceil_div(Nb * p.G, kRowsPerTile);
  r.rg = max(1, ceil_div(r.T, bal::WAVES));
  r.tpg = r.rg == 1 ? max(1, r.T) : quick_div(r.T + r.rg - 1, r.rg);
  r.kg = BT::MAX_KG == 2 && r.tpg <= bal::WAVES / 2 ? 2 : 1;
  r.n_ctx = p.stage != D2SD_STAGE_TREE ? ceil_div(C, bal::KT) : 0;
  r.n_tiles = r.n_ctx + (p.stage != D2SD_STAGE_PREFIX ? ceil_div(Nb, bal::KT) : 0);
  r.cost = BT::cost(r.tpg, r.kg);
  r.work = max(1, r.n_tiles) * r.cost;
  r.streams = r.T > 0 ? p.hkv * r.rg : 0;
  return r;
}

// The part of a stream that one workgroup takes.
struct __attribute__((aligned(16))) BalPiece {
  int b, sidx;          // stream sidx = h * rg + row group of request b
  int h, rgi;
  int node_base, Nb, C;
  int row0;             // first row of the row group
  int tiles, kg;        // its query tiles; key groups
  int t0, t1;           // key tiles
  int index, count;     // of the stream's pieces; count 0: no more pieces
  int last;             // the workgroup's share ends with this piece
  int pad;
};

// The same value, unknown to the optimiser: what a phase derives from its lane
// is computed there again, instead of being kept (and spilled) across the others.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Wait until at most `tiles` of the wave's later tile copies (2 * COPIES DMAs
// each) are outstanding; sync_tiles: and all its LDS reads done, then the
// workgroup barrier.
template <int COPIES>
__device__ __forceinline__ void wait_tiles(int tiles) {
  // s_waitcnt: vmcnt 2 * COPIES * tiles, the other counters at their maxima
  switch (tiles) {
    case 0: __builtin_amdgcn_s_waitcnt(0x0f70); break;
    case 1: __builtin_amdgcn_s_waitcnt(0x0f70 | 2 * COPIES); break;
    case 2: __builtin_amdgcn_s_waitcnt(0x0f70 | 4 * COPIES); break;
    case 3: __builtin_amdgcn_s_waitcnt(0x0f70 | 6 * COPIES); break;
    default: __builtin_amdgcn_s_waitcnt(0x0f70 | ((8 * COPIES) & 15) | ((8 * COPIES) >> 4) << 14); break;   // at most 4
  }
}
template <int COPIES>
__device__ __forceinline__ void sync_tiles(int tiles) {
  switch (tiles) {
    case 0: sync_keep<0>(); break;
    case 1: sync_keep<2 * COPIES>(); break;
    case 2: sync_keep<4 * COPIES>(); break;
    case 3: sync_keep<6 * COPIES>(); break;
    case 4: sync_keep<8 * COPIES>(); break;
    case 5: sync_keep<10 * COPIES>(); break;
    default: sync_keep<12 * COPIES>(); break;   // at most SLOTS - 2 = 6 tiles are ever queued past the next
  }
}

// ---- per-type pieces: copy of one tile, scores, probabilities x V ----

// Where copy wave w puts its blocks of a tile, and which row and byte column
// of the tile a lane fetches. K2, V2: LDS distance of the second blocks (fp32:
// sixteen rows further, on the tile's second page).
template <typename T>
struct BalCopy;
template <>
struct BalCopy<__bf16> {   // block w: rows 8 (w / 2) .., 128-byte half w % 2, of K and of V
  using BT = BalTile<__bf16>;
  static constexpr uint32_t K2 = 0, V2 = 0;
  __device__ static __forceinline__ int krow(int w, int lane) { return 8 * ((w >> 1) & 3) + (lane & 7); }
  __device__ static __forceinline__ int kcol(int w, int lane) { return (w & 1) * 128 + (lane >> 3) * 16; }
  __device__ static __forceinline__ int vrow(int w, int lane) { return 8 * ((w >> 1) & 3) + ((lane >> 2) & 7); }
  __device__ static __forceinline__ int vcol(int w, int lane) {
    return (w & 1) * 128 + (lane >> 5) * 64 + (lane & 3) * 16;
  }
  __device__ static __forceinline__ uint32_t kdst(int w) { return ((w >> 1) & 3) * BT::OCT_STRIDE + (w & 1) * 1024; }
  __device__ static __forceinline__ uint32_t vdst(int w) { return BT::K_BYTES + (w & 7) * 1024; }
};
template <>
struct BalCopy<float> {    // K: rows 8 (w / 4) .., 128-byte quarter w % 4; V: two whole rows
  using BT = BalTile<float>;
  static constexpr uint32_t K2 = 2 * BT::OCT_STRIDE, V2 = 16 * BT::ROW_BYTES;
  __device__ static __forceinline__ int krow(int w, int lane) { return 8 * ((w >> 2) & 1) + (lane & 7); }
  __device__ static __forceinline__ int kcol(int w, int lane) { return (w & 3) * 128 + (lane >> 3) * 16; }
  __device__ static __forceinline__ int vrow(int w, int lane) { return 2 * (w & 7) + (lane >> 5); }
  __device__ static __forceinline__ int vcol(int w, int lane) { return (lane & 31) * 16; }
  __device__ static __forceinline__ uint32_t kdst(int w) { return ((w >> 2) & 1) * BT::OCT_STRIDE + (w & 3) * 1024; }
  __device__ static __forceinline__ uint32_t vdst(int w) { return BT::K_BYTES + (w & 7) * 1024; }
};

// O^T accumulators: bf16 o[dt] holds dims 32 dt .. 32 dt + 31 (slot i of lane
// half hf: dim 32 dt + (i/4) 8 + hf 4 + i%4); fp32 o[dt] holds dims 4 m + dt,
// m = (i/4) 8 + hf 4 + i%4.
__device__ __forceinline__ void bal_scores(const char* slot, int ka, const bf16x8 (&q)[8], f32x16& s) {
  s = f32x16{};
#pragma unroll
  for (int st = 0; st < 8; ++st) {
    const bf16x8 a = __builtin_bit_cast(bf16x8, lds_b128(slot, ka + st * 128));
    s = mfma(a, q[st], s);
  }
}
__device__ __forceinline__ void bal_scores(const char* slot, int ka, const float (&q)[64], f32x16& s) {
  s = f32x16{};
#pragma unroll
  for (int st = 0; st < 16; ++st) {
    if (st % 2 == 0) __builtin_amdgcn_sched_barrier(0);
    const uint4 u = lds_b128(slot, ka + st * 128);
    s = mfma(__uint_as_float(u.x), q[4 * st], s);
    s = mfma(__uint_as_float(u.y), q[4 * st + 1], s);
    s = mfma(__uint_as_float(u.z), q[4 * st + 2], s);
    s = mfma(__uint_as_float(u.w), q[4 * st + 3], s);
  }
}

// Per-lane LDS addresses within a slot: K (A operand) and V (transposed A operand).
template <typename T>
__device__ __forceinline__ int bal_kaddr(int lane) {
  const int r = lane & 31, hf = lane >> 5;
  return (r >> 3) * BalTile<T>::OCT_STRIDE + hf * (int)(sizeof(T) / 2) * 1024 + (r & 7) * 16;
}
template <typename T>
__device__ __forceinline__ int bal_vaddr(int lane);
template <>
__device__ __forceinline__ int bal_vaddr<__bf16>(int lane) {
  const int grp = lane >> 4, i = lane & 15;   // 16-lane group: dims (grp & 1) 16 .., keys + 4 (grp >> 1)
  return BalTile<__bf16>::K_BYTES + (4 * (grp >> 1) + (i >> 2)) * 64 + (grp & 1) * 32 + (i & 3) * 8;
}
template <>
__device__ __forceinline__ int bal_vaddr<float>(int lane) {
  return BalTile<float>::K_BYTES + (lane >> 5) * 4 * BalTile<float>::ROW_BYTES + (lane & 31) * 16;
}

// The exponent reference of a row that has seen no key: below every score,
// and finite, so that a masked score (-inf) less it is still -inf.
constexpr float kNoReference = -3.0e38f;

// Moves the exponent reference of a query row (m, in log2 units) when the
// tile's largest score exceeds it by more than `slack`, rescaling O and l. It is
// the score itself, so that the largest probability is exactly 1 in bf16 (as a
// whole number above it, it left a row's dominant key with a rounding error).
__device__ __forceinline__ void bal_reference(float mx, float slack, float c2, float& m, float& l, f32x16 (&o)[4]) {
  const float top = xhalf_max(mx) * c2;
  if (__ballot(top - m > slack)) {
    const float m_new = fmaxf(m, top);
    const float alpha = __builtin_amdgcn_exp2f(m - m_new);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
    l *= alpha;
    m = m_new;
  }
}
__device__ __forceinline__ float lane_max(const f32x16& s) {
  float mx = s[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
  return mx;
}

// bf16 probabilities of a tile in B-operand order, their sum added to l.
__device__ __forceinline__ void bal_probs(const f32x16& s, float moff, float c2, float& l, bf16x8* pf) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float la = 0.0f, lb = 0.0f;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[8 * t + j], c2, -moff));
#pragma unroll
    for (int j = 0; j < 8; j += 4) {
      la = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[j], v[j + 1]}, ones, la, false);
      lb = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[j + 2], v[j + 3]}, ones, lb, false);
    }
    pf[t] = v;
  }
  l += la + lb;
}
// Online softmax of one 32-key tile, then O^T += V^T P^T (fp32).
__device__ __forceinline__ void bal_update(const char* slot, int va, f32x16& s, float& m_run, float& l_run,
                                           f32x16 (&o)[4], float c2) {
  bal_reference(lane_max(s), 0.0f, c2, m_run, l_run, o);
  const float moff = m_run;
  float lsum = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c2, -moff));
    lsum += s[i];
  }
  l_run += lsum;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i % 2 == 0) __builtin_amdgcn_sched_barrier(0);
    const uint4 u = lds_b128(slot, va + ((i >> 2) * 8 + (i & 3)) * BalTile<float>::ROW_BYTES);
    o[0] = mfma(__uint_as_float(u.x), s[i], o[0]);
    o[1] = mfma(__uint_as_float(u.y), s[i], o[1]);
    o[2] = mfma(__uint_as_float(u.z), s[i], o[2]);
    o[3] = mfma(__uint_as_float(u.w), s[i], o[3]);
  }
}

// Keys of the tile outside `vis` (bit k: key k) get a score of -inf; slot i is
// key (i/4) 8 + hf 4 + i%4.
__device__ __forceinline__ void bal_mask(f32x16& s, uint32_t vis, int hf) {
  const uint32_t w = vis >> (hf * 4);
#pragma unroll
  for (int i = 0; i < 16; ++i) s[i] = ((w >> ((i >> 2) * 8 + (i & 3))) & 1u) ? s[i] : -INFINITY;
}

template <typename T>
struct BalQ;
template <>
struct BalQ<__bf16> { using type = bf16x8[8]; };
template <>
struct BalQ<float> { using type = float[64]; };

// The state of one piece in a wave.
template <typename T>
struct BalWave {
  typename BalQ<T>::type q;
  f32x16 o[4];
  float m, l;
};

// A wave's 32 query rows from global memory to its registers by way of LDS
// (`area`: one K tile's bytes of the wave's own): a lane holds one row, and
// loading it straight would touch 64 lines per instruction, 6000 cycles for
// the twelve waves of a CU. fp32 rows take two passes.
struct BalRows {
  int row0, rows;        // the tile's first row in the request's stack, the stack's rows
  int node_base, h;
  __device__ __forceinline__ size_t global_row(const Params& p, int r) const {   // r < 2^21
    const int n = (int)(((float)r + 0.5f) * p.inv_G);
    return (size_t)((node_base + n) * p.hq + h * p.G + r - n * p.G);
  }
};
template <typename T>
__device__ __forceinline__ void bal_queue_q(const Params& p, const BalRows& rw, char* area, int lane, int pass) {
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    const char* src = static_cast<const char*>(p.q) +
                      rw.global_row(p, min(rw.row0 + 8 * o + (lane & 7), rw.rows - 1)) * BalTile<T>::ROW_BYTES +
                      pass * 128 + (lane >> 3) * 16;
#pragma unroll
    for (int half = 0; half < 2; ++half)
      dma16(src + half * (BalTile<T>::ROW_BYTES / 2), lds_addr(area) + o * BalTile<__bf16>::OCT_STRIDE + half * 1024);
  }
}
__device__ __forceinline__ void bal_read_q(const char* area, int lane, int, bf16x8 (&q)[8]) {
  const int ka = bal_kaddr<__bf16>(lane);
#pragma unroll
  for (int i = 0; i < 8; ++i) q[i] = __builtin_bit_cast(bf16x8, lds_b128(area, ka + i * 128));
}
__device__ __forceinline__ void bal_read_q(const char* area, int lane, int pass, float (&q)[64]) {
  const int ka = bal_kaddr<__bf16>(lane);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint4 u = lds_b128(area, ka + i * 128);
    q[32 * pass + 4 * i] = __uint_as_float(u.x); q[32 * pass + 4 * i + 1] = __uint_as_float(u.y);
    q[32 * pass + 4 * i + 2] = __uint_as_float(u.z); q[32 * pass + 4 * i + 3] = __uint_as_float(u.w);
  }
}

// The wave's output rows, scaled by inv, as type Out to row_at(row) by way of
// LDS, so that a store instruction writes whole rows (four of bf16, two of
// fp32). fp32 goes in two passes of 16 rows.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}
template <typename T, typename Out, typename Row>
__device__ __forceinline__ void bal_store(const BalRows& rw, char* area, int lane, f32x16 (&o)[4], float inv, Row row_at) {
  constexpr int ROW_BYTES = kD * sizeof(Out);
  constexpr int PASSES = sizeof(Out) / 2;
  constexpr int STRIDE = ROW_BYTES + 16;                    // of a staged row
  constexpr int LANES = ROW_BYTES / 16;                     // per row
  constexpr int ROWS = kRowsPerTile / PASSES;               // per pass
  const int hf = lane >> 5, r = lane & 31;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) o[dt] *= inv;
#pragma unroll 1
  for (int pass = 0; pass < PASSES; ++pass) {
    char* mine = area + (r % ROWS) * STRIDE;
    if constexpr (PASSES == 1) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<uint2*>(mine + dt * 64 + q4 * 16 + hf * 8) =
              make_uint2(pack_bf16(o[dt][4 * q4], o[dt][4 * q4 + 1]), pack_bf16(o[dt][4 * q4 + 2], o[dt][4 * q4 + 3]));
    } else if constexpr (sizeof(T) == 2) {
      if (r / ROWS == pass) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<float4*>(mine + dt * 128 + q4 * 32 + hf * 16) =
                make_float4(o[dt][4 * q4], o[dt][4 * q4 + 1], o[dt][4 * q4 + 2], o[dt][4 * q4 + 3]);
      }
    } else {
      if (r / ROWS == pass) {      // a register at a time: four adjacent dims sit in four accumulators
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            *reinterpret_cast<float*>(mine + 16 * ((i >> 2) * 8 + hf * 4 + (i & 3)) + 4 * dt) = o[dt][i];
      }
    }
#pragma unroll
    for (int i = 0; i < ROWS * LANES / kWave; ++i) {
      const int rr = i * (kWave / LANES) + lane / LANES;
      const uint4 v = lds_b128(area, rr * STRIDE + (lane % LANES) * 16);
      const int row = rw.row0 + pass * ROWS + rr;
      if (row < rw.rows) *reinterpret_cast<uint4*>(row_at(row) + (lane % LANES) * 16) = v;
    }
  }
}

// One key tile of the pipeline: the probabilities of tile j from its scores s
// beside the score products of tile j + 1, then O^T += V^T P^T of tile j. The
// scores of j + 1 replace s.
//
// A matrix instruction that waits for the matrix pipe holds the SIMD's vector
// issue, so a burst of them keeps the other waves from issuing anything: two
// waves that ran score products, softmax and V products one after the other
// took as long as one after the other (1235 cycles a tile each). Six vector
// instructions go between two score products here, which they take as long as.
// K fragments are read two products ahead, V fragments during the last score
// products, each ordered by scheduling barriers.
//
// The sum of the probabilities says where a score may exceed the row's
// exponent reference by 2^8; only then are the tile's scores computed again
// (scores_again), the reference moved and the probabilities taken again.
template <typename Again>
__device__ __forceinline__ void bal_tile(const char* ring, int va, int ka, int ka_next, uint4 (&a)[2], f32x16& s,
                                         BalWave<__bf16>& st, float c2, Again scores_again) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  s16x4 v[4][2];
  auto load_v = [&](int ks, int dt) {
    v[dt][0] = lds_tr16(ring, va + (2 * ks) * 2048 + dt * 512);
    v[dt][1] = lds_tr16(ring, va + (2 * ks + 1) * 2048 + dt * 512);
  };
  uint4 kf[8];
  kf[0] = a[0];
  kf[1] = a[1];
  f32x16 sn = {};
  bf16x8 pf[2];
  float ls[2] = {0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (k + 2 < 8) kf[k + 2] = lds_b128(ring, ka + (k + 2) * 128);
    if (k >= 6) load_v(0, k - 6);
    sn = mfma(__builtin_bit_cast(bf16x8, kf[k]), st.q[k], sn);
    const float e0 = __builtin_amdgcn_exp2f(fmaf(s[2 * k], c2, -st.m));
    const float e1 = __builtin_amdgcn_exp2f(fmaf(s[2 * k + 1], c2, -st.m));
    const bf16x2 pr = {(__bf16)e0, (__bf16)e1};
    pf[k >> 2][2 * (k & 3)] = pr[0];
    pf[k >> 2][2 * (k & 3) + 1] = pr[1];
    ls[k & 1] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, ls[k & 1], false);
    __builtin_amdgcn_sched_barrier(0);
  }
  float lt = ls[0] + ls[1];
  if (__ballot(!(lt < 256.0f))) {
    f32x16 r;
    scores_again(r);
    bal_reference(lane_max(r), 0.0f, c2, st.m, st.l, st.o);
    lt = 0.0f;
    bal_probs(r, st.m, c2, lt, pf);
  }
  st.l += lt;
  __builtin_amdgcn_sched_barrier(0);
  load_v(0, 2);
  load_v(0, 3);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const s16x8 a8 = {v[dt][0][0], v[dt][0][1], v[dt][0][2], v[dt][0][3],
                        v[dt][1][0], v[dt][1][1], v[dt][1][2], v[dt][1][3]};
      st.o[dt] = mfma(__builtin_bit_cast(bf16x8, a8), pf[ks], st.o[dt]);
      if (ks == 0) load_v(1, dt);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  a[0] = lds_b128(ring, ka_next);
  a[1] = lds_b128(ring, ka_next + 128);
  s = sn;
  __builtin_amdgcn_sched_barrier(0);
}

template <typename T>
struct BalShared {
  using BT = BalTile<T>;
  __attribute__((aligned(1024))) char ring[BT::SLOTS * BT::SLOT];
  int pid[2 * bal::CHUNK_TILES + 8];
  int pref[bal::MAX_BATCH + 1];
  int node[bal::MAX_BATCH], nb[bal::MAX_BATCH], ctx[bal::MAX_BATCH];
  int streams[bal::MAX_BATCH];   // of the requests before, within the scheduling lane
  int share, end;       // cost units per workgroup; where this one's share ends
  int start;            // what the start of a stream costs
  BalPiece piece[2];
};

// The workgroup's first piece at or after stream sidx of request b, and the
// stream's share limits; written to `out` by lane 0.
template <typename T>
__device__ __forceinline__ void bal_seek(const Params& p, const BalShared<T>& sh, int batch, int b, int sidx,
                                         BalPiece& out, int lane) {
  const int item = blockIdx.x;
  const int share = uni(sh.share), hi = uni(sh.end), start = uni(sh.start);
  BalPiece pc{};
  for (; b < batch;) {
    const int base = uni(sh.pref[b]);
    if (base >= hi) break;
    const BalReq rq = bal_request<T>(p, uni(sh.node[b]), uni(sh.nb[b]), uni(sh.ctx[b]));
    for (; sidx < rq.streams; ++sidx) {
      const int s0 = base + sidx * (start + rq.work);
      if (s0 >= hi) break;
      const int x0 = s0 + start;                            // cost position of tile 0
      const int n = max(1, rq.n_tiles);
      const int i0 = uni(quick_div(x0, share)), i1 = uni(quick_div(x0 + (n - 1) * rq.cost, share));
      if (item < i0 || item > i1) continue;
      pc.b = b; pc.sidx = sidx;
      pc.h = rq.rg == 1 ? sidx : uni(quick_div(sidx, rq.rg));
      pc.rgi = sidx - pc.h * rq.rg;
      pc.node_base = rq.node_base; pc.Nb = rq.Nb; pc.C = rq.C;
      pc.row0 = pc.rgi * rq.tpg * kRowsPerTile;
      pc.last = item < i1;
      pc.tiles = min(rq.tpg, rq.T - pc.rgi * rq.tpg);
      pc.kg = rq.kg;
      pc.t0 = item == i0 ? 0 : uni(quick_div(item * share - x0 + rq.cost - 1, rq.cost));
      pc.t1 = min(rq.n_tiles, item == i1 ? n : uni(quick_div((item + 1) * share - x0 + rq.cost - 1, rq.cost)));
      pc.index = item - i0;
      pc.count = i1 - i0 + 1;
      break;
    }
    if (pc.count) break;
    ++b;
    sidx = 0;
  }
  if (lane == 0) out = pc;
}

// The scheduling wave: costs before each request, the share of a workgroup,
// and the piece this one starts with.
template <typename T>
__device__ __forceinline__ void bal_schedule(const Params& p, BalShared<T>& sh, int batch, int lane) {
  const int per = ceil_div(batch, kWave);
  int node[bal::PER_LANE], end[bal::PER_LANE], ctx[bal::PER_LANE];
#pragma unroll
  for (int k = 0; k < bal::PER_LANE; ++k) {                 // every load before the first use
    const int b = lane * per + k;
    const bool in = k < per && b < batch;
    node[k] = in ? p.node_indptr[b] : 0;
    end[k] = in ? p.node_indptr[b + 1] : 0;
    ctx[k] = in ? p.ctx_len[b] : 0;
  }
  int sum = 0, count = 0, top_cost = 1;
  for (int k = 0; k < per; ++k) {
    const int b = lane * per + k;
    int nd = 0, en = 0, cx = 0;
#pragma unroll
    for (int i = 0; i < bal::PER_LANE; ++i)
      if (i == k) { nd = node[i]; en = end[i]; cx = ctx[i]; }
    nd = clampi(nd, 0, p.total_nodes);
    const int Nb = clampi(en - nd, 0, min(p.max_nodes, p.total_nodes - nd));
    const int C = clampi(cx, 0, p.max_ctx);
    const BalReq r = bal_request<T>(p, nd, Nb, C);
    if (b < batch) {
      sh.node[b] = nd; sh.nb[b] = Nb; sh.ctx[b] = C;
      sh.pref[b] = sum;
      sh.streams[b] = count;
    }
    sum += r.streams * r.work;
    count += r.streams;
    top_cost = max(top_cost, r.streams ? r.cost : 1);
  }
  // The start of a stream counts as four shares of the tiles at most: where
  // shares are short, more would leave workgroups without any tile.
  const int incl = wave_scan<false>(sum), incl_count = wave_scan<false>(count);
  const int start = min(BalTile<T>::OVERHEAD, 4 * ceil_div(lane_of(incl, 63), kBalWorkgroups));
  const int total = lane_of(incl, 63) + start * lane_of(incl_count, 63);
  // A share is at least one tile: every piece then holds a tile.
  const int share = max(ceil_div(total, kBalWorkgroups), lane_of(wave_scan<true>(top_cost), 63));
  const int lo = (int)blockIdx.x * share;
  if (lane == 0) {
    sh.share = share;
    sh.start = start;
    sh.end = min(lo + share, total);
  }
  // the request that holds cost position lo
  int at = -1;
  for (int k = 0; k < per; ++k) {
    const int b = lane * per + k;
    if (b >= batch) break;
    const int before = sh.pref[b] + incl - sum + start * (sh.streams[b] + incl_count - count);
    sh.pref[b] = before;
    if (before <= lo) at = b;
  }
  if (lane == 0) sh.pref[batch] = total;
  if (lo >= total) {
    if (lane == 0) sh.piece[0].count = 0;
    return;
  }
  // requests without rows cost nothing: the last one that starts at or before lo holds it
  const int b = lane_of(wave_scan<true>(at + 1), 63) - 1;
  const BalReq rq = bal_request<T>(p, uni(sh.node[b]), uni(sh.nb[b]), uni(sh.ctx[b]));
  bal_seek<T>(p, sh, batch, b, uni(quick_div(lo - uni(sh.pref[b]), start + rq.work)), sh.piece[0], lane);
}

// One key row of zeros.
__device__ const uint4 bal_zero_row[kD / 4] = {};

// Key tiles [t0, t1) of the piece's stream, page ids of the context ones
// staged from tile t0 on.
template <typename T>
__device__ __forceinline__ void bal_run(const Params& p, BalShared<T>& sh, const BalPiece& pc, int t0, int t1,
                                        int wave_s, int lane, bool active, int kg, const BalRows& rw, const char* q_area, BalWave<T>& st) {
  using BT = BalTile<T>;
  using CP = BalCopy<T>;
  constexpr int PAGE_SHIFT = BT::COPIES == 1 ? 12 : 13;         // bytes of a page of one KV head
  const int step = BT::STEP * (BT::MAX_KG == 2 ? pc.kg : 1);    // tiles
  constexpr int RING = BT::SLOTS * BT::SLOT;
  const int n = t1 - t0;
  const int cw = wave_s - bal::FIRST_COPY;
  const int n_ctx = p.stage != D2SD_STAGE_TREE ? ceil_div(pc.C, bal::KT) : 0;
  // whole context tiles from t0 on
  const int n_full = p.stage != D2SD_STAGE_TREE ? clampi(pc.C / bal::KT - t0, 0, n) : 0;
  const char* kc = static_cast<const char*>(p.k_cache);
  const char* vc = static_cast<const char*>(p.v_cache);
  const uint32_t kdst = lds_addr(sh.ring) + CP::kdst(cw);
  const uint32_t vdst = lds_addr(sh.ring) + CP::vdst(cw);
  // byte offset within a page of the chunk a lane fetches
  const uint32_t koff = (CP::krow(cw, lane) & 15) * BT::ROW_BYTES + CP::kcol(cw, lane);
  const uint32_t voff = (CP::vrow(cw, lane) & 15) * BT::ROW_BYTES + CP::vcol(cw, lane);

  // byte offset of the KV head's part of a page
  auto page_of = [&](int id) { return (size_t)(uint32_t)(clampi(id, 0, p.num_pages - 1) * p.hkv + pc.h) << PAGE_SHIFT; };

  // Queue tile j. Rows past the valid keys take K from the tile's first row
  // (their scores are masked) and zeros for V: their probabilities are 0, and
  // 0 * inf would make a row NaN that is infinite where the first key's V is.
  auto copy = [&](int j, uint32_t dst) {          // dst: byte offset of its slot
    if (j < n_full) {
#pragma unroll
      for (int c = 0; c < BT::COPIES; ++c) {
        const size_t off = page_of(uni(sh.pid[2 * j + (BT::COPIES == 1 ? (cw >> 2) : c)]));
        dma16s(kc + off, koff, dst + kdst + c * CP::K2);
        dma16s(vc + off, voff, dst + vdst + c * CP::V2);
      }
      return;
    }
    const int t = t0 + j;
    const bool tree = t >= n_ctx;
    const int key0 = (tree ? t - n_ctx : t) * bal::KT;
    const int nvalid = (tree ? pc.Nb : pc.C) - key0;
    auto src = [&](const char* cache, const char* rows, int r) {
      const int rs = r < nvalid ? r : 0;
      return tree ? rows + ((size_t)(pc.node_base + key0 + rs) * p.hkv + pc.h) * BT::ROW_BYTES
                  : cache + page_of(sh.pid[2 * j + (rs >> 4)]) + (rs & 15) * BT::ROW_BYTES;
    };
#pragma unroll
    for (int c = 0; c < BT::COPIES; ++c) {
      dma16(src(kc, static_cast<const char*>(p.k_tree), CP::krow(cw, lane) + 16 * c) + CP::kcol(cw, lane),
            dst + kdst + c * CP::K2);
      const int vr = CP::vrow(cw, lane) + 16 * c;
      const char* v = src(vc, static_cast<const char*>(p.v_tree), vr);
      if (vr >= nvalid) v = reinterpret_cast<const char*>(bal_zero_row);
      dma16(v + CP::vcol(cw, lane), dst + vdst + c * CP::V2);
    }
  };

  int cur = 0;                          // byte offset of the slot of the step's first tile
  int j0 = 0;
  auto after = [&](int at) { return at + step * BT::SLOT == RING ? 0 : at + step * BT::SLOT; };
  // Wait until the first `tiles` tiles from j0 on are there and every wave is
  // done with the step before, then queue the tiles that take its slots.
  int queued = 0;
  auto queue = [&](int to) {
    if (cw >= 0)
      for (; queued < to; ++queued) copy(queued, (queued % BT::SLOTS) * BT::SLOT);
    queued = to;
  };
  auto begin = [&](int tiles) {
    sync_tiles<BT::COPIES>(queued - min(j0 + tiles, queued));
    queue(min(j0 + BT::SLOTS, n));
  };
  // Scores outside the context, the tree or a row's ancestors become -inf.
  auto mask = [&](f32x16& sc, int j) {
    const int t = t0 + j;
    const bool tree = t >= n_ctx;
    const int k0 = (tree ? t - n_ctx : t) * bal::KT;
    const int nvalid = (tree ? pc.Nb : pc.C) - k0;
    uint32_t vis = nvalid >= 32 ? ~0u : ((1u << max(nvalid, 0)) - 1u);
    if (tree) {
      const int w = k0 >> 5;
      const int node = (int)(((float)min(rw.row0 + (lane & 31), rw.rows - 1) + 0.5f) * p.inv_G);
      vis &= w < p.mask_words ? p.anc_mask[(size_t)(pc.node_base + node) * p.mask_words + w] : 0u;
    }
    bal_mask(sc, vis, lane >> 5);
  };
  // Half the ring first: the copies of all CUs start together, and a longer
  // queue only delays its own first tiles. The query rows still lie in the
  // last slots.
  const int before_q = min(BT::SLOTS / 2, (RING - pc.tiles * pc.kg * BalTile<__bf16>::K_BYTES) / BT::SLOT);
  queue(min(q_area ? before_q : BT::SLOTS / 2, n));
  if constexpr (BT::COPIES == 1) {
    if (q_area) {
      if (active) {
        wait_tiles<BT::COPIES>(cw >= 0 ? queued : 0);
        bal_read_q(q_area, lane, 0, st.q);
      }
      if (queued < min(4, n)) begin(0);
    }
  }
  if constexpr (BT::COPIES == 1) {
    // Two tiles to a step. A step computes the scores of the next step's first
    // tile and reads the first K fragments of its second, so its wait covers
    // them too. In the steady state every tile a step queues is a whole
    // context tile: the step then chooses nothing, and its page ids are read a
    // step ahead.
    const int ka = bal_kaddr<T>(lane), va = bal_vaddr<T>(lane);
    const int n_steady = n_full - BT::SLOTS;        // steps from j0 <= n_steady queue only whole context tiles
    const int* pid = sh.pid + 2 * BT::SLOTS + (cw >> 2);
    int ph0 = 0, ph1 = 0;
    if (2 <= n_steady) {
      ph0 = pid[0];
      ph1 = pid[2];
    }
    if (n > 0) begin(4);
    auto next_slot = [&](int at) { return at + BT::SLOT == RING ? 0 : at + BT::SLOT; };
    uint4 a[2];
    f32x16 s;
    if (active && n > 0) {
      bal_scores(sh.ring, ka, st.q, s);
      if (n_full == 0) mask(s, 0);
      bal_reference(lane_max(s), 0.0f, p.c2, st.m, st.l, st.o);
      a[0] = lds_b128(sh.ring, ka + BT::SLOT);
      a[1] = lds_b128(sh.ring, ka + BT::SLOT + 128);
    }
    for (; j0 < n;) {
      const int next = next_slot(cur);
      if (active) {
        if (j0 >= n_full) {
          mask(s, j0);
          bal_reference(lane_max(s), 8.0f, p.c2, st.m, st.l, st.o);
        }
        bal_tile(sh.ring, va + cur, ka + next, ka + next_slot(next), a, s, st, p.c2, [&](f32x16& r) {
          bal_scores(sh.ring, ka + cur, st.q, r);
          if (j0 >= n_full) mask(r, j0);
        });
      }
      cur = next;
      ++j0;
      if (j0 & 1) continue;
      if (j0 >= n) break;
      if (j0 <= n_steady) {
        sync_keep<2 * (BT::SLOTS - 6)>();           // six tiles queued ahead, four of them awaited
        if (cw >= 0) {
          const int fill = (cur == 0 ? RING : cur) - 2 * BT::SLOT;
          const size_t off = page_of(uni(ph0));
          dma16s(kc + off, koff, kdst + fill);
          dma16s(vc + off, voff, vdst + fill);
          const size_t off1 = page_of(uni(ph1));
          dma16s(kc + off1, koff, kdst + fill + BT::SLOT);
          dma16s(vc + off1, voff, vdst + fill + BT::SLOT);
          pid += 4;
          ph0 = pid[0];          // the last ones read lie past the list, unused
          ph1 = pid[2];
        }
        queued = j0 + BT::SLOTS;
      } else {
        begin(4);
      }
    }
  } else {
    for (; j0 < n; j0 += step, cur = after(cur)) {
      begin(step);
      const int j = j0 + kg;
      if (active && j < n) {
        f32x16 s;
        bal_scores(sh.ring, bal_kaddr<T>(lane) + cur + kg * BT::SLOT, st.q, s);
        if (j >= n_full) mask(s, j);
        bal_update(sh.ring, bal_vaddr<T>(lane) + cur + kg * BT::SLOT, s, st.m, st.l, st.o, p.c2);
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(bal::THREADS) __attribute__((amdgpu_waves_per_eu(3)))
void cascade_balanced_kernel(Params p) {
  using BT = BalTile<T>;
  __shared__ BalShared<T> sh;
  const int tid = threadIdx.x;
  const int wave_s = uni(tid >> 6);
  const int batch = min(p.batch, bal::MAX_BATCH);

  if (wave_s == 0) bal_schedule<T>(p, sh, batch, tid & 63);
  for (int turn = 0;; turn ^= 1) {
    const int lane = fresh(tid & 63);
    __syncthreads();          // the piece is written; the one before is done with the ring and the page ids
    BalPiece pc;
    {
      const int4* s = reinterpret_cast<const int4*>(&sh.piece[turn]);
      const int4 v0 = s[0], v1 = s[1], v2 = s[2], v3 = s[3];
      pc = BalPiece{uni(v0.x), uni(v0.y), uni(v0.z), uni(v0.w), uni(v1.x), uni(v1.y), uni(v1.z), uni(v1.w),
                    uni(v2.x), uni(v2.y), uni(v2.z), uni(v2.w), uni(v3.x), uni(v3.y), uni(v3.z), 0};
    }
    if (!pc.count) break;
    const int kg = BT::MAX_KG == 2 && wave_s >= pc.tiles ? 1 : 0;
    const int ti = wave_s - kg * pc.tiles;
    const bool active = kg < pc.kg && ti < pc.tiles;
    const BalRows rw{pc.row0 + ti * kRowsPerTile, pc.Nb * p.G, pc.node_base, pc.h};

    BalWave<T> st;
    for (int c0 = pc.t0;; c0 += bal::CHUNK_TILES) {
      const int c1 = min(pc.t1, c0 + bal::CHUNK_TILES);
      const int npg = p.stage != D2SD_STAGE_TREE ? ceil_div(min(pc.C, c1 * bal::KT), D2SD_PAGE_SIZE) - 2 * c0 : 0;
      if (npg > 0) {
        const int* pt = p.page_table + (size_t)pc.b * p.max_pages + 2 * c0;
        const int ln = fresh(lane);
        for (int i = wave_s * kWave; i < npg; i += bal::THREADS)
          dma4(pt + min(i + ln, npg - 1), lds_addr(reinterpret_cast<const char*>(sh.pid)) + 4 * i);
      }
      // The query rows arrive in the last slots of the ring, beside the first
      // tiles' copies (fp32: before them, in two passes).
      char* const area = sh.ring + BT::SLOTS * BT::SLOT - (pc.tiles * pc.kg - wave_s) * BalTile<__bf16>::K_BYTES;
      if (c0 == pc.t0) {
        if (active) bal_queue_q<T>(p, rw, area, fresh(lane), 0);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) st.o[dt] = f32x16{};
        st.m = kNoReference;
        st.l = 0.0f;
        if (sizeof(T) == 4 && active) {
          wait_vmem();
          bal_read_q(area, fresh(lane), 0, st.q);
          __builtin_amdgcn_s_waitcnt(0xc07f);             // lgkmcnt(0): the area is free again
          bal_queue_q<T>(p, rw, area, fresh(lane), 1);
          wait_vmem();
          bal_read_q(area, fresh(lane), 1, st.q);
        }
      }
      // the page ids (the copies of the query rows stay in flight) and nothing of the compiler's
      if (sizeof(T) == 2 && c0 == pc.t0 && active) __builtin_amdgcn_s_waitcnt(0x0f78); else wait_vmem();
      __syncthreads();
      bal_run<T>(p, sh, pc, c0, c1, wave_s, fresh(lane), active, kg, rw, sizeof(T) == 2 && c0 == pc.t0 ? area : nullptr, st);
      if (c1 >= pc.t1) break;
      __syncthreads();
    }
    if (wave_s == bal::WAVES - 1) {
      if (!pc.last) bal_seek<T>(p, sh, batch, pc.b, pc.sidx + 1, sh.piece[turn ^ 1], lane);
      else if (lane == 0) sh.piece[turn ^ 1].count = 0;
      if (lane == 0 && pc.index == 0)
        p.ws_pieces[((size_t)pc.b * p.hkv + pc.h) * p.n_rg_max + pc.rgi] = (int)blockIdx.x << 16 | pc.count;
    }

    if constexpr (BT::MAX_KG == 2) {
      // ---- merge the second key group's state of a query tile into the first's ----
      if (pc.kg > 1) {
        float4* xo = reinterpret_cast<float4*>(sh.ring) + ti * (17 * 64) + lane;   // O, then (m, l)
        __syncthreads();
        if (active && kg == 1) {
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              xo[(dt * 4 + i) * 64] = make_float4(st.o[dt][4 * i], st.o[dt][4 * i + 1], st.o[dt][4 * i + 2], st.o[dt][4 * i + 3]);
          xo[16 * 64] = make_float4(st.m, st.l, 0.f, 0.f);
        }
        __syncthreads();
        if (active && kg == 0) {
          const float4 ml = xo[16 * 64];
          const float mn = fmaxf(st.m, ml.x);
          const float a = __builtin_amdgcn_exp2f(st.m - mn);
          const float a2 = __builtin_amdgcn_exp2f(ml.x - mn);
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float4 v = xo[(dt * 4 + i) * 64];
              st.o[dt][4 * i] = st.o[dt][4 * i] * a + v.x * a2;
              st.o[dt][4 * i + 1] = st.o[dt][4 * i + 1] * a + v.y * a2;
              st.o[dt][4 * i + 2] = st.o[dt][4 * i + 2] * a + v.z * a2;
              st.o[dt][4 * i + 3] = st.o[dt][4 * i + 3] * a + v.w * a2;
            }
          st.l = st.l * a + ml.y * a2;
          st.m = mn;
        }
      }
    }

    // ---- finalise (one piece) or write the piece's partial state ----
    __syncthreads();          // the ring now holds output rows
    if (active && kg == 0) {
      const float l_all = st.l + __shfl_xor(st.l, 32);
      const float inv = l_all > 0.0f ? 1.0f / l_all : 0.0f;
      char* const rows_area = sh.ring + wave_s * BalTile<__bf16>::K_BYTES;
      const bool direct = pc.count == 1;
      const int stream = (pc.b * p.hkv + pc.h) * p.n_rg_max + pc.rgi;
      const int slot = pc.index > 0 ? (int)blockIdx.x : start_slot(p, stream, blockIdx.x);
      const size_t part = (size_t)slot * p.slot_rows;       // the piece's first row in the workspace
      const int ln = fresh(lane);
      const int r = rw.row0 + ln;
      if (ln < kRowsPerTile && r < rw.rows) {
        if (!direct) {
          p.ws_m[part + r - pc.row0] = l_all > 0.0f ? st.m : -INFINITY;
          p.ws_l[part + r - pc.row0] = l_all;
        } else if (p.lse) {
          p.lse[rw.global_row(p, r)] = l_all > 0.0f ? (st.m + __log2f(l_all)) * kLn2 : -INFINITY;
        }
      }
      auto to_out = [&](int row) { return static_cast<char*>(p.out) + rw.global_row(p, row) * BT::ROW_BYTES; };
      auto to_slot = [&](int row) { return static_cast<char*>(p.ws_o) + (part + row - pc.row0) * (kD * sizeof(float)); };
      if constexpr (sizeof(T) == 4) {
        bal_store<T, T>(rw, rows_area, fresh(lane), st.o, inv, [&](int row) { return direct ? to_out(row) : to_slot(row); });
      } else if (direct) {
        bal_store<T, T>(rw, rows_area, fresh(lane), st.o, inv, to_out);
      } else {
        bal_store<T, float>(rw, rows_area, fresh(lane), st.o, inv, to_slot);
      }
    }
  }
}

}  // namespace

hipError_t launch_balanced_attention(const d2sd_attn_args& a, const AttnPlan& plan, void* ws, hipStream_t stream) {
  const Params p = make_params(a, plan, ws);
  if (a.dtype == D2SD_BF16)
    hipLaunchKernelGGL(cascade_balanced_kernel<__bf16>, dim3(plan.workgroups), dim3(bal::THREADS), 0, stream, p);
  else
    hipLaunchKernelGGL(cascade_balanced_kernel<float>, dim3(plan.workgroups), dim3(bal::THREADS), 0, stream, p);
  return hipGetLastError();
}

}  // namespace d2sd
