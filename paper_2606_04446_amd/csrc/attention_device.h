// Device helpers and kernel parameters shared by the attention kernels.
#pragma once

#include <math.h>

#include "common.h"

namespace d2sd {

namespace {

constexpr int kD = 128;
constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct Params {
  const void* q;
  const void* k_cache;
  const void* v_cache;
  const int* page_table;
  const int* ctx_len;
  const void* k_tree;
  const void* v_tree;
  const int* node_indptr;
  const uint32_t* anc_mask;
  void* out;
  float* lse;
  // Partial states: outputs normalised by their row sum, and m and l in fp32.
  // Fixed splits: [n_ch_max, total_rows], outputs in the input dtype. Balanced:
  // [slots, slot_rows], outputs in fp32.
  void* ws_o;
  float* ws_m;
  float* ws_l;
  int* ws_pieces;  // balanced: [batch, hkv, n_rg_max] (first workgroup << 16 | pieces) of a stream, else null
  int batch, hq, hkv, G, stage;
  int total_nodes, max_nodes, max_ctx, num_pages, max_pages, mask_words;
  int split, n_ch_max, n_rg_max, items;
  int slot_rows;
  float c2;  // sm_scale * log2(e)
  float inv_G, inv_hq;   // reciprocals
};

__device__ __forceinline__ f32x16 mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma(float a, float b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint4 zero4() { return make_uint4(0u, 0u, 0u, 0u); }

// s_waitcnt vmcnt(0): wait for every outstanding vector-memory access of the
// wave (gfx9 encoding: vmcnt 0, expcnt and lgkmcnt left at their maxima).
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0f70); }

template <typename T>
__device__ __forceinline__ void store_out(T* dst, const float* v4);
template <>
__device__ __forceinline__ void store_out<__bf16>(__bf16* dst, const float* v) {
  __bf16 h[4] = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
  *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(h);
}
template <>
__device__ __forceinline__ void store_out<float>(float* dst, const float* v) {
  *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 lds_b128(const char* base, int off) {
  return *reinterpret_cast<const uint4*>(base + off);
}
__device__ __forceinline__ s16x4 lds_tr16(const char* base, int off) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(base + off));
}
// LDS DMA copies are issued as inline asm so that the compiler does not
// track them: its own tracking cannot tell ring stages apart and would make
// every later LDS read wait for all copies in flight (vmcnt(0)). The kernel
// orders copies and reads itself (sync_keep); untracked loads can only
// lengthen the compiler's own vmcnt waits, never shorten them. The s_nop
// covers the M0-write to LDS-DMA hazard. Each lane's 16 bytes land at
// M0 + 16 * lane.
__device__ __forceinline__ uint32_t lds_addr(const char* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ void dma16(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(src), "s"(lds)
               : "memory", "m0");
}
__device__ __forceinline__ void dma16s(const char* base, uint32_t lane_off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_off), "s"(base), "s"(lds)
               : "memory", "m0");
}

// Four bytes per lane, at M0 + 4 * lane.
__device__ __forceinline__ void dma4(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :
               : "v"(src), "s"(lds)
               : "memory", "m0");
}

// s_waitcnt vmcnt(n) lgkmcnt(0) then s_barrier; the asm statement is also a
// compiler memory barrier. Waves keep up to n of their own LDS DMAs in flight.
template <int N>
__device__ __forceinline__ void sync_keep() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  // gfx9 s_waitcnt: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]
  __builtin_amdgcn_s_waitcnt((N & 15) | 0x0070 | ((N >> 4) << 14));
  asm volatile("s_barrier" ::: "memory");
}
__device__ __forceinline__ float xhalf_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Balanced: the slot of a stream's first piece, which workgroup `first` writes.
// The other pieces' slots are their workgroups, which hold one each; the first
// ones have slots by stream where there are no more streams than workgroups.
__device__ __forceinline__ int start_slot(const Params& p, int stream, int first) {
  return kBalWorkgroups + (p.batch * p.hkv * p.n_rg_max <= kBalWorkgroups ? stream : first);
}

inline Params make_params(const d2sd_attn_args& a, const AttnPlan& plan, void* ws) {
  Params p{};
  p.q = a.q; p.k_cache = a.k_cache; p.v_cache = a.v_cache; p.page_table = a.page_table;
  p.ctx_len = a.ctx_len; p.k_tree = a.k_tree; p.v_tree = a.v_tree; p.node_indptr = a.node_indptr;
  p.anc_mask = a.anc_mask; p.out = a.out; p.lse = a.lse;
  // [O][m][l], each split- or slot-major, then the piece counts
  char* w = static_cast<char*>(ws);
  const bool balanced = plan.workgroups > 0;
  const size_t states = balanced ? (size_t)plan.slots * plan.slot_rows
                                 : (size_t)plan.n_ch_max * a.total_nodes * a.num_qo_heads;
  const size_t o_bytes = states * kD * (a.dtype == D2SD_BF16 && !balanced ? 2 : 4);
  p.ws_o = w;
  p.ws_m = w ? reinterpret_cast<float*>(w + o_bytes) : nullptr;
  p.ws_l = w ? p.ws_m + states : nullptr;
  p.ws_pieces = w && balanced ? reinterpret_cast<int*>(p.ws_l + states) : nullptr;
  p.slot_rows = plan.slot_rows;
  p.batch = a.batch; p.hq = a.num_qo_heads; p.hkv = a.num_kv_heads; p.G = plan.G; p.stage = a.stage;
  p.total_nodes = a.total_nodes; p.max_nodes = a.max_nodes; p.max_ctx = a.max_ctx_len;
  p.num_pages = a.num_pages; p.max_pages = a.max_pages; p.mask_words = a.mask_words;
  p.split = plan.split; p.n_ch_max = plan.n_ch_max; p.n_rg_max = plan.n_rg_max;
  p.items = (int)plan.items;
  p.c2 = plan.scale * kLog2e;
  p.inv_G = 1.0f / (float)plan.G;
  p.inv_hq = 1.0f / (float)a.num_qo_heads;
  return p;
}

}  // namespace

}  // namespace d2sd
