// Shared tail of the decode kernels (Sec. 4.2, Eq. 6: decode over the
// grafted KV states).  A block has attended one split of one (sequence, kv
// head) and holds, per query head j of the group, its max M_j, sum L_j and
// unnormalised output O_j (base-2 exponent scale).
//   - emit_pair writes two adjacent output dims: normalised into out when the
//     sequence has a single split, else into the split's partial slot with
//     device-coherent stores (bf16 rows for bf16 storage, fp32 otherwise).
//   - merge_splits makes the block count itself in the (sequence, kv head)
//     counter once its partial stores have completed; the block that arrives
//     last folds every split's partial (device-coherent buffer loads) and
//     writes the output, then sets the counter back to zero.  Every access
//     that crosses blocks is device-coherent, so no L2 write-back or
//     invalidation is needed.
#pragma once

#include "fcg_device.hpp"
#include "kernels.hpp"

namespace fcg {

// Element offset of the new token's row (layer, seq, head, pos).  A page the
// step maps comes by value (DecodeArgs::new_page): the device page table gets
// its entry from this launch (enter_page), so no block reads it there.
template <bool PAGED>
__device__ __forceinline__ int64_t new_token_offset(const CacheView& c, int layer, int seq, int head, int pos,
                                                    int new_page) {
  if (PAGED && new_page >= 0)
    return (int64_t)layer * c.layer_stride +
           (((int64_t)new_page * c.n_kv_heads + head) * 16 + (pos & 15)) * c.head_dim;
  return kv_offset<PAGED>(c, layer, seq, head, pos);
}

// The device page-table entries of a page a decode step maps: its physical
// page, and "values not read from the library" (written by one lane of the
// owning split's first kv-head block; later launches read them).
__device__ __forceinline__ void enter_page(const CacheView& c, int seq, int pos, int new_page) {
  int32_t* row = const_cast<int32_t*>(c.page_table) + (int64_t)seq * 2 * c.n_lp;
  row[pos >> 4] = new_page;
  row[c.n_lp + (pos >> 4)] = -1;
}

// partial slot row of (split slot, kv head, query head): [slot][Hkv][G]
__device__ __forceinline__ int64_t part_row(int slot, int Hkv, int hk, int G, int j) {
  return ((int64_t)slot * Hkv + hk) * G + j;
}

template <typename T, int D>
__device__ __forceinline__ void emit_pair(int nsplit, int64_t prow, T* out_row, float* part_o, float* part_ml,
                                          int d, float a0, float a1, float M, float L) {
  if (nsplit == 1) {
    Store<T>::store1(out_row + d, L > 0.f ? a0 / L : 0.f);
    Store<T>::store1(out_row + d + 1, L > 0.f ? a1 / L : 0.f);
    return;
  }
  if constexpr (sizeof(T) == 2) {
    st_dev_u32(reinterpret_cast<uint32_t*>(part_o) + (prow * D + d) / 2, pack_bf16x2(a0, a1));
  } else {
    st_dev(&part_o[prow * D + d], a0);
    st_dev(&part_o[prow * D + d + 1], a1);
  }
  if (d == 0) {
    st_dev(&part_ml[prow * 2 + 0], M);
    st_dev(&part_ml[prow * 2 + 1], L);
  }
}

// Lanes that share one 16-byte chunk of a split set's outputs in merge_splits.
template <typename T, int D, int G>
constexpr int merge_lanes() {
  constexpr int chunks = G * D / (16 / (int)sizeof(T));
  return chunks < 256 ? 256 / chunks : 1;
}

// Called by all 256 lanes after their emit_pair calls, when nsplit > 1.
// LDS: s_buf 256 * 16 / sizeof(T) floats (256 output chunks), s_mt / s_lt
// [merge_lanes][G] floats, s_flag.
// Always inlined: called out of line (a choice the compiler made once more
// kernel instances called it) it made every decode launch ~2 us longer.
template <typename T, int D, int G>
__device__ __forceinline__ void merge_splits(const DecodeArgs& args, int i, int hk, int slot0, int nsplit, int Hkv,
                                             int Hq, T* __restrict__ out, const float* part_o,
                                             const float* part_ml, int* count, float* s_buf, float* s_mt,
                                             float* s_lt, int* s_flag) {
  const int t = threadIdx.x;
  // Ordering of the cross-block merge, stated in the hardware's terms (the
  // atomics are relaxed: release/acquire at agent scope writes back and
  // invalidates the L2 around the add; an earlier merge built on such fences,
  // with a serial merge loop, took 50 us per launch):
  //  1. every partial store is a device-scope (sc1) store, written through to
  //     the device coherence point; s_waitcnt vmcnt(0) returns only once this
  //     wave's stores are acknowledged there, and the barrier makes that hold
  //     for all four waves before the block's counter add is issued;
  //  2. the counter adds are atomic read-modify-writes at that same point, so
  //     the block that reads nsplit - 1 is ordered after every other block's
  //     add, hence after all their acknowledged stores;
  //  3. that block's partial loads are device-scope (sc1) buffer loads served
  //     by the coherence point, issued only after its add returned: they sit
  //     behind a branch on the returned count and two barriers (workgroup
  //     fences), which the compiler does not move memory accesses across.
  // The many-split and split-edge GPU tests exercise exactly this path.
  wait_vm0();        // this wave's partial stores have completed
  __syncthreads();   // ... and every wave's
  if (t == 0) {
    int* c = count + (i * Hkv + hk) * kCountStride;
    const int before = __hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_flag = before == nsplit - 1;
    if (before == nsplit - 1) __hip_atomic_store(c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!*s_flag) return;

  // O = sum_s O_s 2^(M_s - M) / sum_s L_s 2^(M_s - M), M = max_s M_s, per
  // query head.  A split's G rows are one contiguous run of 16-byte chunks: lane
  // (split lane sl, chunk) folds its chunk of the splits sl, sl + NSL, ... into a
  // running (max, sum, output), PF splits' loads in flight at a time, and the NSL
  // lanes of a chunk then meet in LDS.  With G = 4, D = 128 a wave reads one
  // split's 1 KB per load and 32 splits arrive in one round trip; an earlier fold
  // (every lane all G heads of a chunk of 16 split lanes, 24 loads and four
  // unrolled folds, 32 KB through LDS) took 3.0 us of a 7B step's 10.7, mostly
  // its code: only this block runs it, so every instruction is fetched for it.
  constexpr int EPL = 16 / (int)sizeof(T);  // elements per 16-byte chunk
  constexpr int NDC = D / EPL, CH = G * NDC, NSL = merge_lanes<T, D, G>();
  constexpr int PF = 8;
  constexpr uint32_t kFar = 0x80000000u;    // past every partial buffer (< 2^31 bytes): reads zeros, no access
  const int64_t hg = (int64_t)Hkv * G;      // rows per partial slot
  const int64_t row0 = (int64_t)slot0 * hg + (int64_t)hk * G;
  const uint32_t rows_all = (uint32_t)(args.slots * hg);
  const __amdgpu_buffer_rsrc_t ro = buf_rsrc(part_o, rows_all * D * (uint32_t)sizeof(T));
  const __amdgpu_buffer_rsrc_t rml = buf_rsrc(part_ml, rows_all * 8u);
  T* orow = out + ((int64_t)i * Hq + hk * G) * D;
  const int sl = t / (CH < 256 ? CH : 256);
  for (int c = t % (CH < 256 ? CH : 256); c < CH; c += 256) {  // once unless G * D > 256 chunks
    const int j = c / NDC;
    float acc[EPL], m = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
#pragma unroll 1
    for (int sb = sl; sb < nsplit; sb += NSL * PF) {
      u32x4_t x[PF];
      u32x2_t ml[PF];
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        const int sp = sb + p * NSL;
        const uint32_t r = (uint32_t)(row0 + (int64_t)sp * hg);
        ml[p] = ld8_dev(rml, sp < nsplit ? (r + j) * 8u : kFar);
        x[p] = ld16_dev(ro, sp < nsplit ? r * (uint32_t)(D * sizeof(T)) + c * 16u : kFar);
      }
      float mn = m;
#pragma unroll
      for (int p = 0; p < PF; ++p)
        mn = fmaxf(mn, sb + p * NSL < nsplit ? __uint_as_float(ml[p].x) : -INFINITY);
      const float mr = mn == -INFINITY ? 0.f : mn;         // a split always has a visible key; kept for safety
      const float f = __builtin_amdgcn_exp2f(m - mr);      // 0 while nothing was folded
      lsum *= f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] *= f;
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        // past the last split: sum and outputs read as zeros, whatever the weight
        const float wgt = sb + p * NSL < nsplit ? __builtin_amdgcn_exp2f(__uint_as_float(ml[p].x) - mr) : 0.f;
        float y[EPL];
        Store<T>::unpack(make_uint4(x[p].x, x[p].y, x[p].z, x[p].w), y);
        lsum = fmaf(__uint_as_float(ml[p].y), wgt, lsum);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = fmaf(y[e], wgt, acc[e]);
      }
      m = mn;
    }
    if (NSL == 1) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = lsum > 0.f ? acc[e] / lsum : 0.f;
      st16(orow + c * EPL, Store<T>::pack(acc));
      continue;
    }
#pragma unroll
    for (int e = 0; e < EPL; e += 4)
      *reinterpret_cast<float4*>(&s_buf[(sl * CH + c) * EPL + e]) =
          make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
    if (c % NDC == 0) {
      s_mt[sl * G + j] = m;
      s_lt[sl * G + j] = lsum;
    }
  }
  if (NSL == 1) return;
  __syncthreads();
  for (int idx = t; idx < G * D / 2; idx += 256) {
    const int d = 2 * idx, j = d / D;
    float M = -INFINITY;
#pragma unroll
    for (int s2 = 0; s2 < NSL; ++s2) M = fmaxf(M, s_mt[s2 * G + j]);
    float L = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int s2 = 0; s2 < NSL; ++s2) {
      const float ms = s_mt[s2 * G + j];  // -inf: a split lane without a split
      const float wgt = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - M);
      const float2 x = *reinterpret_cast<const float2*>(&s_buf[s2 * G * D + d]);
      L = fmaf(s_lt[s2 * G + j], wgt, L);
      o0 = fmaf(x.x, wgt, o0);
      o1 = fmaf(x.y, wgt, o1);
    }
    Store<T>::store1(orow + d, L > 0.f ? o0 / L : 0.f);
    Store<T>::store1(orow + d + 1, L > 0.f ? o1 / L : 0.f);
  }
}

}  // namespace fcg
