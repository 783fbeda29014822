// Vector-ALU attention for gfx950, fp32 caches: the g query heads of one kv head
// for R consecutive tokens of a sequence per block, over one split [k0, k1) of
// the key positions (fp32 stays in the vector units: the rate of a few tokens
// over a cache is set by loads and latency).
//
// Lane layout: 16 lanes hold a key row (16-byte vectors), so a block's 16 slots
// cover 16 keys per load instruction, every load a coalesced 16-byte vector; a
// step takes U keys per slot, their loads issued together.  Scores are reduced
// across a key's 16 lanes with DPP (quad_perm, row_half_mirror, row_mirror).
// Each slot keeps its own running max / sum / output per query row (online
// softmax in base 2: the query is pre-scaled by log2(e) / sqrt(D)), rescaled
// once per step.  At the end the four slots of a wave merge by lane swaps, the
// four waves through LDS.  A block that covers the whole range writes the
// normalised output; otherwise it writes a partial (max, sum, unnormalised
// output) that the combine kernel merges.
//
// What bounds it: many tokens, the rows' loads through L2 (512 tokens over ~4K
// keys of 4 kv heads, g 8, D 128: 930 us a call, about 9 TB/s of rows); few, the chain of
// upload, append, attention and merge launches (64 tokens over ~2K keys: a pass
// of four such calls and 16 decode steps 287 -> 209 us).  Before, a block held one
// token, a lane had one key's loads in flight and 256 blocks were planned, and
// sixteen slots' outputs were added through LDS row by row behind two barriers
// each.
#include <type_traits>

#include "fcg_device.hpp"
#include "kernels.hpp"

namespace fcg {

// Sum over the 16 lanes of a DPP row; every lane gets the sum.
__device__ __forceinline__ float sum_lanes16(float x) {
  x += dpp_f32<kDppXor1>(x);
  x += dpp_f32<kDppXor2>(x);
  x += dpp_f32<kDppHalfMirror>(x);
  x += dpp_f32<kDppMirror>(x);
  return x;
}

template <int D, int G, int R>
__global__ void __launch_bounds__(256) attn_rows_kernel(const AttnItem* __restrict__ items,
                                                        const TokenMeta* __restrict__ meta,
                                                        const float* __restrict__ qws, int rows_ws, CacheView cv,
                                                        int layer, int Hq, float* __restrict__ out,
                                                        float* __restrict__ part_o, float* __restrict__ part_ml,
                                                        int part_stride_rows) {
  constexpr int NV = D / 64;      // 16-byte vectors per lane and row: dims 64 nv + 4 chunk .. + 3
  constexpr int DPL = 4 * NV;     // dims per lane
  constexpr int ROWS = G * R;     // query rows
  constexpr int U = ROWS * DPL <= 32 ? 4 : ROWS * DPL <= 64 ? 2 : 1;  // keys per slot and step (registers)
  constexpr int STEP = 16 * U;
  __shared__ __align__(16) float s_o[4][ROWS][D];
  __shared__ float s_m[4][ROWS], s_l[4][ROWS];

  const AttnItem it = items[blockIdx.x];
  const int hk = blockIdx.y;
  const int Hkv = cv.n_kv_heads;
  const int t = threadIdx.x, w = t >> 6;
  const int chunk = t & 15, slot = t >> 4;
  const float qscale = 1.4426950408889634f / sqrtf((float)D);

  // a block of fewer than R tokens repeats its last one (not written)
  int pos[R];
#pragma unroll
  for (int r = 0; r < R; ++r) pos[r] = meta[it.rank0 + min(r, it.n_rank - 1)].pos;
  float q[ROWS][DPL];
#pragma unroll
  for (int j = 0; j < ROWS; ++j)
#pragma unroll
    for (int nv = 0; nv < NV; ++nv) {
      const int64_t row = (int64_t)hk * rows_ws + (int64_t)(it.rank0 + min(j / G, it.n_rank - 1)) * G + j % G;
      const float4 x = *reinterpret_cast<const float4*>(qws + row * D + nv * 64 + chunk * 4);
      q[j][nv * 4 + 0] = x.x * qscale;
      q[j][nv * 4 + 1] = x.y * qscale;
      q[j][nv * 4 + 2] = x.z * qscale;
      q[j][nv * 4 + 3] = x.w * qscale;
    }
  float mx[ROWS], sum[ROWS], o[ROWS][DPL];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    mx[j] = -INFINITY;
    sum[j] = 0.f;
#pragma unroll
    for (int e = 0; e < DPL; ++e) o[j][e] = 0.f;
  }
  const float* ck = reinterpret_cast<const float*>(cv.k);
  const float* cvv = reinterpret_cast<const float*>(cv.v);
  const int end = min(it.k1, pos[R - 1] + 1);  // positions ascend
  // MASKED: the step may hold keys past the range or past a token's position
  auto step = [&](int base, auto masked) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked)::value;
    float kx[U][DPL], vx[U][DPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int key = MASKED ? min(base + u * 16 + slot, end - 1) : base + u * 16 + slot;
      const int64_t off = cache_offset(cv, layer, it.seq, hk, key);
      const float* vr = cv.page_size ? v_row<true, float>(cv, layer, it.seq, hk, key) : cvv + off;
#pragma unroll
      for (int nv = 0; nv < NV; ++nv) {
        Store<float>::unpack(ld16(ck + off + nv * 64 + chunk * 4), kx[u] + nv * 4);
        Store<float>::unpack(ld16(vr + nv * 64 + chunk * 4), vx[u] + nv * 4);
      }
    }
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      float s[U], mn = mx[j];
      bool seen[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < DPL; ++e) a = fmaf(q[j][e], kx[u][e], a);
        s[u] = sum_lanes16(a);
        seen[u] = !MASKED || base + u * 16 + slot < min(end, pos[j / G] + 1);
        if (!seen[u]) s[u] = -INFINITY;
        mn = fmaxf(mn, s[u]);
      }
      const float ref = MASKED && mn == -INFINITY ? 0.f : mn;  // nothing seen yet: every weight 0
      const float a = __builtin_amdgcn_exp2f(mx[j] - ref);      // v_exp_f32: -inf gives 0
      mx[j] = mn;
      sum[j] *= a;
#pragma unroll
      for (int e = 0; e < DPL; ++e) o[j][e] *= a;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float p = __builtin_amdgcn_exp2f(s[u] - ref);
        sum[j] += p;
#pragma unroll
        for (int e = 0; e < DPL; ++e) o[j][e] = fmaf(p, seen[u] ? vx[u][e] : 0.f, o[j][e]);
      }
    }
  };
  int base = it.k0;
  const int whole = min(end, pos[0] + 1);
  for (; base + STEP <= whole; base += STEP) step(base, std::false_type{});
  for (; base < end; base += STEP) step(base, std::true_type{});

  // merge the four slots of each wave, then the waves
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const float M = max_rows4(mx[j]);
    const float f = mx[j] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx[j] - M);
    const float L = sum_rows4(sum[j] * f);
#pragma unroll
    for (int e = 0; e < DPL; ++e) o[j][e] = sum_rows4(o[j][e] * f);
    if ((t & 63) < 16) {
#pragma unroll
      for (int nv = 0; nv < NV; ++nv)
        *reinterpret_cast<float4*>(&s_o[w][j][nv * 64 + chunk * 4]) =
            make_float4(o[j][nv * 4], o[j][nv * 4 + 1], o[j][nv * 4 + 2], o[j][nv * 4 + 3]);
      if (chunk == 0) {
        s_m[w][j] = M;
        s_l[w][j] = L;
      }
    }
  }
  __syncthreads();
  for (int idx = t; idx < min(ROWS, it.n_rank * G) * (D / 4); idx += 256) {
    const int j = idx / (D / 4), d = 4 * (idx % (D / 4));
    float M = -INFINITY;
#pragma unroll
    for (int w2 = 0; w2 < 4; ++w2) M = fmaxf(M, s_m[w2][j]);
    float L = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w2 = 0; w2 < 4; ++w2) {
      const float m = s_m[w2][j];
      const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
      const float4 x = *reinterpret_cast<const float4*>(&s_o[w2][j][d]);
      L = fmaf(s_l[w2][j], f, L);
      acc.x = fmaf(x.x, f, acc.x);
      acc.y = fmaf(x.y, f, acc.y);
      acc.z = fmaf(x.z, f, acc.z);
      acc.w = fmaf(x.w, f, acc.w);
    }
    if (it.part < 0) {
      const int tok = meta[it.rank0 + j / G].tok;
      const bool any = L > 0.f;
      *reinterpret_cast<float4*>(out + ((int64_t)tok * Hq + hk * G + j % G) * D + d) =
          make_float4(any ? acc.x / L : 0.f, any ? acc.y / L : 0.f, any ? acc.z / L : 0.f, any ? acc.w / L : 0.f);
    } else {
      const int64_t row = ((int64_t)it.part * Hkv + hk) * part_stride_rows + j;
      *reinterpret_cast<float4*>(part_o + row * D + d) = acc;
      if (d == 0) {
        part_ml[row * 2 + 0] = M;
        part_ml[row * 2 + 1] = L;
      }
    }
  }
}

// Merge split-KV partials: per row, M = max M_s, L = sum L_s 2^(M_s - M),
// O = sum O_s 2^(M_s - M) / L.  Block (row block, kv head, z) merges up to
// kCombRows rows, its item taken from the by-value plan.  Every load that
// does not depend on another is issued first: the (M_s, L_s) pairs into LDS,
// the rows' output tokens and, for the bf16 MFMA partials, the first
// PRE splits' partial outputs of the lane's 4-dim chunk; 32 lanes per
// row then form the scales 2^(M_s - M) / L with shuffles, and each 4-dim
// output chunk is summed over the splits (fp32 partials: LPC lanes per chunk
// taking interleaved splits, their sums added one by one through LDS).
constexpr int kCombRows = 8;
constexpr int kCombMaxParts = 256;
// PRE: the smallest of 4, 16 and 32 that covers every row block of the
// launch (each preload past the last split re-reads it: 7B patch call -0.4 us
// with 16 against 32).
template <typename T, int D, bool MFMA_PART, int PRE>
__global__ void __launch_bounds__(256) combine_kernel(CombineArgs args, const TokenMeta* __restrict__ meta, int Hq,
                                                      int Hkv, const float* __restrict__ part_o,
                                                      const float* __restrict__ part_ml, int part_stride_rows,
                                                      T* __restrict__ out) {
  __shared__ float s_f[kCombRows][kCombMaxParts + 1];  // +1: rows start in different banks
  __shared__ float s_l[kCombRows][kCombMaxParts + 1];
  __shared__ float4 s_acc[256];
  const CombineItem it = args.item[blockIdx.x];
  const int hk = blockIdx.y;
  // every argument in one batch of scalar loads, before any arithmetic on
  // them (else the compiler issues part of the batch after the division)
  asm volatile("" ::"s"(it.rank0), "s"(it.n_rank), "s"(it.n_part), "s"(it.part0), "s"(it.tok0), "s"(meta), "s"(part_o),
               "s"(part_ml), "s"(out), "s"(Hq), "s"(Hkv), "s"(part_stride_rows));
  __builtin_amdgcn_sched_barrier(0);
  const int g = Hq / Hkv;
  const int t = threadIdx.x;
  const int r0 = blockIdx.z * kCombRows;
  const int nr = min(kCombRows, it.n_rank * g - r0);
  const int np = it.n_part;
  if (nr <= 0) return;
  auto prow = [&](int s, int r) { return ((int64_t)(it.part0 + s) * Hkv + hk) * part_stride_rows + r0 + r; };
  constexpr int CPR = D / 4;                  // 4-dim chunks per row
  const int nch = nr * CPR;
  const int lpc = max(1, 256 / nch);          // lanes per chunk, consecutive (any number: 5 for three rows of 16 chunks)
  // chunk c -> (row, 4-dim chunk): neighbouring lanes read neighbouring bytes
  // (rows fastest in the MFMA fragment order, dims fastest in row-major order)
  auto chunk = [&](int c, int* r, int* c4) {
    *r = MFMA_PART ? c % nr : c / CPR;
    *c4 = MFMA_PART ? c / nr : c % CPR;
  };
  // bf16 partial output of split s, row r, chunk c4, in the MFMA accumulator
  // order of the prefill kernel: per 16-row tile and 16-dim tile, 64 lanes x
  // 4 dims, lane = row % 16 + 16 * (4-dim chunk % 4)
  auto mfma_part = [&](int s, int r, int c4) -> uint2 {
    const int rr = r0 + r;
    const int64_t off = ((int64_t)(it.part0 + s) * Hkv + hk) * part_stride_rows * D +
                        (((rr / 16) * (D / 16) + c4 / 4) * 64 + rr % 16 + 16 * (c4 % 4)) * 4;
    return *reinterpret_cast<const uint2*>(reinterpret_cast<const bf16_t*>(part_o) + off);
  };
  int my_r = 0, my_c4 = 0;
  const bool my_chunk = t / lpc < nch;
  chunk(my_chunk ? t / lpc : 0, &my_r, &my_c4);
  uint2 pre[MFMA_PART ? PRE : 1];
  if (MFMA_PART) {
    // lpc is 1 here (nch = 8 rows x D/4 chunks = 256 lanes for a full block)
#pragma unroll
    for (int u = 0; u < PRE; ++u) pre[u] = mfma_part(min(u, np - 1), my_r, my_c4);
  }
  const int out_tok = it.tok0 >= 0 ? it.tok0 + (r0 + my_r) / g : meta[it.rank0 + (r0 + my_r) / g].tok;
  for (int idx = t; idx < nr * np; idx += 256) {
    const int r = idx / np, s = idx % np;
    s_f[r][s] = part_ml[prow(s, r) * 2];
    s_l[r][s] = part_ml[prow(s, r) * 2 + 1];
  }
  __syncthreads();
  {
    // 32 lanes per row: M, L and the scales 2^(M_s - M) / L
    const int r = t / 32, l32 = t % 32;
    if (r < nr) {
      float M = -INFINITY;
      for (int s = l32; s < np; s += 32) M = fmaxf(M, s_f[r][s]);
      M = max_lanes32(M);
      float L = 0.f;
      for (int s = l32; s < np; s += 32) {
        const float ms = s_f[r][s];
        L = fmaf(s_l[r][s], ms == -INFINITY ? 0.f : exp2f(ms - M), L);
      }
      L = sum_lanes32(L);
      const float inv = L > 0.f ? 1.f / L : 0.f;
      for (int s = l32; s < np; s += 32) {
        const float ms = s_f[r][s];
        s_f[r][s] = ms == -INFINITY ? 0.f : exp2f(ms - M) * inv;
      }
    }
  }
  __syncthreads();
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](float4 o, float f) {
    acc.x = fmaf(o.x, f, acc.x);
    acc.y = fmaf(o.y, f, acc.y);
    acc.z = fmaf(o.z, f, acc.z);
    acc.w = fmaf(o.w, f, acc.w);
  };
  auto bf4 = [](uint2 u) { return make_float4(lo_bf16(u.x), hi_bf16(u.x), lo_bf16(u.y), hi_bf16(u.y)); };
  if (MFMA_PART) {
    if (!my_chunk) return;
#pragma unroll
    for (int u = 0; u < PRE; ++u)
      if (u < np) add(bf4(pre[u]), s_f[my_r][u]);
#pragma unroll 8
    for (int s = PRE; s < np; ++s) add(bf4(mfma_part(s, my_r, my_c4)), s_f[my_r][s]);
  } else {
    if (my_chunk) {
#pragma unroll 8
      for (int s = t % lpc; s < np; s += lpc)
        add(*reinterpret_cast<const float4*>(part_o + prow(s, my_r) * D + my_c4 * 4), s_f[my_r][s]);
    }
    if (lpc > 1) {
      s_acc[t] = acc;
      __syncthreads();
      if (t % lpc || !my_chunk) return;
      for (int sub = 1; sub < lpc; ++sub) {
        const float4 a4 = s_acc[t + sub];
        acc.x += a4.x;
        acc.y += a4.y;
        acc.z += a4.z;
        acc.w += a4.w;
      }
    } else if (!my_chunk) {
      return;
    }
  }
  T* dst = out + ((int64_t)out_tok * Hq + hk * g + (r0 + my_r) % g) * D + my_c4 * 4;
  Store<T>::store1(dst + 0, acc.x);
  Store<T>::store1(dst + 1, acc.y);
  Store<T>::store1(dst + 2, acc.z);
  Store<T>::store1(dst + 3, acc.w);
}

int launch_attn_rows(const AttnItem* items, int n_items, const TokenMeta* meta, const void* qws, int rows_ws,
                     const CacheView& cv, int layer, int Hq, void* out, float* part_o, float* part_ml,
                     int part_stride_rows, int tokens, hipStream_t s, KTime tm) {
  if (n_items == 0) return 0;
  const int g = Hq / cv.n_kv_heads;
  dim3 grid(n_items, cv.n_kv_heads);
#define AR(DD, GG, RR)                                                                                       \
  hipExtLaunchKernelGGL((attn_rows_kernel<DD, GG, RR>), grid, dim3(256), 0, s, tm.start, tm.stop, 0, items, meta, \
                        (const float*)qws, rows_ws, cv, layer, Hq, (float*)out, part_o, part_ml, part_stride_rows)
#define AR1(DD, GG) if (tokens == 1) AR(DD, GG, 1); else return -1
#define AR2(DD, GG) if (tokens == 2) AR(DD, GG, 2); else AR1(DD, GG)
#define AR4(DD, GG) if (tokens == 4) AR(DD, GG, 4); else AR2(DD, GG)
  if (cv.head_dim == 64) {  // the instances attn_rows_tokens allows
    switch (g) {
      case 1: AR4(64, 1); break;
      case 2: AR4(64, 2); break;
      case 4: AR2(64, 4); break;
      case 8: AR1(64, 8); break;
      case 16: AR1(64, 16); break;
      default: return -1;
    }
  } else {
    switch (g) {
      case 1: AR4(128, 1); break;
      case 2: AR2(128, 2); break;
      case 4: AR1(128, 4); break;
      case 8: AR1(128, 8); break;
      case 16: AR1(128, 16); break;
      default: return -1;
    }
  }
#undef AR4
#undef AR2
#undef AR1
#undef AR
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : (int)e;
}

int launch_combine(const CombineArgs& args, const TokenMeta* meta, int Hq, int Hkv, int D,
                   const float* part_o, const float* part_ml, int part_stride_rows, void* out, hipStream_t s,
                   bool mfma_part, KTime tm) {
  if (args.n_items == 0) return 0;
  dim3 grid(args.n_items, Hkv, (part_stride_rows + kCombRows - 1) / kCombRows);
  int max_np = 0;
  for (int i = 0; i < args.n_items; ++i) max_np = max(max_np, (int)args.item[i].n_part);
  const int pre = max_np <= 4 ? 4 : max_np <= 16 ? 16 : 32;
#define CBK(T, DD, MP, PR)                                                                                  \
  hipExtLaunchKernelGGL((combine_kernel<T, DD, MP, PR>), grid, dim3(256), 0, s, tm.start, tm.stop, 0, args,   \
                        meta, Hq, Hkv, part_o, part_ml, part_stride_rows, (T*)out)
#define CB(DD)                                                                                               \
  do {                                                                                                       \
    if (!mfma_part) CBK(float, DD, false, 16);                                                               \
    else if (pre == 4) CBK(bf16_t, DD, true, 4);                                                             \
    else if (pre == 16) CBK(bf16_t, DD, true, 16);                                                           \
    else CBK(bf16_t, DD, true, 32);                                                                          \
  } while (0)
  if (D == 64) CB(64); else CB(128);
#undef CB
#undef CBK
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : (int)e;
}

}  // namespace fcg
