// One decode step at one layer on gfx950 matrix cores, bf16 caches (Sec.
// 4.2, Eq. 6: decoding over the reused, grafted KV states).
//
// Per sequence i the new token sits at position pos_i = its current length.
// Block (split s, sequence i, kv head h) attends the token's g query heads
// (g <= 16) over key positions [s * split_keys, min(pos_i + 1, (s + 1) *
// split_keys)).  Its four waves take the split's 16-key tiles in turn (w, w +
// 4, ...); wave w brings its tiles from memory into an LDS ring of its own
// (global_load_lds, whole rows, 1 KB per instruction), so the loop has no
// barrier and the tiles in flight cost no registers.  Per tile:
//   - S^T = K Q^T with v_mfma_f32_16x16x32_bf16: A = the tile's keys (lane l:
//     key l % 16, dims 32 ks + 8 (l / 16) .. + 7), B = the encoded queries,
//     column j = query head j (columns past g are zero).  Lane l then holds the
//     scores of query l % 16 for keys 4 (l / 16) .. + 3.
//   - online softmax in base 2 with one running max per query shared by its
//     four lanes, moved only when a score exceeds it by 2^8 (ballot), so the
//     lanes exchange maxima (two lane swaps) only then;
//   - O^T += V^T P^T with v_mfma_f32_16x16x16_bf16: B = the lane's four
//     probabilities rounded to bf16 (exactly the B layout), A = V^T by the LDS
//     transpose read (ds_read_b64_tr_b16).
// The owner of pos_i encodes the new key and, after its tiles, stores key and
// value into the cache slot and attends to them as a one-key tile.  The four
// waves merge through LDS; the split's result goes to the output or, for a
// sequence with several splits, to its partial slot, and the last block of
// the sequence to finish merges the splits (decode_common.hpp).
//
// What bounds it: many keys, HBM (32 paged tasks of ~6K tokens, 796 MB a call:
// 148.6 -> 125 us, 6.4 TB/s; four tasks of ~22K with g = 8, 369 MB: 68-72 -> 62
// us); one task of ~4K (17.5 MB), the chain of round trips: 10.9 -> 9.1 us, of
// which an empty launch takes 1.8, arguments, encoding and partial store 2.9,
// the tiles 2.2, the arrival count 0.7 and the merge 1.5.  Before, keys went
// straight into registers in the matrix operand layout, 64 bytes of each of 16
// rows per load, and values through a transpose in registers; a paged block
// read its page entries into LDS behind a barrier (six tasks of ~1.8K: 22.9 us
// against 15).
#include "decode_common.hpp"

namespace fcg {
namespace {

typedef __bf16 dm_bf16x8 __attribute__((ext_vector_type(8)));
typedef short dm_i16x4 __attribute__((ext_vector_type(4)));
typedef float dm_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 dm_bf16x2 __attribute__((ext_vector_type(2)));
typedef float dm_f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ dm_f32x4 mma_qk(const uint4& a, const uint4& b, const dm_f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dm_bf16x8, a), __builtin_bit_cast(dm_bf16x8, b),
                                                 c, 0, 0, 0);
}
__device__ __forceinline__ dm_f32x4 mma_pv(const uint2& a, const uint2& b, const dm_f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(dm_i16x4, a), __builtin_bit_cast(dm_i16x4, b),
                                                   c, 0, 0, 0);
}
// two fp32 -> packed bf16, round to nearest even
__device__ __forceinline__ uint32_t dm_cvt_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((dm_f32x2){lo, hi}, dm_bf16x2));
}

}  // namespace

// NB: 16-key tiles in each wave's LDS ring.
template <int D, int G, bool PAGED, int NB>
__global__ void __launch_bounds__(256) decode_mfma_kernel(DecodeArgs args, const bf16_t* __restrict__ q,
                                                          const bf16_t* __restrict__ k,
                                                          const bf16_t* __restrict__ v, CacheView cv,
                                                          const float2* __restrict__ rope,
                                                          bf16_t* __restrict__ out, float* __restrict__ part_o,
                                                          float* __restrict__ part_ml, int* __restrict__ count,
                                                          int layer) {
  static_assert(G >= 1 && G <= 16, "query group");
  constexpr int KS = D / 32;       // 32-deep k steps of S^T
  constexpr int DT = D / 16;       // 16-dim tiles of O^T
  constexpr int HALF = D / 2;
  constexpr int NC = D / 8;        // 16-byte chunks per row
  constexpr int RI = 64 / NC;      // rows one DMA instruction fills
  constexpr int KI = 16 / RI;      // DMA instructions for a tile's keys (and as many for its values)
  constexpr int DPT = 2 * KI;
  constexpr bool NT = NB == 2;     // launches that read much: see the launcher
  constexpr int TILE = 2 * 16 * D * 2;         // bytes of a tile: 16 keys, then 16 values
  constexpr int NCS = HALF / 2;                // 16-byte chunks of a position's (cos, sin) row
  constexpr int QI = (G * NC + 63) / 64;       // DMA instructions for the query rows
  constexpr int NSL = merge_lanes<bf16_t, D, G>();
  static_assert(2 * NC + NCS <= 64 && (1 + QI) * 1024 <= TILE, "the prologue's rows fit one ring buffer");
  static_assert(G * D * 4 <= NB * TILE && 256 * 8 * 4 <= 4 * NB * TILE, "the merges fit the ring");
  __shared__ __align__(16) char s_ring[4 * NB * TILE];
  __shared__ float s_wm[4][16], s_wl[4][16];
  __shared__ float s_mt[NSL * G], s_lt[NSL * G];
  __shared__ __align__(16) bf16_t s_newk[D], s_newv[D];  // the new token's encoded key and value
  __shared__ int s_last;

  const int split = blockIdx.x, i = blockIdx.y, hk = blockIdx.z;
  const int seq = args.seq[i], pos = args.pos[i], slot0 = args.split0[i];
  const int npage = PAGED ? args.new_page[i] : -1;  // a page this step maps, by value
  const int nsplit = args.split0[i + 1] - slot0;
  const int sk = args.split_keys;
  const bf16_t* ck = reinterpret_cast<const bf16_t*>(cv.k);
  const bf16_t* cvv = reinterpret_cast<const bf16_t*>(cv.v);
  // every kernel argument in one batch of scalar loads before the first branch.
  // The batch must not load a dword nothing reads: the compiler may reuse its
  // register for a later load of the batch, which then waits for the first
  // loads to land (a second round trip).  So `layer` comes last (no padding
  // after it) and the unused head_dim, which a merged load covers, is listed.
  asm volatile("" ::"s"(seq), "s"(pos), "s"(slot0), "s"(nsplit), "s"(sk), "s"(q), "s"(k), "s"(v), "s"(ck),
               "s"(cvv), "s"(cv.layer_stride), "s"(cv.max_tokens), "s"(cv.n_kv_heads), "s"(layer), "s"(rope),
               "s"(out), "s"(part_o), "s"(part_ml), "s"(count), "s"(cv.head_dim));
  if (PAGED)
    asm volatile("" ::"s"(cv.page_table), "s"(cv.n_lp), "s"(cv.v_alias), "s"(cv.lib_v), "s"(cv.lib_cap), "s"(npage),
                 "s"(cv.page_size));  // else the load of n_lp .. head_dim covers a dword that nothing reads
  if (split >= nsplit) return;  // padding split of a shorter sequence

  const int Hkv = cv.n_kv_heads;
  const int Hq = Hkv * G;
  const int t = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);  // the wave, in a scalar register
  const int l = t & 63, lr = l & 15, lq = l >> 4;
  const int k0 = split * sk;             // a multiple of 64
  const int k1 = min(pos + 1, k0 + sk);
  const bool owns_new = k1 == pos + 1;   // the last split holds the new token
  const int kend = owns_new ? pos : k1;  // cached keys [k0, kend)
  const int ntile = (kend - k0 + 15) >> 4;
  // the wave's n tiles are w, w + 4, ...; they pass through its own LDS ring,
  // so no barrier until the waves merge
  const int n = (ntile - w + 3) >> 2;
  const bool new_wave = owns_new && w == (ntile & 3);  // encodes, stores and attends the new token
  char* ring = s_ring + w * (NB * TILE);
  const uint32_t ring_lds = lds_addr(ring);

  // A tile of a paged cache is one page: its entries are wave-uniform, read
  // through the scalar cache (this launch writes only the entry of the page it
  // maps, which holds no cached key).
  typedef const __attribute__((address_space(4))) int32_t* cptr;
  const cptr prow = PAGED ? (cptr)(uintptr_t)(cv.page_table + (int64_t)seq * 2 * cv.n_lp + (k0 >> 4)) : (cptr)0;
  struct Entry {
    int32_t page, alias;
  };
  auto entry = [&](int ti) __attribute__((always_inline)) -> Entry {  // of the wave's tile ti (clamped into the split)
    Entry e{0, -1};
    if (PAGED) {
      const int x = max(0, min(w + 4 * ti, ntile - 1));
      e.page = prow[x];
      if (cv.v_alias) e.alias = prow[cv.n_lp + x];
    }
    return e;
  };
  const int64_t head0 = PAGED ? 0 : kv_offset<false>(cv, layer, seq, hk, k0);
  // Tile ti of the wave into its ring buffer.  DMA instruction j fills slots
  // 64 j .. 64 j + 63 of the key (value) rows, lane l the slot of row (64 j + l)
  // / NC at chunk position (64 j + l) % NC.  The chunks of a row are
  // XOR-swizzled so that the fragment reads below meet no bank conflicts (keys:
  // row % NC; values: 2 (row % (NC / 2))), so the lane loads the chunk that
  // belongs there: every instruction reads RI whole rows, 1 KB in one piece.
  auto issue = [&](int ti, const Entry& e) __attribute__((always_inline)) {
    const int tile = w + 4 * ti;
    const bf16_t *kb, *vb;
    if (PAGED) {
      const int64_t off = (int64_t)layer * cv.layer_stride + ((int64_t)e.page * Hkv + hk) * 16 * D;
      kb = ck + off;
      vb = cvv + off;
      if (e.alias >= 0)
        vb = reinterpret_cast<const bf16_t*>(cv.lib_v) + (((int64_t)layer * Hkv + hk) * cv.lib_cap + e.alias) * D;
    } else {
      kb = ck + head0 + (int64_t)tile * 16 * D;
      vb = cvv + head0 + (int64_t)tile * 16 * D;
    }
    const int last = kend - 1 - (k0 + tile * 16);  // keys past the range re-read its last key (masked below)
    const uint32_t lds = ring_lds + (uint32_t)(ti & (NB - 1)) * TILE;
#pragma unroll
    for (int j = 0; j < KI; ++j) {
      const int r = j * RI + l / NC, p = l % NC;
      dma16s<NT>(kb, (uint32_t)(min(r, last) * D + (p ^ (r % NC)) * 8) * 2, lds + j * 1024);
    }
#pragma unroll
    for (int j = 0; j < KI; ++j) {
      const int r = j * RI + l / NC, p = l % NC;
      const uint32_t off = (uint32_t)(min(r, last) * D + (p ^ (2 * (r % (NC / 2)))) * 8) * 2;
      if (NT && !(PAGED && cv.v_alias)) dma16s<true>(vb, off, lds + (KI + j) * 1024);
      else dma16s(vb, off, lds + (KI + j) * 1024);
    }
  };

  // at most `ahead` of the wave's youngest tiles still in flight
  auto wait_tiles = [&](int ahead) __attribute__((always_inline)) {
    if (NB > 3 && ahead >= 3) wait_vm<3 * DPT>();
    else if (NB > 2 && ahead == 2) wait_vm<2 * DPT>();
    else if (ahead == 1) wait_vm<DPT>();
    else wait_vm<0>();
  };

  // ---- prologue: into the ring buffer that stays free, the new token's key and
  // value, the position's (cos, sin) row and the query rows; then the first
  // tiles.  Each wave fetches its own copy, so none waits for another.
  constexpr int PRE = NB - 1;
  Entry nx = entry(0);
  char* stage = ring + (NB - 1) * TILE;
  const uint32_t stage_lds = ring_lds + (NB - 1) * TILE;
  {
    const char* qr = reinterpret_cast<const char*>(q + ((int64_t)i * Hq + hk * G) * D);
    const char* kr = reinterpret_cast<const char*>(k + ((int64_t)i * Hkv + hk) * D);
    const char* vr = reinterpret_cast<const char*>(v + ((int64_t)i * Hkv + hk) * D);
    const char* cr = reinterpret_cast<const char*>(rope + (int64_t)pos * HALF);
    const char* src = l < NC ? kr + l * 16 : l < 2 * NC ? vr + (l - NC) * 16 : cr + min(l - 2 * NC, NCS - 1) * 16;
    if (__builtin_expect((((uintptr_t)q | (uintptr_t)k | (uintptr_t)v) & 15) == 0, 1)) {
      dma16(src, stage_lds);
#pragma unroll
      for (int j = 0; j < QI; ++j)
        dma16s(qr, (uint32_t)min(j * 64 + l, G * NC - 1) * 16, stage_lds + (1 + j) * 1024);
    } else {  // a caller's rows may start at any element: ordinary loads there, LDS DMA takes whole 16-byte words
      st16(stage + l * 16, ld16_any(src));
#pragma unroll 1
      for (int j = 0; j < QI; ++j)
        st16(stage + (1 + j) * 1024 + l * 16, ld16_any(qr + min(j * 64 + l, G * NC - 1) * 16));
    }
  }
#pragma unroll 1  // one copy of the code: every instruction of a short launch is fetched for it
  for (int u = 0; u < min(n, PRE); ++u) {
    const Entry e = nx;
    nx = entry(u + 1);
    issue(u, e);
  }
  wait_tiles(min(n, PRE));  // all but the tiles: the staged rows have landed

  // rotate 8 dims d .. d + 7 given (own dims, partner dims), round to bf16
  const float* cs = reinterpret_cast<const float*>(stage + 2 * NC * 16);
  auto encode8 = [&](int d, const uint4& xa, const uint4& xb) __attribute__((always_inline)) -> uint4 {
    float a[8], b[8], y[8];
    uint4 cw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) cw[e] = ld16(cs + 2 * (d % HALF) + 4 * e);
    const float* c = reinterpret_cast<const float*>(cw);  // (cos, sin) x 8
    Store<bf16_t>::unpack(xa, a);
    Store<bf16_t>::unpack(xb, b);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      y[e] = d < HALF ? fmaf(a[e], c[2 * e], -b[e] * c[2 * e + 1]) : fmaf(a[e], c[2 * e], b[e] * c[2 * e + 1]);
    return make_uint4(dm_cvt_bf16x2(y[0], y[1]), dm_cvt_bf16x2(y[2], y[3]), dm_cvt_bf16x2(y[4], y[5]),
                      dm_cvt_bf16x2(y[6], y[7]));
  };
  uint4 qB[KS];  // Q^T operand: column lr (query head lr; zero past the group)
  {
    uint4 qa[KS];
    const char* row = stage + 1024 + min(lr, G - 1) * (D * 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qa[ks] = ld16(row + (ks * 4 + lq) * 16);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // the rotary partners of the lane's dims are its own dims of another k step
      const uint4 e = encode8(ks * 32 + lq * 8, qa[ks], qa[ks ^ (HALF / 32)]);
      qB[ks] = lr < G ? e : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  if (PAGED && new_wave && hk == 0 && l == 0 && npage >= 0) enter_page(cv, seq, pos, npage);
  if (new_wave && l < NC) {
    // encode the new key; key and value wait in LDS for the end of the loop
    const int dn = l * 8;
    const uint4 kn = encode8(dn, ld16(stage + l * 16), ld16(stage + (l ^ (NC / 2)) * 16));
    const uint4 nv = ld16(stage + (NC + l) * 16);
    st16(&s_newk[dn], kn);
    st16(&s_newv[dn], nv);
  }
  const float qscale = 1.4426950408889634f / sqrtf((float)D);

  float mref = -INFINITY, lsum = 0.f;  // running max (log2 units) of query lr, sum of this lane's keys
  dm_f32x4 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = dm_f32x4{0.f, 0.f, 0.f, 0.f};

  // softmax of a tile's scores (lane: keys 4 lq + r of query lr), the first
  // nvalid keys real; returns the probabilities rounded to bf16
  auto soft = [&](const dm_f32x4& s, int nvalid) __attribute__((always_inline)) -> uint2 {
    float x[4], lmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x[r] = 4 * lq + r < nvalid ? s[r] * qscale : -INFINITY;
      lmax = fmaxf(lmax, x[r]);
    }
    if (__builtin_amdgcn_ballot_w64(lmax > mref + 8.f)) {
      // exact running max of each query over its four lanes
      const float mn = max_rows4(fmaxf(mref, lmax));
      const float f = __builtin_amdgcn_exp2f(mref - mn);  // 0 while nothing was seen
      lsum *= f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] *= f;
      mref = mn;
    }
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(x[r] - mref);  // 0 for keys past the tile's real ones
      lsum += p[r];
    }
    return make_uint2(dm_cvt_bf16x2(p[0], p[1]), dm_cvt_bf16x2(p[2], p[3]));
  };

  for (int ti = 0; ti < n; ++ti) {
    if (ti + NB - 1 < n) {
      wait_lds();  // the buffer's last reads (the prologue's rows, then the tile before) have returned
      const Entry e = nx;
      nx = entry(ti + NB);
      issue(ti + NB - 1, e);
    }
    wait_tiles(min(NB - 1, n - 1 - ti));  // this tile has landed; the later ones stay in flight
    const bf16_t* T = reinterpret_cast<const bf16_t*>(ring + (ti & (NB - 1)) * TILE);
    uint4 kk[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kk[ks] = ld16(&T[(lr * NC + ((ks * 4 + lq) ^ (lr % NC))) * 8]);
    // V^T fragment dt: lane (lr, lq) needs V[4 lq + e][16 dt + lr], e = 0..3; in
    // the transpose read, lane lr of group lq addresses row 4 lq + lr / 4, dims
    // 16 dt + 4 (lr % 4) .. + 3
    uint2 va[DT];
    {
      const int vr = 4 * lq + (lr >> 2), vsw = 2 * (vr % (NC / 2));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        va[dt] = ld_tr8(&T[16 * D + (vr * NC + ((2 * dt + ((lr & 3) >> 1)) ^ vsw)) * 8 + (lr & 1) * 4]);
    }
    dm_f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = mma_qk(kk[ks], qB[ks], s);
    const uint2 pb = soft(s, min(16, kend - k0 - (w + 4 * ti) * 16));
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = mma_pv(va[dt], pb, acc[dt]);
  }

  if (new_wave) {
    // the new token: into its cache slot, and attended as a one-key tile (key
    // row 0, value element (key 0) of each dim)
    if (l < NC) {
      const int64_t off = new_token_offset<PAGED>(cv, layer, seq, hk, pos, npage) + l * 8;
      st16(reinterpret_cast<bf16_t*>(cv.k) + off, ld16(&s_newk[l * 8]));
      st16(reinterpret_cast<bf16_t*>(cv.v) + off, ld16(&s_newv[l * 8]));
    }
    dm_f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 kn = ld16(&s_newk[ks * 32 + lq * 8]);
      s = mma_qk(lr == 0 ? kn : make_uint4(0u, 0u, 0u, 0u), qB[ks], s);
    }
    const uint2 pb = soft(s, 1);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      acc[dt] = mma_pv(make_uint2(lq == 0 ? (uint32_t)s_newv[dt * 16 + lr] : 0u, 0u), pb, acc[dt]);
  }

  // ---- merge the four waves: per query, M over the waves, each wave's output
  // and sum weighted by 2^(m - M).  A wave's outputs go into its own ring, which
  // no other wave reads before the barrier.
  lsum = sum_rows4(lsum);
  wait_lds();
  if (lr < G) {
    float* o = reinterpret_cast<float*>(ring);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *reinterpret_cast<float4*>(&o[lr * D + dt * 16 + 4 * lq]) =
          make_float4(acc[dt][0], acc[dt][1], acc[dt][2], acc[dt][3]);
    if (lq == 0) {
      s_wm[w][lr] = mref;
      s_wl[w][lr] = lsum;
    }
  }
  __syncthreads();
  for (int idx = t; idx < G * D / 2; idx += 256) {
    const int j = idx / (D / 2), d = 2 * (idx % (D / 2));
    float M = -INFINITY;
#pragma unroll
    for (int w2 = 0; w2 < 4; ++w2) M = fmaxf(M, s_wm[w2][j]);
    float L = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < 4; ++w2) {
      const float m = s_wm[w2][j];
      const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
      const float2 o = *reinterpret_cast<const float2*>(s_ring + w2 * (NB * TILE) + (j * D + d) * 4);
      L = fmaf(s_wl[w2][j], f, L);
      a0 = fmaf(o.x, f, a0);
      a1 = fmaf(o.y, f, a1);
    }
    emit_pair<bf16_t, D>(nsplit, part_row(slot0 + split, Hkv, hk, G, j), out + ((int64_t)i * Hq + hk * G + j) * D,
                         part_o, part_ml, d, a0, a1, M, L);
  }
  if (nsplit == 1) return;
  merge_splits<bf16_t, D, G>(args, i, hk, slot0, nsplit, Hkv, Hq, out, part_o, part_ml, count,
                             reinterpret_cast<float*>(s_ring), s_mt, s_lt, &s_last);
}

// ring: 4 where every CU has at most one block of at most 256 keys (plan_decode):
// all of a wave's tiles are requested at once.  2 (two blocks per CU) otherwise; those
// launches also read with the nontemporal hint, the keys
// always and the values unless the tasks share them in the library: whole rows
// read that way arrive at 6.9 TB/s against 6.2 (measured on the kernel, with
// against without: 796 MB 2001 / 2184 us, 369 MB 506 / 553, 131 MB 439 / 460, 44
// MB 425 / 432 per pass; 17.5 MB 1218 / 1201, so not there; shared values
// 1125 / 1097).
int launch_decode_mfma(const DecodeArgs& args, const void* q, const void* k, const void* v, const CacheView& cv,
                       int layer, const float2* rope, int Hq, void* out, float* part_o, float* part_ml,
                       int* count, int ring, hipStream_t s, KTime tm) {
  if (args.n == 0) return 0;
  const int g = Hq / cv.n_kv_heads;
  dim3 grid(args.max_split, args.n, cv.n_kv_heads);
#define DM2(DD, GG, PG, NB)                                                                                   \
  hipExtLaunchKernelGGL((decode_mfma_kernel<DD, GG, PG, NB>), grid, dim3(256), 0, s, tm.start, tm.stop, 0, args,   \
                        (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, cv, rope, (bf16_t*)out, part_o,   \
                        part_ml, count, layer)
#define DM1(DD, GG, PG) { if (ring == 4) DM2(DD, GG, PG, 4); else DM2(DD, GG, PG, 2); }
#define DM(DD, GG)                                                                                            \
  if (cv.page_size) DM1(DD, GG, true)                                                                         \
  else DM1(DD, GG, false)
#define DMG(DD)                                                                                               \
  switch (g) {                                                                                                \
    case 1: DM(DD, 1); break;                                                                                 \
    case 2: DM(DD, 2); break;                                                                                 \
    case 4: DM(DD, 4); break;                                                                                 \
    case 8: DM(DD, 8); break;                                                                                 \
    case 16: DM(DD, 16); break;                                                                               \
    default: return -1;                                                                                       \
  }
  if (cv.head_dim == 64) { DMG(64) } else { DMG(128) }
#undef DMG
#undef DM
#undef DM1
#undef DM2
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? 0 : (int)e;
}

}  // namespace fcg
