// Branch-masked attention over a shared-prefix key/value cache (gfx950).
//
// A row (one lattice node, or one prompt position during prefill) at
// absolute position pos attends to the logical keys 0..pos of its own
// prefix: positions [0, nc) are committed cache entries (shared by every row
// of the sequence), positions [nc, pos] are the entries of its ancestor slots
// and its own slot, listed in `chain`.  Grouped-query heads: query head h
// reads key/value head h / (H / Hkv).
//
// Decode: the keys are cut into splits of 64 logical positions; a split
// kernel writes one (o, max, sum) partial per (row, query head, split) and
// combine_kernel merges a row's splits.  attn_mfma_kernel (bf16, head_dim 64
// and 128) runs the two products on the matrix cores; attn_kernel (fp32
// models, bf16 head_dim 32) is its VALU form: one workgroup per (row group,
// kv head, split) stages the split's committed keys and values in LDS,
// patches in each row's chain entries, and scores, normalises and sums per
// row with one lane per key and then per value dimension.
//
// Every quantity a row computes depends only on its logical key sequence:
// split and tile boundaries are fixed logical positions, each dot product
// and each value sum runs in a fixed key/dimension order whether the key is
// read from the committed cache or a chain entry, and the combine's order
// depends only on the row's split count.  So a node evaluated speculatively
// (tail keys in lattice slots) gets the bits plain decoding gets at the same
// position.  Splits of 64 keys keep a long context spread over many waves:
// 8192 keys x 8 kv heads x 8 sequences is 9216 waves per layer.
//
// Prefill: prefill_attn_kernel computes causal attention over the prompt's
// own keys.
#include "attn_decode.h"

namespace dex {


// Element e of a packed row held as 32-bit words (bf16 pairs or floats).
template <typename T> __device__ __forceinline__ float unpack(const uint32_t *w, int e);
template <> __device__ __forceinline__ float unpack<bf16>(const uint32_t *w, int e) {
  const uint32_t u = w[e >> 1];
  return __uint_as_float((e & 1) ? (u & 0xffff0000u) : (u << 16));
}
template <> __device__ __forceinline__ float unpack<float>(const uint32_t *w, int e) { return __uint_as_float(w[e]); }

// A split record element: the split's output in the cache's element type
// (bf16 rounded to nearest even).
template <typename T> __device__ __forceinline__ T rec_elem(float v);
template <> __device__ __forceinline__ float rec_elem<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 rec_elem<bf16>(float v) { return pf_f2bf(v); }
template <typename T> __device__ __forceinline__ float rec_val(T v);
template <> __device__ __forceinline__ float rec_val<float>(float v) { return v; }
template <> __device__ __forceinline__ float rec_val<bf16>(bf16 v) { return __uint_as_float((uint32_t)v << 16); }

// DPL consecutive record elements (one load) as floats; zeros if !ok.
template <typename T, int DPL>
__device__ __forceinline__ void rec_load(const T *p, bool ok, float (&v)[DPL]) {
  if constexpr (DPL == 2 && sizeof(T) == 2) {
    const uint32_t u = ok ? *(const uint32_t *)p : 0u;
    v[0] = __uint_as_float(u << 16);
    v[1] = __uint_as_float(u & 0xffff0000u);
  } else if constexpr (DPL == 2) {
    const float2 f = ok ? *(const float2 *)p : make_float2(0.f, 0.f);
    v[0] = f.x;
    v[1] = f.y;
  } else {
#pragma unroll
    for (int q = 0; q < DPL; ++q) v[q] = ok ? rec_val<T>(p[q]) : 0.f;
  }
}

// One wave per (row group, kv head, split of 64 logical keys).  Lane i owns
// key s0 + i for the scores and head dimensions [i*DPL, i*DPL + DPL) for the
// value sum.
// ONE: every row of the launch has one split, whose combine (weight
// e^0 = 1) is the division by its sum: the row goes out at once, row r of the
// group's rows as row out0 + r of c.
template <typename T, int HD, bool ONE>
__device__ __forceinline__ void attn_item(const AttnArgs &a, int gi, int kvh, int split, const CombineArgs &c, int out0) {
  constexpr int WORDS = HD * (int)sizeof(T) / 4;     // 32-bit words per key row
  constexpr int V4 = WORDS / 4;                      // 16-byte loads per key row
  constexpr int DPL = HD >= 64 ? HD / 64 : 1;        // value dims per lane
  constexpr int GMAX = 8;
  constexpr int KSTRIDE = WORDS + 4;
  constexpr int EPC = 16 / (int)sizeof(T);           // elements per 16-byte chunk
  __shared__ __attribute__((aligned(16))) float qs[GMAX][HD];
  __shared__ __attribute__((aligned(16))) uint32_t ks[ATT_SPLIT][KSTRIDE];
  __shared__ __attribute__((aligned(16))) uint32_t vs[ATT_SPLIT][WORDS];
  __shared__ __attribute__((aligned(16))) float es[GMAX][ATT_SPLIT];

  const int r0 = a.grp_row0[gi], nr = a.grp_nrows[gi], seq = a.grp_seq[gi];
  const int G = a.n_heads / a.n_kv_heads;
  const int lane = threadIdx.x;
  int maxpos = 0, ncmax = 0;
  for (int r = 0; r < nr; ++r) {
    maxpos = max(maxpos, a.row_pos[r0 + r]);
    ncmax = max(ncmax, a.row_nc[r0 + r]);
  }
  const int s0 = split * ATT_SPLIT;
  if (s0 > maxpos) return;
  const T *kbase = (const T *)a.kc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;
  const T *vbase = (const T *)a.vc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;

  // committed keys and values of the split, loaded together with the first
  // row's queries: each instruction covers four whole key rows (1 KB
  // contiguous), then K goes to one padded LDS row per key (lane i's key
  // row i) and V to the value tile.  Positions past the committed prefix
  // stay zero until a row's chain entries are patched in.
  const int t = s0 + lane;
  uint4 *krow = (uint4 *)&ks[lane][0];
  const int tn = max(0, min(ATT_SPLIT, ncmax - s0));
  // `held` names the key in this lane's LDS row: -2 the committed one at
  // position t, -1 none, else a cache entry of a row's chain
  int held = t - s0 < tn ? -2 : -1;
  constexpr int Q4 = GMAX * HD / 4 / ATT_THREADS;
  float4 qv[Q4];
  auto load_q = [&](int r) {
    const float4 *qsrc = (const float4 *)(a.q + (size_t)r * a.ldq + kvh * G * HD);
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      const int e = lane + i * ATT_THREADS;
      qv[i] = (e < G * HD / 4) ? qsrc[e] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  {
    constexpr int PER = ATT_SPLIT * V4 / ATT_THREADS;   // 16-byte loads per lane
    uint4 v[PER], k[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + i * ATT_THREADS, j = e / V4, c = e % V4;
      const bool ok = j < tn;
      k[i] = ok ? ((const uint4 *)(kbase + (size_t)(s0 + j) * HD))[c] : make_uint4(0, 0, 0, 0);
      v[i] = ok ? ((const uint4 *)(vbase + (size_t)(s0 + j) * HD))[c] : make_uint4(0, 0, 0, 0);
    }
    load_q(r0);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = lane + i * ATT_THREADS;
      *((uint4 *)&ks[e / V4][0] + e % V4) = k[i];
      *((uint4 *)&vs[e / V4][0] + e % V4) = v[i];
    }
  }

  for (int rr = 0; rr < nr; ++rr) {
    const int r = r0 + rr;
    const int pos = a.row_pos[r], nc = a.row_nc[r], coff = a.row_chain_off[r];
    if (s0 > pos) continue;
    if (rr > 0) load_q(r);
    __syncthreads();
    {
      float4 *qdst = (float4 *)&qs[0][0];
#pragma unroll
      for (int i = 0; i < Q4; ++i) qdst[lane + i * ATT_THREADS] = qv[i];
    }
    // this row's chain values at positions [max(nc, s0), pos] of the split
    const int tb = max(nc, s0), te = min(pos, s0 + ATT_SPLIT - 1);
    for (int e = lane; e < (te - tb + 1) * V4; e += ATT_THREADS) {
      const int tj = tb + e / V4, c = e % V4;
      *((uint4 *)&vs[tj - s0][0] + c) = ((const uint4 *)(vbase + (size_t)a.chain[coff + (tj - nc)] * HD))[c];
    }
    // this row's key at logical position t: committed, or its own chain
    const bool valid = t <= pos;
    const int want = (t < nc) ? -2 : (valid ? a.chain[coff + (t - nc)] : -1);
    if (want != -1 && want != held) {
      const uint4 *src = (const uint4 *)(kbase + (size_t)(want == -2 ? t : want) * HD);
#pragma unroll
      for (int i = 0; i < V4; ++i) krow[i] = src[i];
      held = want;
    }
    __syncthreads();
    // scores, one independent chain per head, dimensions in order
    float sacc[GMAX];
#pragma unroll
    for (int g = 0; g < GMAX; ++g) sacc[g] = 0.f;
#pragma unroll 2
    for (int c = 0; c < V4; ++c) {
      const uint4 kw = valid ? krow[c] : make_uint4(0, 0, 0, 0);
      const uint32_t w4[4] = {kw.x, kw.y, kw.z, kw.w};
      float kv[EPC];
#pragma unroll
      for (int e2 = 0; e2 < EPC; ++e2) kv[e2] = unpack<T>(w4, e2);
#pragma unroll
      for (int g = 0; g < GMAX; ++g) {
        if (g < G) {
          const float4 *q4 = (const float4 *)&qs[g][c * EPC];
#pragma unroll
          for (int e4 = 0; e4 < EPC / 4; ++e4) {
            const float4 qq = q4[e4];
            sacc[g] = fmaf(qq.x, kv[4 * e4 + 0], sacc[g]);
            sacc[g] = fmaf(qq.y, kv[4 * e4 + 1], sacc[g]);
            sacc[g] = fmaf(qq.z, kv[4 * e4 + 2], sacc[g]);
            sacc[g] = fmaf(qq.w, kv[4 * e4 + 3], sacc[g]);
          }
        }
      }
    }
    float m[GMAX], l[GMAX];
#pragma unroll
    for (int g = 0; g < GMAX; ++g) {
      if (g >= G) break;
      const float sc = valid ? sacc[g] * a.scale : -INFINITY;
      m[g] = wave_max(sc);
      const float e = valid ? expf(sc - m[g]) : 0.f;
      l[g] = wave_sum(e);
      es[g][lane] = e;
    }
    __syncthreads();
    // value sum over the split's 64 keys in position order (weights of keys
    // past pos are exactly zero and their values finite)
    float o[GMAX][DPL];
#pragma unroll
    for (int g = 0; g < GMAX; ++g)
#pragma unroll
      for (int q = 0; q < DPL; ++q) o[g][q] = 0.f;
    const int d0 = lane * DPL;
    const bool dims_ok = d0 < HD;
    const int dsafe = dims_ok ? d0 : 0;
#pragma unroll 4
    for (int j0 = 0; j0 < ATT_SPLIT; j0 += 4) {
      float v[4][DPL];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int q = 0; q < DPL; ++q) v[jj][q] = unpack<T>(&vs[j0 + jj][0], dsafe + q);
#pragma unroll
      for (int g = 0; g < GMAX; ++g) {
        if (g >= G) break;
        const float4 e4 = *(const float4 *)&es[g][j0];
        const float ev[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int q = 0; q < DPL; ++q) o[g][q] = fmaf(ev[jj], v[jj][q], o[g][q]);
      }
    }
#pragma unroll
    for (int g = 0; g < GMAX; ++g) {
      if (g >= G) break;
      if constexpr (ONE) {
        const int pk = c.row_pk != nullptr ? c.row_pk[out0 + r] : c.row0 + out0 + r;
        const int rm = c.row_pk != nullptr ? pk < 0 : c.rm, ro = c.row_pk != nullptr && rm ? ~pk : pk;
        const int col = (kvh * G + g) * HD + d0;
        T *out = (T *)c.out + (c.out_steps > 0 ? act_off<T>(ro, col, c.out_steps, rm) : (size_t)(out0 + r) * c.ld_out + col);
        if (dims_ok) {
#pragma unroll
          for (int q = 0; q < DPL; ++q) out[q] = rec_elem<T>(rec_val<T>(rec_elem<T>(o[g][q])) / l[g]);
        }
        continue;
      }
      const size_t rec = ((size_t)r * a.n_heads + kvh * G + g) * a.jmax + split;
      T *dst = (T *)a.part + rec * HD;
      if (dims_ok) {
#pragma unroll
        for (int q = 0; q < DPL; ++q) dst[d0 + q] = rec_elem<T>(o[g][q]);
      }
      if (lane == 0) { a.stat[2 * rec] = m[g]; a.stat[2 * rec + 1] = l[g]; }
    }
  }
}

template <typename T, int HD>
__global__ __launch_bounds__(ATT_THREADS) void attn_kernel(AttnArgs a) {
  attn_item<T, HD, false>(a, blockIdx.x, blockIdx.y, blockIdx.z, CombineArgs{}, 0);
}

// out[r][h] = sum_j w_j o_j / sum_j w_j l_j with w_j = e^{m_j - M},
// M = max_j m_j, over the splits j = 0 .. pos/64 of row r (each split record
// holds its output o_j, in the cache's element type, and its float
// (m_j, l_j)).  One workgroup of CMB_WAVES
// waves per (row, head): wave s sums the splits j = s, s + CMB_WAVES, ... in
// order (lanes over head dimensions) and the wave sums are added in wave
// order; the statistics take one fixed reduction.  The arithmetic depends
// only on the row's split count, never on the other rows of the launch.
// DW head dimensions per workgroup (blockIdx.z picks the slice): each
// dimension's sum is computed the same way whatever the slicing, so a
// launch with few rows splits a head over two workgroups for more latency
// hiding, and the bits do not change.
#ifndef CMB_WAVES
#define CMB_WAVES 4
#endif
template <typename T, typename REC, int HD, int DW>
__global__ __launch_bounds__(64 * CMB_WAVES) void combine_kernel(CombineArgs a) {
  // dimensions per lane: 4-byte record loads for bf16 (whole heads: 64
  // lanes x 2; half heads: 32 lanes x 2)
  constexpr int DPL = sizeof(REC) == 2 ? (DW >= 128 ? DW / 64 : 2) : (DW >= 64 ? DW / 64 : 1);
  constexpr int CH = 16;                       // splits per value chunk
  constexpr int NT = 64 * CMB_WAVES;
  extern __shared__ float ws[];                // [jmax] split weights
  __shared__ float red[CMB_WAVES][DW];         // per-wave weighted sums
  __shared__ float sred[2][CMB_WAVES];         // per-wave max and denominator
  const int r = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, s = tid >> 6;
  const int nsplit = a.row_pos[r] / ATT_SPLIT + 1;
  const int nmine = nsplit > s ? (nsplit - s + CMB_WAVES - 1) / CMB_WAVES : 0;
  const REC *src = (const REC *)a.part + ((size_t)r * a.n_heads + h) * a.jmax * HD;
  const float *sst = a.stat + ((size_t)r * a.n_heads + h) * a.jmax * 2;
  const int dl = lane * DPL;                   // this lane's first dimension in the slice
  const int d0 = blockIdx.z * DW + dl;
  const bool dok = dl < DW;
  // the split values do not depend on the statistics: the first chunk is
  // requested before them, each next chunk before the current one is summed
  float va[CH][DPL], vb[CH][DPL];
  auto load_chunk = [&](int i0, float (&v)[CH][DPL]) {
#pragma unroll
    for (int jj = 0; jj < CH; ++jj) {
      const int j = s + (i0 + jj) * CMB_WAVES;
      rec_load<REC, DPL>(src + (size_t)j * HD + d0, dok && i0 + jj < nmine, v[jj]);
    }
  };
  load_chunk(0, va);
  float M = -INFINITY;
  for (int j = tid; j < nsplit; j += NT) M = fmaxf(M, sst[2 * j]);
  M = wave_max(M);
  if (lane == 0) sred[0][s] = M;
  __syncthreads();
  M = sred[0][0];
#pragma unroll
  for (int w = 1; w < CMB_WAVES; ++w) M = fmaxf(M, sred[0][w]);
  float lp = 0.f;
  for (int j = tid; j < nsplit; j += NT) {
    const float w = expf(sst[2 * j] - M);
    ws[j] = w;
    lp = fmaf(w, sst[2 * j + 1], lp);
  }
  lp = wave_sum(lp);
  if (lane == 0) sred[1][s] = lp;
  __syncthreads();
  float lsum = sred[1][0];
#pragma unroll
  for (int w = 1; w < CMB_WAVES; ++w) lsum += sred[1][w];
  float o[DPL];
#pragma unroll
  for (int q = 0; q < DPL; ++q) o[q] = 0.f;
  auto sum_chunk = [&](int i0, const float (&v)[CH][DPL]) {
#pragma unroll
    for (int jj = 0; jj < CH; ++jj) {
      if (i0 + jj >= nmine) break;
      const float w = ws[s + (i0 + jj) * CMB_WAVES];
#pragma unroll
      for (int q = 0; q < DPL; ++q) o[q] = fmaf(w, v[jj][q], o[q]);
    }
  };
  for (int i0 = 0; i0 < nmine; i0 += 2 * CH) {
    if (i0 + CH < nmine) load_chunk(i0 + CH, vb);
    sum_chunk(i0, va);
    if (i0 + CH >= nmine) break;
    if (i0 + 2 * CH < nmine) load_chunk(i0 + 2 * CH, va);
    sum_chunk(i0 + CH, vb);
  }
  if (dok) {
#pragma unroll
    for (int q = 0; q < DPL; ++q) red[s][dl + q] = o[q];
  }
  __syncthreads();
  if (s != 0 || !dok) return;
  // a lane's dimensions share 16 bytes in every layout
  const int pk = a.row_pk != nullptr ? a.row_pk[r] : a.row0 + r, rm = a.row_pk != nullptr ? pk < 0 : a.rm;
  T *out = (T *)a.out + (a.out_steps > 0 ? act_off<T>(a.row_pk != nullptr && rm ? ~pk : pk, h * HD + d0, a.out_steps, rm)
                                         : (size_t)r * a.ld_out + h * HD + d0);
#pragma unroll
  for (int q = 0; q < DPL; ++q) {
    float v = red[0][dl + q];
#pragma unroll
    for (int w = 1; w < CMB_WAVES; ++w) v += red[w][dl + q];
    v = v / lsum;
    if constexpr (sizeof(T) == 2) {
      uint32_t u = __float_as_uint(v);
      u += 0x7fffu + ((u >> 16) & 1u);
      out[q] = (T)(u >> 16);
    } else {
      out[q] = v;
    }
  }
}

// The arguments of segment sg alone: its layer of the cache, its queries,
// rows and row groups, and the split records of its rows in the launch's
// row space (records of element type T).
template <typename T>
static __host__ __device__ inline void attn_seg_view(AttnArgs &a, const AttnSeg &sg) {
  const size_t r0 = (size_t)sg.r0;
  a.kc = sg.kc;
  a.vc = sg.vc;
  a.q += r0 * a.ldq;
  a.row_pos += r0;
  a.row_nc += r0;
  a.row_chain_off += r0;
  a.row_seq += r0;
  a.grp_row0 += sg.g0;
  a.grp_nrows += sg.g0;
  a.grp_seq += sg.g0;
  if (a.grp_nc != nullptr) a.grp_nc += sg.g0;
  a.n_rows = sg.M;
  a.n_splits = sg.n_splits;
  a.part = (T *)a.part + r0 * a.n_heads * a.jmax * a.head_dim;
  a.stat += r0 * a.n_heads * a.jmax * 2;
}

// The segment whose items hold item x.
__device__ __forceinline__ int find_seg(const AttnSegs &g, int x) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < MAX_SEGS; ++i) k += (i < g.n && x >= g.item0[i]) ? 1 : 0;
  return k;
}

// Grouped form: block x is row group x - item0 of the segment that holds it
// (the fp32 model's four stages: one launch instead of four of 7.5 us).
template <typename T, int HD>
__global__ __launch_bounds__(ATT_THREADS) void attn_seg_kernel(AttnArgs a, AttnSegs g) {
  const int k = find_seg(g, blockIdx.x);
  if ((int)blockIdx.z >= g.s[k].n_splits) return;
  attn_seg_view<T>(a, g.s[k]);
  attn_item<T, HD, false>(a, blockIdx.x - g.item0[k], blockIdx.y, blockIdx.z, CombineArgs{}, 0);
}

// Rows of one split (see ONE): attention and combine in one launch.
template <typename T, int HD>
__global__ __launch_bounds__(ATT_THREADS) void attn_one_seg_kernel(AttnArgs a, CombineArgs c, AttnSegs g) {
  const int k = find_seg(g, blockIdx.x);
  attn_seg_view<T>(a, g.s[k]);
  attn_item<T, HD, true>(a, blockIdx.x - g.item0[k], blockIdx.y, 0, c, g.s[k].r0);
}

template <typename T>
static hipError_t launch_attn_t(const AttnArgs &a, const AttnSegs *g, dim3 grid, hipStream_t s) {
  const dim3 block(ATT_THREADS);
  switch (a.head_dim) {
    case 32:
      if (g != nullptr) hipLaunchKernelGGL((attn_seg_kernel<T, 32>), grid, block, 0, s, a, *g);
      else hipLaunchKernelGGL((attn_kernel<T, 32>), grid, block, 0, s, a);
      break;
    case 64:
      if (g != nullptr) hipLaunchKernelGGL((attn_seg_kernel<T, 64>), grid, block, 0, s, a, *g);
      else hipLaunchKernelGGL((attn_kernel<T, 64>), grid, block, 0, s, a);
      break;
    case 128:
      if (g != nullptr) hipLaunchKernelGGL((attn_seg_kernel<T, 128>), grid, block, 0, s, a, *g);
      else hipLaunchKernelGGL((attn_kernel<T, 128>), grid, block, 0, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, typename REC>
static hipError_t launch_comb_t(const CombineArgs &a, int rows, hipStream_t s) {
  const size_t smem = (size_t)a.jmax * 4;
  const dim3 block(64 * CMB_WAVES);
  switch (a.head_dim) {
    case 32: hipLaunchKernelGGL((combine_kernel<T, REC, 32, 32>), dim3(rows, a.n_heads), block, smem, s, a); break;
    case 64: hipLaunchKernelGGL((combine_kernel<T, REC, 64, 64>), dim3(rows, a.n_heads), block, smem, s, a); break;
    case 128:
      // up to 512 (row, head) pairs: half a head per workgroup (latency-bound
      // launches); beyond, a whole head (bandwidth-bound, fewer statistics reads)
      if ((size_t)rows * a.n_heads <= 512)
        hipLaunchKernelGGL((combine_kernel<T, REC, 128, 64>), dim3(rows, a.n_heads, 2), block, smem, s, a);
      else
        hipLaunchKernelGGL((combine_kernel<T, REC, 128, 128>), dim3(rows, a.n_heads, 1), block, smem, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_combine(int dtype, const CombineArgs &a, int rows, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (a.jmax > ATT_MAX_SPLITS) return hipErrorInvalidValue;
  if (dtype != 1) return launch_comb_t<float, float>(a, rows, s);
  return a.rec_f32 ? launch_comb_t<bf16, float>(a, rows, s) : launch_comb_t<bf16, bf16>(a, rows, s);
}

// ------------------------------------------------------------------------
// Decode attention on the matrix cores (bf16 caches, head_dim 64 or 128): one
// wave per work item (attn_mfma_item in attn_decode.h).
template <int HD, typename REC>
__global__ __launch_bounds__(64) void attn_mfma_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t vr[ATT_SPLIT][HD + 16];
  __shared__ int prow[ATT_MAX_PAIRS];
  __shared__ int ppos[ATT_MAX_PAIRS];
  attn_mfma_item<HD, REC>(a, blockIdx.x, blockIdx.y, vr, prow, ppos);
}

// Grouped form: block x runs item x - item0 of the segment whose items hold it.
template <int HD>
__global__ __launch_bounds__(64) void attn_mfma_seg_kernel(AttnArgs a, AttnSegs g) {
  __shared__ __attribute__((aligned(16))) uint16_t vr[ATT_SPLIT][HD + 16];
  __shared__ int prow[ATT_MAX_PAIRS];
  __shared__ int ppos[ATT_MAX_PAIRS];
  const int x = blockIdx.x, k = find_seg(g, x);
  attn_seg_view<bf16>(a, g.s[k]);
  attn_mfma_item<HD, bf16>(a, x - g.item0[k], blockIdx.y, vr, prow, ppos);
}

// Causal prompt attention on the matrix cores (bf16, head_dim 64 or 128).
// Workgroup = (QW blocks of 16 MT queries, kv head, sequence), wave w = query
// head kvh * G + w % G of query block w / G, so that the G QW waves share the
// keys and values: blocks of KB keys stream into a two-slot LDS ring with
// direct global -> LDS transfers, one block ahead of the products.  Per block
// each wave computes
//   S^T = K Q^T   KB / 16 16-key tiles against its MT 16-query tiles, so each
//                 lane holds KB / 4 keys of one query: the online-softmax
//                 statistics are that lane's plus the four quarter-waves',
//                 and the rescaling of O needs no exchange;
//   O^T += V^T P^T  V^T through the LDS transpose read, P^T straight from
//                 the S^T accumulators (k-slot e of a lane is key
//                 32 st + 4 grp + e or 32 st + 16 + 4 grp + e - 4, the keys it
//                 holds), O^T rows = head dims, columns = queries.
// The vector work beside the products bounds it (at 8 x 8192, counters: 245
// vector instructions against 64 products per 64 keys and 32 queries, the two
// hardly overlapping), so: scale and reference enter through one fused
// multiply-add; only the last block is masked; a query's reference is raised
// (and its O rescaled) only once a score exceeds it by 2^8, which leaves
// every rounding relative; a lane's denominator stays its own until the end;
// key rows past the prompt repeat its last one instead of reading zeros.
// KB depends on head_dim alone and every per-query operation on its own keys
// alone, so a prompt's bits depend neither on the batch nor on MT.
// Three waves a SIMD hide more than two with longer blocks do: at 8 x 8192,
// 32 / 8 heads of 128, KB = 32 takes 4.8 ms and KB = 64 5.2 ms (the earlier
// kernel, masked and rescaled per block: 6.8 ms); at head_dim 64 four waves
// fit either way and KB = 64 wins (18 against 23 us at 2 x 1100, 12 heads,
// where one wave per workgroup took 200 us).  Computing block j + 1's scores
// next to block j's softmax, or alternating the two phases between two
// groups of four waves, spills or drops to two waves: 6.3 and 8.4 ms.
// K and V rows have their 16-byte chunks XOR-swizzled (pa_kswz, pa_vswz) so
// that the 16 rows of a K fragment read and the eight rows that half a wave
// reads for a transposed V fragment land in distinct banks.  Query blocks are
// dispatched longest first (the causal triangle), heads and sequences
// innermost: with a multiple of eight of them, a kv head's blocks share an XCD.

// Max over the four lanes r16, r16 + 16, + 32, + 48.
__device__ __forceinline__ float quarters_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int HD> __device__ __forceinline__ int pa_kswz(int row) { return HD == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int HD> __device__ __forceinline__ int pa_vswz(int row) { return HD == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); }

template <int HD, int MT, int KB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(KB == 32 ? 3 : 2)))
void prefill_attn_kernel(PrefillAttnArgs a, int QW, int n_pairs) {
  constexpr int KS = HD / 32, DT = HD / 16, NKT = KB / 16, QB = 16 * MT;
  constexpr int CPR = HD / 8;                      // 16-byte chunks per key row
  constexpr int RPT = 64 / CPR;                    // key rows per 1 KB transfer
  constexpr int NTR = KB / RPT;                    // transfers per block of keys or values
  __shared__ __attribute__((aligned(16))) uint4 kl[2][KB * CPR];
  __shared__ __attribute__((aligned(16))) uint4 vl[2][KB * CPR];

  const int P = a.prompt_len, G = a.n_heads / a.n_kv_heads;
  const int nqb = (P + QB * QW - 1) / (QB * QW);
  const int pair = blockIdx.x % n_pairs, wg0 = (nqb - 1 - (int)blockIdx.x / n_pairs) * QB * QW;
  const int kvh = pair % a.n_kv_heads, seq = pair / a.n_kv_heads;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, nw = G * QW;
  const int r16 = lane & 15, grp = lane >> 4;
  const int tq = lane >> 4, ti = (lane & 15) >> 2, tg = lane & 3;
  const int h = kvh * G + wave % G;
  const int q0 = wg0 + wave / G * QB;
  const size_t row_base = (size_t)seq * P;
  const uint16_t *kbase = (const uint16_t *)a.kc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;
  const uint16_t *vbase = (const uint16_t *)a.vc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;
  const int nblk = (min(wg0 + QB * QW, P) - 1) / KB + 1;            // key blocks of the workgroup
  const int mine = q0 < P ? (min(q0 + QB, P) - 1) / KB + 1 : 0;     // and of this wave

  // block j of the keys (values) into a ring slot: transfer c moves rows
  // RPT c .. + RPT - 1; lane l fills chunk position l mod CPR of row
  // RPT c + l / CPR with the swizzled global chunk.  Rows past the prompt
  // repeat its last one: no stored query sees them.
  auto issue = [&](const uint16_t *src, uint4 *dst, int j, bool isv) {
    const char *blk = (const char *)(src + (size_t)j * KB * HD);
    const int last = P - 1 - j * KB;
    for (int c = wave; c < NTR; c += nw) {
      const int row = c * RPT + lane / CPR;
      const int chunk = lane % CPR ^ (isv ? pa_vswz<HD>(row) : pa_kswz<HD>(row));
      const unsigned off = (unsigned)min(row, last) * (HD * 2) + chunk * 16;
      __builtin_amdgcn_global_load_lds((const void *)(blk + off), (__attribute__((address_space(3))) void *)(dst + c * 64),
                                       16, 0, 0);
    }
  };
  issue(kbase, kl[0], 0, false);
  issue(vbase, vl[0], 0, true);

  // Q^T fragments (B operand): lane (query r16 of tile mt, grp) holds dims
  // 32 st + 8 grp .. +8, rounded to bf16
  pf_bf16x8 qf[MT][KS];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = q0 + mt * 16 + r16;
    const bool ok = row < P;
    const float *src = a.q + (row_base + (ok ? row : 0)) * a.ldq + h * HD + grp * 8;
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      float4 x0 = make_float4(0.f, 0.f, 0.f, 0.f), x1 = x0;
      if (ok) {
        x0 = *(const float4 *)(src + st * 32);
        x1 = *(const float4 *)(src + st * 32 + 4);
      }
      qf[mt][st] = __builtin_bit_cast(pf_bf16x8, make_uint4(pf_pack_bf16(x0.x, x0.y), pf_pack_bf16(x0.z, x0.w),
                                                            pf_pack_bf16(x1.x, x1.y), pf_pack_bf16(x1.z, x1.w)));
    }
  }
  pf_f32x4 o[MT][DT], sc[NKT][MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[mt][dt] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
  float mrun[MT], lrun[MT];                        // reference (log2 units) and this lane's denominator
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) { mrun[mt] = -INFINITY; lrun[mt] = 0.f; }
  const float sl2 = a.scale * 1.44269504088896341f;

  auto scores = [&](const uint4 *K, pf_f32x4 (&sc)[NKT][MT]) {
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) sc[nt][mt] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt) {
        const int row = nt * 16 + r16;
        const pf_bf16x8 kfr = __builtin_bit_cast(pf_bf16x8, K[row * CPR + ((st * 4 + grp) ^ pa_kswz<HD>(row))]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          sc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr, qf[mt][st], sc[nt][mt], 0, 0, 0);
      }
  };
  // raise the reference of the queries whose block maximum calls for it
  auto reference = [&](const pf_f32x4 (&sc)[NKT][MT]) {
    float mx[MT];
    bool up = false;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float m0 = -INFINITY, m1 = -INFINITY;
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt) {
        m0 = fmaxf(fmaxf(m0, sc[nt][mt][0]), sc[nt][mt][1]);
        m1 = fmaxf(fmaxf(m1, sc[nt][mt][2]), sc[nt][mt][3]);
      }
      mx[mt] = quarters_max(fmaxf(m0, m1)) * sl2;
      up |= mx[mt] > mrun[mt] + 8.f;
    }
    if (__any(up)) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        // a query whose own block does not call for it keeps its reference
        // (alpha = 1), so that its bits do not depend on its neighbours
        const float mnew = mx[mt] > mrun[mt] + 8.f ? mx[mt] : mrun[mt];
        const float alpha = mnew == mrun[mt] ? 1.f : __builtin_amdgcn_exp2f(mrun[mt] - mnew);
        mrun[mt] = mnew;
        lrun[mt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[mt][dt] *= alpha;
      }
    }
  };
  // P = exp2(s scale log2 e - reference), rounded to bf16 in the B operand's k-slots
  auto weights = [&](pf_f32x4 (&sc)[NKT][MT], pf_bf16x8 (&pb)[MT][KB / 32]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float mneg = mrun[mt] == -INFINITY ? 0.f : -mrun[mt];
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sc[nt][mt][i], sl2, mneg));
          sc[nt][mt][i] = p;
          lrun[mt] += p;
        }
#pragma unroll
      for (int st = 0; st < KB / 32; ++st)
        pb[mt][st] = __builtin_bit_cast(
            pf_bf16x8, make_uint4(pf_pack_bf16(sc[2 * st][mt][0], sc[2 * st][mt][1]),
                                  pf_pack_bf16(sc[2 * st][mt][2], sc[2 * st][mt][3]),
                                  pf_pack_bf16(sc[2 * st + 1][mt][0], sc[2 * st + 1][mt][1]),
                                  pf_pack_bf16(sc[2 * st + 1][mt][2], sc[2 * st + 1][mt][3])));
    }
  };
  auto values = [&](const uint16_t *V, const pf_bf16x8 (&pb)[MT][KB / 32]) {
#pragma unroll
    for (int st = 0; st < KB / 32; ++st) {
      const int rlo = 32 * st + 4 * tq + ti, rhi = rlo + 16;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int c = 2 * dt + (tg >> 1);
        const pf_bf16x8 vfr = tr_frag(V + (rlo * CPR + (c ^ pa_vswz<HD>(rlo))) * 8 + (tg & 1) * 4,
                                      V + (rhi * CPR + (c ^ pa_vswz<HD>(rhi))) * 8 + (tg & 1) * 4);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          o[mt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vfr, pb[mt][st], o[mt][dt], 0, 0, 0);
      }
    }
  };

  for (int j = 0; j < nblk; ++j) {
    // block j has landed for every wave, and every wave is past block j - 1,
    // whose slots take block j + 1
    lds_ring_step<0>();
    if (j + 1 < nblk) {
      issue(kbase, kl[(j + 1) & 1], j + 1, false);
      issue(vbase, vl[(j + 1) & 1], j + 1, true);
    }
    if (j >= mine) continue;
    pf_bf16x8 pb[MT][KB / 32];
    scores(kl[j & 1], sc);
    if (j + 1 == mine) {                           // the block with the diagonal
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int room = q0 + mt * 16 + r16 - j * KB - grp * 4;   // keys 16 nt + i up to it are seen
#pragma unroll
        for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[nt][mt][i] = nt * 16 + i > room ? -INFINITY : sc[nt][mt][i];
      }
    }
    reference(sc);
    weights(sc, pb);
    values((const uint16_t *)vl[j & 1], pb);
  }
  // O / l -> bf16: lane holds dims 16 dt + 4 grp .. +3 of query q0 + 16 mt + r16
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int query = q0 + mt * 16 + r16;
    float l = lrun[mt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (query >= P) continue;
    const float inv = 1.f / l;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *(uint2 *)((uint16_t *)a.out + pk_off<bf16>((int)row_base + query, h * HD + dt * 16 + grp * 4, a.out_steps)) =
          make_uint2(pf_pack_bf16(o[mt][dt][0] * inv, o[mt][dt][1] * inv),
                     pf_pack_bf16(o[mt][dt][2] * inv, o[mt][dt][3] * inv));
  }
}

template <int HD, int MT, int KB>
static hipError_t launch_prefill_t(const PrefillAttnArgs &a, hipStream_t s) {
  const int G = a.n_heads / a.n_kv_heads, pairs = a.n_kv_heads * a.batch, qw = G >= 4 ? 1 : 4 / G;
  const long long n_wg = (long long)((a.prompt_len + 16 * MT * qw - 1) / (16 * MT * qw)) * pairs;
  if (n_wg > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((prefill_attn_kernel<HD, MT, KB>), dim3((unsigned)n_wg), dim3(64 * G * qw), 0, s, a, qw, pairs);
  return hipGetLastError();
}

// Two query tiles a wave once that leaves four workgroups per compute unit, one
// below (one against two, us; launches of up to 8192 rows, as prompts make them,
// and of one prompt of 16384): 32 / 8 heads of 128, 560 workgroups 43.4 / 48.7,
// 1024 63.6 to 207 / 56.6 to 179, 2048 120 to 790 / 106 to 652; 8 / 8 heads
// of 128, 512 137 / 159, 1024 818 / 705; 12 / 12 heads of 64, 768 14.6 to 170 /
// 15.5 to 181, 1536 642 / 532; 16 / 8 heads of 64, 512 72 / 87, 1024 36 to 214 /
// 35 to 200.  Of 112 shapes the rule misses by at most 2 %, but for 6 % at one
// prompt of 16384 with 8 heads of 128 per kv head (1446 / 1540).
hipError_t launch_prefill_attention(const PrefillAttnArgs &a, hipStream_t s) {
  const int G = a.n_heads / a.n_kv_heads;
  if (G < 1 || G > 8 || a.prompt_len < 1 || a.batch < 1 || a.out_steps < 1) return hipErrorInvalidValue;
  const int span = 32 * (G >= 4 ? 1 : 4 / G);
  const bool two = (long long)((a.prompt_len + span - 1) / span) * a.n_kv_heads * a.batch >= 1024;
  switch (a.head_dim) {
    case 64: return two ? launch_prefill_t<64, 2, 64>(a, s) : launch_prefill_t<64, 1, 64>(a, s);
    case 128: return two ? launch_prefill_t<128, 2, 32>(a, s) : launch_prefill_t<128, 1, 32>(a, s);
    default: return hipErrorInvalidValue;
  }
}

static bool mfma_attention(int dtype, int head_dim) { return dtype == 1 && (head_dim == 64 || head_dim == 128); }

hipError_t launch_attention(int dtype, const AttnArgs &a, int n_groups, hipStream_t s) {
  if (n_groups <= 0 || a.n_heads / a.n_kv_heads > 8) return hipErrorInvalidValue;
  if (a.n_splits < 1 || a.n_splits > a.jmax) return hipErrorInvalidValue;
  dim3 grid(n_groups, a.n_kv_heads, a.n_splits);
  if (a.rec_f32 && !mfma_attention(dtype, a.head_dim)) return hipErrorInvalidValue;
  if (mfma_attention(dtype, a.head_dim)) {
    if (a.n_rows < 1 || a.row_seq == nullptr) return hipErrorInvalidValue;
    const size_t items = 2 * (size_t)a.n_rows + (size_t)n_groups * a.n_splits;
    if (items > 0x7fffffffull) return hipErrorInvalidValue;
    dim3 g2((unsigned)items, a.n_kv_heads);
    if (a.rec_f32) {
      if (a.head_dim == 128) hipLaunchKernelGGL((attn_mfma_kernel<128, float>), g2, dim3(64), 0, s, a);
      else hipLaunchKernelGGL((attn_mfma_kernel<64, float>), g2, dim3(64), 0, s, a);
    } else {
      if (a.head_dim == 128) hipLaunchKernelGGL((attn_mfma_kernel<128, bf16>), g2, dim3(64), 0, s, a);
      else hipLaunchKernelGGL((attn_mfma_kernel<64, bf16>), g2, dim3(64), 0, s, a);
    }
    return hipGetLastError();
  }
  return dtype == 1 ? launch_attn_t<bf16>(a, nullptr, grid, s) : launch_attn_t<float>(a, nullptr, grid, s);
}

// Up to MAX_SEGS segments per launch, a lone segment as a plain launch.
hipError_t launch_attention_seg(int dtype, const AttnArgs &a, const AttnSeg *segs, int n, hipStream_t s) {
  if (segs == nullptr || n < 1 || a.n_heads / a.n_kv_heads > 8 || a.rec_f32) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i) {
    const AttnSeg &sg = segs[i];
    if (sg.M < 1 || sg.r0 < 0 || sg.g0 < 0 || sg.n_groups < 1 || sg.n_splits < 1 || sg.n_splits > a.jmax)
      return hipErrorInvalidValue;
  }
  const bool mfma = dtype == 1 && (a.head_dim == 128 || a.head_dim == 64);
  if (mfma && a.row_seq == nullptr) return hipErrorInvalidValue;
  for (int i0 = 0; i0 < n; i0 += MAX_SEGS) {
    const int c = n - i0 < MAX_SEGS ? n - i0 : MAX_SEGS;
    if (c == 1) {
      AttnArgs b = a;
      if (dtype == 1) attn_seg_view<bf16>(b, segs[i0]);
      else attn_seg_view<float>(b, segs[i0]);
      const hipError_t e = launch_attention(dtype, b, segs[i0].n_groups, s);
      if (e != hipSuccess) return e;
      continue;
    }
    AttnSegs g{};
    g.n = c;
    size_t items = 0;
    int splits = 0;
    for (int i = 0; i < c; ++i) {
      const AttnSeg &sg = segs[i0 + i];
      g.s[i] = sg;
      g.item0[i] = (int)items;
      items += mfma ? 2 * (size_t)sg.M + (size_t)sg.n_groups * sg.n_splits : (size_t)sg.n_groups;
      if (items > 0x7fffffffull) return hipErrorInvalidValue;
      splits = sg.n_splits > splits ? sg.n_splits : splits;
    }
    for (int i = c; i < MAX_SEGS; ++i) g.item0[i] = (int)items;
    hipError_t e = hipSuccess;
    if (!mfma) {
      const dim3 grid((unsigned)items, a.n_kv_heads, splits);
      e = dtype == 1 ? launch_attn_t<bf16>(a, &g, grid, s) : launch_attn_t<float>(a, &g, grid, s);
    } else {
      const dim3 grid((unsigned)items, a.n_kv_heads);
      if (a.head_dim == 128) hipLaunchKernelGGL(attn_mfma_seg_kernel<128>, grid, dim3(64), 0, s, a, g);
      else hipLaunchKernelGGL(attn_mfma_seg_kernel<64>, grid, dim3(64), 0, s, a, g);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------------
// Short contexts (at most SHORT_SPLITS splits a row), bf16, head_dim 64 or
// 128: attention and split combine in one launch.  Workgroup = (row, kv
// head), wave j = split j; the split records stay in LDS and the workgroup
// merges them.  At this length both kernels are chains of memory round trips
// (6 + 4 us and the gap between them for 0.1 MB of keys), so one launch less
// is what counts; a row alone reads its keys again for every row of its
// sequence, and a compute unit fetches all of a row's splits, which is why
// longer rows keep the split kernels.  Every number is computed as there --
// the same products, statistics, bf16 records, and the combine's own order of
// additions -- so a row's bits do not depend on which of the two ran.
template <int HD, int NS, typename REC>
__device__ __forceinline__ void attn_short_row(const AttnArgs &a, const CombineArgs &c, int r, int kvh) {
  constexpr int KS = HD / 32, DT = HD / 16, NKT = ATT_SPLIT / 16, V4 = HD / 8, RPI = 64 / V4;
  __shared__ __attribute__((aligned(16))) uint16_t vr[NS][ATT_SPLIT][HD + 16];
  __shared__ __attribute__((aligned(16))) REC rec[NS][8][HD];
  __shared__ float2 stat[NS][8];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, grp = lane >> 4;
  const int G = a.n_heads / a.n_kv_heads;
  const int pos = a.row_pos[r], nc = a.row_nc[r], coff = a.row_chain_off[r], seq = a.row_seq[r];
  const int s0 = wave * ATT_SPLIT;
  if (s0 <= pos) {
    const uint16_t *kbase = (const uint16_t *)a.kc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;
    const uint16_t *vbase = (const uint16_t *)a.vc + ((size_t)seq * a.n_kv_heads + kvh) * a.kv_entries * HD;
    // Q^T fragment: pair r16 = query head kvh G + r16, dims 32 st + 8 grp .. +8
    const bool pok = r16 < G;
    const float *qsrc = a.q + (size_t)r * a.ldq + (kvh * G + (pok ? r16 : 0)) * HD + grp * 8;
    float4 qv[KS][2];
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      qv[st][0] = pok ? *(const float4 *)(qsrc + st * 32) : make_float4(0.f, 0.f, 0.f, 0.f);
      qv[st][1] = pok ? *(const float4 *)(qsrc + st * 32 + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    uint4 kf[NKT][KS], vv[V4];
    const int vrow = lane / V4, vch = lane % V4;
    const bool full = s0 + ATT_SPLIT <= nc;
    if (full) {                                   // consecutive cache entries s0 ..
      const uint16_t *kb = kbase + (size_t)s0 * HD, *vb = vbase + (size_t)s0 * HD;
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
        for (int st = 0; st < KS; ++st) kf[nt][st] = *(const uint4 *)(kb + (nt * 16 + r16) * HD + st * 32 + grp * 8);
#pragma unroll
      for (int q = 0; q < V4; ++q) vv[q] = *(const uint4 *)(vb + (q * RPI + vrow) * HD + vch * 8);
    } else {
      // lane j looks up the cache entry of key s0 + j: committed below nc,
      // then the row's chain, -1 past the row
      const int kp = s0 + lane;
      const int mine = kp < nc ? kp : (kp <= pos ? a.chain[coff + (kp - nc)] : -1);
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt) {
        const int e = __shfl(mine, nt * 16 + r16, 64);
#pragma unroll
        for (int st = 0; st < KS; ++st)
          kf[nt][st] = e >= 0 ? *(const uint4 *)(kbase + (size_t)e * HD + st * 32 + grp * 8) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < V4; ++q) {
        const int e = __shfl(mine, q * RPI + vrow, 64);
        vv[q] = e >= 0 ? *(const uint4 *)(vbase + (size_t)e * HD + vch * 8) : make_uint4(0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < V4; ++q) *(uint4 *)&vr[wave][q * RPI + vrow][vch * 8] = vv[q];
    pf_f32x4 sc[NKT];
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt) sc[nt] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      const pf_bf16x8 qf = __builtin_bit_cast(
          pf_bf16x8, make_uint4(pf_pack_bf16(qv[st][0].x, qv[st][0].y), pf_pack_bf16(qv[st][0].z, qv[st][0].w),
                                pf_pack_bf16(qv[st][1].x, qv[st][1].y), pf_pack_bf16(qv[st][1].z, qv[st][1].w)));
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt)
        sc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(pf_bf16x8, kf[nt][st]), qf, sc[nt], 0, 0, 0);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = sc[nt][i] * a.scale;
        if (!full && s0 + nt * 16 + grp * 4 + i > pos) v = -INFINITY;
        sc[nt][i] = v;
        mx = fmaxf(mx, v);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float sum = 0.f;
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = (mx == -INFINITY) ? 0.f : expf(sc[nt][i] - mx);
        sum += e;
        sc[nt][i] = e;
      }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    wave_lds_sync();                              // this wave's value rows
    pf_f32x4 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
    const int tq = lane >> 4, ti = (lane & 15) >> 2, tg = lane & 3;
#pragma unroll
    for (int st = 0; st < ATT_SPLIT / 32; ++st) {
      const pf_bf16x8 pfr = __builtin_bit_cast(
          pf_bf16x8, make_uint4(pf_pack_bf16(sc[2 * st][0], sc[2 * st][1]), pf_pack_bf16(sc[2 * st][2], sc[2 * st][3]),
                                pf_pack_bf16(sc[2 * st + 1][0], sc[2 * st + 1][1]),
                                pf_pack_bf16(sc[2 * st + 1][2], sc[2 * st + 1][3])));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            tr_frag(&vr[wave][32 * st + 4 * tq + ti][16 * dt + 4 * tg],
                    &vr[wave][32 * st + 16 + 4 * tq + ti][16 * dt + 4 * tg]),
            pfr, o[dt], 0, 0, 0);
    }
    if (pok) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) rec_store4(&rec[wave][r16][16 * dt + 4 * grp], o[dt]);
      if (grp == 0) stat[wave][r16] = make_float2(mx, sum);
    }
  }
  __syncthreads();
  // the split combine: two dimensions per thread
  const int nsplit = pos / ATT_SPLIT + 1;
  const int pk = c.row_pk != nullptr ? c.row_pk[r] : c.row0 + r, rm = c.row_pk != nullptr ? pk < 0 : c.rm;
  const int ro = c.row_pk != nullptr && rm ? ~pk : pk;
  for (int e = threadIdx.x; e < G * HD / 2; e += 64 * NS) {
    const int h = e / (HD / 2), d0 = 2 * (e % (HD / 2));
    float M = -INFINITY;
#pragma unroll
    for (int j = 0; j < NS; ++j)
      if (j < nsplit) M = fmaxf(M, stat[j][h].x);
    float lp[4] = {0.f, 0.f, 0.f, 0.f}, v0[4] = {0.f, 0.f, 0.f, 0.f}, v1[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NS; ++j)
      if (j < nsplit) {
        const float w = expf(stat[j][h].x - M);
        float o2[2];
        rec_load<REC, 2>(&rec[j][h][d0], true, o2);
        lp[j] = fmaf(w, stat[j][h].y, 0.f);
        v0[j] = fmaf(w, o2[0], 0.f);
        v1[j] = fmaf(w, o2[1], 0.f);
      }
    const float l = (lp[0] + lp[2]) + (lp[1] + lp[3]);   // the wave butterfly's order
    const uint32_t lo = pf_f2bf((v0[0] + v0[1] + v0[2] + v0[3]) / l), hi = pf_f2bf((v1[0] + v1[1] + v1[2] + v1[3]) / l);
    uint16_t *out = (uint16_t *)c.out;
    const int col = (kvh * G + h) * HD + d0;
    *(uint32_t *)(out + (c.out_steps > 0 ? act_off<bf16>(ro, col, c.out_steps, rm) : (size_t)r * c.ld_out + col)) =
        lo | (hi << 16);
  }
}

template <int HD, int NS, typename REC>
__global__ __launch_bounds__(64 * NS) void attn_short_kernel(AttnArgs a, CombineArgs c, int row0) {
  attn_short_row<HD, NS, REC>(a, c, row0 + blockIdx.x, blockIdx.y);
}

// Grouped form: block x is row x - item0 of the segment that holds it.
template <int HD, int NS>
__global__ __launch_bounds__(64 * NS) void attn_short_seg_kernel(AttnArgs a, CombineArgs c, AttnSegs g) {
  const int x = blockIdx.x, k = find_seg(g, x);
  a.kc = g.s[k].kc;
  a.vc = g.s[k].vc;
  attn_short_row<HD, NS, bf16>(a, c, g.s[k].r0 + x - g.item0[k], blockIdx.y);
}

template <int HD, int NS>
static hipError_t launch_short_t(const AttnArgs &a, const CombineArgs &c, const AttnSeg *segs, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += MAX_SEGS) {
    const int cnt = n - i0 < MAX_SEGS ? n - i0 : MAX_SEGS;
    if (cnt == 1) {
      AttnArgs b = a;
      b.kc = segs[i0].kc;
      b.vc = segs[i0].vc;
      const dim3 grid(segs[i0].M, a.n_kv_heads), block(64 * NS);
      if (a.rec_f32) hipLaunchKernelGGL((attn_short_kernel<HD, NS, float>), grid, block, 0, s, b, c, segs[i0].r0);
      else hipLaunchKernelGGL((attn_short_kernel<HD, NS, bf16>), grid, block, 0, s, b, c, segs[i0].r0);
    } else {
      AttnSegs g{};
      g.n = cnt;
      int rows = 0;
      for (int i = 0; i < cnt; ++i) {
        g.s[i] = segs[i0 + i];
        g.item0[i] = rows;
        rows += g.s[i].M;
      }
      for (int i = cnt; i < MAX_SEGS; ++i) g.item0[i] = rows;
      hipLaunchKernelGGL((attn_short_seg_kernel<HD, NS>), dim3(rows, a.n_kv_heads), dim3(64 * NS), 0, s, a, c, g);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

static int short_splits(const AttnSeg *segs, int n) {
  int m = 0;
  for (int i = 0; i < n; ++i) m = segs[i].n_splits > m ? segs[i].n_splits : m;
  return m;
}

template <typename T>
static hipError_t launch_one_t(const AttnArgs &a, const CombineArgs &c, const AttnSeg *segs, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += MAX_SEGS) {
    AttnSegs g{};
    g.n = n - i0 < MAX_SEGS ? n - i0 : MAX_SEGS;
    int groups = 0;
    for (int i = 0; i < MAX_SEGS; ++i) {
      g.item0[i] = groups;
      if (i >= g.n) continue;
      g.s[i] = segs[i0 + i];
      groups += g.s[i].n_groups;
    }
    const dim3 grid(groups, a.n_kv_heads), block(ATT_THREADS);
    switch (a.head_dim) {
      case 32: hipLaunchKernelGGL((attn_one_seg_kernel<T, 32>), grid, block, 0, s, a, c, g); break;
      case 64: hipLaunchKernelGGL((attn_one_seg_kernel<T, 64>), grid, block, 0, s, a, c, g); break;
      case 128: hipLaunchKernelGGL((attn_one_seg_kernel<T, 128>), grid, block, 0, s, a, c, g); break;
      default: return hipErrorInvalidValue;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Rows that share no keys (a row each per group) always gain from the one
// launch.  Rows of a group share theirs in the split kernels, where the one
// launch fetches them for every row, so it loses once its workgroups (row, kv
// head) are many, the sooner the more splits each holds and the fewer (row,
// head) pairs the split kernels fill their columns with.  Stand-alone calls of
// 1 to 256 rows, one launch against split kernels and combine (us), 8 or 12 kv
// heads.  Three or four splits, heads of 128: 256 workgroups 30 / 30 (G 1) and
// 30 / 31 (G 4), 512 42 / 32 and 42 / 36, 2048 88 / 51 and 89 / 72; G 8: 1024
// 59 / 64, 2048 106 / 97 at worst; heads of 64, G 1: 576 31 / 31, 1152 39 / 33,
// 3072 56 / 48; G 4: 2048 55 / 58.  Two splits, heads of 128, G 1: 768 30 / 32,
// 1024 37 / 33; no loss at G 4 and 8, at heads of 64 and with one split.
// Rounds of 176 rows in 64 sequences, four splits, few rows a group, two
// layers' attention: heads of 128, G 1 109 / 80, G 4 111 / 107, G 8 124 / 135;
// heads of 64, G 1 46 / 52; two splits, heads of 128, G 1 47 / 55.
static bool short_pays(const AttnArgs &a, int splits, const AttnSeg *segs, int n) {
  const int G = a.n_heads / a.n_kv_heads;
  long long rows = 0, groups = 0;
  for (int i = 0; i < n; ++i) { rows += segs[i].M; groups += segs[i].n_groups; }
  const long long wgs = rows * a.n_kv_heads;
  if (splits == 1 || rows == groups) return true;
  const bool few = rows < 2 * groups;          // rows a group
  if (a.head_dim == 64) return splits == 2 || G >= 4 || few || wgs <= 512;
  if (splits == 2) return G >= 4 || few || wgs <= 768;
  return G >= 8 ? few || wgs <= 1024 : wgs <= 256;
}

bool attention_short_supported(int dtype, const AttnArgs &a, const AttnSeg *segs, int n) {
  const int splits = short_splits(segs, n);
  if (!mfma_attention(dtype, a.head_dim)) return splits == 1;
  return splits <= SHORT_SPLITS && short_pays(a, splits, segs, n);
}

hipError_t launch_attention_short(int dtype, const AttnArgs &a, const CombineArgs &c, const AttnSeg *segs, int n,
                                  hipStream_t s) {
  if (segs == nullptr || n < 1 || a.row_seq == nullptr || a.n_heads / a.n_kv_heads > 8 ||
      !attention_short_supported(dtype, a, segs, n) || (a.rec_f32 && (n > 1 || !mfma_attention(dtype, a.head_dim))))
    return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (segs[i].M < 1 || segs[i].r0 < 0 || segs[i].n_splits < 1 || segs[i].g0 < 0 || segs[i].n_groups < 1)
      return hipErrorInvalidValue;
  if (!mfma_attention(dtype, a.head_dim))
    return dtype == 1 ? launch_one_t<bf16>(a, c, segs, n, s) : launch_one_t<float>(a, c, segs, n, s);
  const int m = short_splits(segs, n);
  if (a.head_dim == 128) {
    if (m == 1) return launch_short_t<128, 1>(a, c, segs, n, s);
    if (m == 2) return launch_short_t<128, 2>(a, c, segs, n, s);
    return launch_short_t<128, 4>(a, c, segs, n, s);
  }
  if (m == 1) return launch_short_t<64, 1>(a, c, segs, n, s);
  if (m == 2) return launch_short_t<64, 2>(a, c, segs, n, s);
  return launch_short_t<64, 4>(a, c, segs, n, s);
}

}  // namespace dex
