// M-tiled matrix-core GEMM for the prompt prefill on gfx950 (bf16).
//
//   acc[m][n] = sum_k x[m][k] * W[n][k]
//
// Both operands are read in the packed block layout (1 KB per 16 rows x 32 k,
// one MFMA fragment in lane order): the weights as dex_create packs them, the
// activations as the producing kernel wrote them (pk_off).  So every transfer
// is 1 KB of consecutive bytes and a k-step of a 16-row block follows the one
// before it; row-major activations were fetched as sixteen 64-byte halves of
// cache lines per fragment.
//
// gemm_ring_kernel: a workgroup owns BNB weight blocks (16 output columns
// each; a gate/up pair takes two) x BMF input fragments (16 rows each).  The
// stages (KS k-steps of both operands) move global -> LDS with direct
// transfers (global_load_lds, 16 bytes per lane at LDS base + 16 x lane) into
// a ring of NBUF slots, so a workgroup keeps up to (NBUF - 1) stages in
// flight without a staging register, and each wave waits (vmcnt) only for its
// own oldest stage before the per-stage barrier.  A stage's fragments are
// read into registers while the stage before it is multiplied (two register
// sets): with reads and products of one stage back to back, as the first form
// of this kernel had it, the matrix cores idle while all waves read.
//
// Every output element accumulates its k-steps in increasing order from zero
// whatever the tile, so the bits do not depend on which tile was chosen, on
// the number of rows or on the other rows.
//
// The epilogues are those of the decode kernel (RMSNorm row scale, RoPE and
// the key/value cache write; residual add with the next norm's input and its
// sum-of-squares partials; SwiGLU), applied to the accumulators in registers:
// lane (g, r) of a tile holds output columns 4g..4g+3 of input row r, so a
// store to the packed layout puts a tile's 16 rows x 16 columns into 512
// consecutive bytes.  The row scales of a normed GEMM are computed once
// beforehand (row_scale_kernel) rather than by each of its column blocks.
#include "gemm_common.h"

namespace dex {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 tb_bf16x8;
typedef __attribute__((ext_vector_type(4))) float tb_f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int tb_u32x4;

__device__ __forceinline__ uint32_t tb_f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint2 tb_pack4(float a, float b, float c, float d) {
  return make_uint2(tb_f2bf(a) | (tb_f2bf(b) << 16), tb_f2bf(c) | (tb_f2bf(d) << 16));
}

// RMSNorm reciprocal scale of every prompt row, once per normed GEMM: a wave
// per row, with the decode kernels' sum (row_rscale).  The launch is a chain
// of latencies, so a row is one round of loads and a butterfly
// (2 x 1100 rows of 48 partials, 12 layers: 1303 -> 1288 us a prompt; an in-order
// sum staged through LDS took 4.8 us a launch, 97 rows of 256: 656 -> 641 us).
constexpr int RS_ROWS = 4;
__global__ __launch_bounds__(64 * RS_ROWS) void row_scale_kernel(const float *part, int n_part, int M, float inv_d,
                                                                 float eps, float *out) {
  constexpr int NPRE = 4;
  const int m = blockIdx.x * RS_ROWS + threadIdx.x / 64, lane = threadIdx.x & 63;
  if (m >= M) return;
  const float *p = part + (size_t)m * n_part;
  float pre[NPRE];
#pragma unroll
  for (int i = 0; i < NPRE; ++i) pre[i] = lane + 64 * i < n_part ? p[lane + 64 * i] : 0.f;
  const float r = row_rscale<NPRE>(p, n_part, inv_d, eps, lane, pre);
  if (lane == 0) out[m] = r;
}

// Epilogue of one 16 x 16 output tile held by a wave: lane (g, r) holds
// output columns tile*16 + 4g .. +3 of input row m (ok: m < M).  Every lane
// of the wave calls it (the RESID form exchanges values across lanes).
// acc[0] is the tile (SwiGLU: the gate tile, acc[1] the up tile), rsc the
// row's RMSNorm scale.  The QKV epilogue is tb_qkv_block.
template <int EPI, int NT>
__device__ __forceinline__ void tb_epilogue(const GemmArgs &a, int tile, int m, bool ok, const tb_f32x4 (&acc)[NT],
                                            float rsc, int grp) {
  if constexpr (EPI == EPI_PLAIN) {
    if (ok) {
      float *o = a.out + (size_t)m * a.ld_out + tile * 16 + grp * 4;
      *(float4 *)o = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
    }
  } else if constexpr (EPI == EPI_RESID) {
    const int n0 = tile * 16 + grp * 4;
    float hn[4] = {0.f, 0.f, 0.f, 0.f};
    if (ok) {
      float *hp = a.h + (size_t)m * a.ld_h + n0;
      const float4 hv = *(const float4 *)hp;
      hn[0] = hv.x + a.alpha * acc[0][0];
      hn[1] = hv.y + a.alpha * acc[0][1];
      hn[2] = hv.z + a.alpha * acc[0][2];
      hn[3] = hv.w + a.alpha * acc[0][3];
      *(float4 *)hp = make_float4(hn[0], hn[1], hn[2], hn[3]);
      if (a.xb != nullptr) {
        const float *gn = a.g_next + n0;
        *(uint2 *)((uint16_t *)a.xb + pk_off<bf16>(m, n0, a.pk_steps)) =
            tb_pack4(gn[0] * hn[0], gn[1] * hn[1], gn[2] * hn[2], gn[3] * hn[3]);
      }
    }
    // sum of squares over the tile's 16 columns: four per lane, then
    // across the four lane groups that hold the same input row
    float sq = hn[0] * hn[0] + hn[1] * hn[1] + hn[2] * hn[2] + hn[3] * hn[3];
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    if (ok && grp == 0) a.part_out[(size_t)m * a.n_part_out + tile] = sq;
  } else if constexpr (EPI == EPI_SWIGLU) {
    if (ok) {
      float o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gt = acc[0][i] * rsc, up = acc[NT - 1][i] * rsc;
        o[i] = gt / (1.0f + expf(-gt)) * up;
      }
      *(uint2 *)((uint16_t *)a.act + pk_off<bf16>(m, tile * 16 + grp * 4, a.pk_steps)) = tb_pack4(o[0], o[1], o[2], o[3]);
    }
  }
}

// QKV epilogue of the tiles T0 .. T0 + NTL - 1 (consecutive) over NF input
// fragments (lane (g, r) of fragment f: input row mbase + 16 f + r): RMSNorm
// scale, RoPE on the query and key columns (the tile's rows 0..7 hold
// dimensions i of a head, rows 8..15 dimensions i + hd/2: the partner of a
// value sits 32 lanes away), queries to out (fp32), keys and values to the
// cache entry of the row.  The row-table loads, and the RoPE-table loads of
// four tiles at a time, are issued before the stores they feed, so that
// they are not held behind stores to memory the compiler cannot tell apart
// from the tables.
template <int NTL, int NF, typename Acc>
__device__ __forceinline__ void tb_qkv_block(const GemmArgs &a, int T0, int mbase, const float (&rsc)[NF], int r16,
                                             int grp, Acc acc) {
  const int hd = a.head_dim;
  const int nq = a.n_heads * hd, nk = a.n_kv_heads * hd;
  const int n_tiles = (a.N + 15) / 16;
  const bool lo = grp < 2;
  int pos[NF], seq[NF], ent[NF];
  bool ok[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int m = mbase + f * 16 + r16;
    ok[f] = m < a.M;
    const int mm = ok[f] ? m : 0;
    pos[f] = a.row_pos[mm];
    seq[f] = a.row_seq[mm];
    ent[f] = a.row_entry[mm];
  }
  constexpr int CH = NTL < 4 ? NTL : 4;     // tiles per batch of RoPE loads
  static_assert(NTL % CH == 0, "tile batches");
#pragma unroll
  for (int f = 0; f < NF; ++f) {
#pragma unroll
    for (int p0 = 0; p0 < NTL; p0 += CH) {
      float4 cs[CH][2];                        // (cos, sin) of the lane's four pairs
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const int p = p0 + q, tile = T0 + p;
        const int col0 = qkv_col(tile, 0, hd), head_col = col0 - col0 % hd;
        const int i0 = 8 * (tile % (hd / 16)) + (grp & 1) * 4;
        if (tile < n_tiles && head_col < nq + nk) {
          const float4 *rp = (const float4 *)(a.rope + (size_t)pos[f] * (hd / 2) + i0);
          cs[q][0] = rp[0];
          cs[q][1] = rp[1];
        } else {
          cs[q][0] = cs[q][1] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const int p = p0 + q, tile = T0 + p;
        if (tile >= n_tiles) continue;         // uniform across the wave
        const int col0 = qkv_col(tile, 0, hd), head_col = col0 - col0 % hd;
        const int i0 = 8 * (tile % (hd / 16)) + (grp & 1) * 4;
        const tb_f32x4 t = acc(p, f);
        const float c[4] = {cs[q][0].x, cs[q][0].z, cs[q][1].x, cs[q][1].z};
        const float sn[4] = {cs[q][0].y, cs[q][0].w, cs[q][1].y, cs[q][1].w};
        float y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = t[i] * rsc[f];
          const float partner = __shfl_xor(v, 32, 64);
          y[i] = v;
          if (ok[f] && head_col < nq + nk)     // q or k: rotate the pair
            y[i] = lo ? v * c[i] - partner * sn[i] : v * c[i] + partner * sn[i];
        }
        if (!ok[f]) continue;
        const int dim0 = (lo ? 0 : hd / 2) + i0;
        if (head_col < nq) {
          *(float4 *)(a.out + (size_t)(mbase + f * 16 + r16) * a.ld_out + head_col + dim0) =
              make_float4(y[0], y[1], y[2], y[3]);
        } else {
          const bool isk = head_col < nq + nk;
          const int g = (isk ? head_col - nq : head_col - nq - nk) / hd;
          uint16_t *cache = (uint16_t *)(isk ? a.kc : a.vc);
          const size_t base = (((size_t)seq[f] * a.n_kv_heads + g) * a.kv_entries + ent[f]) * hd;
          *(uint2 *)(cache + base + dim0) = tb_pack4(y[0], y[1], y[2], y[3]);
        }
      }
    }
  }
}

#define RING_LDS(p) ((__attribute__((address_space(3))) void *)(p))

// BNB weight blocks x BMF input fragments per workgroup of WN x WM waves,
// stages of KS k-steps, NBUF ring slots.
template <int BNB_, int BMF_, int WN_, int WM_, int KS_, int NBUF_>
struct RingTile {
  static constexpr int BNB = BNB_, BMF = BMF_, WN = WN_, WM = WM_, KS = KS_, NBUF = NBUF_;
  static constexpr int NW = WN * WM, WB = BNB / WN, WF = BMF / WM;
  static constexpr int NBLK = KS * (BNB + BMF);       // 1 KB blocks per stage
  static constexpr int PT = NBLK / NW;                // transfers per wave and stage
  static constexpr int LDS_BYTES = NBUF * NBLK * 1024;
  static_assert(BNB % WN == 0 && BMF % WM == 0 && NBLK % NW == 0 && NBUF >= 2, "ring tile");
  static_assert((NBUF - 1) * PT < 64, "vmcnt field");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// Per-stage barrier with at most `stages` (0 .. NBUF - 1) whole stages of this
// wave's transfers outstanding.
template <typename T, int S = T::NBUF - 1>
__device__ __forceinline__ void ring_wait(int stages) {
  if constexpr (S <= 0) lds_ring_step<0>();
  else if (stages >= S) lds_ring_step<S * T::PT>();
  else ring_wait<T, S - 1>(stages);
}

template <int EPI, typename T>
__global__ __launch_bounds__(64 * T::NW) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_ring_kernel(GemmArgs a, int n_blk_n, int n_wg, int group) {
  constexpr int NT = (EPI == EPI_SWIGLU) ? 2 : 1;     // interleaved gate/up blocks
  constexpr int WB = T::WB, WF = T::WF, KS = T::KS, NBUF = T::NBUF, PT = T::PT;
  constexpr int TPW = T::BNB / NT;                    // output tiles per workgroup
  static_assert(WB % NT == 0, "a wave owns whole gate/up pairs");
  __shared__ __attribute__((aligned(16))) char ring[T::LDS_BYTES];   // [slot][stage block][lane] of 16 bytes

  // Each XCD takes a contiguous run of tiles, `group` input blocks deep, so
  // that the operands its workgroups share stay in its own L2.
  const int xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
  const int base = n_wg / 8, rem = n_wg % 8;
  const int t = xcd * base + min(xcd, rem) + jx;
  const int n_blk_m = n_wg / n_blk_n;
  const int per_group = group * n_blk_n;
  const int g = t / per_group, first_m = g * group;
  const int gsize = min(group, n_blk_m - first_m);
  const int mb = first_m + (t % per_group) % gsize, nb = (t % per_group) / gsize;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, grp = lane >> 4;
  const int wn = wave % T::WN, wm = wave / T::WN;
  const int n_tiles = (a.N + 15) / 16, nsteps = a.nsteps_w;
  const int tile0 = nb * TPW, f0 = mb * T::BMF, n_frag = (a.M + 15) / 16;
  const int nst = (nsteps + KS - 1) / KS;             // stages

  tb_f32x4 acc[WB][WF];
#pragma unroll
  for (int jb = 0; jb < WB; ++jb)
#pragma unroll
    for (int f = 0; f < WF; ++f) acc[jb][f] = tb_f32x4{0.f, 0.f, 0.f, 0.f};

  // this wave's transfers of a stage: block b = wave + NW i is k-step
  // b / (BNB + BMF) of weight block or input fragment b % (BNB + BMF).  Tiles
  // and fragments past the operands read the last one (their outputs are not
  // stored), k-steps past the end the last one too (they are not multiplied).
  auto issue = [&](int st, int slot) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int b = wave + T::NW * i, j = b % (T::BNB + T::BMF);
      const int step = KS == 1 ? st : min(st * KS + b / (T::BNB + T::BMF), nsteps - 1);
      size_t off;
      const char *p;
      if (j < T::BNB) {
        off = (((size_t)min(tile0 + j / NT, n_tiles - 1) * nsteps + step) * NT + j % NT) * 1024;
        p = (const char *)a.wp;
      } else {
        off = ((size_t)min(f0 + j - T::BNB, n_frag - 1) * nsteps + step) * 1024;
        p = (const char *)a.x;
      }
      __builtin_amdgcn_global_load_lds((const void *)(p + off + lane * 16),
                                       RING_LDS(ring + ((size_t)slot * T::NBLK + b) * 1024), 16, 0, 0);
    }
  };
  struct Set {
    tb_u32x4 w[KS][WB], x[KS][WF];
  };
  auto fetch = [&](int slot, Set &s) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const tb_u32x4 *blk = (const tb_u32x4 *)(ring + ((size_t)slot * T::NBLK + k * (T::BNB + T::BMF)) * 1024) + lane;
#pragma unroll
      for (int f = 0; f < WF; ++f) s.x[k][f] = blk[(T::BNB + wm * WF + f) * 64];
#pragma unroll
      for (int jb = 0; jb < WB; ++jb) s.w[k][jb] = blk[(wn * WB + jb) * 64];
    }
  };
  auto mma = [&](int k, const Set &s) {
#pragma unroll
    for (int jb = 0; jb < WB; ++jb)
#pragma unroll
      for (int f = 0; f < WF; ++f)
        acc[jb][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(tb_bf16x8, s.w[k][jb]),
                                                             __builtin_bit_cast(tb_bf16x8, s.x[k][f]), acc[jb][f], 0, 0, 0);
  };
  // One DS read per PER products, so that the reads of the next stage spread
  // over this stage's products.
  constexpr int READS = KS * (WB + WF), PRODS = KS * WB * WF, PER = PRODS / READS > 0 ? PRODS / READS : 1;
  auto interleave = [&]() {
    __builtin_amdgcn_sched_group_barrier(0x020, PT, 0);         // transfers first
#pragma unroll
    for (int i = 0; i < READS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
    }
  };

  // stages 0 .. NBUF - 1 in flight; stage 0 landed, its fragments requested
  for (int s = 0; s < NBUF && s < nst; ++s) issue(s, s);
  ring_wait<T>(min(nst, NBUF) - 1);
  Set A, B;
  fetch(0, A);
  // Iteration st: stage st + 1 has landed for every wave and every wave holds
  // stage st in registers, whose slot therefore takes stage st + NBUF; stage
  // st + 1 is read while stage st is multiplied.
  int st = 0, slot = 0;                                 // slot of stage st
  auto full = [&](const Set &cur, Set &nxt) {           // st + NBUF < nst
    lds_ring_step<(NBUF - 2) * PT>();
    issue(st + NBUF, slot);
    slot = slot + 1 == NBUF ? 0 : slot + 1;
    fetch(slot, nxt);
#pragma unroll
    for (int k = 0; k < KS; ++k) mma(k, cur);
    interleave();
    ++st;
  };
  while (st + NBUF + 1 < nst) {
    full(A, B);
    full(B, A);
  }
  // the last stages: little or nothing left to request
  auto tail = [&](const Set &cur, Set &nxt) {
    if (st + 1 < nst) {
      ring_wait<T>(min(nst - 2 - st, NBUF - 2));
      if (st + NBUF < nst) issue(st + NBUF, slot);
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      fetch(slot, nxt);
    }
#pragma unroll
    for (int k = 0; k < KS; ++k)
      if (KS == 1 || st * KS + k < nsteps) mma(k, cur);
    ++st;
  };
  while (st < nst) {
    tail(A, B);
    if (st >= nst) break;
    tail(B, A);
  }

  float rsc[WF];
#pragma unroll
  for (int f = 0; f < WF; ++f) {
    const int m = (f0 + wm * WF + f) * 16 + r16;
    rsc[f] = (a.row_rsc != nullptr && m < a.M) ? a.row_rsc[m] : 1.f;
  }
  if constexpr (EPI == EPI_QKV) {
    tb_qkv_block<WB, WF>(a, tile0 + wn * WB, (f0 + wm * WF) * 16, rsc, r16, grp, [&](int p, int f) { return acc[p][f]; });
  } else {
#pragma unroll
    for (int p = 0; p < WB / NT; ++p) {
      const int tile = tile0 + wn * (WB / NT) + p;
      if (tile >= n_tiles) continue;          // uniform across the wave
#pragma unroll
      for (int f = 0; f < WF; ++f) {
        const int m = (f0 + wm * WF + f) * 16 + r16;
        tb_f32x4 at[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) at[nt] = acc[p * NT + nt][f];
        tb_epilogue<EPI, NT>(a, tile, m, m < a.M, at, rsc[f], grp);
      }
    }
  }
}

}  // namespace

bool gemm_tiled_supported(int epi, const GemmArgs &a) {
  if (a.M < 1 || a.N < 1 || a.nsteps_w < 1 || a.row_bnd != nullptr || a.row0 != 0 || a.rm) return false;
  if (a.part != nullptr && a.row_rsc == nullptr) return false;   // the row scales come precomputed
  if ((a.M + 127) / 128 > 65535) return false;
  switch (epi) {
    case EPI_PLAIN: return a.N % 16 == 0 && a.ld_out % 4 == 0;
    case EPI_QKV: return a.ld_out % 4 == 0 && a.head_dim % 16 == 0;
    case EPI_RESID: return a.N % 16 == 0 && a.ld_h % 4 == 0;
    case EPI_SWIGLU: return true;
    default: return false;
  }
}

hipError_t launch_row_scale(const float *part, int n_part, int M, float inv_d, float eps, float *out, hipStream_t s) {
  if (part == nullptr || out == nullptr || n_part < 1 || M < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(row_scale_kernel, dim3((unsigned)((M + RS_ROWS - 1) / RS_ROWS)), dim3(64 * RS_ROWS), 0, s, part, n_part, M,
                     inv_d, eps, out);
  return hipGetLastError();
}

template <int EPI, typename T>
static hipError_t launch_ring(const GemmArgs &a, hipStream_t s) {
  constexpr int GROUP = 2048 / (16 * T::BMF);          // rows of a tile group: 2048
  const int tpw = T::BNB / (EPI == EPI_SWIGLU ? 2 : 1);
  const int n_blk_n = ((a.N + 15) / 16 + tpw - 1) / tpw, n_blk_m = ((a.M + 15) / 16 + T::BMF - 1) / T::BMF;
  const long long n_wg = (long long)n_blk_n * n_blk_m;
  if (n_wg > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_ring_kernel<EPI, T>), dim3((unsigned)n_wg), dim3(64 * T::NW), 0, s, a, n_blk_n, (int)n_wg,
                     GROUP);
  return hipGetLastError();
}

// The tiles, largest first, and what they cost: workgroups a compute unit
// holds, a k-step of one workgroup alone (us), how much each further resident
// one adds to it (share), the fixed part of a round (first loads) and of the
// epilogue (QKV, RESID and PLAIN, SWIGLU).  The transfers of operands into LDS
// bound every tile but the largest: by these costs they all bring 64 to 76 GB/s
// into a compute unit, while the counters see the matrix cores busy 8 to 22 %
// of the time, LDS reads 7 to 16 % and no bank conflicts (97 and 512 rows of
// 4096-wide layers, 2200 of 768-wide).  So a larger tile costs less per
// output, and small ones pay where a grid of large ones leaves compute units
// idle.  The 256 x 256 tile has its matrix cores busy 51 to 57 % of the time at
// 8192 rows, LDS reads 21 %, at a clock of about 2.1 GHz.  The constants are a least
// squares fit to measured launches, all four projections of 4096, 2048 and
// 768 wide layers at 65 to 8192 rows; the tile of the least estimated time is
// on average 2 %, at most 16 %, slower than the best of them (whole rounds of
// one workgroup per compute unit, the first form of this rule: 7 and 53 %).
// For instance (us): 4096 x 14336, 97 / 512 / 2200 / 8192 rows: 45 (32 x 64),
// 103 (64 x 128), 286 and 777 (256 x 256, 1.24 PFLOP/s).
typedef RingTile<16, 16, 4, 2, 1, 5> Tile256x256;
typedef RingTile<16, 8, 2, 2, 1, 3> Tile256x128;
typedef RingTile<8, 8, 2, 2, 1, 5> Tile128x128;       // five slots: two resident
typedef RingTile<8, 8, 2, 2, 1, 3> Tile128x128r3;     // three slots: three resident
typedef RingTile<4, 8, 2, 2, 1, 4> Tile64x128;
typedef RingTile<4, 4, 1, 4, 2, 4> Tile64x64;
typedef RingTile<2, 4, 1, 4, 4, 5> Tile32x64;
struct TileCost {
  int blocks, frags, resident;  // weight blocks x input fragments; workgroups per compute unit
  float step, more, fixed, epi[3];
};
static const TileCost kTileCost[] = {
    {16, 16, 1, 0.598f, 0.00f, 13.6f, {13.7f, 7.7f, 1.8f}}, {16, 8, 2, 0.407f, 0.94f, 12.4f, {7.9f, 5.4f, 0.0f}},
    {8, 8, 2, 0.236f, 0.96f, 8.1f, {3.5f, 2.5f, 0.0f}},     {8, 8, 3, 0.316f, 0.60f, 5.8f, {4.3f, 1.9f, 0.0f}},
    {4, 8, 3, 0.198f, 0.69f, 4.1f, {2.2f, 1.2f, 0.0f}},     {4, 4, 2, 0.121f, 0.85f, 3.4f, {0.6f, 1.1f, 0.0f}},
    {2, 4, 1, 0.094f, 0.55f, 2.2f, {1.0f, 1.4f, 0.7f}}};

static int choose_tile(int epi, int n_blocks, int n_frag, int nsteps) {
  const int ei = epi == EPI_QKV ? 0 : epi == EPI_SWIGLU ? 2 : 1;
  int best = 0;
  double best_us = 0.0;
  for (int i = 0; i < (int)(sizeof(kTileCost) / sizeof(kTileCost[0])); ++i) {
    const TileCost &c = kTileCost[i];
    const long long n_wg = (long long)((n_blocks + c.blocks - 1) / c.blocks) * ((n_frag + c.frags - 1) / c.frags);
    auto round_us = [&](int resident) {
      const double share = 1.0 + (resident - 1) * (double)c.more;
      return share * (nsteps * (double)c.step + c.epi[ei]) + c.fixed;
    };
    const long long per_round = 256LL * c.resident, rounds = n_wg / per_round, rest = n_wg % per_round;
    const double us = rounds * round_us(c.resident) + (rest > 0 ? round_us((int)((rest + 255) / 256)) : 0.0);
    if (i == 0 || us < best_us) { best = i; best_us = us; }
  }
  return best;
}

template <int EPI>
static hipError_t launch_tile(const GemmArgs &a, hipStream_t s) {
  switch (choose_tile(EPI, (a.N + 15) / 16 * (EPI == EPI_SWIGLU ? 2 : 1), (a.M + 15) / 16, a.nsteps_w)) {
    case 0: return launch_ring<EPI, Tile256x256>(a, s);
    case 1: return launch_ring<EPI, Tile256x128>(a, s);
    case 2: return launch_ring<EPI, Tile128x128>(a, s);
    case 3: return launch_ring<EPI, Tile128x128r3>(a, s);
    case 4: return launch_ring<EPI, Tile64x128>(a, s);
    case 5: return launch_ring<EPI, Tile64x64>(a, s);
    default: return launch_ring<EPI, Tile32x64>(a, s);
  }
}

hipError_t launch_gemm_tiled(int epi, const GemmArgs &a, hipStream_t s) {
  if (!gemm_tiled_supported(epi, a)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_PLAIN: return launch_tile<EPI_PLAIN>(a, s);
    case EPI_QKV: return launch_tile<EPI_QKV>(a, s);
    case EPI_RESID: return launch_tile<EPI_RESID>(a, s);
    case EPI_SWIGLU: return launch_tile<EPI_SWIGLU>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dex
