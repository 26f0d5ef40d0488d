// Internal declarations shared by the HIP kernels and the host engine.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dex {

// Output column of local tile row r16 (0..15) of QKV tile `tile`: a tile keeps
// the two RoPE partners (i, i + hd/2) of one head together -- rows 0..7 are
// dims 8j..8j+7 and rows 8..15 dims hd/2+8j.. of head tile/(hd/16), j the
// tile's index inside the head.  Shared by weight packing and the epilogues.
__device__ __forceinline__ int qkv_col(int tile, int r16, int hd) {
  const int tph = hd / 16;                 // tiles per head
  const int head = tile / tph, j = tile % tph;
  const int dim = (r16 < 8) ? (8 * j + r16) : (hd / 2 + 8 * j + r16 - 8);
  return head * hd + dim;
}

typedef uint16_t bf16;

// Element offset of (row m, column k) in the packed block layout of `steps`
// k-steps per 16-row block: block (m / 16, k-step) is 1 KB, one matrix-core
// fragment in lane order -- with EPB elements in 16 bytes and 4 EPB columns a
// k-step, 16 bytes of row m % 16, column group (k % 4 EPB) / EPB at lane
// 16 group + m % 16.  Weights and every activation that a GEMM reads are laid
// out so: a fragment is then 1 KB of consecutive bytes, where 16 row-major
// rows are sixteen 64-byte pieces that cost the vector L1 an access per lane
// (64 against 18 per instruction, counted at 64 rows).
template <typename T>
__host__ __device__ __forceinline__ size_t pk_off(int m, int k, int steps) {
  constexpr int EPB = 16 / (int)sizeof(T), KSTEP = 4 * EPB;
  return ((size_t)(m >> 4) * steps + k / KSTEP) * (16 * KSTEP) + (k % KSTEP) / EPB * (16 * EPB) + (m & 15) * EPB +
         k % EPB;
}

// The same element in an activation buffer of either layout: a few rows (rm)
// lie row-major in the same blocks' bytes, rows of `steps` k-steps.  One or
// two rows of a fragment are a sixteenth or an eighth of its lanes, and in
// lane order 64 bytes of a row lie 256 bytes apart (one row: QKV 11.2 against
// 11.7 us, down 19.7 against 19.9; equal at four, 22.1 against 20.1 at eight).
template <typename T>
__host__ __device__ __forceinline__ size_t act_off(int m, int k, int steps, int rm) {
  constexpr int KSTEP = 64 / (int)sizeof(T);
  return rm ? (size_t)m * steps * KSTEP + k : pk_off<T>(m, k, steps);
}

// Step of an LDS ring filled by direct global -> LDS transfers
// (global_load_lds): wait until this wave's transfers are done but for the
// youngest VMCNT ones and its LDS reads have all returned, then meet the
// workgroup's other waves.  Unlike __syncthreads() it leaves the younger
// transfers in flight.  The empty asm statements and the scheduling barriers
// emit nothing; they keep the compiler from moving anything across the wait
// and the barrier.
template <int VMCNT>
__device__ __forceinline__ void lds_ring_step() {
  static_assert(VMCNT >= 0 && VMCNT < 64, "vmcnt field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0070 | (VMCNT & 15) | ((VMCNT >> 4) << 14));   // lgkmcnt 0, expcnt: no wait
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// Sampling-mode Gumbel noise of token v for the slot of sequence `seq` at
// position `pos` (the definition is stated with dex_debug_gumbel in dex.h).
__device__ __forceinline__ unsigned long long sm64_mix(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ unsigned long long gumbel_key(unsigned long long seed, int seq, int pos) {
  return sm64_mix(seed ^ sm64_mix(((unsigned long long)(unsigned)seq << 32) + (unsigned long long)(unsigned)pos));
}
__device__ __forceinline__ float gumbel_noise(unsigned long long key, int v) {
  const unsigned long long z = sm64_mix(key + (unsigned long long)(v + 1) * 0x9E3779B97F4A7C15ull);
  const float u = ((float)(unsigned)(z >> 41) + 0.5f) * (1.0f / 8388608.0f);
  return -logf(-logf(u));
}

// ---------------------------------------------------------------- epilogues
enum Epi {
  EPI_PLAIN = 0,   // y[m][n] (float)
  EPI_QKV = 1,     // rms-scaled, RoPE on q/k, q -> float buffer, k/v -> cache
  EPI_RESID = 2,   // h += alpha * y; next-norm input and sum-of-squares partials
  EPI_SWIGLU = 3,  // rms-scaled gate/up pair -> SiLU(gate) * up
  EPI_LOGITS = 4,  // rms-scaled LM head, DECS mask, per-tile argmax
  EPI_BIAS_SILU = 5,  // SiLU(rms-scaled y + bias) -> act (adapter up-projection)
};

constexpr int GEMM_WAVES = 8;       // split-K ways inside a workgroup
constexpr int GEMM_THREADS = GEMM_WAVES * 64;
constexpr int ATT_SPLIT = 64;       // logical keys per attention split (one wave)
constexpr int ATT_THREADS = 64;
constexpr int ATT_MAX_PAIRS = 64;   // (row, query head) pairs per attention row group
constexpr int ATT_MAX_SPLITS = 4096; // longest context: 262144 positions

struct GemmArgs {
  // Weights in the packed block layout (see PackArgs); nsteps_w k-steps per tile.
  const void *wp;
  int nsteps_w;
  int N;          // output columns (SWIGLU: d_ffn)
  int K;
  const void *x;  // activations [M][K], packed (pk_off, nsteps_w k-steps)
  int row0;       // row 0's row in x, xb and act
  int rm;         // x, xb and act hold their rows row-major (act_off)
  int M;
  // RMSNorm scale from sum-of-squares partials (nullable): per row
  // 1/sqrt(sum(part[m][0..n_part)) * inv_d + eps).
  const float *part;
  int n_part;
  float inv_d, eps;
  // Prompt GEMMs (launch_gemm_tiled): the same scales precomputed per row by
  // launch_row_scale, required there whenever part is set.
  const float *row_rsc;
  // PLAIN / QKV: float output [M][ld_out]
  float *out;
  int ld_out;
  // QKV
  void *kc, *vc;              // this layer's cache base ([B][Hkv][E][hd])
  int kv_entries;             // E
  int n_heads, n_kv_heads, head_dim;
  const int *row_seq, *row_pos, *row_entry;
  const float2 *rope;         // [max_ctx][hd/2] (cos, sin)
  // RESID
  float *h;                   // [M][ld_h] residual stream (in place)
  int ld_h;
  float alpha;
  const float *g_next;        // gain of the next RMSNorm (nullable)
  void *xb;                   // next-norm input g*h (T), packed with pk_steps (nullable)
  float *part_out;            // [M][n_part_out]
  int n_part_out;
  const int *row_bnd;         // nullable: write h/partials to boundary storage instead
  float *bnd_h, *bnd_part;
  // with row_bnd (nullable): the exit head's input, final norm gain ex_g, and
  // partials of the same rows, rows ex_row0 .. of its buffers
  void *ex_xb;
  float *ex_part;
  const float *ex_g;
  int ex_row0, ex_rm;
  const float *bias;          // RESID (nullable): h += alpha * (y + bias); BIAS_SILU: SiLU(y + bias)
  // SWIGLU / BIAS_SILU
  void *act;                  // [M][N] (T), packed with pk_steps
  int pk_steps;               // k-steps of the packed output (xb or act)
  // LOGITS
  const int *mask_tok;        // [M][mask_stride]
  const int *mask_n;          // [M]
  int mask_stride;
  float *logits_tap;          // nullable [M][N]
  float2 *amax;               // [M][n_tiles] (value, index as float bits)
  int n_tiles;
  float temperature;          // > 0: Gumbel-max sampling with the rows of (sample_seed, row_seq, row_pos)
  unsigned long long sample_seed;
};

// Split partials of R rows live in one buffer of R * H * jmax * (hd + 2)
// floats: the split outputs o in the cache's element type ([R][H][jmax][hd],
// filling at most the first R * H * jmax * hd floats), then the statistics
// ([R][H][jmax] of float (max, sum)) at float offset R * H * jmax * hd.
inline float *split_stats(float *part, size_t rows, int n_heads, int jmax, int hd) {
  return part + rows * n_heads * jmax * hd;
}

struct AttnArgs {
  const float *q;             // [R][H*hd], RoPE applied
  int ldq;
  const void *kc, *vc;        // this layer's cache base
  int kv_entries, n_kv_heads, n_heads, head_dim, batch;
  // row groups: consecutive rows of one sequence that share their committed
  // prefix; grp_nc (nullable) is that prefix's length
  const int *grp_row0, *grp_nrows, *grp_seq, *grp_nc;
  const int *row_pos, *row_nc, *row_chain_off, *chain;
  const int *row_seq;         // sequence of each row (matrix-core kernel)
  int n_rows;                 // rows of the launch (matrix-core kernel)
  void *part;                 // [R][H][jmax][hd] split outputs o (element type of the cache, or float)
  float *stat;                // [R][H][jmax][2] their (max, sum)
  int jmax;                   // split stride of `part` and `stat`
  int n_splits;               // splits the launch covers: max over its rows of pos / 64 + 1 (<= jmax)
  float scale;
  int rec_f32;                // matrix-core kernels: float records (plain launches only)
};

struct CombineArgs {
  const void *part;           // as AttnArgs
  const float *stat;
  const int *row_pos;
  int jmax, n_heads, head_dim;
  int rec_f32;                // as AttnArgs
  void *out;                  // [R][H*hd] (T): an activation buffer of out_steps k-steps,
  int ld_out;                 // or rows ld_out apart where out_steps is 0
  int out_steps;
  int row0, rm;               // row r's row and layout there, or from row_pk[r] where set:
  const int *row_pk;          // the row, or ~row for a row-major one
};

// Grouped launches.  The stages of a round are independent and, taken in
// step, all run their j-th layer at the same time: one launch then covers
// that layer step of every stage (a segment each), each segment on its own
// rows of the launch's row space with its own layer's weights and cache.  A
// segment's rows go through exactly the arithmetic of a launch of their own
// (segments never share a workgroup), so grouping changes no result bit.
// A launch takes at most MAX_SEGS segments in its arguments (longer lists go
// out as several launches), and a single segment goes out as a plain launch
// of the same rows: the arguments stay small, which keeps the launch cost of
// short kernels down.
constexpr int MAX_SEGS = 8;

struct GemmSeg {
  const void *wp;             // the segment's layer weights (packed)
  void *kc, *vc;              // QKV: the layer's key/value cache base
  const float *g_next;        // RESID: the next RMSNorm's gain (nullptr: none)
  const int *row_bnd;         // RESID: boundary rows of the segment (nullable)
  float alpha;                // RESID: the layer's residual scale
  int r0, M;                  // rows [r0, r0 + M) of the launch's buffers
  int p0, rm;                 // row0 and rm of its activations (see GemmArgs)
};
struct GemmSegs {
  int n;
  GemmSeg s[MAX_SEGS];
};

// The arguments of segment s alone: its weights and layer, and the
// row-indexed buffers and tables advanced to its first row.
template <typename T, int EPI>
__host__ __device__ inline void gemm_seg_view(GemmArgs &a, const GemmSeg &s) {
  static_assert(EPI == EPI_QKV || EPI == EPI_RESID || EPI == EPI_SWIGLU, "grouped epilogues");
  const size_t r = (size_t)s.r0;
  a.wp = s.wp;
  a.M = s.M;
  a.row0 = s.p0;
  a.rm = s.rm;
  if (a.part != nullptr) a.part += r * a.n_part;
  if constexpr (EPI == EPI_QKV) {
    a.out += r * a.ld_out;
    a.kc = s.kc;
    a.vc = s.vc;
    a.row_seq += r;
    a.row_pos += r;
    a.row_entry += r;
  } else if constexpr (EPI == EPI_RESID) {
    a.h += r * a.ld_h;
    a.alpha = s.alpha;
    a.g_next = s.g_next;
    if (s.g_next == nullptr) a.xb = nullptr;
    a.part_out += r * a.n_part_out;
    a.row_bnd = s.row_bnd;
    a.ex_row0 = s.r0;
    if (s.row_bnd == nullptr) a.ex_xb = nullptr;
  }
}

struct AttnSeg {
  const void *kc, *vc;        // the segment's layer of the cache
  int r0, M;                  // its rows [r0, r0 + M) of the queries and row tables
  int g0, n_groups;           // its row groups [g0, g0 + n_groups) (row0 relative to r0)
  int n_splits;               // 64-key splits up to its deepest row
};
struct AttnSegs {
  int n;
  int item0[MAX_SEGS];        // first work item of each segment (set by the launcher)
  AttnSeg s[MAX_SEGS];
};

// Causal prompt attention on the matrix cores (bf16 keys/values, head_dim 64
// or 128): rows are (sequence, position) in order, keys are the committed
// cache entries 0..position.
struct PrefillAttnArgs {
  const float *q;             // [batch * prompt_len][ldq], RoPE applied
  int ldq;
  const void *kc, *vc;        // this layer's cache base
  int kv_entries, n_kv_heads, n_heads, head_dim, batch, prompt_len;
  float scale;
  void *out;                  // [batch * prompt_len] rows (bf16), packed
  int out_steps;              // with this many k-steps
};
hipError_t launch_prefill_attention(const PrefillAttnArgs &a, hipStream_t s);

// Weight packing.  mode 0: rows in order; 1: QKV, the three segments w0/w1/w2
// concatenated with each tile holding RoPE partner dimensions (i, i + hd/2)
// of one head; 2: gate (w0) and up (w1) blocks interleaved per step.
struct PackArgs {
  const void *w0, *w1, *w2;
  int n0, n1, n2;
  int N, K, mode, head_dim;
  void *out;
  int nsteps;     // filled by launch_pack
};
size_t packed_bytes(int dtype, int N, int K, int mode);
hipError_t launch_pack(int dtype, const PackArgs &a, hipStream_t s);

// Launchers (return the HIP status of the launch).
hipError_t launch_gemm(int dtype, int epi, const GemmArgs &a, int m_blocks, hipStream_t s);
// Prompt-prefill GEMM (bf16, M-tiled) with the QKV / RESID / SWIGLU / PLAIN
// epilogues.  x ends in zeros past K up to the k-step; N a multiple of 16
// except for SWIGLU, no boundary rows, row0 0 (gemm_tiled_supported);
// launch_gemm_tiled returns hipErrorInvalidValue otherwise.  A normed GEMM
// takes its row scales from row_rsc.
bool gemm_tiled_supported(int epi, const GemmArgs &a);
hipError_t launch_gemm_tiled(int epi, const GemmArgs &a, hipStream_t s);
// out[m] = 1 / sqrt(sum(part[m][0..n_part)) * inv_d + eps), m < M: the RMSNorm
// scales launch_gemm_tiled reads, summed as the decode kernels sum them.
hipError_t launch_row_scale(const float *part, int n_part, int M, float inv_d, float eps, float *out, hipStream_t s);
hipError_t launch_attention(int dtype, const AttnArgs &a, int n_groups, hipStream_t s);
hipError_t launch_combine(int dtype, const CombineArgs &a, int rows, hipStream_t s);
// Grouped forms (QKV, RESID and SWIGLU epilogues; the decode attention):
// `a` holds what the segments share, with the row-indexed buffers and tables
// at row 0 of the launch.  The attention's split records then use the row
// space of the launch: part [rows][H][jmax][hd], stat at split_stats(part,
// rows, ...), where rows covers every segment.
hipError_t launch_gemm_seg(int dtype, int epi, const GemmArgs &a, const GemmSeg *segs, int n, hipStream_t s);
hipError_t launch_attention_seg(int dtype, const AttnArgs &a, const AttnSeg *segs, int n, hipStream_t s);
// Attention and combine of short rows in one launch (every segment at most
// SHORT_SPLITS splits on the matrix cores, and few enough rows; one in the
// vector kernel): rows, queries, row tables and c's output rows are all
// indexed by the launch's row space.
constexpr int SHORT_SPLITS = 4;
bool attention_short_supported(int dtype, const AttnArgs &a, const AttnSeg *segs, int n);
hipError_t launch_attention_short(int dtype, const AttnArgs &a, const CombineArgs &c, const AttnSeg *segs, int n,
                                  hipStream_t s);

struct PrepArgs {
  int M, d, n_part;
  int embed_rows;             // rows [0, embed_rows): h = E[token]; the others h = boundary[src]
  const int *row_tok;         // embed token per row
  const int *row_src;         // boundary index per row
  const void *embed;
  const float *bnd_h, *bnd_part;
  const float *g;             // gain of the first RMSNorm the rows meet
  // n_seg > 0: segments of consecutive rows (one per stage of a grouped
  // lane), rows [seg_end[k-1], seg_end[k]) meeting gain seg_g[k] instead of g
  int n_seg;
  int seg_end[MAX_SEGS];
  const float *seg_g[MAX_SEGS];
  float *h, *part;            // [M][d], [M][n_part]
  void *xb;                   // [M][d] (T), an activation buffer of xb_steps k-steps
  int xb_steps;
  int row0, rm;               // row m's row and layout there, or row_pk[m] where set (as CombineArgs)
  const int *row_pk;
  const int *row_out;         // nullable: write h/part to row_out[m] instead of m
};
hipError_t launch_prep(int dtype, const PrepArgs &a, hipStream_t s);

struct ArgmaxArgs {
  const float2 *amax;
  int n_tiles, M;
  int *u_out;                 // [M], in host memory, as commit_out: stored past the caches
  int *cand;                  // [..][N] candidate table (nullable)
  const int *row_cand;        // [M] index into cand (slot*N + stage)
  // verify/commit of the rows that complete an anchor's final stage
  // (nullable): row_commit[m] = i >= 0 writes (token, k*) to commit_out[2i..]
  const int *row_commit;
  int N;
  int *commit_out;
};
hipError_t launch_argmax(const ArgmaxArgs &a, hipStream_t s);

struct CollapseArgs {
  int n_jobs;
  const int *job;             // [n_jobs][6] in pinned host memory: seq, src entry, dst entry, src slot, dst slot, kind (0 kv only, 1 kv + slot state)
  int *job_dev;               // room for them on the device
  void *kc, *vc;              // cache base
  int n_layers, batch, n_kv_heads, kv_entries, head_dim;
  int elem_bytes;
  float *bnd_h, *bnd_part;    // [B][2S][d], [B][2S][n_part]
  int *cand;                  // [B][2S][N]
  int slots2, d, n_part, N, max_ctx, S;
};
hipError_t launch_collapse(const CollapseArgs &a, hipStream_t s);

// n ints from pageable host memory to the device, in stream order; src is free
// to be reused at once.
hipError_t launch_upload(int *dst, const int *src, size_t n, hipStream_t s);

hipError_t launch_gumbel(unsigned long long seed, int seq, int pos, int V, float *out, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, int64_t bytes, hipStream_t s);

}  // namespace dex
