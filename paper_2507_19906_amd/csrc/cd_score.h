// Observation-window scoring of the eviction strategy f (Alg. 1 step 3, SnapKV-style,
// Sec. 4.1.3): S = Q_win K^T on the matrix cores in two passes over K.
//   pass 1 (score_rowstats): per window-query row, max and sum of exp2 of its logits over the
//           keys of one chunk; the chunks are merged into a row log-sum-exp, in small calls by the
//           workgroups of pass 2, else by rowstats_merge.
//   pass 2 (score_votes):    S recomputed, p = exp2(s - lse_row), column sums over the G*w
//           rows of the KV head -> vote[j] for prefix columns j < P.
// A workgroup owns a block of query rows (128, or 256 when the KV head has more than 128 - so that
// such heads stream their keys once per pass, not once per 128 rows) and a chunk of keys; its waves
// own 32 rows each and share the key tiles through LDS.  Pass 1 forms S^T = K Q^T (a lane owns
// one query row per tile: running row statistics stay in registers); pass 2 forms S = Q K^T (a
// lane owns one key: the column sum over rows is an in-lane sum plus a 4-lane tree).
#pragma once
#include "cd_common.h"

#include <type_traits>

namespace cd {

constexpr int kRowBlock = 128;     // query rows per workgroup, doubled for KV heads with more than 128 window rows
constexpr int kRowTiles = 2;       // 16-row tiles of query rows per wave
constexpr int kMaxCalHeads = 8;    // largest GQA group whose calibration logits the vote pass exports
constexpr int kChunkUnit = 64;      // keys per workgroup in the scoring passes: a multiple of this

struct ScoreArgs {
  const void* q_win;
  const void* k;
  const int32_t* seq_off;
  int64_t total_tokens;
  int batch, Hq, Hkv, G, w, B, R, NRB, NCH, max_seq_len;
  int RB;               // window-query rows per row block: 128, or 256 when a KV head has more than 128 (R = G*w)
  int row_stride;       // rows per KV head in rowpart / row_lse: NRB * RB
  int chunk_keys;       // keys per workgroup (multiple of 64); every wave reads all of them for query rows of its own
  float sl2;            // scale * log2(e)
  int keep_k;           // pass 1 leaves K in the last-level cache for pass 2 (K of the whole call fits it)
  float2* rowpart;      // [batch*Hkv][NCH][row_stride] (max, sum) per chunk
  float* row_lse;       // [batch*Hkv][row_stride] log2-domain row log-sum-exp (+inf for padding rows)
  int rows_merged;      // pass 2 finds row_lse complete; otherwise its workgroups merge the partials (or take win_lse) themselves
  const float* win_lse; // [batch][Hq][w] natural-log row log-sum-exp from the caller instead of pass 1, or NULL
  float* vote;          // [NRB][plane]: one plane of votes per row block, each packed like K with one float per row
  int64_t plane;        // floats per plane: total_tokens*Hkv rounded up to a multiple of 64 (planes stay 256-byte aligned)
  float* cal_logit;     // [batch*Hq][zstride] log2-unit logits of the last window query, or NULL
  int zstride;
  uint32_t* zero_words; // words to clear for the selection that follows (its histograms), or NULL
  int64_t zero_count;
};

// Clears `count` words with the threads of the whole grid (a kernel ahead of the selection does this on the side).
__device__ __forceinline__ void clear_words(uint32_t* words, int64_t count) {
  if (!words) return;
  const int64_t nblk = static_cast<int64_t>(gridDim.x) * gridDim.y;
  const int64_t me = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
  for (int64_t t = me; t < count; t += nblk * blockDim.x) words[t] = 0u;
}

// Length of sequence b as the kernels use it: 0 when the offsets break the host-side contract
// (so nothing out of bounds is ever touched).
__device__ __forceinline__ int seq_len_checked(const int32_t* seq_off, int b, int max_seq_len,
                                               int64_t total_tokens, int& off0) {
  off0 = seq_off[b];
  int off1 = seq_off[b + 1];
  int n = off1 - off0;
  if (off0 < 0 || n < 0 || n > max_seq_len || static_cast<int64_t>(off1) > total_tokens) return 0;
  return n;
}

// Layout of a stage of keys in LDS, shared by the waves of a workgroup (which own different query
// rows and all read every key tile from LDS instead of each loading it from memory).  LDS rows
// are 16-byte chunks stored at chunk' = chunk ^ swz(key), chosen so that 16 consecutive lanes
// always touch 16 different 16-byte bank groups of a 256-byte window, both for row-wise writes
// (lanes = consecutive chunks) and for the column-wise fragment reads (lanes = consecutive keys).
template <typename T, int D, int NT = 256>
struct KeyStream {
  static constexpr int EPL = Elem<T>::kPer16B;
  static constexpr int KD = Elem<T>::kStepK;
  static constexpr int NK = D / KD;
  static constexpr int kStageKeys = sizeof(T) == 2 ? 64 : 32;
  static constexpr int KT = kStageKeys / 16;                       // key tiles per stage
  static constexpr int CH = D * static_cast<int>(sizeof(T)) / 16;  // 16-byte chunks per key row
  static constexpr int NLD = kStageKeys * CH / NT;                 // loads per thread per stage
  static constexpr int kStageBytes = kStageKeys * CH * 16;
  static_assert(CH == 8 || CH == 16 || CH == 32, "row size not covered by the LDS swizzle");
  __device__ __forceinline__ static int swz(int key) { return CH == 8 ? ((key >> 1) & 7) : (key & 15); }

  // fragment of key tile kt for mma step kk: lane (i, c) gets key 16 kt + i, chunk 4 kk + c.  The swizzle of a
  // key depends on its position inside its tile only, so a lane needs NK byte offsets for the whole
  // stream; the tile is an immediate of the LDS read.
  struct Frags {
    uint32_t off[NK];
    __device__ __forceinline__ void init(int i, int c) {
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) off[kk] = i * (CH * 16) + (((4 * kk + c) ^ swz(i)) * 16);
    }
    __device__ __forceinline__ u32x4 get(const char* lds, int kt, int kk) const {
      return ld16(lds + off[kk] + kt * (16 * CH * 16));
    }
  };
};

// The same stage layout filled by LDS-direct loads: every lane fetches the 16-byte chunk that
// belongs in "its" LDS slot (slot = threadIdx.x + NT u, in the swizzled order above) and the
// load unit writes it there, so the stage needs no staging registers and no LDS store
// instructions.  A wave instruction fills 1 KiB of contiguous LDS; the caller waits for its
// own loads (vmcnt) before the workgroup barrier that publishes the stage.
template <typename T, int D, int NT = 256>
struct KeyStreamDirect {
  using KS = KeyStream<T, D, NT>;
  static constexpr int CH = KS::CH, NLD = KS::NLD, kStageKeys = KS::kStageKeys;
  // Slot threadIdx.x + NT u holds key key0 + u kKeys: the bits of key0 (< kKeys) and u kKeys do not overlap,
  // so the swizzle of the sum is the exclusive or of the two swizzles and a lane keeps one chunk index.
  static constexpr int kKeys = NT / CH;
  uint32_t key0, ch0;    // of slot threadIdx.x: its stage-local key, its global chunk index

  __device__ __forceinline__ void init(uint32_t tid = threadIdx.x) {
    key0 = tid / CH;
    ch0 = (tid % CH) ^ KS::swz(key0);
  }
  // kStream: the rows are read once and not again soon - non-temporal loads
  template <bool kStream = false>
  __device__ __forceinline__ void issue(const T* kbase, int first_key, int n, char* lds) const {
    const char* sbase = reinterpret_cast<const char*>(kbase) + static_cast<int64_t>(first_key) * (CH * 16);     // uniform
    char* dst = lds + wave_index() * 1024;
    // the loads themselves stand once, behind the choice of the offsets: two copies of them would be merged
    // by the compiler and lose what it knows about the LDS they write (see stage_barrier)
    uint32_t off[NLD];
    if (first_key + kStageKeys <= n) {
#pragma unroll
      for (int u = 0; u < NLD; ++u) off[u] = (key0 + u * kKeys) * (CH * 16) + ((ch0 ^ KS::swz(u * kKeys)) * 16);
    } else {
#pragma unroll
      for (int u = 0; u < NLD; ++u)                            // the tail repeats the last row
        off[u] = min(key0 + u * kKeys, static_cast<uint32_t>(n - 1 - first_key)) * (CH * 16) + ((ch0 ^ KS::swz(u * kKeys)) * 16);
    }
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      if constexpr (kStream) load_to_lds16_stream(sbase + off[u], dst + u * (NT * 16));
      else load_to_lds16(sbase + off[u], dst + u * (NT * 16));
    }
  }
};

// The stage barrier of the streaming kernels: every LDS-direct load this wave has issued has landed, its
// LDS accesses are done, and so are everyone else's.
//
// Whatever follows the barrier inside a stage has to say which LDS it touches, or the compiler puts a wait for
// the loads just issued in front of the first LDS access (it cannot tell the buffer being filled from the
// one being read) and the double buffer hides nothing: the stage functions below therefore take every LDS
// pointer they use as a __restrict parameter, and operands loaded ahead of the stage loop are waited for in
// front of it (operands_ready), where the compiler sees it - the wait of the barrier it does not.
__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void operands_ready() { __builtin_amdgcn_s_waitcnt(0x0F70); }     // vmcnt(0)

// Pass 1: the key stream goes straight into LDS (no staging registers, one barrier per stage), the next
// stage while the current one is computed.
// Bound by HBM at 128 rows (32 layers x 32768 keys: 340 us = 6.3 TB/s, what a plain read of the same size
// reaches), by the chip's power at 256 (131072 keys: 86 -> 75 us with the stage loads overlapped, 8 waves of
// 32 rows and 2048 keys per workgroup; 4 waves of 64 rows: 82 us).
// A workgroup of NR waves keeps 32 NR window-query rows stationary, 32 per wave (128 rows, or 256 so
// that a KV head with up to 256 window rows - G*w - streams its keys once).
template <typename T, int D, int NR>
__global__ __launch_bounds__(NR * 64, sizeof(T) == 2 ? 4 : 2) void score_rowstats_kernel(ScoreArgs a) {
  constexpr int NT = NR * 64;
  using KS = KeyStream<T, D, NT>;
  constexpr int KT = KS::KT, NK = KS::NK, SK = KS::kStageKeys, EPL = KS::EPL, KD = KS::KD;
  constexpr int RT = kRowTiles, WR = 16 * RT, RB = NR * WR;
  // every chunk of a (sequence, KV head, row block) behind the same L2, so that its query rows are fetched
  // from memory once and not once per XCD; when the rows do not divide over the XCDs, the chunk index is
  // rotated instead so that the chunks every sequence has do not all land on the same XCDs
  int chunk, y;
  if (!xcd_rows_interleaved(chunk, y)) chunk = (chunk + y) % static_cast<int>(gridDim.x);
  const int rb = y % a.NRB;
  const int bg = y / a.NRB;
  const int g = bg % a.Hkv;
  const int b = bg / a.Hkv;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  if (n <= a.B) return;
  const int key_base = chunk * a.chunk_keys;
  if (key_base >= n) return;
  const int key_end = min(n, key_base + a.chunk_keys);
  const int nstages = (key_end - key_base + SK - 1) / SK;
  const int P = n - a.w;
  const int lane = threadIdx.x & 63, wv = wave_index();
  const int i = lane & 15, c = lane >> 4;
  const T* kbase = static_cast<const T*>(a.k) + (static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(g) * n) * D;

  __shared__ __attribute__((aligned(16))) char s_k[2][KS::kStageBytes];
  KeyStreamDirect<T, D, NT> ks;
  ks.init();
  if (a.keep_k) ks.template issue<false>(kbase, key_base, n, s_k[0]);
  else ks.template issue<true>(kbase, key_base, n, s_k[0]);

  // stationary rows: row (rt, i) of this wave is row rb*RB + wv*WR + 16 rt + i of the KV head
  const T* q = static_cast<const T*>(a.q_win);
  u32x4 qf[RT][NK];
  int lim[RT];                                   // last key the row sees, -1 for padding rows
  const bool any_rows = rb * RB + wv * WR < a.R;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rho = rb * RB + wv * WR + rt * 16 + i;
    const bool valid = rho < a.R;
    const int hh = valid ? rho / a.w : 0;
    const int wi = valid ? rho - hh * a.w : 0;
    const T* qp = q + (static_cast<int64_t>(b * a.Hq + g * a.G + hh) * a.w + wi) * D + c * EPL;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[rt][kk] = valid ? ld16(qp + kk * KD) : zero16();
    lim[rt] = valid ? P + wi : -1;
  }
  float m[RT], l[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) { m[rt] = -INFINITY; l[rt] = 0.f; }
  typename KS::Frags fr;
  fr.init(i, c);

  // S^T tile kt of a stage: keys 16 kt .. 16 kt + 15 against this wave's rows
  auto mma_tile = [&](const char* lds, int kt, f32x4 (&acc)[RT]) __attribute__((always_inline)) {
    u32x4 kf[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) kf[kk] = fr.get(lds, kt, kk);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) mma_step<T>(acc[rt], kf[kk], qf[rt][kk]);
    }
  };
  // A stage of prefix keys, visible to all rows, as one straight run of code (no branch between the
  // fragment reads, matrix products and exponentials of neighbouring key tiles).  The sum is taken
  // against a reference that need not be the maximum (m + log2 sum exp2(s - m) is the same number for
  // any m that keeps the terms in range): the logit of the chunk's first key.
  auto stage_full = [&](const char* lds, auto first) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      f32x4 t[RT];                               // t[rt][r] <-> key 4 c + r of the tile, row (rt, i)
      mma_tile(lds, kt, t);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if constexpr (decltype(first)::value) {
          if (kt == 0) m[rt] = __shfl(t[rt][0] * a.sl2, i);                 // lane (i, c = 0), r = 0: first key
        }
        const float nm = -m[rt];
        l[rt] += (fast_exp2(fmaf(t[rt][0], a.sl2, nm)) + fast_exp2(fmaf(t[rt][1], a.sl2, nm))) +
                 (fast_exp2(fmaf(t[rt][2], a.sl2, nm)) + fast_exp2(fmaf(t[rt][3], a.sl2, nm)));
      }
    }
  };
  // Any stage: causal mask per row, end of the sequence, running maximum.
  auto stage_masked = [&](const char* lds, int key0) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      f32x4 t[RT];
      mma_tile(lds, kt, t);
      const int kfirst = key0 + 16 * kt + 4 * c;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        float x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = (kfirst + r <= lim[rt]) ? t[rt][r] * a.sl2 : -INFINITY;
        const float tm = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
        const float mn = fmaxf(m[rt], tm);
        const float ms = (mn == -INFINITY) ? 0.f : mn;
        l[rt] = l[rt] * fast_exp2(m[rt] - ms) +
                ((fast_exp2(x[0] - ms) + fast_exp2(x[1] - ms)) + (fast_exp2(x[2] - ms) + fast_exp2(x[3] - ms)));
        m[rt] = mn;
      }
    }
  };
  auto compute = [&](const char* lds, int key0) __attribute__((always_inline)) {
    if (!any_rows) return;
    bool masked = key0 + SK > P;
    if (!masked) {
      float l_old[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) l_old[rt] = l[rt];
      if (key0 == key_base) stage_full(lds, std::true_type{});
      else stage_full(lds, std::false_type{});
      // a sum that outgrew 2^64: the stage is redone against its running maximum
      bool big = false;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) big |= !(l[rt] <= 0x1p+64f);
      masked = __any(big);
      if (masked) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) l[rt] = l_old[rt];
      }
    }
    if (masked) stage_masked(lds, key0);
  };

  // stage s is computed from buffer s & 1 while the loads of stage s + 1 fill the other one; the
  // barrier both publishes stage s and says that everyone is done reading the buffer about to be refilled
  auto step = [&](int st, const char* __restrict cur, char* __restrict nxt) __attribute__((always_inline)) {
    if (st + 1 < nstages) {
      if (a.keep_k) ks.template issue<false>(kbase, key_base + (st + 1) * SK, n, nxt);
      else ks.template issue<true>(kbase, key_base + (st + 1) * SK, n, nxt);
    }
    compute(cur, key_base + st * SK);
  };
  operands_ready();
  for (int st = 0; st < nstages; ++st) {
    stage_barrier();
    step(st, s_k[st & 1], s_k[(st + 1) & 1]);
  }

  // merge the four lanes that hold the same row (different keys) and write the chunk partial
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    merge_ml(m[rt], l[rt], __shfl_xor(m[rt], 16), __shfl_xor(l[rt], 16));
    merge_ml(m[rt], l[rt], __shfl_xor(m[rt], 32), __shfl_xor(l[rt], 32));
    if (c == 0)
      a.rowpart[(static_cast<int64_t>(bg) * a.NCH + chunk) * a.row_stride + rb * RB + wv * WR + rt * 16 + i] = make_float2(m[rt], l[rt]);
  }
}

// Chunk partials first, first + step, ... of one row, merged in that order, kFlight of them on their way at a time.
template <int kFlight>
__device__ __forceinline__ void merge_chunks(const float2* part, int64_t stride, int first, int step, int nch, float& m, float& l) {
  for (int c0 = first; c0 < nch; c0 += kFlight * step) {
    float2 v[kFlight];
#pragma unroll
    for (int u = 0; u < kFlight; ++u) v[u] = c0 + u * step < nch ? part[(c0 + u * step) * stride] : make_float2(-INFINITY, 0.f);
    float mn = m;
#pragma unroll
    for (int u = 0; u < kFlight; ++u) mn = fmaxf(mn, v[u].x);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    l *= fast_exp2(m - ms);
#pragma unroll
    for (int u = 0; u < kFlight; ++u) l += v[u].y * fast_exp2(v[u].x - ms);
    m = mn;
  }
}

// The merge as a launch of its own, where a row has so many partials that every workgroup of pass 2 doing it for its
// rows would read more than its keys: 32 rows per workgroup, every eighth partial per thread, the eight results in order.
constexpr int kMergeRows = 32;
__global__ __launch_bounds__(256) void rowstats_merge_kernel(ScoreArgs a) {
  __shared__ float2 s_ml[8][kMergeRows];
  const int row = threadIdx.x % kMergeRows, grp = threadIdx.x / kMergeRows;
  const int64_t gr = static_cast<int64_t>(blockIdx.x) * kMergeRows + row;      // row_stride is a multiple of kMergeRows
  const int bg = static_cast<int>(gr / a.row_stride);
  const int rho = static_cast<int>(gr % a.row_stride);    // row inside the KV head
  int off0;
  const int n = seq_len_checked(a.seq_off, bg / a.Hkv, a.max_seq_len, a.total_tokens, off0);
  if (n <= a.B) return;                                   // the same in all threads
  const int nch = (n + a.chunk_keys - 1) / a.chunk_keys;
  float m = -INFINITY, l = 0.f;
  if (rho < a.R) merge_chunks<8>(a.rowpart + static_cast<int64_t>(bg) * a.NCH * a.row_stride + rho, a.row_stride, grp, 8, nch, m, l);
  s_ml[grp][row] = make_float2(m, l);
  __syncthreads();
  if (grp != 0) return;
#pragma unroll
  for (int q = 1; q < 8; ++q) merge_ml(m, l, s_ml[q][row].x, s_ml[q][row].y);
  a.row_lse[gr] = (l > 0.f && rho < a.R) ? m + fast_log2(l) : INFINITY;          // padding rows: +inf
}

// NR waves of 32 rows each (4 waves for a block of 128 rows, 8 for 256).  With the stage loads
// overlapped and the stage free of branches: 448 -> 426 us for 32 layers x 32768 keys (HBM, 160 MiB of votes
// and logits written into the read stream), 105 -> 80 us for 131072 keys at 256 rows.  64 rows per wave
// (half the LDS reads) leaves too few waves: 440 us and 90 us or more.
template <typename T, int D, int NR>
__global__ __launch_bounds__(NR * 64, sizeof(T) == 2 ? 4 : 2) void score_votes_kernel(ScoreArgs a) {
  constexpr int NT = NR * 64;
  using KS = KeyStream<T, D, NT>;
  constexpr int KT = KS::KT, NK = KS::NK, SK = KS::kStageKeys, RT = kRowTiles, RB = 16 * RT * NR, EPL = KS::EPL, KD = KS::KD;
  // grid: x = key chunk, y = (sequence, KV head, row block).  Workgroups are dealt to the 8 XCDs
  // round-robin in launch order: the launch index is re-read so that every chunk of a y sits behind the
  // same L2 (the stationary query rows are then fetched from memory once, not once per XCD); when y
  // does not divide over the XCDs the chunk index is rotated by y instead, so that with sequences of
  // different lengths the chunks every sequence has do not all land on the same XCDs.
  clear_words(a.zero_words, a.zero_count);
  int chunk, y;
  if (!xcd_rows_interleaved(chunk, y)) chunk = (chunk + y) % static_cast<int>(gridDim.x);
  const int rb = y % a.NRB;
  const int bg = y / a.NRB;
  const int g = bg % a.Hkv;
  const int b = bg / a.Hkv;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  if (n <= a.B) return;
  const int P = n - a.w;
  const int key_base = chunk * a.chunk_keys;
  if (key_base >= P) return;
  const int key_end = min(P, key_base + a.chunk_keys);
  const int nstages = (key_end - key_base + SK - 1) / SK;
  const int lane = threadIdx.x & 63, wv = wave_index();
  const int i = lane & 15, c = lane >> 4;
  const int64_t head_tok = static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(g) * n;
  const T* kbase = static_cast<const T*>(a.k) + head_tok * D;
  float* vote = a.vote + static_cast<int64_t>(rb) * a.plane + head_tok;

  __shared__ __attribute__((aligned(16))) char s_k[2][KS::kStageBytes];
  __shared__ float s_v[2][NR * 2 * SK];              // partial votes of a stage per row wave and pair of row groups
  __shared__ float s_z[2][kMaxCalHeads * SK];       // exported calibration logits of a stage, per head
  const int row0 = rb * RB + wv * (16 * RT);       // first row of this wave
  // the key stream goes straight into LDS (no staging registers: one more wave per SIMD fits)
  KeyStreamDirect<T, D, NT> ks;
  ks.init();
  ks.template issue<true>(kbase, key_base, n, s_k[0]);
  // stationary rows as operands: lane (i, c) holds piece c of row 16 rt + i
  u32x4 qf[RT][NK];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rho = row0 + rt * 16 + i;
    const bool valid = rho < a.R;
    const int hh = valid ? rho / a.w : 0;
    const int wi = valid ? rho - hh * a.w : 0;
    const T* qp = static_cast<const T*>(a.q_win) + (static_cast<int64_t>(b * a.Hq + g * a.G + hh) * a.w + wi) * D + c * EPL;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[rt][kk] = valid ? ld16(qp + kk * KD) : zero16();
  }
  // S tiles are rows x keys here: lane (i, c) holds key i and rows 16 rt + 4 c + r of the wave
  float lse[RT][4];
  if (a.rows_merged) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        lse[rt][r] = a.row_lse[static_cast<int64_t>(bg) * a.row_stride + row0 + rt * 16 + 4 * c + r];   // padding rows: +inf
  } else {
    // lanes j and j + 32 of the wave: row j of its 32, every other chunk each
    const int rho = row0 + (lane & 31);
    float val = INFINITY;
    if (a.win_lse) {
      if (rho < a.R) {
        const int hh = rho / a.w, wi = rho - hh * a.w;
        val = a.win_lse[static_cast<int64_t>(b * a.Hq + g * a.G + hh) * a.w + wi] * kLog2e;
      }
    } else {
      float m = -INFINITY, l = 0.f;
      const int nch = (n + a.chunk_keys - 1) / a.chunk_keys;
      if (rho < a.R) merge_chunks<16>(a.rowpart + static_cast<int64_t>(bg) * a.NCH * a.row_stride + rho, a.row_stride, lane >> 5, 2, nch, m, l);
      merge_ml(m, l, __shfl_xor(m, 32), __shfl_xor(l, 32));
      if (l > 0.f && rho < a.R) val = m + fast_log2(l);
    }
    if (chunk == 0 && lane < 32) a.row_lse[static_cast<int64_t>(bg) * a.row_stride + rho] = val;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) lse[rt][r] = __shfl(val, 16 * rt + 4 * c + r);
  }

  // Rows that are the last window query of a head (the default calibration query, Alg. 1
  // step 5) also export their logits, so that the calibration pass need not read K again.
  // (the export needs w % 4 == 0, so that such a row is always slot r = 3 of its lane)
  int cal_head[RT];                     // head in group whose last window row is this lane's (rt, r = 3), or -1
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rho = row0 + rt * 16 + 4 * c + 3;
    cal_head[rt] = (a.cal_logit != nullptr && rho < a.R && (rho % a.w) == a.w - 1) ? rho / a.w : -1;
  }
  uint32_t cal_mask = 0;                // heads whose last window row is in this row block
  if (a.cal_logit)
    for (int hh = 0; hh < a.G; ++hh) cal_mask |= ((hh * a.w + a.w - 1) / RB == rb ? 1u : 0u) << hh;
  float* zrow = a.cal_logit ? a.cal_logit + static_cast<int64_t>(b * a.Hq + g * a.G) * a.zstride : nullptr;

  // One stage, without a branch up to the export at its end, so that the fragment reads, matrix products
  // and exponentials of neighbouring key tiles are scheduled into each other.
  typename KS::Frags fr;
  fr.init(i, c);
  auto compute = [&](const char* lds, float* sv, float* sz) __attribute__((always_inline)) {
    float vs[KT], zc[KT][RT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      u32x4 kf[NK];
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) kf[kk] = fr.get(lds, kt, kk);
      float v = 0.f;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) mma_step<T>(acc, qf[rt][kk], kf[kk]);
#pragma unroll
        for (int r = 0; r < 4; ++r) v += fast_exp2(fmaf(acc[r], a.sl2, -lse[rt][r]));
        zc[kt][rt] = acc[3];
      }
      vs[kt] = v;
    }
    // only neighbouring row groups are added here (one lane swap), the rest of the sum is left to the
    // flush; both lanes of a pair hold the sum and store it to the same place
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      float lo, hi;
      pair16(vs[kt], lo, hi);
      sv[(2 * wv + (c >> 1)) * SK + 16 * kt + i] = lo + hi;
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      if (cal_head[rt] >= 0) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) sz[cal_head[rt] * SK + 16 * kt + i] = zc[kt][rt] * a.sl2;
      }
  };
  // after the stage barrier: add the partial votes in a fixed order (row waves ascending, inside a wave
  // (c0 + c1) + (c2 + c3), the inner sums already taken) and store; the second wave stores the exported
  // logits, one coalesced row per head
  auto flush = [&](const float* sv, const float* sz, int key0) __attribute__((always_inline)) {
    if (threadIdx.x < SK) {
      const int key = key0 + threadIdx.x;
      if (key < P) {
        float tot = 0.f;
#pragma unroll
        for (int ww = 0; ww < NR; ++ww)
          tot += sv[2 * ww * SK + threadIdx.x] + sv[(2 * ww + 1) * SK + threadIdx.x];
        __builtin_nontemporal_store(tot, vote + key);    // written once, read by a later kernel: kept out of the caches the K stream uses
      }
    } else if (cal_mask != 0 && threadIdx.x >= 64 && threadIdx.x < 64 + SK) {
      const int t = threadIdx.x - 64;
      const int key = key0 + t;
      if (key < P)
        for (uint32_t left = cal_mask; left; left &= left - 1u) {
          const int hh = __ffs(left) - 1;
          __builtin_nontemporal_store(sz[hh * SK + t], zrow + static_cast<int64_t>(hh) * a.zstride + key);
        }
    }
  };

  // stage s is computed from buffer s & 1 while the loads of stage s + 1 fill the other one; the barrier
  // publishes stage s, says that everyone is done reading the buffer about to be refilled, and hands
  // the partial votes of stage s - 1 to the flush
  auto step = [&](int st, const char* __restrict cur, char* __restrict nxt, float* __restrict sv, float* __restrict sz,
                  const float* __restrict sv_prev, const float* __restrict sz_prev) __attribute__((always_inline)) {
    if (st + 1 < nstages) ks.template issue<true>(kbase, key_base + (st + 1) * SK, n, nxt);
    if (st > 0) flush(sv_prev, sz_prev, key_base + (st - 1) * SK);
    compute(cur, sv, sz);
  };
  operands_ready();
  for (int st = 0; st < nstages; ++st) {
    const int cb = st & 1, ob = cb ^ 1;
    stage_barrier();
    step(st, s_k[cb], s_k[ob], s_v[cb], s_z[cb], s_v[ob], s_z[ob]);
  }
  stage_barrier();
  flush(s_v[(nstages - 1) & 1], s_z[(nstages - 1) & 1], key_base + (nstages - 1) * SK);
}

}  // namespace cd
