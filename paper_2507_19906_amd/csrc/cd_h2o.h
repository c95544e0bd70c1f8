// H2O as the eviction strategy f of Alg. 1 step 3 (Sec. 4.1.3: importance = accumulated
// attention score): every prompt query attends causally to the prompt, and a position's score
// is the probability mass it received, summed over all queries and over the G query heads of
// its KV head.  Unlike the observation-window scoring this is a dense n x n contraction per head
// (matrix-core bound), done in two passes that mirror each other:
//   pass 1 (h2o_rowlse): query rows stay in registers, keys stream through LDS; a lane owns a
//           query row, so the running (max, sum exp2) of its softmax stay in the lane -> row
//           log-sum-exp for every prompt position.
//   pass 2 (h2o_votes):  keys stay in registers, query rows stream through LDS; a lane owns a
//           key, so the column sum of p = exp2(s - lse_row) over all rows that see the key stays
//           in the lane -> vote[j], written once, no atomics, fixed summation order.
// Both passes skip the tiles above the diagonal and mask only the tiles on it.
#pragma once
#include "cd_common.h"
#include "cd_score.h"

#include <type_traits>

namespace cd {

// Both passes run at the chip's power limit (the clock settles near 2 GHz), so what counts is the energy per
// logit: with 64 stationary rows per wave a fragment read from LDS serves 4 row tiles instead of 2.  Together
// with the stage loads overlapped and branch-free full stages, one layer of 32 query heads x 32768 rows:
// both passes 8.7 -> 7.9 ms; 32 rows per wave 8.2 ms, 128 rows 8.0 ms, 32 x 32 x 16 matrix instructions 8.4 ms
// (same cycles, lower clock).  A dense bf16 product of 8192 x 8192 reaches 1.33 PFLOP/s on the same card, at which
// the 8.8 TFLOP of the two passes would take 6.6 ms without a single exponential.
// fp32 keeps 32 rows: 64 would need all 256 registers; so do bf16 calls of few workgroups (the launch decides).
// RT = 16-row tiles of stationary rows per wave; stationary rows (or keys) per workgroup of 4 waves:
constexpr int h2o_block(int tiles) { return 4 * 16 * tiles; }

struct H2oArgs {
  const void* q_full;        // packed like K with Hq heads: sequence b at token seq_off[b], inside [Hq][n_b][D]
  const void* k;
  const int32_t* seq_off;
  int64_t total_tokens;
  int batch, Hq, Hkv, G, B, max_seq_len;
  int lse_stride;            // floats per (sequence, query head) in row_lse; a multiple of the row block
  float sl2;                 // scale * log2(e)
  float* row_lse;            // [batch*Hq][lse_stride], log2 units; rows >= n_b hold +inf
  int splits;                // workgroups that share the stream of a block of stationary rows (or pair of key blocks)
  float2* row_part;          // splits > 1: [batch*Hq][splits][lse_stride] (max, sum) per split, merged into row_lse
  float* vote;               // [G][splits][plane]: a plane per query head of the group and split, each packed like K with one float per row
  int64_t plane;             // floats per plane: total_tokens*Hkv rounded up to a multiple of 64
  void* q_last;              // [batch][Hq][D]: the last prompt query of every head (Q_{-1})
  uint32_t* zero_words;      // words pass 1 clears for the selection that follows, or NULL
  int64_t zero_count;
};

// Row statistics of two sets of keys, a sum that is not a number kept also where no maximum is left: a row that sees such a
// logit has log-sum-exp +inf whichever share it lies in.
__device__ __forceinline__ void merge_rows(float& m, float& l, float m2, float l2) {
  const float sum = l + l2;
  merge_ml(m, l, m2, l2);
  if (sum != sum) l = sum;
}

// Calls of few workgroups leave the chip waiting for the longest stream (the last rows see every key), so those split the
// streams: each of `splits` workgroups takes a share of the stages; row partials are merged by a launch of their own, vote
// shares have planes of their own, which the selection adds in a fixed order like those of the heads.  kSplit stands apart
// so that large calls keep their registers (this pass in fp32, D = 128: 160, three workgroups on a compute unit; 184, two).
template <typename T, int D, int RT, bool kSplit>
__global__ __launch_bounds__(256, 2) void h2o_rowlse_kernel(H2oArgs a) {
  using KS = KeyStream<T, D>;
  constexpr int KT = KS::KT, NK = KS::NK, SK = KS::kStageKeys, EPL = KS::EPL, KD = KS::KD;
  constexpr int WR = 16 * RT, BR = 4 * WR;
  clear_words(a.zero_words, a.zero_count);
  int vx, vh;                                    // row block and (sequence, query head) of this workgroup
  xcd_head_major(vx, vh);
  const int hq = vh % a.Hq, b = vh / a.Hq, g = hq / a.G;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  const T* qbase = static_cast<const T*>(a.q_full) + (static_cast<int64_t>(off0) * a.Hq + static_cast<int64_t>(hq) * n) * D;
  // Q_{-1} of this head, the calibration query of Alg. 1 step 5 (also for prompts within the budget)
  if (vx == 0 && n > 0 && threadIdx.x < D)
    store_elem<T>(static_cast<T*>(a.q_last), static_cast<int64_t>(b * a.Hq + hq) * D + threadIdx.x,
                  load_elem<T>(qbase, static_cast<int64_t>(n - 1) * D + threadIdx.x));
  if (n <= a.B) return;
  const int nrb = (n + BR - 1) / BR;
  const int nsplit = kSplit ? a.splits : 1, split = kSplit ? vx % nsplit : 0;
  const int rbp = nrb - 1 - vx / nsplit;         // late rows (most keys) are launched first
  if (rbp < 0) return;
  const int i0 = rbp * BR;
  const int lane = threadIdx.x & 63, wv = wave_index();
  const int i = lane & 15, c = lane >> 4;
  const T* kbase = static_cast<const T*>(a.k) + (static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(g) * n) * D;
  const int wrow0 = i0 + wv * WR;                // first row of this wave

  __shared__ __attribute__((aligned(16))) char s_k[2][KS::kStageBytes];
  u32x4 qf[RT][NK];
  int lim[RT];                                   // last key the row sees (= its position), -1 for padding rows
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = wrow0 + rt * 16 + i;
    const bool valid = row < n;
    const T* qp = qbase + static_cast<int64_t>(valid ? row : 0) * D + c * EPL;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[rt][kk] = valid ? ld16(qp + kk * KD) : zero16();
    lim[rt] = valid ? row : -1;
  }
  float m[RT], l[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) { m[rt] = -INFINITY; l[rt] = 0.f; }
  typename KS::Frags fr;
  fr.init(i, c);

  const int key_end = min(n, i0 + BR);           // no row of the block sees a key beyond its last row
  const int all = (key_end + SK - 1) / SK, st0 = split * all / nsplit, nstages = (split + 1) * all / nsplit;
  KeyStreamDirect<T, D> ks;
  ks.init();
  if (st0 < nstages) ks.issue(kbase, st0 * SK, n, s_k[st0 & 1]);

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
  // A stage every row of the wave sees completely, as one straight run of code: fragment reads, matrix
  // products and exponentials of neighbouring key tiles have no branch between them and are scheduled
  // into each other.  The sum is taken against a reference m that need not be the row maximum:
  // m + log2(sum of exp2(s - m)) is the same number for any m that keeps the terms in range.  The
  // reference is the logit of the first key of the workgroup's stream (every row sees it: a stage that some row
  // does not see completely is never followed by one that all see).
  auto stage_full = [&](const char* lds, auto first) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      f32x4 t[RT];                    // t[rt][r] <-> key 4 c + r of the tile, row (rt, i)
      mma_tile(lds, kt, t);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if constexpr (decltype(first)::value) {
          if (kt == 0) m[rt] = __shfl(t[rt][0] * a.sl2, i);                 // lane (i, c = 0), result 0: first key
        }
        const float nm = -m[rt];
        l[rt] += (fast_exp2(fmaf(t[rt][0], a.sl2, nm)) + fast_exp2(fmaf(t[rt][1], a.sl2, nm))) +
                 (fast_exp2(fmaf(t[rt][2], a.sl2, nm)) + fast_exp2(fmaf(t[rt][3], a.sl2, nm)));
      }
    }
  };
  // Any stage: per-row causal mask, running maximum.
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
    if (key0 > wrow0 + WR - 1 || wrow0 >= n) return;        // nothing of this stage is visible to the wave
    const bool full = key0 + SK - 1 <= wrow0 && wrow0 + WR <= n;   // every key visible to every (real) row
    bool masked = !full;
    if (full) {
      float l_old[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) l_old[rt] = l[rt];
      if (key0 == st0 * SK) stage_full(lds, std::true_type{});
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
  // barrier both publishes stage s and says that everyone is done reading the buffer about to be
  // refilled
  auto step = [&](int st, const char* __restrict cur, char* __restrict nxt) __attribute__((always_inline)) {
    if (st + 1 < nstages) ks.issue(kbase, (st + 1) * SK, n, nxt);
    compute(cur, st * SK);
  };
  operands_ready();
  for (int st = st0; st < nstages; ++st) {
    stage_barrier();
    step(st, s_k[st & 1], s_k[(st + 1) & 1]);
  }

  // merge the lanes that hold the same row (different keys); padding rows get +inf so that
  // pass 2 turns them into probability 0
  float* out = a.row_lse + static_cast<int64_t>(b * a.Hq + hq) * a.lse_stride;
  float2* part = kSplit ? a.row_part + (static_cast<int64_t>(b * a.Hq + hq) * nsplit + split) * a.lse_stride : nullptr;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    merge_rows(m[rt], l[rt], __shfl_xor(m[rt], 16), __shfl_xor(l[rt], 16));
    merge_rows(m[rt], l[rt], __shfl_xor(m[rt], 32), __shfl_xor(l[rt], 32));
    const int row = wrow0 + rt * 16 + i;
    if (c == 0 && row < a.lse_stride) {
      if constexpr (kSplit) part[row] = make_float2(m[rt], l[rt]);
      else out[row] = (row < n && l[rt] > 0.f) ? m[rt] + fast_log2(l[rt]) : INFINITY;
    }
  }
}

// The row partials of a call whose streams are split, one thread per row up to the end of its last block.
__global__ __launch_bounds__(256) void h2o_rowmerge_kernel(H2oArgs a, int block_rows) {
  const int row = blockIdx.x * 256 + threadIdx.x, head = blockIdx.y, b = head / a.Hq;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  if (n <= a.B || row >= min((n + block_rows - 1) / block_rows * block_rows, a.lse_stride)) return;
  const float2* part = a.row_part + static_cast<int64_t>(head) * a.splits * a.lse_stride + row;
  float m = -INFINITY, l = 0.f;
  for (int s = 0; s < a.splits; ++s) {
    const float2 v = part[static_cast<int64_t>(s) * a.lse_stride];
    merge_rows(m, l, v.x, v.y);
  }
  a.row_lse[static_cast<int64_t>(head) * a.lse_stride + row] = (row < n && l > 0.f) ? m + fast_log2(l) : INFINITY;
}

// fp32 has to fit three workgroups on a compute unit (168 registers a lane; with 184 two fit, and 2 prompts of 2584
// tokens, 32 heads, D = 128, took 599 us instead of 515): the addresses of the row stream are therefore worked out anew
// for every stage - hidden from the compiler, which would keep them in registers or, short of those, in memory - a
// dozen instructions beside 256 matrix products (now 510 us).
template <typename T, int D, int RT, bool kSplit>
__device__ __forceinline__ void h2o_votes(const H2oArgs& a) {
  using KS = KeyStream<T, D>;
  constexpr int KT = KS::KT, NK = KS::NK, SK = KS::kStageKeys, EPL = KS::EPL, KD = KS::KD;
  constexpr int WR = 16 * RT, BR = 4 * WR;
  // grid: x = pair of key blocks (block x and its mirror nblk-1-x: early keys are seen by many
  // rows, late keys by few, so every workgroup gets the same amount of work), y = (sequence, KV
  // head), z = query head of the group and share of its rows; each writes its own plane of votes, which
  // the selection adds up in a fixed order.
  int vx, vh;                                    // block pair and ((sequence, KV head), (head in group, share)) of this workgroup
  xcd_head_major(vx, vh);
  const int bg = vh / static_cast<int>(gridDim.z), pl = vh % static_cast<int>(gridDim.z);   // a group's heads side by side
  const int nsplit = kSplit ? a.splits : 1, hh = pl / nsplit, split = pl - hh * nsplit;
  const int g = bg % a.Hkv, b = bg / a.Hkv;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  if (n <= a.B) return;
  const int nblk = (n + BR - 1) / BR;
  const int lane = threadIdx.x & 63, wv = wave_index();
  const int i = lane & 15, c = lane >> 4;
  const int64_t head_tok = static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(g) * n;
  const T* kbase = static_cast<const T*>(a.k) + head_tok * D;
  const int hq = g * a.G + hh;
  const T* qbase = static_cast<const T*>(a.q_full) + (static_cast<int64_t>(off0) * a.Hq + static_cast<int64_t>(hq) * n) * D;
  const float* lse_row = a.row_lse + static_cast<int64_t>(b * a.Hq + hq) * a.lse_stride;
  float* vote = a.vote + static_cast<int64_t>(pl) * a.plane + head_tok;

  __shared__ __attribute__((aligned(16))) char s_q[2][KS::kStageBytes];
  __shared__ __attribute__((aligned(16))) float s_z[2][64];      // row log-sum-exp of the staged rows
  typename KS::Frags fr;
  fr.init(i, c);

  for (int job = 0; job < 2; ++job) {
    const int blk = job == 0 ? vx : nblk - 1 - vx;
    // uniform over the workgroup: the first half of the blocks as job 0, their mirrors as job 1
    if (job == 0 ? 2 * blk >= nblk : (blk < 0 || blk <= vx)) continue;
    const int j0 = blk * BR;
    const int wkey0 = j0 + wv * WR;                // first key of this wave
    u32x4 kf[RT][NK];
    int kpos[RT];                                  // position of the lane's key; beyond every row for padding keys
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int key = wkey0 + rt * 16 + i;
      const bool valid = key < n;
      const T* kp = kbase + static_cast<int64_t>(valid ? key : 0) * D + c * EPL;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) kf[rt][kk] = valid ? ld16(kp + kk * KD) : zero16();
      kpos[rt] = valid ? key : 0x7fffffff;
    }
    float v[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) v[rt] = 0.f;

    // streamed rows: j0 .. n-1 of this query head, SK per stage, with their log-sum-exp
    const int all = (n - j0 + SK - 1) / SK, st0 = split * all / nsplit, nstages = (split + 1) * all / nsplit;
    auto issue = [&](int st, char* rows, float* z) __attribute__((always_inline)) {   // rows and their log-sum-exp, straight into LDS
      const int q0 = j0 + st * SK;
      uint32_t tid = threadIdx.x;
      if constexpr (sizeof(T) == 4) asm("" : "+v"(tid));
      KeyStreamDirect<T, D> ks;
      ks.init(tid);
      ks.issue(qbase, q0, n, rows);
      if (tid < SK) load_to_lds4(lse_row + q0 + tid, z);
    };
    __syncthreads();                               // the previous job is done with the buffers
    if (st0 < nstages) issue(st0, s_q[st0 & 1], s_z[st0 & 1]);

    // one stage; with kFull every row sees every key of the wave and the stage is one straight run of
    // code, in which the exponentials of a row tile are scheduled into the products of the next
    auto stage = [&](const char* lds, const float* zs, int q0, auto full) __attribute__((always_inline)) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        u32x4 qf[NK];
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) qf[kk] = fr.get(lds, kt, kk);
        f32x4 t[RT];                  // t[rt][r] <-> row 16 kt + 4 c + r of the stage, key (rt, i)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          t[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < NK; ++kk) mma_step<T>(t[rt], qf[kk], kf[rt][kk]);
        }
        const int q = 16 * kt + 4 * c;
        const f32x4 z = *reinterpret_cast<const f32x4*>(zs + q);         // log-sum-exp of four rows; +inf beyond n
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          float p[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            p[r] = fast_exp2(fmaf(t[rt][r], a.sl2, -z[r]));
            if constexpr (!decltype(full)::value) p[r] = (q0 + q + r >= kpos[rt]) ? p[r] : 0.f;
          }
          v[rt] += (p[0] + p[1]) + (p[2] + p[3]);
        }
      }
    };
    auto compute = [&](const char* lds, const float* zs, int st) __attribute__((always_inline)) {
      const int q0 = j0 + st * SK;
      if (q0 + SK - 1 < wkey0 || wkey0 >= n) return;          // no row of the stage sees a key of this wave
      if (q0 >= wkey0 + WR - 1) stage(lds, zs, q0, std::true_type{});
      else stage(lds, zs, q0, std::false_type{});
    };

    auto step = [&](int st, const char* __restrict cur, char* __restrict nxt, const float* __restrict z,
                    float* __restrict z_nxt) __attribute__((always_inline)) {
      if (st + 1 < nstages) issue(st + 1, nxt, z_nxt);
      compute(cur, z, st);
    };
    operands_ready();
    for (int st = st0; st < nstages; ++st) {
      const int cb = st & 1, ob = cb ^ 1;
      stage_barrier();
      step(st, s_q[cb], s_q[ob], s_z[cb], s_z[ob]);
    }

#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float tot = col4_sum(v[rt]);           // the four row groups c, fixed tree
      const int key = wkey0 + rt * 16 + i;
      if (c == 0 && key < n) vote[key] = tot;
    }
  }
}

template <typename T, int D, int RT>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 3 : 2) void h2o_votes_kernel(H2oArgs a) { h2o_votes<T, D, RT, false>(a); }
template <typename T, int D, int RT>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 3 : 2) void h2o_shared_votes_kernel(H2oArgs a) { h2o_votes<T, D, RT, true>(a); }

}  // namespace cd
