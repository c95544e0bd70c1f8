// Pooling, per-KV-head top-k of the pooled scores (the selection inside Alg. 1 step 3), the
// optional "calibration size" cut of the evicted tokens (Sec. 5.3) and the gather of
// KV_compress, one workgroup per (sequence, KV head).
//
// Selection is exact: a most-significant-digit-first radix select on the fp32 bit patterns
// (scores are >= 0, so unsigned order equals numeric order) finds the value of a given rank
// and how many entries equal to it fall inside the rank; an ordered compaction then keeps
// everything above it plus the first equal entries in position order - the "ties to the lower
// index" rule - and emits positions in ascending order.  Integer work only: bit-exact and
// deterministic.  Two ranks are used: k_sel = B - w (the retained prefix tokens) and, when a
// calibration size m is set, k_sel + m (retained + the m most important evicted tokens, which
// form the calibration set; everything below is dropped for good).
//
// Two variants: select_lds_kernel (prefix up to 32768 positions: one workgroup per head
// pools the votes itself and keeps the keys in registers) and the wide_* kernels (longer
// prefixes: many workgroups per head, histograms and counts combined in global memory).
#pragma once
#include "cd_common.h"
#include "cd_score.h"

namespace cd {

constexpr int kSelThreads = 1024;
constexpr int kSelPerThread = 32;              // LDS variant: positions per thread (= one bitmap word)
constexpr int kSelMaxLdsKeys = kSelThreads * kSelPerThread;   // longest prefix the LDS variant takes
constexpr int kSelMaxPool = 15;                // widest pooling kernel the LDS variant takes

// K_c[g][r] = K[g][idx[g][r]], V likewise, 16 bytes per thread and copy.
struct GatherArgs {
  const int32_t* indices;        // [batch][Hkv][B]
  const int32_t* cache_off;
  const void* k; const void* v;
  void* k_c; void* v_c;
  int row_bytes;
  int blocks;                    // workgroups of 256 threads that cover one (sequence, KV head)
};
constexpr int kGatherCopies = 1;                       // independent copies of K and of V in flight per thread
constexpr int kGatherVecs = 256 * kGatherCopies;       // 16-byte pieces per workgroup of 256 threads

// Pieces t0, t0 + NT, ... (kCopies of them, below `total`) of the retained rows of one (sequence, KV head).
template <int NT, int kCopies>
__device__ __forceinline__ void gather_pieces(const GatherArgs& a, const int32_t* idx, int t0, int total, int n, bool keeps_all,
                                              int64_t src_row, int64_t dst_row) {
  const int vec_per_row = a.row_bytes / 16;
  u32x4 kk[kCopies], vv[kCopies];
#pragma unroll
  for (int u = 0; u < kCopies; ++u) {
    const int t = t0 + u * NT;
    if (t < total) {
      const int r = t / vec_per_row, vcol = t - r * vec_per_row;
      // a sequence within the budget keeps every row (its list may be written by this very launch); clamped: the
      // list may be the caller's (a strategy applied outside the library)
      const int src = keeps_all ? r : min(max(idx[r], 0), n - 1);
      const int64_t so = (src_row + src) * a.row_bytes + vcol * 16;
      kk[u] = ld16(static_cast<const char*>(a.k) + so);
      vv[u] = ld16(static_cast<const char*>(a.v) + so);
    }
  }
#pragma unroll
  for (int u = 0; u < kCopies; ++u) {
    const int t = t0 + u * NT;
    if (t < total) {
      const int r = t / vec_per_row, vcol = t - r * vec_per_row;
      const int64_t dof = (dst_row + r) * a.row_bytes + vcol * 16;
      st16(static_cast<char*>(a.k_c) + dof, kk[u]);
      st16(static_cast<char*>(a.v_c) + dof, vv[u]);
    }
  }
}

// Workgroup `block` of the a.blocks (256 threads each) that gather the rows of one (sequence, KV head).
__device__ __forceinline__ void gather_block(const GatherArgs& a, int block, int b, int g, int Hkv, int B, int n, int off0) {
  const int len = min(n, B);
  const int c0 = a.cache_off[b];
  const int cap = a.cache_off[b + 1] - c0;
  if (cap < len) return;                 // capacity contract broken: write nothing
  gather_pieces<256, kGatherCopies>(a, a.indices + (static_cast<int64_t>(b) * Hkv + g) * B,
                                    block * kGatherVecs + static_cast<int>(threadIdx.x), len * (a.row_bytes / 16), n, n <= B,
                                    static_cast<int64_t>(off0) * Hkv + static_cast<int64_t>(g) * n,
                                    static_cast<int64_t>(c0) * Hkv + static_cast<int64_t>(g) * cap);
}

struct SelectArgs {
  const int32_t* seq_off;
  int64_t total_tokens;
  int batch, Hkv, w, B, max_seq_len, W32, NRB, pool_k;
  int calib;               // calibration size m (0 = every evicted token)
  int write_scores;        // LDS variant: also store the pooled scores (inspection only)
  const float* vote;       // [NRB][plane]   (LDS-key variant pools these itself)
  int64_t plane;           // floats per vote plane, a multiple of 64
  float* score;            // [total_tokens*Hkv] pooled scores: written (LDS variant) or read
  int32_t* indices;        // [batch][Hkv][B]
  int32_t* cal_indices;    // [batch][Hkv][calib] positions of the calibration set, or NULL
  int32_t* cache_lens;     // [batch]
  uint32_t* bitmap;        // [batch*Hkv][W32]: bit set = position is NOT in the calibration set
  GatherArgs gather;
  int gather_here;         // LDS variant: the workgroup also gathers the rows it has chosen
};

// The bin of a finished 256-bin histogram in which the count from the top reaches `remaining`;
// updates prefix / remaining like one radix pass.  Lane l holds bins 4l..4l+3 in `hb`.  Called
// by all 64 lanes of a wave.
__device__ __forceinline__ void wide_pick(const u32x4 hb, int shift, uint32_t& prefix, uint32_t& remaining) {
  const int lane = threadIdx.x & 63;
  const uint32_t h0 = hb[0], h1 = hb[1], h2 = hb[2], h3 = hb[3];
  const uint32_t mine = h0 + h1 + h2 + h3;
  const uint32_t upto = wave_inclusive_scan(mine);
  const uint32_t above = last_lane(upto) - upto;      // keys in bins owned by higher lanes
  const uint32_t acc = above + mine;
  const bool hit = above < remaining && remaining <= acc;
  uint32_t cum = above;
  int bin = 0;
  if (cum + h3 >= remaining) bin = 3;
  else { cum += h3; if (cum + h2 >= remaining) bin = 2;
    else { cum += h2; if (cum + h1 >= remaining) bin = 1; else { cum += h1; bin = 0; } } }
  const uint64_t who = __ballot(hit);
  if (who == 0) return;                              // inconsistent histogram: leave the digit 0
  const int src = __ffsll(static_cast<long long>(who)) - 1;
  const uint32_t digit = __shfl(static_cast<uint32_t>(4 * lane + bin), src);
  const uint32_t rem = __shfl(remaining - cum, src);
  prefix |= digit << shift;
  remaining = rem;
}

// Radix select of the `rank`-th largest key (rank >= 1, at most the number of keys).
// `for_each_key(visit)` must call visit(u) once for every key this thread owns.  On return
// thr = that key's bit pattern and need_eq = how many keys equal to thr lie within the rank.
// `hist`: one 256-bin histogram per pass, all zero, with a barrier since they were cleared.  Must be called by
// every thread of the workgroup.  Latency is all there is to it (a head of 8192 scores keeps one compute unit busy for
// some microseconds): one barrier per pass, every wave finds the digit for itself, the last runs of a wave are
// added up before they reach the histogram (selection of 32768 scores 42 -> 33 us, three barriers a pass before).
template <typename ForEach>
__device__ __forceinline__ void radix_select(uint32_t (*hist)[256], uint32_t rank, ForEach&& for_each_key, uint32_t& thr,
                                             uint32_t& need_eq) {
  const int lane = threadIdx.x & 63;
  uint32_t prefix = 0;            // bits decided so far (the high bits of the answer)
  uint32_t remaining = rank;      // rank of the answer among the keys matching `prefix`
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const uint32_t himask = (pass == 0) ? 0u : (0xFFFFFFFFu << (shift + 8));
    {
      // run-length compressed updates: scores share their leading digits, so consecutive keys
      // of a thread mostly fall in the same bin and only bin changes touch the histogram
      uint32_t run_bin = 0, run_len = 0;
      for_each_key([&](uint32_t u) {
        if ((u & himask) == prefix) {
          const uint32_t bin = (u >> shift) & 0xFF;
          if (bin != run_bin && run_len) { atomicAdd(&hist[pass][run_bin], run_len); run_len = 0; }
          run_bin = bin;
          ++run_len;
        }
      });
      // the last runs of a wave are mostly in one bin (the leading digits): one addition then
      const uint32_t first = __builtin_amdgcn_readfirstlane(run_bin);
      if (__all(run_bin == first)) {
        const uint32_t sum = last_lane(wave_inclusive_scan(run_len));
        if (lane == 0 && sum) atomicAdd(&hist[pass][first], sum);
      } else if (run_len) {
        atomicAdd(&hist[pass][run_bin], run_len);
      }
    }
    __syncthreads();
    wide_pick(*reinterpret_cast<const u32x4*>(&hist[pass][4 * lane]), shift, prefix, remaining);
  }
  thr = prefix;
  need_eq = remaining;
}

// Membership of one candidate, given how many greater / equal keys precede it in position order.
struct Cut {
  uint32_t thr, need_eq;
  bool all;              // no cut: every candidate is inside
  // number of inside candidates among the first `pos` positions, from the running counts
  __device__ __forceinline__ uint32_t rank(uint32_t pos, uint32_t gt_before, uint32_t eq_before) const {
    return all ? pos : gt_before + min(eq_before, need_eq);
  }
};

// Members of a cut among the positions of one thread, as bit masks: everything above the threshold, and of the
// keys equal to it the first (need_eq - equal ones at earlier positions), i.e. ties go to the lower index.
__device__ __forceinline__ uint32_t cut_members(const Cut& c, uint32_t gtm, uint32_t eqm, uint32_t eq_before, uint32_t valid) {
  if (c.all) return valid;
  const uint32_t allow = c.need_eq > eq_before ? c.need_eq - eq_before : 0u;
  if (allow < static_cast<uint32_t>(__popc(eqm))) {
    uint32_t kept = 0;
    for (uint32_t t = 0; t < allow; ++t) { const uint32_t low = eqm & (0u - eqm); kept |= low; eqm ^= low; }
    eqm = kept;
  }
  return gtm | eqm;
}

// ---- long prefixes: selection spread over many workgroups ------------------------------------
// One workgroup per head cannot sweep hundreds of thousands of scores quickly, so the prefix is
// cut into segments of kWideSeg positions, one workgroup each, and the radix select becomes a
// chain of launches that meet in global memory, with digits of 12, 12 and 8 bits:
//   wide_pool   average pooling of the votes, scores stored, histogram of the first digit;
//   wide_hist   histogram of the second digit among the keys that match the first;
//   wide_last   per segment: how many keys lie above the 24 bits decided, and the 256-bin histogram of
//               the last digit among those that match them (also added up per head);
//   wide_emit   the counts of the earlier segments follow from what wide_last stored, so the ordered
//               compaction needs no pass of its own for them.
// Nothing waits inside a kernel; every workgroup re-derives the decided digits from the finished
// histograms.  What bounds it is the number of dependent launches (8 heads of 131072 scores are half a megabyte
// each): four of 1024 threads, 34 us, where digits of 8 bits, a count pass and a pooling pass apart took seven
// of 256 threads and 54 us.
constexpr int kWideThreads = 1024;
constexpr int kWidePer = 8;                           // positions per thread
constexpr int kWideSeg = kWideThreads * kWidePer;     // positions per workgroup
constexpr int kWideBins = 4096;                       // bins of the first two digits
constexpr int kWideHistWords = 3 * kWideBins + 2 * 256;   // per head: digit 1 (shared by the cuts), digit 2 per cut, digit 3 per cut
constexpr int kWideSegWords = 2 * 256 + 4;            // per segment: digit 3 per cut, keys above the 24 bits per cut

struct WideArgs {
  SelectArgs s;
  uint32_t* hist;        // [batch*Hkv][kWideHistWords], zero before wide_pool
  uint32_t* seg;         // [batch*Hkv][NSEG][kWideSegWords]
  int NSEG;
};

struct WideHead {
  int n, P, k_sel, b, g, bg;
  int64_t head_tok;
  bool all2;             // no second cut (no calibration size, or it covers every evicted token)
};

__device__ __forceinline__ WideHead wide_head(const SelectArgs& a, int bg) {
  WideHead h;
  h.bg = bg; h.g = bg % a.Hkv; h.b = bg / a.Hkv;
  int off0;
  h.n = seq_len_checked(a.seq_off, h.b, a.max_seq_len, a.total_tokens, off0);
  h.P = h.n - a.w; h.k_sel = a.B - a.w;
  h.head_tok = static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(h.g) * h.n;
  h.all2 = a.calib <= 0 || h.k_sel + a.calib >= h.P;
  return h;
}

struct WideShared {
  uint32_t tot[2][kWideThreads / 64];
  uint32_t digit[2][2], rem[2][2];       // [digit][cut]
};

// One 12-bit digit of both cuts from finished histograms (thread t holds bins 4t..4t+3): the bin in which the
// count from the top reaches `remaining`.  Called by the whole workgroup; `which` = 0, 1.
__device__ __forceinline__ void wide_digit(WideShared& sh, int which, int ncut, const u32x4 (&hb)[2], int shift, uint32_t (&prefix)[2],
                                           uint32_t (&remaining)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_index();
  uint32_t mine[2], inc[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    mine[c] = hb[c][0] + hb[c][1] + hb[c][2] + hb[c][3];
    inc[c] = wave_inclusive_scan(mine[c]);
    if (lane == 63) sh.tot[c][wv] = inc[c];
    if (tid == c) { sh.digit[which][c] = 0; sh.rem[which][c] = remaining[c]; }     // inconsistent histogram: the digit stays 0
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (c >= ncut) continue;
    uint32_t above = last_lane(inc[c]) - inc[c];
    for (int ww = wv + 1; ww < kWideThreads / 64; ++ww) above += sh.tot[c][ww];
    if (above < remaining[c] && remaining[c] <= above + mine[c]) {                   // exactly one thread
      uint32_t cum = above;
      int bin = 3;
      while (bin > 0 && cum + hb[c][bin] < remaining[c]) { cum += hb[c][bin]; --bin; }
      sh.digit[which][c] = 4 * tid + bin;
      sh.rem[which][c] = remaining[c] - cum;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    prefix[c] |= sh.digit[which][c] << shift;
    remaining[c] = sh.rem[which][c];
  }
}

// The first kDigits digits of both cuts.  The histograms are fetched together; only the scans depend on each other.
template <int kDigits>
__device__ __forceinline__ void wide_derive(const WideArgs& a, const WideHead& h, WideShared& sh, uint32_t (&prefix)[2],
                                            uint32_t (&remaining)[2]) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int ncut = h.all2 ? 1 : 2;
  const uint32_t* H = a.hist + static_cast<int64_t>(h.bg) * kWideHistWords;
  u32x4 h1[2], h2[2], h3[2];
  h1[0] = h1[1] = ld16(H + 4 * tid);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    h2[c] = h3[c] = zero16();
    if (kDigits > 1 && c < ncut) h2[c] = ld16(H + (1 + c) * kWideBins + 4 * tid);
    if (kDigits > 2 && c < ncut) h3[c] = ld16(H + 3 * kWideBins + c * 256 + 4 * lane);
  }
  prefix[0] = prefix[1] = 0;
  remaining[0] = h.k_sel;
  remaining[1] = h.k_sel + a.s.calib;
  wide_digit(sh, 0, ncut, h1, 20, prefix, remaining);
  if constexpr (kDigits > 1) wide_digit(sh, 1, ncut, h2, 8, prefix, remaining);
  if constexpr (kDigits > 2) {
    wide_pick(h3[0], 0, prefix[0], remaining[0]);
    if (ncut > 1) wide_pick(h3[1], 0, prefix[1], remaining[1]);
  }
}

// score[j] = (1/k) * sum_{d=-k/2..k/2} vote[j+d], zero outside [0, P), taps left to right; the votes of the row
// blocks are added first, always in the same order.
constexpr int kWideHalo = 64;            // widest half pooling width staged in LDS; wider ones read the votes where they are
__global__ __launch_bounds__(kWideThreads) void wide_pool_kernel(WideArgs a) {
  const SelectArgs& s = a.s;
  const WideHead h = wide_head(s, blockIdx.y);
  const int lo = blockIdx.x * kWideSeg;
  if (h.n <= s.B || lo >= h.P) return;
  const int tid = threadIdx.x;
  __shared__ float s_vote[kWideSeg + 2 * kWideHalo];
  __shared__ uint32_t s_hist[kWideBins];
  const float* vote = s.vote + h.head_tok;
  auto vote_at = [&](int j) {
    float val = 0.f;
    if (j >= 0 && j < h.P)
      for (int rb = 0; rb < s.NRB; ++rb) val += vote[rb * s.plane + j];
    return val;
  };
  const int half = s.pool_k / 2;
  const bool staged = half <= kWideHalo;
  if (staged)
    for (int t = tid; t < kWideSeg + 2 * half; t += kWideThreads) s_vote[t] = vote_at(lo - half + t);
  for (int t = tid; t < kWideBins; t += kWideThreads) s_hist[t] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kWidePer; ++q) {
    const int t = tid + q * kWideThreads, j = lo + t;
    if (j >= h.P) continue;
    float sum = 0.f;
    if (staged) for (int d = 0; d < s.pool_k; ++d) sum += s_vote[t + d];
    else for (int d = -half; d <= half; ++d) sum += vote_at(j + d);
    const float sc = sum / static_cast<float>(s.pool_k);
    s.score[h.head_tok + j] = sc;
    atomicAdd(&s_hist[__builtin_bit_cast(uint32_t, sc) >> 20], 1u);
  }
  __syncthreads();
  uint32_t* H = a.hist + static_cast<int64_t>(h.bg) * kWideHistWords;
  for (int t = tid; t < kWideBins; t += kWideThreads)
    if (const uint32_t v = s_hist[t]) atomicAdd(H + t, v);
}

__global__ __launch_bounds__(kWideThreads) void wide_hist_kernel(WideArgs a) {
  const WideHead h = wide_head(a.s, blockIdx.y);
  const int lo = blockIdx.x * kWideSeg;
  if (h.n <= a.s.B || lo >= h.P) return;
  const int tid = threadIdx.x;
  const uint32_t* gkey = reinterpret_cast<const uint32_t*>(a.s.score) + h.head_tok;
  uint32_t u[kWidePer];                 // issued first: in flight while the digit is derived
#pragma unroll
  for (int q = 0; q < kWidePer; ++q) { const int j = lo + tid + q * kWideThreads; u[q] = j < h.P ? gkey[j] : 0u; }
  __shared__ WideShared sh;
  __shared__ uint32_t s_hist[2][kWideBins];
  for (int t = tid; t < 2 * kWideBins; t += kWideThreads) (&s_hist[0][0])[t] = 0;
  uint32_t prefix[2], remaining[2];
  wide_derive<1>(a, h, sh, prefix, remaining);         // its barriers also publish the cleared histograms
  const int ncut = h.all2 ? 1 : 2;
  for (int c = 0; c < ncut; ++c)
#pragma unroll
    for (int q = 0; q < kWidePer; ++q)
      if (lo + tid + q * kWideThreads < h.P && (u[q] >> 20) == (prefix[c] >> 20)) atomicAdd(&s_hist[c][(u[q] >> 8) & 0xFFF], 1u);
  __syncthreads();
  uint32_t* H = a.hist + static_cast<int64_t>(h.bg) * kWideHistWords + kWideBins;
  for (int t = tid; t < ncut * kWideBins; t += kWideThreads)
    if (const uint32_t v = (&s_hist[0][0])[t]) atomicAdd(H + t, v);
}

__global__ __launch_bounds__(kWideThreads) void wide_last_kernel(WideArgs a) {
  const WideHead h = wide_head(a.s, blockIdx.y);
  const int lo = blockIdx.x * kWideSeg;
  if (h.n <= a.s.B || lo >= h.P) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t* gkey = reinterpret_cast<const uint32_t*>(a.s.score) + h.head_tok;
  uint32_t u[kWidePer];
#pragma unroll
  for (int q = 0; q < kWidePer; ++q) { const int j = lo + tid + q * kWideThreads; u[q] = j < h.P ? gkey[j] : 0u; }
  __shared__ WideShared sh;
  __shared__ uint32_t s_hist[2 * 256 + 2];             // digit 3 per cut, keys above the 24 bits per cut
  if (tid < 2 * 256 + 2) s_hist[tid] = 0;
  uint32_t prefix[2], remaining[2];
  wide_derive<2>(a, h, sh, prefix, remaining);         // its barriers also publish the cleared counters
  const int ncut = h.all2 ? 1 : 2;
  for (int c = 0; c < ncut; ++c) {
    uint32_t gt = 0;
#pragma unroll
    for (int q = 0; q < kWidePer; ++q)
      if (lo + tid + q * kWideThreads < h.P) {
        gt += (u[q] >> 8) > (prefix[c] >> 8) ? 1u : 0u;
        if ((u[q] >> 8) == (prefix[c] >> 8)) atomicAdd(&s_hist[c * 256 + (u[q] & 0xFF)], 1u);
      }
    gt = last_lane(wave_inclusive_scan(gt));
    if (lane == 0 && gt) atomicAdd(&s_hist[512 + c], gt);
  }
  __syncthreads();
  uint32_t* S = a.seg + (static_cast<int64_t>(h.bg) * a.NSEG + blockIdx.x) * kWideSegWords;
  uint32_t* H = a.hist + static_cast<int64_t>(h.bg) * kWideHistWords + 3 * kWideBins;
  if (tid < 2 * 256 + 2) {
    const uint32_t v = s_hist[tid];
    S[tid] = v;
    if (tid < ncut * 256 && v) atomicAdd(H + tid, v);
  }
}

__global__ __launch_bounds__(kWideThreads) void wide_emit_kernel(WideArgs a) {
  const SelectArgs& s = a.s;
  const WideHead h = wide_head(s, blockIdx.y);
  const int seg = blockIdx.x;
  const int lo = seg * kWideSeg;
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_index();
  int32_t* idx = s.indices + static_cast<int64_t>(h.bg) * s.B;
  int32_t* cal = (s.cal_indices && s.calib > 0) ? s.cal_indices + static_cast<int64_t>(h.bg) * s.calib : nullptr;
  if (seg == 0 && h.g == 0 && tid == 0) s.cache_lens[h.b] = min(h.n, s.B);
  if (h.n <= s.B) {                     // nothing to evict: keep every position
    if (seg == 0) {
      for (int r = tid; r < s.B; r += kWideThreads) idx[r] = (r < h.n) ? r : -1;
      if (cal) for (int r = tid; r < s.calib; r += kWideThreads) cal[r] = -1;
    }
    return;
  }
  if (seg == 0) {
    for (int r = tid; r < s.w; r += kWideThreads) idx[h.k_sel + r] = h.P + r;    // the window is always kept
    if (cal) {                                                                   // pad a short calibration set
      const int n_cal = min(s.calib, h.P - h.k_sel);
      for (int r = n_cal + tid; r < s.calib; r += kWideThreads) cal[r] = -1;
    }
  }
  if (lo >= h.P) return;
  const uint32_t* gkey = reinterpret_cast<const uint32_t*>(s.score) + h.head_tok;
  const int j0 = lo + tid * kWidePer;                  // this thread's positions
  uint32_t key[kWidePer];
#pragma unroll
  for (int u = 0; u < kWidePer; ++u) key[u] = j0 + u < h.P ? gkey[j0 + u] : 0u;
  __shared__ WideShared sh;
  __shared__ uint32_t s_pre[4];                        // greater1, equal1, greater2, equal2 of the earlier segments
  __shared__ uint32_t wave_tot[2][kWideThreads / 64];
  if (tid < 4) s_pre[tid] = 0;
  uint32_t prefix[2], remaining[2];
  wide_derive<3>(a, h, sh, prefix, remaining);         // its barriers also publish s_pre
  Cut c1, c2;
  c1.all = false; c1.thr = prefix[0]; c1.need_eq = remaining[0];
  c2.all = h.all2; c2.thr = h.all2 ? 0u : prefix[1]; c2.need_eq = h.all2 ? 0u : remaining[1];
  {
    uint32_t pre[4] = {0, 0, 0, 0};
    const int ncut = h.all2 ? 1 : 2;
    for (int sg = wv; sg < seg; sg += kWideThreads / 64) {      // a wave per earlier segment, four bins per lane
      const uint32_t* S = a.seg + (static_cast<int64_t>(h.bg) * a.NSEG + sg) * kWideSegWords;
      for (int c = 0; c < ncut; ++c) {
        const u32x4 v = ld16(S + c * 256 + 4 * lane);
        const uint32_t d3 = prefix[c] & 0xFF;
        if (lane == 0) pre[2 * c] += S[512 + c];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t bin = 4 * lane + q;
          if (bin > d3) pre[2 * c] += v[q];
          if (bin == d3) pre[2 * c + 1] += v[q];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t sum = last_lane(wave_inclusive_scan(pre[q]));
      if (lane == 0 && sum) atomicAdd(&s_pre[q], sum);
    }
  }
  constexpr uint32_t kAll = (1u << kWidePer) - 1u;
  const uint32_t valid = j0 >= h.P ? 0u : (h.P - j0 >= kWidePer ? kAll : (1u << (h.P - j0)) - 1u);
  uint32_t gtm1 = 0, eqm1 = 0, gtm2 = 0, eqm2 = 0;
#pragma unroll
  for (int u = 0; u < kWidePer; ++u) {
    gtm1 |= (key[u] > c1.thr ? 1u : 0u) << u;
    eqm1 |= (key[u] == c1.thr ? 1u : 0u) << u;
    gtm2 |= (key[u] > c2.thr ? 1u : 0u) << u;
    eqm2 |= (key[u] == c2.thr ? 1u : 0u) << u;
  }
  gtm1 &= valid; eqm1 &= valid; gtm2 &= valid; eqm2 &= valid;
  const uint32_t cnt1 = __popc(gtm1) + (static_cast<uint32_t>(__popc(eqm1)) << 16);      // at most 8192 in a segment
  const uint32_t cnt2 = __popc(gtm2) + (static_cast<uint32_t>(__popc(eqm2)) << 16);
  const uint32_t inc1 = wave_inclusive_scan(cnt1), inc2 = wave_inclusive_scan(cnt2);
  if (lane == 63) { wave_tot[0][wv] = inc1; wave_tot[1][wv] = inc2; }
  __syncthreads();
  uint32_t bef1 = inc1 - cnt1, bef2 = inc2 - cnt2;
  for (int ww = 0; ww < wv; ++ww) { bef1 += wave_tot[0][ww]; bef2 += wave_tot[1][ww]; }
  const uint32_t gt1 = s_pre[0] + (bef1 & 0xFFFFu), eq1 = s_pre[1] + (bef1 >> 16);
  const uint32_t gt2 = s_pre[2] + (bef2 & 0xFFFFu), eq2 = s_pre[3] + (bef2 >> 16);
  const uint32_t keepm = cut_members(c1, gtm1, eqm1, eq1, valid);
  const uint32_t calm = cut_members(c2, gtm2, eqm2, eq2, valid) & ~keepm;
  const uint32_t base1 = c1.rank(j0, gt1, eq1);
  {
    uint32_t pos = base1;
    for (uint32_t m = keepm; m; m &= m - 1u, ++pos) idx[pos] = j0 + (__ffs(m) - 1);
  }
  if (cal) {
    uint32_t pos = c2.rank(j0, gt2, eq2) - base1;
    for (uint32_t m = calm; m; m &= m - 1u, ++pos) cal[pos] = j0 + (__ffs(m) - 1);
  }
  // four neighbouring lanes hold the bytes of one bitmap word (bit = skip in the calibration pass; positions beyond
  // the prefix are marked)
  uint32_t w32 = ~calm & kAll;
#pragma unroll
  for (int q = 1; q < 4; ++q) w32 |= (__shfl_down(~calm, q) & kAll) << (q * kWidePer);
  if ((tid & 3) == 0 && j0 < h.P) s.bitmap[static_cast<int64_t>(h.bg) * s.W32 + (j0 >> 5)] = w32;
}

// The gather as a launch of its own: where no streaming pass or selection kernel carries it.
struct GatherOnlyArgs {
  GatherArgs g;
  const int32_t* seq_off;
  int64_t total_tokens;
  int Hkv, B, max_seq_len;
};
__global__ __launch_bounds__(256) void gather_kv_kernel(GatherOnlyArgs a) {
  const int bg = blockIdx.y;
  const int g = bg % a.Hkv, b = bg / a.Hkv;
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  gather_block(a.g, blockIdx.x, b, g, a.Hkv, a.B, n, off0);
}

// LDS variant for prefixes of up to PER * NT positions (NT = 1024 threads in use: smaller
// workgroups were measured slower, their staging and gather phases have too few threads).
// Thread t owns positions PER*t..PER*t+PER-1: their pooled scores live in its registers for the
// radix passes and the compaction.  PER = 32: their bits are exactly bitmap word t (prefixes up
// to 32768); PER = 16 / 8: half a word / a byte, so that prefixes up to 16384 / 8192 still keep
// every thread busy.  The votes are staged once in LDS
// (padded by one word per 32 so that the stride-32 accesses do not collide).
template <int NT, int PER>
__global__ __launch_bounds__(NT) void select_lds_kernel(SelectArgs a) {
  extern __shared__ uint32_t s_sel[];
  float* s_vote = reinterpret_cast<float*>(s_sel);
  int32_t* s_idx = reinterpret_cast<int32_t*>(s_sel);      // gather_here: the list, once the votes are done with
  const int bg = blockIdx.x;
  const int g = bg % a.Hkv;
  const int b = bg / a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_index();
  int off0;
  const int n = seq_len_checked(a.seq_off, b, a.max_seq_len, a.total_tokens, off0);
  int32_t* idx = a.indices + static_cast<int64_t>(bg) * a.B;
  int32_t* cal = (a.cal_indices && a.calib > 0) ? a.cal_indices + static_cast<int64_t>(bg) * a.calib : nullptr;
  if (g == 0 && tid == 0) a.cache_lens[b] = min(n, a.B);
  const int64_t head_tok = static_cast<int64_t>(off0) * a.Hkv + static_cast<int64_t>(g) * n;

  __shared__ __attribute__((aligned(16))) uint32_t s_hist[2][4][256];
  __shared__ uint32_t wave_tot[2][NT / 64];
  static_assert(PER == 32 || PER == 16 || PER == 8, "a thread owns a whole bitmap word, a half or a byte of one");
  auto pad = [](int j) { return j + (j >> 5); };

  if (n <= a.B) {                       // nothing to evict: keep every position
    for (int r = tid; r < a.B; r += NT) {
      idx[r] = (r < n) ? r : -1;
      if (a.gather_here && r < n) s_idx[r] = r;
    }
    if (cal) for (int r = tid; r < a.calib; r += NT) cal[r] = -1;
  } else {
    const int P = n - a.w;
    const int k_sel = a.B - a.w;
    for (int t = tid; t < 2 * 4 * 256; t += NT) (&s_hist[0][0][0])[t] = 0;
    // ---- stage the votes (row-block partials added first, fixed order) ---------------------
    {
      // 16 bytes per lane from the 16-byte boundary at or below the head's first vote (every vote
      // plane starts 256-byte aligned - the plane stride is a multiple of 64 floats - and a head
      // starts anywhere inside): vector v covers positions
      // 4v - shift .. 4v - shift + 3.  All loads of a thread are in flight together.
      const int64_t plane = a.plane;
      const int shift = static_cast<int>(head_tok & 3);
      const float* vsrc = a.vote + (head_tok - shift);
      f32x4 tmp[PER / 4];
#pragma unroll
      for (int u = 0; u < PER / 4; ++u) {
        const int v4 = tid + u * NT;
        f32x4 val = f32x4{0.f, 0.f, 0.f, 0.f};
        if (4 * v4 - shift < P) {
          val = *reinterpret_cast<const f32x4*>(vsrc + 4 * v4);
          for (int rb = 1; rb < a.NRB; ++rb) val += *reinterpret_cast<const f32x4*>(vsrc + rb * plane + 4 * v4);
        }
        tmp[u] = val;
      }
#pragma unroll
      for (int u = 0; u < PER / 4; ++u) {
        const int jb = 4 * (tid + u * NT) - shift;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int j = jb + x;
          if (j >= 0 && j < P) s_vote[pad(j)] = tmp[u][x];
        }
      }
      // the vectors end `shift` positions short of PER * NT: the last few of a full-length prefix
      const int jt = PER * NT - shift + tid;
      if (tid < shift && jt < P) {
        float val = a.vote[head_tok + jt];
        for (int rb = 1; rb < a.NRB; ++rb) val += a.vote[rb * plane + head_tok + jt];
        s_vote[pad(jt)] = val;
      }
    }
    __syncthreads();
    // ---- pooling: score[j] = (1/k) sum_{d=-k/2..k/2} vote[j+d], zeros outside [0, P), summed
    //      left to right at every position ------------------------------------------------------
    uint32_t key[PER];
    const int j0 = tid * PER;
    {
      // the thread's window of votes: w[x] = vote[j0 - half + x], zeros outside [0, P)
      const int half = a.pool_k / 2;
      const float kf = static_cast<float>(a.pool_k);
      float w[PER + kSelMaxPool - 1];
#pragma unroll
      for (int x = 0; x < PER + kSelMaxPool - 1; ++x) {
        const int jj = j0 - half + x;
        w[x] = (x < PER + a.pool_k - 1 && jj >= 0 && jj < P) ? s_vote[pad(jj)] : 0.f;
      }
      float sum[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) sum[u] = 0.f;
#pragma unroll
      for (int dd = 0; dd < kSelMaxPool; ++dd) {      // taps left to right
        if (dd < a.pool_k) {
#pragma unroll
          for (int u = 0; u < PER; ++u) sum[u] += w[u + dd];
        }
      }
#pragma unroll
      for (int u = 0; u < PER; ++u) key[u] = __builtin_bit_cast(uint32_t, sum[u] / kf);
      if (a.write_scores) {
        // pooled scores go out through LDS so that the global stores are coalesced
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (j0 + u < P) s_sel[pad(j0 + u)] = key[u];
        __syncthreads();
        float* dst = a.score + head_tok;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int j = tid + u * NT;
          if (j < P) dst[j] = __builtin_bit_cast(float, s_sel[pad(j)]);
        }
      }
    }
    auto each_key = [&](auto&& visit) {
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (j0 + u < P) visit(key[u]);
    };
    Cut c1, c2;                          // c1: retained prefix tokens; c2: retained + calibration set
    c1.all = false;
    radix_select(s_hist[0], k_sel, each_key, c1.thr, c1.need_eq);
    c2.all = a.calib <= 0 || k_sel + a.calib >= P;
    c2.thr = 0; c2.need_eq = 0;
    if (!c2.all) radix_select(s_hist[1], k_sel + a.calib, each_key, c2.thr, c2.need_eq);

    // ---- ordered compaction: exclusive scans of the per-thread (greater, equal) counts of
    //      both cuts, greater in the low half-word and equal in the high half-word -------------
    // per-thread bit masks over its PER positions: key above the threshold / equal to it
    constexpr uint32_t kAll = PER == 32 ? 0xFFFFFFFFu : (1u << (PER & 31)) - 1u;
    const uint32_t valid = j0 >= P ? 0u : (P - j0 >= PER ? kAll : (1u << ((P - j0) & 31)) - 1u);
    uint32_t gtm1 = 0, eqm1 = 0, gtm2 = 0, eqm2 = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      gtm1 |= (key[u] > c1.thr ? 1u : 0u) << u;
      eqm1 |= (key[u] == c1.thr ? 1u : 0u) << u;
      gtm2 |= (key[u] > c2.thr ? 1u : 0u) << u;
      eqm2 |= (key[u] == c2.thr ? 1u : 0u) << u;
    }
    gtm1 &= valid; eqm1 &= valid; gtm2 &= valid; eqm2 &= valid;
    const uint32_t cnt1 = __popc(gtm1) + (static_cast<uint32_t>(__popc(eqm1)) << 16);
    const uint32_t cnt2 = __popc(gtm2) + (static_cast<uint32_t>(__popc(eqm2)) << 16);
    const uint32_t inc1 = wave_inclusive_scan(cnt1), inc2 = wave_inclusive_scan(cnt2);
    if (lane == 63) { wave_tot[0][wv] = inc1; wave_tot[1][wv] = inc2; }
    __syncthreads();
    uint32_t bef1 = inc1 - cnt1, bef2 = inc2 - cnt2;
    for (int ww = 0; ww < wv; ++ww) { bef1 += wave_tot[0][ww]; bef2 += wave_tot[1][ww]; }
    const uint32_t gt1 = bef1 & 0xFFFFu, eq1 = bef1 >> 16, gt2 = bef2 & 0xFFFFu, eq2 = bef2 >> 16;
    const uint32_t keepm = cut_members(c1, gtm1, eqm1, eq1, valid);
    const uint32_t calm = cut_members(c2, gtm2, eqm2, eq2, valid) & ~keepm;
    // the cut's members are emitted in position order: a thread's first one lands at the number of
    // members at earlier positions
    const uint32_t base1 = c1.rank(j0, gt1, eq1);
    {
      uint32_t pos = base1;
      for (uint32_t m = keepm; m; m &= m - 1u, ++pos) {
        const int j = j0 + (__ffs(m) - 1);
        idx[pos] = j;
        if (a.gather_here) s_idx[pos] = j;
      }
    }
    if (cal) {
      uint32_t pos = c2.rank(j0, gt2, eq2) - base1;
      for (uint32_t m = calm; m; m &= m - 1u, ++pos) cal[pos] = j0 + (__ffs(m) - 1);
    }
    const uint32_t word = ~calm;            // bit = skip in the calibration pass
    if constexpr (PER == 32) {
      if (j0 < P) a.bitmap[static_cast<int64_t>(bg) * a.W32 + tid] = word;
    } else {
      // 32 / PER neighbouring lanes hold the pieces of one word (positions beyond the prefix were
      // marked "skip" above, so the pieces of idle threads are all ones)
      constexpr int LPW = 32 / PER;
      constexpr uint32_t kMask = (1u << PER) - 1u;
      uint32_t w32 = word & kMask;
#pragma unroll
      for (int q = 1; q < LPW; ++q) w32 |= (__shfl_down(word, q) & kMask) << (q * PER);
      if ((tid & (LPW - 1)) == 0 && j0 < P) a.bitmap[static_cast<int64_t>(bg) * a.W32 + (j0 >> 5)] = w32;
    }
    for (int r = tid; r < a.w; r += NT) {
      idx[k_sel + r] = P + r;
      if (a.gather_here) s_idx[k_sel + r] = P + r;
    }
    if (cal) {                                                              // pad a short calibration set
      const int n_cal = min(a.calib, P - k_sel);
      for (int r = n_cal + tid; r < a.calib; r += NT) cal[r] = -1;
    }
  }
  if (!a.gather_here) return;
  __syncthreads();
  const int len = min(n, a.B);
  const int c0 = a.gather.cache_off[b];
  const int cap = a.gather.cache_off[b + 1] - c0;
  if (cap < len) return;                 // capacity contract broken: write nothing
  // Two copies of K and of V in flight per thread keep the kernel for prefixes up to 8192 below 64 registers and two workgroups on
  // a compute unit: while one selects, the other copies.  480 heads of 300 rows 46 us with four copies, 34 us with two (42 us
  // with eight and one workgroup per unit); 280 heads of 1669 rows 145 / 139 / 141 us; 128 heads of 203 rows 14.7 / 15.4 / 15.0 us.
  constexpr int kCopies = 2;
  const int total = len * (a.gather.row_bytes / 16);
#pragma unroll 1
  for (int t0 = tid; t0 < total; t0 += kCopies * NT)
    gather_pieces<NT, kCopies>(a.gather, s_idx, t0, total, n, n <= a.B, head_tok,
                               static_cast<int64_t>(c0) * a.Hkv + static_cast<int64_t>(g) * cap);
}

}  // namespace cd
