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
constexpr int kSelPerThread = 32;              // LDS variant: most positions per thread (= one bitmap word)
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
static_assert(kGatherCopies == 1, "a workgroup of NT threads takes NT pieces");

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

// Workgroup `block` of those (NT threads each; a.blocks of them with 256) that gather the rows of one (sequence, KV head).
template <int NT = 256>
__device__ __forceinline__ void gather_block(const GatherArgs& a, int block, int b, int g, int Hkv, int B, int n, int off0) {
  const int len = min(n, B);
  const int c0 = a.cache_off[b];
  const int cap = a.cache_off[b + 1] - c0;
  if (cap < len) return;                 // capacity contract broken: write nothing
  gather_pieces<NT, kGatherCopies>(a, a.indices + (static_cast<int64_t>(b) * Hkv + g) * B,
                                    block * NT + static_cast<int>(threadIdx.x), len * (a.row_bytes / 16), n, n <= B,
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

// Sum of tot[0 .. wave - 1] of the workgroup's waves, in every lane (one LDS read and a scan; a loop over the waves waits
// for LDS once per wave).
template <int NT>
__device__ __forceinline__ uint32_t before_wave(const uint32_t* tot, int wave) {
  static_assert(NT / 64 <= 16, "the totals of one row of lanes");
  const int lane = threadIdx.x & 63;
  const uint32_t v = lane < wave ? tot[lane & 15] : 0u;
  return last_lane(wave_inclusive_scan(v));
}
// The same of tot[wave + 1 ..].
template <int NT>
__device__ __forceinline__ uint32_t after_wave(const uint32_t* tot, int wave) {
  static_assert(NT / 64 <= 16, "the totals of one row of lanes");
  const int lane = threadIdx.x & 63;
  const uint32_t v = lane > wave && lane < NT / 64 ? tot[lane & 15] : 0u;
  return last_lane(wave_inclusive_scan(v));
}

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

constexpr int kSelThreadWaves = kSelThreads / 64;
constexpr uint32_t kNoKey = 0x80000000u;               // scores have no sign: a key with this bit is no score
// First digit of the single-workgroup selection: its bits.  Scores crowd in few of its bins (a pooled vote rarely is more than
// an octave from the next), and lanes that add to one word of LDS do so one after the other: the more keys there are, the
// finer the digit (32768 keys within 6 % of each other: 4096 bins 26.8 us, 16384 bins 20.7 us).
__host__ __device__ constexpr int select_bits(int per) { return per == 2 ? 12 : per == 8 ? 13 : 14; }
// Words of its histogram; the first one behind the bins takes the keys that are no score.
__host__ __device__ constexpr int select_first_words(int per) { return (1 << select_bits(per)) + 16; }
// Keys of the bin the first digit ends in that are ranked against each other, instead of two more histograms (bits - 31 to 9,
// and the last 9) over all keys.
constexpr int kSelFewKeys = 256;
constexpr int kSelLastBits = 9;
__host__ __device__ constexpr int select_later_words(int per) { return (1 << (31 - select_bits(per) - kSelLastBits)) + (1 << kSelLastBits); }
static_assert(kSelThreads == 4 * kSelFewKeys && kSelFewKeys % 64 == 0, "four threads a key, sixteen keys a step");
static_assert(2 * kSelFewKeys <= select_later_words(32), "the few keys and their ranks take the place of the later histograms");
__host__ __device__ constexpr int select_hist_words(int per) { return select_first_words(per) + select_later_words(per); }
// Short prefixes: histograms beside the votes, cleared while those are on their way; longer ones: in their place once they
// are pooled, so that two workgroups for 16384 positions fit a compute unit.
__host__ __device__ constexpr bool select_own_hist(int per) { return per <= 8; }
struct SelectShared {
  uint32_t wave_tot[2][kSelThreadWaves];
  uint32_t digit, rem, in_bin, few;
};

template <int NT>
__device__ __forceinline__ void clear_hist(uint32_t* hist, int words, int tid) {
#pragma unroll
  for (int t = tid; t < words / 4; t += NT) *reinterpret_cast<u32x4*>(hist + 4 * t) = zero16();
}

// Where chunk q (16 bytes) of the staged row lies: rows of 16 chunks, rotated by exclusive or, so that both consecutive
// chunks (staging) and chunks PER / 4 apart (windows) of sixteen neighbouring lanes are in different banks.
__device__ __forceinline__ int select_chunk(int q) { return q ^ ((q >> 4) & 15); }
// Slot s of the staged row holds vote s - shift - kSelFront, shift = the head's first vote modulo 4: 16-byte pieces of memory
// are chunks of the row.
constexpr int kSelFront = 8;                           // zeros ahead: two chunks, at least half the widest pooling
static_assert(kSelFront % 4 == 0 && kSelFront >= kSelMaxPool / 2, "the first window starts in the row");
// Chunks a thread's window takes, wherever in a chunk it starts.
__host__ __device__ constexpr int select_window_chunks(int per) { return (per + kSelMaxPool - 1 + 3 + 3) / 4; }
// Bytes of the staged row of a prefix of up to P positions (what the windows read, whole rows of chunks) and of the histograms
// where they take its place.
__host__ __device__ constexpr size_t select_row_bytes(int P, int per) {
  const size_t row = static_cast<size_t>((P - 1 + kSelFront + 3) / 4 + select_window_chunks(per) + 15) / 16 * 16 * 16;
  const size_t hist = select_own_hist(per) ? 0 : select_hist_words(per) * sizeof(uint32_t);
  return row > hist ? row : hist;
}

// The bin of a finished histogram in which the count from the top reaches `remaining`; `remaining` becomes the rank inside it,
// `in_bin` its count.  Thread t looks at bins BPT t .. BPT t + BPT - 1.
template <int NT, int BPT>
__device__ __forceinline__ uint32_t pick_digit(SelectShared& sh, const uint32_t* hist, int bins, uint32_t& remaining, uint32_t& in_bin) {
  constexpr int kChunks = BPT / 4;                             // of 16 bytes
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_index();
  uint32_t mine = 0;
  if (BPT * tid < bins) {
#pragma unroll
    for (int q = 0; q < kChunks; ++q) {                         // sixteen lanes start with different chunks: all banks at once
      const u32x4 c = ld16(hist + BPT * tid + 4 * ((q + tid / (16 / kChunks)) % kChunks));
      mine += (c[0] + c[1]) + (c[2] + c[3]);
    }
  }
  const uint32_t inc = wave_inclusive_scan(mine);
  if (lane == 63) sh.wave_tot[0][wv] = inc;
  if (tid == 0) { sh.digit = 0; sh.rem = remaining; sh.in_bin = ~0u; sh.few = 0; }      // never left so by a consistent histogram
  __syncthreads();
  const uint32_t above = last_lane(inc) - inc + after_wave<NT>(sh.wave_tot[0], wv);
  if (above < remaining && remaining <= above + mine) {         // exactly one thread
    u32x4 c[kChunks];
#pragma unroll
    for (int q = 0; q < kChunks; ++q) c[q] = ld16(hist + BPT * tid + 4 * q);
    uint32_t cum = above, cnt = 0;
    int bin = BPT;
#pragma unroll
    for (int x = BPT - 1; x >= 0; --x)
      if (cum + cnt < remaining) { cum += cnt; cnt = c[x / 4][x % 4]; bin = x; }
    sh.digit = BPT * tid + bin;
    sh.rem = remaining - cum;
    sh.in_bin = cnt;
  }
  __syncthreads();
  remaining = sh.rem;
  in_bin = sh.in_bin;
  return sh.digit;
}

// Radix select of the `rank`-th largest key (rank >= 1, at most the number of keys).
// `for_each_key(visit)` must call visit(u) once for every key this thread owns; keys with kNoKey are none.  On return
// thr = that key's bit pattern and need_eq = how many keys equal to thr lie within the rank.
// `hist`: zero, with a barrier since it was cleared.  Must be called by every thread of the workgroup.
// kSecond: another rank of the same keys; the histogram of the first digit is still there.
template <int NT, int PER, bool kSecond, typename ForEach>
__device__ __forceinline__ void radix_select(uint32_t* hist, SelectShared& sh, uint32_t rank, ForEach&& for_each_key, uint32_t& thr,
                                             uint32_t& need_eq) {
  constexpr int kBits = select_bits(PER), kLow = 31 - kBits, kLater = select_later_words(PER);      // kLow: bits below the first digit
  const int tid = threadIdx.x;
  uint32_t remaining = rank;      // rank of the answer among the keys matching the bits decided so far
  uint32_t in_bin;
  if constexpr (!kSecond)
    for_each_key([&](uint32_t u) __attribute__((always_inline)) { atomicAdd(&hist[u >> kLow], 1u); });
  __syncthreads();                // second: everyone has read what the first left in `sh`
  uint32_t prefix = pick_digit<NT, (1 << kBits) / NT>(sh, hist, 1 << kBits, remaining, in_bin) << kLow;
  uint32_t* h = hist + select_first_words(PER);
  auto clear_again = [&]() {
    if constexpr (kSecond) {
      for (int t = tid; t < kLater; t += NT) h[t] = 0u;
      __syncthreads();
    }
  };
  if (in_bin <= kSelFewKeys) {
    // the keys of the bin in any order, then for each how many are greater, and how many greater or equal (high half): thread t
    // counts for key t modulo 256 over every fourth group of four keys
    uint32_t* list = h;
    uint32_t* ranks = h + kSelFewKeys;
    clear_again();
    for_each_key([&](uint32_t u) __attribute__((always_inline)) {
      if ((u ^ prefix) < (1u << kLow)) list[atomicAdd(&sh.few, 1u)] = (u ^ prefix) + 1u;       // 0: none
    });
    __syncthreads();
    const uint32_t me = tid % kSelFewKeys;
    uint32_t own = 0;
    if (wave_index() % (kSelFewKeys / 64) * 64u < in_bin) {
      own = list[me];
      uint32_t higher = 0, reach = 0;
      for (uint32_t j = 0; j < in_bin; j += 64) {                // four groups in flight; zeros behind the last key
        u32x4 o[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) o[x] = ld16(list + j + 16 * x + 4 * (tid / kSelFewKeys));
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int q = 0; q < 4; ++q) { higher += o[x][q] > own ? 1u : 0u; reach += o[x][q] >= own ? 1u : 0u; }
      }
      if (me < in_bin) atomicAdd(&ranks[me], higher | (reach << 16));
    }
    __syncthreads();
    if (tid < kSelFewKeys && me < in_bin) {
      const uint32_t r = ranks[me], higher = r & 0xFFFFu, reach = r >> 16;
      if (higher < remaining && remaining <= reach) { sh.digit = own - 1u; sh.rem = remaining - higher; }      // equal keys write the same
    }
    __syncthreads();
    thr = prefix | sh.digit;
    need_eq = sh.rem;
    return;
  }
  clear_again();
#pragma unroll 1                  // one copy of the code: fetching it costs more than the loop
  for (int pass = 0; pass < 2; ++pass) {
    const int bins = pass ? 1 << kSelLastBits : 1 << (kLow - kSelLastBits), shift = pass ? 0 : kSelLastBits, decided = pass ? kSelLastBits : kLow;
    for_each_key([&](uint32_t u) __attribute__((always_inline)) {
      if (((u ^ prefix) >> decided) == 0) atomicAdd(&h[(u >> shift) & (bins - 1)], 1u);
    });
    __syncthreads();
    prefix |= pick_digit<NT, 4>(sh, h, bins, remaining, in_bin) << shift;
    h += bins;
  }
  thr = prefix;
  need_eq = remaining;
}

// s / k for an odd k up to kSelMaxPool, rounded as the division rounds it: one correction of s times the rounded reciprocal
// (a test compares every 24-bit significand for every such k).  Sums outside 2^-100 .. 2^100 other than 0 - their
// remainders may leave the range - and what is no number are for the division itself.
__host__ __device__ __forceinline__ float divide_small(float s, float k, float rk) {
  const float q = s * rk;
  return fmaf(fmaf(-k, q, s), rk, q);
}
constexpr uint32_t kDivideLow = 27u << 23, kDivideHigh = 227u << 23;      // bit patterns of 2^-100 and 2^100

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
// each) and, inside them, of dependent trips to memory and LDS: four of 1024 threads, 25 us (10.6 + 4.4 + 5.6 + 10.6 = 31 us
// while the pooling fetched its votes word by word and its taps one after the other, and the totals of the waves were
// added up in loops; digits of 8 bits, a count pass and a pooling pass apart took seven launches of 256 threads and 54 us).
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
    const uint32_t above = last_lane(inc[c]) - inc[c] + after_wave<kWideThreads>(sh.tot[c], wv);
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
  __shared__ __attribute__((aligned(16))) float s_vote[kWideSeg + 2 * kWideHalo + 8];
  __shared__ uint32_t s_hist[kWideBins];
  const float* vote = s.vote + h.head_tok;
  const int half = s.pool_k / 2;
  const bool staged = half <= kWideHalo;
  float sum[kWidePer];
#pragma unroll
  for (int q = 0; q < kWidePer; ++q) sum[q] = 0.f;
  for (int t = tid; t < kWideBins; t += kWideThreads) s_hist[t] = 0;
  if (staged) {
    // 16 bytes per lane from the 16-byte boundary at or below the first vote of the first window (planes start 256-byte
    // aligned), all of a thread's on their way together; vectors that hold no vote of the head are not loaded
    const int64_t first = h.head_tok + lo - half;
    const int shift = static_cast<int>(first & 3);
    const float* src = s.vote + (first - shift);
    constexpr int kVec = (kWideSeg + 2 * kWideHalo + 6 + 4 * kWideThreads - 1) / (4 * kWideThreads);
    f32x4 tmp[kVec];
#pragma unroll
    for (int u = 0; u < kVec; ++u) tmp[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int count = (kWideSeg + 2 * half + shift + 3) / 4;
    for (int rb = 0; rb < s.NRB; ++rb)
#pragma unroll
      for (int u = 0; u < kVec; ++u) {
        const int v4 = tid + u * kWideThreads, j = lo - half - shift + 4 * v4;
        if (v4 < count && j + 3 >= 0 && j < h.P) tmp[u] += *reinterpret_cast<const f32x4*>(src + rb * s.plane + 4 * v4);
      }
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const int v4 = tid + u * kWideThreads, j = lo - half - shift + 4 * v4;
#pragma unroll
      for (int x = 0; x < 4; ++x) tmp[u][x] = (j + x >= 0 && j + x < h.P) ? tmp[u][x] : 0.f;
      if (v4 < count) *reinterpret_cast<f32x4*>(s_vote + 4 * v4) = tmp[u];
    }
    __syncthreads();
    for (int d = 0; d < s.pool_k; ++d)                 // taps left to right, eight positions side by side
#pragma unroll
      for (int q = 0; q < kWidePer; ++q) sum[q] += s_vote[shift + tid + q * kWideThreads + d];
  } else {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kWidePer; ++q) {
      const int j = lo + tid + q * kWideThreads;
      if (j >= h.P) continue;
      for (int i = max(j - half, 0); i <= min(j + half, h.P - 1); ++i) {
        float val = 0.f;
        for (int rb = 0; rb < s.NRB; ++rb) val += vote[rb * s.plane + i];
        sum[q] += val;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kWidePer; ++q) {
    const int j = lo + tid + q * kWideThreads;
    if (j >= h.P) continue;
    const float sc = sum[q] / static_cast<float>(s.pool_k);
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
  // a wave per earlier segment, four bins of its last digit per lane; the first one's on their way while the digits are derived
  const int ncut = h.all2 ? 1 : 2;
  u32x4 bins[2];
  uint32_t upper[2];
  auto fetch = [&](int sg) __attribute__((always_inline)) {
    const uint32_t* S = a.seg + (static_cast<int64_t>(h.bg) * a.NSEG + sg) * kWideSegWords;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bins[c] = c < ncut ? ld16(S + c * 256 + 4 * lane) : zero16();
      upper[c] = c < ncut ? S[512 + c] : 0u;
    }
  };
  if (wv < seg) fetch(wv);
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
    for (int sg = wv; sg < seg; sg += kWideThreads / 64) {
      if (sg != wv) fetch(sg);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint32_t d3 = prefix[c] & 0xFF;
        if (lane == 0) pre[2 * c] += upper[c];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t bin = 4 * lane + q;
          if (bin > d3) pre[2 * c] += bins[c][q];
          if (bin == d3) pre[2 * c + 1] += bins[c][q];
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
  const uint32_t bef1 = inc1 - cnt1 + before_wave<kWideThreads>(wave_tot[0], wv), bef2 = inc2 - cnt2 + before_wave<kWideThreads>(wave_tot[1], wv);
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
// radix passes and the compaction.  PER = 32 covers prefixes up to 32768; 16, 8 and 2 are there so that
// shorter ones (16384, 8192, 2048) still keep every thread busy.
// What bounds it is instruction issue on the one compute unit a head has: each of the 16 waves spends its instructions per key
// in every pass over the keys, some 500 cycles per instruction and pass at 32768 keys.  Hence one wide first digit counted with
// plain LDS atomics and the few keys of its bin ranked directly (four 8-bit digits with run-length compressed counts before),
// windows read 16 bytes at a time from a zero-padded row, a three-instruction division, waves without positions that skip
// all of it, and a second cut only where there is one.  Eight heads, four digits / now, us: 8192 scores 10.0 / 7.5, 16000
// 13.8 / 11.4, 32768 21.5 / 15.8; two heads of 512 8.6 / 5.1; the same with all scores within 6 % of each other 10.1 / 9.2, 14.3 /
// 14.0, 22.2 / 20.7, 8.6 / 5.7; 512 heads of 14000 with the gather of 1024 rows 110 / 98 (two workgroups on a compute unit).
template <int NT, int PER>
__global__ __launch_bounds__(NT) void select_lds_kernel(SelectArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t s_sel[];
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

  constexpr bool kOwnHist = select_own_hist(PER);
  __shared__ __attribute__((aligned(16))) uint32_t s_own[kOwnHist ? select_hist_words(PER) : 4];
  __shared__ SelectShared sh;
  uint32_t* hist = kOwnHist ? s_own : s_sel;

  if (n <= a.B) {                       // nothing to evict: keep every position
    for (int r = tid; r < a.B; r += NT) {
      idx[r] = (r < n) ? r : -1;
      if (a.gather_here && r < n) s_idx[r] = r;
    }
    if (cal) for (int r = tid; r < a.calib; r += NT) cal[r] = -1;
  } else {
    const int P = n - a.w;
    const int k_sel = a.B - a.w;
    const int half = a.pool_k / 2;
    // ---- stage the votes (row-block partials added first, fixed order) into the zero-padded row.  16 bytes per lane from the
    // 16-byte boundary at or below the head's first vote (every vote plane starts 256-byte aligned - the plane stride is a
    // multiple of 64 floats - and a head starts anywhere inside).  All loads of a thread are in flight together.
    const int shift = static_cast<int>(head_tok & 3);
    const float* vsrc = a.vote + (head_tok - shift);
    const int nvec = (P + shift + half + 3) / 4;           // behind the prefix: zeros for the last windows
    constexpr int kVec = PER >= 4 ? PER / 4 + 1 : 1;       // (P + 3 + 7 + 3) / 4 <= NT * kVec
    static_assert(static_cast<int64_t>(NT) * kVec * 4 >= static_cast<int64_t>(NT) * PER + 13, "a thread stages kVec chunks");
    {
      f32x4 tmp[kVec];
#pragma unroll
      for (int u = 0; u < kVec; ++u) tmp[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int rb = 0; rb < a.NRB; ++rb) {
        const float* src = vsrc + rb * a.plane;
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
          const int v4 = tid + u * NT;
          if (4 * v4 - shift < P) tmp[u] += *reinterpret_cast<const f32x4*>(src + 4 * v4);
        }
      }
      if constexpr (kOwnHist) clear_hist<NT>(hist, select_hist_words(PER), tid);
      if (tid < kSelFront / 4) *reinterpret_cast<u32x4*>(s_sel + 4 * select_chunk(tid)) = zero16();
#pragma unroll
      for (int u = 0; u < kVec; ++u) {
        const int v4 = tid + u * NT, first = 4 * v4 - shift;
        if (first < 0 || first + 4 > P) {                  // both ends: neighbouring heads' votes, words that are none
#pragma unroll
          for (int x = 0; x < 4; ++x) tmp[u][x] = (first + x >= 0 && first + x < P) ? tmp[u][x] : 0.f;
        }
        if (v4 < nvec) *reinterpret_cast<f32x4*>(s_sel + 4 * select_chunk(v4 + kSelFront / 4)) = tmp[u];
      }
    }
    __syncthreads();
    // ---- pooling: score[j] = (1/k) sum_{d=-k/2..k/2} vote[j+d], zeros outside [0, P), summed
    //      left to right at every position.  Positions beyond the prefix get a key that matches no digit. ---------------
    uint32_t key[PER];
    const int j0 = tid * PER;
    const bool busy = wv * (64 * PER) < P;         // same in every lane: this wave has positions
#pragma unroll
    for (int u = 0; u < PER; ++u) key[u] = kNoKey;
    if (busy) {
      constexpr int kWin = select_window_chunks(PER);
      float w[4 * kWin];
      // the window of position j starts in slot j + shift + kSelFront - half; a lane without positions takes the last one's
      const int slot0 = min(j0, (P - 1) / PER * PER) + shift + kSelFront - half;
#pragma unroll
      for (int x = 0; x < kWin; ++x)
        *reinterpret_cast<f32x4*>(&w[4 * x]) = *reinterpret_cast<const f32x4*>(s_sel + 4 * select_chunk(slot0 / 4 + x));
      // where in its chunk a window starts is the same in all lanes, with two positions a thread for all odd and all even ones
      const int o = slot0 & 3;
      if (PER == 2 ? (o & 1) != 0 : (__builtin_amdgcn_readfirstlane(o) & 1) != 0) {
#pragma unroll
        for (int x = 0; x + 1 < 4 * kWin; ++x) w[x] = w[x + 1];
      }
      if (PER == 2 ? (o & 2) != 0 : (__builtin_amdgcn_readfirstlane(o) & 2) != 0) {
#pragma unroll
        for (int x = 0; x + 2 < 4 * kWin; ++x) w[x] = w[x + 2];
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
      const float kf = static_cast<float>(a.pool_k), rk = 1.f / kf;
      uint32_t top = 0, low = ~0u;                   // bit patterns; less one, so that 0 is no low one
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        top = max(top, __builtin_bit_cast(uint32_t, sum[u]));
        low = min(low, __builtin_bit_cast(uint32_t, sum[u]) - 1u);
      }
      const bool whole = (wv + 1) * (64 * PER) <= P;      // same in every lane
      if (whole && __all(top < kDivideHigh && low >= kDivideLow)) {
#pragma unroll
        for (int u = 0; u < PER; ++u) key[u] = __builtin_bit_cast(uint32_t, divide_small(sum[u], kf, rk));
      } else {
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (j0 + u < P) key[u] = __builtin_bit_cast(uint32_t, sum[u] / kf) & ~kNoKey;
      }
      if (a.write_scores) {
        uint32_t* dst = reinterpret_cast<uint32_t*>(a.score) + head_tok;
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (j0 + u < P) dst[j0 + u] = key[u];
      }
    }
    if constexpr (!kOwnHist) {
      __syncthreads();
      clear_hist<NT>(hist, select_hist_words(PER), tid);
      __syncthreads();
    }
    auto each_key = [&](auto&& visit) __attribute__((always_inline)) {
      if (!busy) return;
#pragma unroll
      for (int u = 0; u < PER; ++u) visit(key[u]);
    };
    Cut c1, c2;                          // c1: retained prefix tokens; c2: retained + calibration set
    c1.all = false;
    radix_select<NT, PER, false>(hist, sh, k_sel, each_key, c1.thr, c1.need_eq);
    c2.all = a.calib <= 0 || k_sel + a.calib >= P;
    c2.thr = 0; c2.need_eq = 0;
    if (!c2.all) radix_select<NT, PER, true>(hist, sh, k_sel + a.calib, each_key, c2.thr, c2.need_eq);

    // ---- ordered compaction: exclusive scans of the per-thread (greater, equal) counts of
    //      both cuts, greater in the low half-word and equal in the high half-word -------------
    // per-thread bit masks over its PER positions: key above the threshold / equal to it
    constexpr uint32_t kAll = PER == 32 ? 0xFFFFFFFFu : (1u << (PER & 31)) - 1u;
    const uint32_t valid = j0 >= P ? 0u : (P - j0 >= PER ? kAll : (1u << ((P - j0) & 31)) - 1u);
    auto masks = [&](uint32_t thr, uint32_t& gtm, uint32_t& eqm) __attribute__((always_inline)) {
      gtm = eqm = 0;
      if (!busy) return;
#pragma unroll
      for (int u = PER - 1; u >= 0; --u) {           // the sign of a difference is shifted in from below
        gtm = __builtin_amdgcn_alignbit(gtm, thr - key[u], 31);
        eqm = __builtin_amdgcn_alignbit(eqm, key[u] - thr, 31);
      }
      gtm &= valid;
      eqm = ~(gtm | eqm) & valid;                    // eqm held the smaller ones
    };
    uint32_t gtm1, eqm1, gtm2 = 0, eqm2 = 0;
    masks(c1.thr, gtm1, eqm1);
    const uint32_t cnt1 = __popc(gtm1) + (static_cast<uint32_t>(__popc(eqm1)) << 16);
    const uint32_t inc1 = wave_inclusive_scan(cnt1);
    uint32_t cnt2 = 0, inc2 = 0;
    if (!c2.all) {
      masks(c2.thr, gtm2, eqm2);
      cnt2 = __popc(gtm2) + (static_cast<uint32_t>(__popc(eqm2)) << 16);
      inc2 = wave_inclusive_scan(cnt2);
    }
    if (lane == 63) { sh.wave_tot[0][wv] = inc1; sh.wave_tot[1][wv] = inc2; }
    __syncthreads();
    const uint32_t bef1 = inc1 - cnt1 + before_wave<NT>(sh.wave_tot[0], wv), bef2 = inc2 - cnt2 + before_wave<NT>(sh.wave_tot[1], wv);
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
    // the bitmap (bit = skip in the calibration pass; positions beyond the prefix are marked), whole words of it: every
    // thread stores the word, half or byte it owns, with 2 positions a thread every fourth one the byte of four
    if (wv * (64 * PER) < ((P + 31) & ~31)) {
      uint32_t word = ~calm;
      void* bits = a.bitmap + static_cast<int64_t>(bg) * a.W32;
      const bool mine = j0 < ((P + 31) & ~31);
      if constexpr (PER == 32) {
        if (mine) static_cast<uint32_t*>(bits)[tid] = word;
      } else if constexpr (PER == 16) {
        if (mine) static_cast<uint16_t*>(bits)[tid] = static_cast<uint16_t>(word);
      } else if constexpr (PER == 8) {
        if (mine) static_cast<uint8_t*>(bits)[tid] = static_cast<uint8_t>(word);
      } else {
        static_assert(PER == 2, "a thread owns a bitmap word, a half, a byte or two bits");
        word &= 3u;
        word |= __shfl_down(word, 1) << 2;
        word |= __shfl_down(word, 2) << 4;
        if (mine && (tid & 3) == 0) static_cast<uint8_t*>(bits)[tid / 4] = static_cast<uint8_t>(word);
      }
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
