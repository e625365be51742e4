// Saliency and recompute selection (Sec. 3.1 Eq. 1, applied per token against
// its cached input; Sec. 3.3 saliency mask with k = ceil(r L) tokens).
//
// saliency_rows: one wave per token row loads x and xref with 16-byte
//   non-temporal loads (all of a lane's loads issued before the first is
//   used) and accumulates
//   |x - xref| and |xref| in fp64 (exact per-element differences, so only the
//   summation order differs from the definition).
//   Writes s_i = fp32(w_frame * num / (den + xi)) plus, per workgroup of four
//   rows, the sums of num and of den for the step-level value.
// step_delta_sum: step-level Eq. 1 sum of those in a fixed order
//   (deterministic); in echo_select the same sum runs as a second workgroup of
//   select_rows.
// select_rows: one 1024-thread workgroup, the keys held in registers
//   (1) top-K threshold key by a radix select over order-preserving uint32
//       keys in digits of 11, 11 and 10 bits (histograms in LDS);
//   (2) stable compaction in index order: per (1024-key round, wave) counts,
//       one block-wide exclusive scan, then the lane's place within each wave
//       from ballots; ties at the threshold key go to the lowest indices.
// The key set is tiny (4 bytes per token, L2-resident), so one workgroup keeps
// the selection exact and deterministic.  One CU's issue rate is what bounds it:
// 32760 keys are 32 per thread and every instruction per key costs 0.2 us, so the
// passes are kept to a few (a shift and an LDS add in the first, a subtract and a
// compare for the keys outside the digit in the others; a wave's counts in its lanes).
// Four passes of 8 bits with a leader election per 64 keys and a count written
// per (round, wave) took 36.5 us at 32760 keys, this form 24.7; at 75600 keys 147 and 62.6.
// Adds of many lanes to one address follow one another (2 cycles each), which
// matters where most keys tie, as they do over silent frames and unchanged
// tokens: 32760 equal keys took 76 us with a plain add per key, 25 with the
// rules at the digits below (39 with the four passes).
// select_small: saliency, step-level sum and selection of few tokens, one launch.
// select_segments: the same selection per anchor segment, one workgroup per
//   segment (the two-stage form: anchor segments, then min(k, N) tokens each).
// anchor_select: the anchor segments (top-k of per-segment keys, or evenly
//   spaced), one workgroup.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace echo {

constexpr int kSalThreads = 256;
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;

// MAXC > 0: a lane's MAXC chunks of 8 elements of x and xref are all loaded
// before any is used (D <= 512 MAXC); MAXC == 0 streams the row (any D).
template <typename T, int MAXC>
__global__ void __launch_bounds__(kSalThreads)
saliency_rows(const T* __restrict__ x, const T* __restrict__ xref, const float* __restrict__ fw,
              int L, int N, int D, double xi, float* __restrict__ s_out,
              double* __restrict__ num_out, double* __restrict__ den_out) {
  __shared__ double part[2][kSalThreads / kWave];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * (kSalThreads / kWave) + wave;
  const int64_t row = row0 < L ? row0 : L - 1;  // past the end: the last row again, not counted
  const T* xr = x + row * D;
  const T* rr = xref + row * D;
  const int nch = D / 8;
  double num = 0.0, den = 0.0;
  auto add8 = [&](const Raw8<T>& a, const Raw8<T>& b) __attribute__((always_inline)) {
    float fa[8], fb[8];
    a.unpack(fa);
    b.unpack(fb);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double da = fa[j], db = fb[j];
      num += fabs(da - db);
      den += fabs(db);
    }
  };
  if (MAXC > 0) {
    constexpr int R = MAXC > 0 ? MAXC : 1;
    Raw8<T> ra[R], rb[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int c = lane + u * kWave;
      const int cc = c < nch ? c : nch - 1;  // past the row end: in-bounds re-load, not added
      ra[u].load_nt(xr + cc * 8);
      rb[u].load_nt(rr + cc * 8);
    }
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (lane + u * kWave < nch) add8(ra[u], rb[u]);
  } else {
    for (int c = lane; c < nch; c += kWave) {
      Raw8<T> a, b;
      a.load(xr + c * 8);
      b.load(rr + c * 8);
      add8(a, b);
    }
  }
  num = wave_sum(num);
  den = wave_sum(den);
  if (lane == 0) {
    if (row0 < L) {
      const double delta = num / (den + xi);
      const double w = static_cast<double>(fw[row / N]);
      s_out[row] = __double2float_rn(w * delta);
    }
    part[0][wave] = row0 < L ? num : 0.0;
    part[1][wave] = row0 < L ? den : 0.0;
  }
  __syncthreads();
  // one pair of sums per workgroup: a quarter of the rows' pairs, which one
  // workgroup adds up beside the selection
  if (threadIdx.x < 2) {
    double t = part[threadIdx.x][0];
#pragma unroll
    for (int w = 1; w < kSalThreads / kWave; ++w) t += part[threadIdx.x][w];
    (threadIdx.x == 0 ? num_out : den_out)[blockIdx.x] = t;
  }
}

// Step-level Eq. 1 value sum(num) / (sum(den) + xi) in a fixed summation
// order (deterministic), by one 1024-thread workgroup: its own kernel after a
// saliency-only call, or the second workgroup of the select_rows launch.
// num, den: n partial sums.
__device__ __forceinline__ void step_delta_block(const double* __restrict__ num, const double* __restrict__ den,
                                                 int n, double xi, double* __restrict__ step_delta) {
  __shared__ double red_n[kSelWaves], red_d[kSelWaves];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  double a = 0.0, b = 0.0;
  // unrolled so that eight loads of each array are in flight; the additions
  // keep their order
#pragma unroll 8
  for (int i = tid; i < n; i += kSelThreads) {
    a += num[i];
    b += den[i];
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane == 0) {
    red_n[wave] = a;
    red_d[wave] = b;
  }
  __syncthreads();
  if (tid == 0) {
    double sa = 0.0, sb = 0.0;
    for (int w = 0; w < kSelWaves; ++w) {
      sa += red_n[w];
      sb += red_d[w];
    }
    *step_delta = sa / (sb + xi);
  }
}

__global__ void __launch_bounds__(kSelThreads)
step_delta_sum(const double* __restrict__ num, const double* __restrict__ den, int n, double xi,
               double* __restrict__ step_delta) {
  step_delta_block(num, den, n, xi, step_delta);
}

// Order-preserving key: larger float -> larger key; NaN above everything; -0 == +0.
// No float has a key below 0x007fffff (-inf), so 0 stands for "no key".
__device__ __forceinline__ uint32_t rank_key(float s) {
  const uint32_t u = __float_as_uint(s);
  const uint32_t k = u ^ (static_cast<uint32_t>(static_cast<int32_t>(u) >> 31) | 0x80000000u);
  return s != s ? 0xffffffffu : (u == 0x80000000u ? 0x80000000u : k);
}

// lanes of `mask` below this one
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// LDS of one selection
struct TopkLds {
  alignas(16) uint32_t h1[2048 * 4];  // digit 1, four copies side by side (a lane uses copy lane % 4): the keys of a
                          // step lie in a few octaves, so that most lanes of a wave meet in a few bins
  uint32_t h2[2048], h3[1024];
  uint32_t digit[3], above[3], in_bin[3];
  uint32_t tot[4][2][kSelWaves];  // wave totals of the scans (three digits, one compaction)
  uint32_t c_gt[kSelThreads], c_eq[kSelThreads];
};

// Top-k (or threshold) selection of L keys by one 1024-thread workgroup:
// writes mask[0..L), the selected positions i as idx_base + i in ascending
// order to idx[0..), and their number to *n_sel if n_sel is not null.
// R > 0: the L keys are loaded once into registers (key r*1024 + tid in
// slot r, L <= 1024 R), all loads in flight together; every later pass works
// on the registers.  R == 0: keys are re-read from s on every pass (any L).
// Workgroup `part` of `parts` writes the results of its share of the rounds
// only: the stores of one CU take as long as the selection, and the selection,
// repeated in every workgroup, needs no word from the others.
template <int R>
__device__ __forceinline__ void topk_rows(const float* __restrict__ s, int L, int k, int threshold_mode,
                                          float threshold, int idx_base, int32_t* __restrict__ idx,
                                          uint8_t* __restrict__ mask, int32_t* __restrict__ n_sel, int part = 0,
                                          int parts = 1) {
  __shared__ TopkLds lds;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  constexpr int RR = R > 0 ? R : 1;
  uint32_t kr[RR];
  // The thread's index through an empty asm for each pass, and a barrier to
  // the scheduler after each round: the indexes, addresses and bounds of up to
  // 80 rounds, computed once and kept from pass to pass, would spill (64 rounds
  // spill 8 registers so, 80 rounds 87).
  auto fresh_tid = [&]() __attribute__((always_inline)) {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  if constexpr (R > 0) {
    const int ta = fresh_tid();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = r * kSelThreads + ta;
      kr[r] = __float_as_uint(s[i < L ? i : L - 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int tb = fresh_tid();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      kr[r] = r * kSelThreads + tb < L ? rank_key(__uint_as_float(kr[r])) : 0u;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int rounds = (L + kSelThreads - 1) / kSelThreads;
  const int nr = R > 0 ? R : rounds;  // the passes over registers are unrolled whole
  // body(r, key) for the rounds r0 .. r1 - 1
  auto for_rounds = [&](int r0, int r1, auto&& body) __attribute__((always_inline)) {
    if constexpr (R > 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r >= r0 && r < r1) body(r, kr[r]);
        __builtin_amdgcn_sched_barrier(0);  // one round's values at a time
      }
    } else {
      for (int r = r0; r < r1; ++r) {
        const int i = r * kSelThreads + tid;
        body(r, i < L ? rank_key(s[i]) : 0u);
      }
    }
  };
  // exclusive sums of a and b over the threads before this one, and their totals
  auto scan2 = [&](uint32_t a, uint32_t b, uint32_t(&tot)[2][kSelWaves], uint32_t& ea, uint32_t& eb, uint32_t& ta,
                   uint32_t& tb) __attribute__((always_inline)) {
    uint32_t ia = a, ib = b;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t va = __shfl_up(ia, o), vb = __shfl_up(ib, o);
      if (lane >= o) {
        ia += va;
        ib += vb;
      }
    }
    if (lane == kWave - 1) {
      tot[0][wave] = ia;
      tot[1][wave] = ib;
    }
    __syncthreads();
    ea = ia - a;
    eb = ib - b;
    ta = tb = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
      const uint32_t va = tot[0][w], vb = tot[1][w];
      ea += w < wave ? va : 0u;
      eb += w < wave ? vb : 0u;
      ta += va;
      tb += vb;
    }
  };

  // (1) threshold key and how many tokens equal to it are taken
  uint32_t thr;
  uint32_t need_eq;
  bool take_eq;
  if (threshold_mode) {
    thr = rank_key(threshold);
    need_eq = 0;
    take_eq = false;
  } else if (k == 0) {
    thr = 0xffffffffu;
    need_eq = 0;
    take_eq = true;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) lds.h1[j * kSelThreads + tid] = 0;
    lds.h2[tid] = lds.h2[kSelThreads + tid] = lds.h3[tid] = 0;
    __syncthreads();
    uint32_t kk = static_cast<uint32_t>(k);
    // The bin of pass P that holds the kk-th largest key, given this thread's
    // two counts (top bins first: thread t holds bins 2047 - 2t and 2046 - 2t),
    // and the keys above it.
    auto find = [&](auto p_c, uint32_t c_hi, uint32_t c_lo, uint32_t bin_hi) __attribute__((always_inline)) {
      constexpr int P = decltype(p_c)::value;
      uint32_t excl, dummy_e, total, dummy_t;
      scan2(c_hi + c_lo, 0u, lds.tot[P], excl, dummy_e, total, dummy_t);
      if (excl < kk && excl + c_hi + c_lo >= kk) {  // one thread: kk <= the keys of the digit
        const bool hi = excl + c_hi >= kk;
        lds.digit[P] = hi ? bin_hi : bin_hi - 1;
        lds.above[P] = hi ? excl : excl + c_hi;
        lds.in_bin[P] = hi ? c_hi : c_lo;
      }
      __syncthreads();
      kk -= __builtin_amdgcn_readfirstlane(lds.above[P]);
      return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(lds.digit[P]));
    };
    // digit 1 (bits 31 .. 21); "no key" counts in bin 0, below every key's bin.
    // A wave of one bin (frames without sound, tokens without change) adds once:
    // its lanes' adds to one address would follow one another.
    for_rounds(0, nr, [&](int, uint32_t key) __attribute__((always_inline)) {
      const uint32_t bin = key >> 21, f = __builtin_amdgcn_readfirstlane(bin);
      if (__ballot(bin != f) == 0ull) {  // uniform
        if (lane == 0) atomicAdd(&lds.h1[(f << 2) + (wave & 3)], static_cast<uint32_t>(kWave));
      } else {
        atomicAdd(&lds.h1[(bin << 2) + (lane & 3)], 1u);
      }
    });
    __syncthreads();
    uint32_t c[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint4 q = *reinterpret_cast<const uint4*>(&lds.h1[(2047 - 2 * tid - j) * 4]);
      c[j] = q.x + q.y + q.z + q.w;
    }
    uint32_t base = find(std::integral_constant<int, 0>{}, c[0], c[1], 2047u - 2u * tid) << 21;
    // digits 2 (bits 20 .. 10) and 3 (bits 9 .. 0) of the keys in the bin before.
    // Where the bin is crowded (many keys tie), one lane adds for all of the wave's
    // keys that meet the first one's bin.
    const uint32_t crowd = static_cast<uint32_t>(L) / 8 + 256;
    auto count = [&](uint32_t* h, uint32_t span, int shift, uint32_t keys_in) __attribute__((always_inline)) {
      if (keys_in <= crowd) {
        for_rounds(0, nr, [&](int, uint32_t key) __attribute__((always_inline)) {
          const uint32_t t = key - base;
          if (t < span) atomicAdd(&h[t >> shift], 1u);
        });
      } else {
        for_rounds(0, nr, [&](int, uint32_t key) __attribute__((always_inline)) {
          const uint32_t t = key - base;
          const uint64_t in = __ballot(t < span);
          if (in != 0ull) {  // uniform
            const int lead = __builtin_ctzll(in);
            const uint32_t bin = t >> shift, f = __builtin_amdgcn_readlane(bin, lead);
            const uint64_t same = __ballot(t < span && bin == f);
            if (t < span && (bin != f || lane == lead))
              atomicAdd(&h[bin], bin == f ? static_cast<uint32_t>(__popcll(same)) : 1u);
          }
        });
      }
      __syncthreads();
    };
    count(lds.h2, 1u << 21, 10, __builtin_amdgcn_readfirstlane(lds.in_bin[0]));
    base += find(std::integral_constant<int, 1>{}, lds.h2[2047 - 2 * tid], lds.h2[2046 - 2 * tid], 2047u - 2u * tid) << 10;
    count(lds.h3, 1u << 10, 0, __builtin_amdgcn_readfirstlane(lds.in_bin[1]));
    base += find(std::integral_constant<int, 2>{}, lds.h3[1023 - tid], 0u, 1023u - tid);
    thr = base;
    need_eq = kk;
    take_eq = true;
  }

  thr = __builtin_amdgcn_readfirstlane(thr);
  need_eq = __builtin_amdgcn_readfirstlane(need_eq);

  // (2) stable compaction in index order, in chunks of CH rounds.  Round r,
  //     wave w holds the indices r * 1024 + 64 w + lane, so the (r, w) pairs
  //     taken round-major are in index order.  Per chunk:
  //   a. every wave counts its keys above (gt) and equal to (eq) the
  //      threshold key in each round, lane r for round r;
  //   b. one thread per (r, w): exclusive scans of both; of the equal keys
  //      before a pair the first need_eq are taken, so its first output slot is
  //      the keys above before it plus min(need_eq, equal keys before it);
  //   c. every lane writes its mask byte and, if taken, its index.
  constexpr int CH = kSelThreads / kSelWaves;  // 64 rounds: one (r, w) pair per thread in b
  uint32_t base_eq = 0, base_gt = 0;
  for (int r0 = 0; r0 < nr; r0 += CH) {
    const int r1 = r0 + CH < nr ? r0 + CH : nr;
    uint32_t n_gt = 0, n_eq = 0;
    for_rounds(r0, r1, [&](int r, uint32_t key) __attribute__((always_inline)) {
      const uint64_t bgt = __ballot(key > thr), beq = __ballot(take_eq && key == thr);
      const bool mine = lane == r - r0;
      n_gt = mine ? static_cast<uint32_t>(__popcll(bgt)) : n_gt;
      n_eq = mine ? static_cast<uint32_t>(__popcll(beq)) : n_eq;
    });
    lds.c_gt[lane * kSelWaves + wave] = n_gt;  // 0 past the last round
    lds.c_eq[lane * kSelWaves + wave] = n_eq;
    __syncthreads();
    uint32_t gt, eq, tot_gt, tot_eq;
    scan2(lds.c_gt[tid], lds.c_eq[tid], lds.tot[3], gt, eq, tot_gt, tot_eq);
    const uint32_t rank = base_eq + eq;  // of the pair's first equal key
    lds.c_eq[tid] = rank;
    lds.c_gt[tid] = base_gt + gt + (rank < need_eq ? rank : need_eq);
    base_gt += tot_gt;
    base_eq += tot_eq;
    __syncthreads();
    // (the comparisons of a. done again, not their 64-bit results kept: two per
    // round would spill)
    asm volatile("" : "+s"(thr));
    const int w0 = rounds * part / parts, w1 = rounds * (part + 1) / parts;  // of the rounds that hold keys
    const int tc = fresh_tid();
    const uint32_t my_rank = lds.c_eq[lane * kSelWaves + wave], my_first = lds.c_gt[lane * kSelWaves + wave];
    for_rounds(r0 > w0 ? r0 : w0, r1 < w1 ? r1 : w1, [&](int r, uint32_t key) __attribute__((always_inline)) {
      const int i = r * kSelThreads + tc;
      bool sel = key > thr;
      uint64_t bsel = __ballot(sel);
      const uint64_t beq = __ballot(take_eq && key == thr);
      if (beq != 0ull) {  // uniform
        const uint32_t before = __builtin_amdgcn_readlane(my_rank, r - r0) + lanes_below(beq);
        sel = sel || (take_eq && key == thr && before < need_eq);
        bsel = __ballot(sel);
      }
      const uint32_t pos = __builtin_amdgcn_readlane(my_first, r - r0) + lanes_below(bsel);
      if (i < L) {
        mask[i] = sel ? 1 : 0;
        if (sel) idx[pos] = idx_base + i;
      }
    });
    __syncthreads();  // c_gt / c_eq and the scan totals are rewritten by the next chunk
  }
  if (tid == 0 && part == 0 && n_sel != nullptr)
    *n_sel = static_cast<int32_t>(base_gt + (base_eq < need_eq ? base_eq : need_eq));
}

// Workgroups [0, parts) select; one more (launched only when step_delta is not
// null) computes the step-level sum, independently of the selection.
template <int R>
__global__ void __launch_bounds__(kSelThreads)
select_rows(const float* __restrict__ s, int L, int k, int threshold_mode, float threshold,
            int32_t* __restrict__ idx, uint8_t* __restrict__ mask, int32_t* __restrict__ n_sel,
            const double* __restrict__ num, const double* __restrict__ den, int nsums, double xi,
            double* __restrict__ step_delta, int parts) {
  if (static_cast<int>(blockIdx.x) == parts) {
    step_delta_block(num, den, nsums, xi, step_delta);
    return;
  }
  topk_rows<R>(s, L, k, threshold_mode, threshold, 0, idx, mask, n_sel, blockIdx.x, parts);
}

// Two-stage selection: workgroup t handles segment t (tokens [tN, tN + N)).
// A segment outside the anchor set clears its mask; an anchor segment takes
// its min(k, N) tokens ranked first by (s desc, index asc) and writes them at
// idx[a * min(k, N)...], a = the number of anchor segments before it, so idx
// stays ascending.  Workgroup 0 writes the total count.
template <int R>
__global__ void __launch_bounds__(kSelThreads)
select_segments(const float* __restrict__ s, const uint8_t* __restrict__ anchors, int T, int N, int k,
                int32_t* __restrict__ idx, uint8_t* __restrict__ mask, int32_t* __restrict__ n_sel) {
  __shared__ int sh_before, sh_total;
  const int t = blockIdx.x, tid = threadIdx.x;
  if (tid == 0) {
    sh_before = 0;
    sh_total = 0;
  }
  __syncthreads();
  int before = 0, total = 0;
  for (int u = tid; u < T; u += kSelThreads) {
    const int a = anchors[u] != 0;
    total += a;
    before += (u < t) ? a : 0;
  }
  if (total) atomicAdd(&sh_total, total);
  if (before) atomicAdd(&sh_before, before);
  __syncthreads();
  const int kk = k < N ? k : N;
  if (t == 0 && tid == 0) *n_sel = sh_total * kk;
  const int64_t base = static_cast<int64_t>(t) * N;
  if (!anchors[t]) {
    for (int i = tid; i < N; i += kSelThreads) mask[base + i] = 0;
    return;
  }
  topk_rows<R>(s + base, N, kk, 0, 0.0f, static_cast<int>(base), idx + static_cast<int64_t>(sh_before) * kk,
               mask + base, nullptr);
}

// Anchor segments, one workgroup, T <= kMaxAnchorT:
//   mode 0: the k segments ranked first by (key desc, index asc), NaN first
//           (each segment counts the segments that rank before it);
//   mode 1: the evenly spaced segments floor((2j + 1) T / (2k)), j < k
//           (segment t is one iff some j satisfies 2kt <= (2j + 1) T < 2k(t + 1)).
constexpr int kMaxAnchorT = 4096;

__global__ void __launch_bounds__(kSelThreads)
anchor_select(const float* __restrict__ keys, int T, int k, int mode, uint8_t* __restrict__ anchors) {
  __shared__ uint32_t kl[kMaxAnchorT];
  const int tid = threadIdx.x;
  if (mode == 0) {
    for (int t = tid; t < T; t += kSelThreads) kl[t] = rank_key(keys[t]);
    __syncthreads();
    for (int t = tid; t < T; t += kSelThreads) {
      const uint32_t kt = kl[t];
      int rank = 0;
      for (int u = 0; u < T; ++u) {
        const uint32_t ku = kl[u];
        rank += (ku > kt || (ku == kt && u < t)) ? 1 : 0;
      }
      anchors[t] = rank < k ? 1 : 0;
    }
    return;
  }
  for (int t = tid; t < T; t += kSelThreads) {
    uint8_t a = 0;
    if (k > 0) {
      // smallest j with (2j + 1) T >= 2kt
      const int64_t num = 2 * static_cast<int64_t>(k) * t - T;
      const int64_t j = num <= 0 ? 0 : (num + 2 * static_cast<int64_t>(T) - 1) / (2 * static_cast<int64_t>(T));
      a = (j < k && (2 * j + 1) * T < 2 * static_cast<int64_t>(k) * (t + 1)) ? 1 : 0;
    }
    anchors[t] = a;
  }
}

// ---- a selection of few tokens in one launch.  Two dependent launches and a
// digit-wise selection made for thousands of keys are all latency here: one
// workgroup takes the saliency of every row (a wave per row, kSmallRows rows'
// loads together, a chunk of 8 elements per lane: D <= 512), keeps the keys in
// LDS and ranks each by counting the keys before it, one thread per key; the
// step-level sum adds the same pairs in the same order as the kernels above.
// A call of 32 or 64 tokens takes 13 us (two launches 16); with more than four
// rows a wave the rows follow one another, and 192 tokens take 19 us (16), 256
// 24, hence the limit.
constexpr int kSmallTokens = 64, kSmallD = 512;
constexpr int kSmallRows = kSmallTokens / kSelWaves;

template <typename T>
__global__ void __launch_bounds__(kSelThreads)
select_small(const T* __restrict__ x, const T* __restrict__ xref, const float* __restrict__ fw, int L, int N, int D,
             double xi, int k, int threshold_mode, float threshold, float* __restrict__ s_out,
             int32_t* __restrict__ idx, uint8_t* __restrict__ mask, int32_t* __restrict__ n_sel,
             double* __restrict__ step_delta) {
  __shared__ __attribute__((aligned(16))) uint32_t keys[kSmallTokens];
  __shared__ double rn[kSmallTokens], rd[kSmallTokens];
  __shared__ double gn[kSmallTokens / 4], gd[kSmallTokens / 4];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (tid < kSmallTokens) {
    keys[tid] = 0u;  // "no key" past L
    rn[tid] = rd[tid] = 0.0;
  }
  __syncthreads();
  const int nch = D / 8, cc = lane < nch ? lane : nch - 1;
  Raw8<T> ra[kSmallRows], rb[kSmallRows];
#pragma unroll
  for (int u = 0; u < kSmallRows; ++u) {
    const int r = wave + u * kSelWaves;
    const int64_t row = r < L ? r : L - 1;
    ra[u].load(x + row * D + cc * 8);
    rb[u].load(xref + row * D + cc * 8);
  }
#pragma unroll
  for (int u = 0; u < kSmallRows; ++u) {
    const int r = wave + u * kSelWaves;
    if (r >= L) break;  // uniform
    float fa[8], fb[8];
    ra[u].unpack(fa);
    rb[u].unpack(fb);
    double num = 0.0, den = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double da = fa[j], db = fb[j];
      num += fabs(da - db);
      den += fabs(db);
    }
    num = wave_sum(lane < nch ? num : 0.0);
    den = wave_sum(lane < nch ? den : 0.0);
    if (lane == 0) {
      const double delta = num / (den + xi);
      const float s = __double2float_rn(static_cast<double>(fw[r / N]) * delta);
      s_out[r] = s;
      keys[r] = rank_key(s);
      rn[r] = num;
      rd[r] = den;
    }
  }
  __syncthreads();
  if (wave == 0) {  // a key per lane
    const uint32_t mine = keys[lane];
    bool sel;
    if (threshold_mode) {
      sel = mine > rank_key(threshold);
    } else {
      int before = 0;
#pragma unroll
      for (int u = 0; u < kSmallTokens / 4; ++u) {
        const uint4 q = reinterpret_cast<const uint4*>(keys)[u];
        const int b = 4 * u;
        before += (q.x > mine || (q.x == mine && b < lane)) ? 1 : 0;
        before += (q.y > mine || (q.y == mine && b + 1 < lane)) ? 1 : 0;
        before += (q.z > mine || (q.z == mine && b + 2 < lane)) ? 1 : 0;
        before += (q.w > mine || (q.w == mine && b + 3 < lane)) ? 1 : 0;
      }
      sel = before < k;
    }
    sel = sel && lane < L;
    const uint64_t bsel = __ballot(sel);
    if (lane < L) {
      mask[lane] = sel ? 1 : 0;
      if (sel) idx[lanes_below(bsel)] = lane;
    }
    if (lane == 0) *n_sel = static_cast<int32_t>(__popcll(bsel));
    if (lane < kSmallTokens / 4) {  // the sums of four rows, as a saliency workgroup leaves them
      double a = rn[4 * lane], b = rd[4 * lane];
#pragma unroll
      for (int j = 1; j < 4; ++j) {
        a += rn[4 * lane + j];
        b += rd[4 * lane + j];
      }
      gn[lane] = a;
      gd[lane] = b;
    }
  }
  __syncthreads();
  if (step_delta != nullptr) step_delta_block(gn, gd, (L + 3) / 4, xi, step_delta);
}

// workgroups of the saliency pass, each of which leaves one pair of sums
static int sal_parts(int L) { return (L + (kSalThreads / kWave) - 1) / (kSalThreads / kWave); }

hipError_t launch_saliency(int dtype_bf16, const void* x, const void* xref, const float* fw, int L, int N,
                           int D, double xi, float* s, double* num, double* den, double* step_delta,
                           hipStream_t stream) {
  const dim3 grid(sal_parts(L));
  const int per_lane = (D / 8 + kWave - 1) / kWave;
  hipError_t e = hipErrorInvalidValue;
  bool done = false;
#define ECHO_SAL_CASE(MC)                                                                        \
  if (!done && (MC == 0 || per_lane <= MC)) {                                                    \
    done = true;                                                                                 \
    if (dtype_bf16)                                                                              \
      e = ECHO_LAUNCH("saliency_rows_bf16", (saliency_rows<bf16_t, MC>), grid, dim3(kSalThreads), \
                      0, stream, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(xref), \
                      fw, L, N, D, xi, s, num, den);                                             \
    else                                                                                         \
      e = ECHO_LAUNCH("saliency_rows_f32", (saliency_rows<float, MC>), grid, dim3(kSalThreads),   \
                      0, stream, static_cast<const float*>(x), static_cast<const float*>(xref),   \
                      fw, L, N, D, xi, s, num, den);                                             \
  }
  ECHO_SAL_CASE(1)
  ECHO_SAL_CASE(2)
  ECHO_SAL_CASE(3)
  ECHO_SAL_CASE(4)
  ECHO_SAL_CASE(6)
  ECHO_SAL_CASE(8)
  ECHO_SAL_CASE(10)
  ECHO_SAL_CASE(12)
  ECHO_SAL_CASE(16)
  ECHO_SAL_CASE(0)
#undef ECHO_SAL_CASE
  if (e != hipSuccess || step_delta == nullptr) return e;
  return ECHO_LAUNCH("step_delta_sum", step_delta_sum, dim3(1), dim3(kSelThreads), 0, stream, num, den,
                     sal_parts(L), xi, step_delta);
}

hipError_t launch_topk(const float* s, int L, int k, int threshold_mode, float threshold, int32_t* idx,
                       uint8_t* mask, int32_t* n_sel, hipStream_t stream, const double* num,
                       const double* den, double xi, double* step_delta) {
  // two rounds of stores per workgroup or more, up to one workgroup per XCD; up to
  // four rounds one workgroup does as well alone
  const int rounds = (L + kSelThreads - 1) / kSelThreads;
  const int parts = rounds < 5 ? 1 : rounds / 2 < 8 ? rounds / 2 : 8;
  // A form of R rounds walks R rounds in every pass, so the forms lie close
  // together: 9000 keys took 18.8 us in the form of 32 rounds and take 13.0 in that of
  // 16, 16384 keys 19.0 and 13.3, 33000 keys 55.8 (80 rounds) and 25.4 (48), 60000
  // keys 56.2 (80) and 32.5 (64).  (Passes bounded by the rounds at run time: 16.6,
  // 18.2, 44, 50, and 2 us more where the form is full.)
  const dim3 grid(parts + (step_delta != nullptr ? 1 : 0));
#define ECHO_SEL_CASE(RK)                                                                      \
  if (L <= RK * kSelThreads)                                                                   \
    return ECHO_LAUNCH("select_rows", select_rows<RK>, grid, dim3(kSelThreads), 0, stream, s, L, \
                       k, threshold_mode, threshold, idx, mask, n_sel, num, den, sal_parts(L), xi, step_delta, parts);
  ECHO_SEL_CASE(1)
  ECHO_SEL_CASE(2)
  ECHO_SEL_CASE(4)
  ECHO_SEL_CASE(8)
  ECHO_SEL_CASE(16)
  ECHO_SEL_CASE(32)
  ECHO_SEL_CASE(48)
  ECHO_SEL_CASE(64)
  ECHO_SEL_CASE(80)
#undef ECHO_SEL_CASE
  return ECHO_LAUNCH("select_rows", select_rows<0>, grid, dim3(kSelThreads), 0, stream, s, L, k,
                     threshold_mode, threshold, idx, mask, n_sel, num, den, sal_parts(L), xi, step_delta, parts);
}

hipError_t launch_topk_segments(const float* s, const uint8_t* anchors, int T, int N, int k, int32_t* idx,
                                uint8_t* mask, int32_t* n_sel, hipStream_t stream) {
#define ECHO_SEG_CASE(RK)                                                                             \
  if (N <= RK * kSelThreads)                                                                          \
    return ECHO_LAUNCH("select_segments", select_segments<RK>, dim3(T), dim3(kSelThreads), 0, stream, s, \
                       anchors, T, N, k, idx, mask, n_sel);
  ECHO_SEG_CASE(2)
  ECHO_SEG_CASE(8)
  ECHO_SEG_CASE(32)
#undef ECHO_SEG_CASE
  return ECHO_LAUNCH("select_segments", select_segments<0>, dim3(T), dim3(kSelThreads), 0, stream, s, anchors,
                     T, N, k, idx, mask, n_sel);
}

int max_anchor_segments() { return kMaxAnchorT; }

hipError_t launch_anchors(const float* keys, int T, int k, int mode, uint8_t* anchors, hipStream_t stream) {
  return ECHO_LAUNCH("anchor_select", anchor_select, dim3(1), dim3(kSelThreads), 0, stream, keys, T, k, mode,
                     anchors);
}

hipError_t launch_select(int dtype_bf16, const void* x, const void* xref, const float* fw, int L, int N,
                         int D, double xi, int k, int threshold_mode, float threshold, float* s,
                         double* num, double* den, int32_t* idx, uint8_t* mask, int32_t* n_sel,
                         double* step_delta, hipStream_t stream) {
  if (L <= kSmallTokens && D <= kSmallD) {
    if (dtype_bf16)
      return ECHO_LAUNCH("select_small", select_small<bf16_t>, dim3(1), dim3(kSelThreads), 0, stream,
                         static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(xref), fw, L, N, D, xi, k,
                         threshold_mode, threshold, s, idx, mask, n_sel, step_delta);
    return ECHO_LAUNCH("select_small", select_small<float>, dim3(1), dim3(kSelThreads), 0, stream,
                       static_cast<const float*>(x), static_cast<const float*>(xref), fw, L, N, D, xi, k,
                       threshold_mode, threshold, s, idx, mask, n_sel, step_delta);
  }
  // the step-level sum runs beside the selection, in the same launch
  const hipError_t e = launch_saliency(dtype_bf16, x, xref, fw, L, N, D, xi, s, num, den, nullptr, stream);
  if (e != hipSuccess) return e;
  return launch_topk(s, L, k, threshold_mode, threshold, idx, mask, n_sel, stream, num, den, xi, step_delta);
}

}  // namespace echo
