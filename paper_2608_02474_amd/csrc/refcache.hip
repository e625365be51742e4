// Adaptive reference cache (Sec. 3.4, "Memory-efficient Cache Management"):
// a fresh output whose cosine similarity with its chain's current reference
// exceeds tau is stored as an int8 residual against it, otherwise it becomes
// a new full-precision reference; references nobody holds are released.
//
// Chains are the tokens of one spatial row of the latent grid (chain_len
// consecutive indices) and keep their current reference across writes.
// References live in a pool of `capacity` rows with a hold count per slot and
// a stack of free slots.  One update is two launches on one stream:
//   refcache_release  one thread per rewritten token: drop the hold of its old
//                     entry; a slot whose count reaches zero goes back on the
//                     free stack (pushes only);
//   refcache_update   the first workgroups take one chain each: scan the
//                     chain's rewritten tokens in index order, keeping the
//                     current reference row in registers; fp64 similarity, int8
//                     residual or new reference (pops only; a chain's old
//                     reference that only the chain still held is reused in
//                     place).  The rest rebuild the other rows from their
//                     entries, one wave per row.  The fresh output cast(y_sel)
//                     and the saliency reference := x of the rewritten rows are
//                     written by the chains or by further waves (see the rule
//                     at the launch).
// The two parts of refcache_update touch different rows: a token that is not
// rewritten holds its reference, so no chain writes that slot.  A chain is
// bound by latency (its tokens one after another), the other rows by HBM, so
// run together the scan hides behind the stream, and y_sel is read once
// instead of twice (32760 x 5120 bf16, chains of 52, 13104 rewritten: scan
// 123 us, then a fusion pass of 183 us -> 217 us together, 5.7 TB/s of what has
// to be read and written; release 5 us before either).
// Every live slot is held by a token entry or a chain, so capacity >= L +
// number of chains never runs out.  Slot numbers depend on the order of the
// atomic pops; stored values and decisions do not.
#include <math.h>

#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace echo {


__global__ void __launch_bounds__(256)
refcache_init(int L, int n_chains, int capacity, int32_t* __restrict__ refcount,
              int32_t* __restrict__ free_list, int32_t* __restrict__ free_top,
              int32_t* __restrict__ chain_ref, int32_t* __restrict__ ent_slot,
              uint8_t* __restrict__ ent_kind, float* __restrict__ scale) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < capacity) {
    refcount[i] = 0;
    free_list[i] = static_cast<int32_t>(i);
  }
  if (i < L) {
    ent_slot[i] = -1;
    ent_kind[i] = 0;
    scale[i] = 0.0f;
  }
  if (i < n_chains) chain_ref[i] = -1;
  if (i == 0) *free_top = capacity;
}

__global__ void __launch_bounds__(256)
refcache_release(const int32_t* __restrict__ idx, int n_sel, int32_t* __restrict__ refcount,
                 int32_t* __restrict__ free_list, int32_t* __restrict__ free_top,
                 int32_t* __restrict__ ent_slot, uint8_t* __restrict__ ent_kind) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_sel) return;
  const int l = idx[j];
  if (ent_kind[l] == 0) return;
  const int s = ent_slot[l];
  if (atomicSub(&refcount[s], 1) == 1) free_list[atomicAdd(free_top, 1)] = s;
  ent_kind[l] = 0;
  ent_slot[l] = -1;
}

// fp32(a - b) and fp32(fp32(a * b) + c) as separate IEEE operations
__device__ __forceinline__ float sub_rn(float a, float b) {
#pragma clang fp contract(off)
  return a - b;
}
__device__ __forceinline__ float mul_add_rn(float a, float b, float c) {
#pragma clang fp contract(off)
  return a * b + c;
}

template <typename T> __device__ __forceinline__ float rc_round(float v);
template <> __device__ __forceinline__ float rc_round<float>(float v) { return v; }
template <> __device__ __forceinline__ float rc_round<bf16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }

// 4 consecutive elements of a row as stored
template <typename T> struct Raw4;
template <> struct Raw4<bf16_t> {
  uint2 v;
  __device__ void load(const bf16_t* p) { v = *reinterpret_cast<const uint2*>(p); }
  __device__ void load_nt(const bf16_t* p) { v = ldg8_nt(p); }
  __device__ void store_nt(bf16_t* p) const { stg8_nt(p, v); }
  __device__ void unpack(float* f) const {
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xffff0000u);
  }
  __device__ void pack(const float* f) { v = make_uint2(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])); }
  // f holds bf16 values
  __device__ static void store_exact(bf16_t* p, const float* f) {
    const uint32_t a = __float_as_uint(f[0]), b = __float_as_uint(f[1]), c = __float_as_uint(f[2]), d = __float_as_uint(f[3]);
    *reinterpret_cast<uint2*>(p) = make_uint2((a >> 16) | (b & 0xffff0000u), (c >> 16) | (d & 0xffff0000u));
  }
};
template <> struct Raw4<float> {
  uint4 v;
  __device__ void load(const float* p) { v = ldg16(p); }
  __device__ void load_nt(const float* p) { v = ldg16_nt(p); }
  __device__ void store_nt(float* p) const { stg16_nt(p, v); }
  __device__ void unpack(float* f) const { unpack16(v, f, static_cast<const float*>(nullptr)); }
  __device__ void pack(const float* f) { v = pack16(f, static_cast<const float*>(nullptr)); }
  __device__ static void store_exact(float* p, const float* f) { stg16(p, pack16(f, static_cast<const float*>(nullptr))); }
};

// Sum (largest) of the 16 lanes of a row, in every lane of it (DPP rotations).
__device__ __forceinline__ double row_sum(double v) {
  auto ror = [](double x, auto d_c) {
    constexpr int D = decltype(d_c)::value;
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(x));
    const uint64_t r = (static_cast<uint64_t>(dpp_ror<D>(static_cast<uint32_t>(u >> 32))) << 32) |
                       dpp_ror<D>(static_cast<uint32_t>(u));
    return x + __longlong_as_double(static_cast<long long>(r));
  };
  v = ror(v, std::integral_constant<int, 8>{});
  v = ror(v, std::integral_constant<int, 4>{});
  v = ror(v, std::integral_constant<int, 2>{});
  return ror(v, std::integral_constant<int, 1>{});
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, __uint_as_float(dpp_ror<8>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(dpp_ror<4>(__float_as_uint(v))));
  v = fmaxf(v, __uint_as_float(dpp_ror<2>(__float_as_uint(v))));
  return fmaxf(v, __uint_as_float(dpp_ror<1>(__float_as_uint(v))));
}

// dot / (sqrt(yy) sqrt(rr)) > tau, 0 > tau if yy or rr is 0, in fp64.  The
// signed squares decide unless they lie within 1e-12 of each other, a
// thousand times what the rounding of either form can move them (and unless
// an operand is out of the range where their products are exact to that); the
// division and the square roots, in every wave of a chain and for every token,
// cost more than the token's sums.
__device__ __forceinline__ bool similar(double dot, double yy, double rr, float tau) {
  const double t = static_cast<double>(tau), n = yy * rr;
  const double a = dot * fabs(dot), b = t * fabs(t) * n;
  if (n > 1e-200 && n < 1e200 && fabs(t) < 1e50 && fabs(a - b) > 1e-12 * (fabs(a) + fabs(b))) return a > b;
  const double sim = (yy == 0.0 || rr == 0.0) ? 0.0 : dot / (sqrt(yy) * sqrt(rr));
  return sim > t;
}

// One token's sums over the chain's data waves: the similarity's dot product,
// the output's squared norm, the current reference's squared norm (taken
// again only after the reference changed) and the largest residual (the
// residual's scale, if the token becomes one).  One barrier per token: the
// partials alternate between two slots, and a slot is rewritten only after
// the next token's barrier, which every reader reaches after its read.
struct ChainSums {
  double dot, yy, rr;
  float amax;
};

struct ChainLds {
  double d[2][3][16];  // per wave; zero past the last one
  float f[2][16];
  int ref[2];  // slot of the reference that the token before made, -1 = none left
};

// Workgroups [0, chains): one chain each.  Thread t of the W waves owns
// elements 4 t + 256 W u (u < U) of a row; D <= 256 W U, D % 4 == 0.  One wave
// up to D = 768, where the exchange between waves is much of a token's time, four
// waves up to D = 5120: every wave of a chain repeats the decision and the
// reductions, so five, eight and ten waves with fewer elements each were 5 to
// 15% slower there, and two waves at D = 520 to 1024 2 to 21% slower than these
// forms with STREAM.  The next token's row of y_sel is loaded while the current one is
// processed, and a token's stores are issued after that load, whose wait would
// otherwise include them.  Taking a slot from the free stack is two dependent
// memory operations of one wave: a new reference's row is stored after the
// next token's barrier, when the slot is known, and until then stays in
// registers.
// Workgroups from `chains` on: STREAM: one wave per rewritten row first, which
// writes its y and xref, so that a chain's tokens carry no more than they have
// to.  Then one wave per row i, rebuilt from its entry if
// mask[i] == 0; up to 5 of a lane's chunks of 8 elements are loaded before any
// is used.  They run in the waves that the chains leave free, so the registers
// decide how much of the stream runs beside the scan: full bf16 rows, which
// come to 128 and little more, are held to that, four waves per SIMD (D = 5120,
// 32760 rows, 40% rewritten 238 -> 225 us, 83% 350 -> 354; 4096 and 8192 the same
// either way).  Others would spill: D = 4608 bf16 319 -> 687 us, fp32 489 -> 508.
// Streams that nothing reads again before the next step are non-temporal
// (y_sel, x, y, xref, codes); the reference rows, shared by the tokens of a
// chain, keep ordinary accesses.
template <typename T, int W, int U, bool FULL, bool STREAM>
__global__ void __launch_bounds__(W * kWave, sizeof(T) == 2 && FULL ? 4 : 1)
refcache_update(const T* __restrict__ x, const int32_t* __restrict__ idx, const uint8_t* __restrict__ mask,
                int n_sel, int L, int D, int chains, int chain_len, float tau,
                const float* __restrict__ y_sel, T* __restrict__ pool, int32_t* __restrict__ refcount,
                const int32_t* __restrict__ free_list, int32_t* __restrict__ free_top,
                int32_t* __restrict__ chain_ref, int32_t* __restrict__ ent_slot,
                uint8_t* __restrict__ ent_kind, int8_t* __restrict__ codes, float* __restrict__ scale,
                T* __restrict__ xref, T* __restrict__ y_out) {
  __shared__ ChainLds lds;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;

  if (static_cast<int>(blockIdx.x) >= chains) {
    int64_t i = static_cast<int64_t>(blockIdx.x - chains) * W + wave;
    const int nch = D / 8;
    if constexpr (STREAM) {
      if (i < n_sel) {
        const int64_t row = static_cast<int64_t>(idx[i]) * D;
        const float* ys = y_sel + i * D;
        constexpr int B = (W * U + 1) / 2;  // chunks per lane: the whole row at once
        Raw8<float> yr[B];
        Raw8<T> xr[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int c = lane + u * kWave;
          if (c >= nch) continue;
          yr[u].load(ys + c * 8);
          xr[u].load_nt(x + row + c * 8);
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int c = lane + u * kWave;
          if (c >= nch) continue;
          float v[8];
          yr[u].unpack(v);
          stg16_nt(y_out + row + c * 8, pack16(v, static_cast<const T*>(nullptr)));
          if (sizeof(T) == 4) stg16_nt(y_out + row + c * 8 + 4, pack16(v + 4, static_cast<const T*>(nullptr)));
          xr[u].store(xref + row + c * 8);
        }
        return;
      }
      i -= n_sel;
    }
    if (i >= L || mask[i]) return;
    const int kind = ent_kind[i];
    const T* rp = pool + static_cast<int64_t>(ent_slot[i] < 0 ? 0 : ent_slot[i]) * D;
    const float sc = scale[i];
    constexpr int kChunks = (W * U + 1) / 2, kBatches = (kChunks + 4) / 5;
    constexpr int B = (kChunks + kBatches - 1) / kBatches;  // chunks in flight per lane
    for (int c0 = lane; c0 < nch; c0 += B * kWave) {
      Raw8<T> rr[B];
      uint2 cw[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int c = c0 + u * kWave;
        if (c < nch && kind != 0) rr[u].load(rp + c * 8);
        if (c < nch && kind == 2) cw[u] = ldg8_nt(codes + i * D + c * 8);
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int c = c0 + u * kWave;
        if (c >= nch) continue;
        float v[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (kind != 0) rr[u].unpack(v);
        if (kind == 2) {
          const uint32_t w[2] = {cw[u].x, cw[u].y};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int8_t q = static_cast<int8_t>((w[e / 4] >> (8 * (e % 4))) & 0xffu);
            v[e] = mul_add_rn(sc, static_cast<float>(q), v[e]);
          }
        }
        stg16_nt(y_out + i * D + c * 8, pack16(v, static_cast<const T*>(nullptr)));
        if (sizeof(T) == 4) stg16_nt(y_out + i * D + c * 8 + 4, pack16(v + 4, static_cast<const T*>(nullptr)));
      }
    }
    return;
  }

  const int c = blockIdx.x;
  const int lo = c * chain_len, hi = lo + chain_len;
  // rewritten tokens of this chain: idx[j0 .. j1) (idx ascending)
  int a = 0, b = n_sel;
  while (a < b) { const int m = (a + b) >> 1; if (idx[m] < lo) a = m + 1; else b = m; }
  const int j0 = a;
  b = n_sel;
  while (a < b) { const int m = (a + b) >> 1; if (idx[m] < hi) a = m + 1; else b = m; }
  const int j1 = a;
  if (j0 == j1) return;
  if (tid < 16) {
    // the slots of absent waves, before the first token's barrier
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (tid >= W) {
        lds.d[s][0][tid] = lds.d[s][1][tid] = lds.d[s][2][tid] = 0.0;
        lds.f[s][tid] = 0.0f;
      }
  }

  float y[U][4], r[U][4];  // the token's output and the current reference row (stored values)
  float4 ynext[U];         // the next token's row, loaded while this one is processed
  // FULL rows (D = 256 W U) have no bounds to check; in others a thread past
  // the row's end loads its last elements and takes zeros, so that no load
  // sits in a branch, where the compiler could not count it and would wait for
  // every access in flight, the stores included
  auto col = [&](int u) { return 4 * tid + 256 * W * u; };
  auto in = [&](int u) { return FULL || col(u) < D; };
  auto at = [&](int u) { return FULL || col(u) < D ? col(u) : D - 4; };
  auto fetch = [&](int j) __attribute__((always_inline)) {
    const float* yp = y_sel + static_cast<int64_t>(j) * D;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint4 t = ldg16_nt(yp + at(u));
      ynext[u] = make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
    }
  };
  int cr = chain_ref[c];  // the reference's slot
  int lnext = idx[j0];
  bool have = cr >= 0;
  int held = have ? refcount[cr] : 0;  // its holders: only this chain's tokens and the chain (thread 0)
  {
    const T* rp = pool + static_cast<int64_t>(have ? cr : 0) * D;
    Raw4<T> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u].load(rp + at(u));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      raw[u].unpack(r[u]);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[u][e] = have && in(u) ? r[u][e] : 0.0f;
    }
  }
  fetch(j0);
  // the row of the reference that the token of slot `slot` made
  auto store_ref = [&](int slot) __attribute__((always_inline)) {
    cr = lds.ref[slot];
    have = cr >= 0;
    if (!have) return;
    T* rp = pool + static_cast<int64_t>(cr) * D;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (in(u)) Raw4<T>::store_exact(rp + col(u), r[u]);
  };

  double rr = 0.0;    // the reference's squared norm
  bool fresh = true;  // it is to be taken with this token's sums
  bool made = false;  // the token before made a reference whose row is still to be stored
  for (int j = j0; j < j1; ++j) {
    const int l = lnext, slot = (j - j0) & 1;
    const int64_t row = static_cast<int64_t>(l) * D;
    Raw4<T> xr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      y[u][0] = in(u) ? ynext[u].x : 0.0f;
      y[u][1] = in(u) ? ynext[u].y : 0.0f;
      y[u][2] = in(u) ? ynext[u].z : 0.0f;
      y[u][3] = in(u) ? ynext[u].w : 0.0f;
    }
    const int jn = j + 1 < j1 ? j + 1 : j;  // past the last token: loaded again, not used
    lnext = idx[jn];
    fetch(jn);
    ChainSums s{0.0, 0.0, 0.0, 0.0f};
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s.dot += static_cast<double>(y[u][e]) * r[u][e];
        s.yy += static_cast<double>(y[u][e]) * y[u][e];
        s.amax = fmaxf(s.amax, fabsf(sub_rn(y[u][e], r[u][e])));
      }
    if (fresh) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) s.rr += static_cast<double>(r[u][e]) * r[u][e];
      s.rr = wave_sum(s.rr);
    }
    // x only passes through: loaded here, after the sums, its registers are
    // the sums' (loaded a token ahead like y_sel: 238 -> 227 us without)
    if constexpr (!STREAM) {
#pragma unroll
      for (int u = 0; u < U; ++u) xr[u].load_nt(x + row + at(u));
    }
    s.dot = wave_sum(s.dot);
    s.yy = wave_sum(s.yy);
    s.amax = wave_max(s.amax);
    if constexpr (W == 1) {
      __syncthreads();  // the token before's slot is known
      if (made) store_ref(slot ^ 1);
      if (fresh) rr = s.rr;
    } else {
      if (lane == 0) {
        lds.d[slot][0][wave] = s.dot;
        lds.d[slot][1][wave] = s.yy;
        lds.d[slot][2][wave] = s.rr;
        lds.f[slot][wave] = s.amax;
      }
      __syncthreads();
      if (made) store_ref(slot ^ 1);
      s.dot = row_sum(lds.d[slot][0][lane % 16]);
      s.yy = row_sum(lds.d[slot][1][lane % 16]);
      s.amax = row_max(lds.f[slot][lane % 16]);
      if (fresh) rr = row_sum(lds.d[slot][2][lane % 16]);
    }
    bool residual = false;
    if (have) {
      residual = similar(s.dot, s.yy, rr, tau);
    }
    fresh = made = !residual;
    if (tid == 0) {
      if (residual) {
        scale[l] = s.amax > 0.0f ? __fdiv_rn(s.amax, 127.0f) : 0.0f;
        ent_kind[l] = 2;
        ent_slot[l] = cr;
        refcount[cr] = ++held;
      } else {
        // new reference: the chain's old one is reused in place when only the
        // chain held it, otherwise the chain lets go of it and a slot is popped
        int ns = cr;
        if (!(have && held == 1)) {
          const int top = atomicSub(free_top, 1);
          if (top > 0) {
            ns = free_list[top - 1];
            if (have) refcount[cr] = held - 1;
          } else {
            // cannot happen with capacity >= L + chains; kept so that a broken
            // invariant leaves the token without an entry, and its chain with
            // nothing to compare with for the rest of the call, instead of
            // writing outside the pool
            atomicAdd(free_top, 1);
            ns = -1;
          }
        }
        held = 2;  // the token's entry and the chain
        if (ns >= 0) {
          refcount[ns] = 2;
          ent_kind[l] = 1;
          ent_slot[l] = ns;
          scale[l] = 0.0f;
          chain_ref[c] = ns;
        }
        lds.ref[slot] = ns;
      }
    }
    if constexpr (!STREAM) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!in(u)) continue;
        Raw4<T> o;
        o.pack(y[u]);
        o.store_nt(y_out + row + col(u));
        xr[u].store_nt(xref + row + col(u));
      }
    }
    if (residual) {
      const float inv = s.amax > 0.0f ? __fdiv_rn(127.0f, s.amax) : 0.0f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!in(u)) continue;
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float q = rintf(__fmul_rn(sub_rn(y[u][e], r[u][e]), inv));
          q = fminf(fmaxf(q, -127.0f), 127.0f);
          word |= (static_cast<uint32_t>(static_cast<int32_t>(q)) & 0xffu) << (8 * e);
        }
        __builtin_nontemporal_store(word, reinterpret_cast<uint32_t*>(codes + row + col(u)));
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) r[u][e] = rc_round<T>(y[u][e]);
    }
  }
  __syncthreads();  // the last token's slot is known
  if (made) store_ref((j1 - 1 - j0) & 1);
}

hipError_t launch_refcache_init(int L, int n_chains, int capacity, int32_t* refcount, int32_t* free_list,
                                int32_t* free_top, int32_t* chain_ref, int32_t* ent_slot, uint8_t* ent_kind,
                                float* scale, hipStream_t stream) {
  const int n = capacity > L ? capacity : L;
  return ECHO_LAUNCH("refcache_init", refcache_init, dim3((n + 255) / 256), dim3(256), 0, stream, L,
                     n_chains, capacity, refcount, free_list, free_top, chain_ref, ent_slot, ent_kind, scale);
}

template <typename T>
static hipError_t refcache_update_t(const T* x, const int32_t* idx, const uint8_t* mask, int n_sel, int L, int D,
                                    int chain_len, float tau, const float* y_sel, T* pool, int32_t* refcount,
                                    int32_t* free_list, int32_t* free_top, int32_t* chain_ref, int32_t* ent_slot,
                                    uint8_t* ent_kind, int8_t* codes, float* scale, T* xref, T* y,
                                    hipStream_t stream) {
  TimedLaunch scope("refcache_update", stream);
  int chains = 0;
  if (n_sel > 0) {
    chains = L / chain_len;
    hipLaunchKernelGGL(refcache_release, dim3((n_sel + 255) / 256), dim3(256), 0, stream, idx, n_sel, refcount,
                       free_list, free_top, ent_slot, ent_kind);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // The rewritten rows' y and xref by waves of their own, which read y_sel a
  // second time, while the rows are few enough for that read to hit the caches
  // (256 MB behind HBM; a call moves up to six times its rows) and the chains
  // narrow enough that the scan is what the call waits for.  Chains that write
  // / waves that write, us a call: 7080 tokens, chains of 59, 83% rewritten, bf16
  // D = 520 82 / 68, 640 83 / 70, 776 85 / 67, 1016 90 / 70, 1536 105 / 84, 2048 97
  // / 79, fp32 D = 520 75 / 66, 1024 90 / 73 (a scan and then a fusion pass took 80,
  // 82, 83, 86, 107, 112, 84, 95); 32760 tokens, all rewritten, bf16 D = 1024 128
  // / 122, but D = 2048 169 / 185, fp32 D = 1024 140 / 150; 75600 tokens of D = 768
  // bf16, 30% rewritten, 95 / 104.
  const bool stream_rows = D <= 2048 && static_cast<int64_t>(L) * D * sizeof(T) <= (int64_t(1) << 26);
  // the chains first: they take longest and stay resident beside the stream
#define ECHO_RC_LAUNCH(W, U, FULL, STREAM)                                                                          \
  {                                                                                                                 \
    const int64_t rows = static_cast<int64_t>(L) + (STREAM ? n_sel : 0);                                            \
    const dim3 grid(static_cast<unsigned>(chains + (rows + W - 1) / W));                                            \
    hipLaunchKernelGGL((refcache_update<T, W, U, FULL, STREAM>), grid, dim3(W * kWave), 0, stream, x, idx, mask,   \
                       n_sel, L, D, chains, chain_len, tau, y_sel, pool, refcount, free_list, free_top, chain_ref,  \
                       ent_slot, ent_kind, codes, scale, xref, y);                                                  \
    return hipGetLastError();                                                                                       \
  }
#define ECHO_RC_CASE(W, U, STREAM)                         \
  if (D == 256 * W * U) ECHO_RC_LAUNCH(W, U, true, STREAM) \
  if (D <= 256 * W * U) ECHO_RC_LAUNCH(W, U, false, STREAM)
#define ECHO_RC_NARROW(STREAM)                                                              \
  ECHO_RC_CASE(1, 1, STREAM) ECHO_RC_CASE(1, 2, STREAM) ECHO_RC_CASE(1, 3, STREAM)          \
  ECHO_RC_CASE(4, 1, STREAM) ECHO_RC_CASE(4, 2, STREAM)
  if (stream_rows) {
    ECHO_RC_NARROW(true)
  }
  ECHO_RC_NARROW(false)
  ECHO_RC_CASE(4, 4, false)
  ECHO_RC_CASE(4, 5, false)
  ECHO_RC_CASE(8, 4, false)
  ECHO_RC_CASE(16, 4, false)
#undef ECHO_RC_LAUNCH
#undef ECHO_RC_CASE
#undef ECHO_RC_NARROW
  return hipErrorInvalidValue;
}

hipError_t launch_refcache_update(int dtype_bf16, const void* x, const int32_t* idx, const uint8_t* mask,
                                  int n_sel, int L, int D, int chain_len, float tau, const float* y_sel,
                                  void* pool, int32_t* refcount, int32_t* free_list, int32_t* free_top,
                                  int32_t* chain_ref, int32_t* ent_slot, uint8_t* ent_kind, int8_t* codes,
                                  float* scale, void* xref, void* y, hipStream_t stream) {
  if (dtype_bf16)
    return refcache_update_t<bf16_t>(static_cast<const bf16_t*>(x), idx, mask, n_sel, L, D, chain_len, tau,
                                     y_sel, static_cast<bf16_t*>(pool), refcount, free_list, free_top, chain_ref,
                                     ent_slot, ent_kind, codes, scale, static_cast<bf16_t*>(xref),
                                     static_cast<bf16_t*>(y), stream);
  return refcache_update_t<float>(static_cast<const float*>(x), idx, mask, n_sel, L, D, chain_len, tau, y_sel,
                                  static_cast<float*>(pool), refcount, free_list, free_top, chain_ref, ent_slot,
                                  ent_kind, codes, scale, static_cast<float*>(xref), static_cast<float*>(y),
                                  stream);
}

}  // namespace echo
