// fp32 path of the partial DiT block (any head width up to 128), for exactness
// checks and small shapes: a GEMM with the same fused epilogues as the bf16
// one and a streaming-softmax attention, both on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// The shapes are small (tens to hundreds of rows), so what bounds them is the
// latency of a few dependent steps, not a rate: fragments are read straight
// from global memory (a lane's operand is 16 bytes of one row; every operand
// is L2-resident and read by few workgroups), many loads in flight per wave,
// with no LDS staging and no barrier but the one in front of the reduction,
// and the depth (GEMM) or the keys (attention) are divided between the waves
// of a workgroup.
#include <math.h>

#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace echo {

constexpr int F32_WAVES = 4;  // waves of a workgroup, which divide the depth or the keys

__device__ __forceinline__ float gelu_tanh_ref(float z) {
  return 0.5f * z * (1.0f + tanhf(0.7978845608028654f * (z + 0.044715f * z * z * z)));
}

// Output tile of 16 T x 16 T.  The depth goes in chunks of 16: wave w takes the
// chunks w, w + 4, ..., each four MFMAs per 16 x 16 block: in step j lane
// (l16, lq) holds k = 16 c + 4 lq + j of row l16 of A and of B, so a lane's four
// steps are one 16-byte load.  The waves' sums are added in wave order, so a
// row's result depends neither on the tile size nor on the other rows.
// T = 2 reads half the bytes per product, T = 1 has four times the workgroups;
// see launch_gemm_f32.  32 tokens, 16 selected, D 64, F 256 (depths 64 and 256):
// 3.9 - 9.6 us per product with 16 x 16 tiles staged through LDS -> 3.1 - 3.6;
// 600 tokens, 400 selected, D 512, F 1024: the whole step 576 -> 117 us.
// The grid's third dimension picks one of two products (the second may have
// fewer or more tiles than the first: workgroups past a product's end leave).
struct GemmF32Pair {
  GemmF32Args g[2];
};
template <int EPI, int T>  // 0 bias, 1 gelu, 2 gate+residual (same codes as the bf16 GEMM)
__global__ void __launch_bounds__(F32_WAVES * kWave) gemm_f32_nt(GemmF32Pair pair) {
  const GemmF32Args& p = pair.g[blockIdx.z];
  constexpr int TILE = 16 * T, LD = TILE + 1;
  constexpr int UNR = T == 1 ? 4 : 2;  // chunks whose loads are in flight together
  __shared__ float part[F32_WAVES][TILE * LD];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int l16 = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * TILE, n0 = blockIdx.x * TILE;
  if (m0 >= p.M || n0 >= p.N) return;  // uniform
  const float* arow[T];
  const float* brow[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    int m = m0 + 16 * t + l16, n = n0 + 16 * t + l16;  // past the end: the last row again, not stored
    m = m < p.M ? m : p.M - 1;
    n = n < p.N ? n : p.N - 1;
    arow[t] = p.A + (p.a_rows ? static_cast<int64_t>(p.a_rows[m]) : m) * p.lda;
    brow[t] = n < p.n_split ? p.B0 + static_cast<int64_t>(n) * p.ldb : p.B1 + static_cast<int64_t>(n - p.n_split) * p.ldb;
  }
  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int nc = (p.K + 15) / 16;  // K is a multiple of 4: a lane's four elements are all in or all out
  for (int c0 = wave; c0 < nc; c0 += UNR * F32_WAVES) {
    float4 a[UNR][T], b[UNR][T];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int k = 16 * (c0 + u * F32_WAVES) + 4 * lq;
      const int kk = k < p.K ? k : 0;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        a[u][t] = *reinterpret_cast<const float4*>(arow[t] + kk);
        b[u][t] = *reinterpret_cast<const float4*>(brow[t] + kk);
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if (c0 + u * F32_WAVES >= nc) break;  // uniform per wave
      const bool in = 16 * (c0 + u * F32_WAVES) + 4 * lq < p.K;
#pragma unroll
      for (int t = 0; t < T; ++t)
        if (!in) a[u][t] = b[u][t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) {
            const float av = s == 0 ? a[u][i].x : s == 1 ? a[u][i].y : s == 2 ? a[u][i].z : a[u][i].w;
            const float bv = s == 0 ? b[u][j].x : s == 1 ? b[u][j].y : s == 2 ? b[u][j].z : b[u][j].w;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[i][j], 0, 0, 0);
          }
    }
  }
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][(16 * i + 4 * lq + r) * LD + 16 * j + l16] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < TILE * TILE / (F32_WAVES * kWave); ++e) {
    const int i = tid + e * F32_WAVES * kWave, r = i / TILE, c = i % TILE;
    const int row = m0 + r, col = n0 + c;
    if (row >= p.M || col >= p.N) continue;
    float sum = part[0][r * LD + c];
#pragma unroll
    for (int w = 1; w < F32_WAVES; ++w) sum += part[w][r * LD + c];
    const float v = sum + (col < p.n_split ? p.bias0[col] : p.bias1[col - p.n_split]);
    float outv;
    if (EPI == 0) {
      outv = v;
    } else if (EPI == 1) {
      outv = gelu_tanh_ref(v);
    } else {
      const int64_t rr = p.res_rows ? p.res_rows[row] : row;
      outv = p.res[rr * p.ldr + col] + p.gate[col] * v;
    }
    p.C[static_cast<int64_t>(row) * p.ldc + col] = outv;
  }
}

// One workgroup per (16 queries, head).  Keys go in groups of 16: wave w takes
// the groups w, w + 4, ... with a streaming softmax of its own; the waves'
// sums are merged in wave order at the end.  dh is padded to 16 NB with zeros
// (EXACT: dh = 16 NB, rows read 16 bytes at a time).
//   S^T (16 keys x 16 queries) = K Q^T: in step (c, j) lane (l16, lq) holds
//     element 16 c + 4 lq + j of key l16 and of query l16; the lane ends with
//     the scores of query l16 and keys 4 lq + r, r < 4.
//   O^T (16 NB x 16 queries) += V^T P^T: in step r lane (l16, lq) holds
//     V[key 4 lq + r][16 n + l16] and its own probability of that key.
// A group's K and V are loaded while the group before is processed.  One wave
// per query with a key per lane, as before, read each key row element by
// element with the lanes on different rows (32 keys of width 32: 12.5 -> 3.4 us).
template <int NB, bool EXACT>
__global__ void __launch_bounds__(F32_WAVES * kWave)
attn_fwd_f32(const float* __restrict__ q, int64_t ldq, const float* __restrict__ k,
             const float* __restrict__ v, int64_t ldkv, int Mq, int L, int dh, float scale,
             float* __restrict__ out, int64_t ldo) {
  __shared__ float so[F32_WAVES][16 * NB][17];
  __shared__ float sm[F32_WAVES][16], sl[F32_WAVES][16];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int l16 = lane & 15, lq = lane >> 4;
  const int q0 = blockIdx.x * 16, head = blockIdx.y;
  const int64_t hoff = static_cast<int64_t>(head) * dh;
  // elements 16 c + 4 lq .. + 3 of a row
  auto load4 = [&](const float* row, int c) __attribute__((always_inline)) {
    const int d = 16 * c + 4 * lq;
    if constexpr (EXACT) {
      return *reinterpret_cast<const float4*>(row + d);
    } else {
      float4 t;
      t.x = d < dh ? row[d] : 0.0f;
      t.y = d + 1 < dh ? row[d + 1] : 0.0f;
      t.z = d + 2 < dh ? row[d + 2] : 0.0f;
      t.w = d + 3 < dh ? row[d + 3] : 0.0f;
      return t;
    }
  };
  float4 qf[NB], kf[NB], kn[NB];
  float vf[NB][4], vn[NB][4];
  {
    const int qr = q0 + l16 < Mq ? q0 + l16 : Mq - 1;
#pragma unroll
    for (int c = 0; c < NB; ++c) qf[c] = load4(q + static_cast<int64_t>(qr) * ldq + hoff, c);
  }
  // the group at key0; keys past L: row L - 1 again, masked below
  auto fetch = [&](int key0, float4(&kd)[NB], float(&vd)[NB][4]) __attribute__((always_inline)) {
    const int kr = key0 + l16 < L ? key0 + l16 : L - 1;
#pragma unroll
    for (int c = 0; c < NB; ++c) kd[c] = load4(k + static_cast<int64_t>(kr) * ldkv + hoff, c);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = key0 + 4 * lq + r;
      const float* row = v + static_cast<int64_t>(key < L ? key : L - 1) * ldkv + hoff;
#pragma unroll
      for (int n = 0; n < NB; ++n) vd[n][r] = EXACT || 16 * n + l16 < dh ? row[16 * n + l16] : 0.0f;
    }
  };
  f32x4 o[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) o[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // largest (sum) over the lanes of a query: l16, l16 + 16, + 32, + 48
  auto across = [&](float x, auto op) __attribute__((always_inline)) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
  };
  // the running maximum starts at the lowest finite value: a wave without keys,
  // or with none but -inf scores, merges with weight 0, and a NaN score reaches
  // the result through the sums of the wave that has it
  float m = -3.402823466e38f, l = 0.0f;
  int key0 = 16 * wave;
  if (key0 < L) fetch(key0, kn, vn);
  for (; key0 < L; key0 += 16 * F32_WAVES) {
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      kf[n] = kn[n];
#pragma unroll
      for (int r = 0; r < 4; ++r) vf[n][r] = vn[n][r];
    }
    if (key0 + 16 * F32_WAVES < L) fetch(key0 + 16 * F32_WAVES, kn, vn);
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].x, qf[c].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].y, qf[c].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].z, qf[c].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].w, qf[c].w, s, 0, 0, 0);
    }
    float sc[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sc[r] = key0 + 4 * lq + r < L ? s[r] * scale : -INFINITY;
      mx = fmaxf(mx, sc[r]);
    }
    mx = across(mx, [](float a, float b) { return fmaxf(a, b); });
    const float m_new = fmaxf(m, mx);
    const float alpha = expf(m - m_new);
    float pv[4], ps = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool in = key0 + 4 * lq + r < L;
      pv[r] = in ? expf(sc[r] - m_new) : 0.0f;
      ps += pv[r];
#pragma unroll
      for (int n = 0; n < NB; ++n) vf[n][r] = in ? vf[n][r] : 0.0f;
    }
    l = l * alpha + across(ps, [](float a, float b) { return a + b; });
    m = m_new;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n][r] *= alpha;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[n][r], pv[r], o[n], 0, 0, 0);
    }
  }
  // lane (l16, lq) holds O of query l16 at elements 16 n + 4 lq + r
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) so[wave][16 * n + 4 * lq + r][l16] = o[n][r];
  if (lq == 0) {
    sm[wave][l16] = m;
    sl[wave][l16] = l;
  }
  __syncthreads();
  for (int e = tid; e < 16 * dh; e += F32_WAVES * kWave) {
    const int qi = e / dh, d = e % dh;
    if (q0 + qi >= Mq) break;
    float mt = sm[0][qi];
#pragma unroll
    for (int w = 1; w < F32_WAVES; ++w) mt = fmaxf(mt, sm[w][qi]);
    float lt = 0.0f, ot = 0.0f;
#pragma unroll
    for (int w = 0; w < F32_WAVES; ++w) {
      const float f = expf(sm[w][qi] - mt);
      lt += f * sl[w][qi];
      ot += f * so[w][d][qi];
    }
    out[static_cast<int64_t>(q0 + qi) * ldo + hoff + d] = ot / lt;
  }
}

template <int T>
static hipError_t launch_gemm_f32_t(const char* name, int epi, const GemmF32Pair& p, int count, hipStream_t stream) {
  int M = p.g[0].M, N = p.g[0].N;
  if (count > 1) {
    M = p.g[1].M > M ? p.g[1].M : M;
    N = p.g[1].N > N ? p.g[1].N : N;
  }
  const dim3 grid((N + 16 * T - 1) / (16 * T), (M + 16 * T - 1) / (16 * T), count);
  const dim3 block(F32_WAVES * kWave);
  switch (epi) {
    case 0: return ECHO_LAUNCH(name, (gemm_f32_nt<0, T>), grid, block, 0, stream, p);
    case 1: return ECHO_LAUNCH(name, (gemm_f32_nt<1, T>), grid, block, 0, stream, p);
    default: return ECHO_LAUNCH(name, (gemm_f32_nt<2, T>), grid, block, 0, stream, p);
  }
}

static int64_t f32_tiles(const GemmF32Args& a) {
  return static_cast<int64_t>((a.M + 31) / 32) * ((a.N + 31) / 32);
}

hipError_t launch_gemm_f32(const char* name, int epi, const GemmF32Args& a, hipStream_t stream) {
  if (a.M <= 0) return hipSuccess;
  // 32 x 32 tiles once they are two to a CU (below that the 16 x 16 ones, four
  // times as many, finish sooner)
  const GemmF32Pair p{{a, a}};
  return f32_tiles(a) >= 2 * device_cu_count() ? launch_gemm_f32_t<2>(name, epi, p, 1, stream)
                                               : launch_gemm_f32_t<1>(name, epi, p, 1, stream);
}

hipError_t launch_gemm_f32_pair(const char* name, const GemmF32Args& a, const GemmF32Args& b, hipStream_t stream) {
  const GemmF32Pair p{{a, b}};
  return f32_tiles(a) + f32_tiles(b) >= 2 * device_cu_count() ? launch_gemm_f32_t<2>(name, 0, p, 2, stream)
                                                              : launch_gemm_f32_t<1>(name, 0, p, 2, stream);
}

hipError_t launch_attn_f32(const float* q, int64_t ldq, const float* k, const float* v, int64_t ldkv,
                           int Mq, int L, int H, int dh, float* out, int64_t ldo, hipStream_t stream) {
  if (Mq <= 0) return hipSuccess;
  const float scale = static_cast<float>(1.0 / sqrt(static_cast<double>(dh)));
  const dim3 grid((Mq + 15) / 16, H);
#define ECHO_ATT_CASE(NB)                                                                                     \
  if (dh == 16 * NB)                                                                                          \
    return ECHO_LAUNCH("attn_fwd_f32", (attn_fwd_f32<NB, true>), grid, dim3(F32_WAVES * kWave), 0, stream, q, \
                       ldq, k, v, ldkv, Mq, L, dh, scale, out, ldo);                                          \
  if (dh < 16 * NB)                                                                                           \
    return ECHO_LAUNCH("attn_fwd_f32", (attn_fwd_f32<NB, false>), grid, dim3(F32_WAVES * kWave), 0, stream, q, \
                       ldq, k, v, ldkv, Mq, L, dh, scale, out, ldo);
  ECHO_ATT_CASE(1)
  ECHO_ATT_CASE(2)
  ECHO_ATT_CASE(4)
  ECHO_ATT_CASE(8)
#undef ECHO_ATT_CASE
  return hipErrorInvalidValue;
}

}  // namespace echo
