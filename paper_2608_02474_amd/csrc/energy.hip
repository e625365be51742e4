// Audio energy anchor (Sec. 3.3, "Cross-modal Saliency Anchors"): per-segment
// STFT power, pooled into mel-width bands and latent frames.
//
// Kernel 1 (energy_frames): one workgroup per (segment, STFT frame), in fp64.
// For a power-of-two n_fft, an in-place FFT in LDS; for any other even n_fft,
// each thread evaluates whole one-sided bins k directly from the DFT sum over a
// full-period twiddle table.  |X_k|^2 and each band's range of bins go to LDS,
// and one wave per band sums its bins.  Both stay within fp64 rounding of the
// definition.
// Kernel 2 (energy_reduce): one workgroup sums the per-frame band energies of
// each (segment, band) in frame order (one thread each), then each segment's
// bands, and forms e_t and e_t / max e.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace echo {

constexpr int kEnergyThreads = 256;   // energy_reduce
constexpr int kLdsSums = 2048;        // band sums that energy_reduce holds in LDS
constexpr int kFrameThreads = 512;    // energy_frames: one thread per one-sided bin up to n_fft 1022
constexpr int kFftThreads = 256;     // energy_frames_fft

__device__ __forceinline__ int band_of_bin(int k, int n_fft, int sr, int n_bands) {
  const double mel_top = 2595.0 * log10(1.0 + (0.5 * sr) / 700.0);
  const double width = mel_top / n_bands;
  const double f = static_cast<double>(k) * sr / n_fft;
  const double m = 2595.0 * log10(1.0 + f / 700.0);
  int b = static_cast<int>(floor(m / width));
  return b < n_bands - 1 ? b : n_bands - 1;
}

// Bands are ranges of bins: first[band] = its first bin, first[n_bands] = nbins
// (bandof ascends and ends at n_bands - 1).
__device__ __forceinline__ void band_starts(const int* bandof, int nbins, int n_bands, int* first) {
  for (int k = threadIdx.x; k < nbins; k += blockDim.x)
    for (int band = k > 0 ? bandof[k - 1] + 1 : 0; band <= bandof[k]; ++band) first[band] = k;
  if (threadIdx.x == 0) first[n_bands] = nbins;
}

// Per-band sums of the bin powers, one wave per band (lane l takes bins l, l +
// 64, ... of the band; fp64 throughout).
__device__ __forceinline__ void band_sums(const double* pw, const int* first, int n_bands, double* __restrict__ out) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, nw = blockDim.x / kWave;
  for (int band = wave; band < n_bands; band += nw) {
    double acc = 0.0;
    const int k1 = first[band + 1];
    for (int k = first[band] + lane; k < k1; k += kWave) acc += pw[k];
    acc = wave_sum(acc);
    if (lane == 0) out[band] = acc;
  }
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 w) {
  return make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}

// Power-of-two n_fft (16 .. 2048): one workgroup of kFftThreads per (segment,
// frame), decimation in frequency in fp64: natural order in, X_k at position
// bitrev(k).  The chain of dependent steps bounds it (a frame is 2 KB), so
// there are few of them: a thread makes the window and the twiddle of j from
// one sincospi and does the first stage on samples j and j + n_fft/2 as it
// loads them; the band of bin j is worked out while the samples are on their
// way; the other stages go two at a time, and the last two leave the powers of
// the one-sided bins (the even positions and position 1).  Bands are ranges of
// bins, so that a wave sums its band's range and no other.  441 frames of 512:
// 7.2 us; one stage per barrier from a bit-reversed load, a second cosine for
// the window and masked band sums over all bins took 10.4.
__global__ void __launch_bounds__(kFftThreads)
energy_frames_fft(const float* __restrict__ audio, int64_t n_samples, int T, int n_fft, int log2n, int hop,
                  int n_bands, int sr, int max_frames, double* __restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int half = n_fft / 2;
  double2* z = reinterpret_cast<double2*>(lds);               // [n_fft]
  double2* tw = z + n_fft;                                    // [n_fft/2] exp(-2 pi i j / n_fft)
  double* pw = reinterpret_cast<double*>(tw + half);          // [n_fft/2 + 1]
  int* bandof = reinterpret_cast<int*>(pw + half + 1);        // [n_fft/2 + 1]
  int* first = bandof + half + 1;                             // [n_bands + 1] first bin of a band
  const int tid = threadIdx.x;
  const int t = blockIdx.y, f = blockIdx.x;
  const int64_t a = (static_cast<int64_t>(t) * n_samples) / T;
  const int64_t b = (static_cast<int64_t>(t + 1) * n_samples) / T;
  const int64_t len = b - a;
  const int nf = len < n_fft ? 1 : static_cast<int>(1 + (len - n_fft) / hop);
  double* out = part + (static_cast<int64_t>(t) * max_frames + f) * n_bands;
  if (f >= nf) {
    for (int i = tid; i < n_bands; i += kFftThreads) out[i] = 0.0;
    return;
  }
  const int64_t start = a + static_cast<int64_t>(f) * hop;
  const int64_t last = b - 1;
  for (int j = tid; j < half; j += kFftThreads) {
    const int64_t i0 = start + j, i1 = i0 + half;
    const float s0 = audio[i0 < b ? i0 : last], s1 = audio[i1 < b ? i1 : last];
    double sn, cs;
    sincospi(2.0 * j / n_fft, &sn, &cs);
    bandof[j] = band_of_bin(j, n_fft, sr, n_bands);
    const double2 w = make_double2(cs, -sn);
    // periodic Hann 0.5 - 0.5 cos(2 pi n / n_fft); the cosine half a period on is -cs
    const double v0 = i0 < b ? (0.5 - 0.5 * cs) * static_cast<double>(s0) : 0.0;
    const double v1 = i1 < b ? (0.5 + 0.5 * cs) * static_cast<double>(s1) : 0.0;
    const double d = v0 - v1;
    tw[j] = w;
    z[j] = make_double2(v0 + v1, 0.0);
    z[j + half] = make_double2(d * w.x, d * w.y);
  }
  if (tid == 0) bandof[half] = n_bands - 1;  // half the sampling rate: the top of the last band
  __syncthreads();
  band_starts(bandof, half + 1, n_bands, first);
  int left = log2n - 1;  // stages still to do, each on blocks of 2^left
  if (left & 1) {
    const int h = 1 << (left - 1);
    for (int i = tid; i < half; i += kFftThreads) {
      const int pos = i & (h - 1), p0 = 2 * i - pos;
      const double2 x0 = z[p0], x1 = z[p0 + h], w = tw[pos << (log2n - left)];
      z[p0] = cadd(x0, x1);
      z[p0 + h] = cmul(csub(x0, x1), w);
    }
    __syncthreads();
    --left;
  }
  for (; left > 0; left -= 2) {
    const int lq = left - 2, q = 1 << lq;
    for (int i = tid; i < n_fft / 4; i += kFftThreads) {
      const int pos = i & (q - 1), p0 = 4 * i - 3 * pos;
      const double2 x0 = z[p0], x1 = z[p0 + q], x2 = z[p0 + 2 * q], x3 = z[p0 + 3 * q];
      const double2 w1 = tw[pos << (log2n - left)], w2 = tw[pos << (log2n - left + 1)];
      const double2 u0 = cadd(x0, x2), u1 = cadd(x1, x3);
      const double2 u2 = cmul(csub(x0, x2), w1);
      const double2 e = cmul(csub(x1, x3), w1), u3 = make_double2(e.y, -e.x);  // times -i
      if (left > 2) {
        z[p0] = cadd(u0, u1);
        z[p0 + q] = cmul(csub(u0, u1), w2);
        z[p0 + 2 * q] = cadd(u2, u3);
        z[p0 + 3 * q] = cmul(csub(u2, u3), w2);
      } else {  // q == 1, w1 == w2 == 1
        const double2 y0 = cadd(u0, u1), y2 = cadd(u2, u3);
        const int k = static_cast<int>(__brev(static_cast<unsigned>(4 * i)) >> (32 - log2n));
        pw[k] = y0.x * y0.x + y0.y * y0.y;
        pw[k + n_fft / 4] = y2.x * y2.x + y2.y * y2.y;  // bit 1 of the position is bit log2n - 2 of the bin
        if (i == 0) {
          const double2 y1 = csub(u0, u1);
          pw[half] = y1.x * y1.x + y1.y * y1.y;
        }
      }
    }
    __syncthreads();
  }
  band_sums(pw, first, n_bands, out);
}

// groups of threads that share a bin's terms
__host__ __device__ __forceinline__ int dft_groups(int nbins) {
  return nbins <= kFrameThreads / 4 ? 4 : nbins <= kFrameThreads / 2 ? 2 : 1;
}

// Any other even n_fft: the DFT sum of each one-sided bin.  Samples n and n_fft -
// n share their cosine and, but for the sign, their sine, so that a bin takes
// half the terms (sums with the cosines, differences with the sines); threads
// that bins leave idle share the terms.  The table reads (a bank conflict or
// two each) and fp64 multiply-adds bound it.  A call with n_fft 400 and 81000
// samples 41 -> 22 us, 480000 samples 185 -> 121, n_fft 1000 314 -> 211 (all
// terms by one thread per bin -> this).
__global__ void __launch_bounds__(kFrameThreads)
energy_frames(const float* __restrict__ audio, int64_t n_samples, int T, int n_fft, int hop,
              int n_bands, int sr, int max_frames, double* __restrict__ part) {
  extern __shared__ double lds[];
  double* xw = lds;                 // [n_fft] windowed frame; then sums at n, differences at n_fft - n
  double* tc = lds + n_fft;         // [n_fft] cos(2 pi m / n_fft)
  double* ts = lds + 2 * n_fft;     // [n_fft] sin(2 pi m / n_fft)
  double* pw = lds + 3 * n_fft;     // [n_fft/2 + 1] |X_k|^2
  const int tid = threadIdx.x, half = n_fft / 2, nbins = half + 1;
  // G groups of S threads: a bin per thread of a group, the terms divided among the groups
  const int G = dft_groups(nbins), S = kFrameThreads / G;
  double* pre = pw + nbins;          // [kFrameThreads] partial sums of the groups (G > 1)
  double* pim = pre + kFrameThreads;
  int* bandof = reinterpret_cast<int*>(G > 1 ? pim + kFrameThreads : pre);  // [nbins] band of bin k
  int* first = bandof + nbins;                                              // [n_bands + 1] first bin of a band
  const int t = blockIdx.y, f = blockIdx.x;
  const int64_t a = (static_cast<int64_t>(t) * n_samples) / T;
  const int64_t b = (static_cast<int64_t>(t + 1) * n_samples) / T;
  const int64_t len = b - a;
  const int nf = len < n_fft ? 1 : static_cast<int>(1 + (len - n_fft) / hop);
  double* out = part + (static_cast<int64_t>(t) * max_frames + f) * n_bands;
  if (f >= nf) {  // frame slot past this segment's frame count: contributes zero
    for (int i = threadIdx.x; i < n_bands; i += blockDim.x) out[i] = 0.0;
    return;
  }
  const int64_t start = a + static_cast<int64_t>(f) * hop;
  for (int n = tid; n < n_fft; n += kFrameThreads) {
    const int64_t s = start + n;
    const float smp = audio[s < b ? s : b - 1];
    double sn, cs;
    sincospi(2.0 * n / n_fft, &sn, &cs);
    tc[n] = cs;
    ts[n] = sn;
    // periodic Hann; a short segment is padded with zeros
    xw[n] = s < b ? (0.5 - 0.5 * cs) * static_cast<double>(smp) : 0.0;
  }
  for (int k = tid; k < nbins; k += kFrameThreads) bandof[k] = k < half ? band_of_bin(k, n_fft, sr, n_bands) : n_bands - 1;
  __syncthreads();
  for (int n = 1 + tid; n < half; n += kFrameThreads) {
    const double u = xw[n], v = xw[n_fft - n];
    xw[n] = u + v;
    xw[n_fft - n] = u - v;
  }
  band_starts(bandof, nbins, n_bands, first);
  __syncthreads();
  const int g = tid / S;  // terms 1 .. half - 1
  const int per = (half - 1 + G - 1) / G;
  const int n0 = 1 + g * per, n1 = n0 + per < half ? n0 + per : half;
  for (int k0 = 0; k0 < nbins; k0 += S) {
    const int k = k0 + tid % S;
    // four independent partial sums, so that four twiddle reads and FMA chains
    // are in flight at once
    double re[4] = {0.0, 0.0, 0.0, 0.0}, im[4] = {0.0, 0.0, 0.0, 0.0};
    if (k < nbins) {
      int m[4];  // (k * n) mod n_fft for the four current n, advanced by 4k
#pragma unroll
      for (int u = 0; u < 4; ++u) m[u] = (k * (n0 + u)) % n_fft;
      const int step = (4 * k) % n_fft;
      int n = n0;
      for (; n + 4 <= n1; n += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          re[u] = fma(xw[n + u], tc[m[u]], re[u]);
          im[u] = fma(xw[n_fft - n - u], ts[m[u]], im[u]);
          m[u] += step;
          if (m[u] >= n_fft) m[u] -= n_fft;
        }
      }
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (n + u < n1) {
          re[u] = fma(xw[n + u], tc[m[u]], re[u]);
          im[u] = fma(xw[n_fft - n - u], ts[m[u]], im[u]);
        }
    }
    double r = (re[0] + re[1]) + (re[2] + re[3]), i = (im[0] + im[1]) + (im[2] + im[3]);
    if (G > 1) {  // uniform; S >= nbins, one pass
      pre[tid] = r;
      pim[tid] = i;
      __syncthreads();
      for (int h = 1; g == 0 && h < G; ++h) {
        r += pre[tid + h * S];
        i += pim[tid + h * S];
      }
    }
    if (g == 0 && k < nbins) {
      r += xw[0] + ((k & 1) ? -xw[half] : xw[half]);
      pw[k] = r * r + i * i;
    }
  }
  __syncthreads();
  band_sums(pw, first, n_bands, out);
}

// One workgroup: three dependent steps, so that the memory in flight and the
// words between the steps are what it takes; the band sums and the energies
// stay in LDS and registers where they fit (T n_bands <= kLdsSums, T <= the
// threads), in e_scratch otherwise.  21 segments, 8 bands, 21 frames: 2.8 us;
// with 8 loads in flight, band sums through global memory and a tree of
// barriers for the maximum 5.2.
__global__ void __launch_bounds__(kEnergyThreads)
energy_reduce(const double* __restrict__ part, int T, int max_frames, int n_bands,
              float* __restrict__ band_energy, float* __restrict__ frame_energy,
              float* __restrict__ frame_weight, double* __restrict__ e_scratch) {
  __shared__ double sums[kLdsSums];
  __shared__ double red[kEnergyThreads / kWave];
  const int tid = threadIdx.x;
  // (1) one thread per (segment, band): the band's frames summed in frame
  //     order, the loads of kInFlight frames together
  double* bsum = e_scratch + T;
  const bool in_lds = T * n_bands <= kLdsSums;
  constexpr int kInFlight = 24;
  for (int i = tid; i < T * n_bands; i += kEnergyThreads) {
    const int t = i / n_bands, band = i % n_bands;
    const double* src = part + static_cast<int64_t>(t) * max_frames * n_bands + band;
    double acc = 0.0;
    for (int f0 = 0; f0 < max_frames; f0 += kInFlight) {
      double v[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u)
        v[u] = src[static_cast<int64_t>(f0 + u < max_frames ? f0 + u : max_frames - 1) * n_bands];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) acc += f0 + u < max_frames ? v[u] : 0.0;
    }
    if (in_lds) sums[i] = acc;
    else bsum[i] = acc;
    band_energy[i] = static_cast<float>(acc);
  }
  __syncthreads();
  // (2) one thread per segment: its bands in band order
  double local_max = 0.0, e_mine = 0.0;
  for (int t = tid; t < T; t += kEnergyThreads) {
    double tot = 0.0;
    if (in_lds)
      for (int band = 0; band < n_bands; ++band) tot += sums[t * n_bands + band];
    else
      for (int band = 0; band < n_bands; ++band) tot += bsum[t * n_bands + band];
    const double e = sqrt(tot);
    if (t == tid) e_mine = e;
    else e_scratch[t] = e;
    frame_energy[t] = static_cast<float>(e);
    local_max = fmax(local_max, e);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) local_max = fmax(local_max, __shfl_xor(local_max, o));
  if (tid % kWave == 0) red[tid / kWave] = local_max;
  __syncthreads();
  double mx = red[0];
#pragma unroll
  for (int w = 1; w < kEnergyThreads / kWave; ++w) mx = fmax(mx, red[w]);
  for (int t = tid; t < T; t += kEnergyThreads)
    frame_weight[t] = mx > 0.0 ? static_cast<float>((t == tid ? e_mine : e_scratch[t]) / mx) : 1.0f;
}

int energy_max_frames(int64_t n_samples, int T, int n_fft, int hop) {
  // the longest segment has ceil(n / T) samples
  const int64_t longest = (n_samples + T - 1) / T;
  return longest < n_fft ? 1 : static_cast<int>(1 + (longest - n_fft) / hop);
}

hipError_t launch_energy(const float* audio, int64_t n_samples, int T, int sr, int n_fft, int hop,
                         int n_bands, float* band_energy, float* frame_energy, float* frame_weight,
                         double* part, double* e_scratch, hipStream_t stream) {
  const int mf = energy_max_frames(n_samples, T, n_fft, hop);
  hipError_t e;
  if ((n_fft & (n_fft - 1)) == 0) {
    int log2n = 0;
    while ((1 << log2n) < n_fft) ++log2n;
    const size_t lds = sizeof(double) * (3 * n_fft + n_fft / 2 + 1) + sizeof(int) * (n_fft / 2 + 2 + n_bands);
    e = ECHO_LAUNCH("energy_frames", energy_frames_fft, dim3(mf, T), dim3(kFftThreads), lds, stream, audio,
                    n_samples, T, n_fft, log2n, hop, n_bands, sr, mf, part);
  } else {
    const int sums = dft_groups(n_fft / 2 + 1) > 1 ? 2 * kFrameThreads : 0;
    const size_t lds = sizeof(double) * (3 * n_fft + n_fft / 2 + 1 + sums) + sizeof(int) * (n_fft / 2 + 2 + n_bands);
    e = ECHO_LAUNCH("energy_frames", energy_frames, dim3(mf, T), dim3(kFrameThreads), lds, stream, audio,
                    n_samples, T, n_fft, hop, n_bands, sr, mf, part);
  }
  if (e != hipSuccess) return e;
  return ECHO_LAUNCH("energy_reduce", energy_reduce, dim3(1), dim3(kEnergyThreads), 0, stream, part, T,
                     mf, n_bands, band_energy, frame_energy, frame_weight, e_scratch);
}

}  // namespace echo
