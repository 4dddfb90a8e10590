// Auxiliary kernels of the plan: zero fills, per-probe references, the exact
// FP64 mean pre-pass, ring stores for streamed series, per-probe detector
// partial reduction, the exact elastic-mean correction, normalisation and the
// masked detector reduction D_j(m) = sum_k M_j(k) S(m, k) (DetectorSet,
// Sec. II.B.1 of the paper).
#include <algorithm>
#include <type_traits>

#include "tacaw_internal.h"

namespace tacaw {

static inline int blocks_for(int64_t n, int bs, int cap = 65535 * 8) {
  int64_t b = (n + bs - 1) / bs;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

__global__ void fill_zero_kernel(uint4* p, int64_t n16, unsigned char* tail, int ntail) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_fill_zero(void* p, int64_t bytes, hipStream_t st) {
  if (bytes <= 0) return hipSuccess;
  const int64_t n16 = bytes / 16;
  const int ntail = (int)(bytes - n16 * 16);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for(n16, 256, 8192)), dim3(256), 0, st,
                     (uint4*)p, n16, (unsigned char*)p + n16 * 16, ntail);
  return hipGetLastError();
}

// Reference c(k) of a probe: the window-weighted mean of up to kRefSamples
// frames spread over the first chunk (FP64 sum, rounded to FP32 for complex64
// input so that the chunk kernel subtracts exactly this value). Any c keeps the
// mean correction exact; one close to the chunks' own mean keeps the FP32
// transform of psi - c small at bins 0 and +-1, where the correction cancels.
template <typename InT>
__global__ void ref_sampled_kernel(const InT* in, int64_t pstride, int64_t fstride, int32_t nx,
                                   int64_t rs, RefSamples smp, int32_t probe0, int32_t n_probes,
                                   int32_t n_k, double2* cref) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y;
  if (k >= n_k || i >= n_probes) return;
  const InT* src = in + (int64_t)i * pstride + pix_off(k, nx, rs);
  double sx = 0.0, sy = 0.0;
  for (int r = 0; r < smp.n; ++r) {
    const InT v = src[(int64_t)smp.t[r] * fstride];
    sx += smp.wt[r] * (double)v.x;
    sy += smp.wt[r] * (double)v.y;
  }
  sx *= smp.inv_sum;
  sy *= smp.inv_sum;
  if (smp.round32) {
    sx = (double)(float)sx;
    sy = (double)(float)sy;
  }
  cref[(int64_t)(probe0 + i) * n_k + k] = make_double2(sx, sy);
}

hipError_t launch_ref_sampled(const void* in, int in_dtype, int64_t pstride, int64_t fstride,
                              int32_t nx, int64_t rs, const RefSamples& smp, int32_t probe0,
                              int32_t n_probes, int32_t n_k, double2* cref, hipStream_t st) {
  dim3 g((n_k + 255) / 256, n_probes);
  if (in_dtype == 1)
    hipLaunchKernelGGL(ref_sampled_kernel<double2>, g, dim3(256), 0, st, (const double2*)in,
                       pstride, fstride, nx, rs, smp, probe0, n_probes, n_k, cref);
  else
    hipLaunchKernelGGL(ref_sampled_kernel<float2>, g, dim3(256), 0, st, (const float2*)in,
                       pstride, fstride, nx, rs, smp, probe0, n_probes, n_k, cref);
  return hipGetLastError();
}

// Exact FP64 time mean over frames [0, n_used) of each (probe, pixel). Bound by the
// read of the series. A block takes 64 adjacent pixels (512-byte runs of each frame)
// and splits the frames over its kMeanGroups waves, kMeanLoads loads in flight per
// thread; the waves' FP64 sums are added in order through LDS. With one thread per
// pixel for all frames a small grid left the chip idle: 3200 frames of 383^2 pixels
// 1580 -> 704 us (5.3 TB/s), 4 probes x 1024 frames of 48 x 40 268 -> 12 us.
constexpr int kMeanGroups = 16, kMeanLoads = 8;
template <typename InT>
__global__ void __launch_bounds__(64 * kMeanGroups) mean_kernel(
    const InT* __restrict__ in, int64_t pstride, int64_t fstride, int32_t nx, int64_t rs,
    int64_t n_used, int32_t probe0, int32_t n_probes, int32_t n_k, double2* __restrict__ out) {
  __shared__ double2 part[kMeanGroups][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int64_t k = (int64_t)blockIdx.x * 64 + lane;
  const int i = blockIdx.y;
  const bool valid = k < n_k;
  const InT* p = in + (int64_t)i * pstride + pix_off(valid ? k : n_k - 1, nx, rs);
  double sx = 0.0, sy = 0.0;
  int64_t n = g;
  for (; n + (kMeanLoads - 1) * kMeanGroups < n_used; n += kMeanLoads * kMeanGroups) {
    InT v[kMeanLoads];
#pragma unroll
    for (int u = 0; u < kMeanLoads; ++u) v[u] = p[(n + u * kMeanGroups) * fstride];
#pragma unroll
    for (int u = 0; u < kMeanLoads; ++u) {
      sx += (double)v[u].x;
      sy += (double)v[u].y;
    }
  }
  for (; n < n_used; n += kMeanGroups) {
    const InT v = p[n * fstride];
    sx += (double)v.x;
    sy += (double)v.y;
  }
  part[g][lane] = make_double2(sx, sy);
  __syncthreads();
  if (g == 0 && valid) {
#pragma unroll
    for (int r = 1; r < kMeanGroups; ++r) {
      sx += part[r][lane].x;
      sy += part[r][lane].y;
    }
    out[(int64_t)(probe0 + i) * n_k + k] = make_double2(sx / (double)n_used, sy / (double)n_used);
  }
}

hipError_t launch_mean_exact(const void* in, int in_dtype, int64_t pstride, int64_t fstride,
                             int32_t nx, int64_t rs, int64_t n_used, int32_t probe0,
                             int32_t n_probes, int32_t n_k, double2* mu, hipStream_t st) {
  dim3 g((n_k + 63) / 64, n_probes);
  const dim3 b(64 * kMeanGroups);
  if (in_dtype == 1)
    hipLaunchKernelGGL(mean_kernel<double2>, g, b, 0, st, (const double2*)in, pstride, fstride, nx,
                       rs, n_used, probe0, n_probes, n_k, mu);
  else
    hipLaunchKernelGGL(mean_kernel<float2>, g, b, 0, st, (const float2*)in, pstride, fstride, nx,
                       rs, n_used, probe0, n_probes, n_k, mu);
  return hipGetLastError();
}

hipError_t launch_ref_mean(const void* in, int in_dtype, int64_t pstride, int64_t fstride,
                           int32_t nx, int64_t rs, int64_t n_used, int32_t probe0,
                           int32_t n_probes, int32_t n_k, double2* cref, hipStream_t st) {
  return launch_mean_exact(in, in_dtype, pstride, fstride, nx, rs, n_used, probe0, n_probes, n_k,
                           cref, st);
}

// ring[slot][f % D][k] = in[i][f - push_begin][k] for f in [f_lo, f_hi); each
// thread copies 16 bytes (two complex64 or one complex128 element).
template <typename InT>
__global__ void ring_store_kernel(const InT* in, int64_t pstride, int64_t fstride, int32_t nx,
                                  int64_t rs, int64_t push_begin, int64_t f_lo, int32_t n_f,
                                  int32_t probe0, int32_t n_slots, int64_t depth, int32_t n_k,
                                  InT* ring) {
  constexpr int V = 16 / (int)sizeof(InT);  // elements per thread
  const int64_t k0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
  const int fi = blockIdx.y;
  const int i = blockIdx.z;
  if (k0 >= n_k || fi >= n_f) return;
  const int64_t f = f_lo + fi;
  const int slot = (probe0 + i) % n_slots;
  InT* dst = ring + ((int64_t)slot * depth + (f % depth)) * n_k;
  const InT* src = in + (int64_t)i * pstride + (f - push_begin) * fstride;
#pragma unroll
  for (int v = 0; v < V; ++v)
    if (k0 + v < n_k) dst[k0 + v] = src[pix_off(k0 + v, nx, rs)];
}

// The same into a ring stored per pixel tile: element (slot, row, k) at
// ((slot * n_tiles + k / W) * D + row) * W + k % W. A block moves R consecutive frames
// (R = 16, or the largest power of two dividing D; the first frame aligned to R in
// absolute frame index) of 1 KiB of pixels through LDS: a wave reads 1 KiB of one
// frame and writes 1 KiB of consecutive rows of a tile (64 R bytes at W = 8; half rows
// where a row is 2 KiB), so both sides are whole lines. Bound by memory. Copying straight
// from frames to rows gave each wave four 256-byte reads and 16 separate 64-byte rows: 2
// probes x 256 frames of 1024^2 pixels, 4.3 GB in and out, 2190 us, now 2000 us (4.3 TB/s;
// a plain copy reaches 4.76).
// VEC: frames are contiguous and pixels come in pairs (complex64), so a thread moves
// 16 bytes; otherwise element by element.
constexpr int kStorePx = 1024;  // bytes of a frame per block
template <typename InT, bool VEC>
__global__ void __launch_bounds__(256) ring_store_tiled_kernel(
    const InT* __restrict__ in, int64_t pstride, int64_t fstride, int32_t nx, int64_t rs,
    int64_t push_begin, int64_t f_lo, int64_t f_hi, int32_t R, int32_t probe0, int32_t n_slots,
    int64_t depth, int32_t n_k, int32_t tile_w, int32_t n_tiles, InT* __restrict__ ring) {
  constexpr int V = 16 / (int)sizeof(InT);                // elements per 16 bytes
  constexpr int PX = kStorePx / (int)sizeof(InT);         // pixels of a block
  constexpr int LROW = kStorePx / 16 + 4;                 // 16-byte words per frame, padded
  __shared__ uint4 buf[16 * LROW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t fb = (f_lo - f_lo % R) + (int64_t)blockIdx.y * R;  // the block's first frame
  const int i = blockIdx.z;
  const int64_t kb = (int64_t)blockIdx.x * PX;
  const InT* src = in + (int64_t)i * pstride;
  for (int r = wave; r < R; r += 4) {
    const int64_t f = fb + r;
    if (f < f_lo || f >= f_hi) continue;  // uniform per wave
    const int64_t k0 = kb + lane * V;
    InT e[V];
    if (VEC && k0 + V <= n_k) {
      __builtin_memcpy(e, src + (f - push_begin) * fstride + k0, 16);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (k0 + v < n_k) e[v] = src[(f - push_begin) * fstride + pix_off(k0 + v, nx, rs)];
    }
    __builtin_memcpy(&buf[r * LROW + lane], e, 16);
  }
  __syncthreads();
  const int slot = (probe0 + i) % n_slots;
  const int run = min(tile_w, PX);            // pixels of a tile row in this block
  const int wpr = run / V;                    // 16-byte words of that run
  const int n_words = R * (kStorePx / 16);    // words of the block, [tile][row][word]
  const int64_t row0 = fb % depth;            // R divides D and fb: the rows do not wrap
  for (int e = threadIdx.x; e < n_words; e += 256) {
    const int part = e % wpr, r = (e / wpr) % R, t = e / (wpr * R);
    const int64_t k0 = kb + (int64_t)t * run + part * V;
    const int64_t f = fb + r;
    if (k0 >= n_k || f < f_lo || f >= f_hi) continue;
    InT x[V];
    __builtin_memcpy(x, &buf[r * LROW + t * wpr + part], 16);
    const int64_t tile = k0 / tile_w;
    InT* dst = ring + (((int64_t)slot * n_tiles + tile) * depth + row0 + r) * tile_w + (k0 - tile * tile_w);
    if (k0 + V <= n_k) {
      __builtin_memcpy(dst, x, 16);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (k0 + v < n_k) dst[v] = x[v];
    }
  }
}

hipError_t launch_ring_store(const void* in, int in_dtype, int64_t pstride, int64_t fstride,
                             int32_t nx, int64_t rs, int64_t push_begin, int64_t f_lo,
                             int64_t f_hi, int32_t probe0, int32_t n_probes, int32_t n_slots,
                             int64_t depth, int32_t n_k, int32_t tile_w, void* ring,
                             hipStream_t st) {
  const int64_t nf = f_hi - f_lo;
  if (nf <= 0) return hipSuccess;
  if (tile_w > 0) {
    int R = 16;  // halved until it divides D
    while (depth % R != 0) R /= 2;
    const int esz = in_dtype == 1 ? 16 : 8;
    const int px = kStorePx / esz;
    // a block holds whole tile rows, or (128-pixel tiles of complex128) a part of one
    if ((px % tile_w != 0 && tile_w % px != 0) || tile_w % (16 / esz) != 0)
      return hipErrorInvalidValue;
    const int32_t n_tiles = (n_k + tile_w - 1) / tile_w;
    const int64_t fb = f_lo - f_lo % R;
    const dim3 g((unsigned)((n_k + px - 1) / px), (unsigned)((f_hi - fb + R - 1) / R), n_probes);
    const bool vec = rs == nx;
    auto go = [&](auto in_t, auto vec_c) {
      using T = decltype(in_t);
      hipLaunchKernelGGL((ring_store_tiled_kernel<T, decltype(vec_c)::value>), g, dim3(256), 0, st,
                         (const T*)in, pstride, fstride, nx, rs, push_begin, f_lo, f_hi, R, probe0,
                         n_slots, depth, n_k, tile_w, n_tiles, (T*)ring);
    };
    if (in_dtype == 1) {
      if (vec) go(double2{}, std::true_type{});
      else go(double2{}, std::false_type{});
    } else {
      if (vec) go(float2{}, std::true_type{});
      else go(float2{}, std::false_type{});
    }
    return hipGetLastError();
  }
  const int V = in_dtype == 1 ? 1 : 2;
  dim3 g((unsigned)((n_k + 256 * V - 1) / (256 * V)), (unsigned)nf, n_probes);
  if (in_dtype == 1)
    hipLaunchKernelGGL(ring_store_kernel<double2>, g, dim3(256), 0, st, (const double2*)in,
                       pstride, fstride, nx, rs, push_begin, f_lo, (int32_t)nf, probe0, n_slots,
                       depth, n_k, (double2*)ring);
  else
    hipLaunchKernelGGL(ring_store_kernel<float2>, g, dim3(256), 0, st, (const float2*)in, pstride,
                       fstride, nx, rs, push_begin, f_lo, (int32_t)nf, probe0, n_slots, depth,
                       n_k, (float2*)ring);
  return hipGetLastError();
}

// Per-probe detector spectra from the cumulative (tile, detector) partials:
// Dp[d][probe0 + i][m] += sum over the slots s of detector d of
// (part[s][i][m] - part[s][i-1][m]). Block (m-range, d, g) sums a group of at
// most `per` slots, reads every partial once and adds its per-probe differences
// atomically (groups run in parallel).
// Bound by latency, then by the read of the partials: the kPartSlots loads of a probe
// are independent, and four probes are unrolled, so 32 loads per thread are in
// flight. With a loop of runtime length over the slots each load waited for the one
// before: 295 MB of partials (32 probes, 512 bins, 4 masks on 256^2 pixels) 146 us,
// now 101 us (2.9 TB/s); 16 probes of 128^2 57 us, now 18 us.
constexpr int kPartSlots = 8;
__global__ void __launch_bounds__(128) dpart_reduce_kernel(const double* __restrict__ part,
                                                           DetSlots so, int32_t per,
                                                           int32_t n_probes, int32_t n_om,
                                                           int32_t probe0, int32_t n_probe_total,
                                                           double* __restrict__ Dp) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  const int d = blockIdx.y;
  const int g = blockIdx.z;
  if (m >= n_om) return;
  const int s0 = so.off[d] + g * per, s1 = min(so.off[d + 1], s0 + per);
  if (s0 >= s1) return;
  const int64_t per_slot = (int64_t)n_probes * n_om;
  double prev = 0.0;
  if (per == kPartSlots) {
#pragma unroll 4
    for (int i = 0; i < n_probes; ++i) {
      const double* base = part + (int64_t)i * n_om + m;
      double v[kPartSlots], cur = 0.0;
#pragma unroll
      for (int u = 0; u < kPartSlots; ++u)
        v[u] = base[min(s0 + u, s1 - 1) * per_slot];
#pragma unroll
      for (int u = 0; u < kPartSlots; ++u) cur += s0 + u < s1 ? v[u] : 0.0;
      atomicAdd(&Dp[((int64_t)d * n_probe_total + probe0 + i) * n_om + m], cur - prev);
      prev = cur;
    }
    return;
  }
  for (int i = 0; i < n_probes; ++i) {
    const double* base = part + (int64_t)i * n_om + m;
    double cur = 0.0;
    for (int s = s0; s < s1; s += kPartSlots) {
      double v[kPartSlots];
#pragma unroll
      for (int u = 0; u < kPartSlots; ++u) v[u] = base[min(s + u, s1 - 1) * per_slot];
#pragma unroll
      for (int u = 0; u < kPartSlots; ++u) cur += s + u < s1 ? v[u] : 0.0;
    }
    atomicAdd(&Dp[((int64_t)d * n_probe_total + probe0 + i) * n_om + m], cur - prev);
    prev = cur;
  }
}

hipError_t launch_dpart_reduce(const double* dpart, const DetSlots& so, int32_t n_probes,
                               int32_t n_det, int32_t n_om, int32_t probe0, int32_t n_probe_total,
                               double* Dp, hipStream_t st) {
  int most = 0;
  for (int d = 0; d < n_det; ++d) most = max(most, so.off[d + 1] - so.off[d]);
  if (most == 0) return hipSuccess;
  int per = kPartSlots;  // slots per block: enough blocks to fill the chip, few atomics per value
  if ((most + per - 1) / per > 1024) per = (most + 1023) / 1024;
  dim3 g((n_om + 127) / 128, n_det, (most + per - 1) / per);
  hipLaunchKernelGGL(dpart_reduce_kernel, g, dim3(128), 0, st, dpart, so, per, n_probes, n_om,
                     probe0, n_probe_total, Dp);
  return hipGetLastError();
}

// ---- exact elastic-mean correction -----------------------------------------
// For chunk spectra of the reference-subtracted series X'_s and the true
// mean-subtracted X_s = X'_s - delta W (delta = mu - c):
//   sum_s |X_s|^2 = sum_s |X'_s|^2 - 2 Re(conj(delta W) sum_s X'_s) + N_s |delta W|^2
__device__ __forceinline__ double corr_term(const CorrArgs& c, int p, int64_t k, int b) {
  if (c.pcorr) return c.pcorr[((int64_t)p * kMaxCorr + b) * c.n_k + k];
  const double2 cr = c.cref[(int64_t)p * c.n_k + k];
  double2 delta;
  if (c.mean_global) {
    const double2 ms = c.msum[(int64_t)p * c.n_k + k];
    delta = make_double2(ms.x * c.inv_nused, ms.y * c.inv_nused);
  } else {
    delta = make_double2(-cr.x, -cr.y);
  }
  const double2 w = c.wbin[b];
  const double2 dw = make_double2(delta.x * w.x - delta.y * w.y, delta.x * w.y + delta.y * w.x);
  const double2 xs = c.xs[((int64_t)p * kMaxCorr + b) * c.n_k + k];
  // Re(conj(dw) * xs) = dw.x xs.x + dw.y xs.y
  return -2.0 * (dw.x * xs.x + dw.y * xs.y) + c.n_seg * (dw.x * dw.x + dw.y * dw.y);
}

// Dp[d][p][bin_b] += sum_k M_d(k) corr_p(b, k). A block takes kCorrPix pixels of one
// probe; its sums stay in registers (all detector and bin indexes are compile-time),
// are reduced across each wave with lane shuffles and added with one atomic per
// block, detector and bin. Before, runtime-indexed sums lived in scratch and were
// reduced one by one through LDS: 31 us for one probe of 64^2 pixels and one mask,
// now 8.4 us.
constexpr int kCorrPix = 1024;
__global__ void __launch_bounds__(256) correct_Dp_kernel(const CorrArgs c,
                                                         const double* __restrict__ masks,
                                                         int32_t n_det, double* Dp) {
  const int p = blockIdx.y;
  __shared__ double red[4][kMaxDet * kMaxCorr];
  double accd[kMaxDet][kMaxCorr];
#pragma unroll
  for (int d = 0; d < kMaxDet; ++d)
#pragma unroll
    for (int b = 0; b < kMaxCorr; ++b) accd[d][b] = 0.0;
  const int64_t k0 = (int64_t)blockIdx.x * kCorrPix + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kCorrPix / 256; ++u) {
    const int64_t k = k0 + 256 * u;
    if (k < c.n_k) {
      double ct[kMaxCorr];
#pragma unroll
      for (int b = 0; b < kMaxCorr; ++b) ct[b] = (b < c.n_corr) ? corr_term(c, p, k, b) : 0.0;
#pragma unroll
      for (int d = 0; d < kMaxDet; ++d) {
        if (d < n_det) {
          const double m = masks[(int64_t)d * c.n_k + k];
#pragma unroll
          for (int b = 0; b < kMaxCorr; ++b) accd[d][b] += m * ct[b];
        }
      }
    }
  }
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < kMaxDet; ++d) {
    if (d < n_det) {
#pragma unroll
      for (int b = 0; b < kMaxCorr; ++b) {
        double v = accd[d][b];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((threadIdx.x & 63) == 0) red[wave][d * kMaxCorr + b] = v;
      }
    }
  }
  __syncthreads();
  const int e = threadIdx.x;
  if (e < n_det * kMaxCorr && e % kMaxCorr < c.n_corr) {
    const int b = e % kMaxCorr, row = b == 0 ? c.rows[0] : b == 1 ? c.rows[1] : c.rows[2];
    atomicAdd(&Dp[((int64_t)(e / kMaxCorr) * c.n_probe + p) * c.n_om + row],
              (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]));
  }
}

hipError_t launch_correct_Dp(const CorrArgs& c, const double* masks, int32_t n_det, double* Dp,
                             hipStream_t st) {
  const int gx = (c.n_k + kCorrPix - 1) / kCorrPix;
  hipLaunchKernelGGL(correct_Dp_kernel, dim3(gx, c.n_probe), dim3(256), 0, st, c, masks, n_det, Dp);
  return hipGetLastError();
}

// ---- per-chunk mean --------------------------------------------------------
// With its own mean mu_s subtracted, chunk s has at a correction bin b
//   X_s(b) = A_s(b) - delta_s W(b),  A_s(b) = sum_t w(t) e^{-2 pi i b t / L} y'(s H + t),
// where y' = psi - c and delta_s = mu_s - c = (1/L) sum_t y'(s H + t). The chunk
// kernel leaves these bins out of S in this mode; this kernel adds the whole
// sum_s |X_s(b)|^2, formed in FP64 from exact FP64 sums.
// One thread per (probe, pixel) walks the push's frames in time order; the V
// chunks that can hold a frame live in V register slots (chunk s in slot s mod V),
// a chunk's sums are cleared at its first frame and turned into its correction
// at its last. Open sums persist in `open` between pushes.
// Bound by the read of the push. The fast variant keeps its window tables in LDS and
// loads the next kPsegB frames while it adds the current ones. Before, the tables
// came by scalar loads that each batch waited for (16 KB of tables in a 16 KB scalar
// cache), and no load was in flight during the sums: 8 probes x 2048 frames of 256^2,
// L = 512, 8.6 GB: 3420 us, now 1910 us (4.5 TB/s).
constexpr int kPsegU = 16;  // frames in flight per thread (general variant)
constexpr int kPsegB = 8;   // frames per batch of the fast variant, the next one in flight
constexpr int kPsegMaxL = 1024;
template <typename InT, int V, bool FAST>
__global__ void __launch_bounds__(256) pseg_kernel(const PsegArgs a) {
  // Slot state (four double2): the chunk sum of y'; A(0); (P, Q); (R, T) with
  // P = sum e_r y_r, Q = sum e_i y_i, R = sum e_r y_i, T = sum e_i y_r and
  // e = w(t) exp(-2 pi i t / L). The window is real, so bins 1 and L - 1 share
  // them: A(1) = (P - Q, R + T), A(L - 1) = conj(e) y summed = (P + Q, R - T).
  constexpr int Q = 4;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y;
  // fast variant: the window tables in LDS
  __shared__ double s_w[FAST ? kPsegMaxL : 1];
  __shared__ double2 s_e[FAST ? kPsegMaxL : 1];
  if constexpr (FAST) {
    for (int t = threadIdx.x; t < a.L; t += blockDim.x) {
      s_w[t] = a.tw[t].x;
      s_e[t] = a.tw[a.L + t];
    }
    __syncthreads();
  }
  if (k >= a.n_k || i >= a.n_probes) return;
  const int p = a.probe0 + i;
  const InT* src = (const InT*)a.in + (int64_t)i * a.pstride + pix_off(k, a.nx, a.rs);
  const double2 c = a.cref[(int64_t)p * a.n_k + k];
  double2* op = a.open + (int64_t)p * V * Q * a.n_k + k;
  double* cp = a.pcorr + (int64_t)p * kMaxCorr * a.n_k + k;
  double2 st[V][Q];
  double cor[kMaxCorr];
#pragma unroll
  for (int r = 0; r < V; ++r)
#pragma unroll
    for (int q = 0; q < Q; ++q)
      st[r][q] = a.f_lo == 0 ? make_double2(0.0, 0.0) : op[(int64_t)(r * Q + q) * a.n_k];
#pragma unroll
  for (int b = 0; b < kMaxCorr; ++b) cor[b] = a.f_lo == 0 ? 0.0 : cp[(int64_t)b * a.n_k];
  const bool three = a.n_corr == 3;
  const double inv_l = 1.0 / (double)a.L;
  const double* w0 = (const double*)a.tw;  // w(t) = Re tw[0][t], stride 2
  const double2* e1 = a.tw + a.L;         // w(t) exp(-2 pi i t / L)
  constexpr int U = kPsegU;
  // add chunk s's correction from its finished sums and keep its mean
  auto close = [&](const double2 (&z)[Q], int s) {
    const double dx = z[0].x * inv_l, dy = z[0].y * inv_l;
    a.cmean[((int64_t)p * a.Ns + s) * a.n_k + k] = make_double2(c.x + dx, c.y + dy);
    double2 A[kMaxCorr];
    A[0] = z[1];
    A[1] = make_double2(z[2].x - z[2].y, z[3].x + z[3].y);
    A[2] = make_double2(z[2].x + z[2].y, z[3].x - z[3].y);
#pragma unroll
    for (int b = 0; b < kMaxCorr; ++b) {
      if (b == 0 || three) {
        const double2 wb = a.wbin[b];
        const double wx = dx * wb.x - dy * wb.y, wy = dx * wb.y + dy * wb.x;
        const double xr = A[b].x - wx, xi = A[b].y - wy;  // X_s(b) = A_s(b) - delta_s W(b)
        cor[b] += xr * xr + xi * xi;
      }
    }
  };
  if constexpr (FAST) {
    // H divides L (FAST is chosen when L = V H): frame n = j H + u lies in chunks
    // j - q, q = 0..V-1, at t = q H + u, so inside a hop block every frame updates
    // the same V sums with no bookkeeping; chunk j starts at u = 0 and chunk
    // j - V + 1 ends after u = H - 1. Register sq[q] holds chunk j - q (HBM slot
    // (j - q) mod V); sums of chunks that do not exist (j - q < 0, or past the
    // last chunk) are never closed.
    double2 sq[V][Q];
    const int jb = (int)(a.f_lo / a.H);
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int slot = ((jb - q) % V + V) % V;
#pragma unroll
      for (int z = 0; z < Q; ++z) sq[q][z] = st[0][z];
#pragma unroll
      for (int r = 1; r < V; ++r)
        if (slot == r)
#pragma unroll
          for (int z = 0; z < Q; ++z) sq[q][z] = st[r][z];
    }
    constexpr int B = kPsegB;
    InT nxt[B];
    auto fetch = [&](int64_t n0) {
#pragma unroll
      for (int x = 0; x < B; ++x)
        if (n0 + x < a.f_hi) nxt[x] = src[(n0 + x - a.base) * a.fstride];
    };
    int64_t n = a.f_lo;
    fetch(n);
    int j = jb;
    int u0 = (int)(n - (int64_t)j * a.H);
    while (n < a.f_hi) {
      // frames n .. n + cnt of hop block j
      const int cnt = (int)min<int64_t>(min(B, a.H - u0), a.f_hi - n);
      InT v[B];
#pragma unroll
      for (int x = 0; x < B; ++x) v[x] = nxt[x];
      if (n + cnt < a.f_hi) fetch(n + cnt);
      if (u0 == 0) {
#pragma unroll
        for (int z = 0; z < Q; ++z) sq[0][z] = make_double2(0.0, 0.0);
      }
      auto add = [&](int x) {
        const double yr = (double)v[x].x - c.x, yi = (double)v[x].y - c.y;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const int t = q * a.H + u0 + x;
          const double w = s_w[t];
          sq[q][0].x += yr;
          sq[q][0].y += yi;
          sq[q][1].x += w * yr;
          sq[q][1].y += w * yi;
          if (three) {
            const double2 e = s_e[t];
            sq[q][2].x += e.x * yr;
            sq[q][2].y += e.y * yi;
            sq[q][3].x += e.x * yi;
            sq[q][3].y += e.y * yr;
          }
        }
      };
      if (cnt == B) {
#pragma unroll
        for (int x = 0; x < B; ++x) add(x);
      } else {
#pragma unroll
        for (int x = 0; x < B; ++x)
          if (x < cnt) add(x);
      }
      n += cnt;
      u0 += cnt;
      if (u0 == a.H) {  // hop block j is complete
        const int s_end = j - (V - 1);
        if (s_end >= 0 && s_end < a.Ns) close(sq[V - 1], s_end);
#pragma unroll
        for (int q = V - 1; q > 0; --q)
#pragma unroll
          for (int z = 0; z < Q; ++z) sq[q][z] = sq[q - 1][z];
        u0 = 0;
        ++j;
      }
    }
    // back to HBM slots: register q now holds chunk je - q
    const int je = (int)(a.f_hi / a.H);
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int slot = ((je - q) % V + V) % V;
#pragma unroll
      for (int z = 0; z < Q; ++z) op[(int64_t)(slot * Q + z) * a.n_k] = sq[q][z];
    }
#pragma unroll
    for (int b = 0; b < kMaxCorr; ++b) cp[(int64_t)b * a.n_k] = cor[b];
    return;
  } else {
  for (int64_t n0 = a.f_lo; n0 < a.f_hi; n0 += U) {
    InT v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (n0 + u < a.f_hi) v[u] = src[(n0 + u - a.base) * a.fstride];
    // uniform bookkeeping: frame n = n0 + u lies after chunk start sl * H + rem
    int sl = (int)(n0 / a.H);
    int rem = (int)(n0 - (int64_t)sl * a.H);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (n0 + u >= a.f_hi) break;
      const int n = (int)(n0 + u);  // frames below 2^31 (checked by the plan)
      const double yr = (double)v[u].x - c.x, yi = (double)v[u].y - c.y;
      const int smax = min(a.Ns - 1, sl);  // the latest chunk that has started
#pragma unroll
      for (int r = 0; r < V; ++r) {
        const int s = smax - (((smax - r) % V) + V) % V;  // the chunk in slot r
        const int t = n - s * a.H;
        if (s < 0 || t >= a.L) continue;  // no chunk of slot r holds frame n
        if (t == 0) {
#pragma unroll
          for (int q = 0; q < Q; ++q) st[r][q] = make_double2(0.0, 0.0);
        }
        const double w = w0[2 * t];
        st[r][0].x += yr;
        st[r][0].y += yi;
        st[r][1].x += w * yr;
        st[r][1].y += w * yi;
        if (three) {
          const double2 e = e1[t];
          st[r][2].x += e.x * yr;
          st[r][2].y += e.y * yi;
          st[r][3].x += e.x * yi;
          st[r][3].y += e.y * yr;
        }
        if (t == a.L - 1) close(st[r], s);
      }
      if (++rem == a.H) {
        rem = 0;
        ++sl;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < V; ++r)
#pragma unroll
    for (int q = 0; q < Q; ++q) op[(int64_t)(r * Q + q) * a.n_k] = st[r][q];
#pragma unroll
  for (int b = 0; b < kMaxCorr; ++b) cp[(int64_t)b * a.n_k] = cor[b];
  }
}

hipError_t launch_pseg(const PsegArgs& a, int32_t in_dtype, hipStream_t st) {
  if (a.f_hi <= a.f_lo || a.n_probes < 1) return hipSuccess;
  if (a.V < 1 || a.V > kMaxPsegOpen) return hipErrorInvalidValue;
  dim3 g((a.n_k + 255) / 256, a.n_probes);
  const bool fast = a.L == a.V * a.H;
  auto go = [&](auto vt) {
    constexpr int V = decltype(vt)::value;
    if (in_dtype == 1) {
      if (fast)
        hipLaunchKernelGGL((pseg_kernel<double2, V, true>), g, dim3(256), 0, st, a);
      else
        hipLaunchKernelGGL((pseg_kernel<double2, V, false>), g, dim3(256), 0, st, a);
    } else {
      if (fast)
        hipLaunchKernelGGL((pseg_kernel<float2, V, true>), g, dim3(256), 0, st, a);
      else
        hipLaunchKernelGGL((pseg_kernel<float2, V, false>), g, dim3(256), 0, st, a);
    }
  };
  switch (a.V) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    default: go(std::integral_constant<int, 4>{}); break;
  }
  return hipGetLastError();
}

// ---- HBM read ceiling ------------------------------------------------------
// Grid-stride read of 16-byte words, TACAW_READ_U independent loads per thread
// and trip, summed as 64-bit words (wrapping); one atomic per block.
#ifndef TACAW_READ_U
#define TACAW_READ_U 16
#endif
__global__ void __launch_bounds__(256) read_probe_kernel(const uint4* __restrict__ p, int64_t n16,
                                                         unsigned long long* sum) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long acc = 0;
  auto add = [&](const uint4 v) {
    acc += ((unsigned long long)v.y << 32 | v.x) + ((unsigned long long)v.w << 32 | v.z);
  };
  constexpr int U = TACAW_READ_U;
  for (; i + (U - 1) * stride < n16; i += U * stride) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[i + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) add(v[u]);
  }
  for (; i < n16; i += stride) add(p[i]);
  __shared__ unsigned long long red[256];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(sum, red[0]);
}

hipError_t launch_read_probe(const void* p, int64_t bytes, uint64_t* sum, hipStream_t st) {
  hipError_t e = launch_fill_zero(sum, 8, st);
  if (e != hipSuccess) return e;
  const int64_t n16 = bytes / 16;
  const int64_t want = (n16 + TACAW_READ_U * 256 - 1) / (TACAW_READ_U * 256);
  const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(want, 256 * 32));
  hipLaunchKernelGGL(read_probe_kernel, dim3(blocks), dim3(256), 0, st, (const uint4*)p, n16,
                     (unsigned long long*)sum);
  return hipGetLastError();
}

// Column pattern, the chunk transform's loads without its arithmetic: the rows
// (frames) of row_bytes are cut into columns seg_bytes wide (pixel tiles). One
// 512-thread workgroup per column walks all rows; a thread takes 8 bytes,
// seg_bytes / 8 lanes share a row, so a wave load spans 64 / (seg_bytes / 8) rows,
// and 8 row passes are in flight. The workgroup reserves most of the LDS so
// that, like the chunk transform, one runs per CU.
constexpr int kColThreads = 512;
constexpr int kColLds = 96 * 1024;
__global__ void __launch_bounds__(kColThreads) read_probe_columns_kernel(
    const char* __restrict__ p, int64_t n_rows, int64_t row_bytes, int32_t lanes,
    unsigned long long* sum) {
  constexpr int U = 8;
  __shared__ unsigned long long red[kColLds / 8];  // only the first kColThreads are used
  const int rows_per_pass = kColThreads / lanes;
  const int lane = threadIdx.x % lanes, r_off = threadIdx.x / lanes;
  const char* colp = p + (int64_t)blockIdx.x * lanes * 8 + lane * 8;
  unsigned long long acc = 0;
  for (int64_t r0 = r_off; r0 < n_rows; r0 += (int64_t)U * rows_per_pass) {
    unsigned long long v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = r0 + (int64_t)u * rows_per_pass;
      v[u] = r < n_rows ? *(const unsigned long long*)(colp + r * row_bytes) : 0ull;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kColThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(sum, red[0]);
}

hipError_t launch_read_probe_columns(const void* p, int64_t n_rows, int64_t row_bytes,
                                     int32_t seg_bytes, uint64_t* sum, hipStream_t st) {
  hipError_t e = launch_fill_zero(sum, 8, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(read_probe_columns_kernel, dim3((unsigned)(row_bytes / seg_bytes)),
                     dim3(kColThreads), 0, st, (const char*)p, n_rows, row_bytes,
                     seg_bytes / 8, (unsigned long long*)sum);
  return hipGetLastError();
}

// Row factor of the normalised spectrum: S is kept as accumulated, and every reader
// multiplies by it (the same product that a stored normalised copy would hold).
__device__ __forceinline__ double row_factor(double kappa, const double* q, int row) {
  return q ? kappa * q[row] : kappa;
}

// One launch for the whole end of a reduction. Block row y < n_om: output row
// row = (y + the first correction row) mod n_om, so that the correction rows, whose
// blocks walk all probes, start first; S of those rows gets its correction, and out
// = S times the row factor. Further block rows normalise D_p. Bound by memory: S is
// read once and out written once (8 + 8 bytes per value); before, a launch per
// step, and S read, written back normalised and copied: 222 us for 32 probes of
// 256^2 and 512 bins, now 148 us (3.6 TB/s).
constexpr int kFinV = 4;  // values per thread
template <bool CORR>
__global__ void __launch_bounds__(256) finalize_kernel(const CorrArgs c, double* S, double* out,
                                                       double kappa, const double* q, double* Dp,
                                                       int64_t n_dp, double kappa_p) {
  const int y = blockIdx.y;
  if (y >= c.n_om) {
    const int64_t stride = (int64_t)(gridDim.y - c.n_om) * gridDim.x * 256;
    for (int64_t i = ((int64_t)(y - c.n_om) * gridDim.x + blockIdx.x) * 256 + threadIdx.x; i < n_dp;
         i += stride)
      Dp[i] *= row_factor(kappa_p, q, (int)(i % c.n_om));
    return;
  }
  int row = y + (CORR ? c.rows[2] : 0);
  if (row >= c.n_om) row -= c.n_om;
  int b = -1;  // correction bin of this row
  if constexpr (CORR) {
#pragma unroll
    for (int e = 0; e < kMaxCorr; ++e)
      if (e < c.n_corr && c.rows[e] == row) b = e;
  }
  if (b < 0 && !out) return;
  const double f = row_factor(kappa, q, row);
  const int64_t k0 = (int64_t)blockIdx.x * (256 * kFinV) + threadIdx.x;
  double* const Sr = S + (int64_t)row * c.n_k;
  double v[kFinV];
#pragma unroll
  for (int u = 0; u < kFinV; ++u) v[u] = k0 + 256 * u < c.n_k ? Sr[k0 + 256 * u] : 0.0;
  if constexpr (CORR) {
    if (b >= 0) {
      double sum[kFinV];
#pragma unroll
      for (int u = 0; u < kFinV; ++u) sum[u] = 0.0;
#pragma unroll 2
      for (int p = 0; p < c.n_probe; ++p)
#pragma unroll
        for (int u = 0; u < kFinV; ++u)
          sum[u] += corr_term(c, p, min(k0 + 256 * u, (int64_t)c.n_k - 1), b);
#pragma unroll
      for (int u = 0; u < kFinV; ++u) {
        v[u] += sum[u];
        if (k0 + 256 * u < c.n_k) Sr[k0 + 256 * u] = v[u];
      }
    }
  }
  if (out) {
    double* const o = out + (int64_t)row * c.n_k;
#pragma unroll
    for (int u = 0; u < kFinV; ++u)
      if (k0 + 256 * u < c.n_k) o[k0 + 256 * u] = v[u] * f;
  }
}

hipError_t launch_finalize(const CorrArgs& c, bool corr, double* S, double* out, double kappa,
                           const double* q, double* Dp, int64_t n_dp, double kappa_p,
                           hipStream_t st) {
  const unsigned gx = (unsigned)((c.n_k + 256 * kFinV - 1) / (256 * kFinV));
  const int64_t dp_rows = std::min<int64_t>((n_dp + 256 * (int64_t)gx - 1) / (256 * (int64_t)gx), 1024);
  const dim3 g(gx, (unsigned)(c.n_om + dp_rows));
  if (corr)
    hipLaunchKernelGGL(finalize_kernel<true>, g, dim3(256), 0, st, c, S, out, kappa, q, Dp, n_dp, kappa_p);
  else
    hipLaunchKernelGGL(finalize_kernel<false>, g, dim3(256), 0, st, c, S, out, kappa, q, Dp, n_dp, kappa_p);
  return hipGetLastError();
}

// Before the detector sums: D zeroed for their atomics, and D_p copied out
__global__ void detector_prep_kernel(double* D, int64_t n_d, const double* __restrict__ src,
                                     double* __restrict__ dst, int64_t n_dp) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < n_d; i += stride) D[i] = 0.0;
  for (int64_t i = i0; i < n_dp; i += stride) dst[i] = src[i];
}

hipError_t launch_detector_prep(double* D, int64_t n_d, const double* src, double* dst, int64_t n_dp,
                                hipStream_t st) {
  const int64_t n = std::max(n_d, n_dp);
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(detector_prep_kernel, dim3(blocks_for(n, 256, 2048)), dim3(256), 0, st, D, n_d,
                     src, dst, n_dp);
  return hipGetLastError();
}

// D[d][m] += sum over a pixel chunk of M_d(k) S(m, k): each block takes kDetBins
// bins and a chunk of pixels (coalesced rows of S), reduces across each wave
// with lane shuffles and adds one value per (block, bin, detector) atomically.
constexpr int kDetBins = 4;
template <int ND>
__global__ void detector_kernel(const double* S, const double* masks, int32_t L, int32_t n_k,
                                int32_t chunk, double kappa, const double* q, double* D) {
  const int m0 = blockIdx.y * kDetBins;
  const int64_t k0 = (int64_t)blockIdx.x * chunk;
  const int64_t k1 = (k0 + chunk < n_k) ? k0 + chunk : n_k;
  __shared__ double red[4][kDetBins * ND];  // blocks of 4 waves
  double acc[kDetBins][ND], f[kDetBins];
#pragma unroll
  for (int b = 0; b < kDetBins; ++b) {
    f[b] = m0 + b < L ? row_factor(kappa, q, m0 + b) : 0.0;
#pragma unroll
    for (int d = 0; d < ND; ++d) acc[b][d] = 0.0;
  }
  for (int64_t k = k0 + threadIdx.x; k < k1; k += blockDim.x) {
    double mk[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) mk[d] = masks[(int64_t)d * n_k + k];
#pragma unroll
    for (int b = 0; b < kDetBins; ++b) {
      const double sv = (m0 + b < L) ? S[(int64_t)(m0 + b) * n_k + k] * f[b] : 0.0;
#pragma unroll
      for (int d = 0; d < ND; ++d) acc[b][d] += mk[d] * sv;
    }
  }
#pragma unroll
  for (int b = 0; b < kDetBins; ++b) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      double v = acc[b][d];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][b * ND + d] = v;
    }
  }
  __syncthreads();
  const int e = threadIdx.x, b = e / ND, d = e % ND;
  if (e < kDetBins * ND && m0 + b < L)
    atomicAdd(&D[(int64_t)d * L + m0 + b], (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]));
}

template <int ND>
static void launch_det_nd(const double* S, const double* masks, int32_t L, int32_t n_k,
                          double kappa, const double* q, double* D, hipStream_t st) {
  // 16384 pixels per block, fewer while the grid is below 8 blocks per CU and no more than
  // 32 blocks then add to one value (256^2 pixels, 123 bins, 4 masks: 47 us with 16384 pixels per
  // block, 29 us with 2048, 181 us with 512 and one atomic per wave, which queue up). Grids
  // above 2^19 pixels keep 16384 and add more: 64 blocks at 1024^2
  const int64_t rows = (L + kDetBins - 1) / kDetBins;
  int chunk = 16384;
  while (chunk > 512 && (n_k + chunk - 1) / chunk * rows < 2048 && n_k <= 32 * (chunk / 2)) chunk /= 2;
  dim3 g((n_k + chunk - 1) / chunk, (unsigned)rows);
  hipLaunchKernelGGL((detector_kernel<ND>), g, dim3(256), 0, st, S, masks, L, n_k, chunk, kappa, q, D);
}

hipError_t launch_detector(const double* S, const double* masks, int32_t n_det, int32_t L,
                           int32_t n_k, double kappa, const double* q, double* D, hipStream_t st) {
  switch (n_det) {
    case 1: launch_det_nd<1>(S, masks, L, n_k, kappa, q, D, st); break;
    case 2: launch_det_nd<2>(S, masks, L, n_k, kappa, q, D, st); break;
    case 3: launch_det_nd<3>(S, masks, L, n_k, kappa, q, D, st); break;
    case 4: launch_det_nd<4>(S, masks, L, n_k, kappa, q, D, st); break;
    case 5: launch_det_nd<5>(S, masks, L, n_k, kappa, q, D, st); break;
    case 6: launch_det_nd<6>(S, masks, L, n_k, kappa, q, D, st); break;
    case 7: launch_det_nd<7>(S, masks, L, n_k, kappa, q, D, st); break;
    case 8: launch_det_nd<8>(S, masks, L, n_k, kappa, q, D, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// *cnt += number of non-finite values (NaN or +-Inf) in x[i] times the factor of row
// (i / inner) % n_om, i < n (x as it stands when kappa is 1 and q null)
__global__ void count_nonfinite_kernel(const double* __restrict__ x, int64_t n, double kappa,
                                       const double* q, int64_t inner, int32_t n_om,
                                       unsigned long long* cnt) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  unsigned long long c = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    c += isfinite(x[i] * row_factor(kappa, q, q ? (int)((i / inner) % n_om) : 0)) ? 0ull : 1ull;
  if (c) atomicAdd(cnt, c);
}

hipError_t launch_count_nonfinite(const double* x, int64_t n, double kappa, const double* q,
                                  int64_t inner, int32_t n_om, unsigned long long* cnt,
                                  hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(count_nonfinite_kernel, dim3(blocks_for(n, 256, 4096)), dim3(256), 0, st, x,
                     n, kappa, q, inner, n_om, cnt);
  return hipGetLastError();
}

}  // namespace tacaw
