// Range and Doppler transforms (Section 3.3; eqs. (4), (5), (10)-(11)).
//
// The beat signal is x = conj(H) (eq. (13) under stretch processing); the range
// transform X = FFT_m(x) is the paper's inverse transform of the frequency-domain
// echo, up to conjugation and the factor M. The Doppler transform Y = FFT_n(X) puts
// zero Doppler in row N/2; the RDM is |Y|^2. Unnormalised, no window.
//
// Both wait on memory, at 70 to 97% of the copy's rate: a workgroup transforms a block of rows
// (range) or a tile of columns (Doppler, coalesced along the range axis), reading each point once
// and writing it once.
// The radix-4/2/3 Stockham stages (the same stages, in the same order and with the same
// operations as fft_common.h's) are taken two at a time in a thread's registers, up to 16
// points: the first pass takes its points straight from global memory, the last writes them
// back there, and only what lies between goes through LDS (512 points: two exchanges, 256:
// one, where every stage went through LDS with a barrier and two integer divisions a point).
// 192 x 256 x 512 points: range 214 -> 114 us (402 MB), Doppler with Y 240 -> 104 us (503 MB),
// the copy rate of this memory being about 5 TB/s.
// Twiddles come from an FP64-accurate table, tw[i] = exp(-j 2 pi i / L), i < L.
#include <algorithm>

#include "fft_common.h"

namespace rsim {

namespace {

constexpr int kFftMaxPasses = 8;

// The passes of a transform of length L = 2^a 3^b: its Stockham stages (radix 4 while two
// factors of 2 remain, 2 for an odd one, then 3) in pairs, ra[p] then rb[p] (1: a lone stage).
struct FftPlan {
  int L, passes;
  int ra[kFftMaxPasses], rb[kFftMaxPasses];
};
FftPlan make_plan(int L) {
  FftPlan p{};
  p.L = L;
  int stage[16], n = 0;
  for (int r : {4, 2, 3})
    for (; L % r == 0 && L > 1; L /= r) stage[n++] = r;
  for (int i = 0; i < n; i += 2) {
    p.ra[p.passes] = stage[i];
    p.rb[p.passes] = i + 1 < n ? stage[i + 1] : 1;
    ++p.passes;
  }
  return p;
}

__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }

// v <- its R-point DFT, v[q] = sum_i v[i] exp(-j 2 pi i q / R), after the twiddles w[i - 1]
template <int N, typename C>
__device__ __forceinline__ void stage_dft(C (&v)[N], const C *w) {
  using R = decltype(C{}.x);
  C x[N];
  x[0] = v[0];
#pragma unroll
  for (int i = 1; i < N; ++i)
    x[i] = {fma_(w[i - 1].x, v[i].x, -(w[i - 1].y * v[i].y)),
            fma_(w[i - 1].x, v[i].y, w[i - 1].y * v[i].x)};
  if constexpr (N == 4) {
    // X0,2 = (x0 + x2) +/- (x1 + x3), X1,3 = (x0 - x2) -/+ j (x1 - x3)
    const C s02 = {x[0].x + x[2].x, x[0].y + x[2].y}, d02 = {x[0].x - x[2].x, x[0].y - x[2].y};
    const C s13 = {x[1].x + x[3].x, x[1].y + x[3].y}, d13 = {x[1].x - x[3].x, x[1].y - x[3].y};
    v[0] = {s02.x + s13.x, s02.y + s13.y};
    v[1] = {d02.x + d13.y, d02.y - d13.x};
    v[2] = {s02.x - s13.x, s02.y - s13.y};
    v[3] = {d02.x - d13.y, d02.y + d13.x};
  } else if constexpr (N == 2) {
    v[0] = {x[0].x + x[1].x, x[0].y + x[1].y};
    v[1] = {x[0].x - x[1].x, x[0].y - x[1].y};
  } else {
    // X0 = x0 + x1 + x2; X1,2 = x0 - (x1 + x2)/2 -/+ j (sqrt(3)/2)(x1 - x2)
    const R h = R(0.86602540378443864676);
    const C t1 = {x[1].x + x[2].x, x[1].y + x[2].y};
    const C t2 = {fma_(R(-0.5), t1.x, x[0].x), fma_(R(-0.5), t1.y, x[0].y)};
    const C d = {x[1].x - x[2].x, x[1].y - x[2].y};
    v[0] = {x[0].x + t1.x, x[0].y + t1.y};
    v[1] = {fma_(h, d.y, t2.x), fma_(-h, d.x, t2.y)};
    v[2] = {fma_(-h, d.y, t2.x), fma_(h, d.x, t2.y)};
  }
}

// floor(i / d) for 0 <= i < 2^16 and inv = 1 / d: (i + 1/2) / d lies at least 1 / (2 d) from
// a whole number, more than the product's rounding (2^-23 i / d) while i < 2^22.
__device__ __forceinline__ int div_small(int i, float inv) {
  return static_cast<int>((static_cast<float>(i) + 0.5f) * inv);
}

// One pass over `count` sequences of length L after sub-transforms of length ns: a stage of
// radix RA, then one of radix RB (1: none) on sub-transforms of length ns RA. A thread takes
// x_i = load(s, j + i L / R), i < R = RA RB, j < L / R. With k = j mod ns the first stage's
// butterflies r < RB over the points i = r, RB + r, ... carry the twiddles exp(-j 2 pi i k /
// (ns RA)), the second's over their q-th outputs exp(-j 2 pi r (k + q ns) / (ns R)); output q2
// of that goes to store(s, (j - k) R + k + (q + RA q2) ns). The sequences run fastest
// (SEQ_FAST: the Doppler transform's columns lie side by side) or the butterflies.
template <int RA, int RB, bool SEQ_FAST, typename C, typename Load, typename Store>
__device__ __forceinline__ void fft_pass(int L, int ns, int count, const C *tw, Load &&load,
                                         Store &&store) {
  constexpr int R = RA * RB;
  const int span = L / R, step_a = L / (ns * RA), step_b = span / ns;
  const float inv = 1.0f / static_cast<float>(SEQ_FAST ? count : span);
  const float inv_ns = 1.0f / static_cast<float>(ns);
  for (int idx = threadIdx.x; idx < count * span; idx += blockDim.x) {
    const int hi = div_small(idx, inv);
    const int s = SEQ_FAST ? idx - hi * count : hi;
    const int j = SEQ_FAST ? hi : idx - hi * span;
    const int k = j - div_small(j, inv_ns) * ns;
    C y[RB][RA], w[RA > RB ? RA : RB];
#pragma unroll
    for (int i = 0; i < R; ++i) y[i % RB][i / RB] = load(s, j + i * span);
#pragma unroll
    for (int i = 1; i < RA; ++i) w[i - 1] = tw[i * k * step_a];
#pragma unroll
    for (int r = 0; r < RB; ++r) stage_dft<RA>(y[r], w);
    const int o = (j - k) * R + k;
#pragma unroll
    for (int q = 0; q < RA; ++q) {
      if constexpr (RB == 1) {
        store(s, o + q * ns, y[0][q]);
      } else {
        C v[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) v[r] = y[r][q];
#pragma unroll
        for (int r = 1; r < RB; ++r) w[r - 1] = tw[r * (k + q * ns) * step_b];
        stage_dft<RB>(v, w);
#pragma unroll
        for (int q2 = 0; q2 < RB; ++q2) store(s, o + (q + RA * q2) * ns, v[q2]);
      }
    }
  }
}

template <bool SEQ_FAST, typename C, typename Load, typename Store>
__device__ __forceinline__ void fft_pass_any(int ra, int rb, int L, int ns, int count, const C *tw,
                                             Load &&load, Store &&store) {
  switch (ra * 4 + rb) {
    case 4 * 4 + 4: fft_pass<4, 4, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 4 * 4 + 2: fft_pass<4, 2, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 4 * 4 + 3: fft_pass<4, 3, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 4 * 4 + 1: fft_pass<4, 1, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 2 * 4 + 3: fft_pass<2, 3, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 2 * 4 + 1: fft_pass<2, 1, SEQ_FAST>(L, ns, count, tw, load, store); break;
    case 3 * 4 + 3: fft_pass<3, 3, SEQ_FAST>(L, ns, count, tw, load, store); break;
    default: fft_pass<3, 1, SEQ_FAST>(L, ns, count, tw, load, store); break;
  }
}

// The transform of `count` sequences: in(s, i) reads point i of sequence s, out(s, i, v)
// takes point i of its transform; a and b (LDS, at(s, i) the place of a point) carry what
// lies between the passes (b only with more than two).
template <bool SEQ_FAST, typename C, typename In, typename Out, typename At>
__device__ __forceinline__ void fft_run(const FftPlan &plan, int count, const C *tw, C *a, C *b,
                                        In &&in, Out &&out, At &&at) {
  const int L = plan.L, last = plan.passes - 1;
  const auto run = [&](int p, int ns, auto &&load, auto &&store) __attribute__((always_inline)) {
    fft_pass_any<SEQ_FAST>(plan.ra[p], plan.rb[p], L, ns, count, tw, load, store);
  };
  if (last == 0) {
    run(0, 1, in, out);
    return;
  }
  run(0, 1, in, [&](int s, int i, C v) { a[at(s, i)] = v; });
  __syncthreads();
  int ns = plan.ra[0] * plan.rb[0];
  for (int p = 1; p < last; ++p) {
    run(p, ns, [&](int s, int i) { return a[at(s, i)]; },
        [&](int s, int i, C v) { b[at(s, i)] = v; });
    __syncthreads();
    C *t = a;
    a = b;
    b = t;
    ns *= plan.ra[p] * plan.rb[p];
  }
  run(last, ns, [&](int s, int i) { return a[at(s, i)]; }, out);
}

}  // namespace

// Rows of length M: out[row] = FFT(conj_in ? conj(in[row]) : in[row]).
template <typename R>
__global__ void __launch_bounds__(256) range_fft_kernel(const typename Cx2<R>::T *in,
                                                        typename Cx2<R>::T *out, int64_t rows,
                                                        FftPlan plan, int rows_per_wg, int ld,
                                                        int conj_in,
                                                        const typename Cx2<R>::T *tw) {
  using C = typename Cx2<R>::T;
  extern __shared__ __align__(16) unsigned char fft_smem[];
  C *a = reinterpret_cast<C *>(fft_smem);
  C *b = a + rows_per_wg * ld;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * rows_per_wg;
  const int nrow = static_cast<int>(min<int64_t>(rows_per_wg, rows - row0));
  const int M = plan.L;
  const C *src = in + row0 * M;
  C *dst = out + row0 * M;
  fft_run<false>(
      plan, nrow, tw, a, b,
      [&](int s, int i) {
        C v = src[s * M + i];
        if (conj_in) v.y = -v.y;
        return v;
      },
      [&](int s, int i, C v) { dst[s * M + i] = v; },
      // a gap after every eighth point: the first pass writes with the stride of its radix
      [&](int s, int i) { return s * ld + i + (i >> 3); });
}

// Columns of length N (stride M) of each channel's [N][M] plane.
// mode 0 (forward): Y = shift_n(FFT_n(X)), row l holding Doppler index l - floor(N/2) for
//   even and odd N alike; writes rdm = |Y|^2 and y_out if given.
// mode 1 (adjoint input side): Z = FFT_n(conj(unshift_n(G))) written to y_out.
// mode 2 (RDM backward): as mode 1 with G = 2 (dL/dP) Y formed on the fly from
//   gp = dL/dP (rdm-shaped) and in = Y, since P = |Y|^2.
template <typename R>
__global__ void __launch_bounds__(512) doppler_fft_kernel(const typename Cx2<R>::T *in,
                                                          typename Cx2<R>::T *y_out, R *rdm,
                                                          int64_t planes, FftPlan plan, int M,
                                                          int kt, int mode,
                                                          const typename Cx2<R>::T *tw,
                                                          const R *gp) {
  using C = typename Cx2<R>::T;
  extern __shared__ __align__(16) unsigned char fft_smem[];
  const int N = plan.L;
  C *a = reinterpret_cast<C *>(fft_smem);
  C *b = a + kt * N;
  const int tiles = (M + kt - 1) / kt;
  const int64_t plane = blockIdx.x / tiles;
  const int k0 = static_cast<int>(blockIdx.x - plane * tiles) * kt;
  const int ncol = min(kt, M - k0);
  const int64_t base = plane * static_cast<int64_t>(N) * M + k0;
  const int hN = N >> 1;
  const auto at = [&](int c, int i) { return i * kt + c; };
  if (mode == 0) {
    fft_run<true>(
        plan, ncol, tw, a, b, [&](int c, int i) { return in[base + static_cast<int64_t>(i) * M + c]; },
        [&](int c, int i, C v) {
          const int l = i + hN < N ? i + hN : i + hN - N;  // row l <- index l - floor(N/2)
          const int64_t g = base + static_cast<int64_t>(l) * M + c;
          if (rdm) rdm[g] = v.x * v.x + v.y * v.y;
          if (y_out) y_out[g] = v;
        },
        at);
  } else {
    fft_run<true>(
        plan, ncol, tw, a, b,
        [&](int c, int i) {
          // row l of G holds Doppler index l - floor(N/2), conjugated
          const int l = i + hN < N ? i + hN : i + hN - N;
          const int64_t g = base + static_cast<int64_t>(l) * M + c;
          C v = in[g];
          if (mode == 2) {
            const R s = R(2) * gp[g];
            v.x *= s;
            v.y *= s;
          }
          v.y = -v.y;
          return v;
        },
        [&](int c, int i, C v) { y_out[base + static_cast<int64_t>(i) * M + c] = v; }, at);
  }
}

namespace {

// LDS of a transform of `points` points a workgroup: none for one pass, one buffer for two,
// two beyond.
size_t fft_lds(const FftPlan &plan, size_t points, size_t csize) {
  return csize * points * (plan.passes <= 1 ? 0 : plan.passes == 2 ? 1 : 2);
}

// Rows a range workgroup takes, and the LDS stride of a row (a gap after every eighth point).
int range_rows(int M, size_t csize) {
  const int budget = csize == 8 ? 2048 : 1024;  // points per workgroup
  return std::max(1, budget / M);
}
int range_ld(int M) { return M + M / 8 + 1; }

// Columns a Doppler workgroup takes: whole 128-byte lines of a row (256 bytes at best) within
// 64 KB of LDS.
int doppler_cols(const FftPlan &plan, int M, size_t csize) {
  int kt = 256 / static_cast<int>(csize);
  while (kt > 1 &&
         (fft_lds(plan, static_cast<size_t>(kt) * plan.L, csize) > (64u << 10) || kt / 2 >= M))
    kt /= 2;
  return kt;
}

template <typename R>
hipError_t launch_range_t(const void *in, void *out, int64_t rows, int M, int conj_in,
                          const void *tw, hipStream_t s) {
  using C = typename Cx2<R>::T;
  const FftPlan plan = make_plan(M);
  const int rpw = range_rows(M, sizeof(C)), ld = range_ld(M);
  const unsigned grid = static_cast<unsigned>((rows + rpw - 1) / rpw);
  hipLaunchKernelGGL(range_fft_kernel<R>, dim3(grid), dim3(256),
                     fft_lds(plan, static_cast<size_t>(rpw) * ld, sizeof(C)), s,
                     static_cast<const C *>(in), static_cast<C *>(out), rows, plan, rpw, ld, conj_in,
                     static_cast<const C *>(tw));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_doppler_t(const void *in, void *y_out, void *rdm, int64_t planes, int N, int M,
                            int mode, const void *tw, hipStream_t s, const void *gp) {
  using C = typename Cx2<R>::T;
  const FftPlan plan = make_plan(N);
  const int kt = doppler_cols(plan, M, sizeof(C));
  const int tiles = (M + kt - 1) / kt;
  const unsigned grid = static_cast<unsigned>(planes * tiles);
  const int threads = std::min(512, std::max(64, (kt * (N / (plan.ra[0] * plan.rb[0])) + 63) / 64 * 64));
  hipLaunchKernelGGL(doppler_fft_kernel<R>, dim3(grid), dim3(threads),
                     fft_lds(plan, static_cast<size_t>(kt) * N, sizeof(C)), s,
                     static_cast<const C *>(in), static_cast<C *>(y_out), static_cast<R *>(rdm),
                     planes, plan, M, kt, mode, static_cast<const C *>(tw),
                     static_cast<const R *>(gp));
  return hipGetLastError();
}

}  // namespace

size_t fft_smem_bytes(int precision, int N, int M) {
  const size_t csize = precision ? 16 : 8;
  const FftPlan range = make_plan(M), doppler = make_plan(N);
  return std::max(fft_lds(range, static_cast<size_t>(range_rows(M, csize)) * range_ld(M), csize),
                  fft_lds(doppler, static_cast<size_t>(doppler_cols(doppler, M, csize)) * N, csize));
}

hipError_t launch_range_fft(int precision, const void *in, void *out, int64_t rows, int M,
                            int conj_in, const void *tw, hipStream_t s) {
  return precision ? launch_range_t<double>(in, out, rows, M, conj_in, tw, s)
                   : launch_range_t<float>(in, out, rows, M, conj_in, tw, s);
}

hipError_t launch_doppler_fft(int precision, const void *in, void *y_out, void *rdm,
                              int64_t planes, int N, int M, int mode, const void *tw,
                              hipStream_t s, const void *gp) {
  return precision ? launch_doppler_t<double>(in, y_out, rdm, planes, N, M, mode, tw, s, gp)
                   : launch_doppler_t<float>(in, y_out, rdm, planes, N, M, mode, tw, s, gp);
}

}  // namespace rsim
