// NUFFT facet sum, the spread: each run of cell-sorted records (one lit facet, point or
// double-bounce connection of one chirp each) adds its Gaussian grid sources, for every
// channel, into a register window of kNuSlots grid cells, written out once per run (see
// nufft.hip for the transform it belongs to and the kernels around it).
#include <hip/hip_runtime.h>

#include <cstddef>
#include <type_traits>

#include "nufft_common.h"
#include "rsim_internal.h"
#include "rsim_launch.h"

namespace rsim {

namespace {

// Gaussian (from cell S0 on: g_{s+1} = g_s rho_s, rho_{s+1} = rho_s exp(-1/s^2)) times the
// weight cw at the NCELL cells S0 .. S0 + NCELL - 1 of the window (cells past the window's
// end are dropped at compile time; the runs keep every source inside).
template <int S0, int NCELL>
__device__ __forceinline__ void point_cells(float2 (&acc)[kNuSlots], float2 cw, float gw,
                                            float rho, float q_ratio) {
  // the weights are formed here, in the block: hoisted ahead of the chain of blocks (they
  // are the same in every block) they would hold NCELL registers more across it
  asm volatile("" : "+v"(gw), "+v"(rho));
#pragma unroll
  for (int j = 0; j < NCELL; ++j) {
    if (S0 + j < kNuSlots) {
      acc[S0 + j].x = fmaf(gw, cw.x, acc[S0 + j].x);
      acc[S0 + j].y = fmaf(gw, cw.y, acc[S0 + j].y);
      gw *= rho;
      rho *= q_ratio;
    }
  }
}

// Gaussian times the polynomial sum_k c_k (s - pos)^k at the cells S0 .. S0 + NCELL - 1.
template <int S0, int NCELL, int NC>
__device__ __forceinline__ void poly_cells(float2 (&acc)[kNuSlots], const float2 (&c)[NC],
                                           float u0, float gw, float rho, float q_ratio) {
  asm volatile("" : "+v"(u0), "+v"(gw), "+v"(rho));  // formed in the block, as above
#pragma unroll
  for (int j = 0; j < NCELL; ++j) {
    if (S0 + j < kNuSlots) {
      const float xx = u0 + static_cast<float>(j);
      float pr = c[NC - 1].x, pi = c[NC - 1].y;
#pragma unroll
      for (int k = NC - 2; k >= 0; --k) {
        pr = fmaf(pr, xx, c[k].x);
        pi = fmaf(pi, xx, c[k].y);
      }
      acc[S0 + j].x = fmaf(gw, pr, acc[S0 + j].x);
      acc[S0 + j].y = fmaf(gw, pi, acc[S0 + j].y);
      gw *= rho;
      rho *= q_ratio;
    }
  }
}

// Gaussian times c0 + c2 (s - pos)^2 (no linear term: a point source under the delay
// within the chirp) at the cells S0 .. S0 + NCELL - 1.
template <int S0, int NCELL>
__device__ __forceinline__ void even2_cells(float2 (&acc)[kNuSlots], float2 c0, float2 c2,
                                            float u0, float gw, float rho, float q_ratio) {
  asm volatile("" : "+v"(u0), "+v"(gw), "+v"(rho));  // formed in the block, as above
#pragma unroll
  for (int j = 0; j < NCELL; ++j) {
    if (S0 + j < kNuSlots) {
      const float xx = u0 + static_cast<float>(j);
      const float x2 = xx * xx;
      const float pr = fmaf(c2.x, x2, c0.x), pi = fmaf(c2.y, x2, c0.y);
      acc[S0 + j].x = fmaf(gw, pr, acc[S0 + j].x);
      acc[S0 + j].y = fmaf(gw, pi, acc[S0 + j].y);
      gw *= rho;
      rho *= q_ratio;
    }
  }
}

// The window cell s_lo (wave-uniform) selects one straight-line block of NCELL cells. A
// source covers NCELL or fewer cells (its count is floor(2 reach) or one more, NCELL at
// least the larger), so a block may reach up to four cells past the last the runs
// guarantee inside the window; those are dropped (their Gaussian weights are below
// psi(W/2) for every channel). The blocks sit behind independent scalar bit tests rather
// than a switch: every block then updates the window registers in place, where the merge
// of a switch's cases costs register copies of the untouched cells. The tests come in four
// levels (halves, quarters, eighths, blocks): a test that fails is a taken branch, and 23 of
// them a source left the waves waiting for their instructions.
constexpr int kNuTopStart = 22;  // the last block start
template <int NCELL, int S0, typename F>
__device__ __forceinline__ void try_block(uint32_t bit, F &&f) {
  if constexpr (S0 <= kNuTopStart) {
    if (bit & (1u << S0)) f(std::integral_constant<int, S0>{});
  }
}
template <int NCELL, typename F>
__device__ __forceinline__ void select_block(int s_lo, F &&f) {
  const uint32_t bit = 1u << s_lo;
#define RSIM_NU_3(S)                             \
  if (bit & (7u << (S))) {                       \
    try_block<NCELL, (S)>(bit, f);               \
    try_block<NCELL, (S) + 1>(bit, f);           \
    try_block<NCELL, (S) + 2>(bit, f);           \
  }
#define RSIM_NU_6(S)                             \
  if (bit & (0x3Fu << (S))) {                    \
    RSIM_NU_3(S) RSIM_NU_3((S) + 3)              \
  }
#define RSIM_NU_12(S)                            \
  if (bit & (0xFFFu << (S))) {                   \
    RSIM_NU_6(S) RSIM_NU_6((S) + 6)              \
  }
  RSIM_NU_12(0) RSIM_NU_12(12)
#undef RSIM_NU_3
#undef RSIM_NU_6
#undef RSIM_NU_12
  static_assert(kNuTopStart < 24, "every start has a block");
}

// First Gaussian weight of a block and its first step, for a lane's source at pos.
__device__ __forceinline__ void first_cell(int s_lo, float pos, float nc, float &u0, float &gw,
                                           float &rho) {
  u0 = static_cast<float>(s_lo) - pos;
  gw = __builtin_amdgcn_exp2f(nc * u0 * u0);
  rho = __builtin_amdgcn_exp2f(nc * fmaf(2.0f, u0, 1.0f));
}

template <int NCELL>
__device__ __forceinline__ void spread_point(float2 (&acc)[kNuSlots], float2 cw, float pos,
                                             int s_lo, float nc, float q_ratio) {
  float u0, gw, rho;
  first_cell(s_lo, pos, nc, u0, gw, rho);
  select_block<NCELL>(s_lo, [&](auto s0) __attribute__((always_inline)) {
    point_cells<s0(), NCELL>(acc, cw, gw, rho, q_ratio);
  });
}

template <int NCELL>
__device__ __forceinline__ void spread_even2(float2 (&acc)[kNuSlots], float2 c0, float2 c2,
                                             float pos, int s_lo, float nc, float q_ratio) {
  float u0, gw, rho;
  first_cell(s_lo, pos, nc, u0, gw, rho);
  select_block<NCELL>(s_lo, [&](auto s0) __attribute__((always_inline)) {
    even2_cells<s0(), NCELL>(acc, c0, c2, u0, gw, rho, q_ratio);
  });
}

template <int NCELL, int NC>
__device__ __forceinline__ void spread_poly(float2 (&acc)[kNuSlots], const float2 (&c)[NC],
                                            float pos, int s_lo, float nc, float q_ratio) {
  float u0, gw, rho;
  first_cell(s_lo, pos, nc, u0, gw, rho);
  select_block<NCELL>(s_lo, [&](auto s0) __attribute__((always_inline)) {
    poly_cells<s0(), NCELL, NC>(acc, c, u0, gw, rho, q_ratio);
  });
}

// (1 - j 2 pi B m'^2) on the modes is F + j eps F'' on the grid (F = psi P): coefficient
// k of the result is c_k + j eps (c_{k-2} / s^4 - (2k + 1) c_k / s^2 + (k+1)(k+2) c_{k+2}).
template <int NI, int NO>
__device__ __forceinline__ void intra_coeffs(const float2 (&c)[NI], float2 (&o)[NO], float eps,
                                             float inv_s2) {
  const float inv_s4 = inv_s2 * inv_s2;
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const float2 ck = k < NI ? c[k] : make_float2(0.0f, 0.0f);
    const float2 cm2 = (k >= 2 && k - 2 < NI) ? c[k - 2] : make_float2(0.0f, 0.0f);
    const float2 cp2 = (k + 2 < NI) ? c[k + 2] : make_float2(0.0f, 0.0f);
    const float wk = -(2.0f * k + 1.0f) * inv_s2;
    const float wp = static_cast<float>((k + 1) * (k + 2));
    const float dx = cm2.x * inv_s4 + wk * ck.x + wp * cp2.x;
    const float dy = cm2.y * inv_s4 + wk * ck.y + wp * cp2.y;
    o[k] = {ck.x - eps * dy, ck.y + eps * dx};
  }
}

// The part of a record that its channels and cells need, read through scalar loads.
struct NuHead {
  double g1;
  float rt, rr, t0, frac;
  int32_t cell, kind;
  float s[10];
};
static_assert(offsetof(NuRecF<false>, s) - offsetof(NuRecF<false>, g1) == offsetof(NuHead, s) &&
                  offsetof(NuRecF<false>, rt) - offsetof(NuRecF<false>, g1) ==
                      offsetof(NuHead, rt) &&
                  offsetof(NuRecF<false>, kind) - offsetof(NuRecF<false>, g1) ==
                      offsetof(NuHead, kind) &&
                  offsetof(NuRecF<true>, g1) == offsetof(NuRecF<false>, g1),
              "the head's fields are consecutive");

// What a record's channels owe to one element e of their two: u.a, the remainder of the
// path difference and the path difference itself (see the header of nufft.hip).
struct ElemTerm {
  double s;
  float e, dR;
};
// a: its offset from the phase centre, of squared length a2; u: the unit vector to that centre,
// `dist` away
__device__ __forceinline__ ElemTerm element_term(const double *u, float dist, const double (&a)[3],
                                                 float a2) {
  const double s = u[0] * a[0] + u[1] * a[1] + u[2] * a[2];
  const float sf = static_cast<float>(s);
  const float h = fmaf(-sf, sf, a2);
  const float rd = __builtin_amdgcn_rcpf(fmaf(-2.0f, sf, 2.0f * dist));
  const float qd = h * rd;
  const float ed = qd * fmaf(-qd, rd, 1.0f);
  return {s, ed, ed - sf};
}
// With the delay within the chirp: the rate of the element's distance, v the source's velocity
// and `rate` that of the centre's distance.
__device__ __forceinline__ float element_rate(const float *v, float rate, float dist, float dR,
                                              const double (&a)[3]) {
  const float af[3] = {static_cast<float>(a[0]), static_cast<float>(a[1]),
                       static_cast<float>(a[2])};
  const float va = v[0] * af[0] + v[1] * af[1] + v[2] * af[2];
  return fmaf(dist, rate, -va) * __builtin_amdgcn_rcpf(dist + dR);
}

}  // namespace

// One workgroup per (chirp, run) and up to four 64-channel groups (blockIdx.z counts
// further groups); lane = channel. A run's records are taken batch by batch:
//  - staging (STAGED): a lane per (record, element) forms what the record's channels owe to that Tx
//    or Rx element, into LDS: P + Q elements for P Q channels (28 for 192 on the 12 x 16
//    array), where every lane forming its own channel's took a fifth of the kernel's
//    instructions; then a lane per record the first cells of the record's blocks. Arrays with
//    few channels to an element go without (launch_nufft_spread has the rule): a lane forms its
//    own two terms from the record in scalar registers;
//  - spread: per record a lane joins its two elements' terms and adds the record's sources
//    into its register window of kNuSlots cells, which starts at the run's base cell and
//    goes to part[chirp][run][channel][kNuSlots] at the run's end.
// Bound by the waves' latencies (LDS and scalar loads, transcendentals, the blocks' branches)
// at the five waves per SIMD that 96 registers leave, the window taking 64 of them; four
// waves: 95.5 against 88.3 ms. On the 1M-triangle intersection (82M records, 192 channels) the
// element terms and block tests in levels took it from 102.8 to 88.3 ms, the head's load after the
// record's LDS reads to 81.7: 244 VALU instructions a record and wave, of which 162 are the
// cells', at 3.4 cycles each where 2.4 is the least measured (more for exponentials and FP64).
template <bool INTRA, int NCELL, bool STAGED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(INTRA ? 4 : 5, 8)))
nufft_spread_kernel(
    DevScene sc0, RadarConst rc, NuShape ns, const double *elem,
    const NuRecF<INTRA> *__restrict__ sorted, const int4 *__restrict__ runs,
    const int32_t *__restrict__ n_runs, float2 *__restrict__ part, NuBatch bt) {
  extern __shared__ __align__(16) unsigned char spread_smem[];
  const int nl = blockIdx.y;
  const int run = blockIdx.x;
  if (run >= load_uniform(n_runs + nl)) return;  // whole workgroup
  const NuWork w = nu_work(sc0, ns, bt, nl);
  const int E = rc.P + rc.Q, batch = ns.spread_batch;
  ElemTerm *term = reinterpret_cast<ElemTerm *>(spread_smem);             // [batch][E]
  double *off = reinterpret_cast<double *>(term + batch * E);              // [E][3]
  float *rdot = reinterpret_cast<float *>(off + 3 * E);                    // [batch][E] (INTRA)
  int32_t *all_starts = reinterpret_cast<int32_t *>(rdot + (INTRA ? batch * E : 0));
  if constexpr (STAGED) {
    for (int i = threadIdx.x; i < 3 * E; i += blockDim.x) {
      const int k = i % 3;
      off[i] = elem[i] - (i < 3 * rc.P ? rc.tx_c[k] : rc.rx_c[k]);
    }
  }
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int grp = static_cast<int>(blockIdx.z) * 4 + wave;
  const int lane = threadIdx.x & 63;
  const int O = rc.P * rc.Q;
  const bool wave_on = grp * 64 < O;
  const int4 rr = load_uniform(runs + w.run + run);
  const int o = grp * 64 + lane;
  const bool on = o < O;
  const int oc = on ? o : wave_on ? grp * 64 : 0;  // idle lanes: the wave's first channel
  const int p = oc / rc.Q, q = rc.P + oc % rc.Q;
  const int p_first = grp * 64 / rc.Q, q_first = rc.P + grp * 64 % rc.Q;
  int32_t *starts_of = all_starts + wave * batch;  // [waves][batch]
  const float inv_c0 = static_cast<float>(1.0 / kC0), inv_fs = static_cast<float>(1.0 / rc.fs);
  const float df_fs = static_cast<float>(rc.df / rc.fs);
  const float half_m = 0.5f * rc.M, quarter_m2 = 0.25f * rc.M * rc.M, m_f = static_cast<float>(rc.M);
  const float ngf = static_cast<float>(ns.ng);
  const float eps_scale = static_cast<float>(static_cast<double>(ns.ng) * ns.ng / (2.0 * kPi));
  const float inv_s2 = static_cast<float>(1.0 / (ns.sigma * ns.sigma));
  const NuRecF<INTRA> *srec = sorted + w.rec;
  const float nc = static_cast<float>(-1.4426950408889634 / (2.0 * ns.sigma * ns.sigma));
  const float q_ratio = __builtin_amdgcn_exp2f(2.0f * nc);  // exp(-1 / s^2)
  const float kappa = static_cast<float>(ns.kappa);
  const float g2 = static_cast<float>(0.5 * rc.slope / (kC0 * kC0));
  const float reach = static_cast<float>(ns.wave_d) + 0.5f * kNuWidth;
  // the delay within the chirp moves a channel's source by (A + B M) n_g cells, of which the
  // record's frac holds ext[5]
  const auto doppler_shift = [&](float tdot, double g1, float ext5, float &A, float &B)
                                 __attribute__((always_inline)) {
    const float fmt = static_cast<float>(g1 * kC0 - (rc.M / 2) * rc.df);
    A = fmt * tdot * inv_fs;
    B = df_fs * tdot;
    return fmaf(B, m_f, A) * ngf - ext5;
  };
  float2 acc[kNuSlots];
#pragma unroll
  for (int s = 0; s < kNuSlots; ++s) acc[s] = {0.0f, 0.0f};
  // not staged: this lane's two elements
  double at[3] = {}, ar[3] = {};
  float at2 = 0.0f, ar2 = 0.0f;
  if constexpr (!STAGED) {
    if (!wave_on) return;
    double t2 = 0.0, r2 = 0.0;
    for (int k = 0; k < 3; ++k) {
      at[k] = elem[3 * p + k] - rc.tx_c[k];
      ar[k] = elem[3 * q + k] - rc.rx_c[k];
      t2 += at[k] * at[k];
      r2 += ar[k] * ar[k];
    }
    at2 = static_cast<float>(t2);
    ar2 = static_cast<float>(r2);
  }
  for (int b0 = rr.x; b0 < rr.y; b0 += batch) {
    const int nb = min(batch, rr.y - b0);
    if constexpr (STAGED) {
      __syncthreads();  // the offsets are in; the last batch's readers are done
      for (int i = threadIdx.x; i < nb * E; i += blockDim.x) {
        const int rec = i / E, e = i - rec * E;
        const NuRecF<INTRA> *r = srec + b0 + rec;
        const bool tx = e < rc.P;
        const double *u = tx ? r->ut : r->ur;
        const double a[3] = {off[3 * e], off[3 * e + 1], off[3 * e + 2]};
        double aa = 0.0;
        for (int k = 0; k < 3; ++k) aa += a[k] * a[k];
        const float dist = tx ? r->rt : r->rr;
        const ElemTerm T = element_term(u, dist, a, static_cast<float>(aa));
        term[i] = T;
        if constexpr (INTRA)
          rdot[i] = element_rate(r->ext, tx ? r->ext[3] : r->ext[4], dist, T.dR, a);
      }
      __syncthreads();
      if (!wave_on) continue;
      // a lane per record: the first cells of its blocks in this wave (sources at s[0], s[3],
      // s[6]): the lowest cell within `reach` of the source's position for the wave's first
      // channel, clamped to the blocks there are (the runs keep every channel's cells inside the
      // window, so a clamp never drops one of them). Every channel of the wave lies within
      // wave_d cells of the first.
      if (lane < nb) {
        const NuRecF<INTRA> *r = srec + b0 + lane;
        const float dL = term[lane * E + p_first].dR + term[lane * E + q_first].dR;
        float x0 = fmaf(kappa, dL, static_cast<float>(r->cell - rr.z) + r->frac);
        if constexpr (INTRA) {
          const float tdot = (rdot[lane * E + p_first] + rdot[lane * E + q_first]) * inv_c0;
          float A, B;
          x0 += doppler_shift(tdot, r->g1, r->ext[5], A, B);
        }
        int32_t starts = 0;
        for (int j = 0; j < 3; ++j) {
          const int lo = static_cast<int>(ceilf((x0 - r->s[3 * j]) - reach));
          starts |= min(max(lo, 0), kNuTopStart) << (8 * j);
        }
        starts_of[lane] = starts;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    using Head = std::conditional_t<STAGED, NuHead, NuRecF<INTRA>>;  // what a record is read of
    const auto *heads = reinterpret_cast<const unsigned char *>(srec + b0) +
                        (STAGED ? offsetof(NuRecF<INTRA>, g1) : 0);
    const auto head = [&](int i) {
      return load_uniform(reinterpret_cast<const Head *>(heads + i * sizeof(NuRecF<INTRA>)));
    };
    const ElemTerm *tp = term + p, *tq = term + q;
    Head nxt = head(0);
    for (int i = 0; i < nb; ++i) {
      const Head r = nxt;
      ElemTerm T, R;
      uint32_t starts;
      if constexpr (STAGED) {
        T = tp[i * E];
        R = tq[i * E];
        starts = __builtin_amdgcn_readfirstlane(starts_of[i]);
      } else {
        T = element_term(r.ut, r.rt, at, at2);
        R = element_term(r.ur, r.rr, ar, ar2);
      }
      // this channel's path difference dL = -(s_t + s_r) + e_t + e_r, amplitude, phase and
      // grid position
      const float rel_c = static_cast<float>(r.cell - rr.z) + r.frac;
      const double ps = (T.s + R.s) * r.g1;  // turns, up to ~25
      const float pr = static_cast<float>(ps - rint(ps));
      const float dL = T.dR + R.dR;
      float t = (r.t0 - pr) + fmaf(static_cast<float>(r.g1), T.e + R.e, -g2 * dL * dL);
      float xr = fmaf(kappa, dL, rel_c);
      float eps = 0.0f;  // B n_g^2 / (2 pi): weight of F'' for the B m'^2 term
      if constexpr (INTRA) {
        // this channel's tau' (first order in the sample time), its Doppler shift relative
        // to the record's and the constant phase A M/2 + B M^2/4
        float rate;
        if constexpr (STAGED)
          rate = rdot[i * E + p] + rdot[i * E + q];
        else
          rate = element_rate(r.ext, r.ext[3], r.rt, T.dR, at) +
                 element_rate(r.ext, r.ext[4], r.rr, R.dR, ar);
        const float tdot = rate * inv_c0;
        float A, B;
        const float shift = doppler_shift(
            tdot, r.g1, load_uniform(&srec[b0 + i].ext[5]), A, B);
        t += fmaf(A, half_m, B * quarter_m2);
        xr += shift;
        eps = B * eps_scale;
      }
      t -= rintf(t);
      const float amp = __builtin_amdgcn_rcpf((r.rt + T.dR) * (r.rr + R.dR));
      const float qx = __builtin_amdgcn_cosf(t) * amp, qy = -__builtin_amdgcn_sinf(t) * amp;
      if constexpr (!STAGED) {  // the blocks' first cells, a source a lane
        const float x0 = __builtin_bit_cast(
            float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, xr)));
        const float off_l = lane == 0 ? r.s[0] : lane == 1 ? r.s[3] : r.s[6];
        const int lo = min(max(static_cast<int>(ceilf((x0 - off_l) - reach)), 0), kNuTopStart);
        starts = __builtin_amdgcn_readlane(lo, 0) | __builtin_amdgcn_readlane(lo, 1) << 8 |
                 __builtin_amdgcn_readlane(lo, 2) << 16;
      }
      // The next head is asked for when this record's LDS reads are in: one counter holds both
      // kinds of load, so a wait for the LDS would wait for the head, too.
      __builtin_amdgcn_sched_barrier(0);
      nxt = head(i + 1 < nb ? i + 1 : i);
      __builtin_amdgcn_sched_barrier(0);
      // no source for a record of kind 0 (a branch around the work here costs register copies)
      const int n_pts = r.kind == 1 ? 3 : r.kind == 2 ? 1 : 0;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (j < n_pts) {
          const float off_j = r.s[3 * j];
          const float2 cw = {qx * r.s[3 * j + 1] - qy * r.s[3 * j + 2],
                             qx * r.s[3 * j + 2] + qy * r.s[3 * j + 1]};
          // cells some channel reaches: |s - (x_o - off)| <= W/2 with |x_o - x0| <= wave_d,
          // NCELL of them from s_lo
          const int s_lo = static_cast<int>((starts >> (8 * j)) & 31u);
          if constexpr (INTRA) {
            // (1 - j 2 pi B m'^2) on a point's modes: cw (1 - j eps / s^2) + j eps cw / s^4 x^2
            // (intra_coeffs of one coefficient; its linear term is zero)
            const float e2 = eps * inv_s2, e4 = e2 * inv_s2;
            const float2 c0 = {fmaf(e2, cw.y, cw.x), fmaf(-e2, cw.x, cw.y)};
            const float2 c2 = {-e4 * cw.y, e4 * cw.x};
            spread_even2<NCELL>(acc, c0, c2, xr - off_j, s_lo, nc, q_ratio);
          } else {
            spread_point<NCELL>(acc, cw, xr - off_j, s_lo, nc, q_ratio);
          }
        }
      }
      if (r.kind >= 2) {
        const float off_j = r.s[3];
        float2 cq[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
          cq[k] = {qx * r.s[4 + 2 * k] - qy * r.s[5 + 2 * k], qx * r.s[5 + 2 * k] + qy * r.s[4 + 2 * k]};
        const int s_lo = static_cast<int>((starts >> 8) & 31u);
        if constexpr (INTRA) {
          float2 c5[5];
          intra_coeffs(cq, c5, eps, inv_s2);
          spread_poly<NCELL>(acc, c5, xr - off_j, s_lo, nc, q_ratio);
        } else {
          spread_poly<NCELL>(acc, cq, xr - off_j, s_lo, nc, q_ratio);
        }
      }
    }
  }
  if (!on) return;
  float4 *dst = reinterpret_cast<float4 *>(
      part + ((w.run + run) * O + o) * kNuSlots);
#pragma unroll
  for (int s = 0; s < kNuSlots / 2; ++s)
    dst[s] = make_float4(acc[2 * s].x, acc[2 * s].y, acc[2 * s + 1].x, acc[2 * s + 1].y);
}

// Records staged together: 16 KB of element terms at most, 32 records where they fit.
int nufft_spread_batch(int elements) {
  int b = 32;
  while (b > 1 && b * elements * static_cast<int>(sizeof(ElemTerm)) > (16 << 10)) b /= 2;
  return b;
}

size_t nufft_spread_smem_bytes(int elements, int batch, int waves, bool intra) {
  return batch * (elements * (sizeof(ElemTerm) + (intra ? sizeof(float) : 0)) +
                  waves * sizeof(int32_t)) +
         elements * 3 * sizeof(double);
}

namespace {

template <bool INTRA, bool STAGED>
hipError_t launch_spread_t(const DevScene &sc, const RadarConst &rc, const NuShape &ns,
                           const double *elem, const NuRecF<INTRA> *recs, const int4 *runs,
                           const int32_t *n_runs, float2 *part, const NuBatch &bt, dim3 grid,
                           dim3 blk, int ncell, hipStream_t s) {
  const size_t lds =
      STAGED ? nufft_spread_smem_bytes(rc.P + rc.Q, ns.spread_batch, blk.x / 64, INTRA) : 0;
  switch (ncell) {
    case 14:
      hipLaunchKernelGGL((nufft_spread_kernel<INTRA, 14, STAGED>), grid, blk, lds, s, sc, rc, ns, elem,
                         recs, runs, n_runs, part, bt);
      break;
    case 16:
      hipLaunchKernelGGL((nufft_spread_kernel<INTRA, 16, STAGED>), grid, blk, lds, s, sc, rc, ns, elem,
                         recs, runs, n_runs, part, bt);
      break;
    case 20:
      hipLaunchKernelGGL((nufft_spread_kernel<INTRA, 20, STAGED>), grid, blk, lds, s, sc, rc, ns, elem,
                         recs, runs, n_runs, part, bt);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_nufft_spread(const DevScene &sc, const RadarConst &rc, const NuShape &ns0,
                               const double *elem, const void *srec, const int4 *runs,
                               const int32_t *n_runs, float2 *part, const NuBatch &bt,
                               hipStream_t s) {
  const int O = rc.P * rc.Q;
  const int groups = (O + 63) / 64;
  const int per_block = groups < 4 ? groups : 4;
  NuShape ns = ns0;
  dim3 sgrid(static_cast<unsigned>(ns.max_runs), static_cast<unsigned>(ns.n_chirps),
             static_cast<unsigned>((groups + 3) / 4));
  const dim3 blk(64 * per_block);
  const int ncell = nufft_cells_per_source(ns);
  // Staged where a record has at most a quarter as many elements as the workgroup has lanes: with
  // more, the terms cost as much as each lane's own two do, and their way through LDS comes on
  // top. Staged against own terms, spreads of 2k to 60k facets by 8 or 64 chirps in parts of the
  // time without either form's block tests in levels: 12 x 16 elements 0.76 and 0.81, 32 x 32
  // 0.77 and 0.82, 8 x 8 0.72 and 0.74, 2 x 64 0.86 and 0.78, 64 x 1 0.96 and 0.73; with the delay
  // within the chirp 12 x 16 0.82 and 0.82, 8 x 8 0.81 and 0.78, 64 x 1 1.09 and 0.77.
  const bool staged = 4 * (rc.P + rc.Q) <= static_cast<int>(blk.x);
  ns.spread_batch = staged ? nufft_spread_batch(rc.P + rc.Q) : 1024;  // or a whole run
  const auto launch = [&](auto intra, auto stage) {
    return launch_spread_t<intra(), stage()>(sc, rc, ns, elem,
                                             static_cast<const NuRecF<intra()> *>(srec), runs,
                                             n_runs, part, bt, sgrid, blk, ncell, s);
  };
  if (rc.intra) return staged ? launch(std::true_type{}, std::true_type{})
                              : launch(std::true_type{}, std::false_type{});
  return staged ? launch(std::false_type{}, std::true_type{})
                : launch(std::false_type{}, std::false_type{});
}

}  // namespace rsim
