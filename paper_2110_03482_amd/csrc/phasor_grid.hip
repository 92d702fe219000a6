// Phasor sum as a non-uniform Fourier transform along the trial axis (Eqs. 4 and 7 for equal DM
// steps and exact delays), one transform per spin-frequency bin and time chunk.
//
// With trial DMs DM_j = DM_0 + j dDM, Eq. 1 is linear in j, so per bin f and chunk k
//     Y[j] = sum_c X[c] exp(2 pi i f tau[j, c] / L) = sum_c X'[c] exp(2 pi i (j - jc) u[c]),
//     u[c] = f dDM kappa_c / L (turns per trial),  X'[c] = X[c] exp(2 pi i f tau[jc, c] / L),
// i.e. n_chan values at positions u[c] on the unit circle, wanted at the integer frequencies
// j - jc: a type-1 non-uniform FFT (Dutt and Rokhlin 1993; the kernel below is Kaiser and
// Bessel's, as in Fessler and Sutton 2003).  Each X'[c] is spread over the 8 nearest points of an
// M-point grid with weights phi, the grid is transformed, and row j is divided by the transform of
// phi.  That costs 8 n_chan + M log2 M steps per (bin, chunk) where the matrix product takes
// n_dm n_chan: at 1024 channels and 2048 trials 60 times fewer operations.
//
// Accuracy: phi is the width-8 Kaiser-Bessel window with beta = 0.99 * 8 * 0.75 pi, each of its 8
// unit pieces replaced by a polynomial of degree 7 (TapTable), for M >= 2 n (n trials per grid).  The
// row divisors are the transform of those very polynomials (host, float64), so only aliasing is
// left: 5e-8 of the root mean square result at M = 2 n, 2.3e-8 at M = 4 n, against about 3e-7 for
// a float32 sum over 1024 channels.  All arithmetic is float32; positions keep 32 bits below a
// grid cell.
//
// Work decomposition (gfx950): one wave transforms 4096 points at a time, 64 per lane: one column
// (chunk) of M = 4096, or C = 4096 / M columns of the same bin.  A workgroup is 4 waves on 4
// consecutive bins, one workgroup per CU (the four grids take 130 KiB of LDS); it walks the
// columns of its bins, and positions and centre phasors, which the columns share, stay in
// registers.  Per column group a wave
//  - clears its grid and adds the spread values with LDS float atomics (ds_add_f32 without
//    return: nothing waits for them).  A grid belongs to one wave, whose LDS operations execute
//    in order, so the sums are formed in the same order in every run;
//  - transforms in two in-register passes, 64 points over stride M / 64 and M / 64 points over
//    the rest, with one exchange through LDS between them; of the second pass only the quarter of
//    the outputs at each end is wanted;
//  - hands its M / 2 rows to the workgroup through LDS, which writes 4 bins of a row at a time
//    (32 bytes of complex Y, or 16 of power).  Workgroups of one XCD hold neighbouring bins at a
//    time, so the 128-byte lines fill up in its L2.
#include <cmath>

#include "device_math.h"
#include "fdd_internal.h"
#include "fft_block.h"

namespace fdd {

namespace {
constexpr int kGXcds = 8;
constexpr int kGBins = 4;          // bins (waves) per workgroup
constexpr int kTaps = 8;

// phi on its unit pieces: tap i (grid point floor(x) - 3 + i) has the weight P_i(r), tap 7 - i the
// weight P_i(-r), r = x - floor(x) - 1/2; ascending powers of r; integral of phi = 1.
struct TapTable {
  float c[4][8] = {
      {4.143754164e-05f, -3.294314980e-04f, 1.117963969e-03f, -2.119961139e-03f, 2.452127913e-03f, -1.708908042e-03f,
       5.546764968e-04f, 3.850490173e-05f},
      {8.204603541e-03f, -2.957454497e-02f, 4.373736641e-02f, -3.193514291e-02f, 8.690131350e-03f, 3.420751334e-03f,
       -3.035205193e-03f, 4.183040296e-04f},
      {1.155015013e-01f, -2.115766630e-01f, 1.120707457e-01f, 2.270538891e-02f, -4.071746734e-02f, 6.610583888e-03f,
       5.612328843e-03f, -1.892843935e-03f},
      {3.762524780e-01f, -2.150915005e-01f, -1.569267914e-01f, 1.064023631e-01f, 2.958123973e-02f, -2.502987008e-02f,
       -3.147961217e-03f, 3.533136036e-03f}};
};

__device__ __forceinline__ void tap_weights(float r, float (&w)[kTaps]) {
  constexpr TapTable t{};
  const float r2 = r * r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float e = fmaf(fmaf(fmaf(t.c[i][6], r2, t.c[i][4]), r2, t.c[i][2]), r2, t.c[i][0]);
    const float o = fmaf(fmaf(fmaf(t.c[i][7], r2, t.c[i][5]), r2, t.c[i][3]), r2, t.c[i][1]);
    w[i] = fmaf(o, r, e);
    w[7 - i] = fmaf(-o, r, e);
  }
}

// Orders the LDS accesses of the lanes of one wave: its LDS operations execute in program order,
// so only the compiler has to be kept from moving them.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Workgroup barrier that orders LDS accesses only: global loads stay in flight.
__device__ __forceinline__ void grid_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// u, t -> u + w t, u - w t with the second as 2 u - (u + w t): 6 fused operations.
__device__ __forceinline__ void bfly(float2& u, float2& t, float wr, float wi) {
  const float ar = fmaf(-wi, t.y, fmaf(wr, t.x, u.x));
  const float ai = fmaf(wi, t.x, fmaf(wr, t.y, u.y));
  t = make_float2(fmaf(2.0f, u.x, -ar), fmaf(2.0f, u.y, -ai));
  u = make_float2(ar, ai);
}

// Stages LOGB .. LOG2(R) of a decimation-in-time transform with sign +, in place on x (bit-reversed
// order in, natural order out): stage s joins blocks of 2^(s-1).
template <int R, int LOGB>
__device__ __forceinline__ void dit_stages(float2* x) {
  constexpr RootTable<R, true> tab{};
#pragma unroll
  for (int half = 1 << (LOGB - 1); half < R; half *= 2) {
#pragma unroll
    for (int s = 0; s < R; s += 2 * half) {
#pragma unroll
      for (int j = 0; j < half; ++j) {
        float2& u = x[s + j];
        float2& t = x[s + j + half];
        const int m = j * (R / (2 * half));          // exp(2 pi i m / R)
        if (m == 0) {
          const float2 d = f2sub(u, t);
          u = f2add(u, t);
          t = d;
        } else if (4 * m == R) {                     // i t
          const float2 p = make_float2(u.x - t.y, u.y + t.x);
          t = make_float2(u.x + t.y, u.y - t.x);
          u = p;
        } else if (2 * half == R) {                  // last stage: outputs that nobody reads drop out one by one
          const float c = tab.c[m], sn = tab.s[m];
          const float2 p = make_float2(fmaf(-sn, t.y, fmaf(c, t.x, u.x)), fmaf(sn, t.x, fmaf(c, t.y, u.y)));
          t = make_float2(fmaf(sn, t.y, fmaf(-c, t.x, u.x)), fmaf(-sn, t.x, fmaf(-c, t.y, u.y)));
          u = p;
        } else {
          bfly(u, t, tab.c[m], tab.s[m]);
        }
      }
    }
  }
}

// The grid point, counted on through the turns, of the first tap of a channel with `inc` turns per
// bin and trial, at bin f (M points later, so that it is not negative).
template <int LOGM>
__device__ __forceinline__ int64_t first_tap(uint64_t inc, uint32_t f) {
  const uint64_t lo = (uint64_t)(uint32_t)inc * f;
  const uint64_t hi = (inc >> 32) * f + (lo >> 32);   // inc f in units of 2^-32 turns
  return (int64_t)(hi >> (32 - LOGM)) + (1 << LOGM) - 3;
}

template <int LOGM>
struct GridShape {
  static constexpr int M = 1 << LOGM;
  static constexpr int LM = M / 64;                  // lanes per column
  static constexpr int C = 64 / LM;                  // columns per wave
  static constexpr int GP = M + 8;                   // points per column: the grid and a guard of 7
  static constexpr int XP = 65;                      // exchange pitch (points)
  static constexpr int NB = M / 8;                   // buckets of 8 points
  static constexpr int PB = NB > 64 ? NB / 64 : 1;   // buckets per lane of the prefix sum
  // points per wave, 8 modulo 16 so that the rows of two waves read together at the hand-over
  // fall in different banks
  static constexpr int NEED = C * GP > 64 * XP ? C * GP : 64 * XP;
  static constexpr int RP = (NEED + 7) / 16 * 16 + 8;
  static_assert(RP >= NEED && RP % 2 == 0, "wave region too small");
};
}  // namespace

template <int LOGM, bool POWER>
__global__ __launch_bounds__(256, 1) void k_phasor_grid(GridArgs a, int n_bb, int n_split, int per_xcd) {
  using S = GridShape<LOGM>;
  constexpr int M = S::M, LM = S::LM, C = S::C, GP = S::GP, XP = S::XP, NB = S::NB, PB = S::PB;
  __shared__ __align__(16) float2 smem[kGBins * S::RP];
  __shared__ int hist[kGBins * (NB + 1)];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float2* const reg = smem + wave * S::RP;
  int* const cnt = hist + wave * (NB + 1);
  const int N = a.n_chunks;
  const int groups = (N + C - 1) / C;                // column groups per trial block
  const int n_it = groups * a.n_blk;
  const int64_t xrow = (int64_t)N * a.pitch;         // X: points per channel
  const int64_t yrow = xrow;                         // Y: points per trial
  const int jc = a.blk / 2;
  const int n_bat = (a.n_chan + 63) / 64;
  const int steps = (a.n_chan + LM - 1) / LM;        // channels per lane
  const uint32_t inv_steps = (uint32_t)(0xffffffffu / (uint32_t)steps) + 1u;   // steps = 1 is apart
  uint4* const sched = a.sched + ((int64_t)blockIdx.x * kGBins + wave) * a.sched_len;

  // The unit sequence of this workgroup: unit = (split of the iterations, bin block), bin block
  // fastest; each XCD owns a contiguous range and its workgroups take neighbouring units.
  const int xcd = (int)blockIdx.x % kGXcds, slot = (int)blockIdx.x / kGXcds, n_slot = (int)gridDim.x / kGXcds;
  const int n_unit = n_bb * n_split;
  const int u_end = min(n_unit, (xcd + 1) * per_xcd);
  int unit = xcd * per_xcd + slot;

  // twiddles of the second pass, exp(2 pi i l k1 / M) with k1 = lane
  float2 tw[LM];
#pragma unroll
  for (int l = 1; l < LM; ++l) tw[l] = turn_phasor<true>((uint32_t)(l * lane) << (32 - LOGM));
  // row divisors of the rows this thread writes
  constexpr int ROWS = C * (M / 2);                  // 2048 rows handed over per iteration
  constexpr int PER = POWER ? ROWS / 256 : ROWS / 128;
  constexpr int RSTEP = POWER ? 256 : 128;
  const int r0 = POWER ? tid : tid >> 1;
  constexpr int NDEC = (M / 2) / RSTEP > 0 ? ((M / 2) / RSTEP < PER ? (M / 2) / RSTEP : PER) : 1;
  float dec[NDEC];
#pragma unroll
  for (int i = 0; i < NDEC; ++i) dec[i] = a.dec[(r0 + i * RSTEP) & (M / 2 - 1)];

  const int lcol = lane / LM, lrow = lane % LM;       // this lane's column of the group, and its part of it
  for (; unit < u_end; unit += n_slot) {
    const int bb = unit % n_bb, sp = unit / n_bb;
    const int f0 = bb * kGBins;
    const int f = f0 + wave;
    const int itb = (int)((int64_t)n_it * sp / n_split), ite = (int)((int64_t)n_it * (sp + 1) / n_split);
    // The schedule of a bin.  The channels in order of their place on the grid are cut into LM
    // equal parts, one per lane of a column; in step i every lane adds its i-th channel, so the
    // channels added together are `steps` places of the order apart and their 8 points do not
    // meet (no atomics).  Where they would (few points per channel), 2^lq copies of the covered
    // part of the grid stand side by side and lane l adds to copy l mod 2^lq, and where that is
    // not enough a step goes in 2^ls turns.
    int lq = 0, ls = 0, c0 = 0;
    const int64_t ta = first_tap<LOGM>(a.inc_min, (uint32_t)f), tb = first_tap<LOGM>(a.inc_max, (uint32_t)f);
    int lq_most = 0;                                 // copies that the covered part leaves room for
    {
      const int64_t cover = tb - (ta & ~(int64_t)63) + 8;
      while (lq_most < LOGM - 6 && cover <= (M >> (lq_most + 1))) ++lq_most;
      if (lq_most > 0) c0 = (int)(ta & ~(int64_t)63) & (M - 1);
    }
    auto build = [&](int blk) {
      const uint4* tab = a.ctab + (int64_t)blk * a.n_chan;
#pragma unroll
      for (int i = 0; i < (NB + 63) / 64; ++i)
        if (64 * i + lane < NB) cnt[64 * i + lane] = 0;
      wave_order();
      // place of entry e: inc f as turns is a 64-bit fraction, whose top LOGM bits are the cell and
      // the next 32 the place inside it; the first tap lies 3 cells to the left
      auto place = [&](uint4 e, float* r) {
        const uint32_t flo = e.x * (uint32_t)f;
        const uint32_t fhi = e.y * (uint32_t)f + __umulhi(e.x, (uint32_t)f);
        const uint32_t fr = (fhi << LOGM) | (flo >> (32 - LOGM));
        *r = (float)(int32_t)(fr ^ 0x80000000u) * 2.3283064365386963e-10f;   // 2^-32
        return ((fhi >> (32 - LOGM)) + (uint32_t)(M - 3 - c0)) & (uint32_t)(M - 1);
      };
      // Adds the batch to the bucket counts and returns the count before this lane's channel.  The
      // channels come by ascending delay, so those of one bucket are neighbours unless the batch
      // goes round the whole circle.
      auto take = [&](int b, uint32_t bucket, bool act) {
        const int last = min(63, a.n_chan - 1 - 64 * b);
        const uint4 e0 = tab[64 * b], e1 = tab[64 * b + last];
        const int64_t span = first_tap<LOGM>(((uint64_t)e1.y << 32) | e1.x, (uint32_t)f) -
                             first_tap<LOGM>(((uint64_t)e0.y << 32) | e0.x, (uint32_t)f);
        int idx = 0;
        if (span < M - 8) {
          const uint32_t own = act ? bucket : (uint32_t)NB;
          const uint32_t prev = (uint32_t)__shfl_up((int)own, 1, 64);
          const unsigned long long heads = __ballot(lane == 0 || prev != own);
          const int head = 63 - __builtin_clzll(heads & (~0ull >> (63 - lane)));
          const bool tail = lane == 63 || ((heads >> (lane + 1)) & 1ull) != 0;
          if (act) idx = cnt[bucket] + (lane - head);
          wave_order();
          if (act && tail) cnt[bucket] = idx + 1;
        } else if (act) {
          idx = atomicAdd(&cnt[bucket], 1);
        }
        wave_order();
        return idx;
      };
      for (int b = 0; b < n_bat; ++b) {
        const int c = 64 * b + lane;
        const bool act = c < a.n_chan;
        float r;
        const uint32_t cell = place(tab[act ? c : a.n_chan - 1], &r);
        (void)take(b, cell >> 3, act);
      }
      // counts to starts, and the fullest pair of neighbouring buckets: channels at least that many
      // places apart in the order lie more than 8 points apart
      int n[PB + 1], sum = 0, pair = 0;
#pragma unroll
      for (int i = 0; i <= PB; ++i) {
        const int q = lane * PB + i;
        n[i] = q < NB ? cnt[q] : 0;
      }
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        pair = max(pair, n[i] + n[i + 1]);
        sum += n[i];
      }
      int start = sum;
#pragma unroll
      for (int o = 1; o < 64; o *= 2) {
        const int up = __shfl_up(start, o, 64);
        start += lane >= o ? up : 0;
        pair = max(pair, __shfl_xor(pair, o, 64));
      }
      start -= sum;
      wave_order();
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        if (lane * PB + i < NB) cnt[lane * PB + i] = start;
        start += n[i];
      }
      wave_order();
      pair = __builtin_amdgcn_readfirstlane(pair);
      lq = ls = 0;
      while ((steps << (lq + ls)) < pair) {
        if (lq < lq_most) ++lq;
        else ++ls;
      }
      for (int b = 0; b < n_bat; ++b) {
        const int c = 64 * b + lane;
        const bool act = c < a.n_chan;
        const uint4 e = tab[act ? c : a.n_chan - 1];
        const int ch = a.perm[act ? c : a.n_chan - 1];
        float r, sn, cs;
        const uint32_t cell = place(e, &r);
        const PhaseInc cinc = {e.w, e.z};
        sincos_turn(phase_at(cinc, (uint32_t)f), &sn, &cs);
        const uint32_t at = (uint32_t)take(b, cell >> 3, act);
        const uint32_t part = steps == 1 ? at : __umulhi(at, inv_steps);
        if (act)
          sched[(at - part * (uint32_t)steps) * LM + part] =
              make_uint4(__float_as_uint(r), (uint32_t)ch | (cell << 16), __float_as_uint(cs), __float_as_uint(sn));
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");   // entries are read by other lanes
    };
    for (int it = itb; it < ite; ++it) {
      const int blk = it / groups, k0 = (it % groups) * C;
      const bool fresh = it == itb || k0 == 0;       // first columns of the unit, or a new trial block
      // clear the grid
      {
        float4* z = reinterpret_cast<float4*>(reg);
        constexpr int NZ = (S::RP / 2 + 63) / 64;
#pragma unroll
        for (int i = 0; i < NZ; ++i)
          if (64 * i + lane < S::RP / 2) z[64 * i + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
      wave_order();
      if (fresh) build(blk);
      const int k = min(k0 + lcol, N - 1);
      const float2* xk = a.X + (int64_t)k * a.pitch + f;
      {
        float2* const mine = reg + lcol * GP + (lrow & ((1 << lq) - 1)) * (M >> lq);
        const int turn = (lrow >> lq) & ((1 << ls) - 1);
        const int own = min(steps, a.n_chan - lrow * steps);   // this lane's channels (<= 0: none)
        auto entry = [&](int i) {
          const uint4 e = sched[min(i, steps - 1) * LM + lrow];
          return i < own ? e : make_uint4(0u, 0u, 0u, 0u);
        };
        auto value = [&](uint4 e) { return xk[(int64_t)(e.y & 0xffffu) * xrow]; };
        constexpr int G = 4;
        uint4 e0[G], e1[G];
        float2 x0[G];
#pragma unroll
        for (int u = 0; u < G; ++u) e0[u] = entry(u);
#pragma unroll
        for (int u = 0; u < G; ++u) e1[u] = entry(G + u);
#pragma unroll
        for (int u = 0; u < G; ++u) x0[u] = value(e0[u]);
        for (int i = 0; i < steps; i += G) {
          uint4 e2[G];
          float2 x1[G];
#pragma unroll
          for (int u = 0; u < G; ++u) e2[u] = entry(i + 2 * G + u);
#pragma unroll
          for (int u = 0; u < G; ++u) x1[u] = value(e1[u]);
#pragma unroll
          for (int u = 0; u < G; ++u) {
            float w[kTaps];
            tap_weights(__uint_as_float(e0[u].x), w);
            const float cx = __uint_as_float(e0[u].z), cy = __uint_as_float(e0[u].w);
            const float xr = fmaf(cx, x0[u].x, -cy * x0[u].y), xi = fmaf(cx, x0[u].y, cy * x0[u].x);
            float2* p = mine + (e0[u].y >> 16);
            for (int tn = 0; tn < (1 << ls); ++tn) {
              if (i + u < own && turn == tn) {
                float2 g[kTaps];
#pragma unroll
                for (int q = 0; q < kTaps; ++q) g[q] = p[q];
#pragma unroll
                for (int q = 0; q < kTaps; ++q) p[q] = make_float2(fmaf(w[q], xr, g[q].x), fmaf(w[q], xi, g[q].y));
              }
              wave_order();
            }
          }
#pragma unroll
          for (int u = 0; u < G; ++u) {
            e0[u] = e1[u];
            e1[u] = e2[u];
            x0[u] = x1[u];
          }
        }
      }
      wave_order();
      // the 7 guard points past the end of a grid are its first ones
      for (int e = lane; e < 8 * C; e += 64) {
        const int q = e & 7;
        if (q < 7) {
          float2* g = reg + (e >> 3) * GP;
          g[q] = f2add(g[q], g[M + q]);
        }
      }
      wave_order();
      // first pass: lane (column ci, l) transforms the points l + LM a over a
      float2 v[64];
      {
        const float2* g = reg + lcol * GP + lrow;
#pragma unroll
        for (int q = 0; q < 64; ++q) v[q] = g[LM * cx_bitrev(q, 6)];
        // copies: the upper half of the grid joins the lower half, lq times
#pragma unroll
        for (int h = 32; h >= 1; h >>= 1) {
          if (lq >= 6 - cx_log2(h)) {
#pragma unroll
            for (int p = 0; p < h; ++p) {
              const int i0 = cx_bitrev(p, 6), i1 = cx_bitrev(p + h, 6);
              v[i0] = f2add(v[i0], v[i1]);
              v[i1] = make_float2(0.0f, 0.0f);
            }
          }
        }
      }
      dit_stages<64, 1>(v);
      wave_order();
#pragma unroll
      for (int k1 = 0; k1 < 64; ++k1) reg[lane * XP + k1] = v[k1];
      wave_order();
      // second pass: lane k1 transforms the LM points of every column
#pragma unroll
      for (int ci = 0; ci < C; ++ci)
#pragma unroll
        for (int q = 0; q < LM; ++q) v[ci * LM + q] = reg[(ci * LM + cx_bitrev(q, cx_log2(LM))) * XP + lane];
      wave_order();
#pragma unroll
      for (int ci = 0; ci < C; ++ci) {
        float2* x = v + ci * LM;
#pragma unroll
        for (int q = 0; q < LM; q += 2) {            // twiddles and the first stage
          constexpr int LB = cx_log2(LM);
          const int l0 = cx_bitrev(q, LB), l1 = cx_bitrev(q + 1, LB);
          if (l0 != 0) x[q] = cmulf(x[q], tw[l0]);
          bfly(x[q], x[q + 1], tw[l1].x, tw[l1].y);
        }
        dit_stages<LM, 2>(x);
        if (c0 != 0) {                               // the grid begins c0 points (64 at a time) into the circle
          const float2 rot = turn_phasor<true>((uint32_t)((c0 >> 6) * lane) << (32 - (LOGM - 6)));
#pragma unroll
          for (int k2 = 0; k2 < LM; ++k2)
            if (k2 < LM / 4 || k2 >= 3 * (LM / 4)) x[k2] = cmulf(x[k2], rot);
        }
        // rows -M/4 .. M/4 - 1 around the centre
#pragma unroll
        for (int k2 = 0; k2 < LM / 4; ++k2) {
          reg[ci * (M / 2) + M / 4 + 64 * k2 + lane] = x[k2];
          reg[ci * (M / 2) + 64 * k2 + lane] = x[k2 + 3 * (LM / 4)];
        }
      }
      grid_barrier();
      // hand-over: 4 bins of each row
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int ci = (i * RSTEP) / (M / 2);
        const int rb = (i * RSTEP) % (M / 2);        // uniform part of the row
        const int k = k0 + ci;
        const int row = ci * (M / 2) + ((rb + r0) & (M / 2 - 1));
        const int j = ((rb + r0) & (M / 2 - 1)) - M / 4 + jc;   // trial within the block
        const int dm = blk * a.blk + j;
        const bool ok = k < N && j >= 0 && j < a.blk && dm < a.n_dm;
        const float d = dec[i % NDEC];
        if constexpr (POWER) {
          float pw[kGBins];
#pragma unroll
          for (int w = 0; w < kGBins; ++w) {
            float2 y = smem[w * S::RP + row];
            y = make_float2(y.x * d, y.y * d);
            if (f0 + w == 0) y.x += a.dc_add;
            pw[w] = fmaf(y.x, y.x, y.y * y.y);
          }
          if (ok && f0 < a.n_pow_bins)
            *(float4*)(a.P + (int64_t)dm * a.n_pow_bins + f0) = make_float4(pw[0], pw[1], pw[2], pw[3]);
        } else {
          const int h = tid & 1;
          const float2 y0 = smem[(2 * h) * S::RP + row], y1 = smem[(2 * h + 1) * S::RP + row];
          if (ok)
            *(float4*)(a.Yc + (int64_t)dm * yrow + (int64_t)k * a.pitch + f0 + 2 * h) =
                make_float4(y0.x * d, y0.y * d, y1.x * d, y1.y * d);
        }
      }
      grid_barrier();
    }
  }
}

namespace {
template <int LOGM, bool POWER>
hipError_t launch_grid(const GridArgs& a, hipStream_t st) {
  constexpr int C = GridShape<LOGM>::C;
  const int n_bb = ((POWER ? a.n_pow_bins : a.n_bins) + kGBins - 1) / kGBins;
  const int n_it = ((a.n_chunks + C - 1) / C) * a.n_blk;
  // enough units that every CU has several, without cutting the columns of a bin finer than that
  int n_split = 1;
  while (n_split < n_it && (int64_t)n_bb * n_split < 1024) ++n_split;
  const int64_t units = (int64_t)n_bb * n_split;
  if (units > 0x3fffffff) return hipErrorInvalidValue;
  const int per_xcd = (int)((units + kGXcds - 1) / kGXcds);
  const int slots = per_xcd < kGridBlocks / kGXcds ? per_xcd : kGridBlocks / kGXcds;
  hipLaunchKernelGGL((k_phasor_grid<LOGM, POWER>), dim3((unsigned)(kGXcds * slots)), dim3(256), 0, st, a, n_bb,
                     n_split, per_xcd);
  return hipGetLastError();
}

hipError_t launch_grid_m(const GridArgs& a, hipStream_t st) {
  if (a.P != nullptr) return launch_grid<12, true>(a, st);   // one chunk: one column per wave
  switch (a.log_m) {
    case 8: return launch_grid<8, false>(a, st);
    case 9: return launch_grid<9, false>(a, st);
    case 10: return launch_grid<10, false>(a, st);
    case 11: return launch_grid<11, false>(a, st);
    case 12: return launch_grid<12, false>(a, st);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

hipError_t launch_phasor_grid(const GridArgs& a, hipStream_t st) {
  if (a.X == nullptr || a.ctab == nullptr || a.dec == nullptr || a.perm == nullptr || a.sched == nullptr || a.sched_len < (a.n_chan + 63) / 64 * 64 || (a.Yc == nullptr) == (a.P == nullptr) || a.n_dm < 1 ||
      a.n_chan < 1 || a.n_chunks < 1 || a.blk < 1 || 2 * a.blk > (1 << a.log_m) ||
      (int64_t)a.n_blk * a.blk < a.n_dm || (a.n_blk > 1 && a.log_m != 12) || (a.P != nullptr && (a.n_chunks != 1 || a.log_m != 12)))
    return hipErrorInvalidValue;
  return launch_grid_m(a, st);
}

// Row divisors 1 / phihat((idx - M/4) / M), idx < M/2, phihat the Fourier transform of the
// piecewise polynomial phi (8-point Gauss-Legendre per piece: exact for degree 7 times the
// cosine's expansion to well below float64 rounding of the result at |k| <= M/4).
void grid_divisors(int log_m, std::vector<float>* out) {
  static const double kX[8] = {0.0950125098376374, 0.2816035507792589, 0.4580167776572274, 0.6178762444026438,
                               0.7554044083550030, 0.8656312023878318, 0.9445750230732326, 0.9894009349916499};
  static const double kW[8] = {0.1894506104550685, 0.1826034150449236, 0.1691565193950025, 0.1495959888165767,
                               0.1246289712555339, 0.0951585116824928, 0.0622535239386479, 0.0271524594117541};
  const TapTable t{};
  const int half = 1 << (log_m - 1);
  out->resize((size_t)half);
  for (int idx = 0; idx < half; ++idx) {
    const double om = 2.0 * 3.14159265358979323846 * (double)(idx - half / 2) / (double)(2 * half);
    double sum = 0.0;
    for (int i = 0; i < 4; ++i)
      for (int q = 0; q < 16; ++q) {
        const double r = 0.5 * (q < 8 ? kX[q] : -kX[q - 8]), wt = 0.5 * kW[q & 7];
        double p = 0.0;
        for (int d = 7; d >= 0; --d) p = p * r + (double)t.c[i][d];
        sum += 2.0 * wt * p * std::cos(om * ((double)i - 3.5 - r));   // taps i and 7 - i
      }
    (*out)[(size_t)idx] = (float)(1.0 / sum);
  }
}

}  // namespace fdd
