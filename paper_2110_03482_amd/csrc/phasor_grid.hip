// Phasor sum as a non-uniform Fourier transform along the trial axis (Eqs. 4 and 7 for equal DM
// steps and exact delays), one transform per spin-frequency bin and time chunk.
//
// With trial DMs DM_j = DM_0 + j dDM, Eq. 1 is linear in j, so per bin f and chunk k
//     Y[j] = sum_c X[c] exp(2 pi i f tau[j, c] / L) = sum_c X'[c] exp(2 pi i (j - jc) u[c]),
//     u[c] = f dDM kappa_c / L (turns per trial),  X'[c] = X[c] exp(2 pi i f tau[jc, c] / L),
// i.e. n_chan values at positions u[c] on the unit circle, wanted at the integer frequencies
// j - jc: a type-1 non-uniform FFT (Dutt and Rokhlin 1993).  Each X'[c] is spread over the 8 nearest
// points of an M-point grid with weights phi, the grid is transformed, and row j is divided by the
// transform of phi.  That costs 8 n_chan + M log2 M steps per (bin, chunk) where the matrix product takes
// n_dm n_chan: at 1024 channels and 2048 trials 60 times fewer operations.
//
// Accuracy: phi has width 8 and consists of unit pieces of degree 7 (TapTable), for M >= 2 n (n
// trials per grid).  The row divisors are the transform of those very polynomials (host, float64), so
// only aliasing is left: 2.8e-8 at the worst row of M = 2 n and 1.9e-8 on average.  (The
// Kaiser-Bessel window of that width with its best beta, the pieces fitted to it: 1.6e-7 at the
// outermost rows, 5e-8 on average.)  All arithmetic is float32; positions keep 32 bits below a grid
// cell.  A low bin, whose channels all fall in the same cells, has 9e-8 in all, as much from the
// transform as from the sums and the rounding of the divisors.
//
// Work decomposition (gfx950): one wave transforms 4096 points at a time, 64 per lane: one column
// (chunk) of M = 4096, or C = 4096 / M columns of the same bin.  The grid of a wave takes 33 KiB of
// LDS, so there are 4 waves per CU, one per SIMD with up to 512 registers each: 2 workgroups of 2
// waves (neighbouring bins) where the values are staged or read for complex rows, and 1 workgroup of
// 4 where 16 bytes of a row of powers are written at a time.  Neighbouring workgroups of an XCD hold
// neighbouring bins, so the 128-byte lines of X and Y fill up in its L2.  Workgroups are persistent:
// each walks (bin block, part of the columns), and what the columns of a bin share is made once.
//  - k_grid_order sorts the channels by their place on the grid, once per group of bins in which no
//    channel moves far.  From that order every lane gets two runs of channels whose 8 points never
//    meet another lane's in the same step, so the sums are plain read, add and write in LDS and are
//    formed in the same order in every run.  (LDS float atomics take about 240 cycles per wave
//    instruction here: 69 ms where this order takes 14 ms, 1024 channels, 2048 trials, 21 chunks of
//    65536 samples.)
//  - The values of the next columns are loaded during the transform, put into LDS during the
//    hand-over and read from there in the lane's order; with more than 16 steps per column group
//    they are read from memory where they are used.
//  - The transform goes in two in-register passes, 64 points over stride M / 64 and M / 64 points
//    over the rest, with one exchange through LDS between them; of the second pass only the quarter
//    of the outputs at each end is wanted, and the workgroup writes them row by row through LDS.
// Bound: instruction issue and LDS of one wave per SIMD.  At 1024 channels, 2048 trials, 21 chunks of
// 65536 samples, float32: 13.2 to 14.0 ms (matrix product 104 ms; reading X and writing Y once takes
// 3.6 ms); VALU issue 40 % of the cycles, LDS busy in 48 % (half of that bank conflicts), waits for
// memory or LDS 19 %.  512 channels, 2048 trials, one chunk of 2^22 samples, powers: 38 ms (113 ms),
// 18 ns per transform (the other: 20); VALU 37 %, LDS 33 %, waits 24 %: a bin's entries serve
// one column only, and 35 GB are written for 17.
#include <cmath>
#include <mutex>

#include "device_math.h"
#include "fdd_internal.h"
#include "fft_block.h"

namespace fdd {

namespace {
constexpr int kGXcds = 8;

// The work of a launch in units (a bin block and a part of its column groups): n_main of them are the
// first bb_main bin blocks in `split` parts each, whole rounds of the workgroups, and n_tail the other
// bb_tail bin blocks in tail_split parts.  (There are 2^k + 1 bins: with all blocks cut alike, the last
// one would be a round of its own: 200 channels, 301 trials, 15 chunks of 8192 samples 405 -> 373 us per
// call, 1024 channels, 2048 trials, 21 chunks of 65536 22.2 -> 21.6 ms.)  In both, each XCD has a
// contiguous range of at most main_xcd or tail_xcd units, bin blocks fastest, and its workgroups take
// neighbouring ones.
struct GridWork {
  int n_main, bb_main, split, main_xcd;
  int n_tail, bb_tail, tail_split, tail_xcd;
};
struct GridUnit {
  int bb, part, parts;
};
__host__ __device__ inline GridUnit grid_unit(const GridWork& w, int unit) {
  if (unit < w.n_main) return {unit % w.bb_main, unit / w.bb_main, w.split};
  const int t = unit - w.n_main;
  return {w.bb_main + t % w.bb_tail, t / w.bb_tail, w.tail_split};
}
// Unit i of a workgroup (0, 1, ..), or -1 past the last.
__host__ __device__ inline int grid_nth(const GridWork& w, int xcd, int slot, int n_slot, int i) {
  const int m0 = w.main_xcd * xcd, m1 = w.n_main < m0 + w.main_xcd ? w.n_main : m0 + w.main_xcd;
  const int n = m0 + slot < m1 ? (m1 - m0 - slot + n_slot - 1) / n_slot : 0;   // main units of this workgroup
  if (i < n) return m0 + slot + i * n_slot;
  const int t0 = w.tail_xcd * xcd, t1 = w.n_tail < t0 + w.tail_xcd ? w.n_tail : t0 + w.tail_xcd;
  const int t = t0 + slot + (i - n) * n_slot;
  return t < t1 ? w.n_main + t : -1;
}
// The plan of n_bb bin blocks of n_it column groups on `blocks` workgroups: enough units that every
// workgroup has several, without cutting finer than a column group, and the tail cut so that it ends
// soonest (a unit also makes the entries of its bins, about a third of a column group's time).
inline GridWork grid_work(int n_bb, int n_it, int blocks) {
  GridWork w = {};
  w.split = 1;
  while (w.split < n_it && (int64_t)n_bb * w.split < 4 * blocks) ++w.split;
  int step = blocks;                                 // bin blocks whose units are whole rounds
  for (int d = 2; d <= w.split; d *= 2)
    if (w.split % d == 0 && step % 2 == 0) step /= 2;
  w.bb_main = n_bb / step * step;
  w.n_main = w.bb_main * w.split;
  w.main_xcd = w.n_main / kGXcds;
  w.bb_tail = n_bb - w.bb_main;
  if (w.bb_tail > 0) {
    int best = -1;
    for (int ts = w.split; ts <= n_it && ts <= 4096; ++ts) {
      const int64_t units = (int64_t)w.bb_tail * ts, xcd = (units + kGXcds - 1) / kGXcds;
      const int64_t rounds = (xcd + blocks / kGXcds - 1) / (blocks / kGXcds);
      const int64_t cost = rounds * (3 * ((n_it + ts - 1) / ts) + 1);
      if (best >= 0 && cost >= best) continue;
      best = (int)(cost < 0x7fffffff ? cost : 0x7fffffff);
      w.tail_split = ts;
    }
    w.n_tail = w.bb_tail * w.tail_split;
    w.tail_xcd = (w.n_tail + kGXcds - 1) / kGXcds;
  }
  return w;
}
// Bins (waves) per workgroup.
template <bool POWER>
constexpr int grid_bins() {
  return POWER ? 4 : 2;
}
constexpr int kTaps = 8;

// Four powers of a row of the caller's output, which may begin at any float: the compiler is told
// so, and gfx950 writes them in one access all the same.
struct __attribute__((packed, aligned(4))) PowerQuad {
  float a, b, c, d;
};

// phi on its unit pieces: tap i (grid point floor(x) - 3 + i) has the weight P_i(r), tap 7 - i the
// weight P_i(-r), r = x - floor(x) - 1/2; ascending powers of r; integral of phi = 1.
// Made by reweighted least squares: of all such phi the one whose worst ratio of aliases (frequencies
// k + p M, p != 0) to the wanted transform over |k| <= M / 4 is smallest.
struct TapTable {
  float c[4][8] = {{9.869510541e-05f, -6.835844833e-04f, 1.989906188e-03f, -3.184069414e-03f, 3.077049041e-03f, -1.796103199e-03f,
       4.782984615e-04f, 1.403559781e-05f},
      {1.095001679e-02f, -3.583149984e-02f, 4.743985459e-02f, -2.995475382e-02f, 5.496605299e-03f, 4.388341680e-03f,
       -2.684250707e-03f, 3.629339626e-04f},
      {1.229900271e-01f, -2.074640393e-01f, 9.574311972e-02f, 2.762516774e-02f, -3.492985293e-02f, 3.268321743e-03f,
       5.053000525e-03f, -1.630702289e-03f},
      {3.659612536e-01f, -1.936641484e-01f, -1.451727450e-01f, 8.917669952e-02f, 2.635781839e-02f, -1.916933432e-02f,
       -2.856537467e-03f, 3.071275540e-03f}};
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
  static constexpr int GL = kGridGuard;              // guard points before the grid, at least 8
  static constexpr int GP = M + 2 * GL + 8;          // points per column: guard, grid, guard and the 7 taps to the right
  // exchange pitch (points): even, so that two points written at a time stay together, and 4 words
  // modulo the 64 banks, so that 16 lanes of such a write fall in different ones
  static constexpr int XP = 66;
  // staged values lie behind the 2048 rows (or the entries of 16 steps) of a wave
  static constexpr int SO = 2048 + 8;
  static constexpr int NB = M / 8;                   // buckets of 8 points
  static constexpr int PB = NB > 64 ? NB / 64 : 1;   // buckets per lane of the prefix sum
  // points per wave, 8 modulo 16 so that the rows of two waves read together at the hand-over
  // fall in different banks
  static constexpr int NEED = C * GP > 64 * XP ? C * GP : 64 * XP;
  static constexpr int RP = (NEED + 7) / 16 * 16 + 8;
  static_assert(RP >= SO + 16 * 64 && RP >= NEED && RP >= C * GP + 8 && RP % 2 == 0, "wave region too small");
};
}  // namespace

// inc f as turns: its fraction's top LOGM bits are the cell (the result) and the next 32 the place r
// inside it; `far` counts cells on through the turns (modulo 2^32).
template <int LOGM>
__device__ __forceinline__ uint32_t grid_place(uint4 e, uint32_t f, float* r, uint32_t* far) {
  const uint32_t flo = e.x * f;
  const uint32_t c1 = __umulhi(e.x, f);
  const uint32_t fhi = e.y * f + c1;
  const uint32_t turns = __umulhi(e.y, f) + (fhi < c1 ? 1u : 0u);
  const uint32_t fr = (fhi << LOGM) | (flo >> (32 - LOGM));
  *r = (float)(int32_t)(fr ^ 0x80000000u) * 2.3283064365386963e-10f;   // 2^-32
  const uint32_t cell = fhi >> (32 - LOGM);
  *far = (turns << LOGM) + cell;
  return cell;
}

// What the bins fa .. fb of one order have in common: whether their channels go round less than
// once, then a point c0 (a multiple of 64) that the part which they cover begins at, or up to 8
// points before (the low bins begin 3 points before 0, and c0 = 0 saves them a rotation of the
// result), and the copies of it, as a power of two, that the grid has room for.
struct GridCover {
  bool once;
  int c0, copies;
};
template <int LOGM>
__device__ __forceinline__ GridCover grid_cover(const GridArgs& a, uint32_t fa, uint32_t fb) {
  constexpr int M = 1 << LOGM;
  const int64_t ta = first_tap<LOGM>(a.inc_min, fa), tb = first_tap<LOGM>(a.inc_max, fb);
  const int64_t from = (ta + 8) & ~(int64_t)63;
  const int64_t cover = tb + 8 - (from - 8);
  GridCover c = {cover <= M, 0, 0};
  if (!c.once) return c;
  c.c0 = (int)from & (M - 1);
  while (c.copies < LOGM - 6 && cover <= (M >> (c.copies + 1))) ++c.copies;
  return c;
}

// The order of the channels by their place on the grid, for every group of 2^log_gb bins whose
// channels go round the circle more than once (a.places; less than once it is the order of their
// delays), and the turns that a step takes in it (a.turns).  One wave per group: counts per bucket
// of 8 points, their running sum, and every channel's place in it.
template <int LOGM>
__global__ __launch_bounds__(64) void k_grid_order(GridArgs a) {
  using S = GridShape<LOGM>;
  constexpr int M = S::M, LM = S::LM, NB = S::NB, PB = S::PB;
  constexpr int U = 4;                               // batches whose loads and arithmetic go together
  __shared__ int cnt[NB + 1];
  const int lane = (int)threadIdx.x;
  const int g = (int)blockIdx.x;
  const uint32_t fa = (uint32_t)g << a.log_gb, fr = fa + ((1u << a.log_gb) >> 1);
  if (grid_cover<LOGM>(a, fa, fa + (1u << a.log_gb) - 1u).once) return;
  const int n_bat = (a.n_chan + 63) / 64;
  const int q = (a.n_chan + 2 * LM - 1) / (2 * LM);   // channels of a part
  uint16_t* const places = a.places + (int64_t)g * a.sched_len;
  // Adds a batch to the bucket counts and returns the count before this lane's channel.  The
  // channels come by ascending delay, so those of one bucket are neighbours unless the batch goes
  // round the whole circle.
  auto take = [&](uint32_t bucket, uint32_t far, bool act, int last) {
    const uint32_t span = (uint32_t)__builtin_amdgcn_readlane((int)far, last) -
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)far);
    int idx = 0;
    if (span < (uint32_t)(M - 8)) {
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
  auto batches = [&](auto&& use) {
    for (int b0 = 0; b0 < n_bat; b0 += U) {
      uint32_t cell[U], far[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float r;
        const uint32_t c = grid_place<LOGM>(a.ctab[min(64 * (b0 + u) + lane, a.n_chan - 1)], fr, &r, &far[u]);
        cell[u] = (c + (uint32_t)(M - 3)) & (uint32_t)(M - 1);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = 64 * (b0 + u) + lane;
        if (b0 + u < n_bat) use(c, take(cell[u] >> 3, far[u], c < a.n_chan, min(63, a.n_chan - 1 - 64 * (b0 + u))));
      }
    }
  };
#pragma unroll
  for (int i = 0; i < (NB + 63) / 64; ++i)
    if (64 * i + lane < NB) cnt[64 * i + lane] = 0;
  wave_order();
  batches([](int, int) {});
  int n[PB], sum = 0;
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    n[i] = lane * PB + i < NB ? cnt[lane * PB + i] : 0;
    sum += n[i];
  }
  int start = sum;
#pragma unroll
  for (int o = 1; o < 64; o *= 2) {
    const int up = __shfl_up(start, o, 64);
    start += lane >= o ? up : 0;
  }
  start -= sum;
  wave_order();
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    if (lane * PB + i < NB) cnt[lane * PB + i] = start;
    start += n[i];
  }
  if (lane == 0) cnt[NB] = a.n_chan;
  wave_order();
  // the fullest a.window neighbouring buckets: channels that many places apart in the order lie more
  // than 8 (window - 1) points apart at bin fr, and so 8 or more at each bin of the group
  int most = 0;
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int k = lane * PB + i;
    if (k < NB) most = max(most, cnt[min(k + a.window, NB)] - cnt[k]);
  }
#pragma unroll
  for (int o = 1; o < 64; o *= 2) most = max(most, __shfl_xor(most, o, 64));
  int ls = 0;
  while ((q << ls) < most) ++ls;
  if (lane == 0) a.turns[g] = ls;
  wave_order();
  batches([&](int c, int idx) {
    if (c < a.n_chan) places[c] = (uint16_t)idx;
  });
}

// NS > 0: at most NS (16) schedule steps, the values of a column staged in channel order; NS = 0: any
// number, every value read where its step needs it.
template <int LOGM, int NS, bool POWER>
__global__ __launch_bounds__(64 * grid_bins<POWER>(), 1) void k_phasor_grid(GridArgs a, GridWork work) {
  using S = GridShape<LOGM>;
  constexpr int FB = grid_bins<POWER>();
  constexpr int M = S::M, LM = S::LM, C = S::C, GP = S::GP, XP = S::XP, GL = S::GL;
  __shared__ __align__(16) float2 smem[FB * S::RP];
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float2* const reg = smem + wave * S::RP;
  const int N = a.n_chunks;
  const int groups = (N + C - 1) / C;                // column groups per trial block
  const int n_it = groups * a.n_blk;
  const int64_t xrow = (int64_t)N * a.pitch;         // X: points per channel
  const int64_t yrow = xrow;                         // Y: points per trial
  const int jc = a.blk / 2;
  const int n_bat = (a.n_chan + 63) / 64;
  const int q = (a.n_chan + 2 * LM - 1) / (2 * LM);   // channels of a part: a lane has two parts
  const int steps = 2 * q;
  const uint32_t inv_q = (uint32_t)(0xffffffffu / (uint32_t)q) + 1u;   // q = 1 is apart
  uint4* const sched = a.sched + ((int64_t)blockIdx.x * FB + wave) * a.sched_len;   // of this wave (NS = 0)

  // the units of this workgroup
  const int xcd = (int)blockIdx.x % kGXcds, slot = (int)blockIdx.x / kGXcds, n_slot = (int)gridDim.x / kGXcds;
  int nth = 0, unit = grid_nth(work, xcd, slot, n_slot, 0);
  if (unit < 0) return;                              // the whole workgroup, before any barrier

  // twiddles of the second pass, exp(2 pi i l k1 / M) with k1 = lane
  // (l = TB la + lb: two short tables and a product instead of 2 LM registers)
  constexpr int TB = LM > 8 ? 8 : LM, TA = LM / TB;
  float2 twa[TA], twb[TB];
#pragma unroll
  for (int l = 0; l < TA; ++l) twa[l] = turn_phasor<true>((uint32_t)(TB * l * lane) << (32 - LOGM));
#pragma unroll
  for (int l = 0; l < TB; ++l) twb[l] = turn_phasor<true>((uint32_t)(l * lane) << (32 - LOGM));
  auto twiddle = [&](int l) { return l < TB ? twb[l] : l % TB == 0 ? twa[l / TB] : cmulf(twa[l / TB], twb[l % TB]); };
  // row divisors of the rows this thread writes
  constexpr int ROWS = C * (M / 2);                  // 2048 rows handed over per iteration
  // threads per row: one, or one for every two bins of complex rows
  constexpr int TR = POWER ? 1 : FB / 2;
  constexpr int RSTEP = 64 * FB / TR;
  constexpr int PER = ROWS / RSTEP;
  const int r0 = tid / TR, rh = tid % TR;
  constexpr int NDEC = (M / 2) / RSTEP > 0 ? ((M / 2) / RSTEP < PER ? (M / 2) / RSTEP : PER) : 1;
  float dec[NDEC];
#pragma unroll
  for (int i = 0; i < NDEC; ++i) dec[i] = a.dec[(r0 + i * RSTEP) & (M / 2 - 1)];

  const int lcol = lane / LM, lrow = lane % LM;       // this lane's column of the group, and its part of it
  constexpr int NL = NS > 0 ? NS / 2 : 1;            // 16-byte loads of a thread per column group
  constexpr int TP = FB / 2;                         // threads that load one value's bins
  float4 raw[NL];                                    // the values of the next column group
  // Straight-line loads and writes (a value past the last repeats it): a branch among them would
  // make the compiler wait for the loads at the end of the branch.
  const int total = C * a.n_chan;                    // values of a column group
  auto load_raw = [&](int k0, int fa) {
    int to = tid;
    asm volatile("" : "+v"(to));
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int v = min(128 * i + to / TP, total - 1);   // value (column, channel) of this thread's bin pair
      const int ci = C > 1 ? v / a.n_chan : 0, c = v - ci * a.n_chan;
      raw[i] = *reinterpret_cast<const float4*>(a.X + (int64_t)c * xrow + (int64_t)min(k0 + ci, N - 1) * a.pitch + fa +
                                                2 * (to % TP));
    }
  };
  auto put_raw = [&]() {
    int to = tid;
    asm volatile("" : "+v"(to));
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      float2* at = smem + 2 * (to % TP) * S::RP + S::SO + min(128 * i + to / TP, total - 1);
      at[0] = make_float2(raw[i].x, raw[i].y);
      at[S::RP] = make_float2(raw[i].z, raw[i].w);
    }
  };
  auto first_col = [&](const GridUnit& u) { return (int)((int64_t)n_it * u.part / u.parts) % groups * C; };
  if constexpr (NS > 0) {
    const GridUnit u = grid_unit(work, unit);
    load_raw(first_col(u), u.bb * FB);
    put_raw();
    grid_barrier();
  }
  for (int next; unit >= 0; unit = next) {
    next = grid_nth(work, xcd, slot, n_slot, ++nth);
    const GridUnit un = grid_unit(work, unit);
    const int bb = un.bb, sp = un.part;
    const int f0 = bb * FB;
    // a wave past the last bin repeats it (its row pieces fall into the padding of Y)
    const int f = min(f0 + wave, (POWER ? a.n_pow_bins : a.n_bins) - 1);
    const int itb = (int)((int64_t)n_it * sp / un.parts), ite = (int)((int64_t)n_it * (sp + 1) / un.parts);
    // The schedule of a bin.  The channels in order of their place on the grid are cut into 2 LM
    // equal parts of q, two per lane of a column; in step i every lane adds the i-th channel of both,
    // so the channels added together are q places of the order apart and their 8 points do not meet
    // (no atomics, and a lane's two sums are formed side by side).  Where they would (few points per
    // channel), 2^lq copies of the covered part of the grid stand side by side and part v adds to
    // copy v mod 2^lq, and where that is not enough a step goes in 2^ls turns.  The 2^log_gb bins of
    // a group share one order, that of their middle bin fr: no channel moves by more than the guard
    // within them.
    const int grp = f >> a.log_gb;
    const uint32_t fa = (uint32_t)grp << a.log_gb, fr = fa + ((1u << a.log_gb) >> 1);
    const GridCover cov = grid_cover<LOGM>(a, fa, fa + (1u << a.log_gb) - 1u);
    const bool once = cov.once;
    const int c0 = cov.c0;
    int lq = 0, ls = 0;
    if (once) {
      // channels q 2^(lq + ls) apart are at least gap f turns apart
      auto meet = [&](int j) {
        const uint64_t d = a.gap[j];
        if (d == ~0ull) return false;
        const uint64_t hi = (d >> 32) * fa + (((uint64_t)(uint32_t)d * fa) >> 32);
        return (hi >> (32 - LOGM)) < 8u;
      };
      while (lq + ls < LOGM - 5 && meet(lq + ls)) {
        if (lq < cov.copies) ++lq;
        else ++ls;
      }
    } else {
      ls = min(__builtin_amdgcn_readfirstlane(a.turns[grp]), LOGM - 5);
    }
    const uint16_t* const places = a.places + (int64_t)grp * a.sched_len;
    // The entries of this wave's bin, of trial block blk, in their places: in its LDS region (NS > 0;
    // the lanes then take theirs) or its schedule.
    auto entries = [&](int blk) {
      const uint4* tab = a.ctab + (int64_t)blk * a.n_chan;
      constexpr int U = 4;
      for (int b0 = 0; b0 < n_bat; b0 += U) {
        uint4 e[U];
        int ch[U];
        uint32_t at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c = min(64 * (b0 + u) + lane, a.n_chan - 1);
          e[u] = tab[c];
          ch[u] = a.perm[c];
          at[u] = once ? (uint32_t)c : (uint32_t)places[c];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float r, rq, sn, cs;
          uint32_t far, farq;
          const uint32_t cell = grid_place<LOGM>(e[u], (uint32_t)f, &r, &far);
          uint32_t to;                               // first tap within the column
          if (once) {
            to = ((cell + (uint32_t)(M + 8 - 3 - c0)) & (uint32_t)(M - 1)) + (GL - 8);
          } else {
            const uint32_t cq = grid_place<LOGM>(e[u], fr, &rq, &farq);
            to = ((cq + (uint32_t)(M - 3)) & (uint32_t)(M - 1)) + GL + (far - farq);
          }
          const PhaseInc cinc = {e[u].w, e[u].z};
          sincos_turn(phase_at(cinc, (uint32_t)f), &sn, &cs);
          const uint32_t part = q == 1 ? at[u] : __umulhi(at[u], inv_q);
          uint4* const dst = NS > 0 ? reinterpret_cast<uint4*>(reg) : sched;
          if (64 * (b0 + u) + lane < a.n_chan)
            dst[(2 * (at[u] - part * (uint32_t)q) + (part & 1u)) * LM + (part >> 1)] =
                make_uint4(__float_as_uint(r), (uint32_t)ch[u] | (to << 16), __float_as_uint(cs), __float_as_uint(sn));
        }
      }
      if constexpr (NS > 0) wave_order();
      else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");   // entries are read by other lanes
    };
    // The spread runs in groups of G steps.  The values of a column, staged: the workgroup loads
    // them in channel order (the bins of a channel together, during the transform of the column
    // before) and puts each bin's into the region of its wave, from where the wave takes them in
    // schedule order; the entries stay in registers.  Otherwise every lane reads entries and values
    // from memory, three and two groups ahead.
    constexpr int G = 4, R = 4;
    constexpr int NI = NS > 0 ? NS : 1;
    const int n_grp = (steps + G - 1) / G;
    // whether entry i = 2 (step) + (part) of this lane is a channel
    const int own0 = min(q, a.n_chan - 2 * lrow * q), own1 = min(q, a.n_chan - (2 * lrow + 1) * q);
    auto has = [&](int i) { return (i >> 1) < ((i & 1) ? own1 : own0); };
    uint4 eb[R][G];
    float2 xb[R][G];
    uint4 ent[NI];                                   // this lane's entries
    auto load_e = [&](uint4 (&e)[G], int g) {
#pragma unroll
      for (int u = 0; u < G; ++u) e[u] = sched[min(g * G + u, steps - 1) * LM + lrow];
    };
    auto load_x = [&](float2 (&x)[G], const uint4 (&e)[G], int g, int k0) {
      const float2* xk = a.X + (int64_t)min(k0 + lcol, N - 1) * a.pitch + f;
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const uint32_t c = has(g * G + u) ? e[u].y & 0xffffu : 0u;   // an idle lane reads channel 0
        x[u] = xk[(int64_t)c * xrow];
      }
    };
    for (int it = itb; it < ite; ++it) {
      const int blk = it / groups, k0 = (it % groups) * C;
      const bool fresh = it == itb || k0 == 0;       // first columns of the unit, or a new trial block
      if (fresh) entries(blk);
      float2 xs[NI];
      if constexpr (NS > 0) {
        if (fresh) {
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            const uint4 e = reinterpret_cast<const uint4*>(reg)[min(i, steps - 1) * LM + lrow];
            ent[i] = make_uint4(e.x, has(i) ? e.y : 0u, e.z, e.w);   // an idle lane reads channel 0
          }
        }
#pragma unroll
        for (int i = 0; i < NS; ++i)
          xs[i] = reg[S::SO + lcol * a.n_chan + (int)(ent[i].y & 0xffffu)];
        wave_order();
      }
      // clear the grid
      {
        float4* z = reinterpret_cast<float4*>(reg);
        constexpr int NZ = (S::RP / 2 + 63) / 64;
#pragma unroll
        for (int i = 0; i < NZ; ++i)
          if (64 * i + lane < S::RP / 2) z[64 * i + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
      wave_order();
      if constexpr (NS == 0) {
        load_e(eb[0], 0);
        load_e(eb[1], 1);
        load_x(xb[0], eb[0], 0, k0);
        load_x(xb[1], eb[1], 1, k0);
        load_e(eb[2], 2);
      }
      {
        float2* const base = reg + lcol * GP;
        float2* const none = reg + C * GP;           // where idle lanes add
        const int mask = (1 << lq) - 1, tmask = (1 << ls) - 1;
        // the entries 2 i and 2 i + 1: channel i of both parts
        auto step = [&](const uint4* e, const float2* x, int i) {
          float w[2][kTaps], xr[2], xi[2];
          float2* pt[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            tap_weights(__uint_as_float(e[h].x), w[h]);
            const float cx = __uint_as_float(e[h].z), cy = __uint_as_float(e[h].w);
            xr[h] = fmaf(cx, x[h].x, -cy * x[h].y);
            xi[h] = fmaf(cx, x[h].y, cy * x[h].x);
            pt[h] = has(2 * i + h) ? base + ((2 * lrow + h) & mask) * (M >> lq) + (e[h].y >> 16) : none;
          }
          auto add = [&](bool both, int h0) {
            float2 t[2][kTaps];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int k = 0; k < kTaps; ++k)
                if (both || h == h0) t[h][k] = pt[h][k];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int k = 0; k < kTaps; ++k)
                if (both || h == h0) pt[h][k] = make_float2(fmaf(w[h][k], xr[h], t[h][k].x), fmaf(w[h][k], xi[h], t[h][k].y));
          };
          if (ls == 0) {
            add(true, 0);
          } else {
            for (int tn = 0; tn <= tmask; ++tn) {
              if ((((2 * lrow) >> lq) & tmask) == tn) add(false, 0);
              wave_order();
              if ((((2 * lrow + 1) >> lq) & tmask) == tn) add(false, 1);
              wave_order();
            }
          }
          wave_order();
        };
        if constexpr (NS > 0) {
#pragma unroll
          for (int g = 0; g < NS / G; ++g) {
            if (g >= n_grp) break;
#pragma unroll
            for (int u = 0; u < G; u += 2) step(ent + g * G + u, xs + g * G + u, (g * G + u) / 2);
          }
        } else {
          for (int g0 = 0; g0 < n_grp; g0 += R) {
#pragma unroll
            for (int p = 0; p < R; ++p) {
              const int g = g0 + p;
              if (g >= n_grp) break;
              load_x(xb[(p + 2) % R], eb[(p + 2) % R], g + 2, k0);
              load_e(eb[(p + 3) % R], g + 3);
#pragma unroll
              for (int u = 0; u < G; u += 2) step(&eb[p][u], &xb[p][u], (g * G + u) / 2);
            }
          }
        }
        if constexpr (NS > 0) {
          const GridUnit nu = grid_unit(work, next >= 0 ? next : unit);   // (the last one loads in vain)
          const bool same = it + 1 < ite;
          load_raw(same ? (it + 1) % groups * C : first_col(nu), same ? f0 : nu.bb * FB);
        }
      }
      wave_order();
      // the guard points are points of the grid's other end
      constexpr int GG = 2 * GL + 8;
      for (int e = lane; e < GG * C; e += 64) {
        const int q = e % GG;                        // the left guard, then the right one
        float2* g = reg + (e / GG) * GP;
        const int from = q < GL ? q : M + q, to = q < GL ? M + q : q;
        if (from < GP) g[to] = f2add(g[to], g[from]);
      }
      wave_order();
      // first pass: lane (column ci, l) transforms the points l + LM a over a
      float2 v[64];
      {
        const float2* g = reg + lcol * GP + GL + lrow;
#pragma unroll
        for (int q = 0; q < 64; ++q) v[q] = g[LM * cx_bitrev(q, 6)];
        // copies: the upper half of the grid joins the lower half, lq times; the 8 points before c0
        // are then the last ones of the copy, and belong at the end of the grid
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
          if (lq == 6 - cx_log2(h)) {
            constexpr int NA = LM < 8 ? 8 / LM : 1;
#pragma unroll
            for (int p = 0; p < NA && p < h; ++p) {
              const int i0 = cx_bitrev(h - 1 - p, 6), i1 = cx_bitrev(63 - p, 6);
              const bool last = lrow + 8 >= LM;
              v[i1] = last ? v[i0] : v[i1];
              v[i0] = last ? make_float2(0.0f, 0.0f) : v[i0];
            }
          }
        }
      }
      dit_stages<64, 1, true>(v);
      wave_order();
#pragma unroll
      for (int k1 = 0; k1 < 64; ++k1) reg[lane * XP + k1] = v[k1];
      wave_order();
      // second pass: lane k1 transforms the LM points of every column (the tables pass as new
      // values, or their products would be kept in registers across the loop)
#pragma unroll
      for (int l = 0; l < TA; ++l) asm volatile("" : "+v"(twa[l].x), "+v"(twa[l].y));
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
          if (l0 != 0) x[q] = cmulf(x[q], twiddle(l0));
          const float2 w1 = twiddle(l1);
          bfly(x[q], x[q + 1], w1.x, w1.y);
        }
        dit_stages<LM, 2, true>(x);
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
      // the next column's values, waited for before this one's stores are issued
      if constexpr (NS > 0) put_raw();
      // hand-over: the bins of each row (what follows from the thread's place is formed here and
      // not held in registers across the transforms; likewise in load_raw).  Rows that are no trial
      // go to a place of the wave's own: were their stores skipped, the count of stores in flight
      // would be unknown and every wait for the next column's values one for all stores.
      int ro = r0, ho = rh;
      asm volatile("" : "+v"(ro), "+v"(ho));
      float4* const dump = a.dump + (int64_t)(blockIdx.x * FB + wave) * 64 + lane;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int ci = (i * RSTEP) / (M / 2);
        const int rb = (i * RSTEP) % (M / 2);        // uniform part of the row
        const int k = k0 + ci;
        const int row = ci * (M / 2) + ((rb + ro) & (M / 2 - 1));
        const int j = ((rb + ro) & (M / 2 - 1)) - M / 4 + jc;   // trial within the block
        const int dm = blk * a.blk + j;
        const bool ok = k < N && j >= 0 && j < a.blk && dm < a.n_dm;
        const float d = dec[i % NDEC];
        if constexpr (POWER) {
          float pw[FB];
#pragma unroll
          for (int w = 0; w < FB; ++w) {
            float2 y = smem[w * S::RP + row];
            y = make_float2(y.x * d, y.y * d);
            if (f0 + w == 0) y.x += a.dc_add;
            pw[w] = fmaf(y.x, y.x, y.y * y.y);
          }
          PowerQuad* const to = reinterpret_cast<PowerQuad*>(a.P + (int64_t)dm * a.n_pow_bins + f0);
          *(ok && f0 < a.n_pow_bins ? to : reinterpret_cast<PowerQuad*>(dump)) = {pw[0], pw[1], pw[2], pw[3]};
        } else {
          const float2 y0 = smem[(2 * ho) * S::RP + row], y1 = smem[(2 * ho + 1) * S::RP + row];
          float4* const to = reinterpret_cast<float4*>(a.Yc + (int64_t)dm * yrow + (int64_t)k * a.pitch + f0 + 2 * ho);
          *(ok ? to : dump) = make_float4(y0.x * d, y0.y * d, y1.x * d, y1.y * d);
        }
      }
      grid_barrier();
    }
  }
}

namespace {
template <int LOGM, int NS, bool POWER>
hipError_t launch_grid_ns(const GridArgs& a, hipStream_t st) {
  constexpr int C = GridShape<LOGM>::C, FB = grid_bins<POWER>();
  constexpr int kBlocks = kGridWaves / FB;           // four waves per CU
  const int n_bb = ((POWER ? a.n_pow_bins : a.n_bins) + FB - 1) / FB;
  const int n_it = ((a.n_chunks + C - 1) / C) * a.n_blk;
  const GridWork w = grid_work(n_bb, n_it, kBlocks);
  const int most = w.main_xcd > w.tail_xcd ? w.main_xcd : w.tail_xcd;
  const int slots = most < kBlocks / kGXcds ? most : kBlocks / kGXcds;
  hipLaunchKernelGGL((k_phasor_grid<LOGM, NS, POWER>), dim3((unsigned)(kGXcds * slots)), dim3(64 * FB), 0, st, a, w);
  return hipGetLastError();
}

template <int LOGM, bool POWER>
hipError_t launch_grid(const GridArgs& a, hipStream_t st) {
  const int bins = POWER ? a.n_pow_bins : a.n_bins;
  hipLaunchKernelGGL((k_grid_order<LOGM>), dim3((unsigned)grid_groups(bins, a.log_gb)), dim3(64), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int steps = grid_steps(a.n_chan, LOGM);
  if (steps <= 8) return launch_grid_ns<LOGM, 8, POWER>(a, st);
  if (steps <= kGridStaged) return launch_grid_ns<LOGM, kGridStaged, POWER>(a, st);
  return launch_grid_ns<LOGM, 0, POWER>(a, st);
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
  if (a.log_m < kGridLogMin || a.log_m > kGridLogMax || a.X == nullptr || a.ctab == nullptr || a.dec == nullptr ||
      a.perm == nullptr || a.places == nullptr || a.turns == nullptr || a.dump == nullptr ||
      (a.sched == nullptr && grid_steps(a.n_chan, a.log_m) > kGridStaged) || a.sched_len < grid_sched_len(a.n_chan) ||
      a.window < 2 || (a.Yc == nullptr) == (a.P == nullptr) || a.n_dm < 1 || a.n_chan < 1 || a.n_chan > 65535 ||
      a.n_chunks < 1 || a.blk < 1 || 2 * a.blk > (1 << a.log_m) || (int64_t)a.n_blk * a.blk < a.n_dm ||
      (a.n_blk > 1 && a.log_m != 12) || (a.P != nullptr && (a.n_chunks != 1 || a.log_m != 12)) ||
      grid_groups(a.P != nullptr ? a.n_pow_bins : a.n_bins, a.log_gb) > a.n_groups)
    return hipErrorInvalidValue;
  return launch_grid_m(a, st);
}

// Row divisors 1 / phihat((idx - M/4) / M), idx < M/2, phihat the Fourier transform of the
// piecewise polynomial phi (8-point Gauss-Legendre per piece: exact for degree 7 times the
// cosine's expansion to well below float64 rounding of the result at |k| <= M/4).
static std::vector<float> make_divisors(int log_m) {
  static const double kX[8] = {0.0950125098376374, 0.2816035507792589, 0.4580167776572274, 0.6178762444026438,
                               0.7554044083550030, 0.8656312023878318, 0.9445750230732326, 0.9894009349916499};
  static const double kW[8] = {0.1894506104550685, 0.1826034150449236, 0.1691565193950025, 0.1495959888165767,
                               0.1246289712555339, 0.0951585116824928, 0.0622535239386479, 0.0271524594117541};
  const TapTable t{};
  const int half = 1 << (log_m - 1);
  std::vector<float> out((size_t)half);
  for (int idx = half / 2; idx <= half; ++idx) {      // even in idx - half / 2
    const double om = 2.0 * 3.14159265358979323846 * (double)(idx - half / 2) / (double)(2 * half);
    double sum = 0.0;
    for (int i = 0; i < 4; ++i)
      for (int q = 0; q < 16; ++q) {
        const double r = 0.5 * (q < 8 ? kX[q] : -kX[q - 8]), wt = 0.5 * kW[q & 7];
        double p = 0.0;
        for (int d = 7; d >= 0; --d) p = p * r + (double)t.c[i][d];
        sum += 2.0 * wt * p * std::cos(om * ((double)i - 3.5 - r));   // taps i and 7 - i
      }
    if (idx < half) out[(size_t)idx] = (float)(1.0 / sum);
    out[(size_t)(half - idx)] = (float)(1.0 / sum);
  }
  return out;
}

// They depend on the grid alone and take 64 cosines each (half of them): made once per process and size.
const std::vector<float>& grid_divisors(int log_m) {
  static std::once_flag made[kGridLogMax - kGridLogMin + 1];
  static std::vector<float> tab[kGridLogMax - kGridLogMin + 1];
  const int i = log_m - kGridLogMin;
  std::call_once(made[i], [&] { tab[i] = make_divisors(log_m); });
  return tab[i];
}

}  // namespace fdd
