// Phasor sum on the vector ALUs (Eqs. 4 and 7), any number of chunks, FP32.
//
//     Y[dm, k, f] = sum_c X[c, k, f] * exp(+2 pi i f tau[dm, c] / L)
//
// For one spin-frequency bin this is a matrix-vector product per chunk (Sec. 2.3); with a
// single chunk nothing is shared along the chunk axis, so this kernel is the path for the
// single-transform workloads whose delays do not factorise or whose trials are few, and the
// fallback for any shape.
//
// A workgroup owns 4 DMs and 64 FV bins, and its 4 waves share the channels; at the end wave i
// collects DM i through LDS.  Lanes hold neighbouring bins, so X is read and Y written in whole
// lines, and each value read serves 4 DMs.  Per channel and DM a lane evaluates the phasor of its
// first bin from the exact 64-bit increment and multiplies it by those of 64, 128 .. 448 bins, which 8
// lanes evaluate for all; past 8 bins it evaluates again.  Small problems take fewer bins per lane and
// more workgroups, with the same steps to every bin: a result does not depend on FV.
// Bound: instruction issue, 8 operations per channel, bin and DM, and 4 or more for the
// phasors.
//   128 channels, 2048 DMs, one chunk of 65536 samples, rounded delays:  24.4 -> 2.95 ms (it
//   was one DM per thread with 16 neighbouring bins, 128 bytes apart between lanes);
//   64 channels, 64 equally spaced DMs, one chunk of 4096 samples:  37.8 (64 rows of 32 DMs on the
//   matrix cores, of which 2 were in use) -> 22 us; reading the next
//   channel ahead changes nothing.
// Phasors formed step by step by each lane, instead of those of 64 i bins once for all, make the
// large problem 11 % faster (2.64 ms) and the small one 50 % slower (32.7 us).
//
// With P set, the epilogue writes power spectra |Y|^2 for bins below L/2 (Sec. 5) instead of
// the complex result.
#include "device_math.h"
#include "fdd_internal.h"

namespace fdd {

namespace {
constexpr int kDms = 4;           // DMs, and waves, of a workgroup
constexpr int kSeed = 8;          // bins (64 apart) from one evaluated phasor

template <int FV, int NK>
struct ValuLds {
  static constexpr int floats = (kDms - 1) * 2 * NK * FV * 64;
};
}  // namespace

// FV bins of a lane, NK chunks.  FAC: the increments are sums of a coarse and a fine entry (uniform DM
// grids, a.vtab) instead of entries of the (channel, DM) table.
template <int FV, int NK, bool FAC>
__device__ __forceinline__ void phasor_valu_body(const PhasorArgs& a, const int bx, const int by, const int bz) {
  __shared__ float red[ValuLds<FV, NK>::floats];
  const int lane = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int f0 = bx * 64 * FV + lane;
  const int dm0 = by * kDms;
  const int k0 = bz * NK;
  float2 acc[kDms][NK][FV];
#pragma unroll
  for (int d = 0; d < kDms; ++d)
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int i = 0; i < FV; ++i) acc[d][k][i] = make_float2(0.0f, 0.0f);
  // table columns of this lane's DM (a clamped one's results are not stored)
  const int own = min(dm0 + lane / kSeed % kDms, a.n_dm - 1);
  const int ia = FAC ? own / a.n_fine : own, ib = FAC ? own % a.n_fine : 0;
  const int r0 = bx * FV % kSeed;
  const int na = FAC ? a.n_coarse : a.n_dm;
  int at[FV];
#pragma unroll
  for (int i = 0; i < FV; ++i) at[i] = min(f0 + 64 * i, a.n_bins - 1);
  for (int c = wave; c < a.n_chan; c += kDms) {
    const float2* xr = a.X + (int64_t)c * a.n_chunks * a.pitch;
    float2 x[NK][FV];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const float2* xk = xr + (int64_t)min(k0 + k, a.n_chunks - 1) * a.pitch;
#pragma unroll
      for (int i = 0; i < FV; ++i) x[k][i] = xk[at[i]];
    }
    // lane 8 d + i has the increment of DM d and the phasor of 64 i bins
    uint64_t inc;
    {
      const uint4 e = a.ptab[(int64_t)c * na + ia];
      inc = ((uint64_t)e.y << 32) | e.x;
      if constexpr (FAC) {
        const uint4 v = a.vtab[(int64_t)c * a.n_fine + ib];
        inc += ((uint64_t)v.y << 32) | v.x;
      }
    }
    const int hi = (int)(inc >> 32), lo = (int)(uint32_t)inc;
    float2 far;
    sincos_turn(phase_at(PhaseInc{(uint32_t)hi, (uint32_t)lo}, 64u * (uint32_t)(lane % kSeed)), &far.y, &far.x);
#pragma unroll
    for (int d = 0; d < kDms; ++d) {
      const PhaseInc pi = {(uint32_t)__builtin_amdgcn_readlane(hi, kSeed * d), (uint32_t)__builtin_amdgcn_readlane(lo, kSeed * d)};
      float2 w0;
#pragma unroll
      for (int i = 0; i < FV; ++i) {
        if (i % kSeed == 0) sincos_turn(phase_at(pi, (uint32_t)(f0 - 64 * r0 + 64 * i)), &w0.y, &w0.x);
        float2 w = w0;
        if (FV < kSeed || i % kSeed != 0) {
          const int from = kSeed * d + r0 + i % kSeed;
          w = cmul(w0, make_float2(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(far.x), from)),
                                   __int_as_float(__builtin_amdgcn_readlane(__float_as_int(far.y), from))));
        }
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          acc[d][k][i].x = fmaf(w.x, x[k][i].x, fmaf(-w.y, x[k][i].y, acc[d][k][i].x));
          acc[d][k][i].y = fmaf(w.x, x[k][i].y, fmaf(w.y, x[k][i].x, acc[d][k][i].y));
        }
      }
    }
  }
  // wave d sums the waves' parts of DM d, in the order of the waves after its own
#pragma unroll
  for (int d = 0; d < kDms; ++d) {
    if (wave != d) {
      float* to = red + ((wave - d + kDms) % kDms - 1) * (2 * NK * FV * 64) + lane;
#pragma unroll
      for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int i = 0; i < FV; ++i) {
          to[(2 * (k * FV + i)) * 64] = acc[d][k][i].x;
          to[(2 * (k * FV + i) + 1) * 64] = acc[d][k][i].y;
        }
    }
    __syncthreads();
    if (wave == d) {
      const float* from = red + lane;
#pragma unroll
      for (int o = 0; o < kDms - 1; ++o)
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
          for (int i = 0; i < FV; ++i) {
            acc[d][k][i].x += from[(o * 2 * NK * FV + 2 * (k * FV + i)) * 64];
            acc[d][k][i].y += from[(o * 2 * NK * FV + 2 * (k * FV + i) + 1) * 64];
          }
      const int dm = dm0 + d;
      if (dm < a.n_dm) {
        if (a.P != nullptr) {
          if (f0 == 0) acc[d][0][0].x += a.dc_add;
#pragma unroll
          for (int i = 0; i < FV; ++i) {
            const int f = f0 + 64 * i;
            if (f < a.n_bins && f < a.n_pow_bins)
              a.P[(int64_t)dm * a.n_pow_bins + f] = fmaf(acc[d][0][i].x, acc[d][0][i].x, acc[d][0][i].y * acc[d][0][i].y);
          }
        } else {
#pragma unroll
          for (int k = 0; k < NK; ++k) {
            if (k0 + k >= a.n_chunks) continue;
            const int64_t row = ((int64_t)dm * a.n_chunks + k0 + k) * a.pitch;
#pragma unroll
            for (int i = 0; i < FV; ++i) {
              const int f = f0 + 64 * i;
              if (f < a.n_bins) {
                a.Yr[row + f] = acc[d][k][i].x;
                a.Yi[row + f] = acc[d][k][i].y;
              }
            }
          }
        }
      }
    }
    if (d + 1 < kDms) __syncthreads();
  }
}

template <int FV, int NK, bool FAC>
__global__ __launch_bounds__(64 * kDms, 2) void k_phasor_valu(PhasorArgs a) {
  phasor_valu_body<FV, NK, FAC>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Batched form: tile t of beam b is block (t mod n_bb, (t / n_bb) mod n_dmt, t / (n_bb n_dmt))
// of that beam's own launch.
template <int FV, int NK, bool FAC>
__global__ __launch_bounds__(64 * kDms, 2) void k_phasor_valu_grouped(Group<PhasorArgs> g) {
  const int t = blockIdx.y * gridDim.x + blockIdx.x;
  if (t >= g.total) return;
  const int b = group_beam(g.prefix, g.n_beams, t);
  const PhasorArgs& a = g.beams[b];
  const int lt = t - g.prefix[b];
  phasor_valu_body<FV, NK, FAC>(a, lt % a.n_bb, (lt / a.n_bb) % a.n_dmt, lt / (a.n_bb * a.n_dmt));
}

namespace {
constexpr int kAcc = 16;          // NK FV: bins of a lane times chunks

template <int FV, int NK>
hipError_t launch_valu(const PhasorArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((a.n_bins + 64 * FV - 1) / (64 * FV)), (unsigned)((a.n_dm + kDms - 1) / kDms),
                  (unsigned)((a.n_chunks + NK - 1) / NK)), block(64 * kDms);
  if (a.vtab != nullptr) hipLaunchKernelGGL((k_phasor_valu<FV, NK, true>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_phasor_valu<FV, NK, false>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <int NK>
hipError_t launch_valu_nk(const PhasorArgs& a, hipStream_t st) {
  const int fv = phasor_valu_bins(a.n_bins, a.n_dm, a.n_chunks);
  if (fv == kAcc / NK) return launch_valu<kAcc / NK, NK>(a, st);
  if (NK == 1 && fv == 4) return launch_valu<4, NK>(a, st);
  return launch_valu<1, NK>(a, st);
}
}  // namespace

int phasor_valu_chunks(int n_chunks) { return n_chunks <= 2 ? n_chunks : 4; }

// The most bins per lane that leave 512 workgroups, two per CU.
int phasor_valu_bins(int n_bins, int n_dm, int n_chunks) {
  const int nk = phasor_valu_chunks(n_chunks);
  const int64_t rows = (int64_t)((n_dm + kDms - 1) / kDms) * ((n_chunks + nk - 1) / nk);
  const auto blocks = [&](int fv) { return rows * ((n_bins + 64 * fv - 1) / (64 * fv)); };
  return blocks(kAcc / nk) >= 512 ? kAcc / nk : nk == 1 && blocks(4) >= 512 ? 4 : 1;
}

int64_t phasor_valu_tiles(PhasorArgs* a, int nk) {
  const int bins = 64 * kAcc / nk;
  a->n_bb = (a->n_bins + bins - 1) / bins;
  a->n_dmt = (a->n_dm + kDms - 1) / kDms;
  return (int64_t)a->n_bb * a->n_dmt * ((a->n_chunks + nk - 1) / nk);
}

hipError_t launch_phasor_valu_grouped(int nk, bool fac, const Group<PhasorArgs>& g, hipStream_t st) {
  if (g.total <= 0) return hipSuccess;
  if (nk != 1 && nk != 4) return hipErrorInvalidValue;
  const dim3 grid = linear_grid(g.total), block(64 * kDms);
  if (nk == 1 && fac) hipLaunchKernelGGL((k_phasor_valu_grouped<kAcc, 1, true>), grid, block, 0, st, g);
  else if (nk == 1) hipLaunchKernelGGL((k_phasor_valu_grouped<kAcc, 1, false>), grid, block, 0, st, g);
  else if (fac) hipLaunchKernelGGL((k_phasor_valu_grouped<kAcc / 4, 4, true>), grid, block, 0, st, g);
  else hipLaunchKernelGGL((k_phasor_valu_grouped<kAcc / 4, 4, false>), grid, block, 0, st, g);
  return hipGetLastError();
}

hipError_t launch_phasor_valu(const PhasorArgs& a, hipStream_t st) {
  if (a.P != nullptr && a.n_chunks != 1) return hipErrorInvalidValue;
  if (a.n_chunks == 1) return launch_valu_nk<1>(a, st);
  if (a.n_chunks == 2) return launch_valu_nk<2>(a, st);
  return launch_valu_nk<4>(a, st);
}

}  // namespace fdd
