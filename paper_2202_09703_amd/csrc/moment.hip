// The moment form of the factored operator A = C o S (see operator.hip for
// the factoring): the same operator with the fine grid's Q positions per
// sample carried as R moments per sample.
//
// Over one sample period the tabulated pulse is very smooth (its band is far
// below the sampling rate), so for every tap k the Q + 1 table values
// b[(k + 1) Q - t], t = 0 .. Q, are a polynomial of degree R - 1 in
// z = 2 t / Q - 1 to far below FP32 rounding (build_moments bounds the
// remainder by 1e-8 of the pulse's peak: R = 5 at 20 MHz, 6 at 10 MHz for a
// 500 kHz pulse):
//     b[(k + 1) Q - t] = sum_{p < R} G_p[k] z^p.
// A voxel whose echo starts at fine position n Q + t + phi in sample n, with
// weight W, then contributes
//     y[n + 1 + k] += W x sum_p G_p[k] a_p,   a_p = (1 - phi) z_t^p + phi z_{t+1}^p,
// exactly the linear interpolation of the table that operator.hip states.  So
//   S: u_p[n] = sum over the trace's voxels of sample n of W x a_p;
//   C: y[m] = sum_p sum_n u_p[n] G_p[m - 1 - n];
//   C^T: v_p[n] = sum_m r[m] G_p[m - 1 - n];
//   S^T: sum over the traces of W sum_p a_p v_p[n].
// Against the fine grid this cuts the dense products and the traffic between
// the sparse and the dense part by Q / R (6.4 at Q = 32).
//
// Arrays u and v are [trace][R][Ms] floats, Ms = M rounded up to 32, whatever
// the storage type of the traces.
//
// The splat also uses that the medium is layered: when the scan positions are
// a constant whole number of voxels apart, the delay and weight of (scan i,
// receiver j, row, column c) depend on (j, row, c - pitch i) only.  A record
// per (j, row, relative column) holds n, a_0 .. a_{R-1} (times the weight);
// the records of each j are sorted by n once per geometry, and u of one (j, n)
// for all scan positions is then a sum over its records of coefficients times
// consecutive elements of the image (stored by phase of the pitch), in
// registers: no atomics, and a fixed order of the sums.
//
// With attenuation every pair belongs to one of NG templates; a forward or an
// adjoint alone runs with u and v per template (R = 8: six moments and the two
// ends of the window, see k_template_fit), the records sorted by (template,
// sample).  |A| has tables of its own where |b| is b or -b over every cell.
// Grouped ICD's large groups use C and C^T as they are, with a splat and a
// gather over the group's members.

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "storage.h"

namespace umbir {
namespace {

constexpr int kBufferWord3 = 0x00020000;  // word 3 of a raw buffer resource: 32-bit data, no swizzle

typedef float floatx4 __attribute__((ext_vector_type(4)));

// ---- the plan (once per geometry)

// The two legs of (receiver j, row, relative column) at scan position 0.
struct PairLegs {
  uint64_t D;  // Q32.32 samples
  float w;     // product of the apodisations
};

__device__ __forceinline__ PairLegs pair_legs(const Leg* __restrict__ legs, int n_off, int bt, int br, int row,
                                              int rel) {
  const int half = n_off / 2;
  const Leg a = legs[size_t(row) * n_off + leg_slot(abs(bt + 2 * rel), half)];
  const Leg b = legs[size_t(row) * n_off + leg_slot(abs(br + 2 * rel), half)];
  return {uint64_t(a.delay + b.delay), a.apod * b.apod};
}

// Its attenuation template.
__device__ __forceinline__ int pair_template(const double* __restrict__ gunit, int n_off, int bt, int br, int row,
                                             int rel, int glast) {
  if (!gunit) return 0;
  const int half = n_off / 2;
  const double* u = gunit + size_t(row) * n_off;
  return gamma_bin(u[leg_slot(abs(bt + 2 * rel), half)] + u[leg_slot(abs(br + 2 * rel), half)], glast);
}

// The bin of a pair: its sample, after the bins of the templates before its
// own; NG M past the record.
__device__ __forceinline__ int plan_bin(const PairLegs& p, const double* __restrict__ gunit, const MomentShape& ms,
                                        int n_off, int bt, int br, int row, int rel, int M) {
  const uint64_t n = p.D >> 32;
  if (n >= uint64_t(M)) return ms.NG * M;
  return pair_template(gunit, n_off, bt, br, row, rel, ms.NG - 1) * M + int(n);
}

// Lattice bases of scan lane 0 (the leftmost position) for receiver j.
__device__ __forceinline__ void plan_bases(const int* __restrict__ base, const MomentShape& ms, int P, int K, int j,
                                           int* bt, int* br) {
  const int i = ms.reversed ? P - 1 : 0;
  *bt = base[i];
  *br = base[P + i * K + j];
}

// Relative columns per plan block: one histogram of samples per (j, chunk).
constexpr int kPlanChunk = 64;

// Bins a plan block holds in LDS at a time; a block takes slice blockIdx.z.
constexpr int kPlanSlice = 36864;

// Bytes of the histograms: as many receivers at a time as fit, with one launch
// of each of the three kernels per such part (one part up to 64 receivers, 16
// chunks and 16384 bins).
constexpr size_t kPlanCountBytes = size_t(256) << 20;

// counts[j - j0][chunk][b]: records of receiver j and the chunk's relative
// columns in bin b (of NB = NG M); j0: the part's first receiver.
__global__ __launch_bounds__(1024) void k_plan_count(const Leg* __restrict__ legs, const double* __restrict__ gunit,
                                                    const int* __restrict__ base, MomentShape ms, int P, int K, int j0,
                                                    int nz, int n_off, int M, int* __restrict__ counts) {
  extern __shared__ int hist[];
  const int j = j0 + blockIdx.x, ch = blockIdx.y, NB = ms.NG * M;
  const int b0 = blockIdx.z * kPlanSlice, nb = min(NB - b0, kPlanSlice);
  for (int i = threadIdx.x; i < nb; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  int bt, br;
  plan_bases(base, ms, P, K, j, &bt, &br);
  const int r0 = ch * kPlanChunk, rn = min(kPlanChunk, ms.NR - r0);
  for (int i = threadIdx.x; i < nz * kPlanChunk; i += blockDim.x) {
    const int row = i / kPlanChunk, rc = i - row * kPlanChunk;
    if (rc >= rn) continue;
    const PairLegs p = pair_legs(legs, n_off, bt, br, row, ms.rel0 + r0 + rc);
    const int b = plan_bin(p, gunit, ms, n_off, bt, br, row, ms.rel0 + r0 + rc, M);
    if (b >= b0 && b < b0 + nb) atomicAdd(&hist[b - b0], 1);
  }
  __syncthreads();
  int* out = counts + (size_t(blockIdx.x) * gridDim.y + ch) * NB + b0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) out[i] = hist[i];
}

// Per receiver: start[j][n] (the first record of bin n of M, start[j][M] the
// end) and, in place of each count, the first record of (chunk, n).  Records
// of receiver j begin at j * cap.  max_bin receives the largest bin.
__global__ __launch_bounds__(1024) void k_plan_scan(int M, int chunks, int cap, int j0, int* __restrict__ counts,
                                                    int* __restrict__ start, int* __restrict__ max_bin) {
  __shared__ int waves[16];
  const int j = j0 + blockIdx.x, t = threadIdx.x, lane = t & 63;
  int* cj = counts + size_t(blockIdx.x) * chunks * M;
  int at = j * cap, big = 0;
  for (int n0 = 0; n0 < M; n0 += 1024) {  // 1024 bins at a time, neighbours in neighbouring threads
    const int n = n0 + t;
    int c = 0;
    if (n < M)
      for (int k0 = 0; k0 < chunks; k0 += 8) {
        int v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = cj[size_t(min(k0 + k, chunks - 1)) * M + n];
#pragma unroll
        for (int k = 0; k < 8; ++k) c += k0 + k < chunks ? v[k] : 0;
      }
    big = max(big, c);
    int before = c;  // inclusive over the wave, then exclusive over the block
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(before, off, 64);
      if (lane >= off) before += v;
    }
    if (lane == 63) waves[t >> 6] = before;
    __syncthreads();
    before -= c;
    int total = 0;
    for (int w = 0; w < 16; ++w) {
      if (w < t >> 6) before += waves[w];
      total += waves[w];
    }
    __syncthreads();
    if (n < M) {
      int p = at + before;
      start[size_t(j) * (M + 1) + n] = p;
      for (int k0 = 0; k0 < chunks; k0 += 8) {
        int v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = cj[size_t(min(k0 + k, chunks - 1)) * M + n];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (k0 + k >= chunks) break;
          cj[size_t(k0 + k) * M + n] = p;
          p += v[k];
        }
      }
    }
    at += total;
  }
  if (t == 0) start[size_t(j) * (M + 1) + M] = at;
  if (big > 0) atomicMax(max_bin, big);
}

// Keys row * NR + (rel - rel0) of every record into its bin, in any order.
__global__ __launch_bounds__(1024) void k_plan_fill(const Leg* __restrict__ legs, const double* __restrict__ gunit,
                                                   const int* __restrict__ base, MomentShape ms, int P, int K, int j0,
                                                   int nz, int n_off, int M, const int* __restrict__ first,
                                                   unsigned* __restrict__ keys) {
  extern __shared__ int cursor[];
  const int j = j0 + blockIdx.x, ch = blockIdx.y, NB = ms.NG * M;
  const int b0 = blockIdx.z * kPlanSlice, nb = min(NB - b0, kPlanSlice);
  const int* f = first + (size_t(blockIdx.x) * gridDim.y + ch) * NB + b0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) cursor[i] = f[i];
  __syncthreads();
  int bt, br;
  plan_bases(base, ms, P, K, j, &bt, &br);
  const int r0 = ch * kPlanChunk, rn = min(kPlanChunk, ms.NR - r0);
  for (int i = threadIdx.x; i < nz * kPlanChunk; i += blockDim.x) {
    const int row = i / kPlanChunk, rc = i - row * kPlanChunk;
    if (rc >= rn) continue;
    const PairLegs p = pair_legs(legs, n_off, bt, br, row, ms.rel0 + r0 + rc);
    const int b = plan_bin(p, gunit, ms, n_off, bt, br, row, ms.rel0 + r0 + rc, M);
    if (b >= b0 && b < b0 + nb)
      keys[atomicAdd(&cursor[b - b0], 1)] = unsigned(row) * unsigned(ms.NR) + unsigned(r0 + rc);
  }
}

// A bin larger than this would take its wave too long to order (only voxels
// far smaller than a sample period reach it): such a geometry keeps the fine
// grid (the host reads max_bin after the build).
constexpr int kMaxBin = 8192;

// span[g]: the first sample with a record of template g in any receiver, and
// the one past the last ({0, 0}: none).  One block per template.
__global__ __launch_bounds__(256) void k_plan_span(const int* __restrict__ start, int K, int M, int NB,
                                                   int2* __restrict__ span) {
  __shared__ int lo, hi;
  const int g = blockIdx.x;
  if (threadIdx.x == 0) {
    lo = M;
    hi = 0;
  }
  __syncthreads();
  for (int n = threadIdx.x; n < M; n += blockDim.x) {
    bool any = false;
    for (int j = 0; j < K; ++j) {
      const int* s = start + size_t(j) * (NB + 1) + g * M + n;
      any = any || s[1] > s[0];
    }
    if (any) {
      atomicMin(&lo, n);
      atomicMax(&hi, n + 1);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) span[g] = hi > 0 ? make_int2(lo, hi) : make_int2(0, 0);
}

// One wave per (j, n): the bin's keys put in ascending order by counting the
// smaller ones, and the records written in that order: coefficients
// tau a_tx a_rx ((1 - phi) z_t^p + phi z_{t+1}^p) in double, rounded once, and
// the byte offset of the voxel in the phase-major image (lane i of the splat
// adds its scan position) in the word after them.  With attenuation (R = 8) the
// last two coefficients are the weights the pair puts on the table's first and
// last point (see k_moment_fit).
template <int R>
__global__ __launch_bounds__(256) void k_plan_emit(const Leg* __restrict__ legs, const int* __restrict__ base,
                                                   const float* __restrict__ tau, MomentShape ms, int P, int K,
                                                   int n_off, int qs, int M, const int* __restrict__ start,
                                                   const unsigned* __restrict__ keys,
                                                   const int* __restrict__ max_bin, float4* __restrict__ rec4,
                                                   float* __restrict__ rec_hi) {
  if (*max_bin > kMaxBin) return;
  const int j = blockIdx.x;
  const int n = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (n >= M) return;
  const int lane = threadIdx.x & 63;
  const int s = start[size_t(j) * (M + 1) + n], e = start[size_t(j) * (M + 1) + n + 1];
  int bt, br;
  plan_bases(base, ms, P, K, j, &bt, &br);
  for (int i0 = s; i0 < e; i0 += 64) {
    const unsigned key = i0 + lane < e ? keys[i0 + lane] : 0xffffffffu;
    int rank = 0;
    for (int k0 = s; k0 < e; k0 += 64) {  // past the end: no key is smaller than it
      const unsigned other = k0 + lane < e ? keys[k0 + lane] : 0xffffffffu;
#pragma unroll
      for (int k = 0; k < 64; ++k) rank += unsigned(__builtin_amdgcn_readlane(int(other), k)) < key ? 1 : 0;
    }
    if (i0 + lane >= e) continue;
    const int at = s + rank;
    const int row = int(key / unsigned(ms.NR)), rel = ms.rel0 + int(key - unsigned(row) * unsigned(ms.NR));
    const PairLegs p = pair_legs(legs, n_off, bt, br, row, rel);
    const unsigned frac = unsigned(p.D);
    const double t = double(frac >> (32 - qs));
    const double phi = double(unsigned(frac << qs)) * (1.0 / 4294967296.0);
    const double h = 2.0 / double(1 << qs);
    const double z0 = t * h - 1.0, z1 = (t + 1.0) * h - 1.0;
    const double w = double(tau[row]) * double(p.w);
    double p0 = w * (1.0 - phi), p1 = w * phi;
    float a[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      a[q] = float(p0 + p1);
      p0 *= z0;
      p1 *= z1;
    }
    if (R == 8 && ms.NG > 1) {
      const int ti = int(frac >> (32 - qs));
      a[R - 2] = ti == (1 << qs) - 1 ? float(w * phi) : 0.0f;
      a[R - 1] = ti == 0 ? float(w * (1.0 - phi)) : 0.0f;
    }
    rec4[at] = make_float4(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int q = 4; q < R; ++q) rec_hi[size_t(at) * (R - 3) + (q - 4)] = a[q];
    int rq = rel >= 0 ? rel / ms.pitch : -((-rel + ms.pitch - 1) / ms.pitch);  // floor
    const int phase = rel - rq * ms.pitch;
    rec_hi[size_t(at) * (R - 3) + (R - 4)] = __uint_as_float(unsigned((row * ms.pitch + phase) * ms.Lq + rq + P - 1) * 4u);
  }
}

// G_p[k] = sum_t fit[p][t] b[(k + 1) Q - t] (fit: least squares on the Q + 1
// points, R x (Q + 1) doubles), b evaluated in double.  One wave per k.
// absolute: then the same for |b|, which is b or -b over a whole cell (the pulse
// changes sign on the samples only).
__global__ __launch_bounds__(256) void k_moment_fit(int R, int Q, int Lh, double dt, double f_c, double inv2s2,
                                                    double t_c, const double* __restrict__ fit, int absolute,
                                                    float* __restrict__ g) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (k >= Lh) return;
  const int QLh = Q * Lh;
  double acc[8] = {};
  for (int t = lane; t <= Q; t += 64) {
    const int n = (k + 1) * Q - t;
    const double x = n * dt - t_c;
    const double b = n <= 0 || n >= QLh ? 0.0 : sin(2.0 * M_PI * f_c * x) * exp(-x * x * inv2s2);
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p < R) acc[p] += fit[p * (Q + 1) + t] * b;
  }
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    for (int off = 32; off > 0; off >>= 1) acc[p] += __shfl_xor(acc[p], off, 64);
    if (lane == 0 && p < R) {
      g[p * Lh + k] = float(acc[p]);
      if (absolute) {
        const bool neg = sin(2.0 * M_PI * f_c * ((k + 0.5) * Q * dt - t_c)) < 0.0;
        g[(R + p) * Lh + k] = float(neg ? -acc[p] : acc[p]);
      }
    }
  }
}

// The same for the attenuated templates: six coefficients per template and
// window cell from its row of the bank, and a seventh and eighth function.  The
// rows are forced to zero at their ends, where an attenuated response is not:
// the fits of the first and the last cell leave that point out (fit: the three
// matrices without none, the last and the first of the Q + 1 points), and the
// weight a pair puts on it takes the fit's value there away again.
__global__ __launch_bounds__(256) void k_template_fit(int Q, int Lh, const float* __restrict__ bank,
                                                      const double* __restrict__ fit, float* __restrict__ g_all) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (k >= Lh) return;
  const float* b = bank + size_t(blockIdx.y) * (Q * Lh + 2);
  float* g = g_all + size_t(blockIdx.y) * 8 * Lh;
  const double* f = fit + (k == 0 ? 1 : k == Lh - 1 ? 2 : 0) * 6 * (Q + 1);
  double acc[6] = {};
  for (int t = lane; t <= Q; t += 64) {
    const double v = double(b[(k + 1) * Q - t]);
#pragma unroll
    for (int p = 0; p < 6; ++p) acc[p] += f[p * (Q + 1) + t] * v;
  }
  double at_one = 0.0, at_minus = 0.0;  // the fit at t = Q and t = 0
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    for (int off = 32; off > 0; off >>= 1) acc[p] += __shfl_xor(acc[p], off, 64);
    at_one += acc[p];
    at_minus += p & 1 ? -acc[p] : acc[p];
    if (lane == 0) g[p * Lh + k] = float(acc[p]);
  }
  if (lane == 0) {
    g[6 * Lh + k] = k == 0 ? float(-at_one) : 0.0f;
    g[7 * Lh + k] = k == Lh - 1 ? float(-at_minus) : 0.0f;
  }
}

// The dense kernels' operand table F[p][piece][D + 1], D = -1 .. Lh + 7: the 8
// values G_p[D], G_p[D - 1], ..., G_p[D - 7] (zero outside [0, Lh)) split into
// three bf16 pieces.
__global__ __launch_bounds__(256) void k_moment_table(int R, int Lh, int LT, const float* __restrict__ g,
                                                      uint4* __restrict__ F, int* __restrict__ max_bin) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *max_bin = 0;  // for k_plan_scan
  if (i >= R * LT) return;
  const int p = i / LT, D = i - p * LT - 1;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = D - e >= 0 && D - e < Lh ? g[p * Lh + D - e] : 0.0f;
  const Pieces8 pc = split8_bf16x3(make_float4(v[0], v[1], v[2], v[3]), make_float4(v[4], v[5], v[6], v[7]));
#pragma unroll
  for (int q = 0; q < 3; ++q) F[(size_t(p) * 3 + q) * LT + D + 1] = pc.p[q];
}

// ---- the image by phase of the pitch: xp[row][phase][q + P - 1], column
// c = phase + pitch q, zero where c lies outside the grid (x NULL: ones).

__global__ void k_phase_image(const float* __restrict__ x, int nx, int nz, int P, MomentShape ms,
                              float* __restrict__ xp) {
  const int n = nz * ms.pitch * ms.Lq;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int rp = i / ms.Lq, q = i - rp * ms.Lq - (P - 1);
    const int row = rp / ms.pitch, c = rp - row * ms.pitch + ms.pitch * q;
    xp[i] = c >= 0 && c < nx ? (x ? x[row * nx + c] : 1.0f) : 0.0f;
  }
}

// ---- S

// u of receiver bx, samples BINS by .. BINS by + BINS - 1, scan lanes 64 bz ...: a
// wave takes BINS / 4 consecutive samples, 64 records of one at a time: loaded one per
// lane (the next 64 are in flight meanwhile), parked in the wave's own LDS,
// then multiplied G = 64 / S records a step (S lanes, a power of two >= 4, per
// record: one scan position each) on the matrix cores, v_mfma_f32_4x4x1: lane l
// holds coefficient l % 4 of its record (A) and the image element of its scan
// position (B), and the four results of a lane are its moments 0 .. 3; higher
// moments take an FMA each, or a second product.  Records past a sample's end
// have coefficients zero, so steps need no masks and eight image loads are in
// flight together.  Runs of 64 records sum in FP32, the runs in FP64.
//
// The splat this replaces (64-bit LDS atomics on the fine grid) was bound by
// address processing at 118 clocks per 64 (trace, voxel) pairs and CU.  A step
// here costs one coalesced image load (L1), two LDS reads and about five
// vector instructions.
constexpr int kMsWaves = 4;
constexpr int kMsBins = 16;  // samples per block of a full grid: a wave's four follow one another
// With few blocks a wave takes one sample, four times the blocks: the chain of
// record and image loads of one sample, not four, is what a small call waits
// for (8 receivers, 256 samples, 64 x 64 voxels, 128 blocks of 16: 6.2 against
// 9.3 us between events around the launch).  From two blocks of 16 per CU on the longer runs of stores win.
constexpr int kMsBinsFew = 4;
int msplat_bins(long blocks16) { return blocks16 < 512 ? kMsBinsFew : kMsBins; }

// LDS words of a parked record: R coefficients, the offset, padding
template <int R>
__host__ __device__ constexpr int msplat_rec_words() { return R < 8 ? 8 : 12; }

template <int R, int LS>
__device__ __forceinline__ void msplat_steps(const float* recs, int lane, unsigned xl4, __amdgpu_buffer_rsrc_t xrs,
                                             int steps, floatx4& d, float (&dh)[4]) {
  constexpr int W = msplat_rec_words<R>();
  constexpr int G = 64 >> LS;
  constexpr int U = 64 / G < 8 ? 64 / G : 8;  // 64 / G is a multiple of U
  const float* mine = recs + (lane >> LS) * W;
  for (int k0 = 0; k0 < steps; k0 += U) {
    const float* r = mine + k0 * G * W;
    float xv[U], a[U], hi[U][R - 4];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const float* rq = r + q * G * W;
      a[q] = rq[lane & 3];
      if constexpr (R < 8) {
#pragma unroll
        for (int w = 0; w < R - 4; ++w) hi[q][w] = rq[4 + w];
      } else {
        hi[q][0] = rq[4 + (lane & 3)];
      }
      xv[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                            xrs, int(__float_as_uint(rq[R]) + xl4), 0, 0));
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      d = __builtin_amdgcn_mfma_f32_4x4x1f32(a[q], xv[q], d, 0, 0, 0);
      if constexpr (R < 8) {
#pragma unroll
        for (int w = 0; w < R - 4; ++w) dh[w] = fmaf(hi[q][w], xv[q], dh[w]);
      } else {
        floatx4 d2 = {dh[0], dh[1], dh[2], dh[3]};
        d2 = __builtin_amdgcn_mfma_f32_4x4x1f32(hi[q][0], xv[q], d2, 0, 0, 0);
#pragma unroll
        for (int w = 0; w < 4; ++w) dh[w] = d2[w];
      }
    }
  }
}

template <int R, int BINS>
__device__ __forceinline__ void msplat_body(int bx, int by, int bz, const float* __restrict__ xp, int xp_bytes,
                                            const int* __restrict__ start, const float4* __restrict__ rec4,
                                            const float* __restrict__ rec_hi, int P, int K, int M, int sstride, int Ms,
                                            int ls, int reversed, float* __restrict__ u) {
  extern __shared__ __align__(16) float sm[];
  constexpr int W = msplat_rec_words<R>();
  constexpr int NB = BINS / kMsWaves;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int S = 1 << ls, sh = 6 - ls;
  float* recs = sm + wave * 64 * W;           // [64][W]
  float* outu = sm + kMsWaves * 64 * W;       // [R][S][BINS + 1]
  const __amdgpu_buffer_rsrc_t xrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xp), 0, xp_bytes, kBufferWord3);
  const int j = bx, n0 = by * BINS, nw = n0 + NB * wave;
  const unsigned xl4 = unsigned(64 * bz + (lane & (S - 1))) * 4u;  // this lane's scan position
  // the records of the wave's samples: [at[b], at[b + 1])
  const int* sj = start + size_t(j) * sstride;
  int at[NB + 1];
#pragma unroll
  for (int b = 0; b <= NB; ++b) at[b] = sj[min(nw + b, M)];
  float4 v4;
  float vh[R - 3];
  auto load = [&](int c, int e) {  // records c .. c + 63 (past e: e - 1)
    const int i = max(min(c + lane, e - 1), 0);
    v4 = rec4[i];
#pragma unroll
    for (int q = 0; q < R - 3; ++q) vh[q] = rec_hi[size_t(i) * (R - 3) + q];
  };
  load(at[0], at[1]);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int e = at[b + 1];
    double acc[R];
#pragma unroll
    for (int p = 0; p < R; ++p) acc[p] = 0.0;
    if (at[b] == e && b + 1 < NB) load(e, at[b + 2]);
    for (int c = at[b]; c < e; c += 64) {
      {
        const bool in = c + lane < e;
        float* r = recs + lane * W;
        __builtin_amdgcn_wave_barrier();
        *reinterpret_cast<float4*>(r) = in ? v4 : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int q = 0; q < R - 4; ++q) r[4 + q] = in ? vh[q] : 0.0f;
        r[R] = vh[R - 4];
        __builtin_amdgcn_wave_barrier();
      }
      if (c + 64 < e) load(c + 64, e);
      else if (b + 1 < NB) load(e, at[b + 2]);
      floatx4 d = {0.0f, 0.0f, 0.0f, 0.0f};
      float dh[4] = {};
      const int steps = (min(64, e - c) + (1 << sh) - 1) >> sh;
      switch (ls) {
        case 2: msplat_steps<R, 2>(recs, lane, xl4, xrs, steps, d, dh); break;
        case 3: msplat_steps<R, 3>(recs, lane, xl4, xrs, steps, d, dh); break;
        case 4: msplat_steps<R, 4>(recs, lane, xl4, xrs, steps, d, dh); break;
        case 5: msplat_steps<R, 5>(recs, lane, xl4, xrs, steps, d, dh); break;
        default: msplat_steps<R, 6>(recs, lane, xl4, xrs, steps, d, dh); break;
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) acc[p] += double(d[p]);
#pragma unroll
      for (int p = 4; p < R; ++p) acc[p] += double(dh[p - 4]);
    }
    for (int off = S; off < 64; off <<= 1) {
#pragma unroll
      for (int p = 0; p < R; ++p) acc[p] += __shfl_xor(acc[p], off, 64);
    }
    if (lane < S) {
#pragma unroll
      for (int p = 0; p < R; ++p) outu[(p * S + lane) * (BINS + 1) + NB * wave + b] = float(acc[p]);
    }
  }
  __syncthreads();
  // runs of BINS samples of one (trace, moment)
  for (int i = threadIdx.x; i < R * S * BINS; i += blockDim.x) {
    const int b = i & (BINS - 1), ps = i / BINS;
    const int p = ps >> ls, sc = 64 * bz + (ps & (S - 1));
    if (sc < P) {
      const int t = (reversed ? P - 1 - sc : sc) * K + j;
      u[(size_t(t) * R + p) * Ms + n0 + b] = outu[ps * (BINS + 1) + b];
    }
  }
}

template <int R, int BINS = kMsBins>
size_t msplat_lds(int ls) {
  return size_t(kMsWaves * 64 * msplat_rec_words<R>() + R * (1 << ls) * (BINS + 1)) * sizeof(float);
}

template <int R, int BINS>
__global__ __launch_bounds__(64 * kMsWaves) void k_msplat(const float* __restrict__ xp, int xp_bytes,
                                                          const int* __restrict__ start,
                                                          const float4* __restrict__ rec4,
                                                          const float* __restrict__ rec_hi, int P, int K, int M,
                                                          int Ms, int ls, int reversed, float* __restrict__ u,
                                                          CostFold fold) {
  if (fold.out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) {  // uniform
    extern __shared__ __align__(16) float sm[];
    fold_cost(fold, reinterpret_cast<double*>(sm));
  }
  msplat_body<R, BINS>(blockIdx.x, blockIdx.y, blockIdx.z, xp, xp_bytes, start, rec4, rec_hi, P, K, M, M + 1, Ms, ls,
                       reversed, u);
}

// Every template's u (grid z: scan chunks of template 0, of template 1, ...),
// of the samples its span reaches.  A record belongs to one template, so the
// bins are (template, sample) and the records are no more than without
// attenuation.  The fine-grid form fills one dense grid per template: 512
// traces of 65536 positions in 16 templates are 2.1 GB, and writing and reading
// them took 1158 and 1328 us at 256 x 256; u (0.5 GB at most, the spans' share
// of it) takes 139 and 255 us.
__global__ __launch_bounds__(64 * kMsWaves) void k_msplat_att(const float* __restrict__ xp, int xp_bytes,
                                                              const int* __restrict__ start,
                                                              const float4* __restrict__ rec4,
                                                              const float* __restrict__ rec_hi, int P, int K, int M,
                                                              MomentShape ms, const int2* __restrict__ span,
                                                              float* __restrict__ u) {
  const int chunks = (P + 63) / 64, gb = blockIdx.z / chunks;
  const int2 sp = span[gb];
  const int n0 = blockIdx.y * kMsBins;
  if (n0 >= sp.y || n0 + kMsBins <= sp.x) return;  // uniform
  msplat_body<8, kMsBins>(blockIdx.x, blockIdx.y, blockIdx.z - gb * chunks, xp, xp_bytes, start + size_t(gb) * M, rec4, rec_hi,
                 P, K, M, ms.NG * M + 1, ms.Ms, ms.ls, ms.reversed, u + size_t(gb) * P * K * 8 * ms.Ms);
}

// ---- C and C^T: banded Toeplitz products on the bf16 matrix cores, FP32
// products from bf16 pieces (storage.h).  D = A B with 32 traces as rows; the
// Toeplitz operand B[k][col] = G_p[col's d - k] is a table in LDS whose entry
// D holds G_p[D .. D - 7] as one 16-byte word per piece, so every lane's eight
// contraction values are one aligned read and neighbouring lanes read
// neighbouring words.

constexpr int kMcWaves = 8;

// x with the sign bits of `neg` (0 or 1 << 31) flipped
__device__ __forceinline__ float flip_sign(float x, unsigned neg) {
  return __uint_as_float(__float_as_uint(x) ^ neg);
}
__device__ __forceinline__ float4 flip_sign(float4 x, unsigned neg) {
  return make_float4(flip_sign(x.x, neg), flip_sign(x.y, neg), flip_sign(x.z, neg), flip_sign(x.w, neg));
}

__device__ __forceinline__ void stage_table(uint4* tab, const uint4* __restrict__ F, int n) {
  stage_block<uint4>(n, [&](int i) { return F[i]; }, [&](int i, const uint4& v) { tab[i] = v; });
}

// C: a block computes 32 traces x 32 NTC samples; its eight waves take the
// (16 samples of u, moment) items of the window in turn, each item split into
// pieces once and multiplied into every tile it reaches; the waves' sums are
// added in LDS, two tiles at a time, in wave order.  ATT: the templates one
// after the other, each over the samples its span reaches, each summed by
// itself and added to the ones before.
//
// The matrix cores cut the bits of C below the products' grid towards minus
// infinity (a sixth of the largest term's last place in the mean where C is a
// hundredth of the products).  Per trace that is less than FP32 rounding, but it
// adds up over the traces of an image where roundings average out: 3.8e-7 relative L2 of the adjoint at 512 x 512, 2048
// traces, with errors of neighbouring voxels alike.  So every other wave (ATT:
// and template) multiplies the negated samples and is subtracted, here and in
// the correlation: with the gather's partial sums 1.9e-7 at the same time.  The
// items take the moments in turn so that with R = 6 and 8 too each wave gets
// large and small ones, and both kinds of wave each: the attenuated forward at
// 256 x 256 1.2e-7 for 1.93e-7 (1.7e-7 with a moment per wave), 260 for 257 us.
// Without templates an item's six products are summed by themselves, so that
// the sum of the window is rounded once an item: 2.85e-7 before both, 2.4e-7
// with the signs and 1.9e-7 so for a sparse image at 512 x 512 (1.86e-7 on the
// fine grid), 21 us for 20 at 256 x 256.
struct MomentTemplates {
  const int2* span;  // [n]
  int n;
};
template <int R, int NTC, int ST, bool ATT = false>
__device__ __forceinline__ void mconv_body(int bx, int by, const float* __restrict__ u, int Ms,
                                           const uint4* __restrict__ F, int LT, int M, int Lh, int PK,
                                           const typename Store<ST>::T* base, float sign,
                                           const float* __restrict__ g, const float* __restrict__ dbasis,
                                           typename Store<ST>::T* out, MomentTemplates mt = {}) {
  extern __shared__ __align__(16) float sm[];
  uint4* tab = reinterpret_cast<uint4*>(sm);
  const int tr0 = bx * 32, m0 = by * 32 * NTC;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, lk = lane >> 5;
  if constexpr (!ATT) stage_table(tab, F, R * 3 * LT);
  // the epilogue's inputs, fetched while the window multiplies: thread
  // (wave, lane) finishes registers wave and wave + 8 of every tile
  constexpr int E = 2 * NTC;
  float pre_base[E], pre_db[E], pre_g[E];
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int i = wave + 8 * (q & 1);
    const int mm = min(m0 + 32 * (q >> 1) + li, M - 1);
    const int tr = min(tr0 + 8 * (i >> 2) + 4 * lk + (i & 3), PK - 1);
    const size_t idx = size_t(tr) * M + mm;
    pre_base[q] = base ? Store<ST>::get(base[idx]) : 0.0f;
    pre_db[q] = g ? dbasis[idx] : 0.0f;
    pre_g[q] = g ? g[tr] : 0.0f;
  }
  floatx16 acc[NTC];
#pragma unroll
  for (int j = 0; j < NTC; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.0f;
  const float* ut = u + size_t(min(tr0 + li, PK - 1)) * R * Ms;
  // rows n of the window [m0 - Lh, m0 + 32 NTC - 2], in steps of 16 from a
  // multiple of 8 (a group of 8 lies wholly before sample 0 or not at all)
  const int ns = (m0 - Lh) & ~7;
  int s_lo = ns < 0 ? (-ns) >> 4 : 0;
  int s_hi = min((m0 + 32 * NTC - 1 - ns + 15) >> 4, (Ms - ns + 15) >> 4);
  int n_lo = 0, n_hi = Ms;  // rows that hold u (ATT: the groups of 16 written)
  unsigned neg = unsigned(wave & 1) << 31;  // sign flip of this wave's samples
  auto fetch = [&](int q, float4& x, float4& y) {
    const int s = s_lo + q / R, p = (q + q / R) % R;
    const int n = ns + 16 * s + 8 * lk;
    const float* row = ut + p * Ms + min(max(n, 0), Ms - 8);
    x = *reinterpret_cast<const float4*>(row);
    y = *reinterpret_cast<const float4*>(row + 4);
  };
  auto multiply = [&](int q, float4 x, float4 y) {
    const int s = s_lo + q / R, p = (q + q / R) % R;
    const int n0 = ns + 16 * s, n = n0 + 8 * lk;
    if (n < n_lo || (ATT && n >= n_hi)) x = y = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const Pieces8 a = split8_bf16x3(flip_sign(x, neg), flip_sign(y, neg));
    const uint4* tp = tab + p * 3 * LT + 1;
#pragma unroll
    for (int j = 0; j < NTC; ++j) {
      const int dj = m0 + 32 * j - 1 - n0;  // lane's D = dj + li - 8 lk
      if (dj + 31 < 0 || dj - 8 > Lh + 6) continue;  // uniform: no tap meets the tile
      const int D = min(max(dj + li - 8 * lk, -1), LT - 2);
      const uint4 b[3] = {tp[D], tp[LT + D], tp[2 * LT + D]};
      if constexpr (ATT) {
        acc[j] = mfma_bf16x3(a.p, b, acc[j]);
      } else {
        floatx16 t;
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = 0.0f;
        acc[j] += mfma_bf16x3(a.p, b, t);
      }
    }
  };
  auto window = [&]() {
    const int items = (s_hi - s_lo) * R;
    float4 x0, y0, x1, y1;
    if (wave < items) fetch(wave, x0, y0);
    for (int q = wave; q < items; q += 2 * kMcWaves) {
      if (q + kMcWaves < items) fetch(q + kMcWaves, x1, y1);
      multiply(q, x0, y0);
      if (q + kMcWaves < items) {
        if (q + 2 * kMcWaves < items) fetch(q + 2 * kMcWaves, x0, y0);
        multiply(q + kMcWaves, x1, y1);
      }
    }
  };
  if constexpr (ATT) {
    floatx16 tot[NTC];
#pragma unroll
    for (int j = 0; j < NTC; ++j) tot[j] = acc[j];
    const int w_lo = s_lo, w_hi = s_hi;
    for (int gb = 0; gb < mt.n; ++gb) {
      const int2 sp = mt.span[gb];
      n_lo = sp.x & ~15;
      n_hi = (sp.y + 15) & ~15;
      s_lo = max(w_lo, (n_lo - ns) >> 4);
      s_hi = min(w_hi, (n_hi - ns + 15) >> 4);
      if (sp.y > 0 && s_hi > s_lo) {  // uniform
        __syncthreads();  // the table before is read
        stage_table(tab, F + size_t(gb) * R * 3 * LT, R * 3 * LT);
        __syncthreads();
        window();
        const float sgn = neg ? -1.0f : 1.0f;
#pragma unroll
        for (int j = 0; j < NTC; ++j)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            tot[j][i] = fmaf(sgn, acc[j][i], tot[j][i]);
            acc[j][i] = 0.0f;
          }
        neg ^= 0x80000000u;
      }
      ut += size_t(PK) * R * Ms;
    }
#pragma unroll
    for (int j = 0; j < NTC; ++j) acc[j] = tot[j];
  } else {
    __syncthreads();
    window();
  }
  // red[tile of the pair][wave][register][lane]
  constexpr int NP = NTC < 2 ? 1 : 2;
  float* red = sm;
#pragma unroll
  for (int j0 = 0; j0 < NTC; j0 += NP) {
    __syncthreads();  // the table (or the pair before) is read
#pragma unroll
    for (int jj = 0; jj < NP; ++jj)
#pragma unroll
      for (int i = 0; i < 16; ++i) red[((jj * kMcWaves + wave) * 16 + i) * 64 + lane] = acc[j0 + jj][i];
    __syncthreads();
#pragma unroll
    for (int q = 2 * j0; q < 2 * (j0 + NP); ++q) {
      const int i = wave + 8 * (q & 1), jj = (q >> 1) - j0;
      float v = red[(jj * kMcWaves * 16 + i) * 64 + lane];
      for (int w = 1; w < kMcWaves; ++w) {
        const float x = red[((jj * kMcWaves + w) * 16 + i) * 64 + lane];
        v += !ATT && (w & 1) ? -x : x;
      }
      const int mm = m0 + 32 * (q >> 1) + li, tr = tr0 + 8 * (i >> 2) + 4 * lk + (i & 3);
      if (mm < M && tr < PK) {
        float val = sign * v;
        if (base) val += pre_base[q];
        if (g) val -= pre_g[q] * pre_db[q];
        out[size_t(tr) * M + mm] = Store<ST>::put(val);
      }
    }
  }
}

size_t mconv_lds(int R, int LT, int ntc) {
  return std::max(size_t(R) * 3 * LT * sizeof(uint4),
                  size_t(ntc < 2 ? 1 : 2) * kMcWaves * 1024 * sizeof(float));
}

template <int R, int NTC, int ST>
__global__ __launch_bounds__(64 * kMcWaves) void k_mconv(const float* __restrict__ u, int Ms,
                                                         const uint4* __restrict__ F, int LT, int M, int Lh, int PK,
                                                         const typename Store<ST>::T* base, float sign,
                                                         const float* __restrict__ g,
                                                         const float* __restrict__ dbasis,
                                                         typename Store<ST>::T* out) {
  mconv_body<R, NTC, ST>(blockIdx.x, blockIdx.y, u, Ms, F, LT, M, Lh, PK, base, sign, g, dbasis, out);
}

// Eight consecutive samples of a trace row from m on; samples at or past M
// are zero.  `inside` (uniform): every lane's eight lie in the record.
__device__ __forceinline__ void load8(const float* row, int m, int M, bool inside, float (&v)[8]) {
  if (inside) {
    __builtin_memcpy(v, row + m, sizeof(v));  // rows start at any multiple of 4 bytes
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = m + e < M ? row[m + e] : 0.0f;
  }
}

// C^T: a block computes NT tiles of 32 traces x 32 samples x all R moments, with
// 8 / NT waves on each tile; the eight samples of a lane go in reversed, so that
// C's table serves.
// PAIR: v of one template for the gather of pairs, [..][n][R] in place of
// [..][R][n] (vstride: floats between traces).
//
// Four tiles: a tile's two waves share the window's steps (the samples are
// split into pieces once for the R products) and add their sums in LDS; the
// odd one works on negated samples (see C).
template <int R, int NT, bool PAIR>
__device__ __forceinline__ void mcorr_shared_steps(int bx, int by, const float* __restrict__ r,
                                                   const uint4* __restrict__ F, int LT, int M, int Lh, int PK, int Ms,
                                                   float* __restrict__ v, size_t vstride) {
  extern __shared__ __align__(16) float sm[];
  constexpr int KS = kMcWaves / NT;
  uint4* tab = reinterpret_cast<uint4*>(sm);
  const int tr0 = bx * 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, lk = lane >> 5;
  const int jt = wave % NT, ks = wave / NT;
  const int n0 = (by * NT + jt) * 32;
  stage_table(tab, F, R * 3 * LT);
  floatx16 acc[R];
#pragma unroll
  for (int p = 0; p < R; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[p][i] = 0.0f;
  const float* row = r + size_t(min(tr0 + li, PK - 1)) * M;
  // samples m of [n0 + 1, n0 + 31 + Lh], in steps of 16 from n0
  const int steps = n0 < M ? min((Lh + 32 + 15) >> 4, (M - n0 + 15) >> 4) : 0;
  static_assert(KS == 2, "the waves of a tile are added by subtracting the odd one");
  const unsigned neg = unsigned(ks & 1) << 31;
  auto multiply = [&](int s, const float (&x)[8]) {
    const Pieces8 a = split8_bf16x3(flip_sign(make_float4(x[7], x[6], x[5], x[4]), neg),
                                    flip_sign(make_float4(x[3], x[2], x[1], x[0]), neg));
    const int D = min(max(16 * s + 8 * lk + 6 - li, -1), LT - 2);
    const uint4* tp = tab + 1 + D;
#pragma unroll
    for (int p = 0; p < R; ++p) {
      const uint4 b[3] = {tp[(3 * p) * LT], tp[(3 * p + 1) * LT], tp[(3 * p + 2) * LT]};
      acc[p] = mfma_bf16x3(a.p, b, acc[p]);
    }
  };
  auto fetch = [&](int s, float (&x)[8]) {
    load8(row, n0 + 16 * s + 8 * lk, M, n0 + 16 * s + 16 <= M, x);
  };
  __syncthreads();
  float x0[8], x1[8];
  if (ks < steps) fetch(ks, x0);
  for (int s = ks; s < steps; s += 2 * KS) {
    if (s + KS < steps) fetch(s + KS, x1);
    multiply(s, x0);
    if (s + KS < steps) {
      if (s + 2 * KS < steps) fetch(s + 2 * KS, x0);
      multiply(s + KS, x1);
    }
  }
  float* red = sm + size_t(jt) * R * 1024 + lane;
  __syncthreads();
  if (ks == 1) {
#pragma unroll
    for (int p = 0; p < R; ++p)
#pragma unroll
      for (int i = 0; i < 16; ++i) red[(p * 16 + i) * 64] = acc[p][i];
  }
  __syncthreads();
  if (ks != 0 || n0 >= Ms) return;
#pragma unroll
  for (int p = 0; p < R; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[p][i] -= red[(p * 16 + i) * 64];
  if constexpr (PAIR) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int tr = tr0 + 8 * (i >> 2) + 4 * lk + (i & 3);
      if (tr >= PK) continue;
      float4* o = reinterpret_cast<float4*>(v + tr * vstride + size_t(n0 + li) * R);
#pragma unroll
      for (int p = 0; p < R; p += 4) o[p / 4] = make_float4(acc[p][i], acc[p + 1][i], acc[p + 2][i], acc[p + 3][i]);
    }
    return;
  }
#pragma unroll
  for (int p = 0; p < R; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int tr = tr0 + 8 * (i >> 2) + 4 * lk + (i & 3);
      if (tr < PK) v[(size_t(tr) * R + p) * Ms + n0 + li] = acc[p][i];
    }
}

// One or two tiles (few traces or samples: the time of one block is the
// launch's): the waves share the moments, ceil(R NT / 8) each over all of the
// window, so that there are no sums to add up between them; each splits the
// samples for itself.  8.8 against 12.9 us for 8 traces of 256 samples (10 MHz,
// between events around the launch).  With four tiles, moments per wave left the
// adjoint at 256 x 256 at 2.5e-7 with running sums (2.0e-7 with the steps shared,
// 1.8e-7 since every other wave's samples are negated), and adding each step by
// itself, as here, takes registers that halve the blocks of a CU (165 against
// 142 us at 512 x 512).
template <int R, int NT, bool PAIR>
__device__ __forceinline__ void mcorr_shared_moments(int bx, int by, const float* __restrict__ r,
                                                     const uint4* __restrict__ F, int LT, int M, int Lh, int PK,
                                                     int Ms, float* __restrict__ v, size_t vstride) {
  extern __shared__ __align__(16) float sm[];
  constexpr int KS = kMcWaves / NT;
  constexpr int NP = (R + KS - 1) / KS;  // moments per wave
  uint4* tab = reinterpret_cast<uint4*>(sm);
  const int tr0 = bx * 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, lk = lane >> 5;
  const int jt = wave % NT, p0 = wave / NT * NP;
  const int n0 = (by * NT + jt) * 32;
  stage_table(tab, F, R * 3 * LT);
  floatx16 acc[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[p][i] = 0.0f;
  const float* row = r + size_t(min(tr0 + li, PK - 1)) * M;
  // samples m of [n0 + 1, n0 + 31 + Lh], in steps of 16 from n0
  const int steps = n0 < M && p0 < R ? min((Lh + 32 + 15) >> 4, (M - n0 + 15) >> 4) : 0;
  auto multiply = [&](int s, const float (&x)[8], unsigned neg) {
    const Pieces8 a = split8_bf16x3(flip_sign(make_float4(x[7], x[6], x[5], x[4]), neg),
                                    flip_sign(make_float4(x[3], x[2], x[1], x[0]), neg));
    const int D = min(max(16 * s + 8 * lk + 6 - li, -1), LT - 2);
    const uint4* tp = tab + 1 + D + 3 * p0 * LT;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (R % NP != 0 && p0 + p >= R) continue;  // uniform
      const uint4 b[3] = {tp[(3 * p) * LT], tp[(3 * p + 1) * LT], tp[(3 * p + 2) * LT]};
      // a step's six products by themselves: one rounding of the running sum
      // per step, not six (odd steps on negated samples, see C)
      floatx16 t;
#pragma unroll
      for (int i = 0; i < 16; ++i) t[i] = 0.0f;
      t = mfma_bf16x3(a.p, b, t);
      acc[p] += neg ? -t : t;
    }
  };
  auto fetch = [&](int s, float (&x)[8]) {
    load8(row, n0 + 16 * s + 8 * lk, M, n0 + 16 * s + 16 <= M, x);
  };
  float x0[8], x1[8];
  if (steps > 0) fetch(0, x0);
  __syncthreads();
  for (int s = 0; s < steps; s += 2) {
    if (s + 1 < steps) fetch(s + 1, x1);
    multiply(s, x0, 0u);
    if (s + 1 < steps) {
      if (s + 2 < steps) fetch(s + 2, x0);
      multiply(s + 1, x1, 0x80000000u);
    }
  }
  if (n0 >= Ms) return;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int tr = tr0 + 8 * (i >> 2) + 4 * lk + (i & 3);
    if (tr >= PK) continue;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p0 + p >= R) continue;
      if constexpr (PAIR) v[tr * vstride + size_t(n0 + li) * R + p0 + p] = acc[p][i];
      else v[(size_t(tr) * R + p0 + p) * Ms + n0 + li] = acc[p][i];
    }
  }
}

template <int R, int NT, bool PAIR = false>
__device__ __forceinline__ void mcorr_body(int bx, int by, const float* __restrict__ r,
                                           const uint4* __restrict__ F, int LT, int M, int Lh, int PK, int Ms,
                                           float* __restrict__ v, size_t vstride = 0) {
  if constexpr (NT == 4) mcorr_shared_steps<R, NT, PAIR>(bx, by, r, F, LT, M, Lh, PK, Ms, v, vstride);
  else mcorr_shared_moments<R, NT, PAIR>(bx, by, r, F, LT, M, Lh, PK, Ms, v, vstride);
}

// the table, then the sums of one of two waves per tile
size_t mcorr_lds(int R, int LT) {
  return std::max(size_t(R) * 3 * LT * sizeof(uint4), size_t(kMcWaves / 2) * R * 1024 * sizeof(float));
}

template <int R, int NT>
__global__ __launch_bounds__(64 * kMcWaves) void k_mcorr(const float* __restrict__ r, const uint4* __restrict__ F,
                                                         int LT, int M, int Lh, int PK, int Ms,
                                                         float* __restrict__ v) {
  mcorr_body<R, NT>(blockIdx.x, blockIdx.y, r, F, LT, M, Lh, PK, Ms, v);
}

// Every template's v (grid z), over the samples its span reaches: 182 us for 512
// traces of 2048 samples in 16 templates (960 us to the fine grids).
template <int NT>
__global__ __launch_bounds__(64 * kMcWaves) void k_mcorr_att(const float* __restrict__ r,
                                                             const uint4* __restrict__ F, int LT, int M, int Lh,
                                                             int PK, int Ms, int NG, const int2* __restrict__ span,
                                                             float* __restrict__ v) {
  const int gb = blockIdx.z, n0 = int(blockIdx.y) * 32 * NT;
  const int2 sp = span[gb];
  if (n0 >= sp.y || n0 + 32 * NT <= sp.x) return;  // uniform
  mcorr_body<8, NT, true>(blockIdx.x, blockIdx.y, r, F + size_t(gb) * 24 * LT, LT, M, Lh, PK, Ms,
                          v + size_t(gb) * Ms * 8, size_t(NG) * Ms * 8);
}

// ---- S^T

// The windowed gather over moments: blocks of 512 threads take 32 x 64 voxel
// tiles (wave w's load q covers tile row 8 q + w, one lane per column); for
// every trace of group bx the tile's window of v (R planes, from the
// geometry's table of (tile, trace) windows) is copied into LDS with 16-byte
// loads, one trace ahead, into the other of two buffers (one barrier per
// trace), and every voxel evaluates its polynomial at its two table points
// and interpolates.  The window is Q / R times smaller than the fine grid's,
// so two buffers fit.  One partial image per group, traces in order, summed 16
// at a time (a running sum over a group of 256 rounds 256 times at full size:
// 3.1e-7 against 1.9e-7 relative L2 at 512 x 512, at the same time).
//
// A window longer than a buffer (2048 samples at R = 5) is staged into both,
// without a trace in flight beside it, and one longer than both is read from
// memory.  Such windows belong to tiles that straddle the top layer's face:
// one row of tiles of 16 at 512 x 512, 4096 samples, where a third of them read
// from memory paced the whole launch, 1345 us against 1088 us staged.  A
// block's tiles lie a whole generation of blocks apart, so that no block has
// two of them: 927 us, and 880 as it stands.  (Tiles that stop at layers' faces
// instead: 1160 us, and 12 % more of them.)  Bound by its vector instructions (34 per wave and
// trace-voxel, 54 % of the cycles at 256 x 256), the load unit (65 %) and LDS
// (36 %), which the barrier of each trace keeps from overlapping fully.
// Sharing a record between voxels a pitch apart, four traces a barrier and
// windows dealt to the waves piece by piece halved single shares of these but
// not the time (57 .. 95 us against 57 then, 50 now, at 256 x 256; 910 .. 1440 at
// 512 x 512).
constexpr int kMgBufBytes = 40960;  // one window buffer; two per block, two blocks per CU

template <int R>
__host__ __device__ constexpr int mgather_cap() { return kMgBufBytes / (4 * R) / 4 * 4; }

template <int R>
__device__ __forceinline__ void mgather_body(int bx, int by, const float* __restrict__ v, int Ms, int nx, int nz,
                                             int n_off, const Leg* __restrict__ legs,
                                             const float* __restrict__ tau, const int* __restrict__ base, int P,
                                             int K, int qs, int M, int tpg, const int2* __restrict__ gwin,
                                             int tiles_per_block, float* __restrict__ partial) {
  extern __shared__ __align__(16) float sm[];  // [2][R][kCap]
  constexpr int kCap = mgather_cap<R>();
  static_assert(kCap <= 4 * 512, "one 16-byte load per thread and plane");
  constexpr int VPT = kGatherTileRows / 8;
  const int N = nx * nz, PK = P * K;
  const int t0 = bx * tpg, t1 = min(t0 + tpg, PK);
  const int tiles_x = (nx + kGatherTileCols - 1) / kGatherTileCols;
  const int n_tiles = tiles_x * ((nz + kGatherTileRows - 1) / kGatherTileRows);
  const int blocks = (n_tiles + tiles_per_block - 1) / tiles_per_block;
  const int half = n_off / 2;
  // (the wave's number in a scalar register: the rows' offsets then take none of
  // the 128 vector registers that four waves per SIMD leave)
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), lane = int(threadIdx.x & 63);
  const float h = 2.0f / float(1 << qs);
  const __amdgpu_buffer_rsrc_t leg_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<Leg*>(legs), 0, nz * n_off * int(sizeof(Leg)), kBufferWord3);
  struct Legs { int64_t d[VPT]; float p[VPT]; };
  for (int tile = by; tile < n_tiles; tile += blocks) {
    const int tz = tile / tiles_x;
    const int tx = tile - tz * tiles_x;
    int col2[VPT], rowoff[VPT], vox[VPT];
    bool ok[VPT];
    float acc[VPT], tot[VPT];  // of up to 16 traces; of those before
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      const int row = tz * kGatherTileRows + 8 * q + wave;
      const int col = tx * kGatherTileCols + lane;
      ok[q] = row < nz && col < nx;
      const int r = min(row, nz - 1), c = min(col, nx - 1);  // outside the grid: a voxel of the tile, unused
      vox[q] = r * nx + c;
      col2[q] = 2 * c;
      rowoff[q] = r * n_off;
      acc[q] = tot[q] = 0.0f;
    }
    const int2* wt = gwin + size_t(tile) * PK;
    auto load_leg = [&](int bt, Legs& L) {
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        const int o = (rowoff[q] + leg_slot(abs(bt + col2[q]), half)) * int(sizeof(Leg));
        const auto a = __builtin_amdgcn_raw_buffer_load_b64(leg_rs, o, 0, 0);
        L.p[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(leg_rs, o + 8, 0, 0));
        L.d[q] = int64_t((uint64_t(a[1]) << 32) | a[0]);
      }
    };
    // the window of trace t in samples: {first (a multiple of 4), count (a
    // multiple of 4, 0: no voxel of the tile lies in the record)}
    auto window = [&](int t) {
      const int2 w = wt[min(t, t1 - 1)];
      if (w.y == 0 || t >= t1) return make_int2(0, 0);
      const int lo = (w.x >> qs) & ~3;
      const int hi = min((w.x + w.y - 1) >> qs, M - 1);
      return make_int2(lo, (hi + 1 - lo + 3) & ~3);
    };
    const int x4 = 4 * int(threadIdx.x);
    // (unconditional loads: slots past the window read out of range, zero)
    auto stage_load = [&](int2 W, int t, uint4 (&rg)[R]) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(v + size_t(min(t, t1 - 1)) * R * Ms), 0, R * Ms * 4, kBufferWord3);
      const bool in = W.y <= kCap && x4 < W.y;
#pragma unroll
      for (int p = 0; p < R; ++p) {
        const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, in ? (p * Ms + W.x + x4) * 4 : 0x7ffffff0, 0, 0);
        rg[p] = make_uint4(q[0], q[1], q[2], q[3]);
      }
    };
    auto stage_store = [&](int2 W, float* buf, const uint4 (&rg)[R]) {
      if (W.y <= kCap && x4 < W.y) {
#pragma unroll
        for (int p = 0; p < R; ++p) *reinterpret_cast<uint4*>(buf + p * kCap + x4) = rg[p];
      }
    };
    Legs TX, La, Lb;
    // a window of up to both buffers, planes 2 kCap apart
    auto stage_long = [&](int2 W, int t) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(v + size_t(t) * R * Ms), 0, R * Ms * 4, kBufferWord3);
#pragma unroll 1
      for (int x = x4; x < W.y; x += 4 * 512) {
        uint4 q[R];
#pragma unroll
        for (int p = 0; p < R; ++p) {
          const auto d = __builtin_amdgcn_raw_buffer_load_b128(rs, (p * Ms + W.x + x) * 4, 0, 0);
          q[p] = make_uint4(d[0], d[1], d[2], d[3]);
        }
#pragma unroll
        for (int p = 0; p < R; ++p) *reinterpret_cast<uint4*>(sm + p * 2 * kCap + x) = q[p];
      }
    };
    auto add = [&](const Legs& L, int2 W, int t, const float* buf, int plane) {
      if (W.y == 0) return;
      const bool fits = W.y <= plane;
      const float* vt = v + size_t(t) * R * Ms + W.x;
      // the window's samples of the record: it holds every voxel of the tile
      // in the record, and bounds each index here
      const unsigned cnt = unsigned(min(W.y, M - W.x));
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        const uint64_t D = uint64_t(TX.d[q] + L.d[q]);
        const unsigned n = unsigned(D >> 32) - unsigned(W.x);  // in the window
        const bool in = n < cnt;
        const unsigned fr = unsigned(D);
        const float w = TX.p[q] * L.p[q];
        const float z0 = fmaf(float(fr >> (32 - qs)), h, -1.0f), z1 = z0 + h;
        const float phi = float(fr << qs) * 2.3283064365386963e-10f;
        float c[R];
        if (fits) {
          const float* s = buf + (in ? n : 0u);
#pragma unroll
          for (int p = 0; p < R; ++p) c[p] = s[p * plane];
        } else {
          const float* s = vt + (in ? n : 0u);
#pragma unroll
          for (int p = 0; p < R; ++p) c[p] = s[size_t(p) * Ms];
        }
        float f0 = c[R - 1], f1 = c[R - 1];
#pragma unroll
        for (int p = R - 2; p >= 0; --p) {
          f0 = fmaf(f0, z0, c[p]);
          f1 = fmaf(f1, z1, c[p]);
        }
        const float sum = fmaf(w, fmaf(phi, f1 - f0, f0), acc[q]);
        acc[q] = in ? sum : acc[q];
      }
    };
    if (t0 < t1) {
      uint4 rg[R];
      int scan = t0 / K;
      load_leg(base[scan], TX);
      load_leg(base[P + t0], La);
      int2 Wc = window(t0), Wn = window(t0 + 1);
      stage_load(Wc, t0, rg);
      __syncthreads();  // the tile before is done with the buffers
      stage_store(Wc, sm, rg);
      stage_load(Wn, t0 + 1, rg);
      __syncthreads();
      // trace t: window in buffer (t - t0) & 1, legs in L; the window of
      // t + 1 is in rg (in flight)
      auto step = [&](int t, Legs& L, Legs& Ln) {
        float* cur = sm + ((t - t0) & 1) * (kMgBufBytes / 4);
        float* nxt = sm + ((t - t0 + 1) & 1) * (kMgBufBytes / 4);
        if (t + 1 < t1) load_leg(base[P + t + 1], Ln);
        if (t / K != scan) {  // uniform: the next scan position's transmit legs
          scan = t / K;
          load_leg(base[scan], TX);
        }
        const int2 W2 = window(t + 2);
        if (Wc.y > kCap) {  // uniform
          if (Wc.y <= 2 * kCap) {
            stage_long(Wc, t);
            __syncthreads();
          }
          add(L, Wc, t, sm, 2 * kCap);
          __syncthreads();
        } else {
          add(L, Wc, t, cur, kCap);
        }
        stage_store(Wn, nxt, rg);
        stage_load(W2, t + 2, rg);
        Wc = Wn;
        Wn = W2;
        __syncthreads();
      };
      for (int t = t0; t < t1; t += 2) {
        step(t, La, Lb);
        if (t + 1 < t1) step(t + 1, Lb, La);
        if (((t - t0) & 14) == 14) {
#pragma unroll
          for (int q = 0; q < VPT; ++q) {
            tot[q] += acc[q];
            acc[q] = 0.0f;
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < VPT; ++q)
      if (ok[q]) partial[size_t(bx) * N + vox[q]] = (tot[q] + acc[q]) * tau[vox[q] / nx];
  }
}

template <int R>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(R < 8 ? 4 : 2))) void k_mgather(
    const float* __restrict__ v, int Ms, int nx, int nz, int n_off, const Leg* __restrict__ legs,
    const float* __restrict__ tau, const int* __restrict__ base, int P, int K, int qs, int M, int tpg,
    const int2* __restrict__ gwin, int tiles_per_block, float* __restrict__ partial) {
  mgather_body<R>(blockIdx.x, blockIdx.y, v, Ms, nx, nz, n_off, legs, tau, base, P, K, qs, M, tpg, gwin,
                  tiles_per_block, partial);
}

// The gather with attenuation: v is [trace][template][n][8], so that a pair's
// eight values are two 16-byte loads of one 32-byte sector, from L2.  Threads
// take voxels in row-major order, VPT a thread; the legs of trace t + 2 and the
// values of trace t + 1 are in flight while trace t accumulates.  One partial
// image per trace group, traces in order.  Bound by the load unit, a line per
// lane: 158 us at 256 x 256, 512 traces (2 x 139 us from the fine grids, whose
// batches of traces had to fit an L2).
constexpr int kMgAttVpt = 2;
__global__ __launch_bounds__(256) void k_mgather_att(const float* __restrict__ v, MomentShape ms, int nx, int nz,
                                                     int n_off, const Leg* __restrict__ legs,
                                                     const double* __restrict__ gunit, const float* __restrict__ tau,
                                                     const int* __restrict__ base, int P, int K, int qs, int M,
                                                     int tpg, int vox_per_block, float* __restrict__ partial) {
  constexpr int V = kMgAttVpt;
  const int N = nx * nz, PK = P * K;
  const int v_begin = blockIdx.y * vox_per_block, v_end = min(N, v_begin + vox_per_block);
  const int t0 = blockIdx.x * tpg, t1 = min(t0 + tpg, PK);
  const int half = n_off / 2;
  const float h = 2.0f / float(1 << qs);
  const __amdgpu_buffer_rsrc_t leg_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<Leg*>(legs), 0, nz * n_off * int(sizeof(Leg)), kBufferWord3);
  const __amdgpu_buffer_rsrc_t gu_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(gunit), 0, nz * n_off * 8, kBufferWord3);
  const int v_floats = ms.NG * ms.Ms * 8;  // of one trace
  struct Legs { int64_t d[V]; float p[V]; double u[V]; };
  struct Pairs { int at[V]; unsigned fr[V]; float w[V]; };
  struct Values { float4 lo[V], hi[V]; };
  for (int vc = v_begin; vc < v_end; vc += 256 * V) {
    int col2[V], rowoff[V];
    float acc[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int vox = min(vc + q * 256 + int(threadIdx.x), v_end - 1);  // past the end: a voxel of the block, unused
      const int row = vox / nx;
      col2[q] = 2 * (vox - row * nx);
      rowoff[q] = row * n_off;
      acc[q] = 0.0f;
    }
    auto load_leg = [&](int bt, Legs& L) {
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const int o = (rowoff[q] + leg_slot(abs(bt + col2[q]), half)) * int(sizeof(Leg));
        const auto a = __builtin_amdgcn_raw_buffer_load_b64(leg_rs, o, 0, 0);
        L.p[q] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(leg_rs, o + 8, 0, 0));
        L.u[q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(gu_rs, o >> 1, 0, 0));
        L.d[q] = int64_t((uint64_t(a[1]) << 32) | a[0]);
      }
    };
    Legs TX;
    int scan = -1;
    auto pairs = [&](const Legs& L, int t, Pairs& T) {
      t = min(t, t1 - 1);
      if (t / K != scan) {  // uniform
        scan = t / K;
        load_leg(base[scan], TX);
      }
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const uint64_t D = uint64_t(TX.d[q] + L.d[q]);
        const unsigned n = unsigned(D >> 32);
        const int gb = gamma_bin(TX.u[q] + L.u[q], ms.NG - 1);
        T.at[q] = n < unsigned(M) ? (gb * ms.Ms + int(n)) * 32 : 0x7fffff00;  // past the record: reads zero
        T.fr[q] = unsigned(D);
        T.w[q] = TX.p[q] * L.p[q];
      }
    };
    auto values = [&](const Pairs& T, int t, Values& S) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(v + size_t(min(t, t1 - 1)) * v_floats), 0, v_floats * 4, kBufferWord3);
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const auto a = __builtin_amdgcn_raw_buffer_load_b128(rs, T.at[q], 0, 0);
        const auto b = __builtin_amdgcn_raw_buffer_load_b128(rs, T.at[q] + 16, 0, 0);
        S.lo[q] = __builtin_bit_cast(float4, a);
        S.hi[q] = __builtin_bit_cast(float4, b);
      }
    };
    auto add = [&](const Pairs& T, const Values& S) {
#pragma unroll
      for (int q = 0; q < V; ++q) {
        const unsigned fr = T.fr[q], ti = fr >> (32 - qs);
        const float z0 = fmaf(float(ti), h, -1.0f), z1 = z0 + h;
        const float phi = float(fr << qs) * 2.3283064365386963e-10f;
        const float c[6] = {S.lo[q].x, S.lo[q].y, S.lo[q].z, S.lo[q].w, S.hi[q].x, S.hi[q].y};
        float f0 = c[5], f1 = c[5];
#pragma unroll
        for (int p = 4; p >= 0; --p) {
          f0 = fmaf(f0, z0, c[p]);
          f1 = fmaf(f1, z1, c[p]);
        }
        // the forced zeros at the ends of the bank's rows
        if (ti == 0u) f0 += S.hi[q].w;
        if (ti == (1u << qs) - 1u) f1 += S.hi[q].z;
        acc[q] = fmaf(T.w[q], fmaf(phi, f1 - f0, f0), acc[q]);
      }
    };
    if (t0 < t1) {
      Legs L;
      Pairs T0, T1;
      Values S0, S1;
      load_leg(base[P + t0], L);
      pairs(L, t0, T0);
      load_leg(base[P + min(t0 + 1, t1 - 1)], L);
      values(T0, t0, S0);
      for (int t = t0; t < t1; t += 2) {
        // trace t: T0 / S0 (in flight); the legs of t + 1 in L (in flight)
        pairs(L, t + 1, T1);
        load_leg(base[P + min(t + 2, t1 - 1)], L);
        values(T1, t + 1, S1);
        __builtin_amdgcn_sched_barrier(0);
        add(T0, S0);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 >= t1) break;
        pairs(L, t + 2, T0);
        load_leg(base[P + min(t + 3, t1 - 1)], L);
        values(T0, t + 2, S0);
        __builtin_amdgcn_sched_barrier(0);
        add(T1, S1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const int vox = vc + q * 256 + int(threadIdx.x);
      if (vox < v_end) partial[size_t(blockIdx.x) * N + vox] = acc[q] * tau[vox / nx];
    }
  }
}

// ---- grouped ICD: one group's columns of A against e, and their sum

// delay (Q32.32 samples), weight and the two table points of member i of a
// group in trace t
struct IcdMember {
  unsigned n;
  float z0, phi, w;
};
__device__ __forceinline__ IcdMember icd_moment_member(const Leg* __restrict__ legs, int n_off,
                                                       const float* __restrict__ tau, int bt, int br,
                                                       const IcdGroup& gp, int Sr, int Sc, int qs, int i) {
  int row, col;
  icd_member(gp, Sr, Sc, i, &row, &col);
  const PairLegs p = pair_legs(legs, n_off, bt, br, row, col);
  const unsigned fr = unsigned(p.D);
  const float h = 2.0f / float(1 << qs);
  return {unsigned(p.D >> 32), fmaf(float(fr >> (32 - qs)), h, -1.0f), float(fr << qs) * 2.3283064365386963e-10f,
          tau[row] * p.w};
}

// partial[i][t] = A_{t, v_i}^T e_t from v (v_p[n] of e): a block per trace, one
// thread per member, v of the trace in LDS as far as planes fit (`planes`; the
// others are read from memory).
template <int R>
__global__ __launch_bounds__(1024) void k_icd_mdots(const float* __restrict__ v, int Ms, int planes,
                                                    const Leg* __restrict__ legs, int n_off,
                                                    const float* __restrict__ tau, const int* __restrict__ base,
                                                    int P, int K, int qs, int M, IcdGroup gp, int Sr, int Sc,
                                                    float* __restrict__ partial) {
  extern __shared__ __align__(16) float sm[];  // [planes][Ms]
  const int t = blockIdx.x;
  const float* vt = v + size_t(t) * R * Ms;
  const int bt = base[t / K], br = base[P + t];
  const float h = 2.0f / float(1 << qs);
  const int i0 = blockIdx.y * blockDim.x + threadIdx.x;
  // the first member's legs arrive while v is staged
  IcdMember mb = icd_moment_member(legs, n_off, tau, bt, br, gp, Sr, Sc, qs, min(i0, gp.size - 1));
  stage_block<float4>(planes * Ms / 4, [&](int k) { return reinterpret_cast<const float4*>(vt)[k]; },
                      [&](int k, const float4& x) { reinterpret_cast<float4*>(sm)[k] = x; });
  __syncthreads();
  for (int i = i0; i < gp.size; i += gridDim.y * blockDim.x) {
    if (i != i0) mb = icd_moment_member(legs, n_off, tau, bt, br, gp, Sr, Sc, qs, i);
    float f0 = 0.0f, f1 = 0.0f;
    if (mb.n < unsigned(M)) {
      const float z1 = mb.z0 + h;
#pragma unroll
      for (int p = R - 1; p >= 0; --p) {
        const float c = p < planes ? sm[p * Ms + mb.n] : vt[size_t(p) * Ms + mb.n];
        f0 = fmaf(f0, mb.z0, c);
        f1 = fmaf(f1, z1, c);
      }
    }
    partial[size_t(i) * gridDim.x + t] = mb.w * fmaf(mb.phi, f1 - f0, f0);
  }
}

// u_p[n] = sum_i delta_i w a_p of the group's members, `planes` of the R at a
// time in 64-bit fixed point in LDS (bitwise reproducible).  |a_p|, |w| <= 1,
// so the scale of k_icd_scatter keeps every sum below 2^62.
template <int R>
__global__ __launch_bounds__(1024) void k_icd_msplat(float* __restrict__ u, int Ms, int planes,
                                                     const Leg* __restrict__ legs, int n_off,
                                                     const float* __restrict__ tau, const int* __restrict__ base,
                                                     int P, int K, int qs, int M, IcdGroup gp, int Sr, int Sc,
                                                     const float* __restrict__ delta) {
  extern __shared__ __align__(16) unsigned long long sums[];  // [planes][Ms]
  __shared__ float wmax[16];
  const int t = blockIdx.x, tid = int(threadIdx.x);
  const int bt = base[t / K], br = base[P + t];
  const float h = 2.0f / float(1 << qs);
  // the first member's step and legs arrive while the sums are cleared
  const float dl0 = tid < gp.size ? delta[tid] : 0.0f;
  const IcdMember mb0 = icd_moment_member(legs, n_off, tau, bt, br, gp, Sr, Sc, qs, min(tid, gp.size - 1));
  float mx = fabsf(dl0);
  for (int i = tid + int(blockDim.x); i < gp.size; i += blockDim.x) mx = fmaxf(mx, fabsf(delta[i]));
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((tid & 63) == 0) wmax[tid >> 6] = mx;
  ulonglong2* sums2 = reinterpret_cast<ulonglong2*>(sums);
  float* ut = u + size_t(t) * R * Ms;
  for (int p0 = 0; p0 < R; p0 += planes) {
    const int np = min(planes, R - p0);
    for (int k = tid; k < np * Ms / 2; k += blockDim.x) sums2[k] = make_ulonglong2(0ull, 0ull);
    __syncthreads();
    float dmax = 0.0f;
    for (int k = 0; k < int(blockDim.x >> 6); ++k) dmax = fmaxf(dmax, wmax[k]);
    int lg = 0;
    while ((1 << lg) < gp.size) ++lg;
    const int kx = dmax > 0.0f ? 61 - lg - ilogbf(dmax) : 0;
    const double scale = ldexp(1.0, kx), back = ldexp(1.0, -kx);
    for (int i = tid; i < gp.size; i += blockDim.x) {
      const float dl = i == tid ? dl0 : delta[i];
      if (dl == 0.0f) continue;
      const IcdMember mb = i == tid ? mb0 : icd_moment_member(legs, n_off, tau, bt, br, gp, Sr, Sc, qs, i);
      if (mb.n >= unsigned(M)) continue;
      const float z1 = mb.z0 + h;
      float a1 = dl * mb.w * mb.phi, a0 = dl * mb.w * (1.0f - mb.phi);
#pragma unroll
      for (int p = 0; p < R; ++p) {
        if (p >= p0 && p < p0 + np)
          atomicAdd(&sums[(p - p0) * Ms + mb.n],
                    static_cast<unsigned long long>(__double2ll_rn((double(a0) + double(a1)) * scale)));
        a0 *= mb.z0;
        a1 *= z1;
      }
    }
    __syncthreads();
    for (int k = tid; k < np * Ms / 4; k += blockDim.x) {
      const ulonglong2 x = sums2[2 * k], y = sums2[2 * k + 1];
      auto value = [&](unsigned long long s) { return float(double(static_cast<long long>(s)) * back); };
      reinterpret_cast<float4*>(ut + size_t(p0) * Ms)[k] = make_float4(value(x.x), value(x.y), value(y.x), value(y.y));
    }
    __syncthreads();
  }
}

// ---- work-list forms (see the sweeps' in operator.hip): an item runs the
// block (y, z, w) of its problem's own launch.

// Calls f(integral_constant) for the problem's R.
template <typename F>
__device__ __forceinline__ void with_r_device(int R, F&& f) {
  if (R == 5) f(std::integral_constant<int, 5>());
  else if (R == 6) f(std::integral_constant<int, 6>());
  else f(std::integral_constant<int, 8>());
}
template <typename F>
__device__ __forceinline__ void with_tiles_device(int n, F&& f) {
  if (n == 4) f(std::integral_constant<int, 4>());
  else if (n == 2) f(std::integral_constant<int, 2>());
  else f(std::integral_constant<int, 1>());
}

__global__ __launch_bounds__(64 * kMsWaves) void k_msplat_list(const BatchProb* __restrict__ probs,
                                                               const int* __restrict__ active,
                                                               const int4* __restrict__ items, int n_items,
                                                               int which) {
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    if (!active[w.x]) continue;  // uniform: the problem left the batch
    const BatchProb& p = probs[w.x];
    const float* xp = p.P == 1 ? p.x[which] : p.xt;
    with_r_device(p.mom.R, [&](auto rc) {
      msplat_body<decltype(rc)::value, kMsBins>(w.y, w.z, w.w, xp, p.nz * p.mom.pitch * p.mom.Lq * 4, p.mom_start, p.mom_rec4,
                                       p.mom_rec_hi, p.P, p.K, p.M, p.M + 1, p.mom.Ms, p.mom.ls, p.mom.reversed, p.fine);
    });
    __syncthreads();
  }
}

// residual e = y - A x - g D of the iteration
__global__ __launch_bounds__(64 * kMcWaves) void k_mconv_list(const BatchProb* __restrict__ probs,
                                                              const int* __restrict__ active,
                                                              const int4* __restrict__ items, int n_items) {
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    if (!active[w.x]) continue;
    const BatchProb& p = probs[w.x];
    with_r_device(p.mom.R, [&](auto rc) {
      with_tiles_device(p.mom_tiles, [&](auto nc) {
        mconv_body<decltype(rc)::value, decltype(nc)::value, UMBIR_STORAGE_F32>(
            w.y, w.z, p.fine, p.mom.Ms, p.mom_taps, p.mom.LT, p.M, p.Lh, p.P * p.K, p.y, -1.0f, p.g, p.dbasis, p.e);
      });
    });
    __syncthreads();
  }
}

__global__ __launch_bounds__(64 * kMcWaves) void k_mcorr_list(const BatchProb* __restrict__ probs,
                                                              const int* __restrict__ active,
                                                              const int4* __restrict__ items, int n_items) {
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    if (!active[w.x]) continue;
    const BatchProb& p = probs[w.x];
    with_r_device(p.mom.R, [&](auto rc) {
      with_tiles_device(p.mom_tiles, [&](auto nc) {
        mcorr_body<decltype(rc)::value, decltype(nc)::value>(
            w.y, w.z, p.e, p.mom_taps, p.mom.LT, p.M, p.Lh, p.P * p.K, p.mom.Ms, p.fine);
      });
    });
    __syncthreads();
  }
}

__global__ __launch_bounds__(512) void k_mgather_list(const BatchProb* __restrict__ probs,
                                                      const int* __restrict__ active,
                                                      const int4* __restrict__ items, int n_items) {
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    if (!active[w.x]) continue;
    const BatchProb& p = probs[w.x];
    with_r_device(p.mom.R, [&](auto rc) {
      mgather_body<decltype(rc)::value>(w.y, w.z, p.fine, p.mom.Ms, p.nx, p.nz, p.n_off, p.legs, p.tau, p.base, p.P,
                                        p.K, p.qs, p.M, p.tpg, p.gwin, p.vpb, p.partial);
    });
    __syncthreads();
  }
}

template <int NTC>
__global__ __launch_bounds__(64 * kMcWaves) void k_mconv_att(const float* __restrict__ u, int Ms,
                                                             const uint4* __restrict__ F, int LT, int M, int Lh,
                                                             int PK, const float* base, float sign,
                                                             const float* __restrict__ g,
                                                             const float* __restrict__ dbasis, float* out,
                                                             MomentTemplates mt) {
  mconv_body<8, NTC, UMBIR_STORAGE_F32, true>(blockIdx.x, blockIdx.y, u, Ms, F, LT, M, Lh, PK, base, sign, g, dbasis,
                                              out, mt);
}

// ---- launches

const uint4* taps_of(const umbir_geometry& G, bool abs_op) {
  return G.mom_taps + (abs_op ? G.mom.taps_words() : 0);
}

template <int R, int NTC, int ST>
void launch_mconv(const umbir_geometry& G, const float* u, const void* base, float sign, const float* g, bool abs_op,
                  void* out, hipStream_t s) {
  using T = typename Store<ST>::T;
  const dim3 grid(unsigned((G.traces() + 31) / 32), unsigned((G.M + 32 * NTC - 1) / (32 * NTC)));
  UMBIR_LAUNCH("conv", (k_mconv<R, NTC, ST>), grid, dim3(64 * kMcWaves), mconv_lds(R, G.mom.LT, NTC), s, u,
               G.mom.Ms, taps_of(G, abs_op), G.mom.LT, G.M, G.Lh, G.traces(), static_cast<const T*>(base), sign, g, G.dbasis,
               static_cast<T*>(out));
}

template <int R, int NT>
void launch_mcorr(const umbir_geometry& G, const float* r, bool abs_op, float* v, hipStream_t s) {
  const dim3 grid(unsigned((G.traces() + 31) / 32), unsigned((G.mom.Ms / 32 + NT - 1) / NT));
  UMBIR_LAUNCH("corr", (k_mcorr<R, NT>), grid, dim3(64 * kMcWaves), mcorr_lds(R, G.mom.LT), s, r,
               taps_of(G, abs_op), G.mom.LT, G.M, G.Lh, G.traces(), G.mom.Ms, v);
}

// Calls f(integral_constant R, integral_constant storage).
template <typename F>
void with_r(int R, F&& f) {
  if (R == 5) f(std::integral_constant<int, 5>());
  else if (R == 6) f(std::integral_constant<int, 6>());
  else f(std::integral_constant<int, 8>());
}
template <typename F>
void with_storage(int st, F&& f) {
  if (st == UMBIR_STORAGE_F16) f(std::integral_constant<int, UMBIR_STORAGE_F16>());
  else if (st == UMBIR_STORAGE_BF16) f(std::integral_constant<int, UMBIR_STORAGE_BF16>());
  else f(std::integral_constant<int, UMBIR_STORAGE_F32>());
}
template <typename F>
void with_tiles(int n, F&& f) {
  if (n == 4) f(std::integral_constant<int, 4>());
  else if (n == 2) f(std::integral_constant<int, 2>());
  else f(std::integral_constant<int, 1>());
}

// Sample tiles of 32 per block: four where that leaves a block per CU, else
// two likewise, else one (the waves of a block then share one tile's window).
int moment_tiles(const umbir_geometry& G) {
  const long tt = (G.traces() + 31) / 32;
  return tt * ((G.M + 127) / 128) >= 256 ? 4 : tt * ((G.M + 63) / 64) >= 256 ? 2 : 1;
}

float* phase_image(const umbir_geometry& G, void* fine) {
  return reinterpret_cast<float*>(static_cast<char*>(fine) + G.mom.u_bytes);
}

}  // namespace

bool forward_moments_on(const umbir_geometry& G) { return G.form == 1 && G.split && G.mom.R > 0; }

bool adjoint_moments_on(const umbir_geometry& G) {
  return forward_moments_on(G) && G.storage == UMBIR_STORAGE_F32;
}

bool moments_on(const umbir_geometry& G) { return adjoint_moments_on(G) && G.mom.NG == 1; }

bool abs_moments_on(const umbir_geometry& G) { return moments_on(G) && G.mom.absolute; }

// One scan position reads the image as it is.
float* moment_image(const umbir_geometry& G, void* fine) {
  return G.P == 1 ? nullptr : phase_image(G, fine);
}

int run_phase_image(const umbir_geometry& G, const float* x, void* fine, hipStream_t s) {
  if (G.P == 1 && x) return UMBIR_OK;
  const long n = long(G.nz) * G.mom.pitch * G.mom.Lq;
  UMBIR_LAUNCH("prescale", k_phase_image, dim3(unsigned(std::min<long>((n + 255) / 256, 2048))), dim3(256), 0, s, x,
               G.nx, G.nz, G.P, G.mom, phase_image(G, fine));
  return check_hip(hipGetLastError(), "k_phase_image");
}

int run_forward_moments(const umbir_geometry& G, const float* x, void* out, const void* base, float sign,
                        const float* g, bool abs_op, void* fine, hipStream_t s, bool in_place, const CostFold* fold) {
  int st = UMBIR_OK;
  if (!in_place && (st = run_phase_image(G, x, fine, s))) return st;
  float* u = static_cast<float*>(fine);
  const float* xp = G.P == 1 && x ? x : phase_image(G, fine);
  const int xp_bytes = int(size_t(G.nz) * G.mom.pitch * G.mom.Lq * 4);  // P == 1: the image's own bytes
  if (G.mom.NG > 1) {  // (a forward alone: no fold)
    const MomentShape& ms = G.mom;
    const dim3 grid(unsigned(G.K), unsigned(ms.Ms / kMsBins), unsigned((G.P + 63) / 64 * ms.NG));
    UMBIR_LAUNCH("splat", k_msplat_att, grid, dim3(64 * kMsWaves), msplat_lds<8>(ms.ls), s, xp, xp_bytes, G.mom_start,
                 G.mom_rec4, G.mom_rec_hi, G.P, G.K, G.M, ms, G.mom_span, u);
    // tiles differ in how many templates reach them: four to a block only from two
    // blocks per CU on (at one per CU 276 us, with two tiles to a block 257 at the
    // time)
    const long tt = (G.traces() + 31) / 32;
    const int tiles = moment_tiles(G) == 4 && tt * ((G.M + 127) / 128) < 512 ? 2 : moment_tiles(G);
    with_tiles(tiles, [&](auto nc) {
      constexpr int NTC = decltype(nc)::value;
      const dim3 cgrid(unsigned((G.traces() + 31) / 32), unsigned((G.M + 32 * NTC - 1) / (32 * NTC)));
      UMBIR_LAUNCH("conv", (k_mconv_att<NTC>), cgrid, dim3(64 * kMcWaves), mconv_lds(8, ms.LT, NTC), s, u, ms.Ms,
                   G.mom_taps, ms.LT, G.M, G.Lh, G.traces(), static_cast<const float*>(base), sign, g, G.dbasis,
                   static_cast<float*>(out), MomentTemplates{G.mom_span, ms.NG});
    });
    return check_hip(hipGetLastError(), "attenuated moments");
  }
  const CostFold f = fold ? *fold : CostFold{};
  with_r(G.mom.R, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const unsigned chunks = unsigned((G.P + 63) / 64);
    auto launch = [&](auto bc) {
      constexpr int BINS = decltype(bc)::value;
      const size_t lds = std::max<size_t>(fold ? 256 * sizeof(double) : 0, msplat_lds<R, BINS>(G.mom.ls));
      UMBIR_LAUNCH("splat", (k_msplat<R, BINS>), dim3(unsigned(G.K), unsigned(G.mom.Ms / BINS), chunks),
                   dim3(64 * kMsWaves), lds, s, xp, xp_bytes, G.mom_start, G.mom_rec4, G.mom_rec_hi, G.P, G.K, G.M,
                   G.mom.Ms, G.mom.ls, G.mom.reversed, u, f);
    };
    if (msplat_bins(long(G.K) * (G.mom.Ms / kMsBins) * chunks) == kMsBins)
      launch(std::integral_constant<int, kMsBins>());
    else
      launch(std::integral_constant<int, kMsBinsFew>());
  });
  if ((st = check_hip(hipGetLastError(), "k_msplat"))) return st;
  with_r(G.mom.R, [&](auto rc) {
    with_tiles(moment_tiles(G), [&](auto nc) {
      with_storage(G.storage, [&](auto sc) {
        launch_mconv<decltype(rc)::value, decltype(nc)::value, decltype(sc)::value>(G, u, base, sign, g, abs_op, out, s);
      });
    });
  });
  return check_hip(hipGetLastError(), "k_mconv");
}

int run_adjoint_moments(const umbir_geometry& G, const float* r, bool abs_op, void* fine, float* partial,
                        hipStream_t s) {
  float* v = static_cast<float*>(fine);
  if (G.mom.NG > 1) {
    const MomentShape& ms = G.mom;
    with_tiles(moment_tiles(G), [&](auto nc) {
      constexpr int NT = decltype(nc)::value;
      const dim3 grid(unsigned((G.traces() + 31) / 32), unsigned((ms.Ms / 32 + NT - 1) / NT), unsigned(ms.NG));
      UMBIR_LAUNCH("corr", (k_mcorr_att<NT>), grid, dim3(64 * kMcWaves), mcorr_lds(8, ms.LT), s, r, G.mom_taps, ms.LT,
                   G.M, G.Lh, G.traces(), ms.Ms, ms.NG, G.mom_span, v);
    });
    const int tpg = (G.traces() + G.trace_groups - 1) / G.trace_groups;
    // one generation: at most 1024 blocks (four per CU)
    const int chunk = 256 * kMgAttVpt;
    int nb = (G.voxels() + chunk - 1) / chunk;
    nb = std::max(1, std::min(nb, 1024 / G.trace_groups));
    const int vpb = (G.voxels() + nb - 1) / nb;
    UMBIR_LAUNCH("gather", k_mgather_att, dim3(unsigned(G.trace_groups), unsigned(nb)), dim3(256), 0, s, v, ms, G.nx,
                 G.nz, G.n_off, G.legs, G.gunit, G.tau, G.base, G.P, G.K, log2_int(G.Q), G.M, tpg, vpb, partial);
    return check_hip(hipGetLastError(), "attenuated moments");
  }
  with_r(G.mom.R, [&](auto rc) {
    with_tiles(moment_tiles(G), [&](auto nc) {
      launch_mcorr<decltype(rc)::value, decltype(nc)::value>(G, r, abs_op, v, s);
    });
  });
  int st = check_hip(hipGetLastError(), "k_mcorr");
  if (st) return st;
  const int tpg = (G.traces() + G.trace_groups - 1) / G.trace_groups;
  int tpb;
  const dim3 grid(unsigned(G.trace_groups), unsigned(gather_lds_blocks(G.nx, G.nz, G.trace_groups, &tpb)));
  with_r(G.mom.R, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    UMBIR_LAUNCH("gather", k_mgather<R>, grid, dim3(512), size_t(2) * kMgBufBytes, s, v, G.mom.Ms, G.nx, G.nz,
                 G.n_off, G.legs, G.tau, G.base, G.P, G.K, log2_int(G.Q), G.M, tpg, G.gwin, tpb, partial);
  });
  return check_hip(hipGetLastError(), "k_mgather");
}

// Planes of a trace's moments that an ICD block holds in kIcdMomentLds bytes.
constexpr size_t kIcdMomentLds = 81920;  // two blocks per CU
int icd_planes(const umbir_geometry& G, size_t bytes_per_value) {
  return int(std::min<size_t>(G.mom.R, std::max<size_t>(1, kIcdMomentLds / (bytes_per_value * G.mom.Ms))));
}

int run_icd_dots_moments(const umbir_geometry& G, const float* e, bool abs_op, const IcdGroup& gp, int Sr, int Sc,
                         float* mom, float* partial, hipStream_t s) {
  const int planes = icd_planes(G, sizeof(float));
  const int ych = std::max(1, std::min((gp.size + 1023) / 1024, 512 / std::max(G.traces(), 1)));
  with_r(G.mom.R, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    with_tiles(moment_tiles(G), [&](auto nc) { launch_mcorr<R, decltype(nc)::value>(G, e, abs_op, mom, s); });
    UMBIR_LAUNCH("icd_dots", k_icd_mdots<R>, dim3(unsigned(G.traces()), unsigned(ych)), dim3(1024),
                 size_t(planes) * G.mom.Ms * sizeof(float), s, mom, G.mom.Ms, planes, G.legs, G.n_off, G.tau, G.base,
                 G.P, G.K, log2_int(G.Q), G.M, gp, Sr, Sc, partial);
  });
  return check_hip(hipGetLastError(), "icd moment dots");
}

int run_icd_update_moments(const umbir_geometry& G, bool abs_op, const IcdGroup& gp, int Sr, int Sc,
                           const float* delta, float* mom, const float* base, float* e, hipStream_t s) {
  const int planes = icd_planes(G, sizeof(unsigned long long));
  with_r(G.mom.R, [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    UMBIR_LAUNCH("icd_scatter", k_icd_msplat<R>, dim3(unsigned(G.traces())), dim3(1024),
                 size_t(planes) * G.mom.Ms * sizeof(unsigned long long), s, mom, G.mom.Ms, planes, G.legs, G.n_off,
                 G.tau, G.base, G.P, G.K, log2_int(G.Q), G.M, gp, Sr, Sc, delta);
    with_tiles(moment_tiles(G), [&](auto nc) {
      launch_mconv<R, decltype(nc)::value, UMBIR_STORAGE_F32>(G, mom, base, -1.0f, nullptr, abs_op, e, s);
    });
  });
  return check_hip(hipGetLastError(), "icd moment update");
}

void plan_moments(const umbir_geometry& G, int pi, BatchProb& bp, std::vector<int4>* items, size_t* lds) {
  const MomentShape& ms = G.mom;
  bp.mom = ms;
  bp.mom_start = G.mom_start;
  bp.mom_rec4 = G.mom_rec4;
  bp.mom_rec_hi = G.mom_rec_hi;
  bp.mom_taps = G.mom_taps;
  bp.mom_tiles = moment_tiles(G);
  const int tt = (G.traces() + 31) / 32, nt = bp.mom_tiles;
  auto grow = [&](int stage, size_t bytes) { lds[stage] = std::max(lds[stage], bytes); };
  with_r(ms.R, [&](auto rc) { grow(kStMSplat, msplat_lds<decltype(rc)::value>(ms.ls)); });
  grow(kStMConv, mconv_lds(ms.R, ms.LT, nt));
  grow(kStMCorr, mcorr_lds(ms.R, ms.LT));
  grow(kStMGather, size_t(2) * kMgBufBytes);
  for (int z = 0; z < (G.P + 63) / 64; ++z)
    for (int y = 0; y < ms.Ms / kMsBins; ++y)
      for (int j = 0; j < G.K; ++j) items[kStMSplat].push_back(make_int4(pi, j, y, z));
  for (int y = 0; y < (G.M + 32 * nt - 1) / (32 * nt); ++y)
    for (int x = 0; x < tt; ++x) items[kStMConv].push_back(make_int4(pi, x, y, 0));
  for (int y = 0; y < (ms.Ms / 32 + nt - 1) / nt; ++y)
    for (int x = 0; x < tt; ++x) items[kStMCorr].push_back(make_int4(pi, x, y, 0));
  const int nb = gather_lds_blocks(G.nx, G.nz, G.trace_groups, &bp.vpb);
  for (int y = 0; y < nb; ++y)
    for (int x = 0; x < G.trace_groups; ++x) items[kStMGather].push_back(make_int4(pi, x, y, 0));
}

int launch_moment_stage(int stage, const BatchProb* probs, const int* active, const StageLaunch& L, int which,
                        hipStream_t s) {
  const dim3 grid(unsigned(L.grid));
  if (stage == kStMSplat)
    UMBIR_LAUNCH("splat", k_msplat_list, grid, dim3(64 * kMsWaves), L.lds, s, probs, active, L.items, L.n_items, which);
  else if (stage == kStMConv)
    UMBIR_LAUNCH("conv", k_mconv_list, grid, dim3(64 * kMcWaves), L.lds, s, probs, active, L.items, L.n_items);
  else if (stage == kStMCorr)
    UMBIR_LAUNCH("corr", k_mcorr_list, grid, dim3(64 * kMcWaves), L.lds, s, probs, active, L.items, L.n_items);
  else
    UMBIR_LAUNCH("gather", k_mgather_list, grid, dim3(512), L.lds, s, probs, active, L.items, L.n_items);
  return check_hip(hipGetLastError(), "moment work-list stage");
}

// ---- which geometries take the moment form

// |f^(R)| a^R / (R! 2^(R-1)) bounds the remainder of a degree R - 1 fit at the
// Chebyshev points over a half-width a; f's derivatives by its spectrum
// (a Gaussian of width 1 / (2 pi sigma_t) around f_c, unit mass for a pulse of
// unit peak).  The least-squares fit on Q + 1 equispaced points stays within
// a small factor of it.
static double fit_remainder(double f_c, double sigma_t, double half_width, int R) {
  const double sf = 1.0 / (2.0 * M_PI * sigma_t);
  double mean = 0.0, mass = 0.0;
  for (int k = -60; k <= 60; ++k) {  // E (2 pi f a)^R over +- 6 sigma_f
    const double z = 0.1 * k, w = std::exp(-0.5 * z * z);
    mean += w * std::pow(std::fabs(2.0 * M_PI * (f_c + z * sf) * half_width), R);
    mass += w;
  }
  double scale = 1.0;
  for (int k = 2; k <= R; ++k) scale *= k;
  return mean / mass / (scale * std::pow(2.0, R - 1));
}

MomentShape moment_shape(const MomentInput& in) {
  MomentShape ms;
  const int Q = in.Q;
  // the dense part pays from Q >= 2 R on; longer records, or more bins than the
  // plan's grid holds, keep the fine grid
  if (Q < 16 || in.M > 16384 || long(in.M) * in.n_gamma > 262140) return ms;
  // the window must end where the pulse is (numerically) zero: the table's
  // forced zeros at its ends are then no step
  const double tc = 0.5 * in.t_win;
  if (std::fabs(std::sin(2.0 * M_PI * in.f_c * tc)) * std::exp(-tc * tc / (2.0 * in.sigma_t * in.sigma_t)) > 1e-9)
    return ms;
  // 8 moments (a 2 MHz pulse at 20 MHz), 512 traces of 2048 samples at 256 x 256,
  // against the fine grid: forward 62 for 153 us, adjoint 140 for 143, an
  // iteration of both 204 for 294
  int R = 0;
  for (int c : {5, 6, 8})
    if (!R && 2 * c <= Q && fit_remainder(in.f_c, in.sigma_t, 0.5 / in.fs, c) <= 1e-8) R = c;
  if (in.n_gamma > 1) {
    // six coefficients (an attenuated response is smoother than the pulse, so
    // the same remainder relative to its own, smaller peak) and the two ends
    if (Q < 16 || in.Lh < 2 || in.storage != UMBIR_STORAGE_F32 ||
        fit_remainder(in.f_c, in.sigma_t, 0.5 / in.fs, 6) > 1e-8)
      return ms;
    R = 8;
  }
  if (!R) return ms;
  // scan positions a constant whole number of voxels apart
  const int P = in.P, K = in.K;
  long pitch = 1;
  if (P > 1) {
    const long d = long(in.base[0]) - in.base[1];  // 2 x voxels to the right
    if (d == 0 || d % 2) return ms;
    for (int i = 0; i < P; ++i) {
      if (long(in.base[0]) - in.base[i] != d * i) return ms;
      for (int j = 0; j < K; ++j)
        if (long(in.base[P + j]) - in.base[P + size_t(i) * K + j] != d * i) return ms;
    }
    pitch = std::labs(d / 2);
    ms.reversed = d < 0;
  }
  const double NR = double(in.nx) + double(pitch) * (P - 1);
  const double Lq = std::ceil(double(in.nx) / pitch) + 2.0 * (P - 1);
  const double recs = double(K) * in.nz * NR;
  if (recs * 4.0 * (R + 1) > 4e9 || recs > 1e9 || double(in.nz) * pitch * Lq > 1e8) return ms;
  // the plan's grid, and its histogram of one receiver
  const double chunks = std::ceil(NR / kPlanChunk);
  if (chunks > 65535 || chunks * in.M * in.n_gamma * 4.0 > double(kPlanCountBytes)) return ms;
  const int LT = in.Lh + 9;
  if (size_t(R) * 3 * LT * 16 > 150u * 1024 || double(K) * in.M * in.n_gamma > 6.4e7) return ms;
  if (in.n_gamma == 1 && gather_window_bytes(in.nx, in.nz, long(P) * K, long(in.M) * Q, in.storage) == 0) return ms;
  ms.R = R;
  ms.NG = in.n_gamma;
  // |A|: the weights are not negative (an even power of the cosine), and the
  // pulse's sign changes fall on samples
  const double half = in.fs / (2.0 * in.f_c), mid = tc * in.fs;
  ms.absolute = in.n_gamma == 1 && in.beta % 2 == 0 && std::fabs(half - std::round(half)) < 1e-9 * half &&
                std::fabs(mid - std::round(mid)) < 1e-9 * mid;
  ms.Ms = (in.M + 31) & ~31;
  ms.LT = LT;
  ms.pitch = int(pitch);
  ms.Lq = int(Lq);
  ms.NR = int(NR);
  ms.rel0 = -int(pitch) * (P - 1);
  ms.ls = 2;
  while ((1 << ms.ls) < P && ms.ls < 6) ++ms.ls;
  ms.u_bytes = (size_t(ms.NG) * P * K * R * ms.Ms * 4 + 255) & ~size_t(255);
  // the image by phase, and the lanes past the last scan position of it
  ms.work_bytes = ms.u_bytes + (size_t(in.nz) * ms.pitch * ms.Lq * 4 + 255 & ~size_t(255));
  ms.records = size_t(K) * in.nz * ms.NR;
  // one allocation: rec4, rec_hi, taps, start, span
  auto place = [&](size_t bytes) {
    const size_t at = ms.table_bytes;
    ms.table_bytes += (bytes + 255) & ~size_t(255);
    return at;
  };
  (void)place(ms.records * sizeof(float4));
  ms.hi_at = place(ms.records * (R - 3) * sizeof(float));
  ms.taps_at = place((1 + ms.absolute) * ms.taps_words() * sizeof(uint4));
  ms.start_at = place(size_t(K) * (size_t(ms.NG) * in.M + 1) * sizeof(int));
  ms.span_at = place(size_t(ms.NG) * sizeof(int2));
  return ms;
}

// Least-squares fit of degree R - 1 on z_t = 2 t / Q - 1, t = 0 .. Q: the
// R x (Q + 1) matrix taking the values to the coefficients (normal equations
// by Gaussian elimination with pivoting; they are well conditioned at R <= 8).
// Point `skip` is left out.
static std::vector<double> fit_matrix(int R, int Q, int skip = -1) {
  std::vector<double> V(size_t(R) * (Q + 1)), A(size_t(R) * R, 0.0);
  for (int t = 0; t <= Q; ++t) {
    double z = 2.0 * t / Q - 1.0, p = 1.0;
    for (int k = 0; k < R; ++k, p *= z) V[size_t(k) * (Q + 1) + t] = t == skip ? 0.0 : p;
  }
  for (int a = 0; a < R; ++a)
    for (int b = 0; b < R; ++b)
      for (int t = 0; t <= Q; ++t) A[a * R + b] += V[size_t(a) * (Q + 1) + t] * V[size_t(b) * (Q + 1) + t];
  for (int c = 0; c < R; ++c) {
    int piv = c;
    for (int r = c + 1; r < R; ++r)
      if (std::fabs(A[r * R + c]) > std::fabs(A[piv * R + c])) piv = r;
    if (piv != c) {
      for (int k = 0; k < R; ++k) std::swap(A[c * R + k], A[piv * R + k]);
      for (int t = 0; t <= Q; ++t) std::swap(V[size_t(c) * (Q + 1) + t], V[size_t(piv) * (Q + 1) + t]);
    }
    for (int r = 0; r < R; ++r) {
      if (r == c) continue;
      const double f = A[r * R + c] / A[c * R + c];
      for (int k = c; k < R; ++k) A[r * R + k] -= f * A[c * R + k];
      for (int t = 0; t <= Q; ++t) V[size_t(r) * (Q + 1) + t] -= f * V[size_t(c) * (Q + 1) + t];
    }
  }
  for (int r = 0; r < R; ++r)
    for (int t = 0; t <= Q; ++t) V[size_t(r) * (Q + 1) + t] /= A[r * R + r];
  return V;
}

// Queues the plan's kernels (G's legs, bases and tau are queued before on s);
// scratch (a word per record, kPlanCountBytes of histograms at most, small
// tables) is allocated and freed in stream order, *max_bin (a host word that
// lives until the stream was synchronized) receives the largest bin.
// UMBIR_ENOMEM: nothing was queued.
int build_moments(umbir_geometry* G, int* max_bin, hipStream_t s) {
  const MomentShape& ms = G->mom;
  const int R = ms.R, K = G->K, M = G->M, Q = G->Q;
  const int chunks = (ms.NR + kPlanChunk - 1) / kPlanChunk;
  const int NB = ms.NG * M;
  const size_t count_row = size_t(chunks) * NB;  // of one receiver
  const int part = int(std::min<size_t>(K, std::max<size_t>(1, kPlanCountBytes / sizeof(int) / count_row)));
  std::vector<double> fit = fit_matrix(ms.NG > 1 ? 6 : R, Q);
  if (ms.NG > 1)
    for (int skip : {Q, 0}) {
      const std::vector<double> f = fit_matrix(6, Q, skip);
      fit.insert(fit.end(), f.begin(), f.end());
    }
  const size_t fit_bytes = (fit.size() * sizeof(double) + 255) & ~size_t(255);
  const size_t count_bytes = (part * count_row * sizeof(int) + 255) & ~size_t(255);
  const int g_rows = ms.NG * R * (1 + ms.absolute);
  const size_t g_bytes = (size_t(g_rows) * G->Lh * sizeof(float) + 255) & ~size_t(255);
  char* tmp = nullptr;
  int st = check_hip(hipMallocAsync(reinterpret_cast<void**>(&tmp),
                                    fit_bytes + 256 + g_bytes + count_bytes + ms.records * sizeof(unsigned), s),
                     "hipMallocAsync(plan)");
  if (st) return st;
  double* fit_dev = reinterpret_cast<double*>(tmp);
  int* mb = reinterpret_cast<int*>(tmp + fit_bytes);
  float* g = reinterpret_cast<float*>(tmp + fit_bytes + 256);
  int* counts = reinterpret_cast<int*>(tmp + fit_bytes + 256 + g_bytes);
  unsigned* keys = reinterpret_cast<unsigned*>(tmp + fit_bytes + 256 + g_bytes + count_bytes);
  const int cap = G->nz * ms.NR;
  const size_t lds = size_t(std::min(NB, kPlanSlice)) * sizeof(int);
  const unsigned slices = unsigned((NB + kPlanSlice - 1) / kPlanSlice);
  if (!(st = check_hip(hipMemcpyAsync(fit_dev, fit.data(), fit.size() * sizeof(double), hipMemcpyHostToDevice, s),
                       "hipMemcpyAsync(fit)"))) {
    if (ms.NG > 1)
      UMBIR_LAUNCH("moment_fit", k_template_fit, dim3(unsigned((G->Lh + 3) / 4), unsigned(ms.NG)), dim3(256), 0, s, Q,
                   G->Lh, G->bank, fit_dev, g);
    else
      UMBIR_LAUNCH("moment_fit", k_moment_fit, dim3(unsigned((G->Lh + 3) / 4)), dim3(256), 0, s, R, Q, G->Lh,
                   1.0 / (double(Q) * G->fs), G->f_c, 1.0 / (2.0 * G->sigma_t * G->sigma_t), 0.5 * G->t_win, fit_dev, ms.absolute, g);
    // (the templates' rows, and those of |b|, follow one another in g and in the table)
    UMBIR_LAUNCH("moment_table", k_moment_table, dim3(unsigned((g_rows * ms.LT + 255) / 256)), dim3(256), 0, s,
                 g_rows, G->Lh, ms.LT, g, G->mom_taps, mb);
    for (int j0 = 0; j0 < K; j0 += part) {
      const dim3 cg{unsigned(std::min(part, K - j0)), unsigned(chunks), slices};
      UMBIR_LAUNCH("plan_count", k_plan_count, cg, dim3(1024), lds, s, G->legs, G->gunit, G->base, ms, G->P, K, j0,
                   G->nz, G->n_off, M, counts);
      UMBIR_LAUNCH("plan_scan", k_plan_scan, dim3(cg.x), dim3(1024), 0, s, NB, chunks, cap, j0, counts, G->mom_start,
                   mb);
      UMBIR_LAUNCH("plan_fill", k_plan_fill, cg, dim3(512), lds, s, G->legs, G->gunit, G->base, ms, G->P, K, j0, G->nz,
                   G->n_off, M, counts, keys);
    }
    if (ms.NG > 1)
      UMBIR_LAUNCH("plan_span", k_plan_span, dim3(unsigned(ms.NG)), dim3(256), 0, s, G->mom_start, K, M, NB, G->mom_span);
    with_r(R, [&](auto rc) {
      UMBIR_LAUNCH("plan_emit", k_plan_emit<decltype(rc)::value>, dim3(unsigned(K), unsigned((NB + 3) / 4)), dim3(256),
                   0, s, G->legs, G->base, G->tau, ms, G->P, K, G->n_off, log2_int(Q), NB, G->mom_start, keys, mb,
                   G->mom_rec4, G->mom_rec_hi);
    });
    st = check_hip(hipGetLastError(), "moment plan");
    if (!st) st = check_hip(hipMemcpyAsync(max_bin, mb, sizeof(int), hipMemcpyDeviceToHost, s), "hipMemcpyAsync");
  }
  (void)hipFreeAsync(tmp, s);
  return st;
}

bool moment_plan_fits(int max_bin) { return max_bin <= kMaxBin; }

}  // namespace umbir
