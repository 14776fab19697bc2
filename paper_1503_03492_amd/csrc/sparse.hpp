// sparse.hpp -- gfx950 device code of a region's sweep that visits only the
// rounds that can change something.
//
// A window whose increments are zero and whose sum of squares is within its
// bound is left exactly as it is by Algorithm 2 (y = x, t = 1, x' = x, I' = 0),
// and on the images this library is for nearly all windows are in that state
// nearly all of the time: 0.7% of the (window, pixel) units of a 1024 x 1024
// fluorescence frame with sides 1..16 did anything in its first sweep, 0.05%
// in its tenth.  Streaming every increment through the chip (12.3 GB a sweep at
// that size) then is the cost of the sweep, so this job
//   - keeps one "live" bit per round (round: the windows a wave projects
//     together, kernels.hpp): set when an increment of the round may be
//     non-zero.  Increments of rounds whose bit is clear are zero, in memory
//     too, and are not read;
//   - tests all windows of a side at once, from the footprint in LDS, before it
//     visits the side (window_test), and visits in the usual order the rounds
//     that are live or hold a window that might exceed its bound;
//   - repeats the test after a round that changed pixels, for the rounds still
//     to come.
// A visited round does the arithmetic of run_side, in its order, so the result
// is the one of the full visit, bit for bit (but for the sign of zeros).
//
// The test may say "might exceed" of a window that does not (the visit then
// changes nothing), never the reverse.  It compares an FP32 sum with
// r2 (1 - kTestMargin).  All terms are positive, so a sum is within its longest chain
// of roundings of the exact one: test_all carries one sum through all sides (S (S + 3) / 2
// roundings up to side S, 560 at side 32, 3.4e-5), window_test adds 2 S values; a visit's
// own FP32 sum comes on top (below 50 roundings).  A static_assert ties the margin to
// that.
//
// Workgroup = 3 waves: wave 0 (consumer) tests and projects; wave 1 (loader)
// walks the live rounds in visiting order ahead of it and puts their increments
// into a ring of LDS slots, one slot per round; wave 2 (writer) stores the
// updated increments that the consumer left in a second ring, and shares the
// first test with the consumer.  They pass rounds
// on through LDS counters; every wait is bounded, as in region_job.
//
// A side more than half of whose rounds are live is visited round by round
// without tests (a test costs about as much as a visit).  A region more than about a
// quarter of whose rounds are live goes through region_job, which streams whole pages,
// for kDenseSweeps - 1 sweeps, after which a sweep that takes every round for live finds
// the live ones again.  us per sweep of 512 x 512 noise, visited and streamed: sides
// 1..8, share of live rounds 0.14: 260 and 350, 0.25: 376 and 350, 0.34: 432 and 350;
// BF16 increments 0.25: 385 and 376; FP64 0.25: 428 and 445; region side 8 0.22: 338
// and 338.
//
// Measured, us per sweep with its check, a full visit against this: 512 x 512
// sides 1..8, 338 against 158 (264 in the first sweep, 133 in the last of 120);
// 1024 x 1024 sides 1..16, 2550 against 250 (1142, 183).  What bounds it: the chain
// of visits of the slowest region, and instruction fetch (the code of a side, about
// 4 KB, runs for a few rounds per job).
#pragma once

#include "kernels.hpp"
#include "growth.hpp"

namespace smre {

constexpr int kPhaseThreads = 192;  // consumer, loader, writer
constexpr float kTestMargin = 1e-4f;
// Roundings between a sum of the test and the sum a visit decides by: test_all's chain,
// a pixel's conversion from FP64 (twice in its square), the product r2 (1 - margin), and
// the visit's own chain.
constexpr int kTestRoundings = 32 * (32 + 3) / 2 + 2 + 3 + 50;
static_assert(kTestRoundings * (1.0 / (1 << 24)) < 0.5 * kTestMargin, "the test's margin");
// A wait here lasts while the consumer tests and visits rounds that need nothing
// from the ring (a region of side 32 has up to 32768 rounds): ~1 s of sleeps.
constexpr int kSparseSpin = 1 << 24;
constexpr int kDenseSweeps = 32;  // head word of a region that goes over to streaming

// Live bits of a region in HBM: kLiveHead words (word 0: 0 = sparse, 1 = sparse
// with every round taken for live, h > 1 = page streaming for h - 1 sweeps more),
// then live_words(R) words per side.
constexpr int kLiveHead = 4;
__host__ __device__ constexpr int live_words(int R) { return R * R / 32; }

// Rounds of side s in a region with all its anchors: those along an axis, squared.
__host__ __device__ constexpr int block_side(int R, int s) {  // BR = BC of pattern(R, s)
  return R == 8 ? (s <= 1 ? 8 : s <= 3 ? 4 : s <= 7 ? 2 : 1)
       : R == 16 ? (s <= 3 ? 8 : s <= 6 ? 4 : s <= 12 ? 2 : 1)
                 : (s <= 5 ? 8 : s <= 8 ? 4 : s <= 16 ? 2 : 1);
}
__host__ __device__ constexpr int axis_rounds(int R, int s) {
  const int b = block_side(R, s), n = (R + s - 1) / s, a = s < R ? s : R;
  const int rest = R - (n - 1) * s, f = rest < a ? rest : a;
  return f * ((n + b - 1) / b) + (a - f) * ((n - 1 + b - 1) / b);
}
constexpr bool axis_rounds_agree() {
  bool ok = true;
  for (int R = 8; R <= 32; R *= 2)
    for (int s = 1; s <= R + 1 && s <= 32; ++s)
      ok = ok && block_side(R, s) == pattern(R, s).br && block_side(R, s) == pattern(R, s).bc;
  return ok;
}
static_assert(axis_rounds_agree(), "block_side follows pattern");

// Numbering of a side's rounds in visiting order: offsets (ap, bp) raster, then
// blocks (rby, rbx) of BR x BC windows, counted for a region with all R x R
// anchors (in a region cut by the image border some numbers have no round).
// Along an axis, offset a has NRM windows if a < F, else NRM - 1.
template <int R, int S> struct Rounds {
  using SS = SideShape<R, S>;
  static constexpr int BR = SS::BR, BC = SS::BC, NRM = SS::NRM;
  static constexpr int A = S < R ? S : R;  // offsets along an axis
  static constexpr int F = (R - (NRM - 1) * S) < A ? (R - (NRM - 1) * S) : A;
  static constexpr int RB1 = (NRM + BR - 1) / BR, RB2 = F == A ? RB1 : (NRM - 1 + BR - 1) / BR;
  static constexpr int CB1 = (NRM + BC - 1) / BC, CB2 = F == A ? CB1 : (NRM - 1 + BC - 1) / BC;
  static constexpr int CT = F * CB1 + (A - F) * CB2;
  static constexpr int N = (F * RB1 + (A - F) * RB2) * CT;
  static_assert(N <= R * R, "a live bit per round");
  static_assert(N == axis_rounds(R, S) * axis_rounds(R, S), "rounds of a side");

  // number of the round that holds the window anchored at (i, j)
  static __host__ __device__ __forceinline__ int of_window(int i, int j) {
    const int ap = i % S, rby = i / S / BR, bp = j % S, rbx = j / S / BC;
    const int rbn = ap < F ? RB1 : RB2, cbn = bp < F ? CB1 : CB2;
    const int pr = ap < F ? ap * RB1 : F * RB1 + (ap - F) * RB2;
    const int pc = bp < F ? bp * CB1 : F * CB1 + (bp - F) * CB2;
    return pr * CT + rbn * pc + rby * cbn + rbx;
  }

  int ap, bp, rby, rbx;
  int nbr, nbc;  // windows of the round; none when one of them is not positive
  int before;    // windows of the side visited before the round

  // round `id` of a region with rhi x chi anchors
  __host__ __device__ __forceinline__ Rounds(int id, int rhi, int chi) {
    int r, rbn = RB1, cbn = CB1;
    if (RB1 == RB2 || id < F * RB1 * CT) {
      ap = id / (RB1 * CT);
      r = id - ap * (RB1 * CT);
    } else {
      const int t = id - F * RB1 * CT, a = t / (RB2 * CT);
      ap = F + a;
      r = t - a * (RB2 * CT);
      rbn = RB2;
    }
    const int full = F * rbn * CB1;  // rounds of the offsets bp < F
    if (CB1 == CB2 || r < full) {
      bp = rbn == RB1 ? r / (RB1 * CB1) : r / (RB2 * CB1);
      r -= bp * (rbn * CB1);
    } else {
      r -= full;
      const int b = rbn == RB1 ? r / (RB1 * CB2) : r / (RB2 * CB2);
      bp = F + b;
      r -= b * (rbn * CB2);
      cbn = CB2;
    }
    rby = cbn == CB1 ? r / CB1 : r / CB2;
    rbx = r - rby * cbn;
    const int nr = (rhi - ap + S - 1) / S, nc = (chi - bp + S - 1) / S;
    nbr = ap < rhi ? nr - rby * BR : 0;
    nbc = bp < chi ? nc - rbx * BC : 0;
    nbr = nbr < BR ? nbr : BR;
    nbc = nbc < BC ? nbc : BC;
    before = windows_before(ap, rhi) * chi + nr * windows_before(bp, chi) + rby * BR * nc +
             nbr * (rbx * BC);
  }
  __host__ __device__ __forceinline__ bool exists() const { return nbr > 0 && nbc > 0; }

 private:
  // windows along an axis of n anchors with offset below a
  static __host__ __device__ __forceinline__ int windows_before(int a, int n) {
    const int m = (n + S - 1) / S, f = n - (m - 1) * S;
    return a <= f ? a * m : f * m + (a - f) * (m - 1);
  }
};

template <typename TX, typename TQ, int R, int SMAX> struct SparseLds {
  using SH = PhaseShape<TX, TQ, R, SMAX>;
  static constexpr int ES = (int)sizeof(TQ);
  static constexpr int NW = live_words(R);
  static constexpr int NWM = R * R / 64;  // window masks per side
  // a slot holds the largest round, read by all lanes, and the 0..3 bytes by
  // which a round may start off a 4-byte boundary
  static constexpr int max_elem() {
    int m = 0;
    for (int s = 1; s <= SMAX; ++s) {
      const Pattern p = pattern(R, s);
      const int e = p.br * p.bc * s * s + p.gr * p.gc;
      if (e > m) m = e;
    }
    return m;
  }
  static constexpr int SLOT = (max_elem() * ES + 4 + 15) / 16 * 16;
  static constexpr int NIN = SLOT <= 4096 ? 5 : SLOT <= 8192 ? 4 : 2;
  static constexpr int NOUT = SLOT <= 4096 ? 2 : SLOT <= 8192 ? 2 : 1;
  static constexpr int ODUMMY = NOUT * SLOT;  // targets of masked lanes' writes
  static constexpr int LW = R == 8 ? 16 : R == 16 ? 32 : 64;  // footprint columns, padded
  static constexpr int VP = LW + 4;
  // (the same bytes hold the masked lanes' writes and, at other times, the
  // column sums of window_test)
  static constexpr int DUMMY = SH::RING - SH::QD, VSUMS = R * VP * (int)sizeof(float);
  static constexpr int OBYTES = ODUMMY + (DUMMY > VSUMS ? DUMMY : VSUMS);
  __device__ __forceinline__ float* vs() { return (float*)(out + ODUMMY); }

  // (first: the loader's loads take their LDS address from 16 bits)
  __align__(16) unsigned char in[NIN * SLOT];
  TX xs[SH::XSIZE];
  __align__(16) unsigned char out[OBYTES];
  __align__(8) uint64_t win[SMAX + 1][NWM];  // by side: windows that may exceed the bound
  double r2d[40];                         // by side: bounds, test bound
  float r2f[40], rf[40], thr[64];
  float top[2][64];                       // by side: largest sum below the test bound, per wave
  int base[64], index[64], flag[64];      // by side: first increment byte, k (-1: none), win != 0
  int side[40];                           // by k
  uint32_t need[NW];                      // rounds that window_test flags
  uint32_t live[SMAX * NW];               // live bits at the start of the job, by k
  uint32_t now[SMAX * NW];                // and at its end
  __align__(8) int2 odesc[4];             // a round given to the writer: first byte, bytes
  int rounds;                             // of the region, about
  int head;                               // its head word after the job
  int tested, in_ready, in_done, out_ready, out_done, finished, abort, changed;
};

// Sums of S consecutive values t[j] .. t[j + S - 1] for j < N: suffix sums within
// blocks of S plus prefix sums of the next block (3 adds a value, none of them a
// difference).
template <int S, int N> __device__ __forceinline__ void running_sums(const float* t, float* out) {
  constexpr int M = N + S - 1;
  float pre[M];
#pragma unroll
  for (int i = 0; i < M; ++i) pre[i] = (i % S == 0) ? t[i] : pre[i - 1] + t[i];
  float suf = 0.0f;
#pragma unroll
  for (int j = M - 1; j >= 0; --j) {
    // suffix sum of t[j] .. end of its block (only full blocks are used)
    suf = (j % S == S - 1 || j == M - 1) ? t[j] : suf + t[j];
    if (j < N) out[j] = (j % S == 0) ? pre[j + S - 1] : suf + pre[j + S - 1];
  }
}

// Largest of a non-negative value over the wave (not a number: ignored).
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f(v, 0xB1));
  v = fmaxf(v, dpp_f(v, 0x4E));
  v = fmaxf(v, dpp_f(v, 0x141));
  v = fmaxf(v, dpp_f(v, 0x140));
  auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
  v = fmaxf(__int_as_float(p[0]), __int_as_float(p[1]));
  auto q = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  return fmaxf(__int_as_float(q[0]), __int_as_float(q[1]));
}

// Largest over the wave of 16 values at once, halving the number of values a lane
// holds at each exchange: lane l ends with the maximum of
// v[8 l3 + 4 l2 + 2 l1 + l0] (l3..l0: the low bits of l).
__device__ __forceinline__ float wave_max16(const float (&v)[16], int lane) {
  float a[8], b[4], c[2];
  const bool l3 = lane & 8, l2 = lane & 4, l1 = lane & 2, l0 = lane & 1;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    a[i] = fmaxf(l3 ? v[8 + i] : v[i], dpp_f(l3 ? v[i] : v[8 + i], 0x140));
#pragma unroll
  for (int i = 0; i < 4; ++i)
    b[i] = fmaxf(l2 ? a[4 + i] : a[i], dpp_f(l2 ? a[i] : a[4 + i], 0x141));
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = fmaxf(l1 ? b[2 + i] : b[i], dpp_f(l1 ? b[i] : b[2 + i], 0x4E));
  float d = fmaxf(l0 ? c[1] : c[0], dpp_f(l0 ? c[0] : c[1], 0xB1));
  auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(d), __float_as_int(d), false, false);
  d = fmaxf(__int_as_float(p[0]), __int_as_float(p[1]));
  auto q = __builtin_amdgcn_permlane32_swap(__float_as_int(d), __float_as_int(d), false, false);
  return fmaxf(__int_as_float(q[0]), __int_as_float(q[1]));
}

// Test of every window of every side at the start of a job, by two waves:
// a lane owns a window position and grows its window by one row and one column
// at a time (each pixel of the largest window is read once), so all sides cost
// one read and one FMA per pixel of the largest.  The sums of 8 sides at a time
// are taken without a branch between them: with one per side every read waited
// for the one before (16 sides 4.4 us more than one side; 2.8 us now).  Leaves by side the mask of the
// windows that might exceed the bound (masks are zero before) and the largest
// sum below it.
template <typename TX, typename TQ, int R, int SMAX>
__device__ __forceinline__ void test_all(SparseLds<TX, TQ, R, SMAX>& L, int wave, int lane,
                                         int h, int w, int smax) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  constexpr int P = SL::SH::P, SM = SMAX < 32 ? SMAX : 32;
  const int thr = __float_as_int(L.thr[lane]);  // of side `lane`
  for (int g = wave; g < SL::NWM; g += 2) {
    const int i = (g * 64 + lane) / R, j = (g * 64 + lane) % R;
    const int fit = min(h - i, w - j);  // largest window that lies in the image
    const TX* p = L.xs + i * P + j;
    float n = 0.0f;
#pragma unroll
    for (int s0 = 0; s0 < SM; s0 += 16) {
      if (s0 >= smax) break;
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = 0.0f;
#pragma unroll
      for (int s1 = s0; s1 < s0 + 16 && s1 < SM; s1 += 8)
        if (s1 < smax) {
#pragma unroll
          for (int s = s1 + 1; s <= s1 + 8 && s <= SM; ++s) {
            float r = 0.0f;
#pragma unroll
            for (int l = 0; l < s; ++l) {
              const float f = (float)p[(s - 1) * P + l];
              n = __builtin_fmaf(f, f, n);
              if (l < s - 1) {
                const float e = (float)p[l * P + s - 1];
                r = __builtin_fmaf(e, e, r);
              }
            }
            n += r;
            v[s - s0 - 1] = n;
            // (a bound on the reads in flight, thus on their registers)
            if (s >= 8) __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
      for (int s = s0 + 1; s <= s0 + 16 && s <= SM; ++s) {
        float& sum = v[s - s0 - 1];
        const bool over = s <= fit && !(sum < __int_as_float(__builtin_amdgcn_readlane(thr, s)));
        const uint64_t m = __ballot(over);
        if (m != 0 && s <= smax) {
          L.win[s][g] = m;
          L.flag[s] = 1;
        }
        sum = over || s > fit ? 0.0f : sum;
      }
      const float t = wave_max16(v, lane);
      if (lane < 16) {
        // (one wave may own several masks of a side)
        float& o = L.top[wave][s0 + 1 + lane];
        o = g == wave ? t : fmaxf(o, t);
      }
    }
  }
  __asm__ volatile("" ::: "memory");
  if (lane == 0)
    __hip_atomic_fetch_add(&L.tested, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct Sparse {
  int h, w;        // image rows and columns from the region's origin on
  float guard;
  int lane;
  int in_seq, in_seen, in_off;     // live rounds taken from the ring, loaded; next slot
  int out_seq, out_seen, out_off;  // rounds given to the writer, written; next slot
  int nlive;       // rounds live at the end
  Growth grown;    // lane's part of the growth of x^2 summed over pixels
};

// Test of every window of side S against its bound, from the footprint: the
// bits (by lane: word `lane`) of the rounds that hold a window that might exceed
// it, and the largest sum of the others.  Lanes own footprint columns for the
// column sums, then runs of windows of a row for the row sums of those.
template <typename TX, typename TQ, int R, int SMAX, int S>
__device__ __forceinline__ uint32_t window_test(SparseLds<TX, TQ, R, SMAX>& L, int lane, int rhi,
                                                int chi, float thr, float* top) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  constexpr int LW = SL::LW, VP = SL::VP, NW = SL::NW, P = SL::SH::P;
  constexpr int NG = 64 / LW, NR = R / NG;
  constexpr int WPL = R * R / 64, LPR = R / WPL;
  {
    const int col = lane % LW, g = lane / LW;
    const TX* p = L.xs + g * NR * P + col;
    float t[NR + S - 1], v[NR];
#pragma unroll
    for (int i = 0; i < NR + S - 1; ++i) {
      const float f = (float)p[i * P];
      t[i] = f * f;
    }
    running_sums<S, NR>(t, v);
#pragma unroll
    for (int j = 0; j < NR; ++j) L.vs()[(g * NR + j) * VP + col] = v[j];
  }
  __asm__ volatile("" ::: "memory");
  const int row = lane / LPR, c0 = (lane % LPR) * WPL;
  float u[WPL + S - 1], n[WPL];
#pragma unroll
  for (int i = 0; i < WPL + S - 1; ++i) u[i] = L.vs()[row * VP + c0 + i];
  running_sums<S, WPL>(u, n);
  bool over[WPL], any = false;
  float best = 0.0f;
#pragma unroll
  for (int w = 0; w < WPL; ++w) {
    const bool is = row < rhi && c0 + w < chi;
    over[w] = is && !(n[w] < thr);
    any |= over[w];
    best = fmaxf(best, is && !over[w] ? n[w] : 0.0f);
  }
  *top = wave_max(best);
  if (__ballot(any) == 0) return 0;
  if (lane < NW) L.need[lane] = 0;
  __asm__ volatile("" ::: "memory");
#pragma unroll
  for (int w = 0; w < WPL; ++w)
    if (over[w]) {
      const int id = Rounds<R, S>::of_window(row, c0 + w);
      __hip_atomic_fetch_or(&L.need[id >> 5], 1u << (id & 31), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  __asm__ volatile("" ::: "memory");
  return lane < NW ? L.need[lane] : 0;
}

// The same bits from the masks test_all left.
template <typename TX, typename TQ, int R, int SMAX, int S>
__device__ __forceinline__ uint32_t flagged_rounds(SparseLds<TX, TQ, R, SMAX>& L, int lane) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  if (lane < SL::NW) L.need[lane] = 0;
  __asm__ volatile("" ::: "memory");
  for (int g = 0; g < SL::NWM; ++g)
    if ((L.win[S][g] >> lane) & 1) {
      const int id = Rounds<R, S>::of_window((g * 64 + lane) / R, (g * 64 + lane) % R);
      __hip_atomic_fetch_or(&L.need[id >> 5], 1u << (id & 31), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  __asm__ volatile("" ::: "memory");
  return lane < SL::NW ? L.need[lane] : 0;
}

// One side of a region that holds live rounds or windows that might exceed their
// bound: see the head of this file.  grown: growth from test_all to this side,
// slack: what the windows below the bound had left of it then.
template <typename TX, typename TQ, int R, int SMAX, int S, bool KAHAN>
__device__ __forceinline__ void sparse_side(Sparse& c, SparseLds<TX, TQ, R, SMAX>& L, int k,
                                            int qb0, float thr, float grown, float slack) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  using SS = SideShape<R, S>;
  using LS = typename SL::SH;
  using RD = Rounds<R, S>;
  using QS = QStore<TQ, TX>;
  constexpr int GR = SS::GR, GC = SS::GC, G = SS::G, BR = SS::BR, BC = SS::BC;
  constexpr int U = SS::U, V = SS::V, JRL = SS::JRL, JCL = SS::JCL;
  constexpr int P = LS::P, ES = (int)sizeof(TQ), NW = SL::NW;

  const int rhi = min(R, fresh_uniform(c.h) - S + 1), chi = min(R, fresh_uniform(c.w) - S + 1);
  const int lane = fresh(c.lane);
  const uint32_t livew = lane < NW ? L.live[k * NW + lane] : 0;
  const int nrounds = max(1, RD::N * rhi * chi / (R * R));  // (as if spread evenly)
  bool linear = thr < 0.0f;
  if (__ballot(livew != 0))
    linear = linear || 2 * (int)group_sum<64>((float)__popc(livew)) > nrounds;
  bool test = !(grown * kGrowth < slack) && !linear;
  // candidates: the rounds still to visit as far as the last test tells
  uint32_t cand = lane * 32 + 32 <= RD::N ? ~0u : lane * 32 < RD::N ? (1u << (RD::N & 31)) - 1u : 0u;
  uint32_t later = cand;  // rounds after the last one visited
  if (!linear && !test) {
    cand = livew;
    if (__builtin_amdgcn_readfirstlane(L.flag[S]))
      cand |= flagged_rounds<TX, TQ, R, SMAX, S>(L, lane);
  }
  // Growth up to which no window is lifted to its bound (what is left of the slack),
  // and a lane's part of it: a lane holds at least a 64th of a sum that passes it.
  float rest = slack - grown * kGrowth, limit = rest * (1.0f / (64.0f * kGrowth));

  const int wl = lane / G, jj = lane % G;
  const int bry = wl / BC, brx = wl % BC, jr = jj / GC, jc = jj % GC;
  const bool rl = jr < JRL, cl = jc < JCL;
  const int ef = (jr * GC + jc) * ES, el = (jr * JCL + jc) * ES;
  const int lane_x0 = (S * bry + jr) * P + (S * brx + jc);
  const int xdum = LS::XDUMMY + lane;
  const int qdum = SL::ODUMMY + lane * ES;
  const TX r2 = (sizeof(TX) == 8) ? (TX)L.r2d[S] : (TX)L.r2f[S];
  const float rfl = L.rf[S], gr2 = c.guard * L.r2f[S];
  const double r2d = L.r2d[S];
  uint32_t noww = 0;
  int blk = -1, ib = 0;
  uint64_t there = 0, livem = 0;     // block's rounds that exist, that are live
  int pos = 0, start0 = 0, nwin = 0; // lane's round of the block
  for (;;) {
    if (test) {
      // (of the rounds after the last one visited)
      const int l = blk * 2 + (ib >> 5), b = ib & 31;
      if (blk >= 0) later = lane < l ? 0u : lane > l ? later : later & (~1u << b);
      float top;
      cand = (livew | window_test<TX, TQ, R, SMAX, S>(L, lane, rhi, chi, thr, &top)) & later;
      c.grown.tested();
      rest = thr - top;
      limit = rest * (1.0f / (64.0f * kGrowth));
      test = false;
    }
    const uint64_t mw = __ballot(cand != 0);
    if (mw == 0) break;
    // the next block of 64 rounds with candidates: where each lies, one per lane
    const int bk = __builtin_ctzll(mw) / 2;
    if (bk != blk) {
      blk = bk;
      const RD rd(min(blk * 64 + lane, RD::N - 1), rhi, chi);
      there = __ballot(blk * 64 + lane < RD::N && rd.exists());
      pos = (rd.ap + S * BR * rd.rby) * P + (rd.bp + S * BC * rd.rbx);
      start0 = qb0 + rd.before * (S * S * ES);
      nwin = rd.nbr | rd.nbc << 8;
      livem = (uint32_t)__builtin_amdgcn_readlane(livew, 2 * blk) |
              (uint64_t)(uint32_t)__builtin_amdgcn_readlane(livew, 2 * blk + 1) << 32;
    }
    uint64_t m = there & ((uint32_t)__builtin_amdgcn_readlane(cand, 2 * blk) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane(cand, 2 * blk + 1) << 32);
    cand = lane >> 1 == blk ? 0u : cand;
    uint64_t nowm = 0;
    while (m != 0) {
      ib = __builtin_ctzll(m);
      m &= m - 1;
      const bool live_in = (livem >> ib) & 1;
      const int start = __builtin_amdgcn_readlane(start0, ib);
      const int nb = __builtin_amdgcn_readlane(nwin, ib), nbr = nb & 0xFF, nbc = nb >> 8;
      const int bx = lane_x0 + __builtin_amdgcn_readlane(pos, ib);
      // (a round that exists holds at least one window)
      const bool valid = (BR == 1 || bry < nbr) && (BC == 1 || brx < nbc);
      const int woff = (bry * nbc + brx) * (S * S * ES);
      const int bxr = valid ? bx : 0;
      TX xv[U][V], y[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          xv[u][v] = L.xs[bxr + u * GR * P + v * GC];
          y[u][v] = TX(0);
        }
      if (live_in) {
        if (__builtin_expect(c.in_seen <= c.in_seq, 0))
          c.in_seen = wait_ge(&L.in_ready, c.in_seq + 1, &L.abort, kSparseSpin);
        __asm__ volatile("" ::: "memory");
        const unsigned char* q = L.in + c.in_off + (start & 3) + woff;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < V; ++v)
            y[u][v] = QS::get(q + (v == V - 1 ? el : ef) + SS::slot(u, v) * ES);
        ++c.in_seq;
        c.in_off = c.in_off == (SL::NIN - 1) * SL::SLOT ? 0 : c.in_off + SL::SLOT;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) y[u][v] = xv[u][v] + y[u][v];
      const TX n = group_sum<G>(lane_sum<TX, R, S, KAHAN>(y, rl, cl));
      TX t;
      if constexpr (sizeof(TX) == 4) {
        const bool near = fabsf(n - r2) <= gr2;
        t = n > r2 ? rfl * __builtin_amdgcn_rsqf(n) : 1.0f;
        if (__builtin_expect(__ballot(near) != 0, 0)) {
          double pd = 0.0;
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) pd = __builtin_fma((double)y[u][v], (double)y[u][v], pd);
          const double nd = group_sum<G>(pd);
          const float t64 = nd > r2d ? (float)__builtin_sqrt(r2d / nd) : 1.0f;
          t = near ? t64 : t;
        }
      } else {
        t = n > r2 ? __builtin_sqrt(r2 / n) : TX(1);
      }
      // (a sum that is not a number leaves t = 1 and increments that are not zero)
      const bool live_out = __ballot(valid && (t != TX(1) || n != n)) != 0;
      if (live_in || live_out) {
        if (__builtin_expect(c.out_seen <= c.out_seq - SL::NOUT, 0))
          c.out_seen = wait_ge(&L.out_done, c.out_seq - SL::NOUT + 1, &L.abort, kSparseSpin);
        const int qf = valid ? c.out_off + woff + ef : qdum;
        const int ql = valid && cl ? c.out_off + woff + el : qdum;
        const int bxw = valid ? bx : xdum;
        float e = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const bool part_r = (u == U - 1) && (JRL < GR), part_c = (v == V - 1) && (JCL < GC);
            const bool keep = (part_r && part_c) ? (rl && cl) : part_r ? rl : part_c ? cl : true;
            const TX xn = t * y[u][v];
            L.xs[(keep ? bxw : xdum) + u * GR * P + v * GC] = xn;
            const int wq = part_r && !rl ? qdum : v == V - 1 ? ql : qf;
            QS::put(L.out + wq + SS::slot(u, v) * ES, y[u][v] - xn);
            // x'^2 - x^2 where it is positive (or not a number)
            const float d = (float)((xn - xv[u][v]) * (xn + xv[u][v]));
            e += !keep || d <= 0.0f ? 0.0f : d;
          }
        c.grown.add(valid ? e : 0.0f);
        L.odesc[c.out_seq & 3] = int2{start, nbr * nbc * (S * S * ES)};
        lds_store(&L.out_ready, ++c.out_seq);
        lds_store(&L.in_done, c.in_seq);
        c.out_off = c.out_off == (SL::NOUT - 1) * SL::SLOT ? 0 : c.out_off + SL::SLOT;
        nowm |= live_out ? 1ull << ib : 0;
        c.nlive += live_out;
      }
      if (S > 1 && !linear) {  // (side 1: windows do not overlap)
        // Another test if the growth may have lifted a window to its bound, or
        // if the round became live and others that are not live remain, which
        // what it took away may have brought below the bound.
        if (__builtin_expect(__ballot(!(c.grown.since < limit)) != 0, 0))
          test = !(group_sum<64>(c.grown.since) * kGrowth < rest);
        if (live_out && !live_in && ((m & ~livem) != 0 || __ballot((cand & ~livew) != 0) != 0)) test = true;
        if (test) break;
      }
    }
    if (lane >> 1 == blk) noww |= (uint32_t)(nowm >> (lane & 1 ? 32 : 0));
  }
  if (lane < NW) L.now[k * NW + lane] = noww;
}

#define SMRE_SIDE_SWITCH(side, CASE)                                                        \
  switch (side) {                                                                           \
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10)        \
    CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16) CASE(17) CASE(18) CASE(19)        \
    CASE(20) CASE(21) CASE(22) CASE(23) CASE(24) CASE(25) CASE(26) CASE(27) CASE(28)        \
    CASE(29) CASE(30) CASE(31) CASE(32)                                                     \
    default: break;                                                                         \
  }

// Every round of side k's region taken for live.
template <typename TX, typename TQ, int R, int SMAX, int S>
__device__ __forceinline__ void all_live(int h, int w, int lane0,
                                         SparseLds<TX, TQ, R, SMAX>& L, int k) {
  constexpr int NW = live_words(R);
  const int lane = fresh(lane0);
  const int rhi = min(R, fresh_uniform(h) - S + 1), chi = min(R, fresh_uniform(w) - S + 1);
  for (int i = 0; i < NW; i += 2) {
    const int id = i * 32 + lane;
    const bool is = rhi > 0 && chi > 0 && id < Rounds<R, S>::N &&
                    Rounds<R, S>(min(id, Rounds<R, S>::N - 1), rhi, chi).exists();
    const uint64_t m = __ballot(is);
    if (lane == 0) {
      L.live[k * NW + i] = (uint32_t)m;
      L.live[k * NW + i + 1] = (uint32_t)(m >> 32);
    }
  }
}

// Where the increments of 64 rounds of a side lie in the region's stream, lane l
// round `base` + l: bytes [start, end); returns the mask of the live ones.
template <typename TX, typename TQ, int R, int SMAX, int S>
__device__ __forceinline__ uint64_t live_block(int h, int w, int lane0,
                                               const SparseLds<TX, TQ, R, SMAX>& L, int k,
                                               int base, int* start, int* end) {
  using RD = Rounds<R, S>;
  constexpr int ES = (int)sizeof(TQ), NW = live_words(R);
  const int lane = fresh(lane0);
  const int rhi = min(R, fresh_uniform(h) - S + 1), chi = min(R, fresh_uniform(w) - S + 1);
  const RD rd(min(base + lane, RD::N - 1), rhi, chi);
  *start = L.base[S] + rd.before * (S * S * ES);
  *end = *start + rd.nbr * rd.nbc * (S * S * ES);
  const int id = min(base + lane, R * R - 1);
  return __ballot(base + lane < RD::N && ((L.live[k * NW + (id >> 5)] >> (id & 31)) & 1));
}

// 4 bytes per active lane from HBM into LDS, lane l's to lds + 4 l, without
// passing through registers; complete when the wave's vector memory count says so
// (the compiler does not know of the load: wait_loads before anything reads it).
__device__ __forceinline__ void load_to_lds(const void* g, uint32_t lds) {
  __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                   :
                   : "s"(lds), "v"(g)
                   : "memory", "m0");
}
// Wait until at most n loads are in flight (or fewer: a few values suffice).
__device__ __forceinline__ void wait_loads(int n) {
  if (n >= 32) __asm__ volatile("s_waitcnt vmcnt(32)" ::: "memory");
  else if (n >= 16) __asm__ volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if (n >= 12) __asm__ volatile("s_waitcnt vmcnt(12)" ::: "memory");
  else if (n >= 8) __asm__ volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else if (n >= 6) __asm__ volatile("s_waitcnt vmcnt(6)" ::: "memory");
  else if (n >= 4) __asm__ volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else if (n >= 2) __asm__ volatile("s_waitcnt vmcnt(2)" ::: "memory");
  else if (n == 1) __asm__ volatile("s_waitcnt vmcnt(1)" ::: "memory");
  else __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Loader wave: lists live rounds, in visiting order, and copies their increments
// into the ring, as many rounds in flight as the ring has slots.
template <typename TX, typename TQ, int R, int SMAX, typename Addr> struct Loader {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  static constexpr int kMaxLoads = 60;  // in flight (the hardware counts to 63)
  SL& L;
  const Addr& g;  // address of a byte of the region's stream
  int nwords, h, w, lane;
  int word;       // 64 words of live bits from here
  uint64_t some = 0;  // those not zero, not listed yet
  int n = 0, at = 0;  // live rounds of the block, taken
  uint64_t left = 0;  // those not taken
  int start = 0, end = 0;  // lane's round of the block: bytes
  int issued = 0, published = 0, freed = 0;  // rounds: loads issued, in the ring, consumed
  int loads = 0;  // in flight
  uint64_t fifo = 0;  // of the rounds in flight, oldest in the lowest byte
  // the next block with live rounds: lane i takes the i-th of them
  __device__ __forceinline__ void list() {
    n = at = 0;
    while (some == 0) {  // 64 words of live bits at a time, two to a block of rounds
      if (word + 64 >= nwords) return;
      word += 64;
      some = __ballot(word + lane < nwords && L.live[min(word + lane, nwords - 1)] != 0);
    }
    const int i = __builtin_ctzll(some) & ~1, k = (word + i) / SL::NW;
    const int base = (word + i) % SL::NW * 32;
    some &= ~(3ull << i);
    int from = 0, to = 0;
#define SMRE_CASE(S)                                                                          \
  case S:                                                                                     \
    if constexpr (S <= SMAX)                                                                  \
      left = live_block<TX, TQ, R, SMAX, S>(h, w, lane, L, k, base, &from, &to);              \
    break;
    SMRE_SIDE_SWITCH(__builtin_amdgcn_readfirstlane(L.side[k]), SMRE_CASE)
#undef SMRE_CASE
    n = __popcll(left);
    start = from;
    end = to;
  }
  // issue what there is room for
  __device__ __forceinline__ void issue() {
    for (;;) {
      if (at == n) list();
      if (at == n) return;
      if (issued - freed >= SL::NIN) {
        freed = __builtin_amdgcn_readfirstlane(lds_load(&L.in_done));
        if (issued - freed >= SL::NIN) return;
      }
      const int l = __builtin_ctzll(left);
      const int lo = __builtin_amdgcn_readlane(start, l) & ~3;
      const int hi = __builtin_amdgcn_readlane(end, l), nl = (hi - lo + 255) / 256;
      if (loads > 0 && loads + nl > kMaxLoads) return;
      const uint32_t slot = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)
                                (L.in + (issued % SL::NIN) * SL::SLOT);
      for (int u = 0; u < nl; ++u) {
        const int o = lo + (u * 64 + lane) * 4;
        if (o < hi) load_to_lds(g(o), __builtin_amdgcn_readfirstlane(slot + u * 256));
      }
      fifo |= (uint64_t)nl << (8 * (issued - published));
      loads += nl;
      ++issued;
      ++at;
      left &= left - 1;
    }
  }
  __device__ __forceinline__ void run() {
    for (;;) {
      issue();
      if (issued > published) {
        const int nl = (int)(fifo & 0xFF);
        loads -= nl;
        fifo >>= 8;
        wait_loads(loads);
        lds_store(&L.in_ready, ++published);
      } else if (at == n) {
        return;
      } else {
        freed = wait_ge(&L.in_done, issued - SL::NIN + 1, &L.abort, kSparseSpin);
      }
    }
  }
};

template <int ES> struct QWord;
template <> struct QWord<2> { typedef uint16_t T; };
template <> struct QWord<4> { typedef uint32_t T; };
template <> struct QWord<8> { typedef uint64_t T; };

// Writer wave: the consumer's updated rounds from the second ring to HBM.
template <typename TX, typename TQ, int R, int SMAX, typename Addr>
__device__ __forceinline__ void write_rounds(int lane, SparseLds<TX, TQ, R, SMAX>& L,
                                             const Addr& g) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  constexpr int ES = SL::ES;
  typedef typename QWord<ES>::T W;
  for (int seq = 0;; ++seq) {
#pragma nounroll
    for (int spin = 0; __builtin_amdgcn_readfirstlane(lds_load(&L.out_ready)) <= seq; ++spin) {
      // (nothing follows a round published before `finished` was raised)
      if (__builtin_amdgcn_readfirstlane(lds_load(&L.finished)) &&
          __builtin_amdgcn_readfirstlane(lds_load(&L.out_ready)) <= seq)
        return;
      if (spin >= kSparseSpin || lds_load(&L.abort)) {
        lds_store(&L.abort, 1);
        return;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __asm__ volatile("" ::: "memory");
    const int os = seq % SL::NOUT;
    const int2 d = L.odesc[seq & 3];
    const int start = __builtin_amdgcn_readfirstlane(d.x);
    const int n = __builtin_amdgcn_readfirstlane(d.y) / ES;
    const W* src = (const W*)(L.out + os * SL::SLOT);
    // (a few words at a time, read before the first is stored)
    for (int i0 = 0; i0 < n; i0 += 4 * 64) {
      W v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * 64 + lane < n) v[u] = src[i0 + u * 64 + lane];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * 64 + lane < n) *(W*)g(start + (i0 + u * 64 + lane) * ES) = v[u];
    }
    __asm__ volatile("" ::: "memory");
    lds_store(&L.out_done, seq + 1);
  }
}

// One region of one image, whole workgroup; false (nothing done) if the region is
// to be streamed whole.  ready(): waits until the region's pixels may be read;
// loaded(): called by one wave that then has nothing left to do.
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN, typename Ready, typename Loaded>
__device__ __forceinline__ bool sparse_job(const ImageDesc& a, int region, unsigned char* q,
                                           uint32_t* lv, SparseLds<TX, TQ, R, SMAX>& L,
                                           bool shared, const Ready& ready, const Loaded& loaded) {
  using SL = SparseLds<TX, TQ, R, SMAX>;
  constexpr int P = SL::SH::P, NW = SL::NW;
  const int r0 = region / a.nrx * R, c0 = (region - region / a.nrx * a.nrx) * R;
  const int fh = min(a.fr, a.H - r0), fw = min(a.fr, a.W - c0);
  const int tid = fresh(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = a.nsides * NW;
  const TX* xg = (const TX*)a.x + (int64_t)r0 * a.ld + c0;
  // live bits, descriptor: all loads issued before the first is used
  const uint32_t head = lv[0];
  const RegionStream st = a.rs[region];
  constexpr int LW = SL::LW, RPP = kPhaseThreads / LW, NP = (R + SMAX - 1 + RPP - 1) / RPP;
  constexpr int NLV = (SMAX * NW + kPhaseThreads - 1) / kPhaseThreads;
  uint32_t bits[NLV];
#pragma unroll
  for (int i = 0; i < NLV; ++i)
    if (tid + i * kPhaseThreads < nw) bits[i] = lv[kLiveHead + tid + i * kPhaseThreads];
  const bool is = lane < a.nsides;  // (last wave) lane k reads side k
  int s = 1;
  float r2f = 0.0f, rf = 0.0f;
  double r2d = 0.0;
  if (wave == 2) {
    const int k = is ? lane : 0;
    s = a.sides[k];
    r2f = a.r2f[k];
    rf = a.rf[k];
    r2d = a.r2d[k];
  }
  const uint32_t h0 = __builtin_amdgcn_readfirstlane(head);
  if (h0 > 1) return false;
  if (wave == 2) {
    // by side: its index, bounds, first increment byte and test bound (bounds
    // near the ends of FP32's range, where its sums mean little: every window
    // might exceed them)
    const int rh = min(R, a.H - r0 - s + 1), ch = min(R, a.W - c0 - s + 1);
    const bool any = is && rh > 0 && ch > 0;
    const int size = any ? rh * ch * (s * s * (int)sizeof(TQ)) : 0;
    const int ar = axis_rounds(R, s), nr = any ? max(1, ar * ar * rh * ch / (R * R)) : 0;
    int base = 0, at = 0, rounds = 0;
    for (int j = 0; j < a.nsides; ++j) {
      if (lane == j) base = at;
      at += __builtin_amdgcn_readlane(size, j);
      rounds += __builtin_amdgcn_readlane(nr, j);
    }
    L.index[lane] = -1;
    L.flag[lane] = 0;
    for (int i = lane; i < (SMAX + 1) * SL::NWM; i += 64) L.win[i / SL::NWM][i % SL::NWM] = 0;
    L.thr[lane] = 1.0f;
    __asm__ volatile("" ::: "memory");
    if (any) {
      L.index[s] = lane;
      L.base[s] = base;
      L.thr[s] = r2f > 1e-25f && r2f < 1e37f ? r2f * (1.0f - kTestMargin) : -1.0f;
      L.r2f[s] = r2f;
      L.rf[s] = rf;
      L.r2d[s] = r2d;
    }
    if (is) L.side[lane] = s;
    L.rounds = rounds;
    if (lane == 0) {
      L.tested = L.in_ready = L.in_done = L.out_ready = L.out_done = 0;
      L.finished = L.abort = L.changed = 0;
    }
  }
  if (wave < 2) L.top[wave][lane] = 0.0f;
#pragma unroll
  for (int i = 0; i < NLV; ++i)
    if (tid + i * kPhaseThreads < nw) {
      L.live[tid + i * kPhaseThreads] = bits[i];
      L.now[tid + i * kPhaseThreads] = 0;
    }
  if (shared) {
    if (wave == 0) ready();
    __syncthreads();
  }
  {
    // footprint: a thread's loads issued before the first is stored
    TX v[NP];
    const int col = tid % LW, row = tid / LW;
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (row + i * RPP < fh && col < fw)
        v[i] = load_pixel(xg + (int64_t)(row + i * RPP) * a.ld + col, shared);
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (row + i * RPP < fh && col < fw) L.xs[(row + i * RPP) * P + col] = v[i];
  }
  __syncthreads();
  if (h0 == 1) {  // every round taken for live (before the loader reads the bits)
    if (wave == 0)
      for (int k = 0; k < a.nsides; ++k) {
#define SMRE_CASE(n) \
  case n:            \
    if constexpr (n <= SMAX) all_live<TX, TQ, R, SMAX, n>(a.H - r0, a.W - c0, lane, L, k); \
    break;
        SMRE_SIDE_SWITCH(a.sides[k], SMRE_CASE)
#undef SMRE_CASE
      }
    __syncthreads();
  }
  unsigned char* gq = q + a.q_byte + (int64_t)st.first * kPage;
  const uint32_t stride = (uint32_t)st.stride;
  auto g = [gq, stride](int o) {
    return gq + (uint64_t)((uint32_t)o >> 10) * ((uint64_t)stride << 10) + (o & (kPage - 1));
  };
  if (wave == 1) {
    Loader<TX, TQ, R, SMAX, decltype(g)> ld{L, g, nw, a.H - r0, a.W - c0, lane, -64};
    ld.run();
    loaded();
  } else {
    test_all<TX, TQ, R, SMAX>(L, wave / 2, lane, a.H - r0, a.W - c0, a.sides[0]);
    if (wave == 2) write_rounds<TX, TQ, R, SMAX>(lane, L, g);
  }
  if (wave == 0) {
    Sparse c;
    c.h = a.H - r0;
    c.w = a.W - c0;
    c.guard = a.guard;
    c.lane = lane;
    c.in_seq = c.in_seen = c.in_off = c.out_seq = c.out_seen = c.out_off = 0;
    c.nlive = 0;
    c.grown = {0.0f, 0.0f, 0.0f};
    wait_ge(&L.tested, 2, &L.abort, kSparseSpin);
    __asm__ volatile("" ::: "memory");
    // lane: side
    const int index = L.index[lane];
    const float thr = L.thr[lane];
    const float slack = thr - fmaxf(L.top[0][lane], L.top[1][lane]);
    bool due = false;  // holds live rounds or windows that might exceed the bound
    if (index >= 0) {
      due = L.flag[lane] != 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) due |= L.live[index * NW + i] != 0;
    }
    uint64_t left = __ballot(index >= 0);
    float grown = 0.0f;
    for (;;) {
      const uint64_t m = __ballot(due || !(grown * kGrowth < slack)) & left;
      if (m == 0) break;
      const int side = 63 - __builtin_clzll(m);
      left &= (1ull << side) - 1;
      const int k = __builtin_amdgcn_readlane(index, side);
      const int qb = __builtin_amdgcn_readfirstlane(L.base[side]);
      const float th = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(thr), side));
      const float sl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(slack), side));
#define SMRE_CASE(n)                                                                            \
  case n:                                                                                       \
    if constexpr (n <= SMAX)                                                                    \
      sparse_side<TX, TQ, R, SMAX, n, KAHAN>(c, L, k, qb, th, grown, sl);                       \
    break;
      SMRE_SIDE_SWITCH(side, SMRE_CASE)
#undef SMRE_CASE
      __asm__ volatile("" ::: "memory");
      c.grown.side_done();
      grown = group_sum<64>(c.grown.total);
    }
    if (lane == 0) {
      L.changed = c.out_seq;
      L.head = 5 * c.nlive > L.rounds + 8 * a.nsides ? kDenseSweeps : 0;
      lv[0] = L.head;
    }
    lds_store(&L.finished, 1);
  }
  __syncthreads();
  if (L.changed) {  // (else no round was live either: the bits are as they were)
    const int t = fresh(tid), c = t % LW, r = t / LW;
    TX* to = (TX*)a.x + (int64_t)r0 * a.ld + c0;
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (r + i * RPP < fh && c < fw)
        store_pixel(to + (int64_t)(r + i * RPP) * a.ld + c, L.xs[(r + i * RPP) * P + c], shared);
#pragma unroll
    for (int i = 0; i < NLV; ++i)
      if (t + i * kPhaseThreads < nw)
        lv[kLiveHead + t + i * kPhaseThreads] = L.now[t + i * kPhaseThreads];
  }
  return true;
}

// ---------------------------------------------------------------- sweep kernel
// Two uses.
//
// A batch, one colour per launch: work item `it` is items[it]; done / abort / streams
// are those of image i at byte i * flag_stride.
//
// One image, a whole sweep per launch (items null): the jobs of the sweep are its
// regions colour by colour, then, in a sweep that is checked, its check jobs
// (sweep_check).  A workgroup takes the next job by a ticket and waits until the
// jobs it depends on have ended: a region, for the regions around it of earlier
// colours (their footprints overlap its own; later colours come after it); a check
// job, for the regions whose footprints hold its pixels.  Those all have smaller
// tickets, so the smallest job that has not ended never waits for one that no
// workgroup has taken, however few of them the device has room for.  One launch in
// place of the seven of a checked sweep (four colours, two passes over the image, a
// decision), and a region waits for its neighbours only, not for the slowest
// region of the image.
struct PhaseArgs {
  const ImageDesc* imgs;
  const WorkItem* items;
  const int* nitems;
  const int* done;
  int* abort;
  int* streams;        // count of regions that will stream in the sweep after
  int64_t flag_stride;
  unsigned char* q;
  // one image
  int32_t sweep;       // counted from 1
  int32_t nregions[4]; // by colour
  int32_t ncheck;      // check jobs
  int32_t decide;      // the sweep's largest change is compared with tol
  double tol;
  int* progress;       // by region: last sweep that ended
  void* prev;          // image at the end of the sweep before
  Ctrl* ctrl;
  int* host_done;      // (host memory) [0] raised with ctrl->done, [1] ctrl->streams of the
                       // sweep before
};

// Waits, with one wave, until those of a region and the eight around it that `needs`
// names have ended the sweep.
template <typename Needs>
__device__ __forceinline__ void wait_regions(const PhaseArgs& p, const ImageDesc& a, int ry, int rx,
                                             const Needs& needs) {
  const int lane = fresh(threadIdx.x & 63);
  const int y = ry + lane / 3 - 1, x = rx + lane % 3 - 1;
  const bool wait = lane < 9 && y >= 0 && x >= 0 && y < a.nry && x < a.nrx && needs(y, x);
  const int* at = p.progress + (wait ? y * a.nrx + x : 0);
#pragma nounroll
  for (int spin = 0; spin < kSparseSpin; ++spin) {
    const bool open =
        wait && __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < p.sweep;
    if (__ballot(open) == 0) return;
    __builtin_amdgcn_s_sleep(1);
  }
  if (lane == 0) atomicOr(p.abort, 1);
}

// The pixels of a tile of TH x TW at (y0, x0), compared with (and kept for) the sweep
// before: a thread's largest change.
template <typename TX, int TH, int TW, int NT>
__device__ __forceinline__ double check_tile(const PhaseArgs& p, const ImageDesc& a, int y0, int x0,
                                             int tid, bool shared) {
  const int h = min(TH, a.H - y0), w = min(TW, a.W - x0);
  const TX* x = (const TX*)a.x + (int64_t)y0 * a.ld + x0;
  TX* prev = (TX*)p.prev + (int64_t)y0 * a.W + x0;
  constexpr int NB = (TH * TW + NT - 1) / NT;
  constexpr int NU = NB < 4 ? NB : 4;
  double d = 0.0;
  for (int i0 = tid; i0 < TH * TW; i0 += NU * NT) {
    TX v[NU], o[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = i0 + u * NT, r = i / TW, c = i % TW;
      v[u] = o[u] = TX(0);
      if (r < h && c < w) {
        v[u] = load_pixel(x + (int64_t)r * a.ld + c, shared);
        o[u] = prev[(int64_t)r * a.W + c];
      }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = i0 + u * NT, r = i / TW, c = i % TW;
      if (r < h && c < w) prev[(int64_t)r * a.W + c] = v[u];
      d = fmax(d, fabs((double)v[u] - (double)o[u]));
    }
  }
  return d;
}

// The last of a sweep's p.ncheck workgroups to come here with its largest change
// decides.
template <int NT> __device__ __forceinline__ void check_decide(const PhaseArgs& p, double d, int tid) {
  __shared__ double part[NT / 64];
  for (int o = 32; o > 0; o >>= 1) d = fmax(d, __shfl_xor(d, o));
  if ((tid & 63) == 0) part[tid >> 6] = d;
  __syncthreads();
  if (tid == 0) {
    for (int i = 1; i < NT / 64; ++i) d = fmax(d, part[i]);
    Ctrl* c = p.ctrl;
    // (the count follows the maximum: each waits for its result)
    if (d > 0.0) {
      const unsigned long long was = atomicMax(&c->delta_key, dkey(d));
      __asm__ volatile("" ::"v"((uint32_t)was) : "memory");
    }
    if (atomicAdd(&c->arrived, 1) == p.ncheck - 1) {
      const unsigned long long key =
          __hip_atomic_load(&c->delta_key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double last = dkey_inv(key);
      c->last_delta = last;
      c->delta_key = dkey(0.0);
      c->arrived = 0;
      if (last < p.tol) {
        c->done_sweep = p.sweep;
        c->done = 1;
        __hip_atomic_store(p.host_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
}

// Check job b of a sweep in one launch: the pixels of 2 x 2 regions.
template <typename TX, int R, int NT>
__device__ __forceinline__ void sweep_check(const PhaseArgs& p, const ImageDesc& a, int b) {
  const int tid = fresh(threadIdx.x);
  const int nbx = (a.nrx + 1) / 2, by = b / nbx, bx = b - b / nbx * nbx;
  if (tid < 64) wait_regions(p, a, 2 * by, 2 * bx, [](int, int) { return true; });
  __syncthreads();
  const double d = check_tile<TX, 2 * R, 2 * R, NT>(p, a, 2 * by * R, 2 * bx * R, tid, true);
  if (p.decide) check_decide<NT>(p, d, tid);
}

// The check of a sweep after launches of stream_phase: tiles of 64-pixel rows,
// by at most kCheckBlocks workgroups, since each adds to one counter.  (With a
// workgroup per 2 x 2 regions 2048 x 2048 pixels took 80 us, 209 with region side 8;
// 29 now.)
constexpr int kCheckBlocks = 1024, kCheckH = 16, kCheckW = 64;
__host__ __device__ __forceinline__ int check_tiles(int H, int W) {
  return ((H + kCheckH - 1) / kCheckH) * ((W + kCheckW - 1) / kCheckW);
}
template <typename TX> __global__ __launch_bounds__(256) void sweep_check_kernel(PhaseArgs p) {
  if (*p.done) return;
  const ImageDesc& a = *p.imgs;
  const int n = check_tiles(a.H, a.W), nx = (a.W + kCheckW - 1) / kCheckW;
  double d = 0.0;
  for (int t = blockIdx.x; t < n; t += gridDim.x)
    d = fmax(d, check_tile<TX, kCheckH, kCheckW, 256>(p, a, t / nx * kCheckH, t % nx * kCheckW,
                                                      threadIdx.x, false));
  if (p.decide) check_decide<256>(p, d, threadIdx.x);
}

// One image, one colour, every region through region_job: block b takes the b-th
// region of colour (cy, cx).
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
__global__ __launch_bounds__(128) void stream_phase(ImageDesc a, int cy, int cx, int ncx,
                                                    const int* done, int* abort_flag,
                                                    unsigned char* q) {
  __shared__ PhaseLds<TX, TQ, R, SMAX> L;
  if (*done) return;
  const int b = blockIdx.x;
  const int region = (cy + 2 * (b / ncx)) * a.nrx + cx + 2 * (b % ncx);
  reset_counters(L);
  region_job<TX, TQ, R, SMAX, KAHAN>(a, region, q, L, threadIdx.x & 63, false, []() {},
                                         []() {});
  __syncthreads();
  if (threadIdx.x == 0 && L.ctr[2]) atomicOr(abort_flag, 1);
}

// The same for a batch: a persistent grid walks the colour's work list.
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
__global__ __launch_bounds__(128) void stream_batch(const ImageDesc* __restrict__ imgs,
                                                    const WorkItem* __restrict__ items,
                                                    PhaseArgs p) {
  __shared__ PhaseLds<TX, TQ, R, SMAX> L;
  const int n = *p.nitems;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const WorkItem w = items[it];
    const int64_t flag = w.img * p.flag_stride;
    if (*(const int*)((const char*)p.done + flag)) continue;
    reset_counters(L);
    region_job<TX, TQ, R, SMAX, KAHAN>(imgs[w.img], w.region, p.q, L, threadIdx.x & 63, false,
                                       []() {}, []() {});
    __syncthreads();
    if (threadIdx.x == 0 && L.ctr[2]) atomicOr((int*)((char*)p.abort + flag), 1);
  }
}

// Host side of an instance (phase.hip): launches, and workgroups that fit a CU
// (stream: of stream_batch).
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
void launch_stream(const ImageDesc& a, int cy, int cx, int ncx, int grid, const PhaseArgs& p,
                   hipStream_t s);
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
void launch_phase(int grid, const PhaseArgs& p, bool stream, hipStream_t s);
template <typename TX, typename TQ, int R, int SMAX, bool KAHAN> hipError_t phase_blocks(int* n, bool stream);

template <typename TX, typename TQ, int R, int SMAX, bool KAHAN>
__global__ __launch_bounds__(kPhaseThreads, sizeof(TX) == 4 && R <= 16 ? 3 : 2) void region_phase(
    const ImageDesc* __restrict__ imgs, const WorkItem* __restrict__ items, PhaseArgs p) {
  __shared__ union {
    PhaseLds<TX, TQ, R, SMAX> dense;
    SparseLds<TX, TQ, R, SMAX> sparse;
  } L;
  __shared__ int ticket;
  int it = blockIdx.x, n, c1 = 0, c2 = 0, c3 = 0, c4 = 0;
  if (items) {
    n = *p.nitems;
  } else {
    if (*p.done) return;
    c1 = p.nregions[0];
    c2 = c1 + p.nregions[1];
    c3 = c2 + p.nregions[2];
    c4 = c3 + p.nregions[3];
    n = c4 + p.ncheck;
    if (threadIdx.x == 0) ticket = atomicAdd(&p.ctrl->ticket[p.sweep & 1], 1);
    __syncthreads();
    it = __builtin_amdgcn_readfirstlane(ticket);
    if (it == 0 && threadIdx.x == 0) {
      // the counters of the sweep to come, which no launch uses now; first, what
      // the sweep before counted, for the host
      const int o = (p.sweep + 1) & 1;
      __hip_atomic_store(
          p.host_done + 1,
          __hip_atomic_load(&p.ctrl->streams[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      p.ctrl->ticket[o] = p.ctrl->streams[o] = 0;
    }
  }
  while (it < n) {
    int img = 0, region = 0, ry = 0, rx = 0, color = -1;
    const ImageDesc* ap = imgs;
    if (items) {
      const WorkItem w = items[it];
      img = w.img;
      region = w.region;
      ap += img;
    } else if (it < c4) {
      color = it < c1 ? 0 : it < c2 ? 1 : it < c3 ? 2 : 3;
      const int b = it - (color == 0 ? 0 : color == 1 ? c1 : color == 2 ? c2 : c3);
      const int ncx = (ap->nrx + 1 - (color & 1)) / 2;
      ry = (color >> 1) + 2 * (b / ncx);
      rx = (color & 1) + 2 * (b - b / ncx * ncx);
      region = ry * ap->nrx + rx;
    }
    const ImageDesc& a = *ap;
    const int64_t flag = img * p.flag_stride;
    // The ticket of the next job, taken by the wave that loads when it has loaded
    // all: in a job of many rounds near its end, else at once, so that the atomic's 2 us
    // pass under the job.  (Taken at the start of every job it makes the workgroups that
    // start first hold a second region of the first colour each while others already
    // wait for it.  512 x 512, sides 1..8, us per sweep with every region streamed: 507,
    // 335 now; every round taken for live: 1390, 775.  Taken after the job: 347, 780, and
    // 5 to 10 us more a sweep of a quiet image.)
    auto next = [&]() {
      if (!items && (threadIdx.x & 63) == 0) ticket = atomicAdd(&p.ctrl->ticket[p.sweep & 1], 1);
    };
    if (!items && it >= c4) {
      sweep_check<TX, R, kPhaseThreads>(p, a, it - c4);
      if (threadIdx.x < 64) next();
    } else if (!items || !*(const int*)((const char*)p.done + flag)) {
      uint32_t* lv = (uint32_t*)(p.q + a.q_byte + a.live_off) +
                     (int64_t)region * (kLiveHead + a.nsides * live_words(R));
      const bool shared = !items;
      auto ready = [&]() {
        if (color > 0 && shared)
          wait_regions(p, a, ry, rx,
                       [color](int y, int x) { return (y & 1) * 2 + (x & 1) < color; });
      };
      auto ended = [&]() {
        if ((threadIdx.x & 63) == 0)
          __hip_atomic_store(p.progress + region, p.sweep, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      };
      int aborted, head;
      if (!a.stream && sparse_job<TX, TQ, R, SMAX, KAHAN>(a, region, p.q, lv, L.sparse, shared, ready,
                                                      next)) {
        aborted = L.sparse.abort;
        head = L.sparse.head;
        if (shared) {
          // this wave's pixels have arrived, then every wave's
          __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
          __syncthreads();
          if (threadIdx.x < 64) ended();
        }
      } else {
        head = a.stream ? 0 : (int)lv[0] - 1;
        reset_counters(L.dense);
        if (threadIdx.x < 128)
          region_job<TX, TQ, R, SMAX, KAHAN>(a, region, p.q, L.dense, fresh(threadIdx.x & 63),
                                             shared, ready, ended);
        if (threadIdx.x >= 64 && threadIdx.x < 128) next();
        __syncthreads();
        aborted = L.dense.ctr[2];
        if (threadIdx.x == 0) lv[0] = head;
      }
      if (head > 1 && threadIdx.x == 0) atomicAdd((int*)((char*)p.streams + flag), 1);
      // a wait that gave up (a protocol failure): the host reports a device error
      // for that solve only
      if (threadIdx.x == 0 && aborted) atomicOr((int*)((char*)p.abort + flag), 1);
    }
    __syncthreads();  // before the next item's set-up
    if (items) {
      it += gridDim.x;
    } else {
      it = __builtin_amdgcn_readfirstlane(ticket);
    }
  }
}

}  // namespace smre
