// sft_strain.hip -- SFTs of raw strain series on the device (Sec. III.B segmentation,
// Eq. d_SFT) with the per-SFT noise PSD estimate (bias-corrected running median of the SFT's
// own periodogram), gaps detected as segments holding a non-finite sample.
//
// strain_sft_kernel: n a power of two.  One workgroup per segment of n = 2M samples.  The real series is taken as
// M complex points z[m] = x[2m] + i x[2m+1], loaded in natural order into LDS and transformed
// in place by radix-8 decimation-in-frequency passes (FP64); the n/2 + 1 bins of the real
// transform follow from Z[k] and conj(Z[M - k]):
//   X[k] = (Z[k] + conj(Z[M-k])) / 2 - i e^{-2 pi i k / n} (Z[k] - conj(Z[M-k])) / 2.
// The band bins are written as dt X[k]; the PSD of band bin k is 2 median(P) / (T B) over the
// block of N = 2w+1 periodogram values P[j] = |dt X[j]|^2 centred on k (shifted at the ends of
// [0, n/2]), with B the mean of the middle order statistic of N unit exponentials.  The median
// is the sorted block's middle element (ties broken by bin): found by a wavefront-wide sort of
// the union of 64 neighbouring blocks (half widths w <= 96), or by rank counting per bin.
// strain_blue_kernel (n from 82 to 8190), strain_dft_kernel: other even n with a known white PSD.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

#include "../../include/sft.h"

sft_status sft_set_error(sft_status st, const char* msg);

namespace {

constexpr int kStrainBlock = 256;

__device__ inline double2 cmul(double2 a, double2 b)
{
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// Median of each lane's block by a wavefront-wide sort: the 64 lanes of a wavefront take 64
// consecutive band bins, whose blocks of 2w+1 periodogram values lie in a union of at most
// 64 + 2w <= 128 bins.  The union's (value, bin) pairs are sorted once per wavefront by a
// bitonic network held in registers (two pairs per lane, the partner of each compare-exchange
// fetched across lanes; the 28 stages unrolled and free of branches) and stored in the
// wavefront's LDS slot; every lane then finds the (w+1)-th entry of the sorted list that falls in
// its block (a binary search over prefix masks of the list's bins): the block's middle element in
// (value, bin) order, as a sort of the block itself gives.
constexpr int kSortN = 128;
constexpr int kMaxSortW = (kSortN - 64) / 2;   // w <= 32
constexpr int kMaxKeyW = (256 - 64) / 2;         // w <= 96: four 32-bit keys per lane (below)
// LDS bytes of a wavefront's sort slot: the sorted list (64-bit values, or keys), then for every position of
// the list the mask of the union bins (relative to the union's first bin) that it and the entries before
// it hold
__host__ __device__ constexpr int sort_slot(int w)
{
  return w <= kMaxSortW ? kSortN * (int)(sizeof(double) + sizeof(uint4)) : 256 * (4 + 32);
}

__device__ inline void wave_sync()
{
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline bool pair_less(double va, int ia, double vb, int ib)
{
  return (va < vb) | ((va == vb) & (ia < ib));   // no short circuit: selects, not branches
}

// The 32-bit value of lane (lane ^ S) of the wavefront: quad permutes for S = 1, 2, a half-row
// mirror then a quad reversal for S = 4 ((i ^ 7) ^ 3 = i ^ 4 within each 8 lanes), a rotation
// by 8 within each row of 16 for S = 8 (all on the vector ALU); a swizzle in xor mode within 32
// lanes for S = 16 and a backward permute for S = 32.
template <int S>
__device__ inline int lane_xor(int v, int lane)
{
  if constexpr (S == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  else if constexpr (S == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  else if constexpr (S == 4) {
    const int t = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    return __builtin_amdgcn_mov_dpp(t, 0x1B, 0xF, 0xF, false);           // quad_perm [3,2,1,0]
  } else if constexpr (S == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, false);   // row_ror:8
  else if constexpr (S == 16) return __builtin_amdgcn_ds_swizzle(v, 0x401F);   // and 0x1f, xor 0x10
  else return __builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, v);
}

template <int S>
__device__ inline void xchg_pair(double v, int i, int lane, double& pv, int& pi)
{
  const long long b = __double_as_longlong(v);
  const int lo = lane_xor<S>((int)(b & 0xffffffffll), lane);
  const int hi = lane_xor<S>((int)(b >> 32), lane);
  pv = __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
  pi = lane_xor<S>(i, lane);
}

// One compare-exchange stage of the bitonic network on kSortN = 128 (value, bin) pairs held two
// per lane: element `lane` in (a, ia), element `lane + 64` in (b, ib).  Stride 64 pairs the two
// elements of a lane; smaller strides pair an element with the same one of lane ^ STRIDE, and
// the lower member of the pair keeps the smaller (up) or the larger (down) of the two.
template <int SIZE, int STRIDE>
__device__ inline void bitonic_stage(double& a, int& ia, double& b, int& ib, int lane)
{
  if constexpr (STRIDE == 64) {
    // SIZE = 128: every pair ascending
    const bool sw = pair_less(b, ib, a, ia);
    const double ta = a;
    const int tia = ia;
    a = sw ? b : a;
    ia = sw ? ib : ia;
    b = sw ? ta : b;
    ib = sw ? tia : ib;
  } else {
    const bool lower = (lane & STRIDE) == 0;
    const int qlo = lane & ~STRIDE;
    double pa, pb;
    int pia, pib;
    xchg_pair<STRIDE>(a, ia, lane, pa, pia);
    xchg_pair<STRIDE>(b, ib, lane, pb, pib);
    // keep the smaller of the pair when this lane holds the lower member of an ascending pair
    // or the upper member of a descending one
    const bool mina = lower == ((qlo & SIZE) == 0);
    const bool minb = lower == (((qlo + 64) & SIZE) == 0);
    const bool ta = mina ? pair_less(pa, pia, a, ia) : pair_less(a, ia, pa, pia);
    const bool tb = minb ? pair_less(pb, pib, b, ib) : pair_less(b, ib, pb, pib);
    a = ta ? pa : a;
    ia = ta ? pia : ia;
    b = tb ? pb : b;
    ib = tb ? pib : ib;
  }
}

// Inclusive OR-scan of a 32-bit word over the 64 lanes: shifts by 1, 2, 4, 8 within each row of
// 16 lanes (zero shifted in), then the last lane of rows 0 and 2 into rows 1 and 3, and lane 31
// into rows 2 and 3.
__device__ inline uint32_t wave_or_scan(uint32_t x)
{
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);    // row_shr:1
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);    // row_shr:2
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);    // row_shr:4
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);    // row_shr:8
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15
  x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31
  return x;
}

template <int SIZE, int STRIDE>
__device__ inline void bitonic_from(double& a, int& ia, double& b, int& ib, int lane)
{
  bitonic_stage<SIZE, STRIDE>(a, ia, b, ib, lane);
  if constexpr (STRIDE > 1) bitonic_from<SIZE, STRIDE / 2>(a, ia, b, ib, lane);
  else if constexpr (SIZE < kSortN) bitonic_from<SIZE * 2, SIZE>(a, ia, b, ib, lane);
}

// ---- the same medians by a sort of 32-bit keys
// The periodogram is positive, so the upper words of its values order them up to ties.  A key is the upper word
// above the union's largest one minus R, in 32 - B bits, and the bin's place in the union in the B lowest (B = 7
// or 8 for E = 2 or 4 keys per lane): ratios down to 2^-32 (2^-16) keep all 20 mantissa bits of the word, smaller
// values share one key value.  A compare-exchange then is one lane exchange and one instruction instead of three
// exchanges and a 64-bit compare with its selects.  The median found so is exact unless the entry beside it
// in the sorted list has the same upper word (one chunk in thousands on noise): then, unless those are zeros, the
// caller takes the exact path for the whole chunk (the sort of pairs, or rank counting for w > 32).  12288 segments of 4096
// samples, w = 25: 274 us with the pairs alone, 186 us so; 1000 of 1024 samples, w = 50: 510 us by rank
// counting, 15 us so.
template <int E>
struct KeySort {
  static constexpr int N = 64 * E, B = E == 2 ? 7 : 8;
  static constexpr uint32_t R = (1u << (32 - B)) - 2;   // largest upper word of a key; the pads are above
  static constexpr int kBytes = N * 4 + N * 8 * E;      // keys and prefix masks of a wavefront
  uint32_t a[E];      // entry 64 e + lane of the list
  uint32_t sm[6];     // all ones where bit s of the lane is set

  // min (sel = 0) or max (sel = all ones) of x and y
  static __device__ inline uint32_t pick(uint32_t x, uint32_t y, uint32_t sel)
  {
    const uint32_t lo = x < y ? x : y, hi = x < y ? y : x, m = hi < sel ? hi : sel;
    return lo > m ? lo : m;
  }
  template <int SIZE, int STRIDE>
  __device__ inline void stage()
  {
    if constexpr (STRIDE >= 64) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (e & (STRIDE / 64)) continue;
        const uint32_t x = a[e], y = a[e + STRIDE / 64];
        const bool up = ((64 * e) & SIZE) == 0;
        a[e] = up ? min(x, y) : max(x, y);
        a[e + STRIDE / 64] = up ? max(x, y) : min(x, y);
      }
    } else {
      constexpr int LS = STRIDE == 1 ? 0 : STRIDE == 2 ? 1 : STRIDE == 4 ? 2 : STRIDE == 8 ? 3 : STRIDE == 16 ? 4 : 5;
      constexpr int LZ = SIZE == 2 ? 1 : SIZE == 4 ? 2 : SIZE == 8 ? 3 : SIZE == 16 ? 4 : 5;
      const uint32_t up = SIZE < 64 ? sm[LS] ^ sm[LZ] : sm[LS];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint32_t sel = SIZE >= 64 && ((64 * e) & SIZE) ? ~up : up;
        if constexpr (STRIDE == 32) {
          const auto r = __builtin_amdgcn_permlane32_swap(a[e], a[e], false, false);   // both members of each pair
          a[e] = pick(r[0], r[1], sel);
        } else if constexpr (STRIDE == 16) {
          const auto r = __builtin_amdgcn_permlane16_swap(a[e], a[e], false, false);
          a[e] = pick(r[0], r[1], sel);
        } else {
          a[e] = pick(a[e], (uint32_t)lane_xor<STRIDE>((int)a[e], 0), sel);
        }
      }
    }
  }
  template <int SIZE, int STRIDE>
  __device__ inline void from()
  {
    stage<SIZE, STRIDE>();
    if constexpr (STRIDE > 1) from<SIZE, STRIDE / 2>();
    else if constexpr (SIZE < N) from<SIZE * 2, SIZE>();
  }
};

static_assert(KeySort<2>::kBytes <= sort_slot(kMaxSortW) && KeySort<4>::kBytes <= sort_slot(kMaxKeyW), "sort slots");

// largest value over the 64 lanes
__device__ inline uint32_t wave_max(uint32_t x)
{
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true));    // row_shr:1
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true));    // row_shr:2
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true));    // row_shr:4
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true));    // row_shr:8
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));   // row_bcast:15
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));   // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// Medians of the blocks [s0r, s0r + 2w + 1) (one per lane, relative to u0) of the L values U[u0 ..]; slot holds
// KeySort<E>::kBytes of the wavefront's LDS.  False (for the whole wavefront) where a lane of `want` needs
// the exact path.
template <int E>
__device__ inline bool key_medians(const double* U, int u0, int L, int s0r, int w, int lane, bool want, char* slot,
                                   double& med)
{
  using KS = KeySort<E>;
  KS ks;
  uint32_t top = 0, bot = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = 64 * e + lane;
    const uint32_t h = p < L ? (uint32_t)((unsigned long long)__double_as_longlong(U[u0 + p]) >> 32) : 0;
    ks.a[e] = h;
    top = max(top, h);
    bot = max(bot, p < L ? ~h : 0u);
  }
  top = wave_max(top);
  bot = ~wave_max(bot);
  if (top >= 0x7ff00000u) return false;   // an infinity or NaN
  if (top == bot) {
    // one key value for all; one value for all (a detector that recorded zeros): that is every median
    bool same = true;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int p = 64 * e + lane;
      same = same && (p >= L || U[u0 + p] == U[u0]);
    }
    med = U[u0];
    return !__ballot(!same);
  }
  const uint32_t base = top > KS::R ? top - KS::R : 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = 64 * e + lane;
    const uint32_t h = ks.a[e] > base ? ks.a[e] - base : 0;
    ks.a[e] = p < L ? (h << KS::B) | (uint32_t)p : 0xffffffffu;
  }
#pragma unroll
  for (int b = 0; b < 6; ++b) ks.sm[b] = (lane >> b) & 1 ? 0xffffffffu : 0u;
  ks.template from<2, 1>();
  // prefix masks of the sorted list: bit j of entry q is set when union bin j is one of the entries 0..q
  uint32_t* keys = reinterpret_cast<uint32_t*>(slot);
  uint4* pm = reinterpret_cast<uint4*>(slot + KS::N * 4);
  uint32_t carry[2 * E] = {};
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t id = ks.a[e] & (KS::N - 1);
    const uint32_t bit = ks.a[e] == 0xffffffffu ? 0u : 1u << (id & 31);
    uint32_t m[2 * E];
#pragma unroll
    for (int wd = 0; wd < 2 * E; ++wd) {
      m[wd] = wave_or_scan((id >> 5) == (uint32_t)wd ? bit : 0u) | carry[wd];
      carry[wd] = (uint32_t)__builtin_amdgcn_readlane((int)m[wd], 63);
    }
    keys[64 * e + lane] = ks.a[e];
#pragma unroll
    for (int h = 0; h < E / 2; ++h)
      pm[(64 * e + lane) * (E / 2) + h] = make_uint4(m[4 * h], m[4 * h + 1], m[4 * h + 2], m[4 * h + 3]);
  }
  wave_sync();
  // The count of a lane's block entries among the sorted entries 0..q is the popcount of pm[q] under the
  // block's mask and grows with q; the block's median is the entry at which it reaches w + 1.
  uint32_t wm[2 * E];
#pragma unroll
  for (int wd = 0; wd < 2 * E; ++wd) {
    const int lo = min(max(s0r - 32 * wd, 0), 32), hi = min(max(s0r + 2 * w + 1 - 32 * wd, 0), 32);
    wm[wd] = (uint32_t)(((1ull << hi) - 1ull) & ~((1ull << lo) - 1ull));
  }
  int qlo = 0, qhi = KS::N - 1;
#pragma unroll
  for (int it = 0; it < (E == 2 ? 7 : 8); ++it) {
    const int mid = (qlo + qhi) >> 1;
    int c = 0;
#pragma unroll
    for (int h = 0; h < E / 2; ++h) {
      const uint4 p = pm[mid * (E / 2) + h];
      c += __builtin_popcount(p.x & wm[4 * h]) + __builtin_popcount(p.y & wm[4 * h + 1]) +
           __builtin_popcount(p.z & wm[4 * h + 2]) + __builtin_popcount(p.w & wm[4 * h + 3]);
    }
    if (c >= w + 1) qhi = mid;
    else qlo = mid + 1;
  }
  const uint32_t kq = keys[qlo];
  const uint32_t kp = qlo > 0 ? keys[qlo - 1] : 0xffffffffu, kn = qlo < KS::N - 1 ? keys[qlo + 1] : 0xffffffffu;
  const bool tie = (kp >> KS::B) == (kq >> KS::B) || (kn >> KS::B) == (kq >> KS::B);
  med = U[u0 + (int)(kq & (KS::N - 1))];
  wave_sync();
  if (!__ballot(want && tie)) return true;
  // ties among zeros (a constant segment's bins beside its mean): every entry of the lowest key value is 0 (7812
  // such segments of 256 samples, w = 25: pairs alone 37 us, keys and then pairs 50 us, so 29 us)
  bool zeros = !(want && tie) || (kq >> KS::B) == 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = 64 * e + lane;
    if (p < L) {
      const double v = U[u0 + p];
      zeros = zeros && (v == 0.0 || (uint32_t)((unsigned long long)__double_as_longlong(v) >> 32) > base);
    }
  }
  return !__ballot(!zeros);
}

// The exact path: the medians by a sort of (value, bin) pairs, L <= kSortN.
__device__ inline double pair_median(const double* U, int u0, int L, int s0r, int w, int lane, char* slot)
{
  double* sv = reinterpret_cast<double*>(slot);
  uint4* pm = reinterpret_cast<uint4*>(slot + kSortN * 8);
  const int N = 2 * w + 1;
  // the kSortN pairs sorted in registers (two per lane), then stored in sorted order
  double a = lane < L ? U[u0 + lane] : INFINITY, b = lane + 64 < L ? U[u0 + lane + 64] : INFINITY;
  int ia = lane < L ? lane : 0x7fffffff, ib = lane + 64 < L ? lane + 64 : 0x7fffffff;
  bitonic_from<2, 1>(a, ia, b, ib, lane);
  // prefix masks of the sorted list: bit j of pm[q] is set when union bin j is one of the
  // entries 0..q (an OR-scan of one-hot masks over the lanes, the second half of the list
  // on top of the first; the pads set no bit)
  uint32_t sa[4], sb[4];
#pragma unroll
  for (int wd = 0; wd < 4; ++wd) {
    sa[wd] = wave_or_scan((ia >> 5) == wd ? 1u << (ia & 31) : 0u);
    const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)sa[wd], 63);
    sb[wd] = wave_or_scan((ib >> 5) == wd ? 1u << (ib & 31) : 0u) | t;
  }
  sv[lane] = a;
  sv[lane + 64] = b;
  pm[lane] = make_uint4(sa[0], sa[1], sa[2], sa[3]);
  pm[lane + 64] = make_uint4(sb[0], sb[1], sb[2], sb[3]);
  wave_sync();
  // the smallest entry whose prefix holds w + 1 entries of the lane's block
  uint32_t wm[4];
#pragma unroll
  for (int wd = 0; wd < 4; ++wd) {
    const int lo = min(max(s0r - 32 * wd, 0), 32), hi = min(max(s0r + N - 32 * wd, 0), 32);
    wm[wd] = (uint32_t)(((1ull << hi) - 1ull) & ~((1ull << lo) - 1ull));
  }
  int qlo = 0, qhi = kSortN - 1;
#pragma unroll
  for (int it = 0; it < 7; ++it) {
    const int mid = (qlo + qhi) >> 1;
    const uint4 p = pm[mid];
    const int c = __builtin_popcount(p.x & wm[0]) + __builtin_popcount(p.y & wm[1]) +
                  __builtin_popcount(p.z & wm[2]) + __builtin_popcount(p.w & wm[3]);
    if (c >= w + 1) qhi = mid;
    else qlo = mid + 1;
  }
  const double med = sv[qlo];
  wave_sync();
  return med;
}

// Median of the 2w + 1 values P by rank counting, ties broken by position.
__device__ inline double rank_median(const double* P, int w)
{
  const int N = 2 * w + 1;
  for (int a = 0; a < N; ++a) {
    const double pa = P[a];
    int rank = 0;
    for (int b = 0; b < N; ++b) {
      const double pb = P[b];
      rank += (pb < pa || (pb == pa && b < a)) ? 1 : 0;
    }
    if (rank == w) return pa;
  }
  return 0.0;
}

// Transform of the M = 2^LOGM complex points in LDS (natural order in, digit-reversed out), as
// in-place decimation-in-frequency passes of radix 8 (and one of radix 2 or 4 for the leftover
// bits).  Before pass i the data are M / L independent sub-transforms of length L = M / 8^i,
// each contiguous; with L = R L', the work item (g, n1) of sub-transform g reads its R points
// n1 + L' n2, forms their R-point DFT in registers, multiplies output k2 by W_L^{n1 k2} and
// writes it back to the position it read point n2 = k2 from: sub-transform g R + k2, of length
// L', holds the outputs R k1 + k2 of sub-transform g (its k1-th output after the later passes).
// So X[k] ends at position pos(k), the digits of k (radix 8 from the least significant end)
// in reverse order.
template <int LOGM>
struct FftShape {
  static constexpr int M = 1 << LOGM;
  static constexpr int NP = (LOGM + 2) / 3;                              // passes
  static constexpr int lr(int i) { return i < LOGM / 3 ? 3 : LOGM % 3; }  // log2 of pass i's radix
};

// LDS slot of point i: the 16 points of an aligned run (one pass over the 64 banks, 16 bytes
// each) are permuted by an XOR of higher index bits, so that the strided accesses of the later
// passes and the digit-reversed reads of the unfolding spread over the banks (a model of the
// 16-lane groups of a 16-byte LDS read puts their mean conflict degree at ~1.3 instead of ~4.3
// for M = 2048).  A bijection on each run, the identity for M <= 16.
__device__ inline int swz(int i) { return i ^ (((i >> 4) ^ (i >> 7) ^ (i >> 8)) & 15); }

template <int LOGM>
__device__ inline int fft_pos(int k)
{
  int p = 0;
#pragma unroll
  for (int i = 0; i < FftShape<LOGM>::NP; ++i) {
    const int l = FftShape<LOGM>::lr(i);
    p |= ((k >> (3 * i)) & ((1 << l) - 1)) << (LOGM - 3 * i - l);
  }
  return p;
}

// in-place R-point DFT, v[k] <- sum_n v[n] e^{-2 pi i n k / R}, R = 2, 4 or 8
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }   // times -i

__device__ inline void dft4(double2& u0, double2& u1, double2& u2, double2& u3)
{
  const double2 c0 = cadd(u0, u2), c1 = csub(u0, u2), c2 = cadd(u1, u3), c3 = mul_mi(csub(u1, u3));
  u0 = cadd(c0, c2);
  u1 = cadd(c1, c3);
  u2 = csub(c0, c2);
  u3 = csub(c1, c3);
}

template <int R>
__device__ inline void dft_small(double2* v)
{
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
  } else {
    // radix-2 split: even outputs from a_n = v_n + v_{n+4}, odd ones from
    // b_n = (v_n - v_{n+4}) e^{-2 pi i n / 8}, each by a 4-point DFT
    constexpr double c = 0.70710678118654752440;
    double2 a[4], b[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      a[n] = cadd(v[n], v[n + 4]);
      b[n] = csub(v[n], v[n + 4]);
    }
    b[1] = make_double2(c * (b[1].x + b[1].y), c * (b[1].y - b[1].x));
    b[2] = mul_mi(b[2]);
    b[3] = make_double2(c * (b[3].y - b[3].x), -c * (b[3].x + b[3].y));
    dft4(a[0], a[1], a[2], a[3]);
    dft4(b[0], b[1], b[2], b[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = a[k];
      v[2 * k + 1] = b[k];
    }
  }
}

template <int LOGM, int I>
__device__ inline void fft_pass(double2* buf, const double2* __restrict__ tw, int tid)
{
  constexpr int M = 1 << LOGM;
  constexpr int LR = FftShape<LOGM>::lr(I), R = 1 << LR;
  constexpr int LOGL = LOGM - 3 * I, L = 1 << LOGL, LP = L >> LR;
#pragma unroll
  for (int t0 = 0; t0 < M / R; t0 += kStrainBlock) {
    const int t = t0 + tid;
    if (M / R % kStrainBlock == 0 || t < M / R) {
      const int g = t >> (LOGL - LR), n1 = t & (LP - 1);
      const int base = g * L + n1;
      // W_L^{n1 k2} = W_M^{(M / L) n1 k2}; tw holds W_M^j for j < M / 2, W_M^{j + M/2} = -W_M^j.
      // The twiddle loads are issued first, so that their latency overlaps the LDS reads and
      // the R-point DFT.
      double2 wv[R];
      if constexpr (LP > 1) {
#pragma unroll
        for (int k2 = 1; k2 < R; ++k2) wv[k2] = tw[((n1 * k2) << (LOGM - LOGL)) & (M / 2 - 1)];
      }
      double2 v[R];
#pragma unroll
      for (int n2 = 0; n2 < R; ++n2) v[n2] = buf[swz(base + LP * n2)];
      dft_small<R>(v);
      if constexpr (LP > 1) {
#pragma unroll
        for (int k2 = 1; k2 < R; ++k2) {
          const double sg = (((n1 * k2) << (LOGM - LOGL)) & (M / 2)) ? -1.0 : 1.0;
          v[k2] = cmul(v[k2], make_double2(sg * wv[k2].x, sg * wv[k2].y));
        }
      }
#pragma unroll
      for (int k2 = 0; k2 < R; ++k2) buf[swz(base + LP * k2)] = v[k2];
    }
  }
  __syncthreads();
  if constexpr (I + 1 < FftShape<LOGM>::NP) fft_pass<LOGM, I + 1>(buf, tw, tid);
}

// One workgroup per segment of n = 2M samples.  LDS: the M complex points (buf), then, once the
// spectrum is in registers, the M + 1 periodogram values over it, the median's sort slots at
// byte sort_off and one gap flag per wavefront at byte flag_off.  A segment with a non-finite
// sample is transformed like any other (the values are discarded) and its gap is found after
// the transform, so that no LDS word has to stay reserved through it.
template <int LOGM>
__global__ __launch_bounds__(kStrainBlock) void strain_sft_kernel(
    const double* __restrict__ x, int64_t n_total, int32_t n_seg, double dt, int32_t w, double psd_scale,
    int32_t k_lo, int32_t n_bins, double s_white, const double2* __restrict__ tw, const double2* __restrict__ rtw,
    double* __restrict__ bins, double* __restrict__ psd, int32_t* __restrict__ keep, int32_t sort_off,
    int32_t flag_off)
{
  constexpr int M = 1 << LOGM;
  extern __shared__ double2 buf[];
  double* U = reinterpret_cast<double*>(buf);   // the periodogram, after the transform
  const int row = blockIdx.x;
  const int det = row / n_seg, seg = row - det * n_seg;
  const double* xs = x + (int64_t)det * n_total + (int64_t)seg * 2 * M;
  const int tid = threadIdx.x;
  bool bad = false;
  // z[m] = x[2m] + i x[2m+1] (one 16-byte load per point where the segment is 16-byte
  // aligned), in batches of up to 8 points per thread whose loads are all issued before the
  // first is used
  {
    constexpr int NL = (M + kStrainBlock - 1) / kStrainBlock, NB = NL < 8 ? NL : 8;
    const bool al = (reinterpret_cast<uintptr_t>(xs) & 15) == 0;
    const double2* xs2 = reinterpret_cast<const double2*>(xs);
#pragma unroll
    for (int r0 = 0; r0 < NL; r0 += NB) {
      double2 z[NB];
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        const int m = tid + (r0 + r) * kStrainBlock;
        if (M % kStrainBlock == 0 || m < M) z[r] = al ? xs2[m] : make_double2(xs[2 * m], xs[2 * m + 1]);
      }
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        const int m = tid + (r0 + r) * kStrainBlock;
        if (M % kStrainBlock == 0 || m < M) {
          bad |= !(isfinite(z[r].x) && isfinite(z[r].y));
          buf[swz(m)] = z[r];
        }
      }
    }
  }
  __syncthreads();
  double* bo = bins + (int64_t)row * 2 * n_bins;
  double* po = psd + (int64_t)row * n_bins;
  fft_pass<LOGM, 0>(buf, tw, tid);
  // real-transform bins, pair (k, M - k) per work item; rtw[k] = e^{-2 pi i k / n}, k <= M/2.
  // The band bins go out as dt X[k]; the periodogram |X[k]|^2 stays in registers until every
  // item has read the spectrum, then overlays it in LDS.
  constexpr int NPAIR = (M / 2 + kStrainBlock) / kStrainBlock;   // ceil((M/2 + 1) / block)
  double pk[NPAIR], pm[NPAIR];
  double2 rtk[NPAIR];
#pragma unroll
  for (int r = 0; r < NPAIR; ++r) {
    const int k = tid + r * kStrainBlock;
    rtk[r] = rtw[k <= M / 2 ? k : M / 2];   // all issued before the first is used
  }
#pragma unroll
  for (int r = 0; r < NPAIR; ++r) {
    const int k = tid + r * kStrainBlock;
    pk[r] = pm[r] = 0.0;
    if (k <= M / 2) {
      const int kk = (M - k) & (M - 1);  // M - k, with Z[M] = Z[0]
      const double2 a = buf[swz(fft_pos<LOGM>(k))], b = buf[swz(fft_pos<LOGM>(kk))];
      const double2 e = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));   // (Z[k] + conj Z[M-k]) / 2
      const double2 o = make_double2(0.5 * (a.x - b.x), 0.5 * (a.y + b.y));   // (Z[k] - conj Z[M-k]) / 2
      const double2 rt = rtk[r];
      const double2 ro = cmul(rt, o);
      const double2 Xk = make_double2(e.x + ro.y, e.y - ro.x);                // e - i ro
      // X[M - k] from the same pair with the roles exchanged: e' = conj(e), o' = -conj(o),
      // e^{-2 pi i (M-k)/n} = -conj(e^{-2 pi i k / n})
      const double2 ro2 = cmul(make_double2(-rt.x, rt.y), make_double2(-o.x, o.y));
      const double2 Xm = make_double2(e.x + ro2.y, -e.y - ro2.x);
      const int im = M - k - k_lo;   // band index of X[M - k] (the Nyquist bin for k = 0)
      if (k - k_lo >= 0 && k - k_lo < n_bins) {
        bo[2 * (k - k_lo)] = dt * Xk.x;
        bo[2 * (k - k_lo) + 1] = dt * Xk.y;
      }
      if (2 * k != M && im >= 0 && im < n_bins) {
        bo[2 * im] = dt * Xm.x;
        bo[2 * im + 1] = dt * Xm.y;
      }
      pk[r] = fma(Xk.x, Xk.x, Xk.y * Xk.y);
      pm[r] = fma(Xm.x, Xm.x, Xm.y * Xm.y);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NPAIR; ++r) {
    const int k = tid + r * kStrainBlock;
    if (k <= M / 2) {
      U[k] = pk[r];
      if (2 * k != M) U[M - k] = pm[r];
    }
  }
  int* gap = reinterpret_cast<int*>(reinterpret_cast<char*>(buf) + flag_off);
  const bool wave_bad = __ballot(bad) != 0;
  if ((tid & 63) == 0) gap[tid >> 6] = wave_bad ? 1 : 0;
  __syncthreads();
  bool seg_bad = false;
#pragma unroll
  for (int v = 0; v < kStrainBlock / 64; ++v) seg_bad = seg_bad || gap[v] != 0;
  if (seg_bad) {
    // a gap: zeros over the band bins this thread wrote above (same addresses, same thread, so
    // the zeros land last), a zero PSD and keep = 0
#pragma unroll
    for (int r = 0; r < NPAIR; ++r) {
      const int k = tid + r * kStrainBlock;
      if (k <= M / 2) {
        const int im = M - k - k_lo;
        if (k - k_lo >= 0 && k - k_lo < n_bins) {
          bo[2 * (k - k_lo)] = 0.0;
          bo[2 * (k - k_lo) + 1] = 0.0;
        }
        if (2 * k != M && im >= 0 && im < n_bins) {
          bo[2 * im] = 0.0;
          bo[2 * im + 1] = 0.0;
        }
      }
    }
    for (int i = tid; i < n_bins; i += kStrainBlock) po[i] = 0.0;
    if (tid == 0) keep[row] = 0;
    return;
  }
  const int N = 2 * w + 1;
  auto block_of = [&](int k) {   // first bin of the block centred on k, shifted at the ends of [0, M]
    int s0 = k - w;
    s0 = s0 < 0 ? 0 : s0;
    return s0 + 2 * w > M ? M - 2 * w : s0;
  };
  if (s_white > 0.0) {
    // a known white PSD: no estimate
    for (int i = tid; i < n_bins; i += blockDim.x) po[i] = s_white;
  } else if (w <= kMaxSortW || (LOGM >= 7 && w <= kMaxKeyW)) {
    const int lane = tid & 63, wv = tid >> 6;
    // every wavefront walks its chunks of 64 band bins (wave-uniform loop)
    for (int c0 = wv * 64; c0 < n_bins; c0 += blockDim.x) {
      const int kb = k_lo + c0;
      int u0 = kb - w;                          // the union of the chunk's blocks: [u0, u0 + L)
      u0 = u0 < 0 ? 0 : u0;
      u0 = u0 + 2 * w > M ? M - 2 * w : u0;
      int u1 = kb + 63 - w;
      u1 = u1 < 0 ? 0 : u1;
      u1 = u1 + 2 * w > M ? M - 2 * w : u1;
      const int L = u1 + N - u0;                // <= 64 + 2w
      const int i = c0 + lane;
      const int s0r = block_of(k_lo + i) - u0;  // the lane's block in the union
      char* slot = reinterpret_cast<char*>(buf) + sort_off + wv * sort_slot(w);
      double med = 0.0;
      if (w <= kMaxSortW) {
        if (!key_medians<2>(U, u0, L, s0r, w, lane, i < n_bins, slot, med)) med = pair_median(U, u0, L, s0r, w, lane, slot);
      } else if constexpr (LOGM >= 7) {   // 2w <= M
        if (!key_medians<4>(U, u0, L, s0r, w, lane, i < n_bins, slot, med) && i < n_bins) med = rank_median(U + u0 + s0r, w);
      }
      if (i < n_bins) po[i] = psd_scale * (dt * dt) * med;
    }
  } else {
    for (int i = tid; i < n_bins; i += blockDim.x)
      po[i] = psd_scale * (dt * dt) * rank_median(U + block_of(k_lo + i), w);
  }
  if (tid == 0) keep[row] = 1;
}

// ---------------------------------------------------------------------------- lengths that are no power of two
// Bluestein's algorithm (L. I. Bluestein, IEEE Trans. Audio Electroacoust. 18, 451 (1970)): with
// b[j] = e^{i pi j^2 / M} the M-point DFT of z (M = n / 2, packed as above) is
//   Z[k] = conj(b[k]) sum_j (z[j] conj(b[j])) b[k - j],
// a convolution, taken as a cyclic one of length L >= 2M - 1 by two L-point transforms in LDS.
// L = R0 S with R0 in {8, 9, 10, 12} (16 for the largest) and S in {64, 128, 256, 512}: a first
// pass of radix R0 and passes of radix 8 (2 or 4 for the leftover bits) over the R0 sub-transforms
// of S points.  A power of two alone would take 8192 points where 4608 do (106 s at 40 Hz: M =
// 2120), nearly twice the LDS traffic.
//
// Bound: LDS traffic.  Of the eight passes, the first reads the strain itself, the last of the
// forward transform, the multiplication with the spectrum of b and the first of the inverse run
// on the same points in registers: seven round trips of L points, ~1 MB per segment of 4240
// samples, against 71 KB of strain and bins.  The inverse transform is the transposed (decimation
// in time) flow on the conjugate, which takes the digit-reversed order the forward one leaves, so
// nothing is reordered.  One workgroup of nine wavefronts per CU (162 registers; held to 96 for two
// workgroups it spills) cannot hide what the passes wait for, so a thread reads one root per pass at the
// start and forms the twiddles as its powers, and the spectrum of b a pass ahead.  4396 segments of 4240
// samples (129 h at 40 Hz, every bin): 11.9 ms by the defining sum (strain_dft_kernel, 2.1e10 terms), 0.27 ms
// with every twiddle read where it is used, 0.22 ms so (1.7 TB/s of strain, bins and PSD).
template <int R0, int LOGS>
struct BlueShape {
  static constexpr int S = 1 << LOGS, L = R0 * S;
  static constexpr int items = L / 8 > S ? L / 8 : S;
  static constexpr int threads = (items + 63) / 64 * 64;
  // The last pass's operand is read a pass ahead where that pass has one work item per thread and the
  // registers do not cost a wavefront per SIMD: S = 512 up to 12 wavefronts (one workgroup per CU), not
  // S = 64 (20 k segments of 602 samples: 114 us with it, 109 us without).
  static constexpr int last = 1 << FftShape<LOGS>::lr(FftShape<LOGS>::NP - 1);   // its radix
  static constexpr bool ahead = LOGS == 9 && L / last <= threads && threads <= 768;
};

// e^{-2 pi i m / R} of the composite small transforms
template <int R>
struct Unit;
template <>
struct Unit<9> {
  static constexpr double c[9] = {
    1.00000000000000000000, 0.766044443118978035202, 0.173648177666930348852, -0.500000000000000000000,
    -0.939692620785908384054, -0.939692620785908384054, -0.500000000000000000000, 0.173648177666930348852,
    0.766044443118978035202};
  static constexpr double s[9] = {
    0.0, -0.642787609686539326323, -0.984807753012208059367, -0.866025403784438646764, -0.342020143325668733044,
    0.342020143325668733044, 0.866025403784438646764, 0.984807753012208059367, 0.642787609686539326323};
};
template <>
struct Unit<10> {
  static constexpr double c[10] = {
    1.00000000000000000000, 0.809016994374947424102, 0.309016994374947424102, -0.309016994374947424102,
    -0.809016994374947424102, -1.00000000000000000000, -0.809016994374947424102, -0.309016994374947424102,
    0.309016994374947424102, 0.809016994374947424102};
  static constexpr double s[10] = {
    0.0, -0.587785252292473129169, -0.951056516295153572116, -0.951056516295153572116, -0.587785252292473129169,
    0.0, 0.587785252292473129169, 0.951056516295153572116, 0.951056516295153572116, 0.587785252292473129169};
};
template <>
struct Unit<12> {
  static constexpr double c[12] = {
    1.00000000000000000000, 0.866025403784438646764, 0.500000000000000000000, 0.0, -0.500000000000000000000,
    -0.866025403784438646764, -1.00000000000000000000, -0.866025403784438646764, -0.500000000000000000000, 0.0,
    0.500000000000000000000, 0.866025403784438646764};
  static constexpr double s[12] = {
    0.0, -0.500000000000000000000, -0.866025403784438646764, -1.00000000000000000000, -0.866025403784438646764,
    -0.500000000000000000000, 0.0, 0.500000000000000000000, 0.866025403784438646764, 1.00000000000000000000,
    0.866025403784438646764, 0.500000000000000000000};
};
template <>
struct Unit<16> {
  static constexpr double c[16] = {
    1.00000000000000000000, 0.923879532511286756128, 0.707106781186547524401, 0.382683432365089771728, 0.0,
    -0.382683432365089771728, -0.707106781186547524401, -0.923879532511286756128, -1.00000000000000000000,
    -0.923879532511286756128, -0.707106781186547524401, -0.382683432365089771728, 0.0, 0.382683432365089771728,
    0.707106781186547524401, 0.923879532511286756128};
  static constexpr double s[16] = {
    0.0, -0.382683432365089771728, -0.707106781186547524401, -0.923879532511286756128, -1.00000000000000000000,
    -0.923879532511286756128, -0.707106781186547524401, -0.382683432365089771728, 0.0, 0.382683432365089771728,
    0.707106781186547524401, 0.923879532511286756128, 1.00000000000000000000, 0.923879532511286756128,
    0.707106781186547524401, 0.382683432365089771728};
};
template <int R>
__device__ inline double2 unit_root(int m)
{
  return make_double2(Unit<R>::c[m], Unit<R>::s[m]);
}

template <int R>
__device__ inline void dft_any(double2* v);

// R = A B points by B transforms of A points, the twiddles, and A transforms of B points
template <int A, int B>
__device__ inline void dft_ab(double2* v)
{
  double2 y[A * B];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) {
    double2 u[A];
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) u[n1] = v[B * n1 + n2];
    dft_any<A>(u);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) y[k1 * B + n2] = n2 * k1 == 0 ? u[k1] : cmul(u[k1], unit_root<A * B>(n2 * k1));
  }
#pragma unroll
  for (int k1 = 0; k1 < A; ++k1) {
    dft_any<B>(y + k1 * B);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = y[k1 * B + k2];
  }
}

template <int R>
__device__ inline void dft_any(double2* v)
{
  if constexpr (R == 3) {
    constexpr double s3 = 0.86602540378443864676;
    const double2 t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const double2 m = make_double2(fma(-0.5, t.x, v[0].x), fma(-0.5, t.y, v[0].y));
    v[0] = cadd(v[0], t);
    v[1] = make_double2(fma(s3, d.y, m.x), fma(-s3, d.x, m.y));
    v[2] = make_double2(fma(-s3, d.y, m.x), fma(s3, d.x, m.y));
  } else if constexpr (R == 5) {
    constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;
    constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;
    const double2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]), t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
    const double2 m1 = make_double2(fma(c1, t1.x, fma(c2, t2.x, v[0].x)), fma(c1, t1.y, fma(c2, t2.y, v[0].y)));
    const double2 m2 = make_double2(fma(c2, t1.x, fma(c1, t2.x, v[0].x)), fma(c2, t1.y, fma(c1, t2.y, v[0].y)));
    const double2 q1 = make_double2(fma(s1, t3.x, s2 * t4.x), fma(s1, t3.y, s2 * t4.y));
    const double2 q2 = make_double2(fma(s2, t3.x, -s1 * t4.x), fma(s2, t3.y, -s1 * t4.y));
    v[0] = cadd(v[0], cadd(t1, t2));
    v[1] = make_double2(m1.x + q1.y, m1.y - q1.x);
    v[4] = make_double2(m1.x - q1.y, m1.y + q1.x);
    v[2] = make_double2(m2.x + q2.y, m2.y - q2.x);
    v[3] = make_double2(m2.x - q2.y, m2.y + q2.x);
  } else if constexpr (R == 9) {
    dft_ab<3, 3>(v);
  } else if constexpr (R == 10) {
    dft_ab<5, 2>(v);
  } else if constexpr (R == 12) {
    dft_ab<3, 4>(v);
  } else if constexpr (R == 16) {
    dft_ab<4, 4>(v);
  } else {
    dft_small<R>(v);
  }
}

// The powers w, w^2 .. w^(R-1) of a root, each from the two halves of its exponent (three products deep for R <= 9,
// four above)
template <int R>
__device__ inline void powers(double2 w, double2* p)
{
  p[1] = w;
#pragma unroll
  for (int k = 2; k < R; ++k) p[k] = cmul(p[k / 2], p[k - k / 2]);
}

// Pass I over the S-point sub-transforms (FftShape<LOGS>): forward (decimation in frequency, as
// fft_pass), or INV its transpose, which multiplies by the twiddles before the R-point DFT.  The
// last forward pass has no twiddles; it multiplies by the spectrum of b, conjugates and goes on
// with the transpose of itself.  A work item's twiddles are powers of one root per pass, which the
// kernel reads at its start (wp[I]); the spectrum of b (h) is read a pass ahead.
template <int R0, int LOGS, int I, bool INV>
__device__ inline void blue_pass(double2* buf, const double2* wp, const double2* __restrict__ bh, double2* h, int tid)
{
  using Sh = BlueShape<R0, LOGS>;
  using Ff = FftShape<LOGS>;
  constexpr int LR = Ff::lr(I), R = 1 << LR;
  constexpr int LOGL = LOGS - 3 * I, LP = 1 << (LOGL - LR), N = Sh::L / R;
  // the pass before the last reads the spectrum of b for it
  if constexpr (!INV && I == Ff::NP - 2 && Sh::ahead) {
    if (Sh::L / Sh::last == Sh::threads || tid < Sh::L / Sh::last) {
#pragma unroll
      for (int k = 0; k < Sh::last; ++k) h[k] = bh[tid * Sh::last + k];
    }
  }
#pragma unroll
  for (int t0 = 0; t0 < N; t0 += Sh::threads) {
    const int t = t0 + tid;
    if (N % Sh::threads == 0 || t < N) {
      const int n1 = t & (LP - 1);
      const int base = ((t >> (LOGL - LR)) << LOGL) + n1;
      double2 v[R];
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = buf[swz(base + LP * k)];
      if constexpr (LP == 1) {
        if constexpr (!Sh::ahead) {
#pragma unroll
          for (int k = 0; k < R; ++k) h[k] = bh[base + k];
        }
        dft_small<R>(v);
#pragma unroll
        for (int k = 0; k < R; ++k) {
          v[k] = cmul(v[k], h[k]);
          v[k].y = -v[k].y;
        }
        dft_small<R>(v);
      } else {
        double2 wv[R];
        powers<R>(wp[I], wv);   // t and t0 + tid have the same n1: threads is a multiple of LP
        if constexpr (INV) {
#pragma unroll
          for (int k2 = 1; k2 < R; ++k2) v[k2] = cmul(v[k2], wv[k2]);
        }
        dft_small<R>(v);
        if constexpr (!INV) {
#pragma unroll
          for (int k2 = 1; k2 < R; ++k2) v[k2] = cmul(v[k2], wv[k2]);
        }
      }
#pragma unroll
      for (int k = 0; k < R; ++k) buf[swz(base + LP * k)] = v[k];
    }
  }
  __syncthreads();
  if constexpr (!INV && LP > 1) blue_pass<R0, LOGS, I + 1, false>(buf, wp, bh, h, tid);
  else if constexpr (I > 0) blue_pass<R0, LOGS, I - 1, true>(buf, wp, bh, h, tid);
}

// Root of a work item of pass I: W_{2^LOGL}^{n1}, n1 = tid mod LP
template <int R0, int LOGS, int I>
__device__ inline void blue_roots(const double2* __restrict__ ws, double2* wp, int tid)
{
  constexpr int LOGL = LOGS - 3 * I, LP = 1 << (LOGL - FftShape<LOGS>::lr(I));
  if constexpr (LP > 1) {
    static_assert(BlueShape<R0, LOGS>::threads % LP == 0, "one root per thread");
    wp[I] = ws[(tid & (LP - 1)) << (LOGS - LOGL)];
    blue_roots<R0, LOGS, I + 1>(ws, wp, tid);
  }
}

struct BlueTables {
  const double2* b;     // [M] conj(b[j]) = e^{-i pi j^2 / M}
  const double2* bh;    // [L] spectrum of b over L, in the order the forward transform leaves
  const double2* wl;    // [L] e^{-2 pi i j / L}
  const double2* ws;    // [S] e^{-2 pi i j / S}
  const double2* rtw;   // [M/2 + 1] e^{-2 pi i k / n}
};

// One workgroup per segment; the PSD is the given white level (no estimate).
template <int R0, int LOGS>
// (S = 64 held to 128 registers, four wavefronts per SIMD, at 16 to 20 bytes of scratch a lane: 20 k segments of 602
// samples 109 -> 94 us.  The 16 wavefronts of the largest size, L = 8192, leave 128 registers each and spill 148 bytes.)
__global__ __launch_bounds__((BlueShape<R0, LOGS>::threads))
__attribute__((amdgpu_waves_per_eu(LOGS == 6 ? 4 : 1))) void strain_blue_kernel(
    const double* __restrict__ x, int64_t n_total, int32_t n_seg, int32_t M, double dt, double s_white, int32_t k_lo,
    int32_t n_bins, BlueTables tt, double* __restrict__ bins, double* __restrict__ psd, int32_t* __restrict__ keep)
{
  using Sh = BlueShape<R0, LOGS>;
  constexpr int S = Sh::S, NT = Sh::threads;
  extern __shared__ double2 buf[];
  __shared__ int s_bad;
  const int row = blockIdx.x;
  const int det = row / n_seg, seg = row - det * n_seg;
  const double* xs = x + (int64_t)det * n_total + (int64_t)seg * 2 * M;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  bool bad = false;
  // the roots of the passes' twiddles
  double2 wp[FftShape<LOGS>::NP], h[8], w0 = make_double2(1.0, 0.0);
  blue_roots<R0, LOGS, 0>(tt.ws, wp, tid);
  if (tid < S) w0 = tt.wl[tid];
  if (tid < S) {
    // z[j] conj(b[j]), zero from M on, through the radix-R0 pass
    const bool al = (reinterpret_cast<uintptr_t>(xs) & 15) == 0;
    const double2* xs2 = reinterpret_cast<const double2*>(xs);
    double2 v[R0];
#pragma unroll
    for (int k = 0; k < R0; ++k) {
      const int j = tid + S * k;
      v[k] = make_double2(0.0, 0.0);
      if (j < M) {
        const double2 z = al ? xs2[j] : make_double2(xs[2 * j], xs[2 * j + 1]);
        bad |= !(isfinite(z.x) && isfinite(z.y));
        v[k] = cmul(z, tt.b[j]);
      }
    }
    dft_any<R0>(v);
    double2 wv[R0];
    powers<R0>(w0, wv);
#pragma unroll
    for (int k = 0; k < R0; ++k) buf[swz(tid + S * k)] = k == 0 ? v[0] : cmul(v[k], wv[k]);
  }
  if (bad) s_bad = 1;
  __syncthreads();
  blue_pass<R0, LOGS, 0, false>(buf, wp, tt.bh, h, tid);
  if (tid < S) {
    double2 v[R0], wv[R0];
    powers<R0>(w0, wv);
#pragma unroll
    for (int k = 0; k < R0; ++k) v[k] = k == 0 ? buf[swz(tid)] : cmul(buf[swz(tid + S * k)], wv[k]);
    dft_any<R0>(v);
    // Z[j] = conj(b[j]) conj(v): each thread's points are its own, no barrier in between
#pragma unroll
    for (int k = 0; k < R0; ++k) {
      const int j = tid + S * k;
      if (j < M) buf[swz(j)] = cmul(tt.b[j], make_double2(v[k].x, -v[k].y));
    }
  }
  __syncthreads();
  double* bo = bins + (int64_t)row * 2 * n_bins;
  double* po = psd + (int64_t)row * n_bins;
  const bool gap = s_bad != 0;
  // the bins of the real transform, as in strain_sft_kernel, pair (k, M - k) per thread
  for (int k = tid; 2 * k <= M; k += NT) {
    const int im = M - k - k_lo, ik = k - k_lo;
    const bool wk = ik >= 0 && ik < n_bins, wm = 2 * k != M && im >= 0 && im < n_bins;
    if (!wk && !wm) continue;
    const double2 a = buf[swz(k)], b = buf[swz(k == 0 ? 0 : M - k)];
    const double2 e = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    const double2 o = make_double2(0.5 * (a.x - b.x), 0.5 * (a.y + b.y));
    const double2 rt = tt.rtw[k];
    const double2 ro = cmul(rt, o), ro2 = cmul(make_double2(-rt.x, rt.y), make_double2(-o.x, o.y));
    if (wk) {
      bo[2 * ik] = gap ? 0.0 : dt * (e.x + ro.y);
      bo[2 * ik + 1] = gap ? 0.0 : dt * (e.y - ro.x);
    }
    if (wm) {
      bo[2 * im] = gap ? 0.0 : dt * (e.x + ro2.y);
      bo[2 * im + 1] = gap ? 0.0 : dt * (-e.y - ro2.x);
    }
  }
  for (int i = tid; i < n_bins; i += NT) po[i] = gap ? 0.0 : s_white;
  if (tid == 0) keep[row] = gap ? 0 : 1;
}

// The other segments whose length is not a power of two (few or many samples): the band bins by their defining sum
// X[k] = sum_j x_j e^{-2 pi i j k / n} (Eq. d_SFT), one bin per thread, the segment in LDS (read
// as a broadcast), the twiddle advanced by the rotation e^{-2 pi i k / n} and re-anchored from
// the exact table W[m] = e^{-2 pi i m / n} every kAnchor samples (rounding drift <= kAnchor eps).  SHORT segments (n <
// kBlueMinN), one wavefront each, hold the table in LDS too: kShortAnchor twiddles are one entry times the first powers
// of the rotation, all from the table, so that nothing drifts and no product waits for the one before (20 k segments
// of 66 samples, 16 bins: 31 us by the long ones' rotation, 54 us with every twiddle read, 26 us so).
// The PSD is the given white level (no estimate).
constexpr int kAnchor = 256, kShortAnchor = 8;

template <bool SHORT>

__global__ __launch_bounds__(kStrainBlock) void strain_dft_kernel(
    const double* __restrict__ x, int64_t n_total, int32_t n_seg, int32_t n, double dt, double s_white,
    int32_t k_lo, int32_t n_bins, const double2* __restrict__ W, double* __restrict__ bins, double* __restrict__ psd,
    int32_t* __restrict__ keep)
{
  extern __shared__ __align__(16) double xl[];   // the segment, n values; SHORT: then the table, n pairs (n is even)
  __shared__ int s_bad;
  const int row = blockIdx.x;
  const int det = row / n_seg, seg = row - det * n_seg;
  const double* xs = x + (int64_t)det * n_total + (int64_t)seg * n;
  const int tid = threadIdx.x;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  bool bad = false;
  for (int j = tid; j < n; j += blockDim.x) {
    const double v = xs[j];
    bad = bad || !isfinite(v);
    xl[j] = v;
    if constexpr (SHORT) reinterpret_cast<double2*>(xl + n)[j] = W[j];
  }
  if (bad) s_bad = 1;
  __syncthreads();
  double* bo = bins + (int64_t)row * 2 * n_bins;
  double* po = psd + (int64_t)row * n_bins;
  if (s_bad) {
    for (int i = tid; i < n_bins; i += blockDim.x) {
      bo[2 * i] = 0.0;
      bo[2 * i + 1] = 0.0;
      po[i] = 0.0;
    }
    if (tid == 0) keep[row] = 0;
    return;
  }
  if constexpr (SHORT) {
    const double2* wl = reinterpret_cast<const double2*>(xl + n);
    for (int i = tid; i < n_bins; i += blockDim.x) {
      const int k = k_lo + i;
      double2 r[kShortAnchor];   // e^{-2 pi i t k / n}
      int step = 0;
#pragma unroll
      for (int t = 0; t < kShortAnchor; ++t) {
        r[t] = wl[step];
        step += k;
        step = step >= n ? step - n : step;
      }
      double re = 0.0, im = 0.0;
      int idx = 0;   // (j k) mod n
      for (int j = 0; j < n; j += kShortAnchor) {
        const double2 w0 = wl[idx];
#pragma unroll
        for (int t = 0; t < kShortAnchor; ++t) {
          const double2 wv = t ? cmul(w0, r[t]) : w0;
          const double xj = j + t < n ? xl[j + t] : 0.0;
          re = fma(xj, wv.x, re);
          im = fma(xj, wv.y, im);
        }
        idx += step;
        idx = idx >= n ? idx - n : idx;
      }
      bo[2 * i] = dt * re;
      bo[2 * i + 1] = dt * im;
      po[i] = s_white;
    }
    if (tid == 0) keep[row] = 1;
    return;
  }
  for (int i = tid; i < n_bins; i += blockDim.x) {
    const int k = k_lo + i;
    const double2 r = W[k % n];
    const int step = (int)(((int64_t)kAnchor * k) % n);
    double re = 0.0, im = 0.0;
    int idx = 0;   // (j0 k) mod n
    for (int j0 = 0; j0 < n; j0 += kAnchor) {
      double2 wv = W[idx];
      const int j1 = j0 + kAnchor < n ? j0 + kAnchor : n;
      for (int j = j0; j < j1; ++j) {
        const double xj = xl[j];
        re = fma(xj, wv.x, re);
        im = fma(xj, wv.y, im);
        wv = cmul(wv, r);
      }
      idx += step;
      idx = idx >= n ? idx - n : idx;
    }
    bo[2 * i] = dt * re;
    bo[2 * i + 1] = dt * im;
    po[i] = s_white;
  }
  if (tid == 0) keep[row] = 1;
}

}  // namespace

static sft_status strain_fail(sft_status st, const char* msg) { return sft_set_error(st, msg); }

// Segment lengths of strain_blue_kernel.  L = 8192 points (128 KiB of LDS) hold the n - 1 of the convolution, and the
// next size does not fit the 160 KiB of a CU.  The smallest transform, L = 512, takes about the same time for every
// n up to 512, the defining sum (strain_dft_kernel) one that grows with n: 20 k segments, every bin, 36 us against 15
// us at n = 18, 38 us against 32 us at 66.  Below and above these lengths the defining sum.
constexpr int kBlueMinN = 82, kBlueMaxN = 8192;
static bool blue_length(int n) { return (n & (n - 1)) != 0 && n >= kBlueMinN && n <= kBlueMaxN; }

typedef void (*BlueFn)(const double*, int64_t, int32_t, int32_t, double, double, int32_t, int32_t, BlueTables, double*,
                       double*, int32_t*);
struct BlueSize {
  int r0 = 0, logs = 0, threads = 0;
  BlueFn fn = nullptr;
  int S() const { return 1 << logs; }
  int L() const { return r0 << logs; }
};

template <int R0, int LOGS>
static void blue_offer(int need, BlueSize& best)
{
  using Sh = BlueShape<R0, LOGS>;
  if (Sh::L < need || (best.fn && best.L() <= Sh::L)) return;
  best.r0 = R0;
  best.logs = LOGS;
  best.threads = Sh::threads;
  best.fn = strain_blue_kernel<R0, LOGS>;
}

template <int LOGS>
static void blue_offer_s(int need, BlueSize& best)
{
  blue_offer<8, LOGS>(need, best);
  blue_offer<9, LOGS>(need, best);
  blue_offer<10, LOGS>(need, best);
  blue_offer<12, LOGS>(need, best);
}

// the smallest transform that holds the convolution of n / 2 points
static BlueSize blue_size(int n)
{
  BlueSize b;
  blue_offer_s<6>(n - 1, b);
  blue_offer_s<7>(n - 1, b);
  blue_offer_s<8>(n - 1, b);
  blue_offer_s<9>(n - 1, b);
  blue_offer<16, 9>(n - 1, b);
  return b;
}

// Tables of a segment length n, in long double rounded once to FP64: for n a power of two,
// tw[j] = e^{-2 pi i j / M} (j < M/2, M = n/2) and rtw[k] = e^{-2 pi i k / n} (k <= M/2); for the
// lengths of strain_blue_kernel its tables; for other n W[m] = e^{-2 pi i m / n} (m < n).
// Built on a device's first call for n and kept there until the process ends (tens of KB per
// length, up to 0.4 MB for a length that is no power of two), so that later calls only launch.
struct TwTables {
  double2* tw = nullptr;
  double2* rtw = nullptr;
  double2* W = nullptr;
  double2* blue = nullptr;   // one block: b [M], bh [L], wl [L], ws [S], rtw [M/2 + 1]
};

// a complex number in long double (the library's product checks every factor for infinities)
struct Cld {
  long double re = 0.0L, im = 0.0L;
};
static Cld operator+(Cld a, Cld b) { return {a.re + b.re, a.im + b.im}; }
static Cld operator-(Cld a, Cld b) { return {a.re - b.re, a.im - b.im}; }
static Cld operator*(Cld a, Cld b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }

static Cld unit_ld(int64_t num, int64_t den)   // e^{-2 pi i num / den}
{
  const long double a = -2.0L * 3.141592653589793238462643383279502884L * (long double)(num % den) / (long double)den;
  Cld r;
  sincosl(a, &r.im, &r.re);
  return r;
}

// DFT of x[0], x[s], x[2 s], ... (m points, m s of the length whose roots w are) into y, by halving down to an odd
// length
static void host_dft(const Cld* x, int m, int s, const Cld* w, Cld* y)
{
  if (m % 2 == 0) {
    const int h = m / 2;
    host_dft(x, h, 2 * s, w, y);
    host_dft(x + s, h, 2 * s, w, y + h);
    for (int k = 0; k < h; ++k) {
      const Cld e = y[k], o = w[(int64_t)k * s] * y[h + k];
      y[k] = e + o;
      y[h + k] = e - o;
    }
    return;
  }
  for (int k = 0; k < m; ++k) {
    Cld t;
    for (int j = 0; j < m; ++j) t = t + x[(int64_t)j * s] * w[(int64_t)(j * k % m) * s];
    y[k] = t;
  }
}

// The L-th roots of unity serve the DFT, the first pass and (every L / S-th) the others: one sine and cosine each, as
// with the defining sum's table (first call for n = 4240, kernel included: 14.8 ms with a sine and a cosine at every
// use, 1.3 ms so; 2.8 ms by the defining sum).
static std::vector<double2> blue_tables(int n, const BlueSize& z)
{
  const int M = n / 2, L = z.L(), S = z.S();
  std::vector<double2> h;
  h.reserve((size_t)M + 2 * L + S + M / 2 + 1);
  auto put = [&](Cld v) { h.push_back(make_double2((double)v.re, (double)v.im)); };
  std::vector<Cld> w(L), b(L), f(L);
  for (int j = 0; j <= L / 2; ++j) {
    w[j] = unit_ld(j, L);
    w[(L - j) % L] = {w[j].re, -w[j].im};
  }
  for (int64_t j = 0; j < M; ++j) {
    const Cld c = unit_ld(j * j % n, n);   // e^{-i pi j^2 / M}
    put(c);
    b[j] = {c.re, -c.im};
    if (j > 0) b[L - j] = b[j];
  }
  host_dft(b.data(), L, 1, w.data(), f.data());
  // position of output k of the forward transform: radix-R0 digit first, then the S-point order
  std::vector<Cld> r(L);
  for (int k = 0; k < L; ++k) {
    int q = k / z.r0, p = 0, len = S;
    while (len > 1) {
      const int rad = len >= 8 ? 8 : len;
      len /= rad;
      p += (q % rad) * len;
      q /= rad;
    }
    r[(k % z.r0) * S + p] = {f[k].re / (long double)L, f[k].im / (long double)L};
  }
  for (const Cld& v : r) put(v);
  for (int j = 0; j < L; ++j) put(w[j]);
  for (int j = 0; j < S; ++j) put(w[(int64_t)j * z.r0]);
  for (int k = 0; k <= M / 2; ++k) put(unit_ld(k, n));
  return h;
}

static hipError_t upload(const std::vector<double2>& h, double2** d)
{
  hipError_t e = hipMalloc((void**)d, h.size() * sizeof(double2));
  if (e == hipSuccess) e = hipMemcpy(*d, h.data(), h.size() * sizeof(double2), hipMemcpyHostToDevice);
  if (e != hipSuccess && *d) {
    (void)hipFree(*d);
    *d = nullptr;
  }
  return e;
}

static hipError_t twiddle_tables(int n, TwTables& out)
{
  static std::mutex mu;
  static std::map<std::pair<int, int>, TwTables> cache;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  const auto it = cache.find({dev, n});
  if (it != cache.end()) {
    out = it->second;
    return hipSuccess;
  }
  const long double pi = 3.141592653589793238462643383279502884L;
  TwTables t;
  if (blue_length(n)) {
    e = upload(blue_tables(n, blue_size(n)), &t.blue);
  } else if ((n & (n - 1)) != 0) {
    std::vector<double2> W(n);
    for (int m = 0; m < n; ++m) {
      const long double a = -2.0L * pi * (long double)m / (long double)n;
      W[m] = make_double2((double)cosl(a), (double)sinl(a));
    }
    e = upload(W, &t.W);
  } else {
    const int M = n / 2;
    std::vector<double2> tw(M / 2 > 0 ? M / 2 : 1), rtw(M / 2 + 1);
    for (int j = 0; j < M / 2; ++j) {
      const long double a = -2.0L * pi * (long double)j / (long double)M;
      tw[j] = make_double2((double)cosl(a), (double)sinl(a));
    }
    for (int k = 0; k <= M / 2; ++k) {
      const long double a = -2.0L * pi * (long double)k / (long double)n;
      rtw[k] = make_double2((double)cosl(a), (double)sinl(a));
    }
    e = upload(tw, &t.tw);
    if (e == hipSuccess) e = upload(rtw, &t.rtw);
    if (e != hipSuccess && t.tw) (void)hipFree(t.tw);
  }
  if (e != hipSuccess) return e;
  cache[{dev, n}] = t;
  out = t;
  return hipSuccess;
}

extern "C" sft_status sft_make_sfts(const sft_strain_desc* d, const double* x, double* bins, double* psd, int32_t* keep,
                                    void* hip_stream)
{
  if (!d || !x || !bins || !psd || !keep) return strain_fail(SFT_E_INVALID, "sft_make_sfts: null argument");
  const int n = d->n_samples;
  const bool pow2 = (n & (n - 1)) == 0;
  if (n < 16 || n > 16384 || (n & 1))
    return strain_fail(SFT_E_UNSUPPORTED, "sft_make_sfts: n_samples must be even and in [16, 16384]");
  if (!pow2 && !(d->s_white > 0.0))
    return strain_fail(SFT_E_UNSUPPORTED, "sft_make_sfts: the PSD estimate needs n a power of two (else give s_white)");
  if (d->n_det < 1 || d->n_total < n || !(d->dt > 0.0) || !(d->s_white >= 0.0))
    return strain_fail(SFT_E_INVALID, "sft_make_sfts: bad descriptor");
  const int M = n / 2;
  if (d->k_lo < 0 || d->n_bins < 1 || d->k_lo + d->n_bins - 1 > M)
    return strain_fail(SFT_E_INVALID, "sft_make_sfts: band outside [0, n/2]");
  if (!(d->s_white > 0.0) && (d->psd_w < 0 || 2 * d->psd_w + 1 > M + 1))
    return strain_fail(SFT_E_INVALID, "sft_make_sfts: running-median block wider than the spectrum");
  const int64_t n_seg = d->n_total / n;
  if (n_seg * d->n_det > INT32_MAX) return strain_fail(SFT_E_RANGE, "sft_make_sfts: too many segments");
  hipStream_t st = (hipStream_t)hip_stream;
  TwTables tt;
  hipError_t e = twiddle_tables(n, tt);
  if (e != hipSuccess) return strain_fail(SFT_E_DEVICE, hipGetErrorString(e));
  if (blue_length(n)) {
    const BlueSize z = blue_size(n);
    BlueTables bt;
    bt.b = tt.blue;
    bt.bh = bt.b + M;
    bt.wl = bt.bh + z.L();
    bt.ws = bt.wl + z.L();
    bt.rtw = bt.ws + z.S();
    const size_t lds = (size_t)z.L() * sizeof(double2);
    if (lds > 65536) e = hipFuncSetAttribute((const void*)z.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    // One launch, or with more segments than a grid's row holds (2^32 threads in workgroups of up to 1024) launches of
    // 2^21 segments of one detector
    const int64_t rows = n_seg * d->n_det, most = 1 << 21;
    for (int64_t r0 = 0; r0 < rows && e == hipSuccess;) {
      const int64_t det = r0 / n_seg, seg = r0 - det * n_seg;
      const int64_t nr = rows <= most ? rows : std::min(most, n_seg - seg);
      hipLaunchKernelGGL(z.fn, dim3((unsigned)nr), dim3(z.threads), lds, st, x + det * d->n_total + seg * n, d->n_total,
                         (int32_t)n_seg, M, d->dt, d->s_white, d->k_lo, d->n_bins, bt, bins + r0 * 2 * d->n_bins,
                         psd + r0 * d->n_bins, keep + r0);
      e = hipGetLastError();
      r0 += nr;
    }
    if (e != hipSuccess) return strain_fail(SFT_E_DEVICE, hipGetErrorString(e));
    return SFT_OK;
  }
  if (!pow2) {
    const bool is_short = n < kBlueMinN;
    const auto fn = is_short ? strain_dft_kernel<true> : strain_dft_kernel<false>;
    const size_t lds = (size_t)n * (is_short ? sizeof(double) + sizeof(double2) : sizeof(double));
    if (lds > 65536) e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess && n_seg > 0) {
      hipLaunchKernelGGL(fn, dim3((unsigned)(n_seg * d->n_det)), dim3(is_short ? 64 : kStrainBlock), lds, st, x,
                         d->n_total, (int32_t)n_seg, n, d->dt, d->s_white, d->k_lo, d->n_bins, tt.W, bins, psd, keep);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return strain_fail(SFT_E_DEVICE, hipGetErrorString(e));
    return SFT_OK;
  }
  int logM = 0;
  while ((1 << logM) < M) ++logM;
  double2* d_tw = tt.tw;
  double2* d_rtw = tt.rtw;
  double B = 0.0;
  for (int i = 0; i <= d->psd_w; ++i) B += 1.0 / (double)(2 * d->psd_w + 1 - i);
  const double T = d->dt * n;
  const double psd_scale = 2.0 / (T * B);
  // LDS: the M complex points; the periodogram (M + 1 values), the median's sort slots and the
  // gap flags (each 16-byte aligned after the previous) overlay them once the transform is done
  size_t lds = (size_t)M * sizeof(double2);
  int32_t sort_off = 0;
  int32_t flag_off = (int32_t)(((size_t)(M + 1) * sizeof(double) + 15) / 16 * 16);
  if (!(d->s_white > 0.0) && d->psd_w <= kMaxKeyW) {
    sort_off = flag_off;
    flag_off = sort_off + kStrainBlock / 64 * sort_slot(d->psd_w);
  }
  if ((size_t)flag_off + 16 > lds) lds = (size_t)flag_off + 16;
  const void* kern = nullptr;
  switch (logM) {
    case 3: kern = (const void*)strain_sft_kernel<3>; break;
    case 4: kern = (const void*)strain_sft_kernel<4>; break;
    case 5: kern = (const void*)strain_sft_kernel<5>; break;
    case 6: kern = (const void*)strain_sft_kernel<6>; break;
    case 7: kern = (const void*)strain_sft_kernel<7>; break;
    case 8: kern = (const void*)strain_sft_kernel<8>; break;
    case 9: kern = (const void*)strain_sft_kernel<9>; break;
    case 10: kern = (const void*)strain_sft_kernel<10>; break;
    case 11: kern = (const void*)strain_sft_kernel<11>; break;
    case 12: kern = (const void*)strain_sft_kernel<12>; break;
    case 13: kern = (const void*)strain_sft_kernel<13>; break;
    default: break;
  }
  if (e == hipSuccess && !kern) e = hipErrorInvalidValue;   // n in [16, 16384] was checked above
  if (e == hipSuccess && lds > 65536) e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess && n_seg > 0) {
    int32_t a_nseg = (int32_t)n_seg, a_w = d->psd_w, a_klo = d->k_lo, a_nbins = d->n_bins;
    int64_t a_ntot = d->n_total;
    double a_dt = d->dt, a_scale = psd_scale, a_white = d->s_white;
    void* args[] = {(void*)&x, &a_ntot, &a_nseg, &a_dt, &a_w, &a_scale, &a_klo, &a_nbins, &a_white,
                    &d_tw, &d_rtw, &bins, &psd, &keep, &sort_off, &flag_off};
    e = hipLaunchKernel(kern, dim3((unsigned)(n_seg * d->n_det)), dim3(kStrainBlock), args, lds, st);
  }
  if (e != hipSuccess) return strain_fail(SFT_E_DEVICE, hipGetErrorString(e));
  return SFT_OK;
}
