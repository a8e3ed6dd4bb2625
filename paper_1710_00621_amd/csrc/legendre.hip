// Legendre stage of the spherical harmonic transforms on gfx950.
//
// Synthesis (first half of Y, Sect. 2.1):
//     F^{c|s}_m(r) = c_m sum_{l=m..L} lambda_lm(z_r) u^{c|s}_lm
// Adjoint (second half of Y^T, Sect. 3.2):
//     v^{c|s}_lm   = c_m sum_r lambda_lm(z_r) H^{c|s}_m(r)
// with c_0 = 1, c_m = sqrt 2.  North/south ring pairs share the functions:
// lambda_lm(-z) = (-1)^(l+m) lambda_lm(z), so even and odd l - m (E, O) are
// summed separately and F_N = E + O, F_S = E - O.
//
// Recurrence.  With eps_l = sqrt((l^2 - m^2) / (4 l^2 - 1)) the functions obey
// z lambda_l = eps_{l+1} lambda_{l+1} + eps_l lambda_{l-1}.  The kernels run it
// two steps at a time on q_k = lambda_{m+2k+1} / z (a polynomial in z^2 times
// sin^m, so the division is exact at the equator too):
//     lambda_{m+2k+1} = z q_k,    lambda_{m+2k} = eps_{l+1} q_k + eps_l q_{k-1}  (l = m + 2k)
//     z^2 q_k = g_{k+1} q_{k+1} + (eps_{l+1}^2 + eps_l^2) q_k + g_k q_{k-1},
//               g_k = eps_l eps_{l-1}  (l = m + 2k + 1).
// One function per two l serves both parities, which halves the work, the LDS
// traffic and the matrix operands of generating lambda, and E and O become
// columns of one product.  Written for the difference d_k = g_k (q_k -+ q_{k-1}),
//     d_{k+1} = d_k + (y + b_k) q_k,    q_{k+1} = +-(q_k + d_{k+1} / g_{k+1}),
// it takes three FP64 operations per two l with two scalar coefficients:
// near the poles (upper signs) y = -sin^2 theta and b_k = 1 - eps_{l+1}^2 -
// eps_l^2 - g_k - g_{k+1}, near the equator (lower signs) y = -z^2 and b_k =
// eps_{l+1}^2 + eps_l^2 - g_k - g_{k+1}.  Both b_k and y vanish where the
// recurrence's characteristic roots meet, so nothing cancels in q and d.  What
// would add up over the steps is kept out: an error of y is the same in every
// step (a shifted ring), so y is the exact product of two doubles inside the
// FMA that adds b_k, and the tables form b_k without subtracting equal terms
// (grid.hip).
//
// Even functions next to the equator.  There neighbouring q have opposite signs
// and size |lambda / z|, so that eps_{l+1} q_k + eps_l q_{k-1} cancels by a factor
// of 1 / |z|.  The 32 ring pairs next to the equator therefore run in a third
// form: the same recurrence, and
//     lambda_{m+2k} = p_k / eps_{l+1},  p_k = d_k + h_k q_k,  h_k = eps_{l+1} (eps_{l+1} - eps_l)
// (l = m + 2k, d_k with the lower sign), whose terms do not cancel.  They sit
// twice in a tile of their own, whose first half hands on q (for O) and whose
// second half p (for E): the tile costs what any other does, and no wave holds
// more registers.  (Tried: q and p of 64 pairs one after the other in one wave,
// twice the LDS traffic and a longer chain: Nside 128 / L 256 x3, Legendre
// kernels, synthesis 24.8 us instead of 19.9, adjoint 27.8 instead of 20.3; the
// same inside the last belt group's wave, so that no further partial vector is
// written: its loads wait for its own stores, Nside 1024 / L 2000 adjoint 769 us
// instead of 565.)  Without the third form: 18.8, 19.2, 541.
//
// Relative rms error of F_m over all m, random coefficients, by |z| (each
// scheme emulated on the CPU against 80-bit arithmetic; the one-step recurrence
// in l / q alone / with the equator's form):
//                        Nside 256, L 512             Nside 1024, L 2000
//     0      .. 0.0025   7.6e-16 9.4e-15 5.9e-16     1.9e-15 3.0e-14 1.3e-15
//     0.01   .. 0.02     9.4e-16 2.5e-15 7.3e-16     1.8e-15 2.6e-15 1.3e-15
//     0.05   .. 0.1      8.8e-16 8.0e-16 6.4e-16     1.9e-15 1.4e-15 1.3e-15
//     0.3    .. 0.5      1.7e-15 1.2e-15 1.2e-15     3.6e-15 2.4e-15 2.4e-15
//     0.71   .. 0.8      3.6e-15 1.7e-15 1.7e-15     8.0e-15 4.6e-15 4.6e-15
//     0.97   .. 1        5.2e-14 1.1e-15 1.1e-15     3.4e-13 1.8e-15 1.8e-15
//
// Tiles of 64 ring pairs use one form each (grid.hip lays the pairs out in slots
// so that every tile lies well inside one form's range).
//
// Each (ring pair, m) starts at the last multiple of 8 in k at or before the
// first l where |lambda_lm| reaches 2^-100 (start table from grid.hip); before
// it a lane carries zeros, and lanes join at the start of a block of 8 steps.
#include <algorithm>
#include <climits>
#include <map>
#include <mutex>
#include <tuple>
#include <cstdio>
#include <cstdlib>

#include "internal.h"

namespace crs {

namespace {

enum Form { POLAR, BELT, EQUATOR };  // of the recurrence (a tile's)

// Tables and wave-uniform inputs are read through the constant address space
// so that they become scalar (SMEM) loads.
typedef __attribute__((address_space(4))) const double cdouble;
__device__ __forceinline__ cdouble* as_const(const double* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (cdouble*)(((uint64_t)hi << 32) | lo);
}

// minimum over the wave's active lanes (DPP reduction, no LDS round trips)
__device__ __forceinline__ int wave_min(int v) {
  return __builtin_amdgcn_readfirstlane(__ockl_wfred_min_i32(v));
}

// Lane exchanges of doubles.  dpp<CTRL, BANKS>: the DPP control applied to v
// in the banks (groups of four lanes of a row of 16) that BANKS selects, old
// elsewhere.
template <int CTRL, int BANKS>
__device__ __forceinline__ double dpp(double old, double v) {
  const uint64_t u = __double_as_longlong(v), o = __double_as_longlong(old);
  const unsigned lo = __builtin_amdgcn_update_dpp((unsigned)o, (unsigned)u, CTRL, 0xf, BANKS, false);
  const unsigned hi = __builtin_amdgcn_update_dpp((unsigned)(o >> 32), (unsigned)(u >> 32), CTRL, 0xf, BANKS, false);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
constexpr int kDppXor2 = 0x4e;     // quad_perm [2, 3, 0, 1]
constexpr int kDppRor4 = 0x124;    // row_ror: lane i of a row takes lane i - 4 (mod 16)
constexpr int kDppRor8 = 0x128;
constexpr int kDppRor12 = 0x12c;
// v of lane src (any lane of the wave)
__device__ __forceinline__ double lane_get(double v, int src) {
  const uint64_t u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_ds_bpermute(4 * src, (unsigned)u);
  const unsigned hi = __builtin_amdgcn_ds_bpermute(4 * src, (unsigned)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// v + v of lane t ^ 32 and v + v of lane t ^ 16 (gfx950 lane swaps)
__device__ __forceinline__ double add_xor32(double v) {
  const uint64_t u = __double_as_longlong(v);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
  const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  const double x = __longlong_as_double((long long)(((uint64_t)b[0] << 32) | a[0]));
  const double y = __longlong_as_double((long long)(((uint64_t)b[1] << 32) | a[1]));
  return x + y;
}

__device__ __forceinline__ int64_t moff(int L, int m) {
  return (m == 0) ? 0 : (int64_t)(L + 1) + 2 * ((int64_t)(m - 1) * (L + 1) - (int64_t)(m - 1) * m / 2);
}

// LDS traffic of one wave stays in order: only the compiler must not move
// accesses of the wave-private tile across this point.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// map slots of a launch (see LegArgs::mlist)
__device__ __forceinline__ int leg_nslots(const LegArgs& a, int nmaps) {
  return a.mcount ? __builtin_amdgcn_readfirstlane(*a.mcount) : nmaps;
}
__device__ __forceinline__ int leg_map(const LegArgs& a, int slot) { return a.mlist ? a.mlist[slot] : slot; }
// some slot of [s0, s0 + n) holds a map to process
__device__ __forceinline__ bool leg_any(const LegArgs& a, int s0, int n, int ns) {
  if (!a.skip.act) return s0 < ns;
  bool any = false;
  for (int k = 0; k < n && s0 + k < ns; ++k) any = any || !a.skip.off(leg_map(a, s0 + k));
  return any;
}
// Ring pairs p0 .. of a tile: pair p0 + i in slot i, valid below limit.  full:
// all 64 are valid and none is the equator ring, its own pair.  The last tile,
// the equator's, holds its (at most 32) pairs twice: p0 + i % 32 in slot i.
struct TilePairs {
  int p0, limit;
  bool full;
};
template <int F>
__device__ __forceinline__ TilePairs tile_pairs(const LegArgs& a, int tile) {
  TilePairs t;
  t.p0 = F == POLAR ? tile * 64 : F == BELT ? (tile - a.pol_tiles) * 64 + a.pol_pairs : a.npairs - a.eq_pairs;
  t.limit = F == POLAR ? a.pol_pairs : F == BELT ? a.npairs - a.eq_pairs : a.npairs;
  t.full = F != EQUATOR && t.p0 + 64 <= t.limit;
  return t;
}

// XCD-aware order: the 8 XCDs take blocks round-robin; consecutive blocks on
// one XCD share an m-block (same harmonic coefficients, one L2) and small m
// (the longest recurrences) are dispatched first.  Wave w of a block takes
// m = 4 mb + w.
__device__ __forceinline__ void block_coords(int ntiles, int& mb, int& tile) {
  const int b = blockIdx.x;
  const int xcd = b & 7, q = b >> 3;
  tile = q % ntiles;
  mb = (q / ntiles) * 8 + xcd;
}

// ----------------------------------------------------------- recurrence
// State of one lane's ring pair: (q, d) before step k, k a multiple of 8; y =
// -ya yc (yc = ya = z outside the polar form).
struct RecState {
  double ya, yc, q, d;
  int ks;     // the lane's start
  int nx;     // next start in the wave (uniform)
  int first;  // first start in the wave (uniform)
};
template <int F>
__device__ __forceinline__ void rec_init(RecState& r, const LegArgs& a, int m, int slot, bool in) {
  r.ya = in ? a.ya[slot] : 0.0;
  r.yc = F == POLAR && in ? a.yc[slot] : 0.0;
  r.ks = in ? a.ks[(size_t)m * a.nslots + slot] : INT_MAX;
  r.q = r.d = 0.0;
  r.nx = r.first = wave_min(r.ks);
}

// Coefficients of N steps from k0 (scalar registers), and h_k of eight
template <int N>
struct RecCoef {
  double b[N], g[N];
};
template <int N>
__device__ __forceinline__ RecCoef<N> rec_coef(cdouble* b, cdouble* gi, int k0) {
  RecCoef<N> c;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    c.b[i] = b[k0 + i];
    c.g[i] = gi[k0 + i];
  }
  return c;
}

struct RecH {
  double h[8];
};
__device__ __forceinline__ RecH rec_h(cdouble* he, int k0) {
  RecH c;
#pragma unroll
  for (int i = 0; i < 8; ++i) c.h[i] = he[k0 + i];
  return c;
}

// Eight steps of the signed q_k, k = k0 .. k0 + 7, with the coefficients from
// C.b[O] on, each pair (even, odd k) handed to put(i / 2, q_i, q_{i+1}), in the
// equator form with p_i, p_{i+1} (p_k = eps_{m+2k+1} lambda_{m+2k}) after them.
// Lanes whose start is k0 join first.
template <int F, int O, int N, class Put>
__device__ __forceinline__ void rec8(RecState& r, const RecCoef<N>& C, const RecH& H, const LegArgs& a, int m, int slot,
                                     int k0, Put&& put) {
  if (r.nx == k0) {
    if (r.ks == k0) {
      const double2 v = a.st[(size_t)m * a.nslots + slot];
      asm volatile("" ::"v"(v.x), "v"(v.y));  // waited for here, not where the paths meet (prefetches stay in flight)
      r.q = v.x;
      r.d = v.y;
    }
    r.nx = wave_min(r.ks > k0 ? r.ks : INT_MAX);
  }
  const double yc = F == POLAR ? r.yc : r.ya;
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const double t0 = fma(-r.ya, yc, C.b[O + i]), t1 = fma(-r.ya, yc, C.b[O + i + 1]);
    const double qe = r.q;
    const double pe = F == EQUATOR ? fma(H.h[i], qe, r.d) : 0.0;
    r.d = fma(t0, qe, r.d);
    if constexpr (F == POLAR) {
      const double qo = fma(C.g[O + i], r.d, qe);
      put(i / 2, qe, qo);
      r.d = fma(t1, qo, r.d);
      r.q = fma(C.g[O + i + 1], r.d, qo);
    } else {
      const double qo = fma(-C.g[O + i], r.d, -qe);  // the recurrence runs on -qo and -d there
      if constexpr (F == EQUATOR)
        put(i / 2, qe, qo, pe, fma(H.h[i + 1], qo, -r.d));
      else
        put(i / 2, qe, qo);
      r.d = fma(-t1, qo, r.d);
      r.q = fma(C.g[O + i + 1], r.d, -qo);
    }
  }
}
template <int F, int O, int N, class Put>
__device__ __forceinline__ void rec8(RecState& r, const RecCoef<N>& C, const LegArgs& a, int m, int slot, int k0,
                                     Put&& put) {
  static_assert(F != EQUATOR);
  rec8<F, O>(r, C, RecH{}, a, m, slot, k0, put);
}

// Tile groups: the polar tiles in groups of T, then the belt's, so that a wave
// runs one form (chosen once) and its tiles share the coefficients; the
// equator's tile is a group of its own.
struct TileRange {
  int t0, tend, form;
};
template <int T>
__device__ __forceinline__ TileRange tile_range(const LegArgs& a, int tg) {
  const int np = (a.pol_tiles + T - 1) / T, te = a.nslots / 64 - 1;
  if (tg < np) return {tg * T, a.pol_tiles, POLAR};
  const int t0 = a.pol_tiles + (tg - np) * T;
  return t0 < te ? TileRange{t0, te, BELT} : TileRange{te, te + 1, EQUATOR};
}

// Wave-private LDS tile of q: row k / 2 holds the pairs (q_k, q_{k+1}) of 64
// ring pairs as double2.  The row lengths (in double2) are the ones whose A
// operand reads are free of bank conflicts (measured, cycles per instruction:
// 16-byte reads 4.6 at 64 for the synthesis' rows of 16 lanes and at 68 for
// the adjoint's four rows at a time, 8 to 16 at other lengths; 8-byte reads of
// eight rows 4.1 at 65).  LDS writes run at 76 bytes per cycle in any shape,
// which with one map per wave is as tight a bound as the FP64 pipe.
constexpr int kQRowSyn = 64, kQRowAdj4 = 68, kQRowAdj16 = 65;

typedef double v4d __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------- synthesis
// F[pair][col] = sum_k q_k[pair] B[k][col] on the matrix cores: rows = ring
// pairs, K = k, columns = maps x (E, O) x (cos, sin) with B_E = eps_{l+1} u_l
// + eps_{l+2} u_{l+2} (l = m + 2k) and B_O = u_{l+1}, formed as they are loaded.
// C16 groups of four maps take v_mfma_f64_16x16x4 (16 columns), C4 single maps
// v_mfma_f64_4x4x4 (four blocks of four rows share one map's four columns):
// both run at the same FP64 rate (77 TFLOP/s measured) and read the same A
// operand (lane t: row t % 16, k t / 16), so any map count runs without empty
// columns.  Matrix and vector FP64 instructions share the issue pipe (measured:
// they add), which is why the recurrence's three operations per two l matter.
// One wave owns (m, T tiles of 64 ring pairs, 4 C16 + C4 maps); a block of 8
// steps goes through the wave's LDS tile into the A operands.
//
// The equator's tile (T = 1) has q of its ring pairs in rows 0 .. 31 and p of the
// same pairs in rows 32 .. 63, whose E columns take B = u_l / eps_{l+1}: O comes
// from the first rows and E from the others, at the cost of a tile of the belt.
template <int C16, int C4, int T, int F>
__device__ __forceinline__ void syn_wave(const LegArgs& a, int mw, int wave, int t0, int tend, int map0, int ns,
                                         const double* __restrict__ u, int64_t ustride,
                                         double2* __restrict__ phase, int64_t pstride, double2* qsh) {
  static_assert(F != EQUATOR || T == 1);
  constexpr int NG = C16 + C4, NMW = 4 * C16 + C4;
  constexpr int RB = F == EQUATOR ? 2 : 4;  // blocks of 16 rows with ring pairs of their own
  const int L = a.lmax;
  const bool mok = mw <= L;  // a block's last waves may lie past L: they only join its stores
  const int m = min(mw, L);
  double2* qt = qsh + wave * (4 * kQRowSyn);
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15, kq = lane >> 4;
  const int par = (lane >> 1) & 1, cs = lane & 1;
  const int n = L - m;  // largest l - m
  const int K = n / 2 + 1;
  // column g of this lane: map slot
  int cslot[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) cslot[g] = g < C16 ? map0 + 4 * g + ((lane >> 2) & 3) : map0 + 4 * C16 + (g - C16);
  RecState r[T];
  int kst = INT_MAX;
  cdouble* cb = as_const((F == POLAR ? a.bp : a.be) + krow(L, m));
  cdouble* cg = as_const(a.gi + krow(L, m));
  cdouble* ch = as_const(a.he + krow(L, m));
#pragma unroll
  for (int t = 0; t < T; ++t) {
    rec_init<F>(r[t], a, m, (t0 + t) * 64 + lane, t0 + t < tend && mok);
    kst = min(kst, r[t].first);
  }
  v4d D16[T][4][C16 > 0 ? C16 : 1];
  double D4[T][4][C4 > 0 ? C4 : 1];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
      for (int g = 0; g < C16; ++g) D16[t][rb][g] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < C4; ++c) D4[t][rb][c] = 0.0;
    }
  // This lane's k in a block are k0 + 2 kq and k0 + 2 kq + 1: l - m = x, x + 2
  // (and x + 4 for the second's eps_{l+2} term), x = 2 (k0 + 2 kq) + par.
  // Pointers run with k0: u of the lane's part, and (eps_{l+1}, eps_{l+2},
  // eps_{l+3}, eps_{l+4}) of E columns or the fixed (1, 0, 1, 0) of O columns.
  const int k1 = min(kst, K);
  const double* up[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g)
    up[g] = u + (int64_t)leg_map(a, min(cslot[g], ns - 1)) * ustride + moff(L, m) + (m > 0 && cs ? n + 1 : 0) +
            2 * (k1 + 2 * kq) + par;
  const double* ep = par ? a.ep : a.ep + 4 + erow(L, m) + 1 + 2 * (k1 + 2 * kq);
  const int64_t estep = par ? 0 : 16;
  const double* rp = a.re + krow(L, m) + k1 + 2 * kq;  // equator: 1 / eps_{l+1} of the two even l
  double un[NG][3], en[4], rn[2];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) en[i] = ep[i];
    ep += estep;
    if (F == EQUATOR) {
      rn[0] = rp[0];
      rn[1] = rp[1];
      rp += 8;
    }
    if (2 * (k0 + 7) + 3 <= n) {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 3; ++i) un[g][i] = up[g][2 * i];
    } else {
      const int x = 2 * (k0 + 2 * kq) + par;
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const double v = up[g][min(2 * i, n - x)];  // clamped to l = L
          un[g][i] = x + 2 * i <= n ? v : 0.0;
        }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) up[g] += 16;
  };
  RecCoef<8> C{};
  RecH H{};
  if (kst < K) {
    load(kst);
    C = rec_coef<8>(cb, cg, kst);
    if (F == EQUATOR) H = rec_h(ch, kst);
  }
  const bool two = C16 < 2 || map0 + 4 < ns;  // the second group of four has maps
  for (int k0 = kst; k0 < K; k0 += 8) {
    k0 = __builtin_amdgcn_readfirstlane(k0);
    double B0[NG], B1[NG], P0[NG], P1[NG];  // P: equator, rows of p
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (F == EQUATOR) {
        P0[g] = rn[0] * un[g][0];
        P1[g] = rn[1] * un[g][1];
        B0[g] = un[g][0];  // (of O columns)
        B1[g] = un[g][1];
      } else {
        B0[g] = fma(en[1], un[g][1], en[0] * un[g][0]);
        B1[g] = fma(en[3], un[g][2], en[2] * un[g][1]);
      }
    }
    load(k0 + 8);  // past K: in bounds, unused
    RecCoef<8> Cn;
    if (T > 1) Cn = rec_coef<8>(cb, cg, k0 + 8);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (T > 1 && r[t].first > k0) continue;
      if constexpr (F == EQUATOR)
        rec8<F, 0>(r[t], C, H, a, m, (t0 + t) * 64 + lane, k0, [&](int i, double qe, double qo, double pe, double po) {
          qt[i * kQRowSyn + lane] = lane < 32 ? make_double2(qe, qo) : make_double2(pe, po);
        });
      else
        rec8<F, 0>(r[t], C, a, m, (t0 + t) * 64 + lane, k0,
                   [&](int i, double qe, double qo) { qt[i * kQRowSyn + lane] = make_double2(qe, qo); });
      if (T == 1) C = rec_coef<8>(cb, cg, k0 + 8);  // the next block's, during the products
      if (F == EQUATOR) H = rec_h(ch, k0 + 8);
      wave_fence();
      double2 A[4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) A[rb] = qt[kq * kQRowSyn + 16 * rb + i16];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
        for (int g = 0; g < C16; ++g)
          if (g == 0 || two)
            D16[t][rb][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb].x, rb < RB ? B0[g] : P0[g], D16[t][rb][g], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < C4; ++c)
          D4[t][rb][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[rb].x, rb < RB ? B0[C16 + c] : P0[C16 + c], D4[t][rb][c], 0, 0, 0);
      }
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
#pragma unroll
        for (int g = 0; g < C16; ++g)
          if (g == 0 || two)
            D16[t][rb][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb].y, rb < RB ? B1[g] : P1[g], D16[t][rb][g], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < C4; ++c)
          D4[t][rb][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[rb].y, rb < RB ? B1[C16 + c] : P1[C16 + c], D4[t][rb][c], 0, 0, 0);
      }
      wave_fence();
    }
    if (T > 1) C = Cn;
  }
  // Lanes of E columns store the north ring, lanes of O columns the south one
  // (the column t ^ 2 holds the other parity of the same part): c_m (D + z O)
  // and c_m (E - z D).
  const double cm = m == 0 ? (cs ? 0.0 : 1.0) : 1.4142135623730951;
  const int64_t rstep = 2 * (int64_t)(L + 1);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (t0 + t >= tend) break;
    const TilePairs tp = tile_pairs<F>(a, t0 + t);
    if constexpr (F == EQUATOR) {  // E of rows 32 .. 63 beside O of the same pairs
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int g = 0; g < C16; ++g)
#pragma unroll
          for (int q = 0; q < 4; ++q) D16[t][rb][g][q] = par ? D16[t][rb][g][q] : D16[t][rb + 2][g][q];
#pragma unroll
        for (int c = 0; c < C4; ++c) D4[t][rb][c] = par ? D4[t][rb][c] : D4[t][rb + 2][c];
      }
    }
    const double* zt = a.zs + (t0 + t) * 64;
    if constexpr (C16 == 0) {
      // one to three maps: straight to the phase array
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        // D: block (t / 4) % 4, row t / 16 of it, column t % 4
        const int i = 16 * rb + 4 * ((lane >> 2) & 3) + kq;
        const double cz = cm * zt[i];
        const double wd = par ? -cz : cm, wo = par ? cm : cz;
        const int p = tp.p0 + i, ring = par ? a.nring - 1 - p : p;
        const bool ok = mok && (tp.full || (p < tp.limit && !(par && ring == p)));
#pragma unroll
        for (int c = 0; c < C4; ++c) {
          const double D = D4[t][rb][c], o = dpp<kDppXor2, 0xf>(0.0, D);
          double* ob = reinterpret_cast<double*>(phase + (int64_t)leg_map(a, min(cslot[c], ns - 1)) * pstride);
          if (ok && cslot[c] < ns) ob[(int64_t)ring * rstep + 2 * m + cs] = fma(wo, o, wd * D);
        }
      }
    } else {
      // Four or more maps write most of the phase array's bytes per unit of
      // work: the block's four m of a ring are put together in LDS and leave as
      // 64 contiguous bytes instead of four 16-byte pieces (Nside 256 / L 512,
      // 42 maps: see the figures at launch_leg_synth).
      double* xs = reinterpret_cast<double*>(qsh);  // [row 16][N, S][map][wave][cos, sin]
      static_assert(16 * 2 * NMW * 4 <= 4 * 4 * kQRowSyn, "a row block of every map fits the tiles' LDS");
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        __syncthreads();
        auto put = [&](int row, int ms, double D) {
          const double cz = cm * zt[16 * rb + row];
          const double o = dpp<kDppXor2, 0xf>(0.0, D);
          xs[(((row * 2 + par) * NMW + ms) * 4 + wave) * 2 + cs] = fma(par ? cm : cz, o, (par ? -cz : cm) * D);
        };
#pragma unroll
        for (int q = 0; q < 4; ++q)  // D: row kq + 4 q, column t % 16
#pragma unroll
          for (int g = 0; g < C16; ++g) put(kq + 4 * q, 4 * g + ((lane >> 2) & 3), D16[t][rb][g][q]);
#pragma unroll
        for (int c = 0; c < C4; ++c)  // D: block (t / 4) % 4, row t / 16 of it, column t % 4
          put(4 * ((lane >> 2) & 3) + kq, 4 * C16 + c, D4[t][rb][c]);
        __syncthreads();
        const int mo = mw - wave + (threadIdx.x & 3);
        for (int e = threadIdx.x >> 2; e < 32 * NMW; e += 64) {
          const int ms = e % NMW, side = (e / NMW) & 1, row = e / (2 * NMW);
          const int p = tp.p0 + 16 * rb + row, ring = side ? a.nring - 1 - p : p;
          if (mo > L || map0 + ms >= ns || p >= tp.limit || (side && ring == p)) continue;
          phase[(int64_t)leg_map(a, map0 + ms) * pstride + (int64_t)ring * (L + 1) + mo] =
              qsh[e * 4 + (threadIdx.x & 3)];
        }
      }
    }
  }
}

template <int C16, int C4, int T>
__global__ __launch_bounds__(256, C4 == 1 && T == 4 ? 4 : 1) void k_leg_syn(LegArgs a, int nmaps, const double* __restrict__ u,
                                                 int64_t ustride, double2* __restrict__ phase,
                                                 int64_t pstride, int ntg) {
  constexpr int NMW = 4 * C16 + C4;
  __shared__ double2 qsh[4 * 4 * kQRowSyn];
  int mb, tg;
  block_coords(ntg, mb, tg);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = mb * 4 + wave;
  if (mb * 4 > a.lmax) return;  // whole block
  const int map0 = blockIdx.y * NMW;
  const int ns = leg_nslots(a, nmaps);
  if (!leg_any(a, map0, NMW, ns)) return;
  const TileRange tr = tile_range<T>(a, tg);
  if (tr.form == POLAR)
    syn_wave<C16, C4, T, POLAR>(a, m, wave, tr.t0, tr.tend, map0, ns, u, ustride, phase, pstride, qsh);
  else if (tr.form == BELT)
    syn_wave<C16, C4, T, BELT>(a, m, wave, tr.t0, tr.tend, map0, ns, u, ustride, phase, pstride, qsh);
  else
    syn_wave<C16, C4, 1, EQUATOR>(a, m, wave, tr.t0, tr.tend, map0, ns, u, ustride, phase, pstride, qsh);
}

// --------------------------------------------------------------- adjoint
// W[k][col] = sum_p q_k[p] H[p][col] on the matrix cores (rows = k, K = ring
// pairs), with H_E = H_N + H_S and H_O = z (H_N - H_S) held in registers for
// the wave's T tiles of 64 ring pairs, then v_{m+2k} = eps_{l+1} W^E_k + eps_l
// W^E_{k-1} and v_{m+2k+1} = W^O_k: one partial v per T tiles (fixed order, no
// atomics).  In the equator's tile q and H_O sit in slots 0 .. 31, p and H_E in the
// others (zeros elsewhere), and v_{m+2k} = W^E_k / eps_{l+1}.  T sets the partial
// sums' traffic (one (L+1)^2 vector per map and T
// tiles, written here and read by the tile sum).

// Zero partial below the first evaluated k and the row pointers of a column.
struct AdjOut {
  double* vb;  // index l - m of the lane's part
  bool ok;
};
// the map's vector in group tg's partial
__device__ __forceinline__ double* adj_part(const AdjDst& d, int tg, int map) {
  if (tg == 0) return d.v0 + (int64_t)map * d.v0stride;
  return d.v + (int64_t)(tg - (d.g0 == 0 ? 1 : d.g0)) * d.tstride + (int64_t)map * d.vstride;
}
__device__ __forceinline__ AdjOut adj_out(const LegArgs& a, const AdjDst& dst, int tg, int m, int slot, int ns,
                                          int cs) {
  AdjOut o;
  const int L = a.lmax;
  o.ok = slot < ns && !(m == 0 && cs);
  const int mp = leg_map(a, min(slot, ns - 1));
  o.vb = adj_part(dst, tg, mp) + moff(L, m) + (cs && m > 0 ? L - m + 1 : 0);
  return o;
}
// H of N ring pairs i0 + 16 (j / IN) + j % IN of a tile in a lane's column (ph:
// the map's phase array at (ring 0, m, part); par: 0 E, 1 O; in: the tile exists)
template <int F, int N, int IN>
__device__ __forceinline__ void adj_h(const LegArgs& a, const double* ph, int tile, bool in, int i0, int par,
                                      double (&H)[N]) {
  const TilePairs tp = tile_pairs<F>(a, tile);
  const int64_t rstep = 2 * (int64_t)(a.lmax + 1);
  const double* z = a.zs + tile * 64 + i0;
  const double sg = par ? -1.0 : 1.0;
  if (in && tp.full) {
    const double* pn = ph + (int64_t)(tp.p0 + i0) * rstep;
    const double* ps = ph + (int64_t)(a.nring - 1 - tp.p0 - i0) * rstep;
    double hn[N], hs[N], zv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      hn[j] = *pn;
      hs[j] = *ps;
      zv[j] = z[16 * (j / IN) + j % IN];
      const int64_t step = (j % IN == IN - 1 ? 17 - IN : 1) * rstep;
      pn += step;
      ps -= step;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) H[j] = fma(sg, hs[j], hn[j]) * (par ? zv[j] : 1.0);
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int i = 16 * (j / IN) + j % IN;
      const int p = tp.p0 + (F == EQUATOR ? (i0 + i) & 31 : i0 + i), rs = a.nring - 1 - p;
      H[j] = 0.0;
      if (in && p < tp.limit && (F != EQUATOR || (i0 + i < 32) == (par != 0))) {
        const double hn = ph[(int64_t)p * rstep];
        const double hs = rs != p ? ph[(int64_t)rs * rstep] : 0.0;  // the equator ring is its own pair
        H[j] = fma(sg, hs, hn) * (par ? z[i] : 1.0);
      }
    }
  }
}

// One to three maps: v_mfma_f64_4x4x4 with its four blocks on different ring
// pairs, so a map's H takes 8 registers per tile.  Lane t =
// (j = t % 4: column (E cos, E sin, O cos, O sin), b = (t / 4) % 4, i = t / 16);
// operand k index t / 16: pair 16 s + b + 4 (t / 16) of H register s; A rows:
// k = k0 + 8 x + 2 (t % 4) + {0, 1}.  The blocks are summed once per 16 steps.
template <int NM, int T, int F>
__device__ __forceinline__ void adj4_wave(const LegArgs& a, int m, int tg, int t0, int tend, int map0, int ns,
                                          const double2* __restrict__ phase, int64_t pstride, const AdjDst& dst,
                                          double2* qt) {
  const int L = a.lmax;
  const int lane = threadIdx.x & 63;
  const int b = (lane >> 2) & 3, b0 = b & 1, b1 = b >> 1, hi = lane >> 4;
  const int par = (lane >> 1) & 1, cs = lane & 1;
  const int n = L - m, K = n / 2 + 1;
  RecState r[T];
  double H[T][NM][4];
  AdjOut out[NM];
  int kst = INT_MAX;
#pragma unroll
  for (int c = 0; c < NM; ++c) out[c] = adj_out(a, dst, tg, m, map0 + c, ns, cs);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int s0 = (t0 + t) * 64;
    const bool in = t0 + t < tend;
    rec_init<F>(r[t], a, m, s0 + lane, in);
    kst = min(kst, r[t].first);
#pragma unroll
    for (int c = 0; c < NM; ++c) {
      const double* ph =
          reinterpret_cast<const double*>(phase + (int64_t)leg_map(a, min(map0 + c, ns - 1)) * pstride) + 2 * m + cs;
      adj_h<F, 4, 1>(a, ph, t0 + t, in, b + 4 * hi, par, H[t][c]);
    }
  }
  // zero partial below the first evaluated k (all of it if no lane starts)
  const int zend = min(2 * min(kst, K), n + 1);
#pragma unroll
  for (int c = 0; c < NM; ++c)
    if (out[c].ok && par == 0)
      for (int x = lane >> 2; x < zend; x += 16) out[c].vb[x] = 0.0;
  cdouble* cb = as_const((F == POLAR ? a.bp : a.be) + krow(L, m));
  cdouble* cg = as_const(a.gi + krow(L, m));
  cdouble* ch = as_const(a.he + krow(L, m));
  const double* er = a.ep + 4 + erow(L, m);
  const double* rr = a.re + krow(L, m);
  const double cm = m == 0 ? 1.0 : 1.4142135623730951;
  const int kl = 8 * b1 + 2 * (lane >> 4) + b0;  // this lane's k - k0 after the block sums
  // lane of W_{k-1}: the lane of k - 1, whose carry for k = k0 is the last block's k0 + 15
  const int kp = (kl + 15) & 15;
  const int psrc = (lane & 3) + 4 * (2 * (kp >> 3) + (kp & 1)) + 16 * ((kp & 7) >> 1);
  double Wp[NM];
#pragma unroll
  for (int c = 0; c < NM; ++c) Wp[c] = 0.0;
  for (int k0 = kst; k0 < K; k0 += 16) {
    k0 = __builtin_amdgcn_readfirstlane(k0);
    const RecCoef<16> C = rec_coef<16>(cb, cg, k0);
    const double ea = par ? 1.0 : F == EQUATOR ? rr[k0 + kl] : er[2 * (k0 + kl) + 1];
    const double eb = par || F == EQUATOR ? 0.0 : er[2 * (k0 + kl)];
    double D[4][NM];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int c = 0; c < NM; ++c) D[x][c] = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (r[t].first >= k0 + 16) continue;
      const int slot = (t0 + t) * 64 + lane;
      auto put = [&](int i, double qe, double qo) { qt[i * kQRowAdj4 + lane] = make_double2(qe, qo); };
      if constexpr (F == EQUATOR) {
        rec8<F, 0>(r[t], C, rec_h(ch, k0), a, m, slot, k0, [&](int i, double qe, double qo, double pe, double po) {
          put(i, lane < 32 ? qe : pe, lane < 32 ? qo : po);
        });
        rec8<F, 8>(r[t], C, rec_h(ch, k0 + 8), a, m, slot, k0 + 8, [&](int i, double qe, double qo, double pe, double po) {
          put(4 + i, lane < 32 ? qe : pe, lane < 32 ? qo : po);
        });
      } else {
        rec8<F, 0>(r[t], C, a, m, slot, k0, put);
        rec8<F, 8>(r[t], C, a, m, slot, k0 + 8, [&](int i, double qe, double qo) { put(4 + i, qe, qo); });
      }
      wave_fence();
      double2 A[2][4];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int s = 0; s < 4; ++s) A[x][s] = qt[(4 * x + (lane & 3)) * kQRowAdj4 + 16 * s + b + 4 * hi];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int c = 0; c < NM; ++c) {
            D[2 * x][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[x][s].x, H[t][c][s], D[2 * x][c], 0, 0, 0);
            D[2 * x + 1][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[x][s].y, H[t][c][s], D[2 * x + 1][c], 0, 0, 0);
          }
      wave_fence();
    }
#pragma unroll
    for (int c = 0; c < NM; ++c) {
      // sum over the blocks, lane block b keeping D[b] (x = b1, odd k = b0)
      const double r0 = (b1 ? D[2][c] : D[0][c]) + dpp<kDppRor8, 0xf>(0.0, b1 ? D[0][c] : D[2][c]);
      const double r1 = (b1 ? D[3][c] : D[1][c]) + dpp<kDppRor8, 0xf>(0.0, b1 ? D[1][c] : D[3][c]);
      const double y = b0 ? r0 : r1;
      const double W = (b0 ? r1 : r0) + dpp<kDppRor12, 0x5>(dpp<kDppRor4, 0xa>(0.0, y), y);
      const double Wm = lane_get(kl == 15 ? Wp[c] : W, psrc);
      Wp[c] = W;
      const int x = 2 * (k0 + kl) + par;
      if (out[c].ok && x <= n) out[c].vb[x] = cm * fma(eb, Wm, ea * W);
    }
  }
}

template <int NM, int T>
__global__ __launch_bounds__(256) void k_leg_adj4(LegArgs a, int nmaps, int map0, const double2* __restrict__ phase,
                                                  int64_t pstride, AdjDst dst) {
  __shared__ double2 qsh[4][8 * kQRowAdj4];
  int mb, tg;
  block_coords(dst.ng, mb, tg);
  tg += dst.g0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = mb * 4 + wave;
  if (m > a.lmax) return;
  map0 += blockIdx.y * NM;
  const int ns = leg_nslots(a, nmaps);
  if (!leg_any(a, map0, NM, ns)) return;
  const TileRange tr = tile_range<T>(a, tg);
  if (tr.form == POLAR)
    adj4_wave<NM, T, POLAR>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
  else if (tr.form == BELT)
    adj4_wave<NM, T, BELT>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
  else
    adj4_wave<NM, 1, EQUATOR>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
}

// Groups of four maps: v_mfma_f64_16x16x4, column j = t % 16 = 4 map + 2 (E, O)
// + (cos, sin); H takes 32 registers per tile.  K-block 4 s + b holds the ring
// pairs that block b of k_leg_adj4 takes from H register s, and the four
// accumulators b are added as its blocks are: at one number of tiles per wave a
// map's sums do not depend on how many maps run beside it.
template <int T, int F>
__device__ __forceinline__ void adj16_wave(const LegArgs& a, int m, int tg, int t0, int tend, int map0, int ns,
                                           const double2* __restrict__ phase, int64_t pstride, const AdjDst& dst,
                                           double2* qt) {
  const int L = a.lmax;
  const double* qd = reinterpret_cast<const double*>(qt);
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15, kq = lane >> 4;
  const int par = (lane >> 1) & 1, cs = lane & 1;
  const int n = L - m, K = n / 2 + 1;
  const int slot = map0 + ((lane >> 2) & 3);
  const AdjOut out = adj_out(a, dst, tg, m, slot, ns, cs);
  RecState r[T];
  double H[T][16];
  int kst = INT_MAX;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int s0 = (t0 + t) * 64;
    const bool in = t0 + t < tend;
    rec_init<F>(r[t], a, m, s0 + lane, in);
    kst = min(kst, r[t].first);
    const double* ph =
        reinterpret_cast<const double*>(phase + (int64_t)leg_map(a, min(slot, ns - 1)) * pstride) + 2 * m + cs;
    adj_h<F, 16, 4>(a, ph, t0 + t, in, 4 * kq, par, H[t]);
  }
  const int zend = min(2 * min(kst, K), n + 1);
  if (out.ok && par == 0)
    for (int x = kq; x < zend; x += 4) out.vb[x] = 0.0;
  cdouble* cb = as_const((F == POLAR ? a.bp : a.be) + krow(L, m));
  cdouble* cg = as_const(a.gi + krow(L, m));
  cdouble* ch = as_const(a.he + krow(L, m));
  const double* er = a.ep + 4 + erow(L, m);
  const double* rr = a.re + krow(L, m);
  const double cm = m == 0 ? 1.0 : 1.4142135623730951;
  double Wp = 0.0;  // D[3] of the last block: its row 15 sits in lanes 48..63
  for (int k0 = kst; k0 < K; k0 += 16) {
    k0 = __builtin_amdgcn_readfirstlane(k0);
    const RecCoef<16> C = rec_coef<16>(cb, cg, k0);
    v4d D[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) D[b] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (r[t].first >= k0 + 16) continue;
      const int sl = (t0 + t) * 64 + lane;
      auto put = [&](int i, double qe, double qo) { qt[i * kQRowAdj16 + lane] = make_double2(qe, qo); };
      if constexpr (F == EQUATOR) {
        rec8<F, 0>(r[t], C, rec_h(ch, k0), a, m, sl, k0, [&](int i, double qe, double qo, double pe, double po) {
          put(i, lane < 32 ? qe : pe, lane < 32 ? qo : po);
        });
        rec8<F, 8>(r[t], C, rec_h(ch, k0 + 8), a, m, sl, k0 + 8, [&](int i, double qe, double qo, double pe, double po) {
          put(4 + i, lane < 32 ? qe : pe, lane < 32 ? qo : po);
        });
      } else {
        rec8<F, 0>(r[t], C, a, m, sl, k0, put);
        rec8<F, 8>(r[t], C, a, m, sl, k0 + 8, [&](int i, double qe, double qo) { put(4 + i, qe, qo); });
      }
      wave_fence();
      double A[16];
#pragma unroll
      for (int kb = 0; kb < 16; ++kb) A[kb] = qd[(i16 >> 1) * (2 * kQRowAdj16) + 2 * (16 * (kb >> 2) + (kb & 3) + 4 * kq) + (i16 & 1)];
#pragma unroll
      for (int kb = 0; kb < 16; ++kb)
        D[kb & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[kb], H[t][kb], D[kb & 3], 0, 0, 0);
      wave_fence();
    }
    // D: row (k - k0) = kq + 4 q, column t % 16
    const v4d W = (D[0] + D[2]) + (D[1] + D[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // W_{k-1}: the lane group below, or row 4 q - 1 from the last group
      const double prev = q == 0 ? Wp : W[q > 0 ? q - 1 : 0];
      const double Wm = lane_get(kq == 3 ? prev : W[q], (lane + 48) & 63);
      const int x = 2 * (k0 + kq + 4 * q);
      const double ea = par ? 1.0 : F == EQUATOR ? rr[k0 + kq + 4 * q] : er[x + 1];
      const double eb = par || F == EQUATOR ? 0.0 : er[x];
      if (out.ok && x + par <= n) out.vb[x + par] = cm * fma(eb, Wm, ea * W[q]);
    }
    Wp = W[3];
  }
}

template <int T>
__global__ __launch_bounds__(256, 2) void k_leg_adj16(LegArgs a, int nmaps, const double2* __restrict__ phase,
                                                      int64_t pstride, AdjDst dst) {
  __shared__ double2 qsh[4][8 * kQRowAdj16];
  int mb, tg;
  block_coords(dst.ng, mb, tg);
  tg += dst.g0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = mb * 4 + wave;
  if (m > a.lmax) return;
  const int map0 = blockIdx.y * 4;
  const int ns = leg_nslots(a, nmaps);
  if (!leg_any(a, map0, 4, ns)) return;
  const TileRange tr = tile_range<T>(a, tg);
  if (tr.form == POLAR)
    adj16_wave<T, POLAR>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
  else if (tr.form == BELT)
    adj16_wave<T, BELT>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
  else
    adj16_wave<1, EQUATOR>(a, m, tg, tr.t0, tr.tend, map0, ns, phase, pstride, dst, qsh[wave]);
}

// Squared functions (M_diag setup, Sect. 5): v_lm = sum_r lambda_lm^2 G_m(r) of
// one map, one wave per (m, 64 ring pairs).  Each four steps (eight l, 16
// outputs) are reduced over the lanes through a wave-private LDS block in a
// fixed order: four lanes sum 16 columns each, then two lane swaps finish.
constexpr int kRedRow = 65;
__device__ __forceinline__ double add_xor16(double v) {
  const uint64_t u = __double_as_longlong(v);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
  const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  const double x = __longlong_as_double((long long)(((uint64_t)b[0] << 32) | a[0]));
  const double y = __longlong_as_double((long long)(((uint64_t)b[1] << 32) | a[1]));
  return x + y;
}
__global__ __launch_bounds__(256) void k_leg_adj_sq(LegArgs a, const double2* __restrict__ phase,
                                                    AdjDst dst) {
  __shared__ double red[4][16 * kRedRow];
  int mb, tile;
  block_coords(dst.ng, mb, tile);
  tile += dst.g0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = mb * 4 + wave;
  const int L = a.lmax;
  if (m > L) return;
  double* wb = red[wave];
  const int lane = threadIdx.x & 63;
  const int n = L - m, K = n / 2 + 1, slot = tile * 64 + lane;
  RecState r;
  const bool polar = tile < a.pol_tiles;
  if (polar)
    rec_init<POLAR>(r, a, m, slot, true);
  else
    rec_init<EQUATOR>(r, a, m, slot, true);
  // north plus south (the equator's pairs once)
  const bool last = tile == a.nslots / 64 - 1;
  const TilePairs tp = polar ? tile_pairs<POLAR>(a, tile) : last ? tile_pairs<EQUATOR>(a, tile) : tile_pairs<BELT>(a, tile);
  double2 G = make_double2(0.0, 0.0);
  const int pair = tp.p0 + lane, south = a.nring - 1 - pair;
  if (pair < tp.limit && !(last && lane >= 32)) {
    G = phase[(int64_t)pair * (L + 1) + m];
    if (south != pair) {
      const double2 g = phase[(int64_t)south * (L + 1) + m];
      G.x += g.x;
      G.y += g.y;
    }
  }
  const double z = a.zs[slot];
  double* vb = adj_part(dst, tile, 0) + moff(L, m);
  const int np = m == 0 ? 1 : 2;
  const int zend = min(2 * min(r.first, K), n + 1);
  for (int x = lane; x < zend * np; x += 64) vb[x < zend ? x : n + 1 + x - zend] = 0.0;
  cdouble* cb = as_const((polar ? a.bp : a.be) + krow(L, m));
  cdouble* cg = as_const(a.gi + krow(L, m));
  cdouble* ch = as_const(a.he + krow(L, m));
  cdouble* er = as_const(a.ep + 4 + erow(L, m));
  cdouble* re = as_const(a.re + krow(L, m));
  double qm = 0.0;  // q_{k-1}
  for (int k0 = r.first; k0 < K; k0 += 8) {
    k0 = __builtin_amdgcn_readfirstlane(k0);
    const RecCoef<8> C = rec_coef<8>(cb, cg, k0);
    double q[8], le[8];  // le: lambda_{m+2k}
    if (polar) {
      rec8<POLAR, 0>(r, C, a, m, slot, k0, [&](int i, double qe, double qo) {
        q[2 * i] = qe;
        q[2 * i + 1] = qo;
      });
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        le[i] = fma(er[2 * (k0 + i)], qm, er[2 * (k0 + i) + 1] * q[i]);
        qm = q[i];
      }
    } else {
      rec8<EQUATOR, 0>(r, C, rec_h(ch, k0), a, m, slot, k0, [&](int i, double qe, double qo, double pe, double po) {
        q[2 * i] = qe;
        q[2 * i + 1] = qo;
        le[2 * i] = re[k0 + 2 * i] * pe;
        le[2 * i + 1] = re[k0 + 2 * i + 1] * po;
      });
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double lo = z * q[4 * h + i], ev = le[4 * h + i];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const double g = c ? G.y : G.x;
          wb[(4 * i + c) * kRedRow + lane] = ev * ev * g;
          wb[(4 * i + 2 + c) * kRedRow + lane] = lo * lo * g;
        }
      }
      wave_fence();
      const int o = lane & 15, sub = lane >> 4;
      double acc = wb[o * kRedRow + 16 * sub];
#pragma unroll
      for (int i = 1; i < 16; ++i) acc += wb[o * kRedRow + 16 * sub + i];
      acc = add_xor16(acc);
      acc = add_xor32(acc);
      wave_fence();
      const int x = 2 * (k0 + 4 * h) + (o >> 1), c = o & 1;
      if (sub == 0 && x <= n && c < np) vb[c * (n + 1) + x] = acc;
    }
  }
}

}  // namespace

// ------------------------------------------------------------ launchers
// tile groups of T (tile_range)
static int tile_groups(int pol_tiles, int nslots, int T) {
  return (pol_tiles + T - 1) / T + (nslots / 64 - 1 - pol_tiles + T - 1) / T + 1;
}

// Kernel choice: tiles of 64 ring pairs per wave.  More tiles share the operand
// loads of the synthesis and divide the adjoint's partial sums, fewer leave
// more waves in flight.  Measured (ms, T = 1 / 2 / 4; adjoint with its tile sum):
//                          synthesis               adjoint
//   Nside 256 / L 512 x1   0.031 / 0.036 / 0.053   0.034 / 0.034 / 0.046   ( 4104 waves at T = 1)
//   Nside 512 / L 1024 x1  0.131 / 0.096 / 0.107   0.141 / 0.112 / 0.110   (16400)
//   Nside 1024 / L 2000 x1 0.73  / 0.54  / 0.53    0.97  / 0.68  / 0.63    (64032)
//   Nside 1024 / L 2000 x4 1.15  / 1.18            3.14  / 2.13  / 1.80
//   Nside 512 / L 1024 x4  0.236 / 0.230           0.482 / 0.349 / 0.313
//   Nside 256 / L 512 x6                           0.104 / 0.090 / 0.099
//   Nside 256 / L 512 x15                          0.267 / 0.213 / 0.230
// so the rules take the largest T that leaves 8192 waves (synthesis; 16384 from
// three maps on, whose waves run longer) or 4096 (adjoint; 6144 for T = 4).
// The autotuner replaces them per shape.
static int largest_t(long tiles, int L, int tmax, long groups, long want2, long want4) {
  for (int T : {4, 2}) {
    if (T > tmax || T >= 2 * tiles) continue;
    if ((long)(L + 1) * ((tiles + T - 1) / T) * groups >= (T == 4 ? want4 : want2)) return T;
  }
  return 1;
}

// Largest T the synthesis is built for (the sums of T tiles sit in registers;
// from five maps on two tiles leave too few waves and gain nothing).
static int syn_tmax(int nmaps) { return nmaps == 1 ? 4 : nmaps <= 4 ? 2 : 1; }
constexpr int kAdjTmax = 4;

// waves of a launch with one tile and one group of maps per wave, as the rules and
// the figures below count them: tiles of 64 ring pairs, without the padding of
// the polar slots and without the equator's tile
static long leg_waves(int npairs, int L) { return (long)(L + 1) * ((npairs + 63) / 64); }

// Maps of the adjoint: n16 groups of four on the 16-column kernel, then groups of
// nm on the per-map kernel.  Four or three maps per wave cost the same per map
// where the waves fill the GPU (Nside 1024 / L 2000: 1515 and 1138 us), so that
// any count from six on splits exactly; few waves are a matter of latency,
// and there the maps spread over more, shorter ones.  Measured (us, the
// Legendre kernel alone up to Nside 128, else the whole transform; groups of
// 1 / 2 / 3 maps / of four, a remainder padded or on its own kernel):
//   Nside 16 / L 32 x6        8.5 /  10.0 /  11.4 /  11.9   (   33 waves per group)
//   Nside 64 / L 128 x12     20.6 /  18.1 /  20.3 /  22.8   (  258)
//   Nside 64 / L 128 x16     22.6 /  19.0 /  21.9 /  23.6
//   Nside 90 / L 180 x16     61.2 /  56.4 /  54.9 /  54.5   (  543, whole)
//   Nside 128 / L 256 x8     39.8 /  33.2 /  32.3 /  35.8   ( 1028)
//   Nside 128 / L 256 x20     112 /   104 /   104 /   106
//   Nside 150 / L 300 x10     111 /    98 /   103 /    97   ( 1505)
//   Nside 192 / L 384 x4       81 /    69 /    75 /    78   ( 2310)
//   Nside 192 / L 384 x7      116 /   110 /   113 /   104
//   Nside 256 / L 512 x5      140 /   134 /   125 /   141   ( 4104)
//   Nside 256 / L 512 x10     247 /   215 /   223 /   228
//   Nside 256 / L 512 x16     254 /   200 /   211 /   194   (kernel alone)
//   Nside 256 / L 512 x42     936 /   793 /   788 /   815
//   Nside 512 / L 1024 x6     775 /   674 /   619 /   660   (16400)
//   Nside 512 / L 1024 x10   1199 /  1063 /  1084 /  1005
//   Nside 1024 / L 2000 x6   4146 /  3571 /  3175 /  3316   (64032)
//   Nside 1024 / L 2000 x7   4811 /  4544 /  4336 /  3684
struct AdjGroups {
  int n16, nm;  // groups of four, then groups of nm maps (0: none)
};
static AdjGroups adj_groups(int npairs, int L, int nmaps) {
  const long w = leg_waves(npairs, L);
  if (nmaps == 1 || w * nmaps <= 4096) return {0, 1};
  if (nmaps == 2 || w * ((nmaps + 1) / 2) <= 5200) return {0, 2};
  if (nmaps % 3 == 0 || (nmaps == 5 && w < 32768)) return {0, 3};
  if (nmaps % 4 == 0 && w >= 2048) return {nmaps / 4, 0};
  if (w < 16384) return {0, 2};
  if (nmaps == 5) return {1, 1};
  return {nmaps / 4 - (3 - nmaps % 4), 3};  // nmaps = 4 n16 + 3 (4 - nmaps % 4)
}

// tiles per wave of the adjoint by the waves alone
static int adj_waves_t(int npairs, int L, int nmaps) {
  const AdjGroups g = adj_groups(npairs, L, nmaps);
  const int rest = nmaps - 4 * g.n16;
  return largest_t((npairs + 63) / 64, L, kAdjTmax, g.n16 + (g.nm ? (rest + g.nm - 1) / g.nm : 0), 4096, 6144);
}

static LegChoice default_choice(int npairs, int pol_tiles, int nslots, int L, int nmaps) {
  LegChoice c;
  const long tiles = (npairs + 63) / 64;
  c.syn_t = largest_t(tiles, L, syn_tmax(nmaps), 1, nmaps >= 3 ? 16384 : 8192, 8192);
  c.adj_t = adj_waves_t(npairs, L, nmaps);
  // A wave of four tiles with only one or two to run takes nearly as long as a
  // full one, and the equator's group stays one of few: four tiles only where they
  // halve the groups of two and leave three.  Adjoint, us, T = 2 / 4: Nside 256 / L
  // 512 x42 (4 + 4 tiles) 787 / 805, Nside 300 / L 600 x20 (4 + 5) 642 / 754, Nside
  // 320 / L 640 x30 (4 + 6) 1041 / 1264, Nside 384 / L 768 x20 (6 + 6) 1080 / 1083,
  // Nside 448 / L 900 x15 (7 + 7) 1220 / 1127, Nside 512 / L 1024 x6 (8 + 8) 661 / 619.
  if (c.adj_t == 4) {
    const int g4 = tile_groups(pol_tiles, nslots, 4) - 1, g2 = tile_groups(pol_tiles, nslots, 2) - 1;  // (the equator's apart)
    if (2 * g4 > g2 || g4 < 3) c.adj_t = 2;
  }
  return c;
}

static int env_int(const char* name) {
  const char* e = std::getenv(name);
  return e ? std::atoi(e) : 0;
}

static void apply_env(LegChoice& c, int nmaps) {
  auto pick = [](int v, int most) { return v >= 4 && most >= 4 ? 4 : v >= 2 && most >= 2 ? 2 : 1; };
  if (const int v = env_int("CRS_LEG_TS")) c.syn_t = pick(v, syn_tmax(nmaps));
  if (const int v = env_int("CRS_LEG_TA")) c.adj_t = pick(v, kAdjTmax);
}

static std::mutex g_tune_mu;
// (ring pairs, polar tiles, slots, L, maps): the same pairs may be laid out in other tiles
static std::map<std::tuple<int, int, int, int, int>, LegChoice> g_tuned;

LegChoice leg_choice(crs_grid g, int L, int nmaps) {
  const int npairs = (g->nring + 1) / 2;
  LegChoice c;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tuned.find(std::make_tuple(npairs, g->pol_tiles, g->nslots, L, nmaps));
    c = it != g_tuned.end() ? it->second : default_choice(npairs, g->pol_tiles, g->nslots, L, nmaps);
  }
  apply_env(c, nmaps);
  return c;
}

// blocks of a launch over ntg tile groups: four consecutive m each, m-blocks
// rounded up to the XCD order of block_coords
static unsigned leg_blocks(int L, int ntg) { return (unsigned)(((L + 1 + 3) / 4 + 7) / 8 * 8 * ntg); }

void launch_leg_synth(const LegChoice& c, const LegArgs& a, int nmaps, const double* u, int64_t ustride,
                      double2* phase, int64_t pstride, hipStream_t s) {
#define CRS_SYN(G16, G4, TT)                                                                          \
  do {                                                                                                \
    const int ntg = tile_groups(a.pol_tiles, a.nslots, TT), per = 4 * G16 + G4;                       \
    hipLaunchKernelGGL((k_leg_syn<G16, G4, TT>), dim3(leg_blocks(a.lmax, ntg), (nmaps + per - 1) / per), \
                       dim3(256), 0, s, a, nmaps, u, ustride, phase, pstride, ntg);                   \
  } while (0)
  // Large launches carry up to eight maps per wave: the recurrence is shared.
  // Few waves are a matter of latency: one map per wave while all of them are in
  // flight together, then four.  Measured (us, 1 / 4 / up to 8 maps per wave):
  //   Nside 16 / L 32 x6         7.3 /   9.2 /  11.7   (   33 waves per group)
  //   Nside 64 / L 128 x12      17.7 /  17.5 /  19.1   (  258)
  //   Nside 64 / L 128 x24      25.8 /  19.9 /  23.6
  //   Nside 90 / L 180 x16      34.8 /  21.8 /  27.3   (  543)
  //   Nside 128 / L 256 x3      20.3 /  20.1           ( 1028)
  //   Nside 128 / L 256 x8      36.0 /  24.4 /  29.4
  //   Nside 150 / L 300 x8      48.6 /  32.2 /  34.1   ( 1505)
  //   Nside 192 / L 384 x6      63.0 /  41.4 /  39.9   ( 2310)
  //   Nside 256 / L 512 x5       104 /  79.1 /  57.9   ( 4104)
  //   Nside 256 / L 512 x12      221 /   109 /   110
  //   Nside 512 / L 1024 x9     1007 /   573 /   607   (16400)
  //   Nside 512 / L 1024 x16    1798 /   776 /   739
  // Three maps on one tile run as four, one of them empty (without the equator's
  // tile: Nside 256 40 us instead of 52 for three columns, Nside 512 176 and 185).
  const long w = leg_waves(a.npairs, a.lmax);
  if (nmaps > 1 && c.syn_t == 1 && w * nmaps <= 4096) {
    CRS_SYN(0, 1, 1);
  } else if (nmaps > 4 && (w * ((nmaps + 3) / 4) <= 4608 || (nmaps > 8 && nmaps <= 12))) {
    CRS_SYN(1, 0, 1);
  } else {
    switch (nmaps) {
      case 1: if (c.syn_t == 4) CRS_SYN(0, 1, 4); else if (c.syn_t == 2) CRS_SYN(0, 1, 2); else CRS_SYN(0, 1, 1); break;
      case 2: if (c.syn_t == 2) CRS_SYN(0, 2, 2); else CRS_SYN(0, 2, 1); break;
      case 3: if (c.syn_t == 2) CRS_SYN(0, 3, 2); else CRS_SYN(1, 0, 1); break;
      case 4: if (c.syn_t == 2) CRS_SYN(1, 0, 2); else CRS_SYN(1, 0, 1); break;
      case 5: CRS_SYN(1, 1, 1); break;
      case 6: CRS_SYN(1, 2, 1); break;
      default: CRS_SYN(2, 0, 1); break;
    }
  }
#undef CRS_SYN
  CRS_HIP(hipGetLastError());
}

int leg_adjoint_tiles(const LegChoice& c, crs_grid g, bool square) {
  return tile_groups(g->pol_tiles, g->nslots, square ? 1 : c.adj_t);
}

int leg_adjoint_parts(const LegChoice& c, crs_grid g, int L, int nmaps) {
  const int npairs = (g->nring + 1) / 2;
  const int t = std::max(c.adj_t, adj_waves_t(npairs, L, nmaps));
  return std::min(tile_groups(g->pol_tiles, g->nslots, t) - 1, std::max(1, ((npairs + 63) / 64 + 1) / 2));
}

void launch_leg_adjoint(const LegChoice& c, const LegArgs& a, int nmaps, const double2* phase, int64_t pstride,
                        const AdjDst& dst, bool square, hipStream_t s) {
  const unsigned nb = leg_blocks(a.lmax, dst.ng);
  if (square) {
    CRS_CHECK(nmaps == 1, CRS_EINVAL, "the squared adjoint takes one map");
    hipLaunchKernelGGL(k_leg_adj_sq, dim3(nb), dim3(256), 0, s, a, phase, dst);
    CRS_HIP(hipGetLastError());
    return;
  }
  const AdjGroups g = adj_groups(a.npairs, a.lmax, nmaps);
  const int g16 = g.n16;
#define CRS_ADJ16(TT)                                                                                 \
  hipLaunchKernelGGL((k_leg_adj16<TT>), dim3(nb, g16), dim3(256), 0, s, a, nmaps, phase, pstride,     \
                     dst)
#define CRS_ADJ4(N, TT)                                                                               \
  hipLaunchKernelGGL((k_leg_adj4<N, TT>), dim3(nb, (nmaps - 4 * g16 + N - 1) / N), dim3(256), 0, s, a, \
                     nmaps, 4 * g16, phase, pstride, dst)
#define CRS_ADJ4T(N)                                                                                  \
  do {                                                                                                \
    if (c.adj_t == 4) CRS_ADJ4(N, 4);                                                                 \
    else if (c.adj_t == 2) CRS_ADJ4(N, 2);                                                            \
    else CRS_ADJ4(N, 1);                                                                              \
  } while (0)
  if (g16 > 0) {
    if (c.adj_t == 4) CRS_ADJ16(4);
    else if (c.adj_t == 2) CRS_ADJ16(2);
    else CRS_ADJ16(1);
  }
  if (g.nm == 1) CRS_ADJ4T(1);
  else if (g.nm == 2) CRS_ADJ4T(2);
  else if (g.nm == 3) CRS_ADJ4T(3);
#undef CRS_ADJ16
#undef CRS_ADJ4
#undef CRS_ADJ4T
  CRS_HIP(hipGetLastError());
}

// ------------------------------------------------------------ autotuner
// Average time of `reps` launches after one warm-up, with HIP events on s.
template <class F>
static float time_launches(F&& launch, int reps, hipStream_t s) {
  launch();
  hipEvent_t e0, e1;
  CRS_HIP(hipEventCreate(&e0));
  CRS_HIP(hipEventCreate(&e1));
  CRS_HIP(hipEventRecord(e0, s));
  for (int i = 0; i < reps; ++i) launch();
  CRS_HIP(hipEventRecord(e1, s));
  CRS_HIP(hipEventSynchronize(e1));
  float ms = 0.0f;
  CRS_HIP(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return ms / reps;
}

LegChoice leg_autotune(const LegArgs& a0, int nmaps, double* uhat, double2* phase, hipStream_t s) {
  LegArgs a = a0;
  a.skip = MapSkip{};
  const int L = a.lmax;
  const int64_t nalm = (int64_t)(L + 1) * (L + 1);
  const int64_t pst = (int64_t)a.nring * (L + 1);
  LegChoice best = default_choice(a.npairs, a.pol_tiles, a.nslots, L, nmaps);
  const int tiles = a.nslots / 64;
  // the largest partial-sum count of any candidate (one tile per wave; the first goes to uhat)
  DevBuf<double> vpart;
  vpart.alloc((size_t)(tiles - 1) * nmaps * nalm);
  CRS_HIP(hipMemsetAsync(uhat, 0, (size_t)nmaps * nalm * sizeof(double), s));
  CRS_HIP(hipMemsetAsync(phase, 0, (size_t)nmaps * pst * sizeof(double2), s));
  const int reps = 3;
  float tbest = 1e30f;
  for (int t : {1, 2, 4}) {
    if (t > syn_tmax(nmaps) || t >= 2 * tiles) continue;
    LegChoice c = best;
    c.syn_t = t;
    const float ms = time_launches([&] { launch_leg_synth(c, a, nmaps, uhat, nalm, phase, pst, s); }, reps, s);
    if (ms < tbest) {
      tbest = ms;
      best.syn_t = t;
    }
  }
  // the adjoint's candidates are timed with the sum over their partials
  tbest = 1e30f;
  for (int t : {1, 2, 4}) {
    if (t > kAdjTmax || t >= 2 * tiles) continue;
    LegChoice c = best;
    c.adj_t = t;
    const int nt = tile_groups(a.pol_tiles, a.nslots, t);
    const float ms = time_launches([&] {
      launch_leg_adjoint(c, a, nmaps, phase, pst, AdjDst{uhat, nalm, vpart.p, nalm, (int64_t)nmaps * nalm, 0, nt}, false,
                         s);
      launch_tile_sum(nalm, nmaps, vpart.p, nalm, nt - 1, (int64_t)nmaps * nalm, uhat, nalm, s);
    }, reps, s);
    if (ms < tbest) {
      tbest = ms;
      best.adj_t = t;
    }
  }
  CRS_HIP(hipStreamSynchronize(s));
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned[std::make_tuple(a.npairs, a.pol_tiles, a.nslots, L, nmaps)] = best;
  }
  // the environment overrides apply to a tuned choice as to the default one
  apply_env(best, nmaps);
  return best;
}

namespace {
__global__ void k_tile_sum(int64_t nalm, const double* __restrict__ in, int64_t istride, int ntiles, int64_t tstride,
                           double* __restrict__ out, int64_t ostride) {
  const int map = blockIdx.y;
  const double* __restrict__ src = in + (int64_t)map * istride;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nalm; i += (int64_t)gridDim.x * blockDim.x) {
    double acc = out[(int64_t)map * ostride + i];
    for (int t = 0; t < ntiles; ++t) acc += src[(int64_t)t * tstride + i];
    out[(int64_t)map * ostride + i] = acc;
  }
}
}  // namespace

void launch_tile_sum(int64_t nalm, int nmaps, const double* in, int64_t istride, int ntiles, int64_t tstride,
                     double* out, int64_t ostride, hipStream_t s) {
  if (ntiles < 1) return;
  const int64_t nb = std::min<int64_t>((nalm + 255) / 256, 4096);
  hipLaunchKernelGGL(k_tile_sum, dim3((unsigned)nb, nmaps), dim3(256), 0, s, nalm, in, istride, ntiles, tstride,
                     out, ostride);
  CRS_HIP(hipGetLastError());
}

}  // namespace crs
