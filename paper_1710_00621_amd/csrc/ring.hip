// Ring stage of the spherical harmonic transforms: per-ring FFTs in LDS.
//
// Synthesis, second half of Y (Sect. 2.1): on ring r with Nphi pixels at
// phi_j = phi0 + 2 pi j / Nphi,
//     f_j = Re sum_{m=0..L} (F^c_m - i F^s_m) e^{i m phi_j}.
// The m sum is folded onto Nphi bins (m -> m mod Nphi, conjugate partner
// -m) so that f = inverse DFT of a Hermitian spectrum c; rings with
// Nphi < 2L+1 alias exactly as the dense operator does.
// Adjoint, first half of Y^T (Sect. 3.2): H_m = e^{-i m phi0} F^_{m mod Nphi},
// F^_k = sum_j f_j e^{-2 pi i j k / Nphi}, H^c = Re H, H^s = -Im H.
// Round trip (inside A and T^+): synthesis, multiply by a pixel weight
// (tau for A, alpha^2 w^2 tau^+ for T^+; Sect. 2.3 and Sect. 3.3), adjoint --
// the map never leaves LDS.
// Diagonal setup (M_diag, Sect. 5): for a pixel map t, G^c_m = T^_0 +
// Re(e^{-2 i m phi0} T^_{2m}), G^s_m = T^_0 - Re(...), G_0 = (T^_0, 0):
// sum_j t_j cos^2(m phi_j) = (G^c_m)/2 etc.
//
// Transform layout.  The ring data are real, so an even ring (Nphi = 2H, all
// HEALPix rings) runs a complex FFT of length H on z_n = f_{2n} + i f_{2n+1}:
//   synthesis  Z_k = (c_k + c_{k+H}) + i e^{2 pi i k / Nphi} (c_k - c_{k+H}),
//              z = inverse DFT_H(Z);
//   adjoint    Z = DFT_H(z), E_k = (Z_k + conj Z_{H-k}) / 2,
//              O_k = (Z_k - conj Z_{H-k}) / (2i), F^_k = E_k + e^{-2 pi i k / Nphi} O_k.
// Odd rings run a full complex FFT of length Nphi.  The FFT is a mixed-radix
// Stockham autosort in LDS (radix 8, 4, 2, 3, 5, 7 and primes up to a limit that
// grows with the length, see prime_max in grid.hip); a length with a larger
// prime factor is computed by Bluestein's chirp-z identity
// n k = (n^2 + k^2 - (k - n)^2) / 2 as a cyclic convolution of power-of-two
// length M >= 2n - 1 (filter spectrum precomputed per length on the host).
// One block per (ring, map), eight points per thread; rings are launched in
// classes by FFT length (<= 512 << t: 64 << t threads) and, from t = 2, by
// Bluestein or direct transform and whether the FFT has odd radices.
//
// What bounds it.  A block is a chain of dependent steps (ring record, phases,
// the FFT's exchanges through LDS, the store), so time goes with the length of
// the chain and with the LDS traffic of the FFT long before memory is busy:
//   - everything a block knows about its ring is one 128-byte record, and global
//     loads are issued in batches (loops that waited for each load, two levels
//     of tables and radices read per stage were 80 % of a wave's life);
//   - power-of-two lengths have their indices compiled in, a padded layout
//     (half of all LDS cycles were bank conflicts), and the map load, the
//     Bluestein products, the round trip's weights and the map store happen in
//     registers in the FFT's first and last stages: a Bluestein transform of S
//     stages per FFT exchanges 2 S - 2 times through LDS instead of 2 S + 3;
//   - two thirds of a HEALPix grid's cap rings have a prime factor above 7:
//     the direct sums of stage_prime take a fraction of Bluestein's 2 FFTs of 2
//     to 4 times the length.
// Measured, synthesis / adjoint, ms: Nside 256, 42 maps 0.338 / 0.315 -> 0.218 /
// 0.205 (617 MB: 2.8 / 3.0 TB/s of the 5.0 a copy reaches); Nside
// 1024, 6 maps 0.865 / 0.798 -> 0.530 / 0.465; Nside 1024, 1 map 0.171 / 0.163 ->
// 0.147 / 0.147; Nside 2048, 1 map 0.848 / 0.718 -> 0.53 / 0.50; 512 x 1026 GL, 40
// maps 0.479 / 0.498 -> 0.150 / 0.172.
#include <type_traits>

#include "internal.h"

namespace crs {

namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {  // a * conj(b)
  return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// Exact quotient n / d for n * d < 2^32 (multiply-high by ceil(2^32 / d)).
struct FastDiv {
  unsigned d, m;
  __device__ __forceinline__ explicit FastDiv(unsigned dd)
      : d(dd), m(dd <= 1 ? 0u : 0xFFFFFFFFu / dd + 1u) {}  // 32-bit quotient: same value
  // with the multiplier precomputed on the host
  __device__ __forceinline__ FastDiv(unsigned dd, unsigned mm) : d(dd), m(mm) {}
  __device__ __forceinline__ unsigned div(unsigned n) const { return d <= 1 ? n : __umulhi(n, m); }
  __device__ __forceinline__ unsigned mod(unsigned n) const { return n - div(n) * d; }
};

// Twiddles exp(-2 pi i u / n) of an FFT of length n from two LDS tables:
// Wf[u & 63] Wc[u >> 6] (exact table entries; the product adds one rounding).
struct TwCtx {
  const double2* Wf;
  const double2* Wc;
  __device__ __forceinline__ double2 tw(int u) const { return cmul(Wc[u >> 6], Wf[u & 63]); }
};

// cos(2 pi k / R) and sin(2 pi k / R), 1 <= k <= (R-1)/2, for the odd radices
// (values correctly rounded from their closed forms).
__device__ __forceinline__ constexpr double dft_cos(int R, int k) {
  return R == 3 ? -0.5
       : R == 5 ? (k == 1 ? 0.3090169943749474241022934 : -0.8090169943749474241022934)
       : (k == 1 ? 0.6234898018587335305250049
                 : k == 2 ? -0.2225209339563144042889026 : -0.9009688679024191262361023);
}
__device__ __forceinline__ constexpr double dft_sin(int R, int k) {
  return R == 3 ? 0.8660254037844386467637232
       : R == 5 ? (k == 1 ? 0.9510565162951535721164393 : 0.5877852522924731291687060)
       : (k == 1 ? 0.7818314824680298087084445
                 : k == 2 ? 0.9749279121818236070181317 : 0.4338837391175581204757683);
}

// forward DFT of R points; the inverse of a ring is taken as conj(DFT(conj .)),
// the conjugations folded into the steps before and after
template <int R>
__device__ __forceinline__ void small_dft(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 8) {
    // X_k = E_k + w^k O_k, X_{k+4} = E_k - w^k O_k (E, O: 4-point DFTs of the
    // even and odd samples; w = exp(-i pi / 4))
    double2 e[4] = {v[0], v[2], v[4], v[6]};
    double2 o[4] = {v[1], v[3], v[5], v[7]};
    small_dft<4>(e);
    small_dft<4>(o);
    constexpr double h = 0.7071067811865475244008444;  // 1 / sqrt(2)
    double2 t[4];
    t[0] = o[0];
    t[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
    t[2] = make_double2(o[2].y, -o[2].x);
    t[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cadd(e[k], t[k]);
      v[k + 4] = csub(e[k], t[k]);
    }
  } else if constexpr (R == 4) {
    const double2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const double2 t2 = cadd(v[1], v[3]), t3 = csub(v[1], v[3]);
    const double2 mit3 = make_double2(t3.y, -t3.x);  // -i t3
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, mit3);
    v[3] = csub(t1, mit3);
  } else {
    // odd R: with a_s = x_s + x_{R-s}, b_s = x_s - x_{R-s},
    //   y_r = x_0 + sum_s a_s cos(2 pi r s / R) - i sum_s b_s sin(2 pi r s / R),
    //   y_{R-r} the same with the sine term's sign flipped.
    constexpr int H = (R - 1) / 2;
    double2 a[H], b[H];
    double2 y0 = v[0];
#pragma unroll
    for (int s = 1; s <= H; ++s) {
      a[s - 1] = cadd(v[s], v[R - s]);
      b[s - 1] = csub(v[s], v[R - s]);
      y0 = cadd(y0, a[s - 1]);
    }
    double2 out[R];
    out[0] = y0;
#pragma unroll
    for (int r = 1; r <= H; ++r) {
      double2 A = v[0], B = make_double2(0.0, 0.0);
#pragma unroll
      for (int s = 1; s <= H; ++s) {
        const int k = (r * s) % R;
        const double c = dft_cos(R, k <= H ? k : R - k);
        const double sn = k <= H ? dft_sin(R, k) : -dft_sin(R, R - k);
        A.x = fma(a[s - 1].x, c, A.x);
        A.y = fma(a[s - 1].y, c, A.y);
        B.x = fma(b[s - 1].x, sn, B.x);
        B.y = fma(b[s - 1].y, sn, B.y);
      }
      const double2 miB = make_double2(B.y, -B.x);  // -i B
      out[r] = cadd(A, miB);
      out[R - r] = csub(A, miB);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = out[r];
  }
}

// Global loads of a thread that are issued together: a loop that waits for each
// of its loads pays the memory latency once per iteration (that was most of a
// block's life: 80 % of its waves' cycles).
constexpr int kBatch = 4;

// v[r] *= w^r: powers as products of shorter ones (a chain of log2 R products)
template <int R>
__device__ __forceinline__ void twiddle(double2 (&v)[R], double2 w1) {
  double2 w[R];
  w[1] = w1;
#pragma unroll
  for (int r = 2; r < R; ++r) w[r] = cmul(w[(r + 1) / 2], w[r / 2]);
#pragma unroll
  for (int r = 1; r < R; ++r) v[r] = cmul(v[r], w[r]);
}

// One radix-R Stockham stage on x[0..n): butterfly j (k = j mod Ns) reads
// x[j + r n/R], twiddles by omega_n^{r k span} (span = n / (Ns R)), and writes x[(j / Ns) Ns R
// + k + r Ns].  Every thread keeps its butterflies in registers across the
// barrier, so the stage works in place.
template <int R, int NT, int MAXN>
__device__ __forceinline__ void stage(double2* x, int n, int Ns, unsigned nsm, const TwCtx& C) {
  constexpr int MAXIT = (MAXN / R + NT - 1) / NT;
  const int nb = (int)((unsigned)n / (unsigned)R);
  const FastDiv dv((unsigned)Ns, nsm);
  const int span = (int)dv.div((unsigned)nb);  // nb Ns <= n: exact
  const int tid = threadIdx.x;
  double2 v[MAXIT][R];
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int j = tid + NT * it;
    if (j < nb) {
      const int k = (int)dv.mod((unsigned)j);
#pragma unroll
      for (int r = 0; r < R; ++r) v[it][r] = x[j + r * nb];
      if (k != 0) twiddle<R>(v[it], C.tw(k * span));
      small_dft<R>(v[it]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < MAXIT; ++it) {
    const int j = tid + NT * it;
    if (j < nb) {
      const int q = (int)dv.div((unsigned)j);
      const int idx = q * Ns * R + (j - q * Ns);
#pragma unroll
      for (int r = 0; r < R; ++r) x[idx + r * Ns] = v[it][r];
    }
  }
  __syncthreads();
}

// The same for a prime radix p >= 11 (not known at compile time), by the sums
// that the odd radices of small_dft use: a thread computes up to kPairs output
// pairs (r, p - r) of one butterfly, so a point is read p / (2 kPairs) times and
// costs p - 1 FMAs.  cs: exp(-2 pi i t / p), t < p, in LDS.  A block of n / 8
// threads has at least one thread per work item: (n / p) ceil((p - 1) / 12) <=
// 2 n / 17.
constexpr int kPairs = 6;
template <int NT>
__device__ __forceinline__ void stage_prime(double2* x, int n, int p, int Ns, unsigned nsm, const double2* cs, const TwCtx& C) {
  const int nb = (int)((unsigned)n / (unsigned)p), H = (p - 1) / 2;
  const FastDiv dv((unsigned)Ns, nsm), dnb((unsigned)nb);
  const int tid = threadIdx.x;
  if (Ns > 1) {
    const int span = (int)dv.div((unsigned)nb);
    for (int i = nb + tid; i < n; i += NT) {
      const int r = (int)dnb.div((unsigned)i), k = (int)dv.mod((unsigned)(i - r * nb));
      x[i] = cmul(x[i], C.tw(r * k * span));
    }
    __syncthreads();
  }
  const int g = (int)dnb.div((unsigned)tid), j = tid - g * nb, r0 = g * kPairs + 1;
  const bool on = r0 <= H;
  double2 A[kPairs], B[kPairs], y0 = make_double2(0.0, 0.0);
  if (on) {
    int rq[kPairs], kq[kPairs];
    const double2 x0 = x[j];
    y0 = x0;
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      A[q] = x0;
      B[q] = make_double2(0.0, 0.0);
      rq[q] = kq[q] = min(r0 + q, H);
    }
    for (int t = 1; t <= H; ++t) {
      const double2 u = x[j + t * nb], v = x[j + (p - t) * nb];
      const double2 a = cadd(u, v), b = csub(u, v);
      y0 = cadd(y0, a);
#pragma unroll
      for (int q = 0; q < kPairs; ++q) {
        const double2 c = cs[kq[q]];
        kq[q] += rq[q];
        if (kq[q] >= p) kq[q] -= p;
        A[q].x = fma(a.x, c.x, A[q].x);
        A[q].y = fma(a.y, c.x, A[q].y);
        B[q].x = fma(-b.y, c.y, B[q].x);  // i b c.y
        B[q].y = fma(b.x, c.y, B[q].y);
      }
    }
  }
  __syncthreads();
  if (on) {
    const int q1 = (int)dv.div((unsigned)j);
    double2* o = x + (q1 * Ns * p + (j - q1 * Ns));
    if (g == 0) o[0] = y0;
#pragma unroll
    for (int q = 0; q < kPairs; ++q) {
      const int r = r0 + q;
      if (r <= H) {
        o[r * Ns] = cadd(A[q], B[q]);
        o[(p - r) * Ns] = csub(A[q], B[q]);
      }
    }
  }
  __syncthreads();
}

// In-place forward DFT of x[0..n) in LDS, any length.
// POW2: the length is a power of two (radix 8, 4 and 2 only).
template <int NT, int MAXN, bool POW2>
__device__ __forceinline__ void fft_lds(double2* x, int n, const RingInfo* __restrict__ ri, const TwCtx& C, const double2* cs) {
  int Ns = 1;
  for (int st = 0; st < ri->nfac; ++st) {
    const int R = ri->fac[st];
    const unsigned m = ri->facm[st];
    if (R == 8) {
      stage<8, NT, MAXN>(x, n, Ns, m, C);
    } else if (R == 4) {
      stage<4, NT, MAXN>(x, n, Ns, m, C);
    } else if (R == 2) {
      stage<2, NT, MAXN>(x, n, Ns, m, C);
    } else if constexpr (!POW2) {
      if (R == 3) stage<3, NT, MAXN>(x, n, Ns, m, C);
      else if (R == 5) stage<5, NT, MAXN>(x, n, Ns, m, C);
      else if (R == 7) stage<7, NT, MAXN>(x, n, Ns, m, C);
      else if (R > 7) {
        stage_prime<NT>(x, n, R, Ns, m, cs, C);
        cs += R;
      }
    }
    Ns *= R;
  }
}

// Power-of-two lengths M with everything fixed at compile time (conv below), for
// the tier's longest length and its half and quarter: every long FFT of the
// class and, in a launch that merges classes, the next shorter ones (Nside 64,
// 20 maps: 20 us with the quarter, 21 without).
// The data sit in LDS with one word of padding after every 16 (the first
// stages write with a stride of their radix, which without it puts 8 lanes on
// one bank).  pad(i + c) = pad(i) + pad(c) where the low four bits do not carry,
// which holds for every offset below.
__device__ __forceinline__ constexpr int pad(int i) { return i + (i >> 4); }

template <int R, int NT, int M, class F>
__device__ __forceinline__ void each_butterfly(int tid, F&& f) {
  constexpr int NB = M / R, IT = (NB + NT - 1) / NT;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int j = tid + NT * it;
    if (NB % NT == 0 || j < NB) f(it, j);
  }
}
template <int R, int NT, int M>
struct Bfly {
  static constexpr int NB = M / R, IT = (NB + NT - 1) / NT;
  double2 v[IT][R];
};
template <int R, int NT, int M>
__device__ __forceinline__ void rd(int tid, const double2* x, Bfly<R, NT, M>& b) {
  static_assert(M / R % 16 == 0, "offsets of whole padded rows");
  each_butterfly<R, NT, M>(tid, [&](int it, int j) {
#pragma unroll
    for (int r = 0; r < R; ++r) b.v[it][r] = x[pad(j) + r * pad(M / R)];
  });
}
template <int R, int NT, int M, int NS>
__device__ __forceinline__ void dft(int tid, Bfly<R, NT, M>& b, const TwCtx& C) {
  each_butterfly<R, NT, M>(tid, [&](int it, int j) {
    const int k = j & (NS - 1);
    if (NS > 1) twiddle<R>(b.v[it], C.tw(k * (M / (NS * R))));
    small_dft<R>(b.v[it]);
  });
}
template <int R, int NT, int M, int NS>
__device__ __forceinline__ void wr(int tid, double2* x, const Bfly<R, NT, M>& b) {
  each_butterfly<R, NT, M>(tid, [&](int it, int j) {
    const int k = j & (NS - 1);
    double2* o = x + pad((j - k) * R + k);
#pragma unroll
    for (int r = 0; r < R; ++r) o[pad(r * NS)] = b.v[it][r];
  });
}

// Transform of M points: ld(v, j, NB) fills v[r] with point j + r NB, st(v, j, NB)
// takes the results at the same indices.  With `two` a second transform follows:
// the last stage of the first leaves a thread with the points that the first
// stage of the second needs (equal radices), so that mid(v, j, NB) changes them
// in registers and nothing of it passes through LDS.  A transform of S stages
// takes S - 1 exchanges through LDS, two of them 2 S - 2.
// The caller has a barrier before ld (if that reads LDS) and after st (if that
// writes it).
struct NoMid {};
template <int NT, int M, int S, int NS, class Mid, class St>
__device__ __forceinline__ void conv_rest(int tid, double2* x, const TwCtx& C, bool two, Mid&& mid, St&& st) {
  constexpr int R = pow2_radix(ilog2(M), S);
  constexpr bool last = NS * R == M;
  Bfly<R, NT, M> b;
  rd<R, NT, M>(tid, x, b);
  dft<R, NT, M, NS>(tid, b, C);
  __syncthreads();
  if constexpr (!last) {
    wr<R, NT, M, NS>(tid, x, b);
    __syncthreads();
    conv_rest<NT, M, S + 1, NS * R>(tid, x, C, two, mid, st);
  } else {
    if constexpr (!std::is_same_v<std::decay_t<Mid>, NoMid>) {
      if (two) {
        asm volatile("" : "+v"(tid));  // as in transforms()
        each_butterfly<R, NT, M>(tid, [&](int it, int j) { mid(b.v[it], j, M / R); });
        dft<R, NT, M, 1>(tid, b, C);
        wr<R, NT, M, 1>(tid, x, b);
        __syncthreads();
        conv_rest<NT, M, 1, R>(tid, x, C, false, NoMid{}, st);
        return;
      }
    }
    each_butterfly<R, NT, M>(tid, [&](int it, int j) { st(b.v[it], j, M / R); });
  }
}
template <int NT, int M, class Ld, class Mid, class St>
__device__ __forceinline__ void conv(int tid, double2* x, const TwCtx& C, bool two, Ld&& ld, Mid&& mid, St&& st) {
  constexpr int R = pow2_radix(ilog2(M), 0);
  Bfly<R, NT, M> b;
  each_butterfly<R, NT, M>(tid, [&](int it, int j) { ld(b.v[it], j, M / R); });
  dft<R, NT, M, 1>(tid, b, C);
  __syncthreads();
  wr<R, NT, M, 1>(tid, x, b);
  __syncthreads();
  conv_rest<NT, M, 1, R>(tid, x, C, two, mid, st);
}

// Bluestein's identity for a DFT of length n0:
//   X_k = w_k sum_n (x_n w_n) b_{k-n},  w_n = exp(-i pi n^2 / n0), b_d = conj(w_d),
// a cyclic convolution of length M (x holds M words): chirp and zero-pad, DFT,
// filter, inverse DFT, chirp.  bf holds the filter spectrum (M words) followed
// by the chirp w_n (n0 words), both precomputed on the host.  Here: the
// products, x_i = f(x_i, c_i) for i < n with c read in batches.
template <int NT, class F>
__device__ __forceinline__ void mul_table(double2* x, int n, const double2* __restrict__ c, F&& f) {
  for (int i0 = threadIdx.x; i0 < n; i0 += NT * kBatch) {
    double2 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) v[u] = c[min(i0 + u * NT, n - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (i0 + u * NT < n) x[i0 + u * NT] = f(x[i0 + u * NT], v[u]);
  }
}

// Sum of g_m = (F^c_m - i F^s_m) e^{i m phi0} over m = m0, m0 + S, ... <= L,
// e^{i m phi0} = conj(T[t_m]) with t_m = m num mod 2N stepping by tS; four
// loads in flight per step, summed in order of m.
__device__ __forceinline__ double2 sum_g(const double2* __restrict__ ph, int m0, int S, int L, int t,
                                         int tS, int twoN, const double2* __restrict__ T) {
  double2 acc = make_double2(0.0, 0.0);
  int m = m0;
  auto add = [&](double2 F) {
    acc = cadd(acc, cmulc(make_double2(F.x, -F.y), T[t]));
    t += tS;
    if (t >= twoN) t -= twoN;
  };
  for (; m + 3 * S <= L; m += 4 * S) {
    const double2 F0 = ph[m], F1 = ph[m + S], F2 = ph[m + 2 * S], F3 = ph[m + 3 * S];
    add(F0);
    add(F1);
    add(F2);
    add(F3);
  }
  for (; m <= L; m += S) add(ph[m]);
  return acc;
}

// Folded spectrum c_k = (G_k + conj G_{-k}) / 2 with G_k the sum of g_m over
// m = k mod N (0 <= k < N).
__device__ __forceinline__ double2 fold(const double2* __restrict__ ph, int k, int N, int L, int num,
                                        const FastDiv& d2N, int stepN, const double2* __restrict__ T) {
  const double2 a = sum_g(ph, k, N, L, (int)d2N.mod((unsigned)k * (unsigned)num), stepN, 2 * N, T);
  const int m1 = k == 0 ? 0 : N - k;
  const double2 b = sum_g(ph, m1, N, L, (int)d2N.mod((unsigned)m1 * (unsigned)num), stepN, 2 * N, T);
  return make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
}

// All transforms of one ring for a compiled-in length M.  Word i of the ring's
// n0 words: the samples 2 i and 2 i + 1 of an even ring, sample i of an odd one.
// From map `in` or, if that is NULL, from conj Z in x; the result goes to map
// `out` (synthesis) or into x.  bf: Bluestein's filter and chirp (NULL: direct
// transform, n0 = M); wt: the pixel weights of the round trip.
template <int NT, int M>
__device__ __forceinline__ void transforms(double2* x, const TwCtx& C, bool half, int n0,
                                           const double2* __restrict__ bf, const double* __restrict__ wt,
                                           const double* __restrict__ in, double* __restrict__ out) {
  const double2* __restrict__ chirp = bf + M;
  const double* io = in ? in : out ? out : wt;
  const bool a16 = (reinterpret_cast<uintptr_t>(io) & 15) == 0;
  auto pair = [&](const double* __restrict__ p, int i) -> double2 {
    if (!half) return make_double2(p[i], 0.0);
    if (a16) return reinterpret_cast<const double2*>(p)[i];
    return make_double2(p[2 * i], p[2 * i + 1]);
  };
  bool first = true;  // of the two passes of a Bluestein round trip
  auto ld = [&](auto& v, int j, int nb) {
    constexpr int R = sizeof(v) / sizeof(double2);
    if (bf) {
      // n0 <= M / 2: the points r >= R / 2 are the zero padding
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = make_double2(0.0, 0.0);
      double2 c[R / 2];
#pragma unroll
      for (int r = 0; r < R / 2; ++r) {
        const int i = min(j + r * nb, n0 - 1);
        c[r] = chirp[i];
        v[r] = in ? pair(in, i) : x[pad(i)];
      }
#pragma unroll
      for (int r = 0; r < R / 2; ++r) v[r] = j + r * nb < n0 ? cmul(v[r], c[r]) : make_double2(0.0, 0.0);
    } else if (in) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = pair(in, j + r * nb);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = x[pad(j + r * nb)];
    }
  };
  auto mid = [&](auto& v, int j, int nb) {
    constexpr int R = sizeof(v) / sizeof(double2);
    double2 c[R];
    if (bf) {
#pragma unroll
      for (int r = 0; r < R; ++r) c[r] = bf[j + r * nb];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = conj2(cmul(v[r], c[r]));
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) c[r] = pair(wt, j + r * nb);
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = make_double2(v[r].x * c[r].x, -v[r].y * c[r].y);
    }
  };
  auto st = [&](auto& v, int j, int nb) {
    constexpr int R = sizeof(v) / sizeof(double2);
    if (bf) {
      double2 c[R / 2];
#pragma unroll
      for (int r = 0; r < R / 2; ++r) c[r] = chirp[min(j + r * nb, n0 - 1)];
#pragma unroll
      for (int r = 0; r < R / 2; ++r) v[r] = cmulc(c[r], v[r]);
    }
    const bool weigh = bf && wt && first;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = j + r * nb;
      if (bf && (r >= R / 2 || i >= n0)) continue;
      if (out) {
        if (!half) {
          out[i] = v[r].x;
        } else if (a16) {
          reinterpret_cast<double2*>(out)[i] = conj2(v[r]);
        } else {
          out[2 * i] = v[r].x;
          out[2 * i + 1] = -v[r].y;
        }
      } else if (weigh) {
        const double2 w = pair(wt, i);
        x[pad(i)] = make_double2(v[r].x * w.x, -v[r].y * w.y);
      } else {
        x[pad(i)] = v[r];
      }
    }
  };
  for (;;) {
    // opaque to the compiler: it would keep every index and address of the
    // first pass in registers for the second (256 of them instead of 120)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    conv<NT, M>(tid, x, C, bf || wt, ld, mid, st);
    if (out) return;
    __syncthreads();
    if (!(bf && wt && first)) return;
    first = false;
  }
}

// ODD: the class has FFT lengths with odd radices (without it only the
// power-of-two stages are compiled, which takes fewer registers).
template <int NT, int MAXN, bool ODD>
__global__ __launch_bounds__(NT) void k_ring(RingArgs a, int mode, double2* __restrict__ phase,
                                             int64_t pstride, const double* __restrict__ map_in,
                                             double* __restrict__ map_out, int64_t mstride,
                                             const double* const* __restrict__ weights,
                                             int maps_per_weight) {
  extern __shared__ double2 lds[];
  double2* x = lds;
  double2* wf = lds + a.xcap;
  double2* wc = wf + 64;
  double2* cs = wf + a.wcap;  // tables of the prime radices
  double2* G = cs + a.pcap;   // fold scratch (short rings)
  const RingInfo* __restrict__ ri = a.info + blockIdx.x;
  const int map = blockIdx.y;
  if (a.skip.off(map)) return;  // whole block: before any barrier
  const int tid = threadIdx.x;
  const int L = a.lmax;
  const int N = ri->nphi;
  const bool half = (N & 1) == 0;     // two real samples per complex word
  const bool blue = ri->bfoff >= 0;   // Bluestein convolution
  const int n0 = half ? N / 2 : N;
  const int nf = ri->fftn;
  const int64_t off = ri->offset;
  const int num = ri->num;
  const double2* __restrict__ Tg = a.tw + ri->twoff;  // exp(-i pi t / N), t < 2 N
  double2* __restrict__ ph = phase + (int64_t)map * pstride + (int64_t)ri->ring * (L + 1);
  const int twoN = 2 * N;
  const bool fixed = nf == MAXN || nf == MAXN / 2 || nf == MAXN / 4;  // the length is compiled in
  const int sh = fixed ? 4 : 31;                    // x[i] sits at i + (i >> sh)
  {
    // twiddles of the FFT of length nf: at most one entry of each table per
    // thread (nf / 64 <= NT), loaded together
    const bool p2 = (nf & (nf - 1)) == 0;
    const double2* __restrict__ T = p2 ? a.tw2 : Tg;
    const int q = p2 ? kBlueMax / nf : half ? 4 : 2;
    const int nwf = min(64, nf), nwc = (nf + 63) / 64;
    const double2 f = T[q * min(tid & 63, nwf - 1)], c = T[64 * q * min(tid, nwc - 1)];
    if (tid < 64) wf[tid] = f;
    if (tid < nwc) wc[tid] = c;
    if constexpr (ODD) {
      double2* o = cs;
      if (!p2)
        for (int st = 0; st < ri->nfac; ++st) {
          const int p = ri->fac[st];
          if (p <= 7 || !(p & 1)) break;  // the primes come first
          const int qp = (int)((unsigned)twoN / (unsigned)p);
          for (int t = tid; t < p; t += NT) o[t] = Tg[t * qp];
          o += p;
        }
    }
  }
  // No barrier here: the LDS tables are first read after the barrier that
  // follows the fold (synthesis) or the input load (adjoint), so the table
  // copy and those global loads are in flight together.
  const TwCtx fc{wf, wc};
  const double2* __restrict__ bf = blue ? a.bf + ri->bfoff : nullptr;
  const FastDiv d2N((unsigned)twoN), dN((unsigned)N);
  double* xd = reinterpret_cast<double*>(x);
  const double* __restrict__ wt = mode == RING_ROUNDTRIP ? weights[map / maps_per_weight] + off : nullptr;

  // Even rings, H = N / 2 bins, in slots kk = 0 .. (H - 1) / 2 of four bins of the
  // full-length spectrum: kk, H - kk, H + kk, N - kk (slot 0: 0, H, H / 2, 3 H / 2).
  // With T = e^{-i pi kk / N} the phases e^{-i pi b / N} of the four are T, -i conj T,
  // -i T and -conj T, and m = b + c N differs from b by sg^c (sg = -1 on rings
  // with phi0 = pi / N, else 1), so a slot needs T and w = T^2 only, and the sums
  // over c are plain sums of F.
  const int H = n0, nk = (H + 1) / 2;
  const double sg = num ? -1.0 : 1.0;
  const bool even = (H & 1) == 0;
  const bool wide = half && 2 * L <= N;  // every m has its own bin: c = 0, and bins past H are empty
  auto at = [&](int i) { return i + (i >> sh); };
  auto bin = [&](int kk, int i) {
    if (kk) return i == 0 ? kk : i == 1 ? H - kk : i == 2 ? H + kk : N - kk;
    return i == 0 ? 0 : i == 1 ? H : even ? (i == 2 ? H / 2 : H + H / 2) : L + 1;
  };
  if (mode == RING_SYNTH || mode == RING_ROUNDTRIP) {
    const int stepN = (int)d2N.mod((unsigned)N * (unsigned)num);
    const bool shortr = N <= ring_short(NT) && !wide;
    if (shortr) {
      // short ring: all threads fold.  Thread p < S (S = N floor(threads / N))
      // sums g_m over m = p mod S; G_k then adds the S / N partials of bin k.
      const int S = N * (ring_short(NT) / N);
      double2* P = G + N;
      if (tid < S)
        P[tid] = sum_g(ph, tid, S, L, (int)d2N.mod((unsigned)tid * (unsigned)num),
                       (int)d2N.mod((unsigned)S * (unsigned)num), twoN, Tg);
      __syncthreads();
      for (int k = tid; k < N; k += NT) {
        double2 acc = P[k];
        for (int j = k + N; j < S; j += N) acc = cadd(acc, P[j]);
        G[k] = acc;
      }
      __syncthreads();
    }
    if (half) {
      // c_kk, c_{H-kk} (c_k = (G_k + conj G_{-k}) / 2, c Hermitian) and from them
      //   Z_kk = P + R, Z_{H-kk} = conj(P - R), P = c_kk + conj c_{H-kk},
      //   R = i conj(w) (c_kk - conj c_{H-kk});  x holds conj Z
      constexpr int U = 2;
      for (int k0 = tid; k0 < nk; k0 += NT * U) {
        double2 S[U][4], T[U], W[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kk = min(k0 + u * NT, nk - 1);
          W[u] = Tg[2 * kk];
          T[u] = Tg[kk ? kk : H / 2];  // read on rings with num != 0 only
          if (shortr) {
#pragma unroll
            for (int i = 0; i < 4; ++i) S[u][i] = G[min(bin(kk, i), N - 1)];
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (wide && (i == 3 || (i == 2 && kk != 0))) {
                S[u][i] = make_double2(0.0, 0.0);
                continue;
              }
              const int m = bin(kk, i);
              const double2 F = ph[min(m, L)];
              S[u][i] = make_double2(m <= L ? F.x : 0.0, m <= L ? -F.y : 0.0);
            }
          }
        }
        if (!shortr && !wide) {
          double s = sg;
          for (int c = N; c <= L; c += N) {
            double2 F[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int i = 0; i < 4; ++i) F[u][i] = ph[min(bin(min(k0 + u * NT, nk - 1), i) + c, L)];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const bool in = bin(min(k0 + u * NT, nk - 1), i) + c <= L;
                S[u][i].x = fma(s, in ? F[u][i].x : 0.0, S[u][i].x);
                S[u][i].y = fma(-s, in ? F[u][i].y : 0.0, S[u][i].y);
              }
            s *= sg;
          }
        }
        // short rings hold G itself (phases included)
        const bool turn = num && !shortr;
        const double sc = shortr ? 1.0 : sg;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kk = k0 + u * NT;
          const double2(&s)[4] = S[u];
          if (kk >= nk) continue;
          if (kk == 0) {
            const double cH = turn ? -s[1].y : s[1].x;
            x[0] = make_double2(s[0].x + cH, cH - s[0].x);
            if (even) {
              double2 A2 = make_double2(fma(sc, s[3].x, s[2].x), fma(-sc, s[3].y, s[2].y));
              if (turn) A2 = cmulc(A2, T[u]);
              x[at(H / 2)] = A2;
            }
          } else {
            double2 A2 = make_double2(fma(sc, s[3].x, s[0].x), fma(-sc, s[3].y, s[0].y));
            double2 B2 = make_double2(fma(sc, s[2].x, s[1].x), fma(-sc, s[2].y, s[1].y));
            if (turn) {
              A2 = cmulc(A2, T[u]);
              B2 = cmul(B2, T[u]);
              B2 = make_double2(-B2.y, B2.x);
            }
            const double2 Pp = make_double2(0.5 * (A2.x + B2.x), 0.5 * (A2.y - B2.y));
            const double2 Q = make_double2(0.5 * (A2.x - B2.x), 0.5 * (A2.y + B2.y));
            const double2 t = cmulc(Q, W[u]);
            x[at(kk)] = make_double2(Pp.x - t.y, -Pp.y - t.x);
            x[at(H - kk)] = make_double2(Pp.x + t.y, Pp.y - t.x);
          }
        }
      }
    } else {
      for (int k = tid; k < n0; k += NT) {
        if (shortr) {
          const double2 u = G[k], v = G[k == 0 ? 0 : N - k];
          x[at(k)] = make_double2(0.5 * (u.x + v.x), 0.5 * (v.y - u.y));
        } else {
          x[at(k)] = conj2(fold(ph, k, N, L, num, d2N, stepN, Tg));
        }
      }
    }
  } else if (!fixed) {
    const double* in = map_in + (int64_t)map * mstride + off;
    if (half && (reinterpret_cast<uintptr_t>(in) & 15) == 0) {
      const double2* i2 = reinterpret_cast<const double2*>(in);
      for (int j0 = tid; j0 < H; j0 += NT * kBatch) {
        double2 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v[u] = i2[min(j0 + u * NT, H - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          if (j0 + u * NT < H) x[j0 + u * NT] = v[u];
      }
    } else {
      for (int j0 = tid; j0 < N; j0 += NT * kBatch) {
        double v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v[u] = in[min(j0 + u * NT, N - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const int j = j0 + u * NT;
          if (j >= N) continue;
          if (half)
            xd[j] = v[u];
          else
            x[j] = make_double2(v[u], 0.0);
        }
      }
    }
  }
  __syncthreads();
  // The transforms: of conj Z (its conjugate is the ring's samples) in synthesis
  // and round trip, of the ring's samples in adjoint and round trip.
  const bool syn = mode == RING_SYNTH || mode == RING_ROUNDTRIP;
  if (fixed) {
    const double* in = syn ? nullptr : map_in + (int64_t)map * mstride + off;
    double* out = mode == RING_SYNTH ? map_out + (int64_t)map * mstride + off : nullptr;
    if (nf == MAXN) transforms<NT, MAXN>(x, fc, half, n0, bf, wt, in, out);
    else if (nf == MAXN / 2) transforms<NT, MAXN / 2>(x, fc, half, n0, bf, wt, in, out);
    else transforms<NT, MAXN / 4>(x, fc, half, n0, bf, wt, in, out);
    if (mode == RING_SYNTH) return;
  }
  // any other length, one loop, so that the FFT's code is there once
#pragma unroll 1
  for (int tr = fixed ? 2 : syn ? 0 : 1; tr < 2; ++tr) {
    if (blue) {
      mul_table<NT>(x, n0, bf + nf, [](double2 v, double2 c) { return cmul(v, c); });
      for (int i = n0 + tid; i < nf; i += NT) x[i] = make_double2(0.0, 0.0);
      __syncthreads();
    }
#pragma unroll 1
    for (int pass = blue ? 0 : 1; pass < 2; ++pass) {
      fft_lds<NT, MAXN, !ODD>(x, nf, ri, fc, cs);
      if (pass == 0) {
        mul_table<NT>(x, nf, bf, [](double2 v, double2 c) { return conj2(cmul(v, c)); });
        __syncthreads();
      }
    }
    if (blue) {
      mul_table<NT>(x, n0, bf + nf, [](double2 v, double2 c) { return cmulc(c, v); });
      __syncthreads();
    }
    if (tr == 1) break;
    if (mode == RING_SYNTH) {
      double* out = map_out + (int64_t)map * mstride + off;
      if (half && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        double2* o2 = reinterpret_cast<double2*>(out);
        for (int j = tid; j < H; j += NT) o2[j] = conj2(x[j]);
      } else if (half) {
        for (int j = tid; j < N; j += NT) out[j] = j & 1 ? -xd[j] : xd[j];
      } else {
        for (int j = tid; j < N; j += NT) out[j] = x[j].x;
      }
      return;
    }
    const int st = half ? 1 : 2;  // real samples sit in consecutive words, or in the real parts
    for (int j0 = tid; j0 < N; j0 += NT * kBatch) {
      double wv[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) wv[u] = wt[min(j0 + u * NT, N - 1)];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u * NT;
        if (j < N) {
          xd[st * j] *= half && (j & 1) ? -wv[u] : wv[u];
          if (!half) xd[st * j + 1] = 0.0;
        }
      }
    }
    __syncthreads();
  }

  // forward DFT of the real ring data at bin k (0 <= k < N)
  auto spec = [&](int k) -> double2 {
    if (half) {
      const int kk = k >= n0 ? k - n0 : k;
      const int k2 = kk == 0 ? 0 : n0 - kk;
      const double2 Zk = x[at(kk)], Zc = conj2(x[at(k2)]);
      const double2 E = make_double2(0.5 * (Zk.x + Zc.x), 0.5 * (Zk.y + Zc.y));
      const double2 D = csub(Zk, Zc);
      const double2 O = make_double2(0.5 * D.y, -0.5 * D.x);  // D / (2i)
      return cadd(E, cmul(Tg[2 * k], O));
    } else {
      return x[at(k)];
    }
  };
  if (mode == RING_DIAG) {
    const double t0 = spec(0).x;
    for (int m = tid; m <= L; m += NT) {
      if (m == 0) {
        ph[0] = make_double2(t0, 0.0);
      } else {
        const unsigned m2 = d2N.mod(2u * (unsigned)m);
        const int k = (int)dN.mod(m2);
        const double2 X = cmul(spec(k), Tg[(int)d2N.mod(m2 * (unsigned)num)]);
        ph[m] = make_double2(t0 + X.x, t0 - X.x);
      }
    }
    return;
  }
  if (half && N > ring_short(NT)) {
    // Slots as in the fold: with E, O of (Z_kk, conj Z_{H-kk}) the bins are F^_kk =
    // E + w O and F^_{H-kk} = conj(E - w O); H of the other two are sg conj of
    // these two, and m = b + c N repeats its bin with sg^c.
    constexpr int U = 2;
    for (int k0 = tid; k0 < nk; k0 += NT * U) {
      double2 T[U], W[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kk = min(k0 + u * NT, nk - 1);
        W[u] = Tg[2 * kk];
        T[u] = Tg[kk ? kk : H / 2];  // read on rings with num != 0 only
      }
      auto slot = [&](int kk, double2 Wk, double2 Tk) {
        if (kk >= nk) return;
        double2 V[4];  // (H^c, H^s) of the four bins
        if (kk == 0) {
          const double2 Z = x[0];
          V[0] = make_double2(Z.x + Z.y, 0.0);
          V[1] = num ? make_double2(0.0, Z.x - Z.y) : make_double2(Z.x - Z.y, 0.0);
          double2 v = even ? conj2(x[at(H / 2)]) : Z;
          if (num) v = cmul(v, Tk);
          V[2] = conj2(v);
          V[3] = make_double2(sg * v.x, sg * v.y);
        } else {
          const double2 Zk = x[at(kk)], Zc = conj2(x[at(H - kk)]);
          const double2 E = make_double2(0.5 * (Zk.x + Zc.x), 0.5 * (Zk.y + Zc.y));
          const double2 D = csub(Zk, Zc);
          const double2 wO = cmul(Wk, make_double2(0.5 * D.y, -0.5 * D.x));  // O = D / (2i)
          double2 v0 = cadd(E, wO), v1 = conj2(csub(E, wO));
          if (num) {
            v0 = cmul(v0, Tk);
            v1 = cmulc(v1, Tk);
            v1 = make_double2(v1.y, -v1.x);
          }
          V[0] = conj2(v0);
          V[1] = conj2(v1);
          V[2] = make_double2(sg * v1.x, sg * v1.y);
          V[3] = make_double2(sg * v0.x, sg * v0.y);
        }
        double s = 1.0;
        for (int c = 0; c <= L; c += N) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (wide && (i == 3 || (i == 2 && kk != 0))) continue;
            const int m = bin(kk, i) + c;
            if (m <= L) ph[m] = make_double2(s * V[i].x, s * V[i].y);
          }
          s *= sg;
        }
      };
      slot(k0, W[0], T[0]);
      slot(k0 + NT, W[1], T[1]);
    }
    return;
  }
  for (int m = tid; m <= L; m += NT) {
    // H_m = e^{-i m phi0} F^_{m mod N};  e^{-i m phi0} = T[m num mod 2N]
    const unsigned mm = d2N.mod((unsigned)m);
    const double2 h = cmul(spec((int)dN.mod(mm)), Tg[(int)d2N.mod(mm * (unsigned)num)]);
    ph[m] = make_double2(h.x, m == 0 ? 0.0 : -h.y);
  }
}

}  // namespace

RingArgs ring_args(crs_grid g, int lmax);

void launch_ring(crs_grid g, int lmax, RingMode mode, int nmaps, double2* phase, int64_t pstride,
                 const double* map_in, double* map_out, int64_t mstride,
                 const double* const* weights, int maps_per_weight, hipStream_t s, MapSkip skip) {
  CRS_CHECK(lmax < 65536, CRS_EUNSUPPORTED, "lmax above 65535 is not supported by the ring stage");
  RingArgs base = ring_args(g, lmax);
  base.skip = skip;
  const int mpw = maps_per_weight < 1 ? 1 : maps_per_weight;
  const int md = (int)mode;
  auto launch_class = [&](const RingClass& rc, const RingInfo* info) {
    if (rc.rings.empty()) return;
    RingArgs a = base;
    a.xcap = rc.xcap;
    a.wcap = rc.wcap;
    a.pcap = rc.pcap;
    a.info = info;
    const dim3 grid((unsigned)rc.rings.size(), nmaps);
    const size_t words = (size_t)rc.xcap + rc.wcap + rc.pcap + rc.gcap;
    const size_t lds = words * sizeof(double2);
    CRS_CHECK(lds <= kMaxLds, CRS_EUNSUPPORTED, "ring class needs " + std::to_string(lds) + " bytes of LDS");
    switch (rc.tier * 2 + (rc.odd ? 1 : 0)) {
#define CRS_RING(T, NT, MAXN, ODD)                                                                   \
  case T * 2 + ODD:                                                                                  \
    hipLaunchKernelGGL((k_ring<NT, MAXN, ODD>), grid, dim3(NT), lds, s, a, md, phase, pstride,       \
                       map_in, map_out, mstride, weights, mpw);                                      \
    break;
      CRS_RING(0, 64, 512, false)
      CRS_RING(0, 64, 512, true)
      CRS_RING(1, 128, 1024, false)
      CRS_RING(1, 128, 1024, true)
      CRS_RING(2, 256, 2048, false)
      CRS_RING(2, 256, 2048, true)
      CRS_RING(3, 512, 4096, false)
      CRS_RING(3, 512, 4096, true)
      CRS_RING(4, 1024, 8192, false)
      CRS_RING(4, 1024, 8192, true)
#undef CRS_RING
      default: throw Error{CRS_EUNSUPPORTED, "ring FFT length above 8192"};
    }
    CRS_HIP(hipGetLastError());
  };
  // Launches on a stream run one after another, so a class of a few hundred
  // blocks would leave most CUs idle for a whole block's duration: the
  // classes with fewer than kMinClassBlocks blocks (the first `nsmall` in
  // order of ring count) run together as one launch, the others on their own.
  // Where that launch's blocks are small (up to 256 threads) it takes further
  // classes up to kMergedBlocks blocks, which all fit on the GPU in two or
  // three turns.  Ring stage in us, separate / merged: Nside 256 x2 30.7 / 22.8,
  // x4 40.9 / 33.3, x6 47.1 / 43.9, x8 53.1 / 54.2; Nside 512 x1 45.1 / 35.2, x2 65.0 /
  // 58.0, x3 84.2 / 81.4, x4 100 / 104; with blocks of 512 threads Nside 1024 x1 147 /
  // 171, x2 202 / 279.
  constexpr int64_t kMinClassBlocks = 1024, kMergedBlocks = 6144;
  constexpr int kMergedTier = 2;
  const int ncls = (int)g->ring_classes.size();
  int nsmall = 0;
  while (nsmall < ncls) {
    const RingClass& m = g->ring_prefix[nsmall];
    const int64_t own = (int64_t)g->ring_classes[g->ring_small_order[nsmall]].rings.size() * nmaps;
    if (own >= kMinClassBlocks &&
        (m.tier > kMergedTier || (int64_t)m.rings.size() * nmaps >= kMergedBlocks))
      break;
    ++nsmall;
  }
  bool small[kMaxRingClasses] = {};
  for (int k = 0; k < nsmall; ++k) small[g->ring_small_order[k]] = true;
  for (int c = 0; c < ncls; ++c)
    if (!small[c]) launch_class(g->ring_classes[c], g->d_ring_class[c].p);
  if (nsmall > 0) launch_class(g->ring_prefix[nsmall - 1], g->d_ring_prefix[nsmall - 1].p);
}

}  // namespace crs
