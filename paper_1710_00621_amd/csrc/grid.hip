// Ring grids (HEALPix RING, Gauss-Legendre), per-ring FFT tables and the
// per-(grid, lmax) Legendre plans.
//
// HEALPix RING geometry follows Gorski et al. (2005); the paper uses HEALPix
// sky maps and recommends Gauss-Legendre grids where exact quadrature is
// wanted (Sect. 2.1, Sect. 2.2 below eq:Q).
#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace crs {

namespace {

// sin(pi x), cos(pi x) with exact argument reduction (x a ratio of integers
// reduced modulo 2 by the caller); accurate to a few ulps.
void host_sincospi(double x, double* s, double* c) {
  x = std::fmod(x, 2.0);
  if (x < 0) x += 2.0;
  // reduce to [0, 0.5] using symmetries
  double sign_s = 1.0, sign_c = 1.0;
  if (x >= 1.0) { x -= 1.0; sign_s = -1.0; sign_c = -1.0; }
  if (x > 0.5) { x = 1.0 - x; sign_c = -sign_c; }
  double ss, cc;
  if (x <= 0.25) {
    ss = std::sin(M_PI * x);
    cc = std::cos(M_PI * x);
  } else {
    double y = 0.5 - x;
    ss = std::cos(M_PI * y);
    cc = std::sin(M_PI * y);
  }
  *s = sign_s * ss;
  *c = sign_c * cc;
}

// Radices of an FFT of length n: the power-of-two part 2^e in as few stages
// as possible (radix 8, with 2^4 as 4 x 4 and a remaining 2^2 as one radix
// 4), then the odd prime factors in increasing order.
std::vector<int> factorize(int n) {
  std::vector<int> f;
  int e = 0;
  while (n % 2 == 0) { ++e; n /= 2; }
  for (int p = 3; p * p <= n; p += 2)
    while (n % p == 0) { f.push_back(p); n /= p; }
  if (n > 1) f.push_back(n);
  std::sort(f.begin(), f.end(), std::greater<int>());
  for (int s = 0; pow2_radix(e, s) > 0; ++s) f.push_back(pow2_radix(e, s));
  if (f.empty()) f.push_back(1);
  return f;
}

// Largest prime factor of an FFT length n0 that the ring kernel computes
// directly (p - 1 FMAs per point); a length with a larger one goes through
// Bluestein's convolution of 2 n0 .. 4 n0 points.  The direct sums are long
// serial loops, which short rings (few blocks, a short FFT) cannot hide: ring
// stage in us with the line at 7 / 19 / 31 / 61 / 97 for every length,
//   Nside 64, 20 maps (n0 <= 128):    20.9  20.4  21.5  25.7  25.2
//   33 x 65 GL, 1 map (n0 = 65):       9.2  10.2  10.3  10.7  10.3
//   Nside 256, 1 map (n0 <= 512):     15.9  17.2  17.0  19.8  23.8
//   Nside 256, 42 maps (n0 <= 512):    218   218   218   231   239
//   Nside 1024, 6 maps (n0 <= 2048):   554   544   530   530   532
//   Nside 1024, 4 maps, adjoint:       355   344   348   339   345
//   512 x 1026 GL, 40 maps (n0 = 513 = 19 3^3): 306 through Bluestein, 152 directly
int prime_max(int n0) { return n0 <= 128 ? 7 : n0 <= 512 ? 19 : n0 <= 1024 ? 31 : 61; }

// In-place radix-2 complex FFT (forward, exp(-2 pi i jk / n)), n a power of two.
void host_fft_pow2(std::vector<double2>& x) {
  const int n = (int)x.size();
  for (int i = 1, j = 0; i < n; ++i) {
    int bit = n >> 1;
    for (; j & bit; bit >>= 1) j ^= bit;
    j ^= bit;
    if (i < j) std::swap(x[i], x[j]);
  }
  for (int len = 2; len <= n; len <<= 1) {
    const int h = len / 2;
    for (int k = 0; k < h; ++k) {
      double sv, cv;
      host_sincospi(-2.0 * k / len, &sv, &cv);
      for (int i = k; i < n; i += len) {
        const double2 u = x[i], v = x[i + h];
        const double2 t = make_double2(v.x * cv - v.y * sv, v.x * sv + v.y * cv);
        x[i] = make_double2(u.x + t.x, u.y + t.y);
        x[i + h] = make_double2(u.x - t.x, u.y - t.y);
      }
    }
  }
}

// Bluestein filter for a length-n DFT by a length-M cyclic convolution
// (M >= 2n - 1): b_d = exp(+i pi d^2 / n) for |d| < n, wrapped to M, and
// its forward DFT divided by M (so that the device inverse FFT needs no
// scaling).  Phases are reduced exactly: d^2 mod 2n.
std::vector<double2> bluestein_filter(int n, int M) {
  std::vector<double2> b(M, make_double2(0.0, 0.0));
  for (int d = 0; d < n; ++d) {
    double sv, cv;
    const long long t = ((long long)d * d) % (2LL * n);
    host_sincospi((double)t / n, &sv, &cv);
    b[d] = make_double2(cv, sv);
    if (d) b[M - d] = b[d];
  }
  host_fft_pow2(b);
  for (auto& v : b) v = make_double2(v.x / M, v.y / M);
  // followed by the chirp w_d = exp(-i pi d^2 / n), d < n
  for (int d = 0; d < n; ++d) {
    double sv, cv;
    const long long t = ((long long)d * d) % (2LL * n);
    host_sincospi((double)t / n, &sv, &cv);
    b.push_back(make_double2(cv, -sv));
  }
  return b;
}

// P_n(cos th) and P_{n-1}(cos th) by the Legendre recurrence written for
// D_j = P_j - P_{j-1} and t = 1 - cos th = 2 sin^2(th / 2):
//   D_j = ((j - 1) D_{j-1} - (2j - 1) t P_{j-1}) / j,   P_j = P_{j-1} + D_j.
// It carries the deviation of P_j from P_j(1) = 1 explicitly, with t taken
// from th, so the values keep full relative precision near the pole (the
// recurrence in x = cos th inherits the rounding of x, which near the poles
// moves P_{n-1} by about 1e-6 relative at n = 4000).
void legendre_theta(int n, double th, double& pn, double& pm1) {
  const double sh = std::sin(0.5 * th);
  const double t = 2.0 * sh * sh;
  double prev = 1.0, p = 1.0 - t, d = -t;  // P_0, P_1, D_1
  for (int j = 2; j <= n; ++j) {
    d = ((j - 1.0) * d - (2.0 * j - 1.0) * t * p) / j;
    prev = p;
    p += d;
  }
  pn = n == 0 ? 1.0 : p;
  pm1 = n == 0 ? 0.0 : prev;
}

// Gauss-Legendre nodes (descending) and weights: Newton iteration on theta
// for the nodes of the northern half (theta <= pi / 2), the southern half by
// symmetry; weights w = 2 sin^2 th / (n P_{n-1}(cos th))^2.
void gl_nodes(int n, std::vector<double>& z, std::vector<double>& st, std::vector<double>& w) {
  z.resize(n);
  st.resize(n);
  w.resize(n);
  for (int k = 0; k < (n + 1) / 2; ++k) {
    double th = M_PI * (k + 0.75) / (n + 0.5);
    double pn = 0, pm1 = 0;
    for (int it = 0; it < 100; ++it) {
      legendre_theta(n, th, pn, pm1);
      // d/dth P_n(cos th) = n (cos th P_n - P_{n-1}) / sin th
      const double dth = pn * std::sin(th) / (n * (std::cos(th) * pn - pm1));
      th -= dth;
      if (std::fabs(dth) < 1e-16) break;
    }
    legendre_theta(n, th, pn, pm1);
    const double s = std::sin(th);
    const double x = (2 * k + 1 == n) ? 0.0 : std::cos(th);
    const double wk = 2.0 * s * s / ((n * pm1) * (n * pm1));
    z[k] = x;
    st[k] = s;
    w[k] = wk;
    z[n - 1 - k] = -x;
    st[n - 1 - k] = s;
    w[n - 1 - k] = wk;
  }
}

}  // namespace

// Ring pairs in slots, tiles of 64, for the Legendre kernels: every tile runs
// one form of the recurrence (legendre.hip), whose errors grow as 1 / sin(2
// theta) away from its own end.  The 32 pairs next to the equator sit in the
// last tile, each in slots i and 32 + i: the even functions are taken from the
// second.  Beyond them (|z| 0.08 at Nside 256, 0.02 at Nside 1024) the even
// functions' cancellation 1 / |z| is below the sqrt(L) by which rounding adds up
// in any form.  The polar pairs and the belt's are padded to whole tiles; their
// boundary lies between 35 and 55 degrees where the tiles are fewest (adjoint, us,
// against the nearest multiple of 64: Nside 32 / L 64 x65 44 and 48, Nside 37 / L 90
// x20 27 and 32, Nside 96 / L 192 x20 72 and 76), then the groups of four and of two
// that the kernels take, without padding of the polar slots if it can (Nside 256 /
// L 512 x42: 787, with both parts padded 800), and next to 45 degrees.
static void slot_layout(crs_grid g) {
  const int np = (g->nring + 1) / 2;
  const double lo = 0.329, hi = 0.671;  // cos^2 of 55 and 35 degrees
  int p45 = 0;
  while (p45 < np && g->z[p45] * g->z[p45] >= 0.5) ++p45;
  auto up = [](int n, int unit) { return (n + unit - 1) / unit; };
  std::array<int, 5> best = {INT_MAX, 0, 0, 0, 0};
  for (int c = 0; c <= np; ++c) {
    const bool in = (c == 0 || g->z[c - 1] * g->z[c - 1] >= lo) && (c == np || g->z[c] * g->z[c] <= hi);
    if (!in && c != p45) continue;
    const int belt = np - c - std::min(32, np - c), a = up(c, 64), b = up(belt, 64);
    const std::array<int, 5> key = {a + b, up(a, 4) + up(b, 4), up(a, 2) + up(b, 2), c % 64 != 0, std::abs(c - p45)};
    if (key < best) {
      best = key;
      g->pol_pairs = c;
      g->pol_tiles = a;
      g->eq_pairs = std::min(32, np - c);
      g->nslots = 64 * (a + b + 1);
    }
  }
}

// Two doubles whose product is sin^2 theta = (1 - z)(1 + z) to about 2^-60: the
// recurrence takes the product inside an FMA, so its rounding does not enter.
// Neighbouring doubles a give products a fl(sin^2 / a) with residuals spread
// over an ulp; the best of 64 is taken.
static void sin2_factors(double z, double* fa, double* fc) {
  const double w = 1.0 - z;  // exact for z >= 1/2
  const double p = std::fma(-w, w, 2.0 * w), pe = std::fma(-w, w, 2.0 * w - p);  // sin^2 = 2 w - w^2 = p + pe
  double a = w, best = HUGE_VAL;
  for (int i = 0; i < 64; ++i, a = std::nextafter(a, 2.0)) {
    const double c = p / a;
    const double r = std::fabs(std::fma(a, c, -p) - pe);
    if (r < best) {
      best = r;
      *fa = a;
      *fc = c;
    }
  }
}

// Uploads per-ring tables (lengths, offsets, phi0, FFT factors, twiddles).
void grid_finalize(crs_grid g, hipStream_t s) {
  int nr = g->nring;
  g->offset.resize(nr);
  int64_t off = 0;
  for (int r = 0; r < nr; ++r) {
    g->offset[r] = off;
    off += g->nphi[r];
  }
  g->npix = off;
  for (int r = 0; r < nr; ++r)
    CRS_CHECK(g->nphi[r] <= kMaxRing, CRS_EUNSUPPORTED,
              "ring length above 8192 pixels is not supported");
  // Per ring: the complex FFT that the ring kernels run.  Even Nphi uses a
  // half-length complex transform (two real samples per complex word); a
  // length whose largest prime factor exceeds prime_max goes through
  // Bluestein's chirp convolution with a power-of-two FFT.
  std::vector<RingInfo> info(nr);
  std::map<int, int64_t> tw_of, bf_of;
  std::vector<double2> tw, bf;
  g->ring_classes.clear();
  std::map<int, int> class_of;
  bool any_pow2 = false;
  for (int r = 0; r < nr; ++r) {
    const int n = g->nphi[r];
    RingInfo& ri = info[r];
    ri = RingInfo{};
    ri.ring = r;
    ri.nphi = n;
    ri.num = g->phi0_num[r];
    ri.offset = g->offset[r];
    ri.bfoff = -1;
    const bool half = (n % 2) == 0;
    const int n0 = half ? n / 2 : n;
    auto f0 = factorize(n0);
    const int pmax = f0[0];  // the largest odd prime, if there is one
    bool blue = (pmax & 1) && pmax > prime_max(n0);
    CRS_CHECK(n0 <= 4096 || !(pmax & 1) || pmax <= 7, CRS_EUNSUPPORTED,
              "ring FFT above 8192 points (an odd ring longer than 4096 pixels with a prime factor above 7)");
    int nf = n0;
    if (blue) {
      nf = 1;
      while (nf < 2 * n0 - 1) nf *= 2;
      auto it = bf_of.find(n0);
      if (it == bf_of.end()) {
        bf_of[n0] = (int64_t)bf.size();
        ri.bfoff = (int64_t)bf.size();
        auto spec = bluestein_filter(n0, nf);
        bf.insert(bf.end(), spec.begin(), spec.end());
      } else {
        ri.bfoff = it->second;
      }
    }
    auto ff = factorize(nf);
    CRS_CHECK((int)ff.size() <= kRingStages, CRS_EUNSUPPORTED, "too many FFT factors");
    ri.nfac = (int)ff.size();
    ri.fftn = nf;
    unsigned ns = 1;
    for (size_t i = 0; i < ff.size(); ++i) {
      ri.fac[i] = ff[i];
      ri.facm[i] = ns <= 1 ? 0u : (unsigned)(0xFFFFFFFFull / ns + 1);
      ns *= (unsigned)ff[i];
    }
    any_pow2 = any_pow2 || (nf & (nf - 1)) == 0;
    auto it = tw_of.find(n);
    if (it == tw_of.end()) {
      int64_t o = (int64_t)tw.size();
      tw_of[n] = o;
      for (int t = 0; t < 2 * n; ++t) {
        double sv, cv;
        host_sincospi((double)t / (double)n, &sv, &cv);
        tw.push_back(make_double2(cv, -sv));
      }
      ri.twoff = o;
    } else {
      ri.twoff = it->second;
    }
    int tier = 0;
    while (ring_tier_maxfft(tier) < nf) ++tier;
    // classes by (tier, Bluestein, odd radix) from the 256-thread tier up: a
    // class without odd radices runs a kernel built for power-of-two FFTs
    // only (107 to 115 instead of 127 registers), and Bluestein's longer
    // buffers do not set the LDS size of the direct rings.  The smaller tiers
    // stay whole (the difference is less than an extra launch costs).
    bool odd = false;
    for (int v : ff) odd = odd || (v % 2) != 0;
    const int key = tier >= 2 ? tier * 4 + (blue ? 2 : 0) + (odd ? 1 : 0) : tier * 4;
    auto ci = class_of.find(key);
    if (ci == class_of.end()) {
      class_of[key] = (int)g->ring_classes.size();
      g->ring_classes.emplace_back();
      g->ring_classes.back().tier = tier;
      ci = class_of.find(key);
    }
    RingClass& rc = g->ring_classes[ci->second];
    rc.rings.push_back(r);
    rc.blue = rc.blue || blue;
    rc.odd = rc.odd || odd;
    rc.xcap = std::max(rc.xcap, nf + nf / 16);
    rc.wcap = std::max(rc.wcap, 64 + (nf + 63) / 64);
    int pw = 0;
    for (int v : ff) pw += v > 7 && (v & 1) ? v : 0;
    rc.pcap = std::max(rc.pcap, pw);
    const int nt = ring_tier_threads(tier);
    if (n <= ring_short(nt)) rc.gcap = std::max(rc.gcap, n + n * (ring_short(nt) / n));
  }
  // largest tier first
  std::stable_sort(g->ring_classes.begin(), g->ring_classes.end(),
                   [](const RingClass& x, const RingClass& y) { return x.tier > y.tier; });
  g->d_ring_class.clear();
  std::vector<std::vector<RingInfo>> hold;  // uploaded from: alive until the sync below
  auto records = [&](const std::vector<int>& rings) -> const std::vector<RingInfo>& {
    hold.emplace_back();
    for (int r : rings) hold.back().push_back(info[r]);
    return hold.back();
  };
  for (auto& rc : g->ring_classes) {
    g->d_ring_class.emplace_back();
    g->d_ring_class.back().upload(records(rc.rings), s);
  }
  // Launches with few maps merge the classes that would have too few blocks
  // to fill the GPU on their own into one launch (run by the kernel of their
  // largest tier).  Which classes are small depends on the map count, but
  // they are always the first ones in order of ring count, so the merged
  // class of every such prefix is prepared here.
  const int ncls = (int)g->ring_classes.size();
  CRS_CHECK(ncls <= kMaxRingClasses, CRS_EUNSUPPORTED, "too many ring classes");
  g->ring_small_order.resize(ncls);
  for (int c = 0; c < ncls; ++c) g->ring_small_order[c] = c;
  std::stable_sort(g->ring_small_order.begin(), g->ring_small_order.end(), [&](int x, int y) {
    return g->ring_classes[x].rings.size() < g->ring_classes[y].rings.size();
  });
  g->ring_prefix.clear();
  g->d_ring_prefix.clear();
  RingClass acc;
  for (int k = 0; k < ncls; ++k) {
    const RingClass& rc = g->ring_classes[g->ring_small_order[k]];
    acc.tier = std::max(acc.tier, rc.tier);
    acc.blue = acc.blue || rc.blue;
    acc.odd = acc.odd || rc.odd;
    acc.xcap = std::max(acc.xcap, rc.xcap);
    acc.wcap = std::max(acc.wcap, rc.wcap);
    acc.pcap = std::max(acc.pcap, rc.pcap);
    acc.rings.insert(acc.rings.end(), rc.rings.begin(), rc.rings.end());
    RingClass m = acc;
    std::sort(m.rings.begin(), m.rings.end());
    // fold scratch for the merged kernel's block size
    const int nt = ring_tier_threads(m.tier);
    m.gcap = 0;
    for (int r : m.rings) {
      const int n = g->nphi[r];
      if (n <= ring_short(nt)) m.gcap = std::max(m.gcap, n + n * (ring_short(nt) / n));
    }
    g->ring_prefix.push_back(m);
    g->d_ring_prefix.emplace_back();
    g->d_ring_prefix.back().upload(records(m.rings), s);
  }
  std::vector<double2> t2;
  if (any_pow2) {
    t2.resize(kBlueMax);
    for (int t = 0; t < kBlueMax; ++t) {
      double sv, cv;
      host_sincospi(2.0 * t / kBlueMax, &sv, &cv);
      t2[t] = make_double2(cv, -sv);
    }
    g->d_tw2.upload(t2, s);
  }
  if (!bf.empty()) g->d_bf.upload(bf, s);
  slot_layout(g);
  std::vector<double> zs(g->nslots, 0.0), ss(g->nslots, 1.0), ya(g->nslots, 0.0), yc(g->nslots, 0.0);
  for (int p = 0; p < (nr + 1) / 2; ++p) {
    const bool polar = p < g->pol_pairs;
    const int e = p - ((nr + 1) / 2 - g->eq_pairs);  // pair of the equator's tile
    const int i = polar ? p : e >= 0 ? g->nslots - 64 + e : p - g->pol_pairs + 64 * g->pol_tiles;
    zs[i] = g->z[p];
    ss[i] = g->sint[p];
    // sin^2 theta of the ring's z as stored: the functions are those at the
    // pixel centres the grid reports
    ya[i] = yc[i] = g->z[p];
    if (polar) sin2_factors(g->z[p], &ya[i], &yc[i]);
    if (e >= 0)
      for (auto* v : {&zs, &ss, &ya, &yc}) (*v)[i + 32] = (*v)[i];
  }
  g->d_tw.upload(tw, s);
  g->d_zs.upload(zs, s);
  g->d_ss.upload(ss, s);
  g->d_ya.upload(ya, s);
  g->d_yc.upload(yc, s);
  CRS_HIP(hipStreamSynchronize(s));
}

void build_healpix(crs_grid g, int nside) {
  g->kind = 0;
  g->nside = nside;
  int nr = 4 * nside - 1;
  g->nring = nr;
  g->z.resize(nr);
  g->sint.resize(nr);
  g->nphi.resize(nr);
  g->phi0_num.resize(nr);
  g->phi0_den.resize(nr);
  g->ringw.assign(nr, 4.0 * M_PI / (12.0 * nside * (double)nside));
  double ns = nside;
  for (int k = 0; k < nr; ++k) {
    int i = k + 1;
    if (i < nside || i > 3 * nside) {
      int ii = (i < nside) ? i : 4 * nside - i;
      double om = (double)ii * ii / (3.0 * ns * ns);  // 1 - |z|
      double zz = 1.0 - om;
      g->z[k] = (i < nside) ? zz : -zz;
      g->sint[k] = std::sqrt(om * (2.0 - om));
      g->nphi[k] = 4 * ii;
      g->phi0_num[k] = 1;   // phi0 = pi / (4 ii) = pi / nphi
      g->phi0_den[k] = 4 * ii;
    } else {
      double zz = 4.0 / 3.0 - (2.0 * i) / (3.0 * ns);
      g->z[k] = zz;
      g->sint[k] = std::sqrt((1.0 - zz) * (1.0 + zz));
      g->nphi[k] = 4 * nside;
      bool shifted = ((i - nside) % 2) == 0;
      g->phi0_num[k] = shifted ? 1 : 0;
      g->phi0_den[k] = 4 * nside;
    }
  }
}

void build_gl(crs_grid g, int nrings, int nphi) {
  g->kind = 1;
  g->nring = nrings;
  g->nphi_gl = nphi;
  std::vector<double> w;
  gl_nodes(nrings, g->z, g->sint, w);
  g->nphi.assign(nrings, nphi);
  g->phi0_num.assign(nrings, 0);
  g->phi0_den.assign(nrings, nphi);
  g->ringw.resize(nrings);
  for (int r = 0; r < nrings; ++r) g->ringw[r] = w[r] * 2.0 * M_PI / nphi;
}

// ----------------------------------------------------------- Legendre plan
// Coefficients of the recurrence in legendre.hip.  With eta_l = (4 m^2 - 1) /
// (4 (4 l^2 - 1)), eps_l^2 = 1/4 - eta_l; g = eps_l eps_{l-1} = 1/4 - delta with
// delta = (eta_l / 4 + eta_{l-1} eps_l^2) / (1/4 + g).  At l = m + 2k + 1
//     1 - eps_{l+1}^2 - eps_l^2 - g_k - g_{k+1} = (eta_l + eta_{l+1}) + (delta_k + delta_{k+1})
//     eps_{l+1}^2 + eps_l^2 - g_k - g_{k+1} = eps_l s_l - eps_{l+1} s_{l+2},
// s_l = eps_l - eps_{l-1} = (eta_{l-1} - eta_l) / (eps_l + eps_{l-1}) with eta_{l-1} - eta_l =
// (4 m^2 - 1) / ((2l - 3)(2l - 1)(2l + 1)): the second, O(m^2 / l^3), is multiplied
// by q, l times lambda next to the equator, and as (delta_k + delta_{k+1}) - (eta_l
// + eta_{l+1}) its rounding, O(m^2 / l^2), was up to 300 times what the functions
// need there (6e-13 at L 2000).  h_k = eps_l s_l.
__global__ void k_rec_tables(int L, double* __restrict__ bp, double* __restrict__ be, double* __restrict__ gi,
                             double* __restrict__ he, double* __restrict__ re, double* __restrict__ ep) {
  const int m = blockIdx.y;
  const int K = (L - m) / 2 + 1;
  const double m2 = 4.0 * (double)m * m - 1.0;
  auto eta = [&](double l) { return m2 / (4.0 * (4.0 * l * l - 1.0)); };
  auto eps2 = [&](double l) { return (l - m) * (l + m) / (4.0 * l * l - 1.0); };
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < K; k += gridDim.x * blockDim.x) {
    const double l = m + 2.0 * k + 1.0;
    const double e0 = eps2(l - 1.0), e1 = eps2(l), e2 = eps2(l + 1.0), e3 = eps2(l + 2.0);
    const double g0 = sqrt(e0 * e1), g1 = sqrt(e2 * e3);
    const double d0 = (eta(l) * 0.25 + eta(l - 1.0) * e1) / (0.25 + g0);
    const double d1 = (eta(l + 2.0) * 0.25 + eta(l + 1.0) * e3) / (0.25 + g1);
    // eta_{j-1} - eta_j
    auto deta = [&](double j) { return m2 / ((2.0 * j - 3.0) * (2.0 * j - 1.0) * (2.0 * j + 1.0)); };
    const double r0 = sqrt(e0), r1 = sqrt(e1), r2 = sqrt(e2), r3 = sqrt(e3);
    const double s0 = deta(l) / (r1 + r0), s2 = deta(l + 2.0) / (r3 + r2);
    const int64_t o = krow(L, m) + k;
    bp[o] = (eta(l) + eta(l + 1.0)) + (d0 + d1);
    be[o] = r1 * s0 - r2 * s2;
    gi[o] = 1.0 / g1;
    he[o] = r1 * s0;
    re[o] = 1.0 / r1;
    // eps of l - 1 and l (row entries m + 2k, m + 2k + 1; the row ends at L + 1)
    double* er = ep + 4 + erow(L, m);
    er[2 * k] = r0;
    if (2 * k + 1 <= L + 1 - m) er[2 * k + 1] = r1;
    if (k == K - 1 && 2 * k + 2 <= L + 1 - m) er[2 * k + 2] = r2;
  }
  if (m == 0 && blockIdx.x == 0 && threadIdx.x < 4) ep[threadIdx.x] = threadIdx.x & 1 ? 0.0 : 1.0;
}

// Start of every (slot, m): the recurrence from lambda_mm with a power of two
// carried beside it, up to the first l with |lambda_l| >= thr; (q, d) as they
// were at the last multiple of 8 in k.  counts: triples from the first l with
// |lambda| >= thr (0) and >= thr_lo (1) on.
__global__ void k_start_table(const double* __restrict__ bp, const double* __restrict__ be,
                              const double* __restrict__ gi, const double* __restrict__ ep,
                              const double* __restrict__ zs, const double* __restrict__ ss,
                              const double* __restrict__ ya, const double* __restrict__ yc,
                              const double* __restrict__ pm_mant,
                              const int* __restrict__ pm_exp, int L, int nslots, int pol_pairs, int pol_tiles, int eq_pairs,
                              int npairs, double thr, double thr_lo, int* __restrict__ ks_out,
                              double2* __restrict__ st_out, unsigned long long* __restrict__ counts) {
  const int slot = blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  const bool polar = slot < 64 * pol_tiles;
  // the slot's ring pair (-1: none), and whether it is counted (once)
  const int e = slot - (nslots - 64);
  int p = polar ? slot : slot - 64 * pol_tiles + pol_pairs;
  if (polar ? p >= pol_pairs : e < 0 && p >= npairs - eq_pairs) p = -1;
  if (e >= 0) p = (e & 31) < eq_pairs ? npairs - eq_pairs + (e & 31) : -1;
  const bool counted = e < 32;
  unsigned long long n0 = 0, n1 = 0;
  if (slot < nslots) {
    int ksv = INT_MAX;
    double2 stv = make_double2(0.0, 0.0);
    if (p >= 0) {
      const double z = zs[slot], s = ss[slot], a = ya[slot], c = yc[slot];
      // lambda_mm = P_m sin^m(theta), carried as mantissa * 2^e
      double mant = pm_mant[m];
      long e = pm_exp[m];
      if (m > 0) {
        // powers of two doubles: squaring one would add up m / 2 of its roundings
        struct Num {
          double h, l;
          long e;
        };
        auto norm = [](double h, double l, long e) {
          int t;
          const double f = frexp(h, &t);
          return Num{f, ldexp(l, -t), e + t};
        };
        auto mul = [&](const Num& u, const Num& v) {
#pragma clang fp contract(off)
          const double q = u.h * v.h, r = fma(u.h, v.h, -q) + (u.h * v.l + u.l * v.h), h = q + r;
          return norm(h, r - (h - q), u.e + v.e);
        };
        Num base = norm(s, 0.0, 0), r{1.0, 0.0, 0};
        for (int j = m; j; j >>= 1) {
          if (j & 1) r = mul(r, base);
          base = mul(base, base);
        }
        const Num v = norm(fma(mant, r.h, mant * r.l), 0.0, e + r.e);
        mant = v.h;
        e = v.e;
      }
      const double* b = (polar ? bp : be) + krow(L, m);
      const double* g = gi + krow(L, m);
      const double* ee = ep + 4 + erow(L, m);
      const int K = (L - m) / 2 + 1;
      double q = mant / ee[1], d = 0.0, qm = 0.0;  // q_k, d_k and the signed q_{k-1}
      double sq = 0.0, sd = 0.0;
      long se = 0;
      int lo_l = L + 1;
      for (int k = 0; k < K; ++k) {
        if ((k & 7) == 0) {
          sq = q;
          sd = d;
          se = e;
        }
        const double sg = polar || !(k & 1) ? 1.0 : -1.0;  // the equator form carries (-1)^k q_k
        const double le = fabs(ee[2 * k + 1] * (sg * q) + ee[2 * k] * qm), lo = fabs(z * q);
        const int l = m + 2 * k;
        if (lo_l > L && e > -2000) {
          if (ldexp(le, (int)e) >= thr_lo) lo_l = l;
          else if (l + 1 <= L && ldexp(lo, (int)e) >= thr_lo) lo_l = l + 1;
        }
        int hit = -1;
        if (e > -2000) {
          if (ldexp(le, (int)e) >= thr) hit = l;
          else if (l + 1 <= L && ldexp(lo, (int)e) >= thr) hit = l + 1;
        }
        if (hit >= 0) {
          ksv = k & ~7;
          stv = make_double2(ldexp(sq, (int)se), ldexp(sd, (int)se));
          n0 = counted ? (unsigned long long)(L - hit + 1) : 0;
          break;
        }
        qm = sg * q;
        d = fma(fma(-a, c, b[k]), q, d);
        q = fma(g[k], d, q);
        if (fabs(q) > 0x1p600) {
          q *= 0x1p-600;
          qm *= 0x1p-600;
          d *= 0x1p-600;
          e += 600;
        }
      }
      if (counted && lo_l <= L) n1 = (unsigned long long)(L - lo_l + 1);
    }
    ks_out[(size_t)m * nslots + slot] = ksv;
    st_out[(size_t)m * nslots + slot] = stv;
  }
  for (int off = 32; off > 0; off >>= 1) {
    n0 += __shfl_xor(n0, off, 64);
    n1 += __shfl_xor(n1, off, 64);
  }
  if ((threadIdx.x & 63) == 0 && (n0 | n1)) {
    atomicAdd(counts, n0);
    atomicAdd(counts + 1, n1);
  }
}

__global__ void k_fill(double* __restrict__ p, int64_t n, double v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

constexpr double kSkipThreshold = 0x1p-100;  // a lane starts at most 15 l before |lambda| reaches this
constexpr double kFp64Normal = 0x1p-1022;    // smallest normal float64
constexpr int kTabPad = 64;                  // table words read past the last row (values unused)

ShtPlan& get_plan(crs_grid g, int lmax, hipStream_t s) {
  auto it = g->plans.find(lmax);
  if (it != g->plans.end()) return *it->second;
  auto plan = std::make_unique<ShtPlan>();
  const int L = lmax;
  plan->lmax = L;
  plan->npairs = (g->nring + 1) / 2;
  plan->nslots = g->nslots;
  // P_m = lambda_00 prod_{k<=m} sqrt((2k+1)/(2k)) as mantissa/exponent
  std::vector<double> pmm(L + 1);
  std::vector<int> pme(L + 1);
  {
    int e;
    double mant = std::frexp(1.0 / std::sqrt(4.0 * M_PI), &e);
    long ee = e;
    pmm[0] = mant;
    pme[0] = (int)ee;
    for (int m = 1; m <= L; ++m) {
      mant *= std::sqrt((2.0 * m + 1.0) / (2.0 * m));
      int t;
      mant = std::frexp(mant, &t);
      ee += t;
      pmm[m] = mant;
      pme[m] = (int)ee;
    }
  }
  const int64_t nk = krow(L, L) + 1 + kTabPad, ne = 4 + erow(L, L) + 2 + kTabPad;
  for (auto* t : {&plan->bp, &plan->be, &plan->gi, &plan->he, &plan->re}) {
    t->alloc((size_t)nk);
    hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, s, t->p + nk - kTabPad, (int64_t)kTabPad, 0.0);
  }
  plan->ep.alloc((size_t)ne);
  hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, s, plan->ep.p + ne - kTabPad, (int64_t)kTabPad, 0.0);
  hipLaunchKernelGGL(k_rec_tables, dim3((L / 2 + 256) / 256, L + 1), dim3(256), 0, s, L, plan->bp.p, plan->be.p,
                     plan->gi.p, plan->he.p, plan->re.p, plan->ep.p);
  CRS_HIP(hipGetLastError());
  DevBuf<double> dpm;
  DevBuf<int> dpe;
  DevBuf<unsigned long long> dcnt;
  unsigned long long cnt[2] = {0, 0};
  dpm.upload(pmm, s);
  dpe.upload(pme, s);
  dcnt.upload(cnt, 2, s);
  plan->ks.alloc((size_t)(L + 1) * plan->nslots);
  plan->st.alloc((size_t)(L + 1) * plan->nslots);
  hipLaunchKernelGGL(k_start_table, dim3((plan->nslots + 127) / 128, L + 1), dim3(128), 0, s, plan->bp.p, plan->be.p,
                     plan->gi.p, plan->ep.p, g->d_zs.p, g->d_ss.p, g->d_ya.p, g->d_yc.p, dpm.p, dpe.p, L, plan->nslots,
                     g->pol_pairs, g->pol_tiles, g->eq_pairs, plan->npairs, kSkipThreshold, kFp64Normal, plan->ks.p, plan->st.p,
                     dcnt.p);
  CRS_HIP(hipGetLastError());
  CRS_HIP(hipMemcpyAsync(cnt, dcnt.p, sizeof(cnt), hipMemcpyDeviceToHost, s));
  CRS_HIP(hipStreamSynchronize(s));
  plan->eff_triples = (int64_t)cnt[0];
  plan->fp64_triples = (int64_t)cnt[1];
  plan->nominal_triples = (int64_t)plan->npairs * ((int64_t)(L + 1) * (L + 2) / 2);
  auto& ref = *plan;
  g->plans[lmax] = std::move(plan);
  return ref;
}

}  // namespace crs

using namespace crs;

extern "C" {

int crs_grid_healpix(int nside, crs_grid* out) {
  return guarded([&] {
    CRS_CHECK(out != nullptr, CRS_EINVAL, "out is NULL");
    CRS_CHECK(nside >= 1, CRS_EINVAL, "nside must be >= 1");
    CRS_CHECK(nside <= 2048, CRS_EUNSUPPORTED, "nside above 2048 is not supported");
    auto g = std::make_unique<crs_grid_s>();
    CRS_HIP(hipGetDevice(&g->device));
    build_healpix(g.get(), nside);
    grid_finalize(g.get(), nullptr);
    *out = g.release();
    return CRS_OK;
  });
}

int crs_grid_gauss_legendre(int nrings, int nphi, crs_grid* out) {
  return guarded([&] {
    CRS_CHECK(out != nullptr, CRS_EINVAL, "out is NULL");
    CRS_CHECK(nrings >= 1 && nphi >= 1, CRS_EINVAL, "nrings and nphi must be >= 1");
    CRS_CHECK(nphi <= kMaxRing, CRS_EUNSUPPORTED, "nphi above 8192 is not supported");
    // an odd ring is transformed at full length: above 4096 pixels its length
    // must be 7-smooth (Bluestein's convolution would exceed 8192 points)
    if (nphi % 2 == 1 && nphi > kMaxRing / 2) {
      int n = nphi;
      for (int p : {3, 5, 7})
        while (n % p == 0) n /= p;
      CRS_CHECK(n == 1, CRS_EUNSUPPORTED, "odd nphi above 4096 must have no prime factor above 7");
    }
    auto g = std::make_unique<crs_grid_s>();
    CRS_HIP(hipGetDevice(&g->device));
    build_gl(g.get(), nrings, nphi);
    grid_finalize(g.get(), nullptr);
    *out = g.release();
    return CRS_OK;
  });
}

int crs_grid_info(crs_grid g, int* nrings, int64_t* npix) {
  return guarded([&] {
    CRS_CHECK(g != nullptr, CRS_EINVAL, "grid is NULL");
    if (nrings) *nrings = g->nring;
    if (npix) *npix = g->npix;
    return CRS_OK;
  });
}

int crs_grid_pixel_centres(crs_grid g, double* z, double* phi) {
  return guarded([&] {
    CRS_CHECK(g != nullptr, CRS_EINVAL, "grid is NULL");
    CRS_CHECK(z != nullptr && phi != nullptr, CRS_EINVAL, "z or phi is NULL");
    for (int r = 0; r < g->nring; ++r) {
      int n = g->nphi[r];
      for (int j = 0; j < n; ++j) {
        z[g->offset[r] + j] = g->z[r];
        // phi = pi * (num/den + 2 j / n)
        double x = (double)g->phi0_num[r] / g->phi0_den[r] + 2.0 * j / n;
        phi[g->offset[r] + j] = M_PI * x;
      }
    }
    return CRS_OK;
  });
}

int crs_grid_weights(crs_grid g, double* w) {
  return guarded([&] {
    CRS_CHECK(g != nullptr, CRS_EINVAL, "grid is NULL");
    CRS_CHECK(w != nullptr, CRS_EINVAL, "w is NULL");
    for (int r = 0; r < g->nring; ++r)
      for (int j = 0; j < g->nphi[r]; ++j) w[g->offset[r] + j] = g->ringw[r];
    return CRS_OK;
  });
}

int crs_grid_destroy(crs_grid g) {
  return guarded([&] {
    delete g;
    return CRS_OK;
  });
}

}  // extern "C"
