// Internal declarations of the crsolve HIP library (gfx950, float64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <functional>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../../include/crsolve.h"

namespace crs {

// ---------------------------------------------------------------- errors
struct Error {
  int code;
  std::string msg;
};
void set_error(int code, const std::string& msg);
int fail(int code, const std::string& msg);  // sets and returns code

#define CRS_HIP(call)                                                              \
  do {                                                                             \
    hipError_t e_ = (call);                                                        \
    if (e_ != hipSuccess)                                                          \
      throw ::crs::Error{CRS_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)}; \
  } while (0)

#define CRS_CHECK(cond, code, msg)                          \
  do {                                                      \
    if (!(cond)) throw ::crs::Error{(code), (msg)};         \
  } while (0)

// Runs f() and turns exceptions into status codes.
template <class F>
int guarded(F&& f) {
  try {
    return f();
  } catch (const Error& e) {
    return fail(e.code, e.msg);
  } catch (const std::bad_alloc&) {
    return fail(CRS_ENOMEM, "host allocation failed");
  } catch (const std::exception& e) {
    return fail(CRS_EINVAL, e.what());
  }
}

// Device buffer owned by a handle.
template <class T>
struct DevBuf {
  T* p = nullptr;
  size_t n = 0;
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  DevBuf(DevBuf&& o) noexcept : p(o.p), n(o.n) {
    o.p = nullptr;
    o.n = 0;
  }
  DevBuf& operator=(DevBuf&& o) noexcept {
    if (this != &o) {
      release();
      p = o.p;
      n = o.n;
      o.p = nullptr;
      o.n = 0;
    }
    return *this;
  }
  ~DevBuf() { release(); }
  void release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    n = 0;
  }
  void alloc(size_t count) {
    if (count <= n && p) return;
    release();
    if (count == 0) return;
    hipError_t e = hipMalloc(&p, count * sizeof(T));
    if (e != hipSuccess) {
      p = nullptr;
      throw Error{CRS_ENOMEM, "hipMalloc of " + std::to_string(count * sizeof(T)) + " bytes failed"};
    }
    n = count;
  }
  void upload(const T* host, size_t count, hipStream_t s) {
    alloc(count);
    if (count) CRS_HIP(hipMemcpyAsync(p, host, count * sizeof(T), hipMemcpyHostToDevice, s));
  }
  void upload(const std::vector<T>& v, hipStream_t s) { upload(v.data(), v.size(), s); }
};

constexpr int kMaxRing = 8192;   // pixels per ring (the FFT stays LDS resident)
constexpr int kBlueMax = 8192;   // longest Bluestein convolution (power of two)
constexpr size_t kMaxLds = 160 * 1024;  // LDS bytes one workgroup may use (gfx950)

// ---------------------------------------------------------------- grids
// Per-(grid, lmax) Legendre plan: start table and recurrence tables.  Ring
// pairs sit in slots in tiles of 64 (grid.hip): the polar ones first, padded
// to whole tiles, then the others, the last (up to 32) twice in a tile of their own.
struct ShtPlan {
  int lmax = 0;
  int npairs = 0, nslots = 0;
  int64_t eff_triples = 0;     // (ring pair, l, m) triples with |lambda| >= 2^-100
  int64_t fp64_triples = 0;    // triples whose |lambda| reaches the float64 normal range
  int64_t nominal_triples = 0; // npairs * (L+1)(L+2)/2
  DevBuf<double> bp, be, gi;   // rows of m (krow): recurrence coefficients b_k (polar, equator form), 1 / g_{k+1}
  DevBuf<double> he, re;       // rows of m (krow): h_k and 1 / eps_{m+2k+1} (equator form)
  DevBuf<double> ep;           // (1, 0, 1, 0), then rows of m (erow): eps_lm, l = m .. L + 1
  DevBuf<int> ks;              // [L+1][nslots]: first k evaluated, a multiple of 8 (INT_MAX = never)
  DevBuf<double2> st;          // [L+1][nslots]: (q, d) there
};
// Row of m in the triangles of the recurrence: K = (L - m) / 2 + 1 steps per m
// (sum over n = L - m + 1 .. L of n / 2 + 1), and L - m + 2 values of eps.
__host__ __device__ inline int64_t krow(int L, int m) {
  const int64_t n = L - m, a = L;
  return (a * a / 4 + a) - (n * n / 4 + n);
}
__host__ __device__ inline int64_t erow(int L, int m) { return (int64_t)m * (L + 2) - (int64_t)m * (m - 1) / 2; }

// Rings are launched in classes by FFT length tier (ring_tier_maxfft(t),
// ring_tier_threads(t) threads per block) and, from tier 2 up, by Bluestein
// or direct transform and whether the FFT has odd radices.
struct RingClass {
  std::vector<int> rings;
  bool blue = false;  // some ring of the class uses Bluestein's convolution
  bool odd = false;   // some FFT length of the class has odd radices
  int tier = 0;
  int xcap = 1;       // complex LDS words: ring data / convolution, with its padding,
  int wcap = 0;       //   FFT twiddles,
  int pcap = 0;       //   tables of the prime radices,
  int gcap = 0;       //   fold scratch (rings shorter than the block)
};
// tiers: FFT length <= 512 << t with 64 << t threads (eight points per thread;
// the longest FFT is a Bluestein convolution of kBlueMax words)
constexpr int kMaxRingClasses = 20;  // at most 4 per tier
inline int ring_tier_threads(int tier) { return 64 << tier; }
inline int ring_tier_maxfft(int tier) { return 512 << tier; }
// Rings of at most this many pixels are folded by that many threads of the
// block (below 1024: the partial sums share the LDS with the longest FFT).
__host__ __device__ constexpr int ring_short(int nt) { return nt < 512 ? nt : 512; }

// Radix of stage s of an FFT of length 2^e (e <= 13), 0 past the last.  The
// sequences read the same in both directions (the last stage of one transform
// and the first of the next then hold the same points, see ring.hip).
__host__ __device__ constexpr int pow2_radix(int e, int s) {
  constexpr int r[14][5] = {{0, 0, 0, 0, 0},   {2, 0, 0, 0, 0},  {4, 0, 0, 0, 0},    {8, 0, 0, 0, 0},   {4, 4, 0, 0, 0},
                            {4, 2, 4, 0, 0},   {8, 8, 0, 0, 0},  {4, 8, 4, 0, 0},    {8, 4, 8, 0, 0},   {8, 8, 8, 0, 0},
                            {8, 4, 4, 8, 0},  {8, 4, 2, 4, 8}, {8, 8, 8, 8, 0}, {8, 8, 2, 8, 8}};
  return s < 5 ? r[e][s] : 0;
}
__host__ __device__ constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

// One ring of a launch class: everything the kernel needs to know about it in
// one 128-byte record, read with the block index (one dependent load).
constexpr int kRingStages = 10;  // radices of an FFT length up to 8192
struct RingInfo {
  int ring, nphi;
  int num;              // phi0 = pi num / nphi, 0 or 1
  int fftn;             // FFT length: nphi / 2 (even), nphi (odd) or the Bluestein length
  int64_t offset;       // first pixel
  int64_t twoff;        // into tw
  int64_t bfoff;        // into bf, -1: direct transform
  int nfac;
  int fac[kRingStages];
  unsigned facm[kRingStages];  // per stage: FastDiv multiplier of the stride Ns before it
  int pad;
};
static_assert(sizeof(RingInfo) == 128, "one record per 128 bytes");

// Workspace of the public transforms (sht_synth / sht_adjoint).
struct GridWork {
  DevBuf<double2> phase;
  DevBuf<double> vpart;
};

}  // namespace crs

struct crs_grid_s {
  int kind = 0;  // 0 HEALPix, 1 Gauss-Legendre
  int nside = 0, nring = 0, nphi_gl = 0;
  int64_t npix = 0;
  std::vector<double> z, sint, ringw;
  std::vector<int> nphi, phi0_num, phi0_den;  // phi0 = pi * num / den
  std::vector<int64_t> offset;
  // device ring tables
  crs::DevBuf<double2> d_bf;      // Bluestein filter spectra per distinct length
  crs::DevBuf<double2> d_tw2;     // exp(-2 pi i t / kBlueMax), t < kBlueMax (power-of-two FFTs)
  // ring pair slots (see slot_layout): polar pairs and tiles, pairs of the
  // equator's tile, all slots; per slot z of the north ring, sin(theta), and
  // ya, yc with ya yc = sin^2 (polar) or z^2
  int pol_pairs = 0, pol_tiles = 0, eq_pairs = 0, nslots = 0;
  crs::DevBuf<double> d_zs, d_ss, d_ya, d_yc;
  crs::DevBuf<double2> d_tw;      // twiddles exp(-2 pi i t / N) per distinct N
  std::vector<crs::RingClass> ring_classes;  // by (tier, Bluestein, odd radix)
  std::vector<crs::DevBuf<crs::RingInfo>> d_ring_class;
  std::vector<int> ring_small_order;         // classes by ring count, ascending
  std::vector<crs::RingClass> ring_prefix;   // [k]: the first k + 1 of them merged
  std::vector<crs::DevBuf<crs::RingInfo>> d_ring_prefix;
  std::map<int, std::unique_ptr<crs::ShtPlan>> plans;
  std::unique_ptr<crs::GridWork> work;
  int device = 0;
};

namespace crs {

ShtPlan& get_plan(crs_grid g, int lmax, hipStream_t s);

// ------------------------------------------------------------ kernels API
// Legendre stage on plain harmonic vectors (legendre.hip).
// Optional skip of finished systems: map j is skipped when
// act[kActStride * mapsys[j]] == 0 (both NULL: nothing is skipped).
constexpr int kActStride = 8;
struct MapSkip {
  const int* mapsys = nullptr;
  const double* act = nullptr;
  __device__ __forceinline__ bool off(int map) const {
    return act != nullptr && act[kActStride * mapsys[map]] == 0.0;
  }
};

struct LegArgs {
  const double *bp, *be, *gi, *he, *re, *ep;  // ShtPlan tables
  const int* ks;
  const double2* st;
  const double *zs, *ya, *yc;       // per slot
  int lmax, npairs, nring, nslots, pol_tiles, pol_pairs, eq_pairs;
  MapSkip skip;
  // optional compaction: the launch's map slots s < *mcount are the maps
  // mlist[s] (ascending), the slots past *mcount are empty; without it slot
  // s is map s.  Both device pointers, set together.
  const int* mlist = nullptr;
  const int* mcount = nullptr;
};
// Tiles of 64 ring pairs per wave of the Legendre kernels for a (grid layout,
// L, maps) shape.  leg_choice gives the autotuned choice for the shape if one
// was recorded (leg_autotune), else the measured default rules; the
// environment variables CRS_LEG_TS and CRS_LEG_TA override either (tuning and
// tests).  A caller takes the choice once and passes the same one to
// leg_adjoint_tiles and the launches.
struct LegChoice {
  int syn_t = 1, adj_t = 1;
};
LegChoice leg_choice(crs_grid g, int lmax, int nmaps);
// Times every valid variant of both transforms on the given buffers (their
// contents are overwritten; vpart is allocated internally) and records the
// fastest per transform for the shape.  Returns the recorded choice.
LegChoice leg_autotune(const LegArgs& a, int nmaps, double* uhat, double2* phase, hipStream_t s);
// phase: [nmaps][nring][L+1] double2 (cos, sin parts)
void launch_leg_synth(const LegChoice& c, const LegArgs& a, int nmaps, const double* u, int64_t ustride,
                      double2* phase, int64_t pstride, hipStream_t s);
// Adjoint: one partial vector per tile group and map, as many groups as
// returned here for the same choice and square flag as the launch.  The first
// group's goes to v0 + map v0stride (the result's own place: only the others
// need scratch, and launch_tile_sum adds them to it), the following ones to
// v + i tstride + map vstride.  g0, ng: the launch's groups (all: 0, the count;
// with g0 > 0 group g0 + i goes to v + i tstride).
struct AdjDst {
  double* v0;
  int64_t v0stride;
  double* v;
  int64_t vstride, tstride;
  int g0, ng;
};
// all groups to v[group][map][nalm]
inline AdjDst adj_dst(double* v, int64_t nalm, int nmaps, int ng) {
  const int64_t t = (int64_t)nmaps * nalm;
  return {v, nalm, v + t, nalm, t, 0, ng};
}
int leg_adjoint_tiles(const LegChoice& c, crs_grid g, bool square);
// Partial vectors per map that an adjoint with little scratch keeps beside its
// result: one per 128 ring pairs, or one per tile group after the first where that
// is fewer, at the tiles per wave that the waves alone would give (the groups
// may be more: small grids, whose tiles are padded, and shapes that run fewer tiles
// per wave than their waves allow).
int leg_adjoint_parts(const LegChoice& c, crs_grid g, int L, int nmaps);
void launch_leg_adjoint(const LegChoice& c, const LegArgs& a, int nmaps, const double2* phase, int64_t pstride,
                        const AdjDst& dst, bool square, hipStream_t s);

// Ring FFT stage.
enum RingMode { RING_SYNTH = 0, RING_ADJOINT = 1, RING_ROUNDTRIP = 2, RING_DIAG = 3 };
struct RingArgs {
  const RingInfo* info;  // records of the launch (set by launch_ring per class)
  const double2* tw;    // per distinct Nphi: exp(-i pi t / Nphi), t < 2 Nphi
  const double2* bf;    // per Bluestein length: filter spectrum [fftn], then the chirp [n0]
  const double2* tw2;
  int lmax;
  int xcap, wcap, pcap;  // LDS words per launch class (RingClass)
  MapSkip skip;
};
// maps j = 0..nmaps-1 use weight weights[j / maps_per_weight] (RING_ROUNDTRIP).
void launch_ring(crs_grid g, int lmax, RingMode mode, int nmaps, double2* phase, int64_t pstride,
                 const double* map_in, double* map_out, int64_t mstride,
                 const double* const* weights, int maps_per_weight, hipStream_t s,
                 MapSkip skip = MapSkip{});

// out[map] += sum_t in[t][map] elementwise over the packed alm index, in order of t.
void launch_tile_sum(int64_t nalm, int nmaps, const double* in, int64_t istride, int ntiles, int64_t tstride,
                     double* out, int64_t ostride, hipStream_t s);

// Profiling hooks (no-ops unless profiling is on).  A scope brackets its
// launches with HIP events on the stream.  On a stream that is being
// captured into a graph the event records become graph nodes; the pairs are
// then handed to the graph's owner (prof_take_captured), which accounts them
// after every replay (prof_account) and frees them (prof_release).
// Work of a launch, three ways: the Legendre flops counted over the (ring
// pair, l, m) triples whose |lambda| reaches the float64 normal range (w[0],
// the headline count), over all triples (w[1], nominal) and over the triples
// the kernels evaluate (w[2], |lambda| >= 2^-100); ring launches carry their
// algorithmic bytes in all three.
struct Work3 {
  double w[3] = {0.0, 0.0, 0.0};
};
struct ProfRecord {
  int family;
  Work3 work;
  int tag;  // owner's label (a group index) for replay-time work, -1: fixed
  hipEvent_t e0, e1;
};
struct ProfScope {
  int family;
  Work3 work;
  int tag;
  hipStream_t s;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  bool captured = false;
  ProfScope(int fam, const Work3& w, hipStream_t st, int tag = -1);
  ~ProfScope();
};
enum { FAM_LEG_SYNTH = 0, FAM_LEG_ADJ = 1, FAM_RING = 2, FAM_COUNT = 3 };
bool prof_enabled();
void prof_disable_in_graphs();  // if a graph cannot hold event records
std::vector<ProfRecord> prof_take_captured();
// Accounts one replay; work (optional) gives each record's work for this
// replay (records of finished systems' maps do less), else the recorded work.
void prof_account(const std::vector<ProfRecord>& recs,
                  const std::function<Work3(const ProfRecord&)>& work = nullptr);
void prof_release(std::vector<ProfRecord>& recs);
Work3 leg_work(const ShtPlan& p, int nmaps);
Work3 bytes_work(double bytes);

}  // namespace crs
