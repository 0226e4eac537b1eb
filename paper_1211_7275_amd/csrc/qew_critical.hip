// qew_critical.hip -- critical force f_c^s and critical configuration u_c^s of
// samples periodic in u (Sec. III A of arXiv:1211.7275), on the device.
//
// The critical configuration is the pinned solution of
//   c d2u/dx2 + F_p(u, x) + f = 0                       (Sec. III A)
// with the largest f.  The Middleton theorems (no passing) make it reachable
// without integrating Eq. (1) in time:
//   - from a configuration whose forces are all >= 0, moving any site forward
//     to the first zero of its own force (neighbours held) keeps every force
//     >= 0 (the neighbours' forces only grow) and never passes a pinned
//     configuration that lies ahead (at a site of a pinned configuration ahead,
//     with neighbours behind theirs, the force is <= 0, so the first zero comes
//     no later).  Repeating such moves therefore climbs to the leftmost pinned
//     configuration ahead, if one exists;
//   - in a sample periodic in u the translates by M of a pinned configuration
//     are pinned too, so a line that advances by M everywhere has passed none:
//     there is no pinned configuration at that drive.
// Each workgroup owns one sample and runs a bisection on f: a trial drive is
// "pinned" when the forward moves converge (every |force| <= tol_force) and
// "depinned" when every site has advanced by M from the trial's start (the
// last pinned configuration), all in LDS within one launch.  The moves are
// applied to the even and then the odd sites (never two neighbours at once).
// The very first configuration (at the lower drive) is relaxed by moving each
// site to the nearest zero of its own force in the direction of the force,
// which lowers the line's energy at every move.
//
// Only the Catmull-Rom kinds (continuous forces) are handled; the local
// force of a site is a polynomial in its offset within a cell, and its first
// zero is found on the monotone pieces between the polynomial's turning
// points by Newton steps kept inside a shrinking bracket.
#include "qew_device.hpp"
#include "qew_internal.hpp"

#include <type_traits>

namespace qew {

namespace {

// Threads of a workgroup: one per pair of sites, at most this many.
constexpr int kCritMaxBlock = 1024;
constexpr int kMaxCells = 64;        // cells one move may cross (then it stops at the cell edge)
constexpr int kBisect = 64;          // bound on the bracketed Newton steps of one zero
constexpr int kCheckEvery = 4;       // sweeps between convergence checks

// Columns of the node ring: the even sites, the odd sites, and (odd L) the
// last site, each class padded to whole sets of LDS banks, so that a wave's
// lanes fall on different banks whatever slots they address.
__host__ __device__ __forceinline__ int ring_half(int L) { return ((L >> 1) + 31) & ~31; }
__host__ __device__ __forceinline__ int ring_row(int L) { return 2 * ring_half(L) + ((L & 1) ? 32 : 0); }

// Local force of site j as a cubic in the offset s of cell n:
//   g(s) = A - 2c (n + s) + F_p(n + s),  A = c (u_{j-1} + u_{j+1}) + f.
// The random-bond kind's is a quadratic (b3 = 0): two operations less in every
// dependent chain below.
template <int KIND>
struct Cubic {
  double b0, b1, b2, b3;
  __device__ double at(double s) const {
    if constexpr (KIND == kRB) return b0 + s * (b1 + s * b2);
    else return b0 + s * (b1 + s * (b2 + s * b3));
  }
  __device__ double slope(double s) const {
    if constexpr (KIND == kRB) return b1 + s * (2.0 * b2);
    else return b1 + s * (2.0 * b2 + s * (3.0 * b3));
  }
};

constexpr double kEps = 2.220446049250313e-16;

// 1 / b (b != 0) to about an ulp: the hardware reciprocal refined by one
// Newton step, and a / b from it.  The quotients below steer bracketed searches
// and place turning points, where an ulp more or less changes nothing, and the
// full IEEE division sequence is a long dependent chain on the critical path.
__device__ __forceinline__ double recip(double b) {
  const double r = __builtin_amdgcn_rcp(b);
  return fma(fma(-b, r, 1.0), r, r);
}
__device__ __forceinline__ double quot(double a, double b) { return a * recip(b); }

// A point next to the zero of g on [lo, hi], where g is monotone with
// g(lo) = glo > 0 >= g(hi) = ghi (up) or glo >= 0 > ghi (down).  The answer
// lies on the near side of the zero -- g > 0 (up) or g < 0 (down) -- so a move
// there never passes it.  Newton steps are taken from the end with the
// smaller |g| and kept inside the bracket (a step that leaves it becomes the
// midpoint).  When that end is the far-side one and already within `tol` of
// zero, the next point is placed as far on the near side of the Newton
// estimate of the zero as the end lies on the other side, so that a function
// that keeps the Newton steps on the far side still yields a near-side point.
// Stops once the near-side end has |g| <= tol or the bracket is a few ulp
// wide.
//
// A single wave issues dependent FP64 operations back to back (4 cycles each,
// measured), so the loop is written for few instructions, not for short chains:
// its direction is fixed at compile time.
template <bool UP, int KIND>
__device__ __forceinline__ double bracketed_zero(const Cubic<KIND>& g, double lo, double hi, double glo,
                                                 double ghi, double tol) {
  for (int it = 0; it < kBisect; ++it) {
    if (fabs(UP ? glo : ghi) <= tol || hi - lo <= 4.0 * kEps) break;
    const bool from_lo = fabs(glo) <= fabs(ghi);
    const double e = from_lo ? lo : hi;
    const double ge = from_lo ? glo : ghi;
    // a zero slope gives a NaN here, which the test of the bracket sends to the midpoint
    double x = e - quot(ge, g.slope(e));
    if (from_lo != UP && fabs(ge) <= tol) {
      const double off = fmax(fabs(e - x), 4.0 * kEps);
      x = UP ? x - off : x + off;
    }
    x = (x > lo && x < hi) ? x : 0.5 * (lo + hi);
    const double gx = g.at(x);
    const bool to_lo = UP ? (gx > 0.0) : (gx >= 0.0);
    lo = to_lo ? x : lo;
    glo = to_lo ? gx : glo;
    hi = to_lo ? hi : x;
    ghi = to_lo ? ghi : gx;
  }
  return UP ? lo : hi;
}

// The strength-scaled nodes n-1 .. n+2 of site j: the Catmull-Rom window of
// cell n.  The random-bond kind makes them one at a time: four FP64
// Box-Muller transforms at once would hold more registers than 1024 threads
// per workgroup leave (measured: the sequential form is faster there, the
// interleaved one for the uniform nodes).
template <int KIND>
__device__ void node_window(uint32_t j, int32_t n, uint32_t id, const CritParams& q, double p[4]) {
  if constexpr (KIND == kRF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = q.strength * node_f64<KIND>(j, n - 1 + i, id, q.k0, q.k1, q.period);
  } else {
#pragma unroll 1
    for (int i = 0; i < 4; ++i) p[i] = q.strength * node_f64<KIND>(j, n - 1 + i, id, q.k0, q.k1, q.period);
  }
}

// Local force in cell n from its window p.
template <int KIND>
__device__ __forceinline__ Cubic<KIND> cubic_of(const double p[4], int32_t n, double A, double c) {
  // Catmull-Rom in s: value = 1/2 [2 p1 + d1 s + d2 s^2 + d3 s^3]
  const double d1 = p[2] - p[0];
  const double d2 = 2.0 * p[0] - 5.0 * p[1] + 4.0 * p[2] - p[3];
  const double d3 = -p[0] + 3.0 * p[1] - 3.0 * p[2] + p[3];
  Cubic<KIND> g;
  const double lin = A - 2.0 * c * (double)n;
  if constexpr (KIND == kRF) {  // F_p = value
    g.b0 = lin + p[1];
    g.b1 = -2.0 * c + 0.5 * d1;
    g.b2 = 0.5 * d2;
    g.b3 = 0.5 * d3;
  } else {  // random bond: F_p = -d value / ds
    g.b0 = lin - 0.5 * d1;
    g.b1 = -2.0 * c - d2;
    g.b2 = -1.5 * d3;
    g.b3 = 0.0;
  }
  return g;
}

// Turning points of g (roots of g') strictly inside (lo, hi), ascending: `n` of
// them.  Written with selects: a branch costs the wave some ten instructions.
struct Turns {
  int n;
  double t0, t1;
};

template <int KIND>
__device__ __forceinline__ Turns turning_points(const Cubic<KIND>& g, double lo, double hi) {
  if constexpr (KIND == kRB) {
    const double b = 2.0 * g.b2;
    const double r = quot(-g.b1, b);  // b = 0: not a number or infinite, so not inside
    return Turns{(r > lo && r < hi) ? 1 : 0, r, r};
  } else {
    const double a = 3.0 * g.b3, b = 2.0 * g.b2, c = g.b1;
    const double disc = b * b - 4.0 * a * c;
    const bool two = disc > 0.0 && a != 0.0;
    const double q = -0.5 * (b + copysign(sqrt(disc), b));
    double r0 = quot(q, a);
    const double r1 = quot(c, q);
    bool is0 = two;
    const bool is1 = two && q != 0.0;
    if (__any(!two && !(disc < 0.0))) {  // rare: g' linear, or a double root
      if (!two) {
        const bool linear = a == 0.0;
        r0 = quot(linear ? -c : -b, linear ? b : 2.0 * a);
        is0 = linear ? b != 0.0 : disc == 0.0;
      }
    }
    const double x0 = is1 ? fmin(r0, r1) : r0, x1 = fmax(r0, r1);
    const bool in0 = is0 && x0 > lo && x0 < hi;
    const bool in1 = is1 && x1 > lo && x1 < hi;
    return Turns{(in0 ? 1 : 0) + (in1 ? 1 : 0), in0 ? x0 : x1, x1};
  }
}

// Where a move found its zero: the monotone piece [a, b] of the local force in
// its cell, with the values at its ends.
struct Piece {
  double a, b, ga, gb;
};

// First monotone piece of [s0, 1] on which g (g(s0) = g0 > 0) reaches 0.  The
// ends of all pieces are evaluated side by side.
template <int KIND>
__device__ __forceinline__ bool piece_up(const Cubic<KIND>& g, double s0, double g0, Piece& pc) {
  const Turns t = turning_points(g, s0, 1.0);
  const double e0 = t.n > 0 ? t.t0 : 1.0;
  const double v0 = g.at(e0), v2 = g.at(1.0);
  if constexpr (KIND == kRB) {  // at most one turning point
    const bool first = v0 <= 0.0;
    pc = Piece{first ? s0 : e0, first ? e0 : 1.0, first ? g0 : v0, first ? v0 : v2};
    return first || v2 <= 0.0;
  } else {
    const double e1 = t.n > 1 ? t.t1 : 1.0;
    const double v1 = g.at(e1);
    const bool first = v0 <= 0.0, second = !first && t.n >= 1 && v1 <= 0.0;
    pc = Piece{first ? s0 : (second ? e0 : e1), first ? e0 : (second ? e1 : 1.0),
               first ? g0 : (second ? v0 : v1), first ? v0 : (second ? v1 : v2)};
    return first || second || (t.n >= 2 && v2 <= 0.0);
  }
}

// Last monotone piece of [0, s0] (going down from s0) on which g (g(s0) = g0 < 0) reaches 0.
template <int KIND>
__device__ __forceinline__ bool piece_down(const Cubic<KIND>& g, double s0, double g0, Piece& pc) {
  const Turns t = turning_points(g, 0.0, s0);
  pc = Piece{t.n == 0 ? 0.0 : (t.n == 1 ? t.t0 : t.t1), s0, 0.0, g0};
  pc.ga = g.at(pc.a);
  for (int i = t.n; i > 0 && !(pc.ga >= 0.0); --i) {
    pc.b = pc.a;
    pc.gb = pc.ga;
    pc.a = (i == 2) ? t.t0 : 0.0;
    pc.ga = g.at(pc.a);
  }
  return pc.ga >= 0.0;
}

}  // namespace

// Node cache of the kernel (RING): the last kRing nodes of every site, node n
// in slot n mod kRing, in LDS.  A thread knows the range [lo, hi] its sites
// hold.  The window of a cell is 4 nodes, so 4 more fit ahead of it: whenever
// one lane of a wave has to make a node, every lane with room makes its own
// next one in the same pass, and most passes are saved (a pass costs the wave
// the same whether 1 or 64 lanes take part).
constexpr int kRing = 8;

// One workgroup per sample, one thread per pair of neighbouring sites (2t,
// 2t + 1), so every lane moves a site in both halves of a sweep.
//
// Bound by latency: a sweep is a chain of FP64 operations on one to sixteen
// waves of one CU, and a wave waits for its slowest lane.  The kernel
// therefore keeps the node windows (RING) instead of making the four nodes of
// a window for every visit, and a wave first walks the cells with all its
// lanes until each knows the piece that holds its zero, then takes the Newton
// steps of all lanes together, instead of one after the other cell by cell.
// Measured (windows made on each visit and the Newton steps inside the walk,
// then this form; the same sweeps and the same bits): 32 random-bond samples of
// 256 x 256 to 1e-3 202 -> 55 ms, 48 random-field samples of 63 x 64 to 1e-4
// 114 -> 81 ms.  What is left is instruction issue of one wave per SIMD: some
// 4.3 Newton steps of about 390 cycles and 1.3 (RF) to 3.5 (RB) cells of about
// 1300 cycles per half-sweep.
// LDS: u[L] (the trial), the ring, reduction flags.  The last pinned
// configuration (the trial's start) stays in registers with RING, else in LDS.
template <int KIND, bool RING, int BLOCK>
__global__ void __launch_bounds__(BLOCK)
    k_critical(CritParams q, const uint32_t* __restrict__ did, double* __restrict__ u_io,
               double* __restrict__ f_out, int64_t* __restrict__ st_out) {
  extern __shared__ double sh[];
  const int L = q.L;
  const int npairs = L >> 1;  // sites 2t and 2t + 1 for t < npairs; an odd L's last site is a third class
  const int half = ring_half(L);
  const int row = ring_row(L);
  double* u = sh;
  double* aux = sh + L;  // RING: [kRing][row] nodes; else v[L]
  int* red = reinterpret_cast<int*>(aux + (RING ? kRing * row : L));  // [2][kCritMaxBlock / 64] flags
  const int s = blockIdx.x;
  const int nt = blockDim.x;
  const int nw = nt >> 6;
  const uint32_t id = did[s];
  double* u_s = u_io + (int64_t)s * L;
  for (int j = threadIdx.x; j < L; j += nt) u[j] = u_s[j];
  __syncthreads();

  int64_t sweeps = 0;
  int status = 0;
  int parity = 0;
  // A site whose force is within tol_force / 4 of zero is left where it is,
  // and a move stops once the force left at the site is within tol_force / 64:
  // a converged line (every |force| <= tol_force) is reached without chasing
  // zeros to the last ulp.
  const double skip = 0.25 * q.tol_force;
  const double stop = q.tol_force * (1.0 / 64.0);
  // This thread's site of each class (even, odd, and an odd L's last): the range
  // of nodes it holds (empty at first) and, with RING, its place in the last
  // pinned configuration.  The classes take turns in (lo, hi, v), so that the code
  // of a phase exists once.
  int lo = 0, hi = -1, lo1 = 0, hi1 = -1, lo2 = 0, hi2 = -1;
  double v = 0.0, v1 = 0.0, v2 = 0.0;
  const int classes = (L & 1) ? 3 : 2;
  auto next_class = [&]() {
    const int l = lo, h = hi;
    const double w = v;
    lo = lo1;
    hi = hi1;
    v = v1;
    lo1 = classes == 3 ? lo2 : l;
    hi1 = classes == 3 ? hi2 : h;
    v1 = classes == 3 ? v2 : w;
    lo2 = l;
    hi2 = h;
    v2 = w;
  };
  // fn(site, its ring column) for this thread's sites of class c.
  auto each_of_class = [&](int c, auto&& fn) {
    const int count = c < 2 ? npairs : 1;
    for (int t = threadIdx.x; t < count; t += nt) fn(c < 2 ? 2 * t + c : L - 1, aux + c * half + t);
  };
  auto make_node = [&](int j, int32_t n) -> double {
    return q.strength * node_f64<KIND>((uint32_t)j, n, id, q.k0, q.k1, q.period);
  };
  // One pass of node making: the calling lanes with room above (their window's
  // cell is n) make node hi + 1.
  auto fill_up = [&](double* ring, int j, int32_t n, int& lo_c, int& hi_c) {
    if (hi_c < n + (kRing - 2)) {
      hi_c += 1;
      ring[(hi_c & (kRing - 1)) * row] = make_node(j, hi_c);
      if (lo_c < hi_c - (kRing - 1)) lo_c = hi_c - (kRing - 1);
    }
  };
  // The window n-1 .. n+2 of site j.
  auto window = [&](double* ring, int j, int32_t n, int& lo_c, int& hi_c, double p[4]) {
    if constexpr (RING) {
      if (lo_c > n - 1 || hi_c < n - 2) {  // nothing usable (start, or the line was put back)
        lo_c = n - 1;
        hi_c = n - 2;
      }
#pragma unroll 1
      for (int pass = 0; pass < 4; ++pass) {
        if (!__any(hi_c < n + 2)) break;
        fill_up(ring, j, n, lo_c, hi_c);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = ring[((n - 1 + i) & (kRing - 1)) * row];
    } else {
      node_window<KIND>((uint32_t)j, n, id, q, p);
    }
  };
  // Move of site j at drive f, neighbours held: forward to the first zero of its
  // force (FORWARD), or to the nearest one in the direction of its force.
  auto move = [&](auto forward, int j, double* ring, int& lo_c, int& hi_c, double f) {
    constexpr bool FORWARD = decltype(forward)::value;
    const double ul = u[j == 0 ? L - 1 : j - 1];
    const double ur = u[j == L - 1 ? 0 : j + 1];
    const double A = q.c * (ul + ur) + f;
    const double x = u[j];
    const double nf = floor(x);
    int32_t n = (int32_t)nf;
    double sx = x - nf;
    double p[4];
    window(ring, j, n, lo_c, hi_c, p);
    Cubic<KIND> g = cubic_of<KIND>(p, n, A, q.c);
    double g0 = g.at(sx);
    const int d = (FORWARD || g0 > 0.0) ? 1 : -1;
    const bool moves = FORWARD ? g0 > skip : fabs(g0) > skip;
    // Walk the cells: every lane still searching looks at one cell per trip.
    bool search = moves, found = false;
    Piece pc{0.0, 0.0, 0.0, 0.0};
    for (int cell = 0; cell < kMaxCells; ++cell) {
      if (!__any(search)) break;
      if (search) {
        if (cell > 0) {
          g = cubic_of<KIND>(p, n, A, q.c);
          g0 = g.at(sx);
        }
        if (FORWARD || d > 0) found = piece_up(g, sx, g0, pc);
        else found = piece_down(g, sx, g0, pc);
        search = !found;
        if (search) {  // no zero in the rest of the cell: on to the next one
          n += d;
          sx = d > 0 ? 0.0 : 1.0;
        }
      }
      if constexpr (RING) {
        if (__any(search && d > 0 && hi_c < n + 2)) fill_up(ring, j, n, lo_c, hi_c);
        if (!FORWARD && search && d < 0 && lo_c > n - 1) {
          lo_c = n - 1;
          if (hi_c > lo_c + (kRing - 1)) hi_c = lo_c + (kRing - 1);
          ring[(lo_c & (kRing - 1)) * row] = make_node(j, lo_c);
        }
        if (search) {
          if (FORWARD || d > 0) {
            p[0] = p[1];
            p[1] = p[2];
            p[2] = p[3];
            p[3] = ring[((n + 2) & (kRing - 1)) * row];
          } else {
            p[3] = p[2];
            p[2] = p[1];
            p[1] = p[0];
            p[0] = ring[((n - 1) & (kRing - 1)) * row];
          }
        }
      } else if (search) {
        const double nd = make_node(j, d > 0 ? n + 2 : n - 1);
        if (FORWARD || d > 0) {
          p[0] = p[1];
          p[1] = p[2];
          p[2] = p[3];
          p[3] = nd;
        } else {
          p[3] = p[2];
          p[2] = p[1];
          p[1] = p[0];
          p[0] = nd;
        }
      }
    }
    if (moves) {
      // a move past kMaxCells cells is continued in the next sweep
      if (found) {
        if (FORWARD || d > 0) sx = bracketed_zero<true>(g, pc.a, pc.b, pc.ga, pc.gb, stop);
        else sx = bracketed_zero<false>(g, pc.a, pc.b, pc.ga, pc.gb, stop);
      }
      u[j] = (double)n + sx;
    }
  };
  // One sweep at drive f: the even sites, then the odd ones (the last site
  // alone when L is odd, since it neighbours site 0).
  auto sweep = [&](auto forward, double f) {
#pragma unroll 1
    for (int c = 0; c < classes; ++c) {
      each_of_class(c, [&](int j, double* ring) { move(forward, j, ring, lo, hi, f); });
      next_class();
      __syncthreads();
    }
  };
  // Whether every |force| <= tol_force (bit 0) and every site has advanced
  // by M over the start v (bit 1).
  auto check = [&](double f, bool forward) -> int {
    bool pinned = true, passed = forward;
#pragma unroll 1
    for (int c = 0; c < classes; ++c) {
      each_of_class(c, [&](int j, double* ring) {
        const double x = u[j];
        const double nf = floor(x);
        double p[4];
        window(ring, j, (int32_t)nf, lo, hi, p);
        const double A = q.c * (u[j == 0 ? L - 1 : j - 1] + u[j == L - 1 ? 0 : j + 1]) + f;
        const Cubic<KIND> g = cubic_of<KIND>(p, (int32_t)nf, A, q.c);
        pinned &= fabs(g.at(x - nf)) <= q.tol_force;
        if (forward) passed &= x - (RING ? v : aux[j]) >= (double)q.period;
      });
      next_class();
    }
    int* flags = red + parity * (kCritMaxBlock / 64);
    parity ^= 1;  // the next check writes the other half, so one barrier is enough
    const int mine = (__all(pinned) ? 1 : 0) | (__all(passed) ? 2 : 0);
    if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = mine;
    __syncthreads();
    int all = 3;
    for (int i = 0; i < nw; ++i) all &= flags[i];
    return all;
  };
  // Relax at drive f from the configuration in u; returns 0 pinned, 1
  // depinned (advanced by M over v everywhere), 2 undecided.
  auto relax = [&](auto forward, double f) -> int {
    for (int64_t k = 0; k < q.max_sweeps; k += kCheckEvery) {
#pragma unroll 1
      for (int i = 0; i < kCheckEvery; ++i) sweep(forward, f);
      sweeps += kCheckEvery;
      const int all = check(f, decltype(forward)::value);
      if (all & 1) return 0;
      if (all & 2) return 1;
    }
    return 2;
  };
  // fn(j, v_j) for this thread's sites: the trial's start v is kept (v = u) or
  // put back (u = v).
  auto each_site = [&](auto&& fn) {
    if constexpr (RING) {
      for (int c = 0; c < classes; ++c) {
        each_of_class(c, [&](int j, double*) { fn(j, v); });
        next_class();
      }
    } else {
      for (int j = threadIdx.x; j < L; j += nt) fn(j, aux[j]);
    }
  };
  auto keep = [&]() { each_site([&](int j, double& w) { w = u[j]; }); };
  auto put_back = [&]() { each_site([&](int j, double& w) { u[j] = w; }); };

  double f_lo = q.f_lo, f_hi = q.f_hi;
  int r = relax(std::false_type{}, f_lo);
  if (r != 0) {
    status = 1;  // no pinned configuration reached at the lower drive
  } else {
    keep();
    __syncthreads();
    for (int round = 0; round < q.max_rounds && f_hi - f_lo >= q.tol_f; ++round) {
      const double f_mid = 0.5 * (f_lo + f_hi);
      r = relax(std::true_type{}, f_mid);
      if (r == 0) {
        f_lo = f_mid;
        keep();
      } else if (r == 1) {
        f_hi = f_mid;
        put_back();
      } else {
        status = 2;  // a trial undecided within max_sweeps
        break;
      }
      __syncthreads();
    }
    if (status == 0 && f_hi - f_lo >= q.tol_f) status = 3;  // out of rounds
  }
  __syncthreads();
  if (status == 0) put_back();  // the last pinned configuration
  __syncthreads();
  for (int j = threadIdx.x; j < L; j += nt) u_s[j] = u[j];
  if (threadIdx.x == 0) {
    f_out[2 * s] = f_lo;
    f_out[2 * s + 1] = f_hi;
    st_out[2 * s] = status;
    st_out[2 * s + 1] = sweeps;
  }
}

// The ring needs one pair of sites per thread and kRing nodes per site in LDS.
static bool critical_ring(int L) { return L <= 2 * kCritMaxBlock; }

size_t critical_lds_bytes(int L) {
  const size_t flags = 2 * (kCritMaxBlock / 64) * sizeof(int);
  return ((size_t)L + (critical_ring(L) ? (size_t)kRing * ring_row(L) : (size_t)L)) * sizeof(double) + flags;
}

// Threads per workgroup: one per pair of sites, whole waves, at most kCritMaxBlock.
static int critical_block(int L) {
  const int pairs = L >> 1;
  const int t = ((pairs + 63) / 64) * 64;
  return t < 64 ? 64 : (t > kCritMaxBlock ? kCritMaxBlock : t);
}

hipError_t launch_critical(int kind, const CritParams& q, int n_samples, const uint32_t* did, double* u_io,
                           double* f_out, int64_t* st_out, hipStream_t st) {
  const size_t lds = critical_lds_bytes(q.L);
  const bool ring = critical_ring(q.L);
  auto go = [&](auto kernel) -> hipError_t {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(n_samples), dim3(critical_block(q.L)), lds, st, q, did, u_io, f_out, st_out);
    return hipGetLastError();
  };
  // The random-bond kernel has a form for at most 512 threads, whose FP64
  // Box-Muller transforms then fit the registers without spills.
  if (kind == kRF) return ring ? go(&k_critical<kRF, true, kCritMaxBlock>) : go(&k_critical<kRF, false, kCritMaxBlock>);
  if (critical_block(q.L) <= 512) return go(&k_critical<kRB, true, 512>);
  return ring ? go(&k_critical<kRB, true, kCritMaxBlock>) : go(&k_critical<kRB, false, kCritMaxBlock>);
}

}  // namespace qew
