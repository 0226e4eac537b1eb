// qew_kernels.hip -- gfx950 kernels of the QEW integrator.
//
// Eq. (1) of arXiv:1211.7275 (eta = 1) on periodic chains, explicit Euler
// (Sec. III B), pinning force from counter-based random values at integer u
// with a Catmull-Rom spline, and the FP64 observables of Eqs. (3)-(5).
//
// Kernels:
//   k_step_plain   one FP64 Euler step per launch, one thread per site, four
//                  Philox nodes regenerated per site update.  HBM traffic is
//                  16 B per update (read u, write u; neighbours hit L1/L2).
//   k_blocked_plain
//                  several FP64 steps per launch on overlapping tiles, nodes
//                  made when a site enters a cell.
//   k_lanes        the same in both precisions for small problems: narrow tiles,
//                  every lane makes its own nodes, no request path.
//   k_step_split1  the same on the split state (int32 cell + FP32 offset).
//   k_step_fused   `nsub` split Euler steps per launch.  Each workgroup owns
//                  a tile of 256*P consecutive sites held in registers (P
//                  per thread), `halo` of them on each side recomputed
//                  redundantly; the four nodes of each site's cell stay in
//                  LDS (and in HBM between launches).  A site whose cell
//                  changes needs one new node; each wave gathers its sites'
//                  requests into LDS and serves them with its own lanes, so
//                  Philox costs one pass per wave and sub-step instead of
//                  one per changed site slot.
//   k_meas_*       per-tile FP64 partials of sum F, sum (u-K), sum (u-K)^2.
//   k_meas_final   per-sample combine (Chan et al. pairwise update) into
//                  v, ubar, w2.
#include "qew_device.hpp"
#include "qew_internal.hpp"

#include <type_traits>

namespace qew {

namespace {

__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Wave-wide lane shifts by one (DPP wave_shr:1 / wave_shl:1): lane l receives
// x of lane l - 1 (resp. l + 1); lane 0 (resp. 63) receives 0.
__device__ __forceinline__ float from_lower_lane(float x) {
  const int v = __float_as_int(x);
  return __int_as_float(__builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float from_upper_lane(float x) {
  const int v = __float_as_int(x);
  return __int_as_float(__builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, true));
}

// A pointer into LDS (32-bit, address space 3).
typedef __attribute__((address_space(3))) float lds_f32;

// Node c + d of cell c.  Nodes are numbered modulo 2^32 (the generator's counter
// word), so that the windows of the last cells go on past the largest integer.
__device__ __forceinline__ int32_t node_after(int32_t c, int d) { return (int32_t)((uint32_t)c + (uint32_t)d); }

// Between two rounds of the request slots of a wave: no lane's next request may
// be written before every lane has read its reply from the slot.  The wave's LDS
// operations complete in program order, so only the compiler has to keep it.
__device__ __forceinline__ void slots_read() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t mbcnt64(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Deterministic FP64 sum of three values over a group of kBlock threads (thread
// `tid` of it; fixed reduction order; the whole workgroup takes part).
__device__ __forceinline__ void group_sum3(double& a, double& b, double& c, int tid, double* lds /*[3*4]*/) {
  a = wave_sum_f64(a);
  b = wave_sum_f64(b);
  c = wave_sum_f64(c);
  const int w = tid >> 6;
  if ((tid & 63) == 0) {
    lds[w * 3 + 0] = a;
    lds[w * 3 + 1] = b;
    lds[w * 3 + 2] = c;
  }
  __syncthreads();
  if (tid == 0) {
    double x = 0.0, y = 0.0, z = 0.0;
    for (int i = 0; i < kBlock / 64; ++i) {
      x += lds[i * 3 + 0];
      y += lds[i * 3 + 1];
      z += lds[i * 3 + 2];
    }
    a = x;
    b = y;
    c = z;
  }
}
__device__ __forceinline__ void block_sum3(double& a, double& b, double& c, double* lds) {
  group_sum3(a, b, c, (int)threadIdx.x, lds);
}

}  // namespace

// Per-sample combine of tile partials: mean and sum of squared deviations by
// the pairwise update of Chan, Golub and LeVeque, in a fixed order.
struct Moments {
  double n, mean, m2, sf;
};

__device__ __forceinline__ Moments combine(const Moments& a, const Moments& b) {
  if (a.n == 0.0) return b;
  if (b.n == 0.0) return a;
  const double n = a.n + b.n;
  const double d = b.mean - a.mean;
  Moments r;
  r.n = n;
  r.mean = a.mean + d * (b.n / n);
  r.m2 = (a.m2 + b.m2) + d * d * (a.n * b.n / n);
  r.sf = a.sf + b.sf;
  return r;
}

__device__ __forceinline__ Moments moments_of(const Partial& p, int len) {
  const double n = (double)len;
  return Moments{n, p.shift + p.s1 / n, p.s2 - p.s1 * (p.s1 / n), p.sum_f};
}

// Sample s's v, ubar, w2 at measurement o.mi.
__device__ __forceinline__ void write_series(const Tables& t, const MeasOut& o, int s, const Moments& m) {
  const double L = (double)t.L[s];
  double* out = o.series + ((int64_t)s * o.n_meas + o.mi) * 3;
  const double v = m.sf / L;
  out[0] = v;
  out[1] = m.mean;
  out[2] = (m.m2 > 0.0 ? m.m2 : 0.0) / L;
  if (o.v_host) o.v_host[s] = v;  // pinned host memory
}

// What a measuring launch does with its sums.  kFinal (every sample has at
// most kFinalTiles tiles): a workgroup takes a whole sample, kBlock threads per
// tile, combines its tiles in k_meas_final's order and writes the series: a
// measurement is one launch less (L = 1024 x 4 over 10^4 steps with 50: 3.98 ->
// 3.82 ms).  Four tiles of a sample on one CU cost more than that launch (24
// lines of 2^14 sites with 60 measurements: 4.67 -> 4.85 ms).
enum { kNoMeas = 0, kPartials = 1, kFinal = 2 };
constexpr int meas_block(int mode) { return mode == kFinal ? kBlock * kFinalTiles : kBlock; }

// The measurement tile of this thread's group, and the thread within it.
struct TileOf {
  int tile, s, tid;
  bool valid;
};
template <int MODE>
__device__ __forceinline__ TileOf tile_of(const Tables& t) {
  if constexpr (MODE == kFinal) {
    const int s = blockIdx.x;
    const int tile = t.mt_first[s] + uniform_i32((int)(threadIdx.x / kBlock));
    return TileOf{tile, s, (int)(threadIdx.x % kBlock), tile < t.mt_first[s + 1]};
  } else {
    const int tile = blockIdx.x;  // one index for all of the tile's table entries: their loads then overlap
    return TileOf{tile, t.mt_s[tile], (int)threadIdx.x, true};
  }
}

struct MeasLds {
  double sum[3 * (kBlock / 64) * kFinalTiles];
  Moments m[kFinalTiles];
};

template <int MODE>
__device__ __forceinline__ void emit(const Tables& t, const MeasOut& o, const TileOf& w, int len, double sf, double s1,
                                     double s2, double shift, MeasLds& lds) {
  if constexpr (MODE == kPartials) {
    block_sum3(sf, s1, s2, lds.sum);
    if (threadIdx.x == 0) o.part[w.tile] = Partial{sf, s1, s2, shift};
  } else {
    const int g = threadIdx.x / kBlock;
    group_sum3(sf, s1, s2, w.tid, lds.sum + g * 3 * (kBlock / 64));
    if (w.tid == 0) lds.m[g] = w.valid ? moments_of(Partial{sf, s1, s2, shift}, len) : Moments{0.0, 0.0, 0.0, 0.0};
    __syncthreads();
    if (threadIdx.x == 0) {
      Moments m = lds.m[0];
      if (blockDim.x > kBlock) m = combine(m, lds.m[1]);
      write_series(t, o, w.s, m);
    }
  }
}

// ---------------------------------------------------------------------------
// Initialisation: flat start u = 0 (Sec. II).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_init_plain(Tables t, double* u) {
  const int tile = blockIdx.x;
  const int s = t.mt_s[tile];
  const int p0 = t.mt_p0[tile], len = t.mt_len[tile];
  const int64_t base = t.off[s];
  for (int q = threadIdx.x; q < len; q += kBlock) u[base + p0 + q] = 0.0;
}

template <int KIND>
__global__ void __launch_bounds__(kBlock)
    k_init_split(Tables t, SplitBuf b, Phys ph, int with_nodes) {
  const int tile = blockIdx.x;
  const int s = t.mt_s[tile];
  const int p0 = t.mt_p0[tile], len = t.mt_len[tile];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  for (int q = threadIdx.x; q < len; q += kBlock) {
    const int j = p0 + q;
    const int32_t c = 0;
    b.cell[base + j] = 0;
    b.frac[base + j] = 0.0f;
    if (with_nodes) {
      float4 nd;
      nd.x = node_f32<KIND>(j, c - 1, id, keys, ph.period);
      nd.y = node_f32<KIND>(j, c, id, keys, ph.period);
      nd.z = node_f32<KIND>(j, c + 1, id, keys, ph.period);
      nd.w = node_f32<KIND>(j, c + 2, id, keys, ph.period);
      b.nodes[base + j] = nd;
    }
  }
}

// Rebuild of the fused path's node cache for the state in `b` (after
// one-step stretches or a written state): the nodes of every site's cell.
template <int KIND>
__global__ void __launch_bounds__(kBlock) k_refresh_nodes(Tables t, SplitBuf b, Phys ph) {
  const int tile = blockIdx.x;
  const int s = t.mt_s[tile];
  const int p0 = t.mt_p0[tile], len = t.mt_len[tile];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  for (int q = threadIdx.x; q < len; q += kBlock) {
    const int j = p0 + q;
    const int32_t c = b.cell[base + j];
    float4 nd;
    nd.x = node_f32<KIND>(j, c - 1, id, keys, ph.period);
    nd.y = node_f32<KIND>(j, c, id, keys, ph.period);
    nd.z = node_f32<KIND>(j, c + 1, id, keys, ph.period);
    nd.w = node_f32<KIND>(j, c + 2, id, keys, ph.period);
    b.nodes[base + j] = nd;
  }
}

// ---------------------------------------------------------------------------
// One-step kernels (one Euler step per launch).
// ---------------------------------------------------------------------------
// MODE != kNoMeas: also measure the input state (the same loop, forces and
// reduction order as k_meas_plain, so the sums are the same bits), so a
// measured step reads the state once.
template <int KIND, int MODE>
__global__ void __launch_bounds__(meas_block(MODE))
    k_step_plain(Tables t, const double* __restrict__ uin, double* __restrict__ uout, Phys ph,
                 MeasOut o) {
  constexpr bool MEAS = MODE != kNoMeas;
  const TileOf w = tile_of<MODE>(t);
  const int s = w.s;
  const int p0 = w.valid ? t.mt_p0[w.tile] : 0, len = w.valid ? t.mt_len[w.tile] : 0;
  const int L = t.L[s];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const double f = t.f[s];
  const PlainPhys pp{ph.c, ph.dt, ph.strength};
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  const double K = MEAS ? uin[base + p0] : 0.0;
  double sf = 0.0, s1 = 0.0, s2 = 0.0;
  for (int q = w.tid; q < len; q += kBlock) {
    const int j = p0 + q;
    const int jm = (j == 0) ? L - 1 : j - 1;
    const int jp = (j == L - 1) ? 0 : j + 1;
    const double u = uin[base + j];
    const double F = plain_force<KIND>(uin[base + jm], u, uin[base + jp], (uint32_t)j, id, keys, f,
                                       ph.period, pp);
    uout[base + j] = u + ph.dt * F;
    if constexpr (MEAS) {
      sf += F;
      const double x = u - K;
      s1 += x;
      s2 += x * x;
    }
  }
  if constexpr (MEAS) {
    __shared__ MeasLds lds;
    emit<MODE>(t, o, w, len, sf, s1, s2, K, lds);
  }
}

template <int KIND>
__device__ __forceinline__ void nodes_of(uint32_t j, int32_t c, uint32_t id, const Phys& ph,
                                         const VectorKeys& keys, float& p0, float& p1, float& p2,
                                         float& p3) {
  if (ph.strength == 0.0) {
    p0 = p1 = p2 = p3 = 0.0f;
    return;
  }
  // Catmull-Rom needs nodes c-1..c+2, Case 3 c..c+1, Case 4 c only.
  constexpr bool cubic = (KIND == kRF || KIND == kRB);
  p0 = cubic ? node_f32<KIND>(j, c - 1, id, keys, ph.period) : 0.0f;
  p1 = node_f32<KIND>(j, c, id, keys, ph.period);
  p2 = (KIND != kRFPc) ? node_f32<KIND>(j, c + 1, id, keys, ph.period) : 0.0f;
  p3 = cubic ? node_f32<KIND>(j, c + 2, id, keys, ph.period) : 0.0f;
}

// MODE != kNoMeas: also measure the input state, as k_meas_split does (same
// loop, forces and reduction order).
template <int KIND, int MODE>
__global__ void __launch_bounds__(meas_block(MODE))
    k_step_split1(Tables t, SplitBuf in, SplitBuf out, Phys ph, MeasOut o) {
  constexpr bool MEAS = MODE != kNoMeas;
  const TileOf w = tile_of<MODE>(t);
  const int s = w.s;
  const int p0 = w.valid ? t.mt_p0[w.tile] : 0, len = w.valid ? t.mt_len[w.tile] : 0;
  const int L = t.L[s];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const float f = t.f32[s];
  const SplitPhys sp{ph.cf, ph.dtf, ph.sgn_strf};
  const int32_t Kc = MEAS ? in.cell[base + p0] : 0;
  const double Kr = MEAS ? (double)in.frac[base + p0] : 0.0;
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  double sf = 0.0, s1 = 0.0, s2 = 0.0;
  for (int q = w.tid; q < len; q += kBlock) {
    const int j = p0 + q;
    const int jm = (j == 0) ? L - 1 : j - 1;
    const int jp = (j == L - 1) ? 0 : j + 1;
    int32_t c = in.cell[base + j];
    float r = in.frac[base + j];
    float n0, n1, n2, n3;
    nodes_of<KIND>((uint32_t)j, c, id, ph, keys, n0, n1, n2, n3);
    const float4 a = spline_coef<KIND>(n0, n1, n2, n3, sp.sgn_str, f);
    const float F = split_force<KIND>(c, r, in.cell[base + jm], in.frac[base + jm],
                                      in.cell[base + jp], in.frac[base + jp], a, sp.c);
    if constexpr (MEAS) {
      sf += (double)F;
      const double x = (double)(c - Kc) + ((double)r - Kr);  // exact
      s1 += x;
      s2 += x * x;
    }
    c += (int32_t)split_advance(r, F, sp.dt);
    out.cell[base + j] = c;
    out.frac[base + j] = r;
  }
  if constexpr (MEAS) {
    __shared__ MeasLds lds;
    emit<MODE>(t, o, w, len, sf, s1, s2, (double)Kc + Kr, lds);
  }
}

// ---------------------------------------------------------------------------
// Fused temporally blocked kernel (split precision).
//
// One workgroup owns one tile of T = 256 P consecutive sites of one sample at
// a time: positions p0 - halo .. p0 - halo + T - 1 (periodic in the sample).
// Thread t holds sites t P .. t P + P - 1 in registers: the cell as an exact
// float relative to the tile's first cell (no int/float conversion per step),
// the offset, and the coefficients of f + F_p of the current cell.  The four
// raw nodes of every site live in LDS, slot-major (node index i * 256 + t).
// Each sub-step:
//   1. every site takes one Euler step (neighbours within a thread directly,
//      across lanes by DPP wave shifts, across waves through a double-buffered
//      LDS edge array);
//   2. a site whose cell changed posts a request (its LDS node index and its
//      new and old cells) into its wave's region of the request list;
//   3. the same wave serves its requests, lane q taking request q: shift the
//      node window, generate the missing node (all four after a jump of two
//      or more cells), store the window, and write the new coefficients into
//      the request slot; the requesters then read them back.  Requests,
//      windows and replies belong to one wave and a wave's LDS operations
//      complete in order, so this needs no workgroup barrier;
//   4. the wave publishes its end sites; one workgroup barrier.
// A wave serves kReqPerWave requests at a time; further ones (a burst of
// simultaneous cell changes) take further rounds, or on wide tiles their lanes
// regenerate the windows themselves.  After nsub <= halo sub-steps the sites within `halo` of either
// tile end hold garbage (the tile ends reflect), and the valid part
// [halo, halo + len) is written back with its nodes.  Every value equals what
// the one-step kernel computes: the float cell differences are exact integers
// (checked: a tile whose cells spread over 2^23 or more raises the error flag).
// ---------------------------------------------------------------------------
constexpr int kReqPerWave = 64;

// Waves per SIMD the register allocation must allow (LDS allows the same).
constexpr int fused_min_waves(int P) { return P == 6 ? 5 : (P <= 8 ? 4 : (P == 12 ? 3 : 2)); }

// Whether a kernel exists that serves a burst in rounds.  Tiles of 12 or more sites per
// thread have none (the rounds' code costs their common path 3 %), nor has the
// sparse random-field kernel, whose registers then allow a wave per SIMD less or
// spill (2^20 x 4, f = 0.8, us per step with rounds and without: 1024-site tiles
// 6.25, 4.80; 1536-site ones 4.84, 4.05).
constexpr bool has_rounds(int kind, int P, bool sparse) { return P <= 8 && !(sparse && kind == kRF); }

template <int KIND, int P, bool SPARSE, bool ROUNDS>
__global__ void __launch_bounds__(kBlock, fused_min_waves(P))
    k_step_fused(Tables t, SplitBuf in, SplitBuf out, Phys ph, int halo, int nsub) {
  constexpr int T = kBlock * P;
  constexpr int NW = kBlock / 64;
  constexpr int RQ = kReqPerWave;
  __shared__ float4 s_nodes[T];
  __shared__ int4 s_req[NW * (RQ + 1)];  // per wave: RQ requests, then one sink slot
  // End sites of each wave, double-buffered: [parity][cell, offset][slot][end],
  // wave w in slot w + 1.  A wave reaches its own and its neighbours' entries
  // through one LDS pointer held in a vector register, so every access is an
  // immediate offset of it (no per-access address moves); cells and offsets
  // are stored as single words, so no two registers need to be adjacent.
  __shared__ float s_edge[2][2][NW + 2][2];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = uniform_i32(tid >> 6);
  // The elastic constant and the time step are kept in vector registers:
  // on gfx950 a VALU instruction with a scalar-register operand issues more
  // slowly than its all-vector form (measured for an FP32 add: 0.24 against
  // 0.35 wave instructions per SIMD cycle), and every site update uses both.
  float cel = ph.cf, dt = ph.dtf;
  asm volatile("" : "+v"(cel));
  asm volatile("" : "+v"(dt));
  const float g = ph.sgn_strf;
  // Unit disorder strength (g = +1 for force values, -1 for potential
  // values): the service pass then forms the coefficients without the four
  // multiplications by g (exactly the same values).
  const bool unit_g = g == kind_sign<KIND>();
  lds_f32* eb = (lds_f32*)&s_edge[0][0][wv][0];  // slot wv: the left neighbour's entries
  asm volatile("" : "+v"(eb));
  // entry of parity `pa`, word q (0 cell, 1 offset), slot wv + ds, end e
  auto edge = [&](int pa, int q, int ds, int e) -> lds_f32& {
    return eb[((pa * 2 + q) * (NW + 2) + ds) * 2 + e];
  };

  for (int ti = blockIdx.x; ti < t.n_ft; ti += gridDim.x) {
    const int s = uniform_i32(t.ft_s[ti]);
    const int p0 = uniform_i32(t.ft_p0[ti]);
    const int len = uniform_i32(t.ft_len[ti]);
    const int L = uniform_i32(t.L[s]);
    const int64_t base = uniform_i64(t.off[s]);
    const uint32_t id = (uint32_t)uniform_i32((int)t.did[s]);
    const float f = t.f32[s];
    const int start = p0 - halo;
    int start_mod = start % L;
    if (start_mod < 0) start_mod += L;
    constexpr int VW = (P % 4 == 0) ? 4 : 2;  // sites per vector load / store
    const bool contiguous = start >= 0 && start + T <= L && (start % VW) == 0;
    // The tile crosses the end of its chain: only then does a site's column
    // need wrapping in the service pass.
    const bool wraps = start_mod + T > L;
    const int32_t cbase = uniform_i32(in.cell[base + start_mod]);

    float c[P];  // cell - cbase, an exact integer
    float r[P];
    float4 a[P];
    bool far = false;
    if (contiguous) {
      const int64_t gi = base + start + tid * P;
#pragma unroll
      for (int v = 0; v < P / VW; ++v) {
        int32_t cc[VW];
        float rr[VW];
        if constexpr (VW == 4) {
          const int4 cv = *reinterpret_cast<const int4*>(in.cell + gi + 4 * v);
          const float4 rv = *reinterpret_cast<const float4*>(in.frac + gi + 4 * v);
          cc[0] = cv.x; cc[1] = cv.y; cc[2] = cv.z; cc[3] = cv.w;
          rr[0] = rv.x; rr[1] = rv.y; rr[2] = rv.z; rr[3] = rv.w;
        } else {
          const int2 cv = *reinterpret_cast<const int2*>(in.cell + gi + 2 * v);
          const float2 rv = *reinterpret_cast<const float2*>(in.frac + gi + 2 * v);
          cc[0] = cv.x; cc[1] = cv.y;
          rr[0] = rv.x; rr[1] = rv.y;
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          const int32_t d = cc[e] - cbase;
          far |= (uint32_t)(d + (1 << 23)) >= (1u << 24);
          c[VW * v + e] = (float)d;
          r[VW * v + e] = rr[e];
        }
      }
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const float4 nd = in.nodes[gi + i];
        s_nodes[i * kBlock + tid] = nd;
        a[i] = spline_coef<KIND>(nd.x, nd.y, nd.z, nd.w, g, f);
      }
    } else {
      int pos = (start_mod + tid * P) % L;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int32_t cc = in.cell[base + pos] - cbase;
        far |= (uint32_t)(cc + (1 << 23)) >= (1u << 24);
        c[i] = (float)cc;
        r[i] = in.frac[base + pos];
        const float4 nd = in.nodes[base + pos];
        s_nodes[i * kBlock + tid] = nd;
        a[i] = spline_coef<KIND>(nd.x, nd.y, nd.z, nd.w, g, f);
        pos = (pos + 1 == L) ? 0 : pos + 1;
      }
    }
    if (__ballot(far) && lane == 0) atomicOr(t.err, 1);
    if (lane == 0) {
      edge(0, 0, 1, 0) = c[0];
      edge(0, 1, 1, 0) = r[0];
    }
    if (lane == 63) {
      edge(0, 0, 1, 1) = c[P - 1];
      edge(0, 1, 1, 1) = r[P - 1];
    }
    __syncthreads();

    // One sub-step; the loop runs it twice per trip so that the state
    // arrays alternate between two register sets without copies.
    auto substep = [&](const int par) __attribute__((always_inline)) {
      // Neighbours of this thread's end sites.  The tile ends reflect.
      float cle = from_lower_lane(c[P - 1]);
      float rle = from_lower_lane(r[P - 1]);
      float cre = from_upper_lane(c[0]);
      float rre = from_upper_lane(r[0]);
      if (lane == 0) {
        if (wv > 0) {
          cle = edge(par, 0, 0, 1);
          rle = edge(par, 1, 0, 1);
        } else {
          cle = c[0];
          rle = r[0];
        }
      }
      if (lane == 63) {
        if (wv < NW - 1) {
          cre = edge(par, 0, 2, 0);
          rre = edge(par, 1, 2, 0);
        } else {
          cre = c[P - 1];
          rre = r[P - 1];
        }
      }

      // Wave priorities (s_setprio): a wave takes its steps and posts its
      // requests at the highest priority, serves and reads them back at the
      // lowest, and publishes its edges towards the barrier in between.  The
      // SIMD then issues the long, independent step chains first and fills
      // their gaps with the latency-bound request path of the other waves.
      __builtin_amdgcn_s_setprio(3);
      // Euler step of every site (Jacobi: old values of the neighbours); a
      // site that changed cell posts a request into this wave's region, at
      // byte offset kb[i] of s_req.  Requests past the region's RQ entries go
      // to its sink slot and are served by their own lane below.
      uint32_t kb[P];
      uint32_t nreq = 0u;  // wave-uniform
      const int rbase = wv * (RQ + 1);
      const uint32_t rbase_b = (uint32_t)rbase * (uint32_t)sizeof(int4);
      const uint32_t sink_b = rbase_b + (uint32_t)RQ * (uint32_t)sizeof(int4);
      float oc[P];          // cells before the step
      float dl = c[0] - cle;  // cell difference to the left neighbour
      float pr = rle;
      // All steps first (independent chains the scheduler can interleave),
      // then the requests of the sites that changed cell.
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const float nc = (i + 1 < P) ? c[i + 1] : cre;
        const float nr = (i + 1 < P) ? r[i + 1] : rre;
        const float dr = nc - c[i];
        const float lap = (dr - dl) + fmaf(-2.0f, r[i], pr + nr);
        const float F = fmaf(cel, lap, spline_eval<KIND>(a[i], r[i]));
        dl = dr;
        pr = r[i];
        oc[i] = c[i];
        c[i] = oc[i] + split_advance(r[i], F, dt);
      }
      // The sparse variant first checks whether any site of the wave changed
      // cell and skips the request bookkeeping when none did.
      bool book = true;
      if constexpr (SPARSE) {
        uint64_t any_move = 0u;
#pragma unroll
        for (int i = 0; i < P; ++i) any_move |= __ballot(c[i] != oc[i]);
        book = any_move != 0u;
      }
      if (book) {
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const bool mv = c[i] != oc[i];
        const uint64_t moved = __ballot(mv);
        const uint32_t cnt = (uint32_t)__popcll(moved);
        // The wave-uniform part stays one scalar operand of the address;
        // requests past the region land in its sink slot.
        kb[i] = min(mbcnt64(moved) * (uint32_t)sizeof(int4) +
                        (uint32_t)uniform_i32((int)(rbase_b + nreq * (uint32_t)sizeof(int4))),
                    sink_b);
        if (mv) {
          // The two cells go in the order of their registers, which swap
          // roles every sub-step: {new, old} on even sub-steps, {old, new}
          // on odd ones, so the three words stay one store without copies.
          const float w1 = par ? oc[i] : c[i];
          const float w2 = par ? c[i] : oc[i];
          *reinterpret_cast<int3*>(reinterpret_cast<char*>(s_req) + kb[i]) =
              make_int3(i * kBlock + tid, __float_as_int(w1), __float_as_int(w2));
        }
        nreq += cnt;
      }
      // Serve this wave's requests with this wave's lanes: lane q takes request
      // q.  The requests, their node windows and the replies belong to this
      // wave only, and a wave's LDS operations complete in program order, so
      // no workgroup barrier is needed between posting, serving and reading.
      __builtin_amdgcn_s_setprio(0);
      auto serve = [&](uint32_t nserve) __attribute__((always_inline)) {
        __builtin_amdgcn_wave_barrier();
        if ((uint32_t)lane < nserve) {
          const int slot = rbase + lane;
          const int4 rq = s_req[slot];  // {node index, cells (relative to cbase) in sub-step order}
          const int ni = rq.x;
          const float cnew = __int_as_float(par ? rq.z : rq.y);
          const float move = cnew - __int_as_float(par ? rq.y : rq.z);
          const int32_t cell = cbase + (int32_t)cnew;
          const int lp = (int)(((uint32_t)ni % kBlock) * P + (uint32_t)ni / kBlock);  // tile-local position
          int j = start_mod + lp;
          if (wraps) {
            if (j >= L) j -= L;
            if (j >= L) j %= L;
          }
          float4 w4 = s_nodes[ni];
          if (move == 1.0f) {
            w4 = make_float4(w4.y, w4.z, w4.w, node_f32<KIND>((uint32_t)j, cell + 2, id, ph.k0, ph.k1, ph.period));
          } else if (move == -1.0f) {
            w4 = make_float4(node_f32<KIND>((uint32_t)j, cell - 1, id, ph.k0, ph.k1, ph.period), w4.x, w4.y, w4.z);
          } else if constexpr (ROUNDS || P > 8) {
#pragma unroll 1
            for (int i = 0; i < 4; ++i)
              w4 = make_float4(w4.y, w4.z, w4.w,
                               node_f32<KIND>((uint32_t)j, node_after(cell, i - 1), id, ph.k0, ph.k1, ph.period));
          } else {  // jumps are what this kernel is for
            w4 = make_float4(node_f32<KIND>((uint32_t)j, node_after(cell, -1), id, ph.k0, ph.k1, ph.period),
                             node_f32<KIND>((uint32_t)j, cell, id, ph.k0, ph.k1, ph.period),
                             node_f32<KIND>((uint32_t)j, node_after(cell, 1), id, ph.k0, ph.k1, ph.period),
                             node_f32<KIND>((uint32_t)j, node_after(cell, 2), id, ph.k0, ph.k1, ph.period));
          }
          s_nodes[ni] = w4;
          float4 co;
          if (unit_g) co = spline_coef<KIND>(w4.x, w4.y, w4.z, w4.w, kind_sign<KIND>(), f);
          else co = spline_coef<KIND>(w4.x, w4.y, w4.z, w4.w, g, f);
          s_req[slot] = make_int4(__float_as_int(co.x), __float_as_int(co.y), __float_as_int(co.z),
                                  __float_as_int(co.w));
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
      };
      auto read_back = [&](int i, uint32_t at) __attribute__((always_inline)) {
        const int4 v = *reinterpret_cast<const int4*>(reinterpret_cast<const char*>(s_req) + at);
        a[i] = make_float4(__int_as_float(v.x), __int_as_float(v.y), __int_as_float(v.z), __int_as_float(v.w));
      };
      const uint32_t nserve = nreq < (uint32_t)RQ ? nreq : (uint32_t)RQ;
      if (nserve > 0u) {
        serve(nserve);
        // Requesters read their new coefficients (a request past the region
        // reads its sink slot and is served below).
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (c[i] != oc[i]) read_back(i, kb[i]);
        __builtin_amdgcn_wave_barrier();
      }
      // Rare: more requests than the region holds (a burst of cell changes).
      // Those past it are posted and served in further rounds (ROUNDS), or their
      // lanes make their windows themselves.  At 2^22 x 4 on 2048-site tiles, k = 56,
      // ms per launch, own windows and rounds: f = 1.0 0.692, 0.678; f = 2.5 1.165, 1.042;
      // random bond f = 4 2.563, 1.392.
      if constexpr (ROUNDS) {
#pragma unroll 1
        for (uint32_t done = RQ; done < nreq; done += RQ) {
          slots_read();
          uint32_t first = 0u;
          bool mine[P];
#pragma unroll
          for (int i = 0; i < P; ++i) {
            const bool mv = c[i] != oc[i];
            const uint64_t moved = __ballot(mv);
            const uint32_t r = first + mbcnt64(moved) - done;
            mine[i] = mv && r < (uint32_t)RQ;
            kb[i] = rbase_b + r * (uint32_t)sizeof(int4);
            if (mine[i])
              *reinterpret_cast<int3*>(reinterpret_cast<char*>(s_req) + kb[i]) = make_int3(
                  i * kBlock + tid, __float_as_int(par ? oc[i] : c[i]), __float_as_int(par ? c[i] : oc[i]));
            first += (uint32_t)__popcll(moved);
          }
          serve(nreq - done < (uint32_t)RQ ? nreq - done : (uint32_t)RQ);
#pragma unroll
          for (int i = 0; i < P; ++i)
            if (mine[i]) read_back(i, kb[i]);
        }
      } else if (nreq > (uint32_t)RQ) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
          if (c[i] != oc[i] && kb[i] == sink_b) {
            int j = start_mod + tid * P;
            asm volatile("" : "+v"(j));  // keep this rare path's index arithmetic here
            j += i;
            if (j >= L) j -= L;
            if (j >= L) j %= L;
            const int32_t cell = cbase + (int32_t)c[i];
            const float4 w4 = make_float4(node_f32<KIND>((uint32_t)j, cell - 1, id, ph.k0, ph.k1, ph.period),
                                          node_f32<KIND>((uint32_t)j, cell, id, ph.k0, ph.k1, ph.period),
                                          node_f32<KIND>((uint32_t)j, cell + 1, id, ph.k0, ph.k1, ph.period),
                                          node_f32<KIND>((uint32_t)j, cell + 2, id, ph.k0, ph.k1, ph.period));
            s_nodes[i * kBlock + tid] = w4;
            a[i] = spline_coef<KIND>(w4.x, w4.y, w4.z, w4.w, g, f);
          }
        }
      }
      }  // book
      __builtin_amdgcn_s_setprio(2);
      // Publish this wave's end sites for the neighbouring waves' next sub-step.
      if (lane == 0) {
        edge(par ^ 1, 0, 1, 0) = c[0];
        edge(par ^ 1, 1, 1, 0) = r[0];
      }
      if (lane == 63) {
        edge(par ^ 1, 0, 1, 1) = c[P - 1];
        edge(par ^ 1, 1, 1, 1) = r[P - 1];
      }
      __syncthreads();
    };
    int sub = 0;
    for (; sub + 2 <= nsub; sub += 2) {
      substep(0);
      substep(1);
    }
    if (sub < nsub) substep(0);

    // Write the valid part: tile-local q in [halo, halo + len).
    int qb = tid * P;
    asm volatile("" : "+v"(qb));
    const int64_t g0 = base + p0 + (qb - halo);
    if (qb >= halo && qb + P <= halo + len && (g0 % VW) == 0) {
#pragma unroll
      for (int v = 0; v < P / VW; ++v) {
        if constexpr (VW == 4) {
          *reinterpret_cast<int4*>(out.cell + g0 + 4 * v) =
              make_int4(cbase + (int32_t)c[4 * v], cbase + (int32_t)c[4 * v + 1],
                        cbase + (int32_t)c[4 * v + 2], cbase + (int32_t)c[4 * v + 3]);
          *reinterpret_cast<float4*>(out.frac + g0 + 4 * v) =
              make_float4(r[4 * v], r[4 * v + 1], r[4 * v + 2], r[4 * v + 3]);
        } else {
          *reinterpret_cast<int2*>(out.cell + g0 + 2 * v) =
              make_int2(cbase + (int32_t)c[2 * v], cbase + (int32_t)c[2 * v + 1]);
          *reinterpret_cast<float2*>(out.frac + g0 + 2 * v) = make_float2(r[2 * v], r[2 * v + 1]);
        }
      }
#pragma unroll
      for (int i = 0; i < P; ++i) out.nodes[g0 + i] = s_nodes[i * kBlock + tid];
    } else {
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int q = qb + i;
        if (q >= halo && q < halo + len) {
          const int64_t gi = base + p0 + (q - halo);
          out.cell[gi] = cbase + (int32_t)c[i];
          out.frac[gi] = r[i];
          out.nodes[gi] = s_nodes[i * kBlock + tid];
        }
      }
    }
    __syncthreads();  // s_nodes and s_edge are reused by the next tile
  }
}

// ---------------------------------------------------------------------------
// Temporally blocked FP64 kernel: nsub <= halo Euler steps per launch.
//
// The one-step kernel makes the four nodes of every site at every step (some
// 200 vector operations); a site changes its cell only every 20 steps or so.
// Here a workgroup keeps a tile of T = 256 P consecutive sites (the valid part
// and `halo` more on each side, recomputed redundantly) in registers with the
// coefficients of their current cells, and makes one node when a site enters a
// new cell.  The request path is that of k_step_fused: sites that changed cell
// post a request in LDS, the same wave serves them one per lane and the
// requesters read their new coefficients back.
//
// Bound by VALU issue: 16 FP64 operations of 4 cycles per site and step (some
// 10 us per step at 2^22 x 4), 6 to post a site's cell change, and a service
// pass of some 90 instructions per wave and sub-step, whose 64 lanes about 17
// requests of a wave's 384 sites fill to a quarter.  A launch costs 110 us more
// for loads and the nodes of its tiles.  1536 sites are what lets four waves
// per SIMD have their registers and LDS, and leave a wave's request region room
// on fast lines.  us per step at 2^22 x 4, k = 64 (one step per launch: 97):
//                                      1536 sites  2048 sites
//   RF, f = 0.5 / 1.0 / 2.4          23.2 / 25.2 / 27.1  23.7 / 25.6 / 33.5
//   RB linear, the same drives       66.0 / 63.0 / 37.4  88.2 / 79.8 / 43.2
//   RF without interpolation         53.9 / 31.5 / 31.3  62.3 / 46.3 / 41.3
// (RF, f = 1: 3072 sites 28.0, 1024 sites 29.2; k = 48 to 96 within 3 %.)
// Random bond, whose windows take twice the LDS, on 1024-site tiles: 42
// against 406 us.
//
// Same results as the one-step kernel, bit for bit: the coefficients are the
// sums of spline_f64 (halved, which is exact), the steps its operations in its
// order.
// ---------------------------------------------------------------------------
// Coefficients of F_p in the offset s of a cell with (scaled) nodes p0..p3:
// a0 + s (a1 + s (a2 + s a3)) rounds as spline_f64 does.
template <int KIND>
struct CoefD {
  static constexpr int N = KIND == kRF ? 4 : (KIND == kRB ? 3 : 1);
  double a[N];
};

template <int KIND>
__device__ __forceinline__ CoefD<KIND> coef_f64(double p0, double p1, double p2, double p3) {
  CoefD<KIND> c;
  if constexpr (KIND == kRBLin) {
    c.a[0] = -(p2 - p1);
  } else if constexpr (KIND == kRFPc) {
    c.a[0] = p1;
  } else {
    const double c1 = p2 - p0;
    const double c2 = 2.0 * p0 - 5.0 * p1 + 4.0 * p2 - p3;
    const double c3 = -p0 + 3.0 * p1 - 3.0 * p2 + p3;
    if constexpr (KIND == kRF) {
      c.a[0] = p1;
      c.a[1] = 0.5 * c1;
      c.a[2] = 0.5 * c2;
      c.a[3] = 0.5 * c3;
    } else {
      c.a[0] = -0.5 * c1;
      c.a[1] = -c2;
      c.a[2] = -0.5 * (3.0 * c3);
    }
  }
  return c;
}

template <int KIND>
__device__ __forceinline__ double pin_f64(const CoefD<KIND>& c, double s) {
  if constexpr (KIND == kRF) return c.a[0] + s * (c.a[1] + s * (c.a[2] + s * c.a[3]));
  else if constexpr (KIND == kRB) return c.a[0] + s * (c.a[1] + s * c.a[2]);
  else return c.a[0];
}

// Unscaled nodes kept for a site of cell n, nodes n + kLow .. n + kHigh (the
// random-field values are exact in FP32).
template <int KIND>
struct WindowD {
  static constexpr int kLow = (KIND == kRF || KIND == kRB) ? -1 : 0;
  static constexpr int kHigh = (KIND == kRF || KIND == kRB) ? 2 : (KIND == kRBLin ? 1 : 0);
  static constexpr int kCount = kHigh - kLow + 1;
  using type = std::conditional_t<KIND == kRF, float, double>;
  type v[kCount];
  __device__ __forceinline__ void push_up(double x) {
#pragma unroll
    for (int i = 0; i + 1 < kCount; ++i) v[i] = v[i + 1];
    v[kCount - 1] = (type)x;
  }
  __device__ __forceinline__ void push_down(double x) {
#pragma unroll
    for (int i = kCount - 1; i > 0; --i) v[i] = v[i - 1];
    v[0] = (type)x;
  }
  __device__ __forceinline__ CoefD<KIND> coef(double strength, bool unit) const {
    if constexpr (KIND == kRF) {
      if (unit) {
        // Unit strength: the nodes are multiples of 2^-24 below 1, every sum of
        // coef_f64 is exact, and so is this shorter form of it.
        const double q0 = v[0], q1 = v[1], q2 = v[2], q3 = v[3];
        CoefD<KIND> c;
        c.a[0] = q1;
        c.a[1] = 0.5 * (q2 - q0);
        c.a[2] = fma(-0.5, q3, fma(2.0, q2, fma(-2.5, q1, q0)));
        c.a[3] = fma(1.5, q1 - q2, 0.5 * (q3 - q0));
        return c;
      }
    }
    double p[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < kCount; ++i) p[i + 1 + kLow] = strength * (double)v[i];
    return coef_f64<KIND>(p[0], p[1], p[2], p[3]);
  }
};

__device__ __forceinline__ double from_lower_lane(double x) {
  const uint64_t v = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x138, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x138, 0xF, 0xF, true);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double from_upper_lane(double x) {
  const uint64_t v = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x130, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x130, 0xF, 0xF, true);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// Waves per SIMD the register allocation must allow.  Random bond: no more fit
// the LDS.  Linear random bond: the Box-Muller transform and its windows spill
// at four (107 us per step at 2^22 x 4 against 63).  The other two spill 3 and 6
// registers at four, and run faster than at three all the same (see above).
constexpr int blocked_min_waves(int kind) { return kind == kRF || kind == kRFPc ? 4 : 3; }

template <int KIND, int P>
__global__ void __launch_bounds__(kBlock, blocked_min_waves(KIND))
    k_blocked_plain(Tables t, const double* __restrict__ uin, double* __restrict__ uout, Phys ph, int halo,
                    int nsub) {
  constexpr int T = kBlock * P;
  constexpr int NW = kBlock / 64;
  constexpr int RQ = kReqPerWave;
  constexpr int NC = CoefD<KIND>::N;
  using Win = WindowD<KIND>;
  // A request: the new cell and the site's index; its reply: the coefficients.
  // Every access to a slot goes through these types: it holds a cell and an index
  // first and four coefficients later, and the order of the two must hold.
  typedef double __attribute__((may_alias)) slot_f64;
  typedef int __attribute__((may_alias)) slot_i32;
  struct __align__(16) Req {
    slot_f64 cell;
    slot_i32 site, pad;
    slot_f64 more[2];
  };
  __shared__ __align__(16) Win s_win[T];  // nodes of the site's cell, slot-major
  __shared__ int s_cell[T];
  __shared__ Req s_req[NW * (RQ + 1)];     // per wave: RQ requests, then one sink slot
  __shared__ double s_edge[2][NW + 2][2];  // end sites of each wave, double-buffered

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = uniform_i32(tid >> 6);
  const double cel = ph.c, dt = ph.dt, str = ph.strength;
  const bool unit = str == 1.0;
  const int s = uniform_i32(t.ft_s[blockIdx.x]);
  const int p0 = uniform_i32(t.ft_p0[blockIdx.x]);
  const int len = uniform_i32(t.ft_len[blockIdx.x]);
  const int L = uniform_i32(t.L[s]);
  const int64_t base = uniform_i64(t.off[s]);
  const uint32_t id = (uint32_t)uniform_i32((int)t.did[s]);
  const double f = t.f[s];
  const int start = p0 - halo;
  int start_mod = start % L;
  if (start_mod < 0) start_mod += L;
  // Column of tile-local position lp (wrapped only in tiles that cross their chain's end).
  const bool wraps = start_mod + T > L;
  auto column = [&](int lp) -> int {
    int j = start_mod + lp;
    if (wraps) {
      if (j >= L) j -= L;
      if (j >= L) j %= L;
    }
    return j;
  };
  // The window of a site of column j that moved by `move` cells to cell n (one
  // node; all of them after a jump or at the start, move = 0).
  auto advance_window = [&](Win& w, int j, int32_t n, int move) {
    if (__all(move == 1)) {  // the usual case: every site of the wave moved forward by one
      w.push_up(node_f64<KIND>((uint32_t)j, node_after(n, Win::kHigh), id, ph.k0, ph.k1, ph.period));
      return;
    }
    const bool down = move == -1;
    const int first = move == 1 ? Win::kHigh : Win::kLow, last = down ? first : Win::kHigh;
#pragma unroll 1
    for (int m = first; m <= last; ++m) {
      const double x = node_f64<KIND>((uint32_t)j, node_after(n, m), id, ph.k0, ph.k1, ph.period);
      if (down) w.push_down(x);
      else w.push_up(x);
    }
  };

  double u[P], nf[P];
  CoefD<KIND> a[P];
  {
    const int j = column(tid * P);
    if ((P % 2) == 0 && start >= 0 && start + T <= L && (start & 1) == 0) {
      const double2* src = reinterpret_cast<const double2*>(uin + base + start + tid * P);
#pragma unroll
      for (int i = 0; i < P / 2; ++i) {
        const double2 x = src[i];
        u[2 * i] = x.x;
        u[2 * i + 1] = x.y;
      }
    } else {
      int jj = j;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        u[i] = uin[base + jj];
        jj = (jj + 1 == L) ? 0 : jj + 1;
      }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      nf[i] = floor(u[i]);
      s_cell[i * kBlock + tid] = (int32_t)nf[i];
    }
    int jj = j;
#pragma unroll 1
    for (int i = 0; i < P; ++i) {
      Win w{};
      advance_window(w, jj, s_cell[i * kBlock + tid], 0);
      s_win[i * kBlock + tid] = w;
      jj = (jj + 1 == L) ? 0 : jj + 1;
    }
#pragma unroll
    for (int i = 0; i < P; ++i) a[i] = s_win[i * kBlock + tid].coef(str, unit);
  }
  if (lane == 0) s_edge[0][wv + 1][0] = u[0];
  if (lane == 63) s_edge[0][wv + 1][1] = u[P - 1];
  __syncthreads();

  const uint32_t rbase_b = (uint32_t)(wv * (RQ + 1)) * (uint32_t)sizeof(Req);
  const uint32_t sink_b = rbase_b + (uint32_t)RQ * (uint32_t)sizeof(Req);
  for (int sub = 0; sub < nsub; ++sub) {
    const int par = sub & 1;
    // Neighbours of this thread's end sites.  The tile ends reflect.
    double ul = from_lower_lane(u[P - 1]);
    double ur = from_upper_lane(u[0]);
    if (lane == 0) ul = wv > 0 ? s_edge[par][wv][1] : u[0];
    if (lane == 63) ur = wv < NW - 1 ? s_edge[par][wv + 2][0] : u[P - 1];

    __builtin_amdgcn_s_setprio(3);
    bool mv[P];
    uint64_t moved[P];
    uint64_t any_moved = 0u;
    double pl = ul;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const double nr = (i + 1 < P) ? u[i + 1] : ur;
      const double lap = fma(-2.0, u[i], nr + pl);  // 2 u is exact: one rounding, as (nr + pl) - 2 u
      const double F = ((cel * lap) + f) + pin_f64<KIND>(a[i], u[i] - nf[i]);
      pl = u[i];
      u[i] = u[i] + dt * F;
      const double fl = floor(u[i]);
      mv[i] = fl != nf[i];
      moved[i] = __ballot(mv[i]);
      any_moved |= moved[i];
      nf[i] = fl;
    }
    if (any_moved != 0u) {
      uint32_t kb[P];
      uint32_t nreq = 0u;  // wave-uniform
      // Requests past the region land in its sink slot; they come in later rounds.
#pragma unroll
      for (int i = 0; i < P; ++i) {
        kb[i] = min(mbcnt64(moved[i]) * (uint32_t)sizeof(Req) +
                        (uint32_t)uniform_i32((int)(rbase_b + nreq * (uint32_t)sizeof(Req))),
                    sink_b);
        if (mv[i]) {
          Req* rq = reinterpret_cast<Req*>(reinterpret_cast<char*>(s_req) + kb[i]);
          rq->cell = nf[i];
          rq->site = i * kBlock + tid;
        }
        nreq += (uint32_t)__popcll(moved[i]);
      }
      __builtin_amdgcn_s_setprio(0);
      // Lane q serves request q of this wave; a wave's LDS operations complete in order.
      auto serve = [&](uint32_t count) {
        __builtin_amdgcn_wave_barrier();
        if ((uint32_t)lane < count) {
          Req* rq = &s_req[wv * (RQ + 1) + lane];
          const int ni = rq->site;
          const int32_t n = (int32_t)rq->cell;
          Win w = s_win[ni];
          // Beyond the 32-bit cells all sites share the last one: no move, a whole window.
          const int move = (int)((uint32_t)n - (uint32_t)s_cell[ni]);
          advance_window(w, column((int)(((uint32_t)ni % kBlock) * P + (uint32_t)ni / kBlock)), n, move);
          s_win[ni] = w;
          s_cell[ni] = n;
          const CoefD<KIND> c = w.coef(str, unit);
          slot_f64* reply = reinterpret_cast<slot_f64*>(rq);
#pragma unroll
          for (int q = 0; q < NC; ++q) reply[q] = c.a[q];
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
      };
      auto read_back = [&](int i, uint32_t at) {
        const slot_f64* reply = reinterpret_cast<const slot_f64*>(reinterpret_cast<const char*>(s_req) + at);
#pragma unroll
        for (int q = 0; q < NC; ++q) a[i].a[q] = reply[q];
      };
      serve(nreq < (uint32_t)RQ ? nreq : (uint32_t)RQ);
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (mv[i]) read_back(i, kb[i]);
      // A burst of more cell changes than the region holds: further rounds.
      for (uint32_t done = RQ; done < nreq; done += RQ) {
        slots_read();
        uint32_t first = 0u;
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const uint32_t r = first + mbcnt64(moved[i]) - done;
          kb[i] = rbase_b + r * (uint32_t)sizeof(Req);
          if (mv[i] && r < (uint32_t)RQ) {
            Req* rq = reinterpret_cast<Req*>(reinterpret_cast<char*>(s_req) + kb[i]);
            rq->cell = nf[i];
            rq->site = i * kBlock + tid;
          }
          first += (uint32_t)__popcll(moved[i]);
        }
        serve(nreq - done < (uint32_t)RQ ? nreq - done : (uint32_t)RQ);
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (mv[i] && kb[i] - rbase_b < (uint32_t)(RQ * sizeof(Req))) read_back(i, kb[i]);
      }
    }
    __builtin_amdgcn_s_setprio(2);
    if (lane == 0) s_edge[par ^ 1][wv + 1][0] = u[0];
    if (lane == 63) s_edge[par ^ 1][wv + 1][1] = u[P - 1];
    __syncthreads();
  }

  // Write the valid part: tile-local q in [halo, halo + len).
  const int q0 = tid * P;
  double* dst = uout + base + p0 - halo + q0;
  if ((P % 2) == 0 && q0 >= halo && q0 + P <= halo + len && ((p0 - halo) & 1) == 0) {
#pragma unroll
    for (int i = 0; i < P / 2; ++i) reinterpret_cast<double2*>(dst)[i] = make_double2(u[2 * i], u[2 * i + 1]);
  } else {
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (q0 + i >= halo && q0 + i < halo + len) dst[i] = u[i];
  }
}

// ---------------------------------------------------------------------------
// Temporally blocked kernel for small problems, both precisions: nsub <= halo
// Euler steps per launch on tiles of 256 P sites with P = 1 or 2.
//
// When there are only a few sites per CU, a sub-step costs what its longest
// dependent chain costs.  The request path of the wide-tile kernels (post in
// LDS, serve, read back) is such a chain, some 1300 cycles, so here every lane
// serves its own sites: the window of the current cell and the node after it
// stay in registers, up to kSpare nodes further ahead in LDS.  A site that
// enters the next cell only forms its coefficients.  When a lane has no node
// left, the whole wave makes one node ahead for every lane with room, in one
// pass of the generator.  The edges are published before that work, so the
// barrier finds them written, by every lane (a taken branch costs some 40
// cycles here, as much as ten operations).  FP64, four chains of 1024 sites: 0.35
// us per step on 256-site tiles (the request path on them: 1.04, one step per
// launch: 4.1), of which 0.2 us are the steps, the edges and the barrier.  Split
// state, the same chains: 0.32 us against 0.92 of the 1024-site request tiles.
// Measured and dropped: the nodes ahead in registers (0.34), coefficients of
// unit strength in a branch of their own (0.37).
// ---------------------------------------------------------------------------
constexpr int kSpare = 4;

template <int KIND>
struct LanesD {  // FP64 state
  using Buf = const double*;
  using Out = double*;
  using node_t = typename WindowD<KIND>::type;
  using edge_t = double;
  static constexpr int kHigh = WindowD<KIND>::kHigh;
  struct Consts {
    double c, dt, str, f;
    bool unit;
  };
  static __device__ __forceinline__ Consts consts(const Phys& ph, const Tables& t, int s) {
    return {ph.c, ph.dt, ph.strength, t.f[s], ph.strength == 1.0};
  }
  static __device__ __forceinline__ int32_t cell_base(Buf, int64_t) { return 0; }
  struct Site {
    double u, nf;
    CoefD<KIND> a;
    WindowD<KIND> w;
  };
  static __device__ __forceinline__ bool load(Buf in, int64_t g, int32_t, Site& x) {
    x.u = in[g];
    x.nf = floor(x.u);
    return false;
  }
  static __device__ __forceinline__ int32_t cell(const Site& x, int32_t) { return (int32_t)x.nf; }
  static __device__ __forceinline__ edge_t edge(const Site& x) { return x.u; }
  static __device__ __forceinline__ edge_t lower(const edge_t& e) { return from_lower_lane(e); }
  static __device__ __forceinline__ edge_t upper(const edge_t& e) { return from_upper_lane(e); }
  static constexpr bool kWindowInHbm = false;
  static __device__ __forceinline__ void load_window(Buf, int64_t, Site&) {}
  static __device__ __forceinline__ node_t node(uint32_t j, int32_t n, uint32_t id, const Phys& ph) {
    return (node_t)node_f64<KIND>(j, n, id, ph.k0, ph.k1, ph.period);
  }
  static __device__ __forceinline__ void coef(Site& x, const Consts& k) { x.a = x.w.coef(k.str, k.unit); }
  // One step with the old values of the neighbours; returns the cells moved.
  static __device__ __forceinline__ double step(Site& x, edge_t l, edge_t r, const Consts& k) {
    const double lap = fma(-2.0, x.u, r + l);  // 2 u is exact: one rounding, as (r + l) - 2 u
    const double F = ((k.c * lap) + k.f) + pin_f64<KIND>(x.a, x.u - x.nf);
    x.u = x.u + k.dt * F;
    const double fl = floor(x.u);
    const double d = fl - x.nf;
    x.nf = fl;
    return d;
  }
  static __device__ __forceinline__ void store(Out out, int64_t g, const Site& x, int32_t) { out[g] = x.u; }
};

template <int KIND>
struct LanesS {  // split state; the window comes from and returns to the node cache in HBM
  using Buf = SplitBuf;
  using Out = SplitBuf;
  using node_t = float;
  static constexpr int kHigh = 2;
  struct edge_t {
    float c, r;
  };
  struct Consts {
    float c, dt, g, f;
  };
  static __device__ __forceinline__ Consts consts(const Phys& ph, const Tables& t, int s) {
    return {ph.cf, ph.dtf, ph.sgn_strf, t.f32[s]};
  }
  static __device__ __forceinline__ int32_t cell_base(const Buf& in, int64_t g) { return uniform_i32(in.cell[g]); }
  struct Window {
    float v[4];
    __device__ __forceinline__ void push_up(float x) {
      v[0] = v[1];
      v[1] = v[2];
      v[2] = v[3];
      v[3] = x;
    }
  };
  struct Site {
    float c, r;  // cell relative to the tile's first (an exact integer), offset
    float4 a;
    Window w;
  };
  static __device__ __forceinline__ bool load(const Buf& in, int64_t g, int32_t cbase, Site& x) {
    const int32_t d = in.cell[g] - cbase;
    x.c = (float)d;
    x.r = in.frac[g];
    return (uint32_t)(d + (1 << 23)) >= (1u << 24);  // the difference must be exact in FP32
  }
  static __device__ __forceinline__ int32_t cell(const Site& x, int32_t cbase) { return node_after(cbase, (int32_t)x.c); }
  static __device__ __forceinline__ edge_t edge(const Site& x) { return {x.c, x.r}; }
  static __device__ __forceinline__ edge_t lower(const edge_t& e) { return {from_lower_lane(e.c), from_lower_lane(e.r)}; }
  static __device__ __forceinline__ edge_t upper(const edge_t& e) { return {from_upper_lane(e.c), from_upper_lane(e.r)}; }
  static constexpr bool kWindowInHbm = true;
  static __device__ __forceinline__ void load_window(const Buf& in, int64_t g, Site& x) {
    const float4 nd = in.nodes[g];
    x.w.v[0] = nd.x;
    x.w.v[1] = nd.y;
    x.w.v[2] = nd.z;
    x.w.v[3] = nd.w;
  }
  static __device__ __forceinline__ node_t node(uint32_t j, int32_t n, uint32_t id, const Phys& ph) {
    return node_f32<KIND>(j, n, id, ph.k0, ph.k1, ph.period);
  }
  static __device__ __forceinline__ void coef(Site& x, const Consts& k) {
    x.a = spline_coef<KIND>(x.w.v[0], x.w.v[1], x.w.v[2], x.w.v[3], k.g, k.f);
  }
  static __device__ __forceinline__ float step(Site& x, edge_t l, edge_t r, const Consts& k) {
    const float lap = ((r.c - x.c) - (x.c - l.c)) + fmaf(-2.0f, x.r, l.r + r.r);
    const float F = fmaf(k.c, lap, spline_eval<KIND>(x.a, x.r));
    const float d = split_advance(x.r, F, k.dt);
    x.c += d;
    return d;
  }
  static __device__ __forceinline__ void store(const Out& out, int64_t g, const Site& x, int32_t cbase) {
    out.cell[g] = cbase + (int32_t)x.c;
    out.frac[g] = x.r;
    out.nodes[g] = make_float4(x.w.v[0], x.w.v[1], x.w.v[2], x.w.v[3]);
  }
};

template <class A, int P>
__global__ void __launch_bounds__(kBlock, P == 1 ? 4 : 3)
    k_lanes(Tables t, typename A::Buf in, typename A::Out out, Phys ph, int halo, int nsub) {
  constexpr int T = kBlock * P;
  constexpr int NW = kBlock / 64;
  using node_t = typename A::node_t;
  using edge_t = typename A::edge_t;
  __shared__ node_t s_ahead[kSpare][T];    // node m of a site in row m mod kSpare
  // End sites of each wave, double-buffered, and behind them a place for every
  // other lane to write to, so that the publishing needs no branch.
  constexpr int kOther = (NW + 2) * 2;  // from one buffer to the other
  __shared__ edge_t s_edge[2 * kOther + kBlock + kOther];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = uniform_i32(tid >> 6);
  const int s = uniform_i32(t.ft_s[blockIdx.x]);
  const int p0 = uniform_i32(t.ft_p0[blockIdx.x]);
  const int len = uniform_i32(t.ft_len[blockIdx.x]);
  const int L = uniform_i32(t.L[s]);
  const int64_t base = uniform_i64(t.off[s]);
  const uint32_t id = (uint32_t)uniform_i32((int)t.did[s]);
  const typename A::Consts k = A::consts(ph, t, s);
  int start_mod = (p0 - halo) % L;
  if (start_mod < 0) start_mod += L;
  const int32_t cbase = A::cell_base(in, base + start_mod);

  typename A::Site x[P];
  int col[P];        // columns of this thread's sites
  node_t next[P];    // the node after the window, valid while ahead > 0
  int ahead[P];      // nodes made beyond the window, at most kSpare
  bool far = false;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    col[i] = (start_mod + tid * P + i) % L;
    far |= A::load(in, base + col[i], cbase, x[i]);
    A::load_window(in, base + col[i], x[i]);
    next[i] = (node_t)0;
    ahead[i] = 0;
  }
  if (__ballot(far) && lane == 0) atomicOr(t.err, 1);
  // The whole window of cell n, made anew.
  auto fresh = [&](typename A::Site& y, int j) {
    const int32_t n = A::cell(y, cbase);
#pragma unroll 1
    for (int m = A::kHigh + 1 - (int)(sizeof(y.w.v) / sizeof(y.w.v[0])); m <= A::kHigh; ++m)
      y.w.push_up(A::node((uint32_t)j, node_after(n, m), id, ph));
  };
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if constexpr (!A::kWindowInHbm) fresh(x[i], col[i]);
    A::coef(x[i], k);
  }
  // Lanes 0 and 63 publish their wave's ends and read its neighbours' ends, one
  // LDS access each.  Beyond the tile's ends stand their first values: what
  // that spoils stays within nsub sites of the end.
  // Entry (w, e): end e of wave w - 1.
  const int own = 2 * (wv + 1) + (lane == 63 ? 1 : 0);
  edge_t* const mine = &s_edge[lane == 0 || lane == 63 ? own : 2 * kOther + tid];
  const edge_t* const theirs = &s_edge[lane == 63 ? 2 * (wv + 2) : 2 * wv + 1];
  *mine = A::edge(lane == 63 ? x[P - 1] : x[0]);
  if (tid == 0) s_edge[1] = s_edge[kOther + 1] = A::edge(x[0]);
  if (tid == kBlock - 1) s_edge[2 * (NW + 1)] = s_edge[kOther + 2 * (NW + 1)] = A::edge(x[P - 1]);
  __syncthreads();

  auto substep = [&](const int par) __attribute__((always_inline)) {
    // Neighbours of this thread's end sites.
    const edge_t across = theirs[par * kOther];
    edge_t el = A::lower(A::edge(x[P - 1])), er = A::upper(A::edge(x[0]));
    el = lane == 0 ? across : el;
    er = lane == 63 ? across : er;
    decltype(A::step(x[0], el, er, k)) d[P];  // cells moved
    edge_t prev = el;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const edge_t nb = (i + 1 < P) ? A::edge(x[i + 1 < P ? i + 1 : i]) : er;
      const edge_t old = A::edge(x[i]);
      d[i] = A::step(x[i], prev, nb, k);
      prev = old;
    }
    mine[(par ^ 1) * kOther] = A::edge(lane == 63 ? x[P - 1] : x[0]);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (__ballot(d[i] != 0) == 0u) continue;
      const bool up = d[i] == 1;
      if (__ballot(up && ahead[i] == 0) != 0u) {
        if (ahead[i] < kSpare) {
          const int32_t m = node_after(A::cell(x[i], cbase), (up ? A::kHigh : A::kHigh + 1) + ahead[i]);
          const node_t nd = A::node((uint32_t)col[i], m, id, ph);
          s_ahead[m & (kSpare - 1)][i * kBlock + tid] = nd;
          if (ahead[i] == 0) next[i] = nd;
          ahead[i] += 1;
        }
      }
      if (up) {
        x[i].w.push_up(next[i]);
        A::coef(x[i], k);
        ahead[i] -= 1;
        next[i] = s_ahead[node_after(A::cell(x[i], cbase), A::kHigh + 1) & (kSpare - 1)][i * kBlock + tid];
      }
      const bool other = d[i] != 0 && !up;
      // Backwards, or more than one cell: the whole window.  Rare on lines that
      // move forward; the main path of the kinds whose force jumps, whose sites hop
      // between two cells, and of lines under a negative drive, for which the rules
      // of the geometry therefore end the narrow tiles early.
      if (__ballot(other) != 0u) {
        if (other) {
          fresh(x[i], col[i]);
          A::coef(x[i], k);
          ahead[i] = 0;
        }
      }
    }
    __syncthreads();
  };
  int sub = 0;
  for (; sub + 2 <= nsub; sub += 2) {
    substep(0);
    substep(1);
  }
  if (sub < nsub) substep(0);

  // Write the valid part: tile-local q in [halo, halo + len).
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int q = tid * P + i;
    if (q >= halo && q < halo + len) A::store(out, base + p0 - halo + q, x[i], cbase);
  }
}

// ---------------------------------------------------------------------------
// Measurement partials (Eqs. (3)-(5)) of the state at one step.
// ---------------------------------------------------------------------------
template <int KIND, int MODE>
__global__ void __launch_bounds__(meas_block(MODE))
    k_meas_plain(Tables t, const double* __restrict__ u, Phys ph, MeasOut o) {
  __shared__ MeasLds lds;
  const TileOf w = tile_of<MODE>(t);
  const int s = w.s;
  const int p0 = w.valid ? t.mt_p0[w.tile] : 0, len = w.valid ? t.mt_len[w.tile] : 0;
  const int L = t.L[s];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const double f = t.f[s];
  const PlainPhys pp{ph.c, ph.dt, ph.strength};
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  const double K = u[base + p0];  // shift: the tile's first site (exactly 0 for a flat tile)
  double sf = 0.0, s1 = 0.0, s2 = 0.0;
  for (int q = w.tid; q < len; q += kBlock) {
    const int j = p0 + q;
    const int jm = (j == 0) ? L - 1 : j - 1;
    const int jp = (j == L - 1) ? 0 : j + 1;
    const double uj = u[base + j];
    sf += plain_force<KIND>(u[base + jm], uj, u[base + jp], (uint32_t)j, id, keys, f, ph.period,
                            pp);
    const double x = uj - K;
    s1 += x;
    s2 += x * x;
  }
  emit<MODE>(t, o, w, len, sf, s1, s2, K, lds);
}

template <int KIND, int MODE>
__global__ void __launch_bounds__(meas_block(MODE)) k_meas_split(Tables t, SplitBuf b, Phys ph, MeasOut o) {
  __shared__ MeasLds lds;
  const TileOf w = tile_of<MODE>(t);
  const int s = w.s;
  const int p0 = w.valid ? t.mt_p0[w.tile] : 0, len = w.valid ? t.mt_len[w.tile] : 0;
  const int L = t.L[s];
  const int64_t base = t.off[s];
  const uint32_t id = t.did[s];
  const float f = t.f32[s];
  const SplitPhys sp{ph.cf, ph.dtf, ph.sgn_strf};
  const int32_t Kc = b.cell[base + p0];  // shift: the tile's first site
  const double Kr = (double)b.frac[base + p0];
  const VectorKeys keys = vector_keys(ph.k0, ph.k1);
  double sf = 0.0, s1 = 0.0, s2 = 0.0;
  for (int q = w.tid; q < len; q += kBlock) {
    const int j = p0 + q;
    const int jm = (j == 0) ? L - 1 : j - 1;
    const int jp = (j == L - 1) ? 0 : j + 1;
    const int32_t c = b.cell[base + j];
    const float r = b.frac[base + j];
    float n0, n1, n2, n3;
    if (b.nodes) {  // the node cache of the fused path holds the same four values
      const float4 nd = b.nodes[base + j];
      n0 = nd.x;
      n1 = nd.y;
      n2 = nd.z;
      n3 = nd.w;
    } else {
      nodes_of<KIND>((uint32_t)j, c, id, ph, keys, n0, n1, n2, n3);
    }
    const float4 a = spline_coef<KIND>(n0, n1, n2, n3, sp.sgn_str, f);
    const float F = split_force<KIND>(c, r, b.cell[base + jm], b.frac[base + jm], b.cell[base + jp],
                                      b.frac[base + jp], a, sp.c);
    sf += (double)F;
    const double x = (double)(c - Kc) + ((double)r - Kr);  // exact
    s1 += x;
    s2 += x * x;
  }
  emit<MODE>(t, o, w, len, sf, s1, s2, (double)Kc + Kr, lds);
}

// Per-sample combine of tile partials (more than kFinalTiles of them).
__global__ void __launch_bounds__(kBlock)
    k_meas_final(Tables t, MeasOut o) {
  __shared__ Moments lds[kBlock];
  const int s = blockIdx.x;
  const int t0 = t.mt_first[s], t1 = t.mt_first[s + 1];
  Moments acc{0.0, 0.0, 0.0, 0.0};
  for (int ti = t0 + threadIdx.x; ti < t1; ti += kBlock) {
    acc = combine(acc, moments_of(o.part[ti], t.mt_len[ti]));
  }
  lds[threadIdx.x] = acc;
  __syncthreads();
  for (int stride = kBlock / 2; stride >= 1; stride >>= 1) {
    if ((int)threadIdx.x < stride) lds[threadIdx.x] = combine(lds[threadIdx.x], lds[threadIdx.x + stride]);
    __syncthreads();
  }
  if (threadIdx.x == 0) write_series(t, o, s, lds[0]);
}

// Disorder average over samples of one measurement index per workgroup:
// two passes (mean, then squared deviations) in a fixed order.
__device__ __forceinline__ double block_sum1(double v, double* lds) {
  v = wave_sum_f64(v);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < kBlock / 64; ++i) s += lds[i];
  __syncthreads();
  return s;
}

__global__ void __launch_bounds__(kBlock)
    k_ensemble(int S, int n_meas, const double* __restrict__ series, double* __restrict__ out) {
  __shared__ double lds[kBlock / 64];
  const int mi = blockIdx.x;
  double mean[3], m2[3];
  for (int q = 0; q < 3; ++q) {
    double acc = 0.0;
    for (int s = threadIdx.x; s < S; s += kBlock) acc += series[((int64_t)s * n_meas + mi) * 3 + q];
    mean[q] = block_sum1(acc, lds) / (double)S;
    double dev = 0.0;
    for (int s = threadIdx.x; s < S; s += kBlock) {
      const double e = series[((int64_t)s * n_meas + mi) * 3 + q] - mean[q];
      dev += e * e;
    }
    m2[q] = block_sum1(dev, lds);
  }
  if (threadIdx.x == 0) {
    // series layout per sample: {v, ubar, w2}; output rows: v, se, w2, se, ubar, se, w2 about ensemble ubar
    const int src[3] = {0, 2, 1};
    for (int r = 0; r < 3; ++r) {
      const int q = src[r];
      out[(2 * r) * n_meas + mi] = mean[q];
      out[(2 * r + 1) * n_meas + mi] = S > 1 ? sqrt(m2[q] / (double)(S - 1) / (double)S) : 0.0;
    }
    out[6 * n_meas + mi] = mean[2] + m2[1] / (double)S;
  }
}

// u = cell + offset of a chain in the split state.
__global__ void __launch_bounds__(kBlock)
    k_join_split(const int32_t* __restrict__ cell, const float* __restrict__ frac, double* __restrict__ u, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) u[i] = (double)cell[i] + (double)frac[i];
}

__global__ void k_fill_i32(int* p, int64_t n, int value) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = value;
}

__global__ void k_fill_f64(double* p, int64_t n, double value) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = value;
}

// ---------------------------------------------------------------------------
// Debug kernels.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock)
    k_philox_fill(const uint4* __restrict__ ctr, uint32_t k0, uint32_t k1, uint4* __restrict__ out,
                  int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  uint4 x = ctr[i];
  philox4x32_10(x.x, x.y, x.z, x.w, k0, k1);
  out[i] = x;
}

template <int KIND>
__global__ void __launch_bounds__(kBlock)
    k_force_eval(double strength, uint32_t k0, uint32_t k1, int32_t period, int precision,
                 const uint32_t* __restrict__ did, const int32_t* __restrict__ jj,
                 const int32_t* __restrict__ cell, const double* __restrict__ frac,
                 double* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t j = (uint32_t)jj[i];
  const uint32_t id = did[i];
  if (precision == 0) {
    const double u = (double)cell[i] + frac[i];
    const double nf = floor(u);
    const int32_t c = (int32_t)nf;
    double p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = strength * node_f64<KIND>(j, c - 1 + q, id, k0, k1, period);
    out[i] = spline_f64<KIND>(p, u - nf);
  } else {
    const int32_t c = cell[i];
    const float r = (float)frac[i];
    const float p0 = node_f32<KIND>(j, c - 1, id, k0, k1, period);
    const float p1 = node_f32<KIND>(j, c, id, k0, k1, period);
    const float p2 = node_f32<KIND>(j, c + 1, id, k0, k1, period);
    const float p3 = node_f32<KIND>(j, c + 2, id, k0, k1, period);
    const float sg = kind_sign<KIND>() * (float)strength;
    out[i] = (double)spline_eval<KIND>(spline_coef<KIND>(p0, p1, p2, p3, sg, 0.0f), r);
  }
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
#define QEW_KIND_DISPATCH(kind, KERNEL, ...)                      \
  do {                                                            \
    switch (kind) {                                               \
      case kRF: hipLaunchKernelGGL(KERNEL<kRF>, __VA_ARGS__); break;       \
      case kRB: hipLaunchKernelGGL(KERNEL<kRB>, __VA_ARGS__); break;       \
      case kRBLin: hipLaunchKernelGGL(KERNEL<kRBLin>, __VA_ARGS__); break; \
      default: hipLaunchKernelGGL(KERNEL<kRFPc>, __VA_ARGS__); break;      \
    }                                                             \
  } while (0)

hipError_t launch_init_plain(const Tables& t, double* u, hipStream_t st) {
  hipLaunchKernelGGL(k_init_plain, dim3(t.n_mt), dim3(kBlock), 0, st, t, u);
  return hipGetLastError();
}

hipError_t launch_init_split(const Tables& t, SplitBuf b, const Phys& ph, int kind, bool nodes,
                             hipStream_t st) {
  QEW_KIND_DISPATCH(kind, k_init_split, dim3(t.n_mt), dim3(kBlock), 0, st, t, b, ph, nodes ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_refresh_nodes(const Tables& t, SplitBuf b, const Phys& ph, int kind,
                                hipStream_t st) {
  QEW_KIND_DISPATCH(kind, k_refresh_nodes, dim3(t.n_mt), dim3(kBlock), 0, st, t, b, ph);
  return hipGetLastError();
}

// Launch KERNEL (a template on its measuring mode) as `o` asks.
#define QEW_MEAS_LAUNCH(o, NONE, PARTIALS, FINAL, ...)                                                                  \
  do {                                                                                                                  \
    if ((o).groups > 0) hipLaunchKernelGGL(FINAL, dim3((o).n_samples), dim3(kBlock * (o).groups), 0, st, __VA_ARGS__);  \
    else if ((o).part) hipLaunchKernelGGL(PARTIALS, dim3(t.n_mt), dim3(kBlock), 0, st, __VA_ARGS__);                    \
    else hipLaunchKernelGGL(NONE, dim3(t.n_mt), dim3(kBlock), 0, st, __VA_ARGS__);                                      \
  } while (0)

template <int KIND>
static void launch_plain_kind(const Tables& t, const double* uin, double* uout, const Phys& ph,
                              const MeasOut& o, hipStream_t st) {
  QEW_MEAS_LAUNCH(o, (k_step_plain<KIND, kNoMeas>), (k_step_plain<KIND, kPartials>), (k_step_plain<KIND, kFinal>), t,
                  uin, uout, ph, o);
}

hipError_t launch_step_plain(const Tables& t, const double* uin, double* uout, const Phys& ph,
                             int kind, const MeasOut& o, hipStream_t st) {
  switch (kind) {
    case kRF: launch_plain_kind<kRF>(t, uin, uout, ph, o, st); break;
    case kRB: launch_plain_kind<kRB>(t, uin, uout, ph, o, st); break;
    case kRBLin: launch_plain_kind<kRBLin>(t, uin, uout, ph, o, st); break;
    default: launch_plain_kind<kRFPc>(t, uin, uout, ph, o, st); break;
  }
  return hipGetLastError();
}

// False: no kernel of this tile.
template <int KIND>
static bool launch_blocked_kind(const Tables& t, const double* uin, double* uout, const Phys& ph, int tile,
                                int halo, int nsub, hipStream_t st) {
  const dim3 g(t.n_ft), b(kBlock);
  constexpr int wide = blocked_wide_tile(KIND) / kBlock;
  if (tile == wide * kBlock) hipLaunchKernelGGL((k_blocked_plain<KIND, wide>), g, b, 0, st, t, uin, uout, ph, halo, nsub);
  else if (tile == 256) hipLaunchKernelGGL((k_lanes<LanesD<KIND>, 1>), g, b, 0, st, t, uin, uout, ph, halo, nsub);
  else if (KIND < kRBLin && tile == 512) {
    if constexpr (KIND < kRBLin)
      hipLaunchKernelGGL((k_lanes<LanesD<KIND>, 2>), g, b, 0, st, t, uin, uout, ph, halo, nsub);
  } else return false;
  return true;
}

hipError_t launch_blocked_plain(const Tables& t, const double* uin, double* uout, const Phys& ph, int kind,
                                int tile, int halo, int nsub, hipStream_t st) {
  bool ok = false;
  switch (kind) {
    case kRF: ok = launch_blocked_kind<kRF>(t, uin, uout, ph, tile, halo, nsub, st); break;
    case kRB: ok = launch_blocked_kind<kRB>(t, uin, uout, ph, tile, halo, nsub, st); break;
    case kRBLin: ok = launch_blocked_kind<kRBLin>(t, uin, uout, ph, tile, halo, nsub, st); break;
    default: ok = launch_blocked_kind<kRFPc>(t, uin, uout, ph, tile, halo, nsub, st); break;
  }
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

template <int KIND>
static void launch_split1_kind(const Tables& t, SplitBuf in, SplitBuf out, const Phys& ph,
                               const MeasOut& o, hipStream_t st) {
  QEW_MEAS_LAUNCH(o, (k_step_split1<KIND, kNoMeas>), (k_step_split1<KIND, kPartials>), (k_step_split1<KIND, kFinal>), t,
                  in, out, ph, o);
}

hipError_t launch_step_split1(const Tables& t, SplitBuf in, SplitBuf out, const Phys& ph, int kind,
                              const MeasOut& o, hipStream_t st) {
  switch (kind) {
    case kRF: launch_split1_kind<kRF>(t, in, out, ph, o, st); break;
    case kRB: launch_split1_kind<kRB>(t, in, out, ph, o, st); break;
    case kRBLin: launch_split1_kind<kRBLin>(t, in, out, ph, o, st); break;
    default: launch_split1_kind<kRFPc>(t, in, out, ph, o, st); break;
  }
  return hipGetLastError();
}

template <int KIND, int P>
static const void* fused_ptr() {
  return reinterpret_cast<const void*>(&k_step_fused<KIND, P, false, has_rounds(KIND, P, false)>);
}

static const void* fused_fn(int tile) {
  switch (tile) {
    case 1024: return fused_ptr<kRF, 4>();
    case 1536: return fused_ptr<kRF, 6>();
    case 2048: return fused_ptr<kRF, 8>();
    case 3072: return fused_ptr<kRF, 12>();
    default: return fused_ptr<kRF, 16>();
  }
}

int fused_max_grid(int tile) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const void* fn = fused_fn(tile);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, 0) != hipSuccess) return 0;
  if (per_cu < 1) per_cu = 1;
  return cus * per_cu;
}

bool fused_fits(int tile) {
  int dev = 0, max_lds = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return false;
  hipFuncAttributes attr{};
  const void* fn = fused_fn(tile);
  if (hipFuncGetAttributes(&attr, fn) != hipSuccess) return false;
  return (int)attr.sharedSizeBytes <= max_lds;
}

struct FusedLaunch {
  const Tables& t;
  SplitBuf in, out;
  const Phys& ph;
  int halo, nsub;
  bool rounds;
  dim3 g, b;
  hipStream_t st;
  template <int KIND, int P, bool SPARSE>
  void run() const {
    if constexpr (has_rounds(KIND, P, SPARSE)) {
      // Without interpolation a few small tiles have bursts whose rounds nobody hides:
      // 1024-site tiles, f = 0.6, us per step with rounds and without, 69 tiles 1.58,
      // 1.49, 273 1.60, 1.51, 1092 2.15, 2.16 (f = 0.2: 2.80, 2.99).
      const bool few = KIND == kRFPc && P == 4 && t.n_ft <= 512;
      if ((rounds && !few) || SPARSE) {
        hipLaunchKernelGGL((k_step_fused<KIND, P, SPARSE, true>), g, b, 0, st, t, in, out, ph, halo, nsub);
        return;
      }
    }
    if constexpr (!(SPARSE && has_rounds(KIND, P, SPARSE)))  // a sparse launch is no fast line's
      hipLaunchKernelGGL((k_step_fused<KIND, P, SPARSE, false>), g, b, 0, st, t, in, out, ph, halo, nsub);
  }
};

// False: no kernel of this tile and variant.
template <int KIND, bool SPARSE>
static bool launch_fused_kind(const Tables& t, SplitBuf in, SplitBuf out, const Phys& ph, int tile,
                              int halo, int nsub, bool rounds, dim3 g, dim3 b, hipStream_t st) {
  const FusedLaunch l{t, in, out, ph, halo, nsub, rounds, g, b, st};
  switch (tile) {
    case 256:  // narrow tiles: one workgroup per tile, no sparse variant
      if constexpr (!SPARSE) hipLaunchKernelGGL((k_lanes<LanesS<KIND>, 1>), dim3(t.n_ft), b, 0, st, t, in, out, ph, halo, nsub);
      return !SPARSE;
    case 512:  // for the spline kinds
      if constexpr (!SPARSE && KIND < kRBLin)
        hipLaunchKernelGGL((k_lanes<LanesS<KIND>, 2>), dim3(t.n_ft), b, 0, st, t, in, out, ph, halo, nsub);
      return !SPARSE && KIND < kRBLin;
    case 1024: l.template run<KIND, 4, SPARSE>(); return true;
    case 1536: l.template run<KIND, 6, SPARSE>(); return true;
    case 2048: l.template run<KIND, 8, SPARSE>(); return true;
    case 3072: l.template run<KIND, 12, SPARSE>(); return true;
    case 4096: l.template run<KIND, 16, SPARSE>(); return true;
    default: return false;
  }
}

template <bool SPARSE>
static bool launch_fused_variant(const Tables& t, SplitBuf in, SplitBuf out, const Phys& ph, int kind,
                                 int tile, int halo, int nsub, bool rounds, dim3 g, dim3 b, hipStream_t st) {
  switch (kind) {
    case kRF: return launch_fused_kind<kRF, SPARSE>(t, in, out, ph, tile, halo, nsub, rounds, g, b, st);
    case kRB: return launch_fused_kind<kRB, SPARSE>(t, in, out, ph, tile, halo, nsub, rounds, g, b, st);
    case kRBLin: return launch_fused_kind<kRBLin, SPARSE>(t, in, out, ph, tile, halo, nsub, rounds, g, b, st);
    default: return launch_fused_kind<kRFPc, SPARSE>(t, in, out, ph, tile, halo, nsub, rounds, g, b, st);
  }
}

hipError_t launch_step_fused(const Tables& t, SplitBuf in, SplitBuf out, const Phys& ph, int kind,
                             int tile, int halo, int nsub, int grid, bool sparse, bool rounds, hipStream_t st) {
  const dim3 g(grid), b(kBlock);
  const bool ok = sparse ? launch_fused_variant<true>(t, in, out, ph, kind, tile, halo, nsub, rounds, g, b, st)
                         : launch_fused_variant<false>(t, in, out, ph, kind, tile, halo, nsub, rounds, g, b, st);
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

template <int KIND>
static void launch_meas_plain_kind(const Tables& t, const double* u, const Phys& ph, const MeasOut& o, hipStream_t st) {
  QEW_MEAS_LAUNCH(o, (k_meas_plain<KIND, kPartials>), (k_meas_plain<KIND, kPartials>), (k_meas_plain<KIND, kFinal>), t, u,
                  ph, o);
}

hipError_t launch_meas_plain(const Tables& t, const double* u, const Phys& ph, int kind,
                             const MeasOut& o, hipStream_t st) {
  switch (kind) {
    case kRF: launch_meas_plain_kind<kRF>(t, u, ph, o, st); break;
    case kRB: launch_meas_plain_kind<kRB>(t, u, ph, o, st); break;
    case kRBLin: launch_meas_plain_kind<kRBLin>(t, u, ph, o, st); break;
    default: launch_meas_plain_kind<kRFPc>(t, u, ph, o, st); break;
  }
  return hipGetLastError();
}

template <int KIND>
static void launch_meas_split_kind(const Tables& t, SplitBuf b, const Phys& ph, const MeasOut& o, hipStream_t st) {
  QEW_MEAS_LAUNCH(o, (k_meas_split<KIND, kPartials>), (k_meas_split<KIND, kPartials>), (k_meas_split<KIND, kFinal>), t, b,
                  ph, o);
}

hipError_t launch_meas_split(const Tables& t, SplitBuf b, const Phys& ph, int kind, const MeasOut& o,
                             hipStream_t st) {
  switch (kind) {
    case kRF: launch_meas_split_kind<kRF>(t, b, ph, o, st); break;
    case kRB: launch_meas_split_kind<kRB>(t, b, ph, o, st); break;
    case kRBLin: launch_meas_split_kind<kRBLin>(t, b, ph, o, st); break;
    default: launch_meas_split_kind<kRFPc>(t, b, ph, o, st); break;
  }
  return hipGetLastError();
}

hipError_t launch_meas_final(const Tables& t, const MeasOut& o, hipStream_t st) {
  hipLaunchKernelGGL(k_meas_final, dim3(o.n_samples), dim3(kBlock), 0, st, t, o);
  return hipGetLastError();
}

hipError_t launch_ensemble(int n_samples, int n_meas, const double* series, double* out,
                           hipStream_t st) {
  if (n_meas <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ensemble, dim3(n_meas), dim3(kBlock), 0, st, n_samples, n_meas, series, out);
  return hipGetLastError();
}

hipError_t launch_join_split(const int32_t* cell, const float* frac, double* u, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_join_split, dim3((uint32_t)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, cell, frac, u, n);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int* p, int64_t n, int value, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((uint32_t)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, p, n,
                     value);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, int64_t n, double value, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f64, dim3((uint32_t)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, p, n,
                     value);
  return hipGetLastError();
}

hipError_t launch_philox_fill(const uint32_t* ctr, uint32_t k0, uint32_t k1, uint32_t* out,
                              int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_philox_fill, dim3((uint32_t)blocks), dim3(kBlock), 0, st,
                     reinterpret_cast<const uint4*>(ctr), k0, k1, reinterpret_cast<uint4*>(out), n);
  return hipGetLastError();
}

hipError_t launch_force_eval(int kind, double strength, uint32_t k0, uint32_t k1, int32_t period,
                             int precision, const uint32_t* did, const int32_t* j,
                             const int32_t* cell, const double* frac, double* out, int64_t n,
                             hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + kBlock - 1) / kBlock;
  QEW_KIND_DISPATCH(kind, k_force_eval, dim3((uint32_t)blocks), dim3(kBlock), 0, st, strength, k0, k1,
                    period, precision, did, j, cell, frac, out, n);
  return hipGetLastError();
}

}  // namespace qew
