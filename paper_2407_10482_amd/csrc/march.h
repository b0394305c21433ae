// Per-ray march over the sample lattice with the occupancy distance grid
// (Sec. 4.3, Eq. 9), shared by the forward and backward kernels.
//
// Box domain: lattice t_k = t0 + k*step inside the cube ROI; a grid read
// returning G = g > 0 proves the next floor(g * (voxel/step) / |d|) - 1
// lattice points empty (they lie within g voxels of the read point, less
// one step), so the march jumps over them without reading.
// Contracted domain: lattice of equal contracted arc length,
// t_{k+1} = t_k + step / |J(x_k) d|, in the image of the contraction
// x -> (2 - 1/|x|) x/|x| (|x| > 1); a read with g > 0 opens a known-empty
// ball of radius g*voxel - voxel/1024 around the read point, and lattice
// points inside it are visited without a read.  Either way the sampled
// lattice points are exactly those an exhaustive occupancy march samples.
#pragma once

#include <type_traits>

#include "device.h"

namespace ngprt {

struct MarchState {
  float o[3], d[3];
  float t0, t1;       // box: entry/exit
  float t;            // contract: current lattice t
  float rho;          // box: (vox/step)/|d|
  float dn, dn2;      // |d|, |d|^2
  float dt_in;        // contract: step / |d|, the lattice spacing inside the unit ball
  int k;              // lattice index of the next point to visit
  float bc[3], br2;   // contract: known-empty ball, centre and squared radius (< 0: none)
  float t_lo;         // optional start: contract: lattice points with t < t_lo are not read
                      // (box: the caller sets k to the first lattice point at or after it)
  float t_hi;         // optional end: a lattice point with t > t_hi stops the march
  bool stopped_at_hi; // the march ended at t_hi (and can be resumed)
  bool done;
};

template <int DOM>
__device__ __forceinline__ void march_init(const SceneArgs& S, const float* o, const float* d,
                                           bool in_range, MarchState& m) {
  bool valid = in_range;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    m.o[a] = in_range ? o[a] : 0.0f;
    m.d[a] = in_range ? d[a] : 0.0f;
    valid = valid && isfinite(m.o[a]) && isfinite(m.d[a]);
  }
  m.dn2 = (m.d[0] * m.d[0] + m.d[1] * m.d[1]) + m.d[2] * m.d[2];
  m.dn = sqrtf(m.dn2);
  m.k = 0;
  m.br2 = -1.0f;
  m.bc[0] = m.bc[1] = m.bc[2] = 0.0f;
  m.t = 0.0f;
  m.t_lo = -__int_as_float(0x7F800000);
  m.t_hi = __int_as_float(0x7F800000);
  m.stopped_at_hi = false;
  if (DOM == DOM_BOX) {
    const float lo = S.lo, hi = -S.lo;
    float t0 = 0.0f, t1 = __int_as_float(0x7F800000);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (m.d[a] != 0.0f) {
        float ta = (lo - m.o[a]) / m.d[a];
        float tb = (hi - m.o[a]) / m.d[a];
        t0 = fmaxf(t0, fminf(ta, tb));
        t1 = fminf(t1, fmaxf(ta, tb));
      } else {
        valid = valid && (m.o[a] >= lo) && (m.o[a] <= hi);
      }
    }
    valid = valid && (t0 < t1) && (m.dn2 > 0.0f);
    m.t0 = t0;
    m.t1 = t1;
    m.rho = S.v_over_step / m.dn;
  } else {
    valid = valid && (m.dn2 > 0.0f);
    m.dt_in = S.step / m.dn;
  }
  m.done = !valid;
}

// Grid-domain position -> grid coordinate u in [0,1]^3 and voxel index.
__device__ __forceinline__ uint32_t voxel_of(const SceneArgs& S, const float p[3], float u[3]) {
  int q[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[a] = (p[a] - S.lo) * S.inv_ext;
    int i = (int)floorf(u[a] * S.Rf);
    q[a] = i < 0 ? 0 : (i > S.R - 1 ? S.R - 1 : i);
  }
  return uint32_t(q[0]) + uint32_t(S.R) * (uint32_t(q[1]) + uint32_t(S.R) * uint32_t(q[2]));
}

// Occupancy pyramid level j: the cell of grid coordinate u, and whether it
// is empty (levels x fastest, 32 voxels per word).
__device__ __forceinline__ void pyr_cell(const float u[3], int Rj, int q[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int i = (int)floorf(u[a] * (float)Rj);
    q[a] = i < 0 ? 0 : (i > Rj - 1 ? Rj - 1 : i);
  }
}
__device__ __forceinline__ bool pyr_empty(const SceneArgs& S, int j, const float u[3]) {
  const int Rj = S.pyrR[j];
  int q[3];
  pyr_cell(u, Rj, q);
  const uint32_t w = S.pyr[j][(size_t(q[2]) * Rj + q[1]) * size_t(Rj >> 5) + size_t(q[0] >> 5)];
  return !((w >> (q[0] & 31)) & 1u);
}

// Read the voxel v of the lattice point (p, u, kcur, tcur): returns true when
// it is a sample (its voxel is occupied); otherwise moves the march past what
// the read proves empty (m.k in the box, where it is the next index already;
// the known-empty ball in the contracted domain).
// PYR: the scene marches an occupancy pyramid (S.pyr_n > 0) instead of one
// occupancy grid; a template flag so the single-grid march carries none of it.
template <int DOM, bool PYR>
__device__ __forceinline__ bool read_voxel(const SceneArgs& S, MarchState& m, bool naive, int& reads,
                                           const float p[3], const float u[3], int kcur, float tcur, uint32_t v) {
  if (PYR) {
    // multi-level occupancy (Eq. 9's s_O branch): levels coarse to fine;
    // reads counts marching points (lattice points checked), whatever the
    // number of levels read there
    ++reads;
    // the coarsest empty level decides.  The distance grid's word carries
    // it for the levels at and above the grid's resolution (one read for
    // the code and G); only when all of those are occupied are the finer
    // levels read, coarse to fine.  The exhaustive march reads level 0.
    int lev = -1;
    uint32_t word = 0;
    if (naive) {
      lev = pyr_empty(S, 0, u) ? 0 : -1;
    } else if (S.pwide) {
      word = S.pwide[v];
      // the finest level is the one below the distance grid: the word also
      // holds the voxel's 8 children there (level-0 cell = the voxel's
      // coordinates doubled plus the child offsets, exactly, since u * 2R
      // and u * R differ by a power of two)
      const uint32_t code = (word >> 9) & 7u;
      if (code) {
        lev = int(code);
      } else {
        int q0[3];
        pyr_cell(u, S.pyrR[0], q0);
        const uint32_t c = uint32_t(q0[0] & 1) | (uint32_t(q0[1] & 1) << 1) | (uint32_t(q0[2] & 1) << 2);
        lev = ((word >> (16 + c)) & 1u) ? -1 : 0;
      }
    } else {
      word = S.grid[v];
      const uint32_t code = (word >> 9) & 7u;
      if (code) {
        lev = S.pyr_jg + int(code) - 1;
      } else {
        for (int j = S.pyr_jg - 1; j >= 0; --j)
          if (pyr_empty(S, j, u)) {
            lev = j;
            break;
          }
      }
    }
    if (lev < 0) {
      if (!naive && DOM == DOM_CONTRACT) m.br2 = -1.0f;
      return true;
    }
    if (naive) return false;
    const int Rl = S.pyrR[0] >> lev;          // the resolutions halve
    int qe[3];
    pyr_cell(u, Rl, qe);
    const bool use_g = S.use_dist && Rl < S.R;
    const uint32_t g = use_g ? (word & 0xFFu) : 0u;
    // the level's voxel: powers of two throughout, so exact
    const float vj = ldexpf(S.vox, lev - S.pyr_jg);
    if (DOM == DOM_BOX) {
      float te = __int_as_float(0x7F800000);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (m.d[a] != 0.0f) {
          const float b = S.lo + (float)(qe[a] + (m.d[a] > 0.0f ? 1 : 0)) * vj;
          te = fminf(te, (b - m.o[a]) / m.d[a]);
        }
      }
      const float jo = floorf((te - tcur) / S.step);
      int jump = jo >= 1.0f ? (jo < (float)kMaxLattice ? (int)jo : kMaxLattice) : 1;
      if (use_g && g > 0) {
        const float jf = floorf((float)g * m.rho);
        const int jg = jf < (float)kMaxLattice ? (int)jf : kMaxLattice;
        jump = jg > jump ? jg : jump;
      }
      m.k = kcur + jump;
    } else {
      float r = __int_as_float(0x7F800000);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float lower = S.lo + (float)qe[a] * vj;
        const float upper = S.lo + (float)(qe[a] + 1) * vj;
        r = fminf(r, fminf(p[a] - lower, upper - p[a]));
      }
      const float margin = S.vox * 0.0009765625f;
      const float ro = r - margin;
      const float rg = (use_g && g > 0) ? (float)g * S.vox - margin : -__int_as_float(0x7F800000);
      const float rb = fmaxf(ro, rg);
      m.br2 = rb > 0.0f ? rb * rb : -1.0f;
      m.bc[0] = p[0]; m.bc[1] = p[1]; m.bc[2] = p[2];
    }
    return false;
  }
  const uint32_t word = S.grid[v];
  ++reads;
  const bool occupied = (word & 0x100u) != 0;
  const uint32_t g = word & 0xFFu;
  if (!naive) {
    if (DOM == DOM_BOX) {
      if (!occupied && g > 0) {
        const float jf = floorf((float)g * m.rho);
        const int jump = jf < (float)kMaxLattice ? (int)jf : kMaxLattice;
        m.k = kcur + (jump > 1 ? jump : 1);
      }
    } else {
      const float rb = (float)g * S.vox - S.vox * 0.0009765625f;
      m.br2 = !occupied && g > 0 ? rb * rb : -1.0f;
      m.bc[0] = p[0]; m.bc[1] = p[1]; m.bc[2] = p[2];
    }
  }
  return occupied;
}

// Contracted domain: the image p of the lattice point at tcur, the advance dt of
// t to the next one, and whether the ray ends there.
__device__ __forceinline__ void contract_point(const SceneArgs& S, const MarchState& m, float tcur, float p[3],
                                               float& dt, bool& end) {
  float x[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = m.o[a] + tcur * m.d[a];
  const float r2 = (x[0] * x[0] + x[1] * x[1]) + x[2] * x[2];
  end = end || !isfinite(r2);
  // inside the unit ball x is its own image and |J d| = |d|: the quotient
  // step / |J d| taken once per ray
  float s = 1.0f;
  dt = m.dt_in;
  if (r2 > 1.0f) {
    const float r = sqrtf(r2);
    const float inv_r = 1.0f / r;
    s = (2.0f - inv_r) * inv_r;
    const float xd = ((x[0] * m.d[0] + x[1] * m.d[1]) + x[2] * m.d[2]) * inv_r;
    end = end || (inv_r < S.step && xd >= 0.0f);
    const float perp2 = fmaxf(m.dn2 - xd * xd, 0.0f);
    const float rad = xd * (inv_r * inv_r);
    const float jn = sqrtf((s * s) * perp2 + rad * rad);
    dt = S.step / jn;
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) p[a] = s * x[a];
}

// Visit this lane's next lattice point.  Returns true with (u, ts, ks) set
// when it is a sample (its voxel is occupied); sets m.done when the ray leaves
// the domain.  Call it only while !m.done.
// A step of the contracted march is a serial chain of some 170 instructions
// that a wave executes alone or nearly so (its longest gaps are what a launch
// ends with), so it branches only where whole waves skip something: outside
// the unit ball, and where a point takes a read.  (With a branch for each of
// the ray's ends, the ball and the read's outcomes the loop was 428
// instructions where it is 274: one 1920x1080 view of the baked model with the
// pyramid 3.87 -> 3.46 ms, one 1200x800 view 4.37 -> 4.12 ms, 256x256
// contracted 1.68 -> 1.30 ms.)
// LO: honour m.t_hi and, in the contracted domain, m.t_lo (points before it are
// visited without a read).
template <int DOM, bool PYR, bool LO = false>
__device__ __forceinline__ bool march_step(const SceneArgs& S, MarchState& m, bool naive,
                                           int& reads, float u[3], float& ts, int& ks) {
  const int kcur = m.k;
  float p[3], tcur, dt = 0.0f;
  bool end = kcur >= kMaxLattice, need = true;
  if (DOM == DOM_BOX) {
    tcur = m.t0 + (float)kcur * S.step;
    end = end || !(tcur < m.t1);
#pragma unroll
    for (int a = 0; a < 3; ++a) p[a] = m.o[a] + tcur * m.d[a];
  } else {
    tcur = m.t;
    contract_point(S, m, tcur, p, dt, end);
    // points in the known-empty ball take no read
    const float e0 = p[0] - m.bc[0], e1 = p[1] - m.bc[1], e2 = p[2] - m.bc[2];
    need = !((e0 * e0 + e1 * e1) + e2 * e2 < m.br2);
    if (LO) need = need && !(tcur < m.t_lo);
  }
  // a stop at t_hi leaves the march at this point: a resumed ray visits it
  if (LO && !end && tcur > m.t_hi) {
    m.done = true;
    m.stopped_at_hi = true;
    return false;
  }
  m.done = end;
  m.k = kcur + 1;
  if (DOM == DOM_CONTRACT) m.t = tcur + dt;
  if (end || !need) return false;
  ts = tcur;
  ks = kcur;
  const uint32_t v = voxel_of(S, p, u);
  return read_voxel<DOM, PYR>(S, m, naive, reads, p, u, kcur, tcur, v);
}

// The grid coordinate of the lattice point at t: the values march_step took
// there, by the same operations.
template <int DOM>
__device__ __forceinline__ void lattice_coord(const SceneArgs& S, const MarchState& m, float t, float u[3]) {
  float x[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = m.o[a] + t * m.d[a];
  if (DOM == DOM_CONTRACT) {
    const float r2 = (x[0] * x[0] + x[1] * x[1]) + x[2] * x[2];
    if (r2 > 1.0f) {
      const float inv_r = 1.0f / sqrtf(r2);
      const float s = (2.0f - inv_r) * inv_r;
#pragma unroll
      for (int a = 0; a < 3; ++a) x[a] = s * x[a];
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) u[a] = (x[a] - S.lo) * S.inv_ext;
}

// Samples a wave's march has found ahead of their evaluation: a ring of
// kAhead entries per lane in this wave's LDS slab (entry e of lane i at
// e * 64 + i, so a wave's accesses are consecutive words; a lane touches its
// own entries only, so no barrier is needed).
//
// Why: the lanes of a wave reach their next sample after different numbers of
// lattice points, and a wave that marched every lane to its next sample before
// each evaluation paid the longest gap of the 64 rays at each of its ~16
// evaluations: on a 1920x1080 view of the contracted scene 249 march steps
// a wave on average where its longest ray takes 165, and 7,800 on the wave
// with the most silhouettes, which alone then held the launch for 6 ms.  Here
// the wave marches only while some lane has no sample at hand, and the others
// use those steps to run ahead, so gaps at different samples overlap.  A lane
// that has run ahead of its ray's termination has only spent steps the wave
// took anyway; its entries are dropped and its read count is the last
// evaluated sample's.
constexpr int kAhead = 8;

struct SampleRing {
  float* t;             // this wave's slab: kAhead * 64 lattice t
  int32_t* reads;       // grid reads of the ray up to and including the entry's
  int32_t* k;           // lattice index (NULL: not kept)
  int head, count;
};

constexpr int kRingWords = kAhead * 64;

// March until every lane that can still find a sample has one in its ring
// (or no ray of the wave goes on).  All 64 lanes must call it together.
template <int DOM, bool PYR, bool LO, bool KEEP_K>
__device__ __forceinline__ void march_ahead(const SceneArgs& S, MarchState& m, bool naive, int& reads,
                                            SampleRing& q, int lane) {
  while (__ballot(!m.done && q.count == 0) != 0) {
    if (!m.done && q.count < kAhead) {
      float u[3], ts;
      int ks;
      if (march_step<DOM, PYR, LO>(S, m, naive, reads, u, ts, ks)) {
        const int at = ((q.head + q.count) & (kAhead - 1)) * 64 + lane;
        q.t[at] = ts;
        q.reads[at] = reads;
        if (KEEP_K) q.k[at] = ks;
        ++q.count;
      }
    }
  }
}

// Rays spread over S neighbouring lanes (S = 1: a lane a ray): the lanes of a
// ray march alike and take one each of its next S samples.  Values of slot J's
// lane reach the ray's other lanes by a swizzle within the group.
template <int S, int J>
__device__ __forceinline__ float slot_value(float v) {
  static_assert(S <= 32, "a swizzle stays within 32 lanes");
  if constexpr (S == 1) return v;
  else return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), (J << 5) | (0x1F & ~(S - 1))));
}

template <int S, int J>
__device__ __forceinline__ int slot_value(int v) {
  return __float_as_int(slot_value<S, J>(__int_as_float(v)));
}

// the group's slots whose b is set, as bits 0 .. S - 1 (the whole wave calls it)
template <int S>
__device__ __forceinline__ uint32_t slot_bits(bool b, int lane) {
  if constexpr (S == 1) return b ? 1u : 0u;
  else return uint32_t(__ballot(b) >> (lane & ~(S - 1))) & ((1u << S) - 1u);
}

// f(integral_constant<int, J>) for the slots in order
template <int S, int J = 0, class F>
__device__ __forceinline__ void each_slot(F&& f) {
  f(std::integral_constant<int, J>{});
  if constexpr (J + 1 < S) each_slot<S, J + 1>(f);
}

// The next samples of the wave's 64 / S rays, one a lane, in slot order: the
// wave marches until every ray that goes on has one, then at most two turns
// more to fill the other slots (neighbouring samples are a step apart; a ray in
// a longer gap is not waited for).  Returns whether this lane has a sample.
//
// A turn takes S lattice points of a ray at once, one a lane: a march is a
// serial chain, and its grid reads (half a microsecond each) are what a small
// launch waits for.  The points' positions do not depend on the reads (box: t0
// + k step; contracted: every lane follows the ray's t through S steps), so all
// S words are requested together; the decisions are then taken in order from
// the lanes' answers: box: a read that proves a gap names the next point;
// contracted: the lanes test their points against the ball the last read
// opened.  Visits, decisions and read counts are those of one point after
// another; points beyond a gap had their word read for nothing.
// Measured against every lane marching its ray point by point (16 lanes a ray,
// 4,096 rays): 8 levels in the box 0.107 -> 0.068 ms, 16 levels contracted 0.445
// -> 0.333, baked with the pyramid 0.740 -> 0.539 contracted, 0.100 -> 0.060 in
// the box; a training step of 4,087 rays 0.443 -> 0.354 ms.
template <int DOM, bool PYR, int S>
__device__ __forceinline__ bool march_slots(const SceneArgs& A, MarchState& m, int slot, int& reads, float u[3],
                                            float& ts, int& ks, int& reads_at) {
  const int lane = threadIdx.x & 63;
  const int first = lane & ~(S - 1);                      // the ray's first lane
  int found = 0;
  bool have = false;
  for (int fill = 0;;) {
    if (__ballot(!m.done && found < S) == 0) break;
    if (__ballot(!m.done && found == 0) == 0 && ++fill > 2) break;
    if (!m.done && found < S) {
      // this lane's point, and what its read decides
      const int k = m.k + slot;
      bool end = false, ball = false;                     // ball: inside the one the turn begins with
      float p[3] = {0.f, 0.f, 0.f}, t = m.t, t_end = m.t;
      if (DOM == DOM_BOX) {
        t = m.t0 + (float)k * A.step;
        end = !(t < m.t1);
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] = m.o[a] + t * m.d[a];
      } else {
        // every lane follows the ray's t and keeps its own point
#pragma unroll 1
        for (int j = 0; j < S; ++j) {
          float pj[3], dt;
          bool ej = false;
          contract_point(A, m, t_end, pj, dt, ej);
          if (j == slot) {
            t = t_end;
            end = ej;
#pragma unroll
            for (int a = 0; a < 3; ++a) p[a] = pj[a];
          }
          t_end = t_end + dt;
        }
        const float e0 = p[0] - m.bc[0], e1 = p[1] - m.bc[1], e2 = p[2] - m.bc[2];
        ball = (e0 * e0 + e1 * e1) + e2 * e2 < m.br2;
      }
      end = end || k >= kMaxLattice;
      MarchState q = m;
      float v[3] = {0.f, 0.f, 0.f};
      bool occ = false;
      if (!end && !ball) {
        int r = 0;
        q.k = k + 1;
        const uint32_t vox = voxel_of(A, p, v);
        occ = read_voxel<DOM, PYR>(A, q, false, r, p, v, k, t, vox);
      }
      const uint32_t ends = slot_bits<S>(end, lane), occs = slot_bits<S>(occ, lane);
      const uint32_t balls = slot_bits<S>(ball && !end, lane);
      int cur = balls == 0 ? 0 : __ffs(int(~balls)) - 1;  // the first point outside the ball
      int src = -1;
      while (cur < S && found < S) {
        if ((ends >> cur) & 1u) {
          m.done = true;
          break;
        }
        // back in the turn's first ball after leaving it (another ball has
        // replaced it): not read, so the next turn begins here
        if ((balls >> cur) & 1u) break;
        ++reads;
        const int from = (first + cur) << 2;
        if ((occs >> cur) & 1u) {
          if (found == slot) {
            src = from;
            reads_at = reads;
          }
          ++found;
          m.br2 = -1.0f;
          ++cur;
        } else if (DOM == DOM_BOX) {
          cur = __builtin_amdgcn_ds_bpermute(from, q.k) - m.k;
        } else {
          m.br2 = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(q.br2)));
#pragma unroll
          for (int a = 0; a < 3; ++a)
            m.bc[a] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(q.bc[a])));
          const float e0 = p[0] - m.bc[0], e1 = p[1] - m.bc[1], e2 = p[2] - m.bc[2];
          const bool inside = (e0 * e0 + e1 * e1) + e2 * e2 < m.br2;
          const uint32_t out = slot_bits<S>(end || !inside, lane) & ~((2u << cur) - 1u);
          cur = out ? __ffs(int(out)) - 1 : S;
        }
      }
      if (src >= 0) have = true;
      // every lane's shuffle, whether it takes a sample of this turn or not
      const int at = src >= 0 ? src : lane << 2;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float x = __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v[a])));
        u[a] = src >= 0 ? x : u[a];
      }
      const float st = __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(t)));
      const int sk = __builtin_amdgcn_ds_bpermute(at, k);
      ts = src >= 0 ? st : ts;
      ks = src >= 0 ? sk : ks;
      // move on to the first point not visited
      if (DOM == DOM_CONTRACT) {
        const float tc = __int_as_float(
            __builtin_amdgcn_ds_bpermute((first + (cur < S ? cur : 0)) << 2, __float_as_int(t)));
        m.t = cur < S ? tc : t_end;
      }
      m.k += cur;
    }
  }
  return have;
}

}  // namespace ngprt
