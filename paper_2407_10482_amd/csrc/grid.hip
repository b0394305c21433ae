// Occupancy distance grid G on the GPU (Sec. 4.3, Eq. 9).
//
// G_p = min(255, floor(box-gap distance from voxel p to the nearest
// occupied voxel)), in voxel units.  The box gap to an occupied voxel q
// equals the Euclidean distance from p to the 3x3x3 block around q, so G is
// the integer square root of the squared Euclidean distance transform of the
// 26-dilated occupancy.  The transform is separable and exact in integers:
// per-row distance along x, then min over y' of f + (y - y')^2, then the
// same along z.  Distances are held up to 255 (bytes; squares in 16 bits):
// anything farther gives G = 255 whatever the other axes add.
//
// What bounds it: the line minima.  Taken plainly (a thread per x row with
// strided accesses, then a minimum over all R entries of a line per voxel, 8.6 G
// candidates at 256^3) they are 5.0 of the 5.5 ms of a 512^3 .. 32^3 pyramid
// load.  So x distances come from bit rows by leading / trailing zero counts,
// and a line's minimum is searched outwards from the voxel in groups
// (edt_line_kernel): the cost follows the distances more than R, and the load
// takes 0.26 ms.
//
// Packed grid word (uint16): low byte G, bit 8 set when the voxel is occupied.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace ngprt {

typedef unsigned short us2 __attribute__((ext_vector_type(2)));

constexpr int kFar = 255;               // distances are clamped here
constexpr int kFarSq = kFar * kFar;     // fits 16 bits
constexpr int kTileX = 64;              // x columns of a line tile; rows of the scratch are padded to it

// uint8 occupancy -> bit rows: word w of row (y, z) holds voxels 32 w .. 32 w + 31
// (x fastest; bits at or beyond R are 0).  One thread a word.
__global__ void pack_rows_kernel(const uint8_t* __restrict__ occ, uint32_t* __restrict__ bits, int R, int wpr,
                                 int64_t n_words) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n_words) return;
  const int64_t row = i / wpr;
  const int x0 = int(i - row * wpr) * 32;
  const int m = R - x0 < 32 ? R - x0 : 32;
  const uint8_t* src = occ + row * R + x0;
  uint32_t w = 0;
  for (int b = 0; b < m; ++b) w |= (src[b] != 0 ? 1u : 0u) << b;
  bits[i] = w;
}

// Distance along x to the nearest voxel of the 26-dilated occupancy, clamped
// to 255, as bytes in rows of P.  One wave a row: lane w < wpr holds dilated
// word w and, by scans over the words, the nearest set voxel before and after
// it; then each lane takes four neighbouring voxels of one word.
__global__ void __launch_bounds__(256) edt_x_kernel(const uint32_t* __restrict__ bits, uint8_t* __restrict__ dx,
                                                    int R, int wpr, int P) {
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= int64_t(R) * R) return;
  const int y = int(row % R), z = int(row / R);
  uint32_t m = 0;
  if (lane < wpr) {
    for (int dz = -1; dz <= 1; ++dz) {
      const int zz = z + dz;
      if (zz < 0 || zz >= R) continue;
      for (int dy = -1; dy <= 1; ++dy) {
        const int yy = y + dy;
        if (yy < 0 || yy >= R) continue;
        m |= bits[(int64_t(zz) * R + yy) * wpr + lane];
      }
    }
  }
  const uint32_t before = __shfl_up(m, 1, 64), after = __shfl_down(m, 1, 64);
  uint32_t w = m | (m << 1) | (m >> 1);
  if (lane > 0) w |= before >> 31;
  if (lane < 63) w |= after << 31;
  const int left_in_word = R - 32 * lane;               // voxels of this word inside the row
  if (left_in_word < 32) w = left_in_word > 0 ? (w & ((1u << left_in_word) - 1u)) : 0u;
  // the nearest set voxel in the words before and after each word (scans
  // over the row's at most 32 words)
  int last = w ? 32 * lane + 31 - __clz(int(w)) : -(kFar + 1);
  int first = w ? 32 * lane + __ffs(int(w)) - 1 : 2048;
#pragma unroll
  for (int d = 1; d < 32; d <<= 1) {
    const int p = __shfl_up(last, d, 64), q = __shfl_down(first, d, 64);
    last = lane >= d && p > last ? p : last;
    first = lane + d < 64 && q < first ? q : first;
  }
  const int last_before = __shfl_up(last, 1, 64), first_after = __shfl_down(first, 1, 64);
  // four neighbouring voxels a lane (of one word), 256 a turn
  uint8_t* dst = dx + row * P;
  for (int c = 0; 256 * c < P; ++c) {
    const int word = (8 * c + (lane >> 3)) & 63;
    const uint32_t m4 = __shfl(w, word, 64);
    int before4 = __shfl(last_before, word, 64);
    const int after4 = __shfl(first_after, word, 64);
    if (word == 0) before4 = -(kFar + 1);
    const int x0 = 256 * c + 4 * lane;
    if (x0 < P) {
      uint32_t packed = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int x = x0 + e, bit = x & 31;
        const uint32_t lo = m4 & (0xFFFFFFFFu >> (31 - bit)), hi = m4 >> bit;
        const int l = lo ? bit - (31 - __clz(int(lo))) : x - before4;
        const int r = hi ? __ffs(int(hi)) - 1 : after4 - x;
        int best = l < r ? l : r;
        best = best < kFar ? best : kFar;
        packed |= uint32_t(best) << (8 * e);
      }
      *reinterpret_cast<uint32_t*>(dst + x0) = packed;
    }
  }
}

// Occupancy pyramid, for the level codes and child bits of the packed words
// (see pyramid_word).
struct PyrLevels {
  const uint32_t* bits[kMaxPyr];
};

// Level codes of the march (Eq. 9's multi-level occupancy): for a voxel of
// the distance grid (pyramid level jg, resolution R), the coarsest level
// j >= jg whose cell holding the voxel is empty, as 1 + j - jg in bits 9-11
// of the voxel's word (0: occupied at every level >= jg).  Level j's cell is
// the voxel's coordinates shifted right by j - jg (the resolutions halve).
// With jg == 1 the finest level holds exactly the voxel's 2x2x2 children:
// wide (when given) gets the word in bits 0-15 and child (dx, dy, dz)'s
// occupancy in bit 16 + dx + 2 dy + 4 dz.
// Both voxels x, x + 1 (x even) at once: they share every word read, and above
// level jg their cell.
__device__ __forceinline__ void pyramid_words(uint32_t word[2], int x, int y, int z, int R, int jg, int nl,
                                              bool children, const PyrLevels& P) {
  uint32_t code[2] = {0, 0};
  for (int j = nl - 1; j > jg; --j) {
    const int m = j - jg, Rj = R >> m;
    const int cx = x >> m, cy = y >> m, cz = z >> m;
    const uint32_t w = P.bits[j][(size_t(cz) * Rj + cy) * size_t(Rj >> 5) + size_t(cx >> 5)];
    if (!((w >> (cx & 31)) & 1u)) {
      code[0] = code[1] = uint32_t(1 + m);
      break;
    }
  }
  // level jg's own bit is the voxel's occupied bit
#pragma unroll
  for (int e = 0; e < 2; ++e)
    word[e] |= (code[e] ? code[e] : ((word[e] & 0x100u) ? 0u : 1u)) << 9;
  if (children) {
    const int Rf = 2 * R, wpr = Rf >> 5;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int fy = 2 * y + (c & 1), fz = 2 * z + (c >> 1);
      const uint32_t w = P.bits[0][(size_t(fz) * Rf + fy) * size_t(wpr) + size_t((2 * x) >> 5)] >> ((2 * x) & 31);
      word[0] |= (w & 3u) << (16 + 2 * c);
      word[1] |= ((w >> 2) & 3u) << (16 + 2 * c);
    }
  }
}

// One line pass of the transform: out = min over the line's entries j of
// in(j) + (own - j)^2, on tiles of a whole line by TX columns staged in LDS.
// AXIS 1: lines along y of one z, in = squares of the x distances (bytes),
// out = 16-bit squares.  AXIS 2: lines along z of one y, in = the y pass's
// squares, out = the packed grid word (G = integer square root, occupied bit
// from the bit rows and, for a pyramid, level codes and the wide word).
// A lane owns two neighbouring columns, as packed 16-bit integers, and eight
// consecutive entries of the line, so a candidate entry read once from LDS
// serves 16 outputs with a saturating add (of a squared distance that is
// uniform over the wave) and a min each.  Candidates are taken in groups of
// eight by increasing distance of the groups: a group whose smallest entry
// plus the bound on the distance improves none of the wave's outputs is not
// read, and the search ends when the bound alone reaches them all.  Past the
// line's ends the edge entry is read again: its sum is then no smaller than
// the one taken at its true distance.
// Measured (512^3 .. 32^3 pyramid, 256^3 distance grid): the whole load and
// export 5,562 us with a minimum over the whole line per voxel, 1,348 us with
// an outward search entry by entry per voxel, 259 us so.
template <int AXIS, int TX, bool PYR>
__global__ void __launch_bounds__(256) edt_line_kernel(const void* __restrict__ in, uint16_t* __restrict__ out,
                                                       uint32_t* __restrict__ wide,
                                                       const uint32_t* __restrict__ bits, int R, int wpr, int P,
                                                       int jg, int nl, PyrLevels lev) {
  extern __shared__ uint32_t tile[];                    // [R][TX / 2] pairs of 16-bit squares
  constexpr int TP = TX / 2;
  const int x0 = int(blockIdx.x) * TX;
  const int other = int(blockIdx.y);                    // z (AXIS 1) or y (AXIS 2)
  const int64_t line0 = AXIS == 1 ? int64_t(other) * R : int64_t(other);   // first row of the line
  const int64_t step = AXIS == 1 ? 1 : int64_t(R);                         // rows between its entries
  int near = 0;
  if (AXIS == 1) {
    const uint8_t* src = reinterpret_cast<const uint8_t*>(in);
    for (int t = threadIdx.x; t < R * (TX / 4); t += 256) {
      const int j = t / (TX / 4), c = t - j * (TX / 4);
      const uint32_t q = *reinterpret_cast<const uint32_t*>(src + (line0 + j * step) * P + x0 + 4 * c);
      const uint32_t b0 = q & 255u, b1 = (q >> 8) & 255u, b2 = (q >> 16) & 255u, b3 = q >> 24;
      near |= (q != 0xFFFFFFFFu) ? 1 : 0;
      tile[j * TP + 2 * c] = (b0 * b0) | ((b1 * b1) << 16);
      tile[j * TP + 2 * c + 1] = (b2 * b2) | ((b3 * b3) << 16);
    }
  } else {
    const uint16_t* src = reinterpret_cast<const uint16_t*>(in);
    constexpr uint32_t far2 = uint32_t(kFarSq) | (uint32_t(kFarSq) << 16);
    for (int t = threadIdx.x; t < R * (TP / 2); t += 256) {
      const int j = t / (TP / 2), c = t - j * (TP / 2);
      const uint2 q = *reinterpret_cast<const uint2*>(src + (line0 + j * step) * P + x0 + 4 * c);
      near |= (q.x != far2 || q.y != far2) ? 1 : 0;
      tile[j * TP + 2 * c] = q.x;
      tile[j * TP + 2 * c + 1] = q.y;
    }
  }
  near = __syncthreads_or(near);                        // a tile with nothing within 255 keeps its 255^2
  const int groups = (R + 7) / 8;
  uint32_t* gmin = tile + R * TP;                       // [groups][TP] smallest entry of each group
  for (int t = threadIdx.x; t < groups * TP; t += 256) {
    const int gi = t / TP, c = t - gi * TP;
    us2 m = __builtin_bit_cast(us2, tile[8 * gi * TP + c]);
    for (int b = 1; b < 8 && 8 * gi + b < R; ++b)
      m = __builtin_elementwise_min(m, __builtin_bit_cast(us2, tile[(8 * gi + b) * TP + c]));
    gmin[t] = __builtin_bit_cast(uint32_t, m);
  }
  __syncthreads();
  const int cp = int(threadIdx.x) % TP, slot = int(threadIdx.x) / TP;
  constexpr int SLOTS = 256 / TP;
  const uint32_t* col = tile + cp;
  // every wave takes the same number of turns (the votes below need all lanes);
  // a turn past the last group repeats it and writes nothing
  for (int turn = 0; turn * SLOTS < groups; ++turn) {
    const int gi = turn * SLOTS + slot;
    const int own = gi < groups ? gi : groups - 1;
    us2 best[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int r = 8 * own + e < R ? 8 * own + e : R - 1;
      best[e] = __builtin_bit_cast(us2, col[r * TP]);
    }
    if (near) {
      us2 worst = {kFarSq, kFarSq};
      for (int D = 0; 8 * D < R + 8; ++D) {
        const int bd = D > 0 ? 8 * D - 7 : 0, bound = bd * bd;      // least distance of the groups
        const unsigned w = worst.x > worst.y ? worst.x : worst.y;
        if (__ballot(w > unsigned(bound)) == 0) break;
        const us2 bnd = {(unsigned short)bound, (unsigned short)bound};   // < 255^2 here
        for (int side = 0; side < (D > 0 ? 2 : 1); ++side) {
          const int shift = side ? -D : D;
          const int c = own + shift;
          const bool inside = c >= 0 && c < groups;
          const us2 least =
              __builtin_elementwise_add_sat(__builtin_bit_cast(us2, gmin[(inside ? c : own) * TP + cp]), bnd);
          if (__ballot(inside && (least.x < worst.x || least.y < worst.y)) == 0) continue;
          us2 v[8];
#pragma unroll
          for (int b = 0; b < 8; ++b) {
            int r = 8 * c + b;
            r = r < 0 ? 0 : (r < R ? r : R - 1);
            v[b] = __builtin_bit_cast(us2, col[r * TP]);
          }
#pragma unroll
          for (int o = -7; o <= 7; ++o) {
            const int dist = 8 * shift + o;                          // candidate minus output
            const int sq = dist * dist < 65535 ? dist * dist : 65535;
            const us2 dd = {(unsigned short)sq, (unsigned short)sq};
#pragma unroll
            for (int b = 0; b < 8; ++b) {
              const int e = b - o;
              if (e >= 0 && e < 8)
                best[e] = __builtin_elementwise_min(best[e], __builtin_elementwise_add_sat(v[b], dd));
            }
          }
          worst = best[0];
#pragma unroll
          for (int e = 1; e < 8; ++e) worst = __builtin_elementwise_max(worst, best[e]);
        }
      }
    }
    if (gi >= groups) continue;
#pragma unroll
    for (int e8 = 0; e8 < 8; ++e8) {
      const int j = 8 * gi + e8;
      if (j >= R) break;
      const int64_t row = line0 + j * step;
      if (AXIS == 1) {
        *reinterpret_cast<uint32_t*>(out + row * P + x0 + 2 * cp) = __builtin_bit_cast(uint32_t, best[e8]);
      } else {
        const int x = x0 + 2 * cp;
        if (x < R) {
          const uint32_t w = bits[row * wpr + (x >> 5)] >> (x & 31);
          uint32_t word[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            // exact floor: below 2^16 a correctly rounded square root never reaches the next integer
            const int g = (int)sqrtf((float)best[e8][e]);
            word[e] = uint32_t(g > kFar ? kFar : g) | (((w >> e) & 1u) << 8);
          }
          if (PYR) {
            // R is a multiple of 32: both columns exist and the pair is aligned
            pyramid_words(word, x, other, j, R, jg, nl, wide != nullptr, lev);
            *reinterpret_cast<uint32_t*>(out + row * R + x) = (word[0] & 0xFFFFu) | (word[1] << 16);
            if (wide) *reinterpret_cast<uint2*>(wide + row * R + x) = make_uint2(word[0], word[1]);
          } else {
            out[row * R + x] = uint16_t(word[0]);
            if (x + 1 < R) out[row * R + x + 1] = uint16_t(word[1]);
          }
        }
      }
    }
  }
}

__global__ void pack_grid_kernel(const uint8_t* __restrict__ occ, const uint8_t* __restrict__ given,
                                 uint16_t* __restrict__ grid, int64_t n) {
  const int64_t v = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (v >= n) return;
  grid[v] = uint16_t(uint32_t(given[v]) | (occ[v] ? 0x100u : 0u));
}

// VEC voxels a thread (4: out on a 4-byte boundary and n a multiple of 4)
template <int VEC>
__global__ void unpack_dist_kernel(const uint16_t* __restrict__ grid, uint8_t* __restrict__ out,
                                   int64_t n) {
  const int64_t v = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * VEC;
  if (v >= n) return;
  if constexpr (VEC == 4) {
    const uint2 q = *reinterpret_cast<const uint2*>(grid + v);
    *reinterpret_cast<uint32_t*>(out + v) =
        (q.x & 0xFFu) | ((q.x >> 8) & 0xFF00u) | ((q.y & 0xFFu) << 16) | ((q.y << 8) & 0xFF000000u);
  } else {
    out[v] = uint8_t(grid[v] & 0xFFu);
  }
}

static unsigned blocks_for(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

template <int TX, bool PYR>
static int launch_edt_lines(ngprt_ctx* ctx, const uint8_t* dx, uint16_t* sq, const uint32_t* bits, uint32_t* wide,
                            int wpr, int P, int jg, int nl, const PyrLevels& lev, hipStream_t st) {
  const int R = ctx->desc.occ_res;
  const dim3 g(unsigned(P / TX), unsigned(R));
  const size_t lds = size_t(R + (R + 7) / 8) * TX * sizeof(uint16_t);   // the tile and its groups' minima
  hipLaunchKernelGGL((edt_line_kernel<1, TX, false>), g, dim3(256), lds, st, dx, sq, nullptr, nullptr, R, wpr, P, 0,
                     0, PyrLevels{});
  int rc = check_launch(ctx, "edt_line_kernel(y)");
  if (rc) return rc;
  hipLaunchKernelGGL((edt_line_kernel<2, TX, PYR>), g, dim3(256), lds, st, sq, ctx->grid, wide, bits, R, wpr, P, jg,
                     nl, lev);
  return check_launch(ctx, "edt_line_kernel(z)");
}

// The passes over the bit rows.  dx: the x distances (bytes) in rows of P
// voxels; sq: the y pass's squares (16 bits).  A line tile takes
// R * columns * 2 bytes of LDS: 64 columns up to R = 256, 32 up to 512 and 16
// above keep it at 32 KB, so four workgroups share a CU.
static int build_from_bits(ngprt_ctx* ctx, const uint32_t* bits, int wpr, uint8_t* dx, uint16_t* sq, int P, bool pyr,
                           uint32_t* wide, int jg, const PyrLevels& lev, hipStream_t st) {
  const int R = ctx->desc.occ_res;
  hipLaunchKernelGGL(edt_x_kernel, dim3(blocks_for(int64_t(R) * R, 4)), dim3(256), 0, st, bits, dx, R, wpr, P);
  int rc = check_launch(ctx, "edt_x_kernel");
  if (rc) return rc;
  const int nl = ctx->desc.occ_levels;
#define NGPRT_EDT(TX)                                                                           \
  return pyr ? launch_edt_lines<TX, true>(ctx, dx, sq, bits, wide, wpr, P, jg, nl, lev, st)     \
             : launch_edt_lines<TX, false>(ctx, dx, sq, bits, wide, wpr, P, jg, nl, lev, st)
  if (R <= 256) NGPRT_EDT(64);
  if (R <= 512) NGPRT_EDT(32);
  NGPRT_EDT(16);
#undef NGPRT_EDT
}

static int padded_row(int R) { return (R + kTileX - 1) / kTileX * kTileX; }

int launch_build_distance(ngprt_ctx* ctx, const uint8_t* occ, const uint8_t* dist, hipStream_t st) {
  const int R = ctx->desc.occ_res;
  const int64_t n = int64_t(R) * R * R;
  if (dist) {
    hipLaunchKernelGGL(pack_grid_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, occ, dist, ctx->grid, n);
    return check_launch(ctx, "pack_grid_kernel");
  }
  const int wpr = (R + 31) / 32, P = padded_row(R);
  const int64_t rows = int64_t(R) * R;
  uint32_t* bits = nullptr;
  uint8_t* dx = nullptr;
  uint16_t* sq = nullptr;
  if (dev_malloc_async((void**)&bits, size_t(rows) * wpr * sizeof(uint32_t), st) != hipSuccess ||
      dev_malloc_async((void**)&dx, size_t(rows) * P, st) != hipSuccess ||
      dev_malloc_async((void**)&sq, size_t(rows) * P * sizeof(uint16_t), st) != hipSuccess) {
    if (bits) (void)hipFreeAsync(bits, st);
    if (dx) (void)hipFreeAsync(dx, st);
    (void)hipGetLastError();
    return fail(ctx, NGPRT_E_ALLOC, "distance grid scratch allocation failed");
  }
  hipLaunchKernelGGL(pack_rows_kernel, dim3(blocks_for(rows * wpr, 256)), dim3(256), 0, st, occ, bits, R, wpr,
                     rows * wpr);
  int rc = check_launch(ctx, "pack_rows_kernel");
  if (rc == NGPRT_OK) rc = build_from_bits(ctx, bits, wpr, dx, sq, P, false, nullptr, 0, PyrLevels{}, st);
  (void)hipFreeAsync(bits, st);
  (void)hipFreeAsync(dx, st);
  (void)hipFreeAsync(sq, st);
  return rc;
}

int launch_export_distance(ngprt_ctx* ctx, uint8_t* out, hipStream_t st) {
  const int R = ctx->desc.occ_res;
  const int64_t n = int64_t(R) * R * R;
  // 23 us a voxel a thread, 10 us four at a time (256^3)
  if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 3u) == 0)
    hipLaunchKernelGGL(unpack_dist_kernel<4>, dim3(blocks_for(n / 4, 256)), dim3(256), 0, st, ctx->grid, out, n);
  else
    hipLaunchKernelGGL(unpack_dist_kernel<1>, dim3(blocks_for(n, 256)), dim3(256), 0, st, ctx->grid, out, n);
  return check_launch(ctx, "unpack_dist_kernel");
}

// ---------------------------------------------------------------------------
// Multi-level occupancy: bit grids (x fastest, 32 voxels per word; R is a
// multiple of 32, so voxel v sits in word v >> 5 at bit v & 31).
__global__ void pyr_pack_kernel(const uint8_t* __restrict__ occ, uint32_t* __restrict__ out,
                                int64_t n_words) {
  const int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (w >= n_words) return;
  const uint8_t* src = occ + w * 32;
  uint32_t bits = 0;
  for (int i = 0; i < 32; ++i) bits |= (src[i] != 0 ? 1u : 0u) << i;
  out[w] = bits;
}

// level of resolution Rc from the level of resolution 2 Rc: a voxel is
// occupied when any of its 2x2x2 children is
__global__ void pyr_pool_kernel(const uint32_t* __restrict__ fine, uint32_t* __restrict__ coarse,
                                int Rc) {
  const int64_t wpr = Rc >> 5;                       // words per coarse row
  const int64_t n_words = int64_t(Rc) * Rc * wpr;
  const int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (w >= n_words) return;
  const int64_t xw = w % wpr;
  const int64_t y = (w / wpr) % Rc;
  const int64_t z = w / (wpr * Rc);
  const int64_t Rf = 2 * int64_t(Rc), wpr_f = Rf >> 5;
  uint64_t acc = 0;
  for (int dz = 0; dz < 2; ++dz)
    for (int dy = 0; dy < 2; ++dy) {
      const int64_t row = ((2 * z + dz) * Rf + (2 * y + dy)) * wpr_f;
      acc |= uint64_t(fine[row + 2 * xw]) | (uint64_t(fine[row + 2 * xw + 1]) << 32);
    }
  uint32_t bits = 0;
  for (int i = 0; i < 32; ++i)
    if ((acc >> (2 * i)) & 3u) bits |= 1u << i;
  coarse[w] = bits;
}

int launch_build_pyramid(ngprt_ctx* ctx, const uint8_t* occ_fine, hipStream_t st) {
  const ngprt_desc& d = ctx->desc;
  const int nl = d.occ_levels;
  for (int j = 0; j < nl; ++j) {
    if (!ctx->pyr[j]) {
      const int64_t Rj = int64_t(d.occ_fine_res) >> j;
      if (dev_malloc((void**)&ctx->pyr[j], size_t(Rj * Rj * Rj / 32) * sizeof(uint32_t)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, NGPRT_E_ALLOC, "occupancy pyramid allocation failed");
      }
    }
  }
  const int64_t nR = int64_t(d.occ_res) * d.occ_res * d.occ_res;
  if (int64_t(d.occ_fine_res) == 2 * int64_t(d.occ_res) && !ctx->pwide) {
    if (dev_malloc((void**)&ctx->pwide, size_t(nR) * sizeof(uint32_t)) != hipSuccess) {
      (void)hipGetLastError();
      return fail(ctx, NGPRT_E_ALLOC, "occupancy pyramid allocation failed");
    }
  }
  const int64_t R0 = d.occ_fine_res;
  const int64_t w0 = R0 * R0 * R0 / 32;
  hipLaunchKernelGGL(pyr_pack_kernel, dim3(blocks_for(w0, 256)), dim3(256), 0, st, occ_fine, ctx->pyr[0], w0);
  int rc = check_launch(ctx, "pyr_pack_kernel");
  for (int j = 1; j < nl && rc == NGPRT_OK; ++j) {
    const int Rc = int(R0 >> j);
    const int64_t wc = int64_t(Rc) * Rc * Rc / 32;
    hipLaunchKernelGGL(pyr_pool_kernel, dim3(blocks_for(wc, 256)), dim3(256), 0, st, ctx->pyr[j - 1],
                       ctx->pyr[j], Rc);
    rc = check_launch(ctx, "pyr_pool_kernel");
  }
  if (rc) return rc;
  // the distance grid comes from the pyramid level of its resolution
  int jg = -1;
  for (int j = 0; j < nl; ++j)
    if ((R0 >> j) == d.occ_res) jg = j;
  if (jg < 0) return fail(ctx, NGPRT_E_SHAPE, "occ_res is not a pyramid resolution");
  // the grid's resolution is a multiple of 32 here, so the level's words are
  // the transform's bit rows
  const int P = padded_row(d.occ_res);
  const int64_t rows = int64_t(d.occ_res) * d.occ_res;
  uint8_t* dx = nullptr;
  uint16_t* sq = nullptr;
  if (dev_malloc_async((void**)&dx, size_t(rows) * P, st) != hipSuccess ||
      dev_malloc_async((void**)&sq, size_t(rows) * P * sizeof(uint16_t), st) != hipSuccess) {
    if (dx) (void)hipFreeAsync(dx, st);
    (void)hipGetLastError();
    return fail(ctx, NGPRT_E_ALLOC, "pyramid scratch allocation failed");
  }
  PyrLevels lev = {};
  for (int j = 0; j < nl; ++j) lev.bits[j] = ctx->pyr[j];
  rc = build_from_bits(ctx, ctx->pyr[jg], d.occ_res / 32, dx, sq, P, true, jg == 1 ? ctx->pwide : nullptr, jg, lev,
                       st);
  (void)hipFreeAsync(dx, st);
  (void)hipFreeAsync(sq, st);
  return rc;
}

}  // namespace ngprt
