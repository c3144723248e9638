// The paper's own particle-mesh coupling (Sec. II A): density on the mesh
// nodes from the cubic spline kernel of Eq. (15) with smoothing length h,
// Eq. (9), and the quantum force on each particle by the kernel gradient,
// Eq. (14): a_i = dx^3 sum_j Q_j grad W(x_j - q_i) (dx = 1 in cell units; the
// sign makes a = -grad Q, the particle derivative of the discrete K_rho).
// About 4/3 pi h^3 nodes lie within h of a particle (180 for h = 3.5 cells).
//
// The density is summed in integers: each kernel value W (per unit particle
// mass, cells^-3, at most 8 / (pi h^3)) is rounded once to a multiple of 2^-40
// and added as an unsigned 64-bit integer, in the units of the
// cloud-in-cell deposit (one particle = 2^40), into the context's mass mesh.
// Integer sums commute, so the mesh is bitwise independent of particle order
// and scheduling (tiled or direct, run to run), the density contrast is
// formed from it by the exact subtraction of the mean (the forward z pass),
// and near-empty nodes keep their full relative precision (no sum starting
// from -1), which is what the FP64 path of the Q stencil reads there.
#include <cfloat>
#include <utility>

#include "cic.h"
#include "internal.h"

namespace fdm {

namespace {

// Cell and fraction in [0, 1) of one 32-bit position word.
struct SplinePos {
  int logn, fixed;
  float unit;   // 2^-(32 - logn)
};
__device__ __forceinline__ void cell_frac(const SplinePos& sp, uint32_t raw, int& i, float& f) {
  if (sp.fixed) {
    const int b = 32 - sp.logn;
    i = (int)(raw >> b);
    f = (float)(raw & ((1u << b) - 1u)) * sp.unit;
  } else {
    const float x = __uint_as_float(raw);
    const float fl = floorf(x);
    i = (int)fl & ((1 << sp.logn) - 1);
    f = x - fl;
  }
}
__device__ __forceinline__ void load_cell(const SplinePos& sp, const uint32_t* __restrict__ pos,
                                          int64_t np, int64_t p, int i[3], float f[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) cell_frac(sp, pos[d * np + p], i[d], f[d]);
}

// The kernel functions take s = (r / h)^2, formed by every path as the sum
// (x^2 + y^2) + z^2 of squared scaled offsets, so that all paths round alike.
__device__ __forceinline__ float scaled(int o, float f, float inv_h) {
  return ((float)o - f) * inv_h;
}
__device__ __forceinline__ float square(float v) {
#pragma clang fp contract(off)
  return v * v;
}
__device__ __forceinline__ float clamp01(float v) { return fminf(fmaxf(v, 0.0f), 1.0f); }

// W / (2 c) of Eq. (15), c = 8 / (pi h^3), as the truncated powers
// (1 - q)^3 - 4 (1/2 - q)^3 (each zero where its argument is negative), which
// equal both branches of the equation without one; zero beyond the support.
// INNER false: q >= 1/2 is known, up to the rounding of q, whose cube adds
// nothing.  q from the hardware square root (about 1 ulp).
template <bool INNER>
__device__ __forceinline__ float spline_w(float s) {
  const float q = __builtin_amdgcn_sqrtf(s);
  const float t = clamp01(1.0f - q);
  float w = t * t * t;
  if constexpr (INNER) {
    const float u = clamp01(0.5f - q);
    w = fmaf(-4.0f, u * u * u, w);
  }
  return w;
}
// -(dW/dq) / (6 c q): (1 - q)^2 / q, or 2 - 3 q for q <= 1/2 (finite at 0).
template <bool INNER>
__device__ __forceinline__ float spline_g(float s) {
  const float ri = __builtin_amdgcn_rsqf(INNER ? fmaxf(s, 0x1p-100f) : s);
  const float q = s * ri;
  const float t = clamp01(1.0f - q);
  float g = t * t * ri;
  if constexpr (INNER) g = s <= 0.25f ? fmaf(-3.0f, q, 2.0f) : g;
  return g;
}

// Integer units of a kernel value, plus the bits of 2^52: rint(w unit) lands
// in the low mantissa bits of w unit + 2^52 (doubles are one apart there);
// unit = 2 c 2^40.  One fma, rounded once, ties to even.
__device__ __forceinline__ unsigned long long spline_units(float w, double unit) {
  return (unsigned long long)__double_as_longlong(fma((double)w, unit, 0x1p52));
}
constexpr unsigned long long kUnitMask = 0x000FFFFFFFFFFFFFull;

// Nodes that any particle of a cell can reach, at compile time, for supports
// h <= H2 / 2.  Along x and y the particle's fraction is folded into
// [0, 1/2] (offset o of a folded axis is node 1 - o), along z it is in
// [0, 1); the smallest distance over the fraction's range decides.  For
// h <= 3.5 these are 256 nodes on 43 rows, of which 180 are inside on
// average; the kernel is zero on the others.  All lanes of a wave run the
// same nodes: per-particle spans visited fewer (a wave about 290 all the
// same, the longest of its lanes' spans), at 45 instructions each.
template <int H2>
struct Reach {
  static constexpr int R = (H2 + 1) / 2 - 1;   // node offsets -R .. R + 1
  static constexpr int SPAN = 2 * R + 2;
  static constexpr double fold(int o) { return o <= 0 ? -o : o - 0.5; }
  static constexpr double full(int o) { return o <= 0 ? -o : o - 1.0; }
  static constexpr bool row(int a, int b) { return 4 * (fold(a) * fold(a) + fold(b) * fold(b)) < H2 * H2; }
  static constexpr bool node(int a, int b, int c) {
    return 4 * (fold(a) * fold(a) + fold(b) * fold(b) + full(c) * full(c)) < H2 * H2;
  }
  static constexpr bool inner(int a, int b, int c) {   // can lie within h / 2
    return 16 * (fold(a) * fold(a) + fold(b) * fold(b) + full(c) * full(c)) < H2 * H2;
  }
};
template <int R, class F, int... I>
__device__ __forceinline__ void each_offset_(F&& fn, std::integer_sequence<int, I...>) {
  (fn(std::integral_constant<int, I - R>()), ...);
}
// fn(std::integral_constant<int, o>) for o = -R .. R + 1
template <int H2, class F>
__device__ __forceinline__ void each_offset(F&& fn) {
  each_offset_<Reach<H2>::R>(fn, std::make_integer_sequence<int, Reach<H2>::SPAN>());
}

// A particle's axes folded into [0, 1/2], and its squared scaled offsets.
template <int H2>
struct Folded {
  using Rc = Reach<H2>;
  bool mx, my;
  float dy[Rc::SPAN], dz[Rc::SPAN];
  float fx, inv_h;
  __device__ __forceinline__ Folded(const float f[3], float ih) : inv_h(ih) {
    mx = f[0] > 0.5f;
    my = f[1] > 0.5f;
    fx = mx ? 1.0f - f[0] : f[0];
    const float fy = my ? 1.0f - f[1] : f[1];
#pragma unroll
    for (int k = 0; k < Rc::SPAN; ++k) {
      dy[k] = scaled(k - Rc::R, fy, ih);
      dz[k] = scaled(k - Rc::R, f[2], ih);
    }
  }
  // rows(a, b, x^2 + y^2) for every row that can be reached
  template <class F>
  __device__ __forceinline__ void rows(F&& fn) const {
    each_offset<H2>([&](auto a) {
      const float dx2 = square(scaled(a.value, fx, inv_h));
      each_offset<H2>([&](auto b) {
        if constexpr (Rc::row(a.value, b.value)) fn(a, b, dx2 + square(dy[b.value + Rc::R]));
      });
    });
  }
  __device__ __forceinline__ float dz2(int c) const { return square(dz[c + Rc::R]); }
};

// Offsets o in [lo, hi] along one axis that may satisfy (o - f)^2 <= rem,
// rem being h^2 less the other axes' squared distances: the integers in
// [f - sqrt(rem), f + sqrt(rem)], widened to the enclosing integers, so that
// any error of the square root below one cell never drops a node; the nodes
// outside the support that it lets through add nothing.
__device__ __forceinline__ void axis_span(float f, float rem, int lo, int hi, int& a, int& b) {
  const float w = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f));
  a = max(lo, (int)floorf(f - w));
  b = min(hi, (int)ceilf(f + w));
}

// fn(node index, x, y, z scaled offsets, s) for the nodes around a particle at
// any h (loops over the particle's own spans).
template <class F>
__device__ __forceinline__ void each_node(int logn, const int i[3], const float f[3], float h,
                                          float inv_h, int lo, int hi, F&& fn) {
  const int mask = (1 << logn) - 1;
  const float h2 = h * h;
  for (int a = lo; a <= hi; ++a) {
    const float da = (float)a - f[0], ra = h2 - da * da;
    if (ra < 0.0f) continue;
    const float dx = scaled(a, f[0], inv_h);
    int b0, b1;
    axis_span(f[1], ra, lo, hi, b0, b1);
    for (int b = b0; b <= b1; ++b) {
      const float db = (float)b - f[1], rb = ra - db * db;
      if (rb < 0.0f) continue;
      const float dy = scaled(b, f[1], inv_h);
      const float dxy2 = square(dx) + square(dy);
      const int row = ((((i[0] + a) & mask) << logn) + ((i[1] + b) & mask)) << logn;
      int c0, c1;
      axis_span(f[2], rb, lo, hi, c0, c1);
      for (int c = c0; c <= c1; ++c) {
        const float dz = scaled(c, f[2], inv_h);
        fn(row + ((i[2] + c) & mask), dx, dy, dz, dxy2 + square(dz));
      }
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_spline_deposit(const uint32_t* __restrict__ pos,
                                                           int64_t np, SplinePos sp, float h,
                                                           float inv_h, double unit, int lo,
                                                           int hi,
                                                           unsigned long long* __restrict__ mass) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
    int i[3];
    float f[3];
    load_cell(sp, pos, np, p, i, f);
    each_node(sp.logn, i, f, h, inv_h, lo, hi, [&](int node, float, float, float, float s) {
      const unsigned long long v = spline_units(spline_w<true>(s), unit) & kUnitMask;
      if (v != 0ull) atomicAdd(&mass[node], v);
    });
  }
}

// One particle's nodes by a whole wave, for the few that left their tile
// (a lane that walks its nodes alone holds its wave for 180 of them): a lane
// takes the columns lane, lane + 64, ... of the SPAN x SPAN columns around
// the particle.  fn(node index, x, y, z scaled offsets, s).
template <int H2, class F>
__device__ __forceinline__ void each_node_wave(int logn, const int i[3], const float f[3],
                                               float inv_h, F&& fn) {
  using Rc = Reach<H2>;
  const int mask = (1 << logn) - 1;
  for (int col = threadIdx.x & 63; col < Rc::SPAN * Rc::SPAN; col += 64) {
    const int a = col / Rc::SPAN - Rc::R, b = col % Rc::SPAN - Rc::R;
    const float dx = scaled(a, f[0], inv_h), dy = scaled(b, f[1], inv_h);
    const float dxy2 = square(dx) + square(dy);
    const int row = ((((i[0] + a) & mask) << logn) + ((i[1] + b) & mask)) << logn;
#pragma unroll
    for (int k = 0; k < Rc::SPAN; ++k) {
      const float dz = scaled(k - Rc::R, f[2], inv_h);
      fn(row + ((i[2] + k - Rc::R) & mask), dx, dy, dz, dxy2 + square(dz));
    }
  }
}
// Whether a lane's particle, far from its tile, is taken by the lane itself:
// where many of a wave are, the positions are not those that were sorted (a
// second state on a sorted context, say), and one after the other they would
// take a wave each.  Those near their tile, as after some steps without a
// sort, stay with the waves.  128^3 particles in lattice order on a context
// that sorted others, h = 3.5: force 3080 -> 790 us (unsorted 409; the blocks
// are those of the sort), density 17.5 -> 11.7 ms (unsorted 11.5).  Three
// cells rms after a sort two steps take 10.5 ms, 30 with the near ones taken
// by lanes too.
constexpr int kManyFar = 16;
__device__ __forceinline__ bool by_lane(bool far) {
  return far && __popcll(__ballot(far)) > kManyFar;
}
// fn(lane, its cell, its fraction) for every lane of the wave with `which`
// set; the whole wave runs it, the arguments are uniform.
template <class F>
__device__ __forceinline__ void each_lane(bool which, const int i[3], const float f[3], F&& fn) {
  for (unsigned long long m = __ballot(which); m != 0ull; m &= m - 1) {
    const int lane = __ffsll((long long)m) - 1;
    int iu[3];
    float fu[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      iu[d] = __builtin_amdgcn_readlane(i[d], lane);
      fu[d] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f[d]), lane));
    }
    fn(lane, iu, fu);
  }
}

// Tiled form for a sorted context: a block sums the kernel values of one piece
// of a tile's particles into an LDS window covering every node they reach
// (offsets -R .. R + 1 from the tile), then adds the window's non-zero nodes
// to the mesh; particles that left their tile are taken one after the other by
// their wave, into the window where it covers a node (all but a layer or two
// of the nodes just after a tile's face) and to the mesh elsewhere: 14 steps
// after the sort of a 256^3 Zel'dovich state the deposit takes 1.58 ms, 3.21
// with every node of theirs added to the mesh (1.35 right after it).
// Each add carries the bits of 2^52 on top of its integer; they only reach
// bits 52 and up, which the flush drops: a piece's sum at a node stays below
// 2^52 (at most 3/2 kPiece particles of at most 8 / (pi h^3) < 0.32 each, in
// 2^-40).
//
// What bounds it is the kernel arithmetic (8 to 12 instructions per node) and
// the LDS adds (11 cycles per wave instruction at scattered addresses): 1.4
// ms at 256^3 with one particle per cell and h = 3.5, against 3.88 with
// per-particle spans; 10^6 particles in one object at 128^3, h = 4: 0.20
// against 0.99 ms.  512 threads per block (1.53 ms with all nodes of the
// particles out of their tile on the mesh): 256 take 1.74 ms, 1024 1.56.
constexpr int kSplineBlock = 512;
static_assert(3 * kPiece / 2 * 32 / 100 < (1u << (52 - kMassShift)), "a piece's sum at a node");
constexpr int kSplineGrid = 4096;
constexpr int kSplineH2Max = 10;   // the widest window: h <= 5
template <int H2>
__host__ __device__ constexpr int spline_window(int logn) {
  return ((1 << tile_lx(logn)) + Reach<H2>::SPAN - 1) * ((1 << tile_ly(logn)) + Reach<H2>::SPAN - 1) *
         ((1 << tile_lz(logn)) + Reach<H2>::SPAN - 1);
}

// The tile of a piece and the geometry of a window with BEFORE cells in front
// of it and E - BEFORE behind, on each axis.
template <int BEFORE, int E>
struct TileWindow {
  static constexpr int kNear = 8;
  static constexpr int WX = (1 << kTileLX) + E, WY = (1 << kTileLY) + E;
  int o[3], tz, wz;
  __device__ __forceinline__ TileWindow(int logn, int tile) {
    const int lz = tile_lz(logn), nty = logn - kTileLY, ntz = logn - lz;
    o[0] = (tile >> (nty + ntz)) << kTileLX;
    o[1] = ((tile >> ntz) & ((1 << nty) - 1)) << kTileLY;
    o[2] = (tile & ((1 << ntz) - 1)) << lz;
    tz = 1 << lz;
    wz = tz + E;
  }
  // window index of the particle's own cell, or -1 if it left the tile
  __device__ __forceinline__ int cell(int logn, const int i[3]) const {
    const int mask = (1 << logn) - 1;
    const int rx = (i[0] - o[0]) & mask, ry = (i[1] - o[1]) & mask, rz = (i[2] - o[2]) & mask;
    if (rx >= (1 << kTileLX) || ry >= (1 << kTileLY) || rz >= tz) return -1;
    return ((rx + BEFORE) * WY + ry + BEFORE) * wz + rz + BEFORE;
  }
  // whether a cell is within kNear of the tile
  __device__ __forceinline__ bool near(int logn, const int i[3]) const {
    const int mask = (1 << logn) - 1;
    return ((i[0] - o[0] + kNear) & mask) < (1 << kTileLX) + 2 * kNear &&
           ((i[1] - o[1] + kNear) & mask) < (1 << kTileLY) + 2 * kNear &&
           ((i[2] - o[2] + kNear) & mask) < tz + 2 * kNear;
  }
  // window index of a mesh node, or -1 outside the window
  __device__ __forceinline__ int node(int logn, int n) const {
    const int mask = (1 << logn) - 1;
    const int rx = ((n >> (2 * logn)) - o[0] + BEFORE) & mask;
    const int ry = ((n >> logn) - o[1] + BEFORE) & mask, rz = (n - o[2] + BEFORE) & mask;
    return rx < WX && ry < WY && rz < wz ? (rx * WY + ry) * wz + rz : -1;
  }
  // fn(window index, mesh index) for this thread's nodes of the window
  template <class F>
  __device__ __forceinline__ void each(int logn, F&& fn) const {
    const int mask = (1 << logn) - 1;
    for (int row = threadIdx.x >> 6; row < WX * WY; row += kSplineBlock / 64) {
      const int lx = row / WY, ly = row % WY;
      const int base = ((((o[0] - BEFORE + lx) & mask) << logn) +
                        ((o[1] - BEFORE + ly) & mask)) << logn;
      const int z = threadIdx.x & 63;
      if (z < wz) fn(row * wz + z, base + ((o[2] - BEFORE + z) & mask));
    }
  }
};
template <int H2>
using SplineTile = TileWindow<Reach<H2>::R, Reach<H2>::SPAN - 1>;
using GradTile = TileWindow<1, 3>;   // the nodes of interp_grad
__host__ __device__ constexpr int grad_window(int logn) {
  return GradTile::WX * GradTile::WY * ((1 << tile_lz(logn)) + 3);
}

template <int H2>
__global__ void __launch_bounds__(kSplineBlock, 4) k_spline_deposit_tiled(
    const uint32_t* __restrict__ pos, int64_t np, SplinePos sp, TileMap tm, float h, float inv_h,
    double unit, unsigned long long* __restrict__ mass) {
  using Rc = Reach<H2>;
  using Tile = SplineTile<H2>;
  extern __shared__ unsigned long long win[];
  const unsigned used = __builtin_amdgcn_readfirstlane(tm.used[1]);
  for (unsigned b = blockIdx.x; b < used; b += gridDim.x) {
    const uint4 pc = tm.pieces[b];
    const Tile tile(sp.logn, (int)__builtin_amdgcn_readfirstlane(pc.x));
    const unsigned p1 = __builtin_amdgcn_readfirstlane(pc.z);
    for (int c = threadIdx.x; c < Tile::WX * Tile::WY * tile.wz; c += kSplineBlock) win[c] = 0ull;
    __syncthreads();
    for (unsigned p = __builtin_amdgcn_readfirstlane(pc.y); p < p1; p += kSplineBlock) {
      const bool valid = p + threadIdx.x < p1;
      int i[3] = {0, 0, 0}, at = 0;
      float f[3] = {0.0f, 0.0f, 0.0f};
      if (valid) {
        load_cell(sp, pos, np, p + threadIdx.x, i, f);
        at = tile.cell(sp.logn, i);
      }
      if (valid && at >= 0) {
        const Folded<H2> fo(f, inv_h);
        const int px = Tile::WY * tile.wz, py = tile.wz;
        const int sx = fo.mx ? -px : px, sy = fo.my ? -py : py;
        const int base = at + (fo.mx ? px : 0) + (fo.my ? py : 0) - Rc::R;
        fo.rows([&](auto a, auto bb, float dxy2) {
          unsigned long long* row = win + (base + a.value * sx + bb.value * sy);
          each_offset<H2>([&](auto c) {
            if constexpr (Rc::node(a.value, bb.value, c.value)) {
              const float w =
                  spline_w<Rc::inner(a.value, bb.value, c.value)>(dxy2 + fo.dz2(c.value));
              // a third of the lanes are outside: skipping their adds of zero
              // spares the LDS (1638 -> 1527 us)
              if (w > 0.0f) atomicAdd(row + (c.value + Rc::R), spline_units(w, unit));
            }
          });
        });
      }
      const bool own = by_lane(at < 0 && !tile.near(sp.logn, i));
      if (own)
        each_node(sp.logn, i, f, h, inv_h, -Rc::R, Rc::R + 1,
                  [&](int node, float, float, float, float s) {
          const unsigned long long v = spline_units(spline_w<true>(s), unit) & kUnitMask;
          if (v != 0ull) atomicAdd(&mass[node], v);
        });
      each_lane(at < 0 && !own, i, f, [&](int, const int iu[3], const float fu[3]) {
        each_node_wave<H2>(sp.logn, iu, fu, inv_h, [&](int node, float, float, float, float s) {
          const unsigned long long v = spline_units(spline_w<true>(s), unit) & kUnitMask;
          const int w = tile.node(sp.logn, node);
          if (v == 0ull) return;
          if (w >= 0)
            atomicAdd(win + w, v);
          else
            atomicAdd(&mass[node], v);
        });
      });
    }
    __syncthreads();
    tile.each(sp.logn, [&](int w, int node) {
      const unsigned long long v = win[w] & kUnitMask;
      if (v != 0ull) atomicAdd(&mass[node], v);
    });
    __syncthreads();
  }
}

// Force of one particle from its rows: at(a, b) gives an accessor of Q along
// the row, at offsets c from the particle's cell.  Nodes of the reach beyond
// the support and the node that the particle sits on enter as Q times zero: a
// force that is not finite has to be taken again from its own spans, where
// they stay out (checking each product instead costs a tenth of the kernel).
template <int H2, class At>
__device__ __forceinline__ void force_rows(const Folded<H2>& fo, At&& at, float g[3]) {
  using Rc = Reach<H2>;
  float gx = 0.0f, gy = 0.0f, gz = 0.0f;
  fo.rows([&](auto a, auto b, float dxy2) {
    auto q = at(a, b);
    float sum = 0.0f;
    each_offset<H2>([&](auto c) {
      if constexpr (Rc::node(a.value, b.value, c.value)) {
        const float v =
            q(c.value) * spline_g<Rc::inner(a.value, b.value, c.value)>(dxy2 + fo.dz2(c.value));
        sum += v;
        gz = fmaf(v, fo.dz[c.value + Rc::R], gz);
      }
    });
    gx = fmaf(sum, scaled(a.value, fo.fx, fo.inv_h), gx);
    gy = fmaf(sum, fo.dy[b.value + Rc::R], gy);
  });
  g[0] = fo.mx ? -gx : gx;
  g[1] = fo.my ? -gy : gy;
  g[2] = gz;
}

// Force of one particle from its own spans, Q read from the mesh and only
// inside the support (r = 0 adds nothing).
__device__ __forceinline__ void own_force(int logn, const int i[3], const float f[3], float h,
                                          float inv_h, int lo, int hi,
                                          const float* __restrict__ qmesh, float g[3]) {
  g[0] = g[1] = g[2] = 0.0f;
  each_node(logn, i, f, h, inv_h, lo, hi, [&](int node, float x, float y, float z, float s) {
    float q = 0.0f;
    if (!(s > 1.0f || s == 0.0f))
      q = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(qmesh) +
                                          ((uint32_t)node << 2));
    const float v = q * spline_g<true>(s);
    g[0] = fmaf(v, x, g[0]);
    g[1] = fmaf(v, y, g[1]);
    g[2] = fmaf(v, z, g[2]);
  });
}

// (The sums are made opaque first: seen through, the check has the compiler
// keep the operands of every term, thousands of bytes of scratch per lane.)
__device__ __forceinline__ bool all_finite(float (&g)[3]) {
  asm volatile("" : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]));
  return fabsf(g[0]) <= FLT_MAX && fabsf(g[1]) <= FLT_MAX && fabsf(g[2]) <= FLT_MAX;
}

// Any particle order, any h.
__global__ void __launch_bounds__(kBlock) k_spline_qforce(const uint32_t* __restrict__ pos,
                                                          int64_t np, SplinePos sp,
                                                          const float* __restrict__ qmesh, float h,
                                                          float inv_h, float coef, int lo, int hi,
                                                          float* __restrict__ acc) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
    int i[3];
    float f[3], g[3];
    load_cell(sp, pos, np, p, i, f);
    own_force(sp.logn, i, f, h, inv_h, lo, hi, qmesh, g);
#pragma unroll
    for (int d = 0; d < 3; ++d) acc[d * np + p] = coef * g[d];
  }
}

// The nodes of the reach at compile time, Q read from the mesh (any particle
// order).
template <int H2>
__global__ void __launch_bounds__(kBlock) k_spline_qforce_fixed_reach(
    const uint32_t* __restrict__ pos, int64_t np, SplinePos sp, const float* __restrict__ qmesh,
    float h, float inv_h, float coef, float* __restrict__ acc) {
  using Rc = Reach<H2>;
  const int mask = (1 << sp.logn) - 1;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
    int i[3];
    float f[3], g[3];
    load_cell(sp, pos, np, p, i, f);
    const Folded<H2> fo(f, inv_h);
    uint32_t yo[Rc::SPAN], zo[Rc::SPAN];
#pragma unroll
    for (int k = 0; k < Rc::SPAN; ++k) {
      const int o = k - Rc::R;
      yo[k] = (uint32_t)((i[1] + (fo.my ? 1 - o : o)) & mask) << (sp.logn + 2);
      zo[k] = (uint32_t)((i[2] + o) & mask) << 2;
    }
    force_rows<H2>(fo, [&](auto a, auto b) {
      const uint32_t row = ((uint32_t)((i[0] + (fo.mx ? 1 - a.value : a.value)) & mask)
                            << (2 * sp.logn + 2)) | yo[b.value + Rc::R];
      return [=, &zo](int c) {
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(qmesh) +
                                               (row | zo[c + Rc::R]));
      };
    }, g);
    if (!all_finite(g)) own_force(sp.logn, i, f, h, inv_h, -Rc::R, Rc::R + 1, qmesh, g);
#pragma unroll
    for (int d = 0; d < 3; ++d) acc[d * np + p] = coef * g[d];
  }
}

// One particle's force by a whole wave, as each_node_wave (the lanes' sums w
// are still to be added up): Q is loaded inside the support only, and all of a
// column's nodes before the first is used.
template <int H2>
__device__ __forceinline__ void wave_force(int logn, const int i[3], const float f[3],
                                           float inv_h, const float* __restrict__ qmesh,
                                           float w[3]) {
  using Rc = Reach<H2>;
  const int mask = (1 << logn) - 1;
  w[0] = w[1] = w[2] = 0.0f;
  for (int col = threadIdx.x & 63; col < Rc::SPAN * Rc::SPAN; col += 64) {
    const int a = col / Rc::SPAN - Rc::R, b = col % Rc::SPAN - Rc::R;
    const float dx = scaled(a, f[0], inv_h), dy = scaled(b, f[1], inv_h);
    const float dxy2 = square(dx) + square(dy);
    const int row = ((((i[0] + a) & mask) << logn) + ((i[1] + b) & mask)) << logn;
    float q[Rc::SPAN];
#pragma unroll
    for (int k = 0; k < Rc::SPAN; ++k) {
      const float s = dxy2 + square(scaled(k - Rc::R, f[2], inv_h));
      q[k] = 0.0f;
      if (s <= 1.0f && s != 0.0f) q[k] = qmesh[row + ((i[2] + k - Rc::R) & mask)];
    }
#pragma unroll
    for (int k = 0; k < Rc::SPAN; ++k) {
      const float dz = scaled(k - Rc::R, f[2], inv_h);
      const float t = q[k] * spline_g<true>(dxy2 + square(dz));
      w[0] = fmaf(t, dx, w[0]);
      w[1] = fmaf(t, dy, w[1]);
      w[2] = fmaf(t, dz, w[2]);
    }
  }
}

// The factors of one pass of the spline step over the particles: the closing
// half-kick of the previous step, the opening one of the next and its drift.
struct SplineStep {
  float* vel;
  const float* phi;
  float cg, cq, og, oq;
  double fd;
  int close, open;
};

// v += fg g_phi + fq g_q, and the drift of one coordinate word: fixed point,
// the displacement rounded to the nearest unit, 32-bit wrap; float, wrapped
// into [0, N).
__device__ __forceinline__ float spline_kick(float v, float gphi, float gq, float fg, float fq) {
  return fmaf(fq, gq, fmaf(fg, gphi, v));
}
__device__ __forceinline__ uint32_t spline_drift(const SplinePos& sp, uint32_t raw, float v,
                                                 double fd) {
  if (sp.fixed) {
    const double units = (double)v * fd * (double)(1ull << (32 - sp.logn));
    return raw + (uint32_t)(int64_t)llrint(units);
  }
  const float n = (float)(1 << sp.logn);
  float x = fmaf((float)fd, v, __uint_as_float(raw));
  x -= n * floorf(x * (1.0f / n));
  return __float_as_uint(x >= n ? 0.0f : x);
}

// Sorted context: Q of the piece's window staged in LDS.  Bound by its
// arithmetic (11 to 14 instructions per node): 1.18 ms at 256^3 with one
// particle per cell and h = 3.5, against 2.98 with per-particle spans and Q
// read from the mesh; 10^6 particles in one object at 128^3: 0.17 against
// 0.45 ms.
// STEP: also -grad phi from its own window, the kicks and the drift, so that
// the particles' traffic (60 bytes each) runs under the arithmetic
// (256^3, h = 3.5: 1.48 ms in place of 1.18 and 0.54 for the separate passes).
// Waves per SIMD, which set the register budget: four blocks per CU for the
// force up to h = 3.5, three for the step up to h = 2.5 (held to 80 registers;
// at 86, two blocks, two steps at 128^3 and h = 2 take 541 us instead of 520),
// two where the windows leave no room for more.
constexpr int force_waves(int h2, bool step) { return step ? (h2 <= 5 ? 6 : 5) : h2 <= 7 ? 8 : 5; }
template <int H2, bool STEP>
__global__ void __launch_bounds__(kSplineBlock, force_waves(H2, STEP)) k_spline_qforce_tiled(
    uint32_t* __restrict__ pos, int64_t np, SplinePos sp, TileMap tm,
    const float* __restrict__ qmesh, float h, float inv_h, float coef, float* __restrict__ acc,
    SplineStep st) {
  using Tile = SplineTile<H2>;
  extern __shared__ float qwin[];
  float* pwin = qwin + spline_window<H2>(sp.logn);
  const unsigned used = __builtin_amdgcn_readfirstlane(tm.used[1]);
  for (unsigned b = blockIdx.x; b < used; b += gridDim.x) {
    const uint4 pc = tm.pieces[b];
    const Tile tile(sp.logn, (int)__builtin_amdgcn_readfirstlane(pc.x));
    const GradTile gtile(sp.logn, (int)__builtin_amdgcn_readfirstlane(pc.x));
    const unsigned p1 = __builtin_amdgcn_readfirstlane(pc.z);
    tile.each(sp.logn, [&](int w, int node) { qwin[w] = qmesh[node]; });
    if constexpr (STEP) gtile.each(sp.logn, [&](int w, int node) { pwin[w] = st.phi[node]; });
    __syncthreads();
    for (unsigned p = __builtin_amdgcn_readfirstlane(pc.y); p < p1; p += kSplineBlock) {
      const bool valid = p + threadIdx.x < p1;
      int i[3] = {0, 0, 0}, at = 0;
      float f[3] = {0.0f, 0.0f, 0.0f}, g[3], gp[3], v[3];
      if (valid) {
        load_cell(sp, pos, np, p + threadIdx.x, i, f);
        at = tile.cell(sp.logn, i);
        if constexpr (STEP) {
          const int gat = gtile.cell(sp.logn, i) - (GradTile::WY + 1) * gtile.wz - 1;
          const int mask = (1 << sp.logn) - 1;
          if (at >= 0)
            interp_grad(f, [&](int a, int bb, int c) {
              return pwin[gat + (a * GradTile::WY + bb) * gtile.wz + c];
            }, gp);
          else
            interp_grad(f, [&](int a, int bb, int c) {
              return st.phi[((((((i[0] + a - 1) & mask) << sp.logn) + ((i[1] + bb - 1) & mask))
                              << sp.logn)) + ((i[2] + c - 1) & mask)];
            }, gp);
#pragma unroll
          for (int d = 0; d < 3; ++d) v[d] = st.vel[d * np + p + threadIdx.x];
        }
      }
      const bool lane_own = by_lane(at < 0 && !tile.near(sp.logn, i));
      bool own = lane_own;
      if (valid && at >= 0) {
        const Folded<H2> fo(f, inv_h);
        const int px = Tile::WY * tile.wz, py = tile.wz;
        const int sx = fo.mx ? -px : px, sy = fo.my ? -py : py;
        const int base = at + (fo.mx ? px : 0) + (fo.my ? py : 0) - Reach<H2>::R;
        force_rows<H2>(fo, [&](auto a, auto bb) {
          const float* row = qwin + (base + a.value * sx + bb.value * sy);
          return [row](int c) { return row[c + Reach<H2>::R]; };
        }, g);
        own = !all_finite(g);
      }
      if (own) own_force(sp.logn, i, f, h, inv_h, -Reach<H2>::R, Reach<H2>::R + 1, qmesh, g);
      each_lane(at < 0 && !lane_own, i, f, [&](int lane, const int iu[3], const float fu[3]) {
        float w[3];
        wave_force<H2>(sp.logn, iu, fu, inv_h, qmesh, w);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          for (int off = 32; off > 0; off >>= 1) w[d] += __shfl_xor(w[d], off, 64);
          if ((int)(threadIdx.x & 63) == lane) g[d] = w[d];
        }
      });
      if (valid) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int64_t k = d * np + p + threadIdx.x;
          const float gq = coef * g[d];
          if constexpr (STEP) {
            if (st.close) v[d] = spline_kick(v[d], gp[d], gq, st.cg, st.cq);
            if (st.open) {
              v[d] = spline_kick(v[d], gp[d], gq, st.og, st.oq);
              pos[k] = spline_drift(sp, pos[k], v[d], st.fd);
            }
            st.vel[k] = v[d];
          } else {
            acc[k] = gq;
          }
        }
      }
    }
    __syncthreads();
  }
}

// Half-kick of the spline step: v += fg g_phi + fq g_q, arrays [3][np].
__global__ void __launch_bounds__(kBlock) k_spline_kick(float* __restrict__ vel,
                                                        const float* __restrict__ gphi,
                                                        const float* __restrict__ gq, int64_t n,
                                                        float fg, float fq) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    vel[i] = spline_kick(vel[i], gphi[i], gq[i], fg, fq);
}

// Drift of the spline step: x += fd v, periodic.
__global__ void __launch_bounds__(kBlock) k_spline_drift(uint32_t* __restrict__ pos,
                                                         const float* __restrict__ vel,
                                                         int64_t n, SplinePos sp, double fd) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    pos[i] = spline_drift(sp, pos[i], vel[i], fd);
}

unsigned spline_grid(int64_t n) {
  int64_t b = (n + kBlock - 1) / kBlock;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return (unsigned)b;
}

// Node offsets from the particle's cell that can lie within h: the node
// j = i + o is within reach when |o - f| <= h for some f in [0, 1).
void spline_range(float h, int& lo, int& hi) {
  lo = -(int)floorf(h);
  hi = (int)floorf(h) + 1;
}

SplinePos spline_pos(bool fixed, int logn) {
  SplinePos sp;
  sp.logn = logn;
  sp.fixed = fixed;
  sp.unit = ldexpf(1.0f, logn - 32);
  return sp;
}

// Up to this many particles, too few to hide the latency of the own spans'
// loops, a force in any order takes all nodes of the reach (h up to 5 cells):
// 32768 at 32^3 20 to 29 us, own spans 55 to 63.  Beyond, the loads bound it
// and the own spans have fewer: 2^17 at 64^3, h = 3.5, in lattice order,
// random order and clumps 57, 98 and 96 us (reach 35, 112, 112; h = 3.01: 39,
// 66, 65 against 35, 112, 112), 128^3 particles 421, 1928, 1623 against 544,
// 2802, 2293.
constexpr int64_t kReachMax = 1 << 16;
// Tiles in the order of a sort.  Each costs its window, whatever it holds; up
// to four per CU that is one round of blocks, beyond it takes enough particles
// to share it.  At 256^3 (8192 tiles; lattice and random order, in us):
//   force, h = 3.5:   2^17 particles 163, 164 (spans 106, 129),
//                     2^18 162, 162 (173, 214), 2^19 172, 175 (298, 571)
//   force, h = 2:     2^18 78, 78 (47, 53), 2^19 80, 80 (76, 128)
//   density, h = 5:   2^14 828, 943 (direct 498, 504), 2^16 1050 (1530, 1580)
//   two steps, h = 3.5: 2^15 2785, 2764 as one pass, 1815, 1851 in separate ones
bool tiles_pay(int64_t np, int tiles, int per_tile) {
  return tiles <= 1024 || np >= (int64_t)per_tile * tiles;
}
bool force_tiles_pay(int64_t np, int tiles, int h2) {
  return tiles_pay(np, tiles, h2 <= 5 ? 64 : 32);
}
// (clumps, h = 3.5: 2^14 in tiles 211, direct 260)
bool deposit_tiles_pay(int64_t np, int tiles, int h2) {
  return h2 < kSplineH2Max || tiles_pay(np, tiles, 4);
}
// So few in tiles of more than one pass of a block are too few blocks: 32768
// at 32^3 (16 tiles) 49 us in lattice order and 66 in clumps, 20 and 22 by the
// reach; within one pass the tiles win (64^3: 18 against 25).
constexpr bool few_blocks(int64_t np, int tiles) {
  return np <= kReachMax && np > (int64_t)kSplineBlock * tiles;
}

// The reach class of h, in half cells (0: wider than the fixed classes).
int spline_class(float h) {
  const int h2 = (int)ceilf(2.0f * h);
  return h2 <= kSplineH2Max ? h2 : 0;
}
#define FDM_REACH_SWITCH(h2, MACRO) \
  switch (h2) {                     \
    case 4: MACRO(4); break;        \
    case 5: MACRO(5); break;        \
    case 6: MACRO(6); break;        \
    case 7: MACRO(7); break;        \
    case 8: MACRO(8); break;        \
    case 9: MACRO(9); break;        \
    case 10: MACRO(10); break;      \
    default: return hipErrorInvalidValue; \
  }

float spline_force_coef(float h) { return (float)(-48.0 / (M_PI * (double)h * h * h * h)); }

unsigned piece_grid(int64_t np, int tiles) {
  const unsigned bound = piece_bound(np, tiles);
  return bound < (unsigned)kSplineGrid ? bound : (unsigned)kSplineGrid;
}

// Windows above 64 KiB of LDS need the launch limit raised.
hipError_t allow_lds(const void* kernel, int bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

hipError_t launch_spline_deposit(bool fixed, int logn, const void* pos, int64_t np, float h,
                                 const TileMap* tm, unsigned long long* mass, hipStream_t s) {
  int lo, hi;
  spline_range(h, lo, hi);
  const SplinePos sp = spline_pos(fixed, logn);
  const uint32_t* words = static_cast<const uint32_t*>(pos);
  const double unit = ldexp(16.0 / (M_PI * (double)h * h * h), kMassShift);
  const int h2 = spline_class(h);
  if (tm && h2 && deposit_tiles_pay(np, tm->tiles, h2)) {
    const dim3 g(piece_grid(np, tm->tiles));
#define T_(H2)                                                                                   \
  {                                                                                              \
    const int lds = 8 * spline_window<H2>(logn);                                                 \
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_spline_deposit_tiled<H2>), lds); \
    if (e != hipSuccess) return e;                                                               \
    hipLaunchKernelGGL((k_spline_deposit_tiled<H2>), g, dim3(kSplineBlock), lds, s, words, np,   \
                       sp, *tm, h, 1.0f / h, unit, mass);                                        \
  }
    FDM_REACH_SWITCH(h2, T_)
#undef T_
  } else {
    hipLaunchKernelGGL(k_spline_deposit, dim3(spline_grid(np)), dim3(kBlock), 0, s, words, np, sp,
                       h, 1.0f / h, unit, lo, hi, mass);
  }
  return hipGetLastError();
}

hipError_t launch_spline_qforce(bool fixed, int logn, const void* pos, int64_t np,
                                const float* q, float h, const TileMap* tm, float* acc,
                                hipStream_t s) {
  int lo, hi;
  spline_range(h, lo, hi);
  const SplinePos sp = spline_pos(fixed, logn);
  const uint32_t* words = static_cast<const uint32_t*>(pos);
  const float coef = spline_force_coef(h);
  const int h2 = spline_class(h);
  if (tm && h2 && !few_blocks(np, tm->tiles) && force_tiles_pay(np, tm->tiles, h2)) {
    const dim3 g(piece_grid(np, tm->tiles));
#define T_(H2)                                                                                  \
  {                                                                                             \
    const int lds = 4 * spline_window<H2>(logn);                                                \
    const hipError_t e =                                                                        \
        allow_lds(reinterpret_cast<const void*>(&k_spline_qforce_tiled<H2, false>), lds);       \
    if (e != hipSuccess) return e;                                                              \
    hipLaunchKernelGGL((k_spline_qforce_tiled<H2, false>), g, dim3(kSplineBlock), lds, s,       \
                       const_cast<uint32_t*>(words), np, sp, *tm, q, h, 1.0f / h, coef, acc,    \
                       SplineStep());                                                           \
  }
    FDM_REACH_SWITCH(h2, T_)
#undef T_
  } else if (h2 && np <= kReachMax) {
#define L_(H2)                                                                              \
  hipLaunchKernelGGL((k_spline_qforce_fixed_reach<H2>), dim3(spline_grid(np)), dim3(kBlock), 0, \
                     s, words, np, sp, q, h, 1.0f / h, coef, acc)
    FDM_REACH_SWITCH(h2, L_)
#undef L_
  } else {
    hipLaunchKernelGGL(k_spline_qforce, dim3(spline_grid(np)), dim3(kBlock), 0, s, words, np, sp,
                       q, h, 1.0f / h, coef, lo, hi, acc);
  }
  return hipGetLastError();
}

hipError_t launch_spline_kick(float* vel, const float* gphi, const float* gq, int64_t np,
                              float fg, float fq, hipStream_t s) {
  const int64_t n = 3 * np;
  hipLaunchKernelGGL(k_spline_kick, dim3(spline_grid(n)), dim3(kBlock), 0, s, vel, gphi, gq, n,
                     fg, fq);
  return hipGetLastError();
}

hipError_t launch_spline_drift(bool fixed, int logn, void* pos, const float* vel, int64_t np,
                               double fd, hipStream_t s) {
  const int64_t n = 3 * np;
  hipLaunchKernelGGL(k_spline_drift, dim3(spline_grid(n)), dim3(kBlock), 0, s,
                     static_cast<uint32_t*>(pos), vel, n, spline_pos(fixed, logn), fd);
  return hipGetLastError();
}

bool spline_step_fused(float h, int64_t np, int tiles) {
  const int h2 = spline_class(h);
  return h2 && force_tiles_pay(np, tiles, h2);
}

hipError_t launch_spline_push(bool fixed, int logn, void* pos, float* vel, int64_t np,
                              const float* phi, const float* q, float h, const TileMap& tm,
                              const SplineKicks& k, hipStream_t s) {
  const SplinePos sp = spline_pos(fixed, logn);
  const float coef = spline_force_coef(h);
  const SplineStep st = {vel, phi, k.close_g, k.close_q, k.open_g, k.open_q,
                         k.drift, k.close, k.open};
  const dim3 g(piece_grid(np, tm.tiles));
#define T_(H2)                                                                                  \
  {                                                                                             \
    const int lds = 4 * (spline_window<H2>(logn) + grad_window(logn));                          \
    const hipError_t e =                                                                        \
        allow_lds(reinterpret_cast<const void*>(&k_spline_qforce_tiled<H2, true>), lds);        \
    if (e != hipSuccess) return e;                                                              \
    hipLaunchKernelGGL((k_spline_qforce_tiled<H2, true>), g, dim3(kSplineBlock), lds, s,        \
                       static_cast<uint32_t*>(pos), np, sp, tm, q, h, 1.0f / h, coef, nullptr, st); \
  }
  FDM_REACH_SWITCH(spline_class(h), T_)
#undef T_
  return hipGetLastError();
}

}  // namespace fdm
