// Differentiable windowed SSD of the deformation (an addition of this
// library, not in the paper): forward loss per window and its adjoint with
// respect to the node displacement field, with the Gauss-Newton diagonal.
//
// The tiled forms (win = 2 step) cache the nodes of a tile in LDS; the
// backward forms each pixel's terms 2 m r dB'/du and 2 m (dB'/du)^2 once per
// tile, splits them into left/right node-column partials per pixel row and
// lets every node sum its partials over its rows.  The general forms gather
// per node with per-pixel weights.  No atomics anywhere, so the results are
// bitwise reproducible.
#include <type_traits>

#include "dev_common.h"
#include "piv_internal.h"

namespace piv {
namespace {

struct SsdArgs {
  const float* A;
  const float* B;
  const float* U;
  int W, H, nx, ny, win, step;
  float* loss;
  const float* g;       // NULL: every window's upstream gradient is 1
  float* gU;
  float* D;
  int64_t lstride;      // floats per pair of loss
  int64_t gstride;      // floats per pair of gU and D
  const uint8_t* mask;
  // (tiled adjoint, nullable) per node tile: [tile][2] = the tile's sum of
  // the GN diagonal (both components) and of the window losses (each pixel
  // counted by the tile owning its base node), pair stride pstride floats
  float* part;
  int64_t pstride;
};

__device__ __forceinline__ float ldA(const float* I, int W, int H, int y, int x) {
  return ((unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H) ? I[(int64_t)y * W + x] : 0.0f;
}

// clamped bilinear node coordinates of a pixel: base node and fractions
__device__ __forceinline__ void node_coord(float p, int n, int step, int& b, float& f) {
  const float c = 0.5f * (float)(step - 1);
  float t = fminf(fmaxf((p - c) / (float)step, 0.0f), (float)(n - 1));
  b = min((int)t, max(n - 2, 0));
  f = t - (float)b;
}

__device__ __forceinline__ void disp_at(const float* U, int nx, int ny, int step, int x, int y, float& u,
                                        float& v) {
  int bx, by;
  float fx, fy;
  node_coord((float)x, nx, step, bx, fx);
  node_coord((float)y, ny, step, by, fy);
  int bx1 = nx > 1 ? bx + 1 : bx, by1 = ny > 1 ? by + 1 : by;
  const int np = nx * ny;
  const float* P = U;
  u = (1.0f - fy) * ((1.0f - fx) * P[by * nx + bx] + fx * P[by * nx + bx1]) +
      fy * ((1.0f - fx) * P[by1 * nx + bx] + fx * P[by1 * nx + bx1]);
  P = U + np;
  v = (1.0f - fy) * ((1.0f - fx) * P[by * nx + bx] + fx * P[by * nx + bx1]) +
      fy * ((1.0f - fx) * P[by1 * nx + bx] + fx * P[by1 * nx + bx1]);
}

// weight of node index `b` in the clamped interpolation of coordinate p
__device__ __forceinline__ float node_weight(float p, int n, int step, int b) {
  int bb;
  float f;
  node_coord(p, n, step, bb, f);
  float w = 0.0f;
  if (b == bb) w += 1.0f - f;
  if (b == (n > 1 ? bb + 1 : bb)) w += f;
  return w;
}

// residual r = B(p+u) - A(p) and the floor-cell gradient of the sample
__device__ __forceinline__ void residual(const SsdArgs& a, const float* A, const float* B, const float* U,
                                         int x, int y, float& r, float& gx, float& gy) {
  float u, v;
  disp_at(U, a.nx, a.ny, a.step, x, y, u, v);
  float qx = (float)x + u, qy = (float)y + v;
  float x0 = floorf(qx), y0 = floorf(qy);
  float fx = qx - x0, fy = qy - y0;
  int ix = (int)x0, iy = (int)y0;
  float p00 = ldA(B, a.W, a.H, iy, ix), p01 = ldA(B, a.W, a.H, iy, ix + 1);
  float p10 = ldA(B, a.W, a.H, iy + 1, ix), p11 = ldA(B, a.W, a.H, iy + 1, ix + 1);
  float bs = (1.0f - fy) * ((1.0f - fx) * p00 + fx * p01) + fy * ((1.0f - fx) * p10 + fx * p11);
  r = bs - ldA(A, a.W, a.H, y, x);
  gx = (1.0f - fy) * (p01 - p00) + fy * (p11 - p10);
  gy = (1.0f - fx) * (p10 - p00) + fx * (p11 - p01);
}

__device__ __forceinline__ int fdiv(int p, int q) { return p >= 0 ? p / q : -((-p + q - 1) / q); }

// Forward: a workgroup owns a TN x TN tile of windows; squared residuals of
// the tile's pixel region go to LDS, then every window sums its block.
__global__ __launch_bounds__(256) void k_ssd_forward(SsdArgs a, int TN) {
  extern __shared__ float s_r2[];
  const int pair = blockIdx.z;
  if (slot_off(a.mask, pair)) return;
  const int t = threadIdx.x;
  const int np = a.nx * a.ny;
  const int64_t img = (int64_t)a.W * a.H;
  const float* A = a.A + pair * img;
  const float* B = a.B + pair * img;
  const float* U = a.U + (int64_t)pair * 2 * np;
  const int h = (a.win - a.step) / 2;
  const int ta = blockIdx.y * TN, tb = blockIdx.x * TN;
  const int RW = (TN - 1) * a.step + a.win;
  const int y0 = ta * a.step - h, x0 = tb * a.step - h;
  for (int idx = t; idx < RW * RW; idx += 256) {
    int y = y0 + idx / RW, x = x0 + idx % RW;
    float r, gx, gy;
    residual(a, A, B, U, x, y, r, gx, gy);
    s_r2[idx] = r * r;
  }
  __syncthreads();
  // one window per 4 threads (TN*TN <= 64)
  const int w = t >> 2, p = t & 3;
  const int wi = w / TN, wj = w % TN;
  float s = 0.0f;
  if (w < TN * TN) {
    for (int i = p; i < a.win; i += 4) {
      const float* row = s_r2 + (wi * a.step + i) * RW + wj * a.step;
      for (int j = 0; j < a.win; ++j) s += row[j];
    }
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  if (w < TN * TN && p == 0) {
    int aa = ta + wi, bb = tb + wj;
    if (aa < a.ny && bb < a.nx) a.loss[(int64_t)pair * a.lstride + aa * a.nx + bb] = s;
  }
}

// Backward: a workgroup owns a TN x TN tile of nodes.  Pass 1 writes per
// pixel of the tile's support region: 2 m r gx, 2 m r gy, 2 m gx^2, 2 m gy^2
// (m = sum of upstream gradients of the windows holding the pixel).  Pass 2:
// 16 threads per node gather weight * term over the node's support rows,
// then reduce over their 16 lanes.
__global__ __launch_bounds__(256) void k_ssd_backward(SsdArgs a, int TN) {
  extern __shared__ float s_t[];
  const int pair = blockIdx.z;
  if (slot_off(a.mask, pair)) return;
  const int t = threadIdx.x;
  const int np = a.nx * a.ny;
  const int64_t img = (int64_t)a.W * a.H;
  const float* A = a.A + pair * img;
  const float* B = a.B + pair * img;
  const float* U = a.U + (int64_t)pair * 2 * np;
  const float* G = a.g ? a.g + (int64_t)pair * np : nullptr;
  const int h = (a.win - a.step) / 2;
  const int ta = blockIdx.y * TN, tb = blockIdx.x * TN;
  // pixel support of the tile's nodes (clamped interpolation extends the
  // edge nodes' support to the outermost window pixel)
  const int lo_all = -h, hi_x = a.nx * a.step + h - 1, hi_y = a.ny * a.step + h - 1;
  int ylo = ta == 0 ? lo_all : (ta - 1) * a.step + a.step / 2;   // > centre of node ta-1
  int xlo = tb == 0 ? lo_all : (tb - 1) * a.step + a.step / 2;
  int tae = min(ta + TN, a.ny) - 1, tbe = min(tb + TN, a.nx) - 1;
  int yhi = tae == a.ny - 1 ? hi_y : (tae + 1) * a.step + (a.step - 1) / 2;  // < centre of node tae+1
  int xhi = tbe == a.nx - 1 ? hi_x : (tbe + 1) * a.step + (a.step - 1) / 2;
  const int RH = yhi - ylo + 1, RW = xhi - xlo + 1;
  float* T0 = s_t;
  float* T1 = T0 + RH * RW;
  float* T2 = T1 + RH * RW;
  float* T3 = T2 + RH * RW;
  for (int idx = t; idx < RH * RW; idx += 256) {
    int y = ylo + idx / RW, x = xlo + idx % RW;
    // m(p): windows whose block holds the pixel, i.e. the a with
    // a step - h <= y <= a step - h + win - 1 (ceiling for the lower bound)
    int a0 = max(fdiv(y + h - a.win + a.step, a.step), 0), a1 = min(fdiv(y + h, a.step), a.ny - 1);
    int b0 = max(fdiv(x + h - a.win + a.step, a.step), 0), b1 = min(fdiv(x + h, a.step), a.nx - 1);
    float m = 0.0f;
    for (int i = a0; i <= a1; ++i)
      for (int j = b0; j <= b1; ++j) m += G ? G[i * a.nx + j] : 1.0f;
    float r = 0.0f, gx = 0.0f, gy = 0.0f;
    if (m != 0.0f) residual(a, A, B, U, x, y, r, gx, gy);
    T0[idx] = 2.0f * m * r * gx;
    T1[idx] = 2.0f * m * r * gy;
    T2[idx] = 2.0f * m * gx * gx;
    T3[idx] = 2.0f * m * gy * gy;
  }
  __syncthreads();
  const int nd = t >> 4, lane = t & 15;
  const int na = ta + nd / TN, nb = tb + nd % TN;
  float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
  const bool act = nd < TN * TN && na < a.ny && nb < a.nx;
  if (act) {
    // node support rows/cols, intersected with the region
    int sy0 = na == 0 ? lo_all : (na - 1) * a.step + a.step / 2;
    int sy1 = na == a.ny - 1 ? hi_y : (na + 1) * a.step + (a.step - 1) / 2;
    int sx0 = nb == 0 ? lo_all : (nb - 1) * a.step + a.step / 2;
    int sx1 = nb == a.nx - 1 ? hi_x : (nb + 1) * a.step + (a.step - 1) / 2;
    for (int y = sy0 + lane; y <= sy1; y += 16) {
      float wy = node_weight((float)y, a.ny, a.step, na);
      if (wy == 0.0f) continue;
      const int ro = (y - ylo) * RW - xlo;
      for (int x = sx0; x <= sx1; ++x) {
        float wx = node_weight((float)x, a.nx, a.step, nb);
        float w = wx * wy;
        s0 += w * T0[ro + x];
        s1 += w * T1[ro + x];
        s2 += w * w * T2[ro + x];
        s3 += w * w * T3[ro + x];
      }
    }
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    s0 += __shfl_xor(s0, o);
    s1 += __shfl_xor(s1, o);
    s2 += __shfl_xor(s2, o);
    s3 += __shfl_xor(s3, o);
  }
  if (act && lane == 0) {
    const int i = na * a.nx + nb;
    float* gU = a.gU + (int64_t)pair * a.gstride;
    gU[i] = s0;
    gU[np + i] = s1;
    if (a.D) {
      float* D = a.D + (int64_t)pair * a.gstride;
      D[i] = s2;
      D[np + i] = s3;
    }
  }
}

// ---------------------------------------------------------------------------
// Tiled forms for 16 px windows on an 8 px step (the plans' geometry).  A
// workgroup owns an 8 x 8 tile (of windows forward, of nodes backward); its
// pixel region is nine strips of eight rows by nine cells of eight columns,
// strip k = 0 .. ny holding the rows 8 k - 4 .. 8 k + 3: the rows of a strip
// share their base node row, the windows that hold them and, with the nearest
// node, only two owners.  A thread takes a strip's eight pixels of one
// column, so the lanes of a wave read neighbouring columns: three cache lines
// a gather, where groups of four pixels of a row per lane touch nine (the
// forward then took 69 us, 64 pairs of 512 x 512, instead of 38).
// ---------------------------------------------------------------------------
constexpr int kStep = 8;                 // the step, and the pixels of a strip or cell
constexpr int kTile = 8;                 // windows or nodes a side
constexpr int kStrips = kTile + 1;       // strips and cells a side
constexpr int kCols = kStrips * kStep;   // region columns
constexpr int kNodes = kTile + 2;        // cached node rows and columns, from ta - 1 and tb - 1 on

// What a strip's rows (or a cell's columns) share: the cache index of the base
// node and the fractions towards the next node, f0 + e df for row e.  The
// node coordinate (y - 3.5) / 8 is clamped to the grid, so the first strip
// rests on node 0 and the last on node n - 1.
struct SsdCell {
  int base;
  float f0, df;
};

__device__ __forceinline__ SsdCell ssd_cell_of(int k, int n, int t0) {
  SsdCell c;
  c.base = min(max(k - 1, 0), max(n - 2, 0)) - (t0 - 1);
  c.df = k > 0 && k < n ? 0.125f : 0.0f;
  c.f0 = k <= 0 || n <= 1 ? 0.0f : k < n ? 0.0625f : 1.0f;
  return c;
}

// fraction of row e (kInside: no strip of the tile is clamped)
template <bool kInside>
__device__ __forceinline__ float ssd_fraction(const SsdCell& c, int e) {
  return kInside ? 0.0625f + 0.125f * (float)e : c.f0 + (float)e * c.df;
}

// Deals the region's columns: item(st, j) for strip st, column j.  A wave
// takes the first 64 columns of a strip, whose rows' values it then holds in
// scalar registers; the last cell's eight columns of all strips come last.
template <class Item>
__device__ __forceinline__ void ssd_deal(int t, Item item) {
  const int lane = t & 63;
  int w = __builtin_amdgcn_readfirstlane(t >> 6);
  for (; w < kStrips; w += 4) item(w, lane);
  const int st = (w - kStrips) * 8 + (lane >> 3);
  if (st < kStrips) item(st, 64 + (lane & 7));
}

// Loads the tile's node cache.  Returns (the same in every thread) whether
// the tile is interior: no strip or cell is clamped, every pixel of the
// region lies in the frames and so does every bilinear sample with its right
// and lower neighbours, with a pixel to spare.  The samples of region pixel x
// lie at x + u with u between the cached nodes' extremes (the interpolation
// stays within them), so the nodes decide; a NaN node makes the tile not
// interior.
__device__ __forceinline__ bool ssd_nodes(const SsdArgs& a, const float* U, int ta, int tb,
                                          float (&node)[2][kNodes][kNodes]) {
  const int t = threadIdx.x;
  const int np = a.nx * a.ny;
  const int tae = min(ta + kTile, a.ny) - 1, tbe = min(tb + kTile, a.nx) - 1;
  const int ylo = ta * kStep - kStep / 2, yhi = (tae + 1) * kStep + kStep / 2 - 1;
  const int xlo = tb * kStep - kStep / 2, xhi = (tbe + 1) * kStep + kStep / 2 - 1;
  bool inside = ta > 0 && tb > 0 && tae < a.ny - 1 && tbe < a.nx - 1 && yhi < a.H && xhi < a.W;
  if (t < kNodes * kNodes) {
    const int r = t / kNodes, q = t - (t / kNodes) * kNodes;
    const int i = min(max(ta - 1 + r, 0), a.ny - 1) * a.nx + min(max(tb - 1 + q, 0), a.nx - 1);
    const float u = U[i], v = U[np + i];
    node[0][r][q] = u;
    node[1][r][q] = v;
    inside = inside && (float)xlo + u >= 1.0f && (float)xhi + u <= (float)(a.W - 3) && (float)ylo + v >= 1.0f &&
             (float)yhi + v <= (float)(a.H - 3);
  }
  return __syncthreads_and(inside ? 1 : 0) != 0;
}

// Four-byte reads of a frame at byte offsets from its base, 32 bits (a frame
// holds fewer than 2^30 pixels, a side fewer than 2^15).  kInside: plain
// reads, both columns of a cell's row in one.  Else through a buffer
// descriptor of the frame: a pixel beyond the frame gets the offset kBeyond,
// which the hardware answers with zero, without a branch (a frame ends
// before it).
struct __attribute__((aligned(4))) SsdTwo {
  float x, y;
};
constexpr uint32_t kBeyond = 0xfffffffcu;

struct SsdFrame {
  const char* base;
  __amdgpu_buffer_rsrc_t rsrc;
};

__device__ __forceinline__ SsdFrame ssd_frame(const SsdArgs& a, const float* I) {
  SsdFrame f;
  f.base = reinterpret_cast<const char*>(I);
  f.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(I), 0, (int)(4u * (uint32_t)a.W * (uint32_t)a.H),
                                             0x00020000);
  return f;
}

__device__ __forceinline__ float ssd_beyond(const SsdFrame& f, bool in, uint32_t o) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(f.rsrc, (int)(in ? o : kBeyond), 0, 0));
}

// the bilinear cell of B at (ix, iy)
template <bool kInside>
__device__ __forceinline__ void ssd_corners(const SsdArgs& a, const SsdFrame& f, int ix, int iy, float& p00, float& p01,
                                            float& p10, float& p11) {
  const uint32_t ow = 4u * (uint32_t)a.W;
  if constexpr (kInside) {
    const uint32_t o = (uint32_t)__umul24((uint32_t)iy, ow) + 4u * (uint32_t)ix;
    const SsdTwo top = *reinterpret_cast<const SsdTwo*>(f.base + o);
    const SsdTwo bot = *reinterpret_cast<const SsdTwo*>(f.base + (o + ow));
    p00 = top.x;
    p01 = top.y;
    p10 = bot.x;
    p11 = bot.y;
  } else {
    const bool x0 = (uint32_t)ix < (uint32_t)a.W, x1 = (uint32_t)ix + 1u < (uint32_t)a.W;
    const bool y0 = (uint32_t)iy < (uint32_t)a.H, y1 = (uint32_t)iy + 1u < (uint32_t)a.H;
    const uint32_t o = (uint32_t)__mul24(iy, (int)ow) + 4u * (uint32_t)ix;   // (right where it is used)
    p00 = ssd_beyond(f, x0 && y0, o);
    p01 = ssd_beyond(f, x1 && y0, o + 4u);
    p10 = ssd_beyond(f, x0 && y1, o + ow);
    p11 = ssd_beyond(f, x1 && y1, o + ow + 4u);
  }
}

// A at the pixel (x, y) (zero outside the frame)
template <bool kInside>
__device__ __forceinline__ float ssd_a(const SsdArgs& a, const SsdFrame& f, int x, int y) {
  const uint32_t o = (uint32_t)__mul24(y, 4 * a.W) + 4u * (uint32_t)x;
  if constexpr (kInside) return *reinterpret_cast<const float*>(f.base + o);
  else return ssd_beyond(f, (uint32_t)x < (uint32_t)a.W && (uint32_t)y < (uint32_t)a.H, o);
}

// One column of a strip: for each of its eight pixels, with (u, v) =
// disp(e), use(e, r, gx, gy) gets the residual r = B(x + u, y + v) - A(x, y)
// and the sample's floor-cell gradient: with top/bottom the row
// interpolations of the cell, bs = top + ey (bottom - top), dbs/dy =
// bottom - top and dbs/dx the row differences interpolated in y.  Four
// pixels' reads are in flight together.
template <bool kInside, class Disp, class Use>
__device__ __forceinline__ void ssd_column(const SsdArgs& a, const SsdFrame& A, const SsdFrame& B, int x, int y0, Disp disp,
                                           Use use) {
  const float xf = (float)x, yf = (float)y0;
#pragma unroll
  for (int h = 0; h < kStep; h += 4) {
    float ex[4], ey[4], av[4], p00[4], p01[4], p10[4], p11[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float u, v;
      disp(h + e, u, v);
      const float qx = xf + u, qy = (yf + (float)(h + e)) + v;
      const float x0 = floorf(qx), y0f = floorf(qy);
      ex[e] = qx - x0;
      ey[e] = qy - y0f;
      ssd_corners<kInside>(a, B, (int)x0, (int)y0f, p00[e], p01[e], p10[e], p11[e]);
      av[e] = ssd_a<kInside>(a, A, x, y0 + h + e);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float d0 = p01[e] - p00[e], d1 = p11[e] - p10[e];
      const float top = p00[e] + ex[e] * d0, bot = p10[e] + ex[e] * d1;
      const float gy = bot - top;
      use(h + e, (top + ey[e] * gy) - av[e], d0 + ey[e] * (d1 - d0), gy);
    }
  }
}

// Forward: the squared residuals of every column of a strip are summed in its
// thread, then 4 threads per window add a quarter of its 2 strips x 16
// columns each.  Bound by the address rate of the vector caches (23 million
// accesses, some 16 a gather, or 38 us at one a cycle and CU; 41 VALU
// operations a pixel are 22 us): 64 pairs of 512 x 512 38 us (57 us with a
// thread per pixel, which weighed its four nodes by itself and read the
// cell's corners one by one).
__global__ __launch_bounds__(256, 6) void k_ssd_forward_t(SsdArgs a) {
  __shared__ float node[2][kNodes][kNodes];
  __shared__ __attribute__((aligned(16))) float s_r2[kStrips][kCols];
  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(a.mask, pair)) return;
  const int t = threadIdx.x;
  const int np = a.nx * a.ny;
  const int64_t img = (int64_t)a.W * a.H;
  const SsdFrame A = ssd_frame(a, a.A + pair * img), B = ssd_frame(a, a.B + pair * img);
  const float* U = a.U + (int64_t)pair * 2 * np;
  const int ta = wg.y * kTile, tb = wg.x * kTile;
  const bool interior = ssd_nodes(a, U, ta, tb, node);
  auto squares = [&](auto inside) {
    constexpr bool kIn = decltype(inside)::value;
    ssd_deal(t, [&](int st, int j) __attribute__((always_inline)) {
      if (ta + st > a.ny || tb + j / kStep > a.nx) return;   // no window of the tile holds it
      const SsdCell row = ssd_cell_of(ta + st, a.ny, ta), col = ssd_cell_of(tb + j / kStep, a.nx, tb);
      const float fx = ssd_fraction<kIn>(col, j & (kStep - 1));
      const int rb = kIn ? st : row.base, cb = kIn ? j / kStep : col.base;
      const float uT = node[0][rb][cb] + fx * (node[0][rb][cb + 1] - node[0][rb][cb]);
      const float uB = node[0][rb + 1][cb] + fx * (node[0][rb + 1][cb + 1] - node[0][rb + 1][cb]);
      const float vT = node[1][rb][cb] + fx * (node[1][rb][cb + 1] - node[1][rb][cb]);
      const float vB = node[1][rb + 1][cb] + fx * (node[1][rb + 1][cb + 1] - node[1][rb + 1][cb]);
      const float du = uB - uT, dv = vB - vT;
      float s = 0.0f;
      ssd_column<kIn>(
          a, A, B, tb * kStep - kStep / 2 + j, (ta + st) * kStep - kStep / 2,
          [&](int e, float& u, float& v) {
            const float fy = ssd_fraction<kIn>(row, e);
            u = uT + fy * du;
            v = vT + fy * dv;
          },
          [&](int, float r, float, float) { s += r * r; });
      s_r2[st][j] = s;
    });
  };
  if (interior) squares(std::true_type{});
  else squares(std::false_type{});
  __syncthreads();
  const int w = t >> 2, p = t & 3;
  const int wi = w / kTile, wj = w - (w / kTile) * kTile;
  const int aa = ta + wi, bb = tb + wj;
  const bool act = aa < a.ny && bb < a.nx;
  float s = 0.0f;
  if (act) {
    const float4* q = reinterpret_cast<const float4*>(&s_r2[wi + (p >> 1)][(wj + (p & 1)) * kStep]);
    const float4 lo = q[0], hi = q[1];
    s = ((lo.x + lo.y) + (lo.z + lo.w)) + ((hi.x + hi.y) + (hi.z + hi.w));
  }
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  if (act && p == 0) a.loss[(int64_t)pair * a.lstride + aa * a.nx + bb] = s;
}

// Sum over a 256-thread workgroup in a fixed order (every thread gets it).
__device__ __forceinline__ float tile_sum(float x, float* red) {
  const int t = threadIdx.x;
  __syncthreads();
  red[t] = x;
  __syncthreads();
#pragma unroll
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  return red[0];
}

// Backward, 8 x 8 nodes per workgroup.  Every pixel of the nodes' support
// region contributes to the two node rows and two node columns of its
// bilinear cell (weights 1-f and f, squared for the diagonal), so the
// adjoint separates: pass 1 sums each column of a strip into upper/lower node
// row partials of the four terms 2 m r gx, 2 m r gy, 2 m gx^2, 2 m gy^2 (m,
// the sum of the upstream gradients of the windows holding the pixel, is
// constant along it); pass 2 sums a node's partials over its columns with
// the column weights.  The displacement is interpolated down the two node
// columns and then across, the order that decides in which cell a sample at a
// cell's edge falls.  Bound by VALU issue (0.92 of it; 88 operations a
// pixel with the node sums, half again as many at the frames' border): 64 pairs of 512 x 512 50 us (99 us with a thread per
// eight pixels of a row, whose gathers touched a cache line per lane and whose
// node sums read every row's partials).
constexpr int kPartPlane = kCols + 1;               // odd: the terms' planes on different banks,
constexpr int kPartStrip = 8 * kPartPlane + 1;      // and the strips of a wave's node rows too

template <bool kPart>
__global__ __launch_bounds__(256, 6) void k_ssd_backward_t(SsdArgs a) {
  __shared__ float node[2][kNodes][kNodes];
  __shared__ float s_part[kStrips * kPartStrip];       // [strip][term*2 + side][column]
  __shared__ float s_g[kNodes][kNodes];                // upstream gradients of the windows from ta - 1 and tb - 1 on
  __shared__ float s_red[kPart ? 256 : 1];             // fixed-order tile sums
  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(a.mask, pair)) return;
  const int t = threadIdx.x;
  const int np = a.nx * a.ny;
  const int64_t img = (int64_t)a.W * a.H;
  const SsdFrame A = ssd_frame(a, a.A + pair * img), B = ssd_frame(a, a.B + pair * img);
  const float* U = a.U + (int64_t)pair * 2 * np;
  const float* G = a.g ? a.g + (int64_t)pair * np : nullptr;
  const int ta = wg.y * kTile, tb = wg.x * kTile;
  const int tae = min(ta + kTile, a.ny) - 1, tbe = min(tb + kTile, a.nx) - 1;
  if (t < kNodes * kNodes) {
    const int r = t / kNodes, q = t - (t / kNodes) * kNodes;
    const int gi = ta - 1 + r, gj = tb - 1 + q;
    s_g[r][q] = (unsigned)gi < (unsigned)a.ny && (unsigned)gj < (unsigned)a.nx ? (G ? G[gi * a.nx + gj] : 1.0f) : 0.0f;
  }
  const bool interior = ssd_nodes(a, U, ta, tb, node);   // (ends with a barrier)
  float lsum = 0.0f;   // this thread's share of the tile's loss (owned pixels)
  auto columns = [&](auto in) {
    constexpr bool kIn = decltype(in)::value;
    ssd_deal(t, [&](int st, int j) __attribute__((always_inline)) {
      const int kr = ta + st, cj = j / kStep, kc = tb + cj;
      if (kr > tae + 1 || kc > tbe + 1) return;   // beyond the nodes' support
      // windows kr - 1 and kr of the rows hold the strip, kc - 1 and kc of the columns
      const float m = ((s_g[st][cj] + s_g[st][cj + 1]) + s_g[st + 1][cj]) + s_g[st + 1][cj + 1];
      float acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
      if (m != 0.0f) {
        const SsdCell row = ssd_cell_of(kr, a.ny, ta), col = ssd_cell_of(kc, a.nx, tb);
        const int rb = kIn ? st : row.base, cb = kIn ? cj : col.base;
        const float fx = ssd_fraction<kIn>(col, j & (kStep - 1));
        const float u0 = node[0][rb][cb], u1 = node[0][rb][cb + 1];
        const float du0 = node[0][rb + 1][cb] - u0, du1 = node[0][rb + 1][cb + 1] - u1;
        const float v0 = node[1][rb][cb], v1 = node[1][rb][cb + 1];
        const float dv0 = node[1][rb + 1][cb] - v0, dv1 = node[1][rb + 1][cb + 1] - v1;
        float l0 = 0.0f, l1 = 0.0f;            // the loss of the strip's upper and lower half
        ssd_column<kIn>(
            a, A, B, kc * kStep - kStep / 2 + (j & (kStep - 1)), kr * kStep - kStep / 2,
            [&](int e, float& u, float& v) {
              const float fy = ssd_fraction<kIn>(row, e);
              const float uL = u0 + fy * du0, uR = u1 + fy * du1;
              const float vL = v0 + fy * dv0, vR = v1 + fy * dv1;
              u = uL + fx * (uR - uL);
              v = vL + fx * (vR - vL);
            },
            [&](int e, float r, float gx, float gy) {
              const float f = ssd_fraction<kIn>(row, e);
              const float wl = 1.0f - f, wr = f;
              const float t0 = r * gx, t1 = r * gy, t2 = gx * gx, t3 = gy * gy;
              acc[0] += wl * t0; acc[1] += wr * t0;
              acc[2] += wl * t1; acc[3] += wr * t1;
              acc[4] += (wl * wl) * t2; acc[5] += (wr * wr) * t2;
              acc[6] += (wl * wl) * t3; acc[7] += (wr * wr) * t3;
              if constexpr (kPart) (e < kStep / 2 ? l0 : l1) += r * r;
            });
        if constexpr (kPart) {
          // a pixel counts at the tile of its nearest node: of row kr - 1 in
          // the strip's upper half and kr in its lower (clamped to the grid),
          // and so for the columns
          const int nn = min(max(kc - ((j & (kStep - 1)) < kStep / 2 ? 1 : 0), 0), a.nx - 1);
          const int n0 = min(max(kr - 1, 0), a.ny - 1), n1 = min(kr, a.ny - 1);
          float lacc = 0.0f;
          if (nn >= tb && nn < tb + kTile) {
            if (n0 >= ta && n0 < ta + kTile) lacc += l0;
            if (n1 >= ta && n1 < ta + kTile) lacc += l1;
            lsum += m * lacc;
          }
        }
      }
      const float m2 = 2.0f * m;
#pragma unroll
      for (int k = 0; k < 8; ++k) s_part[st * kPartStrip + k * kPartPlane + j] = m2 * acc[k];
    });
  };
  if (interior) columns(std::true_type{});
  else columns(std::false_type{});
  __syncthreads();
  // pass 2: thread = (node, term); a node collects the upper partials of the
  // strips based on its row and the lower partials of the strips based on the
  // row before, over the columns of the cells based on its column and on the
  // column before with their weights
  const int term = t & 3, nd = t >> 2;
  const int na = ta + nd / kTile, nb = tb + (nd & (kTile - 1));
  float dsum = 0.0f;   // this thread's GN diagonal value (terms 2, 3)
  if (na <= tae && nb <= tbe) {
    const bool sq = term >= 2;
    float s = 0.0f;
    // cells kc and strips kr next to the node: n and n + 1, and at the grid's
    // ends those clamped to the end nodes' cells
    for (int kc = max(nb - 1, tb); kc <= min(nb + 2, tbe + 1); ++kc) {
      const SsdCell col = ssd_cell_of(kc, a.nx, 1);
      const bool left = col.base == nb, right = a.nx > 1 && col.base + 1 == nb;
      if (!left && !right) continue;
      float c[kStep];
#pragma unroll
      for (int e = 0; e < kStep; ++e) c[e] = 0.0f;
      for (int kr = max(na - 1, ta); kr <= min(na + 2, tae + 1); ++kr) {
        const SsdCell row = ssd_cell_of(kr, a.ny, 1);
        const bool up = row.base == na, low = a.ny > 1 && row.base + 1 == na;
        if (!up && !low) continue;
        const float* q = &s_part[(kr - ta) * kPartStrip + (2 * term + (up ? 0 : 1)) * kPartPlane + (kc - tb) * kStep];
#pragma unroll
        for (int e = 0; e < kStep; ++e) c[e] += q[e];
      }
#pragma unroll
      for (int e = 0; e < kStep; ++e) {
        const float f = col.f0 + (float)e * col.df;
        const float w = left ? 1.0f - f : f;
        s += (sq ? w * w : w) * c[e];
      }
    }
    const int idx = na * a.nx + nb;
    if (term < 2) {
      a.gU[(int64_t)pair * a.gstride + term * np + idx] = s;
    } else {
      if (a.D) a.D[(int64_t)pair * a.gstride + (term - 2) * np + idx] = s;
      dsum = s;
    }
  }
  if constexpr (kPart) {
    // fixed-order sums over the workgroup (bitwise reproducible)
    const float ls = tile_sum(lsum, s_red);
    const float ds = tile_sum(dsum, s_red);
    if (t == 0) {
      float* o = a.part + (int64_t)pair * a.pstride + 2 * (wg.y * ((a.nx + kTile - 1) / kTile) + wg.x);
      o[0] = ds;
      o[1] = ls;
    }
  }
}

SsdArgs make_args(const Plan& P, const float* A, const float* B, const float* U) {
  SsdArgs a;
  a.A = A;
  a.B = B;
  a.U = U;
  a.W = P.p.width;
  a.H = P.p.height;
  a.nx = P.nx;
  a.ny = P.ny;
  a.win = P.p.win;
  a.step = P.p.step;
  a.loss = nullptr;
  a.g = nullptr;
  a.gU = nullptr;
  a.D = nullptr;
  a.lstride = (int64_t)P.nx * P.ny;
  a.gstride = 2 * (int64_t)P.nx * P.ny;
  a.mask = P.slot_mask;
  a.part = nullptr;
  a.pstride = 0;
  return a;
}

// Refinement update, one workgroup per pair: the total window loss into the
// history, and U <- U - tau gU / (D + lambda) with lambda = lam_rel mean(D).
// Sums run in a fixed order (per-thread strided partials, then a fixed
// tree), so results are bitwise reproducible.  A node component whose
// D + lambda is not positive is left unchanged.
constexpr int kUpdT = 256;

__device__ __forceinline__ float block_sum(float x, float* red) {
  const int t = threadIdx.x;
  red[t] = x;
  __syncthreads();
#pragma unroll
  for (int o = kUpdT / 2; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  const float r = red[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(kUpdT) void k_ssd_update(float* U, const float* gU, const float* D,
                                                      const float* loss, int64_t wstride, int np, float tau,
                                                      float lam_rel, float* hist, int hstride, int k,
                                                      int update, const uint8_t* mask) {
  __shared__ float red[kUpdT];
  const int pair = blockIdx.x;
  if (slot_off(mask, pair)) return;
  const int t = threadIdx.x;
  if (hist) {
    const float* L = loss + (int64_t)pair * wstride;
    float s = 0.0f;
    for (int i = t; i < np; i += kUpdT) s += L[i];
    s = block_sum(s, red);
    if (t == 0) hist[(int64_t)pair * hstride + k] = s;
  }
  if (!update) return;
  const float* G = gU + (int64_t)pair * wstride;
  const float* Dp = D + (int64_t)pair * wstride;
  float* Up = U + (int64_t)pair * 2 * np;
  float s = 0.0f;
  for (int i = t; i < 2 * np; i += kUpdT) s += Dp[i];
  s = block_sum(s, red);
  const float lam = lam_rel * (s / (float)(2 * np));
  for (int i = t; i < 2 * np; i += kUpdT) {
    const float den = Dp[i] + lam;
    if (den > 0.0f) Up[i] -= tau * G[i] / den;
  }
}

// Refinement update from the adjoint's tile sums: every workgroup adds the
// pair's tile sums in the same fixed order (so all agree on lambda and the
// loss), the first writes the loss into the history, and each updates its
// share of U.
__global__ __launch_bounds__(kUpdT) void k_ssd_update_tiles(float* U, const float* gU, const float* D,
                                                            const float* part, int64_t wstride, int np, int ntiles,
                                                            float tau, float lam_rel, float* hist, int hstride,
                                                            int k, const uint8_t* mask) {
  __shared__ float red[kUpdT];
  const int pair = blockIdx.y;
  if (slot_off(mask, pair)) return;
  const int t = threadIdx.x;
  const float* pp = part + (int64_t)pair * wstride;
  float ds = 0.0f, ls = 0.0f;
  for (int i = t; i < ntiles; i += kUpdT) {
    ds += pp[2 * i];
    ls += pp[2 * i + 1];
  }
  ds = block_sum(ds, red);
  ls = block_sum(ls, red);
  if (hist && blockIdx.x == 0 && t == 0) hist[(int64_t)pair * hstride + k] = ls;
  const float lam = lam_rel * (ds / (float)(2 * np));
  const float* G = gU + (int64_t)pair * wstride;
  const float* Dp = D + (int64_t)pair * wstride;
  float* Up = U + (int64_t)pair * 2 * np;
  for (int i = blockIdx.x * kUpdT + t; i < 2 * np; i += gridDim.x * kUpdT) {
    const float den = Dp[i] + lam;
    if (den > 0.0f) Up[i] -= tau * G[i] / den;
  }
}

}  // namespace

hipError_t launch_ssd_forward(const Plan& P, const float* A, const float* B, const float* U, int n,
                              float* loss, hipStream_t s) {
  SsdArgs a = make_args(P, A, B, U);
  a.loss = loss;
  if (!loss) {   // the workspace's window losses
    a.loss = reinterpret_cast<float*>(P.ws + P.off_loss);
    a.lstride = (int64_t)(P.per_pair / sizeof(float));
  }
  // tile: at most 8 x 8 windows with a pixel region of at most 96 x 96
  if (a.step == 8 && a.win == 16) {
    dim3 grid((a.nx + 7) / 8, (a.ny + 7) / 8, n);
    hipLaunchKernelGGL(k_ssd_forward_t, grid, dim3(256), 0, s, a);
    return hipGetLastError();
  }
  int TN = max(1, min(8, (96 - a.win) / a.step + 1));
  int RW = (TN - 1) * a.step + a.win;
  size_t lds = sizeof(float) * (size_t)RW * RW;
  dim3 grid((a.nx + TN - 1) / TN, (a.ny + TN - 1) / TN, n);
  hipLaunchKernelGGL(k_ssd_forward, grid, dim3(256), lds, s, a, TN);
  return hipGetLastError();
}

hipError_t launch_ssd_backward(const Plan& P, const float* A, const float* B, const float* U,
                               const float* g, int n, float* gU, float* D, hipStream_t s) {
  SsdArgs a = make_args(P, A, B, U);
  a.g = g;
  a.gU = gU;
  a.D = D;
  if (!gU) {   // the workspace's gradient and diagonal
    a.gU = reinterpret_cast<float*>(P.ws + P.off_gu);
    a.D = reinterpret_cast<float*>(P.ws + P.off_dd);
    a.gstride = (int64_t)(P.per_pair / sizeof(float));
  }
  if (a.step == 8 && a.win == 16) {
    dim3 grid((a.nx + 7) / 8, (a.ny + 7) / 8, n);
    hipLaunchKernelGGL((k_ssd_backward_t<false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
  }
  // 16 threads per node -> 16 nodes per workgroup; support region of a
  // 4 x 4 node tile spans (TN+1) step + h px plus edge extension
  const int TN = 4;
  const int h = (a.win - a.step) / 2;
  int RWmax = (TN + 1) * a.step + 2 * h + 2;
  size_t lds = sizeof(float) * 4 * (size_t)RWmax * RWmax;
  if (lds > 65536) return hipErrorInvalidValue;
  dim3 grid((a.nx + TN - 1) / TN, (a.ny + TN - 1) / TN, n);
  hipLaunchKernelGGL(k_ssd_backward, grid, dim3(256), lds, s, a, TN);
  return hipGetLastError();
}

bool ssd_tiled(const Plan& P) { return P.p.step == 8 && P.p.win == 16; }

hipError_t launch_ssd_refine_step(const Plan& P, const float* A, const float* B, float* U, int n, float tau,
                                  float lam_rel, float* hist, int hstride, int k, hipStream_t s) {
  SsdArgs a = make_args(P, A, B, U);
  a.gU = reinterpret_cast<float*>(P.ws + P.off_gu);
  a.D = reinterpret_cast<float*>(P.ws + P.off_dd);
  a.gstride = (int64_t)(P.per_pair / sizeof(float));
  a.part = reinterpret_cast<float*>(P.ws + P.off_part);
  a.pstride = a.gstride;
  dim3 grid((a.nx + 7) / 8, (a.ny + 7) / 8, n);
  hipLaunchKernelGGL((k_ssd_backward_t<true>), grid, dim3(256), 0, s, a);
  if (hipError_t e = hipGetLastError()) return e;
  const int np = P.nx * P.ny;
  const int ntiles = (int)(grid.x * grid.y);
  dim3 gu((unsigned)max(1, min(64, (2 * np + 4 * kUpdT - 1) / (4 * kUpdT))), n);
  hipLaunchKernelGGL(k_ssd_update_tiles, gu, dim3(kUpdT), 0, s, U, a.gU, a.D, a.part, a.gstride, np, ntiles, tau,
                     lam_rel, hist, hstride, k, P.slot_mask);
  return hipGetLastError();
}

hipError_t launch_ssd_update(const Plan& P, float* U, int n, float tau, float lam_rel, float* hist, int hstride,
                             int k, int update, hipStream_t s) {
  const int64_t ws_f = (int64_t)(P.per_pair / sizeof(float));
  hipLaunchKernelGGL(k_ssd_update, dim3(n), dim3(kUpdT), 0, s, U,
                     reinterpret_cast<const float*>(P.ws + P.off_gu), reinterpret_cast<const float*>(P.ws + P.off_dd),
                     reinterpret_cast<const float*>(P.ws + P.off_loss), ws_f, P.nx * P.ny, tau, lam_rel, hist,
                     hstride, k, update, P.slot_mask);
  return hipGetLastError();
}

}  // namespace piv
