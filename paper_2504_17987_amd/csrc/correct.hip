// Correction kernels (Sec. 2 of the paper): deform the pair by the
// interpolated predictor, correlate every window with the deformed frame B
// over the search shifts (Pearson coefficient), pick the best shift and fit
// a 3-point Gaussian per axis.
//
// Implementations of the same definition:
//  * k_correct_generic -- one workgroup per window; any window/step/radius.
//  * k_correct_rows    -- 32 px windows at 50% overlap (below).
//  * k_correct_bands   -- 16 px windows at 50% overlap, frame B deformed
//    (below).
//  * k_correct_halves  -- 24 px windows (u16) with frame B deformed, 16 px
//    windows with both (below).
//  * k_correct_tiled   -- the other cases of 50%-overlap windows (win = 2 step):
//    a workgroup owns a TW x TH tile of windows; the deformed B' tile and the
//    A tile live in LDS; each thread correlates one step x step cell with a
//    band of SYG shift rows, so every pixel-shift product is formed once and
//    shared by the four windows that contain the cell; window sums are then
//    assembled from cell sums.
//
// Numerics (FP32): all sums are taken about an integer offset K (the rounded
// mean intensity of the tile; of the window in k_correct_generic and
// k_correct_rows), which leaves the coefficient unchanged and keeps
// E[x^2] - E[x]^2 well conditioned.  A window counts as flat when its
// variance is below 1e-6 of its second moment about K (an exact zero cannot
// be certified in FP32); a flat window has coefficient 0.
#include <type_traits>

#include "dev_common.h"
#include "piv_internal.h"

namespace piv {
namespace {

constexpr float kFlatRel = 1e-6f;

struct CorrArgs {
  const uint8_t* A;
  const uint8_t* B;
  int64_t pitch, stride;   // bytes per row / per pair
  int W, H, nx, ny;
  int win, step, R;        // R: searched radius (1 in fixed-centre mode)
  int central;             // deform both frames by -u/2, +u/2
  int fixed;               // fixed-centre 5-point stencil
  const float* pred;       // [n][2][ny][nx] or null
  float* disp;
  int64_t dstride;         // floats per pair of disp
  float* peak;             // nullable
  uint8_t* flags;
  const uint8_t* mask;
};

// tie key: smaller is preferred among equal coefficients (|sx|+|sy|, sy, sx)
constexpr int kKeyNone = 0x7fffffff;   // a shift that takes no part in the peak search
__device__ __forceinline__ int tie_key(int sy, int sx) {
  return ((abs(sx) + abs(sy)) << 12) | ((sy + 32) << 6) | (sx + 32);
}

__device__ __forceinline__ bool better(float r1, int k1, float r2, int k2) {
  return r1 > r2 || (r1 == r2 && k1 < k2);
}

// 3-point Gaussian offset on coefficients floored at 1e-3; nocurv when the
// log-parabola does not open downward.
__device__ __forceinline__ float gauss3(float cm, float c0, float cp, bool& nocurv) {
  float lm = logf(fmaxf(cm, 1e-3f)), l0 = logf(fmaxf(c0, 1e-3f)), lp = logf(fmaxf(cp, 1e-3f));
  float den = 2.0f * (lm - 2.0f * l0 + lp);
  nocurv = !(den < 0.0f);
  return nocurv ? 0.0f : (lm - lp) / den;
}

// displacement at pixel (x, y) from a node field read through `node(c, a, b)`
// (clamped to the hull of node centres), bilinear.
template <typename NodeFn>
__device__ __forceinline__ void interp_u(float x, float y, int nx, int ny, int step, NodeFn node,
                                         float& u, float& v) {
  const float c = 0.5f * (float)(step - 1);
  float tx = (x - c) / (float)step, ty = (y - c) / (float)step;
  tx = fminf(fmaxf(tx, 0.0f), (float)(nx - 1));
  ty = fminf(fmaxf(ty, 0.0f), (float)(ny - 1));
  int bx = min((int)tx, max(nx - 2, 0)), by = min((int)ty, max(ny - 2, 0));
  float fx = tx - (float)bx, fy = ty - (float)by;
  int bx1 = nx > 1 ? bx + 1 : bx, by1 = ny > 1 ? by + 1 : by;
  u = (1.0f - fy) * ((1.0f - fx) * node(0, by, bx) + fx * node(0, by, bx1)) +
      fy * ((1.0f - fx) * node(0, by1, bx) + fx * node(0, by1, bx1));
  v = (1.0f - fy) * ((1.0f - fx) * node(1, by, bx) + fx * node(1, by, bx1)) +
      fy * ((1.0f - fx) * node(1, by1, bx) + fx * node(1, by1, bx1));
}

// The correction is relative to the deformation applied to the window, so
// it is added to the window mean of the interpolated predictor.  Bilinear
// interpolation with clamping is separable, so the mean is a product of
// per-axis node weights: for 50%-overlap windows (win = 2 step, step even)
// these are (1/4, 1/2, 1/4) inside, (3/4, 1/4) on the first node and
// (1/4, 3/4) on the last.
__device__ __forceinline__ void half_overlap_weights(int b, int n, float& wm, float& w0, float& wp) {
  if (n == 1) { wm = 0.0f; w0 = 1.0f; wp = 0.0f; }
  else if (b == 0) { wm = 0.0f; w0 = 0.75f; wp = 0.25f; }
  else if (b == n - 1) { wm = 0.25f; w0 = 0.75f; wp = 0.0f; }
  else { wm = 0.25f; w0 = 0.5f; wp = 0.25f; }
}

template <typename NodeFn>
__device__ __forceinline__ void window_mean_half_overlap(int a, int b, int nx, int ny, NodeFn node,
                                                         float& pu, float& pv) {
  float wy[3], wx[3];
  half_overlap_weights(a, ny, wy[0], wy[1], wy[2]);
  half_overlap_weights(b, nx, wx[0], wx[1], wx[2]);
  pu = pv = 0.0f;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      float w = wy[i] * wx[j];
      if (w != 0.0f) {
        pu += w * node(0, a + i - 1, b + j - 1);
        pv += w * node(1, a + i - 1, b + j - 1);
      }
    }
}

// Four consecutive pixels of row y from pixel x on (zero outside the image),
// with aligned word loads realigned by alignbyte.
template <typename T, bool kAligned = false>
__device__ __forceinline__ void load4(const uint8_t* img, int64_t pitch, int H, int rowbytes, int y, int x,
                                      float (&v)[4]) {
  // rows outside the image read row 0 or H-1 and are zeroed afterwards
  const uint32_t rowok = (unsigned)y < (unsigned)H ? 0xffffffffu : 0u;
  const uint8_t* row = img + (int64_t)min(max(y, 0), H - 1) * pitch;
  if constexpr (sizeof(T) == 1 && kAligned) {
    const uint32_t w = masked_word(row, rowbytes, x) & rowok;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (float)((w >> (8 * k)) & 0xffu);
  } else if constexpr (sizeof(T) == 2 && kAligned) {
    const uint32_t lo = masked_word(row, rowbytes, 2 * x) & rowok, hi = masked_word(row, rowbytes, 2 * x + 4) & rowok;
    v[0] = (float)(lo & 0xffffu);
    v[1] = (float)(lo >> 16);
    v[2] = (float)(hi & 0xffffu);
    v[3] = (float)(hi >> 16);
  } else if constexpr (sizeof(T) == 1) {
    const int xb = x, xa = xb & ~3, sh = xb & 3;
    uint32_t w = __builtin_amdgcn_alignbyte(masked_word(row, rowbytes, xa + 4), masked_word(row, rowbytes, xa), sh);
    w &= rowok;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (float)((w >> (8 * k)) & 0xffu);
  } else if constexpr (sizeof(T) == 2) {
    const int xb = 2 * x, xa = xb & ~3, sh = xb & 3;
    uint32_t w0 = masked_word(row, rowbytes, xa), w1 = masked_word(row, rowbytes, xa + 4),
             w2 = masked_word(row, rowbytes, xa + 8);
    uint32_t lo = __builtin_amdgcn_alignbyte(w1, w0, sh) & rowok, hi = __builtin_amdgcn_alignbyte(w2, w1, sh) & rowok;
    v[0] = (float)(lo & 0xffffu);
    v[1] = (float)(lo >> 16);
    v[2] = (float)(hi & 0xffffu);
    v[3] = (float)(hi >> 16);
  } else {
    if (y < 0 || y >= H) {
      v[0] = v[1] = v[2] = v[3] = 0.0f;
      return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = pixf<T>(img, pitch, rowbytes / 4, H, y, x + k);
  }
}

// Fit and compose one vector from its coefficient lookup rho(sy, sx).
template <typename RhoFn>
__device__ __forceinline__ void finish_vector(const CorrArgs& g, int pair, int a, int b, int sy, int sx,
                                              bool flat, float pu, float pv, RhoFn rho) {
  const int R = g.R;
  uint8_t fl = flat ? PIV_F_FLAT : 0;
  float c0 = rho(sy, sx);
  float ex = 0.0f, ey = 0.0f;
  bool nc;
  if (!g.fixed && (sx == -R || sx == R)) fl |= PIV_F_BORDER;
  else {
    ex = gauss3(rho(sy, sx - 1), c0, rho(sy, sx + 1), nc);
    if (nc) fl |= PIV_F_NOCURV;
  }
  if (!g.fixed && (sy == -R || sy == R)) fl |= PIV_F_BORDER;
  else {
    ey = gauss3(rho(sy - 1, sx), c0, rho(sy + 1, sx), nc);
    if (nc) fl |= PIV_F_NOCURV;
  }
  if (g.fixed) {
    ex = fminf(fmaxf(ex, -1.0f), 1.0f);
    ey = fminf(fmaxf(ey, -1.0f), 1.0f);
  }
  const int np = g.nx * g.ny, i = a * g.nx + b;
  float* D = g.disp + (int64_t)pair * g.dstride;
  D[i] = pu + (float)sx + ex;
  D[np + i] = pv + (float)sy + ey;
  if (g.peak) g.peak[(int64_t)pair * np + i] = c0;
  g.flags[(int64_t)pair * np + i] = fl;
}

// ---------------------------------------------------------------------------
// Generic: one workgroup per window.  The window and its B' box are staged
// in LDS; a thread takes one shift and one of H parts of the window's rows
// (H = as many parts as fit the workgroup, so that a window with many shifts
// still gives every SIMD several waves), the parts' sums meet in LDS in a
// fixed order, and a thread per shift forms the coefficient.
// ---------------------------------------------------------------------------
constexpr int kGenT = 1024;

template <typename T>
__global__ __launch_bounds__(kGenT) void k_correct_generic(CorrArgs g) {
  extern __shared__ float s_mem[];
  __shared__ float s_red[kGenT], s_red2[kGenT];
  __shared__ int s_key[kGenT];
  __shared__ float s_K;
  const int pair = blockIdx.z;
  if (slot_off(g.mask, pair)) return;
  const int a = blockIdx.y, b = blockIdx.x, t = threadIdx.x;
  const int win = g.win, R = g.R, S = 2 * R + 1, BWd = win + 2 * R, S2 = S * S;
  const int H = max(1, min(win, kGenT / S2));   // row parts per shift
  float* sA = s_mem;                 // [win][win]
  float* sB = sA + win * win;        // [BWd][BWd]
  float* sRho = sB + BWd * BWd;      // [S][S]
  float* sPart = sRho + S2;          // [3][H][S2]: P, S, Q of each shift's row parts
  const uint8_t* Ai = g.A + (int64_t)pair * g.stride;
  const uint8_t* Bi = g.B + (int64_t)pair * g.stride;
  const float* Pn = g.pred ? g.pred + (int64_t)pair * 2 * g.nx * g.ny : nullptr;
  const int np = g.nx * g.ny;
  auto node = [&](int c, int y, int x) { return Pn[c * np + y * g.nx + x]; };
  const int h = (win - g.step) / 2, oy = a * g.step - h, ox = b * g.step - h;
  const float sgnA = -0.5f, sgnB = g.central ? 0.5f : 1.0f;
  // fixed-order tree over the workgroup (every thread returns the total)
  auto tree2 = [&](float x, float y, float& sx_, float& sy_) {
    s_red[t] = x;
    s_red2[t] = y;
    __syncthreads();
    for (int o = kGenT / 2; o > 0; o >>= 1) {
      if (t < o) {
        s_red[t] += s_red[t + o];
        s_red2[t] += s_red2[t + o];
      }
      __syncthreads();
    }
    sx_ = s_red[0];
    sy_ = s_red2[0];
    __syncthreads();
  };

  float part = 0.0f;
  for (int idx = t; idx < win * win; idx += kGenT) {
    int y = oy + idx / win, x = ox + idx % win;
    float v;
    if (g.central && Pn) {
      float u, w;
      interp_u((float)x, (float)y, g.nx, g.ny, g.step, node, u, w);
      v = bilin<T>(Ai, g.pitch, g.W, g.H, x + sgnA * u, y + sgnA * w);
    } else {
      v = pixf<T>(Ai, g.pitch, g.W, g.H, y, x);
    }
    sA[idx] = v;
    part += v;
  }
  {
    float tot, unused;
    tree2(part, 0.0f, tot, unused);
    if (t == 0) s_K = rintf(tot / (float)(win * win));
    __syncthreads();
  }
  const float K = s_K;
  for (int idx = t; idx < win * win; idx += kGenT) sA[idx] -= K;
  for (int idx = t; idx < BWd * BWd; idx += kGenT) {
    int y = oy - R + idx / BWd, x = ox - R + idx % BWd;
    float v;
    if (Pn) {
      float u, w;
      interp_u((float)x, (float)y, g.nx, g.ny, g.step, node, u, w);
      v = bilin<T>(Bi, g.pitch, g.W, g.H, x + sgnB * u, y + sgnB * w);
    } else {
      v = pixf<T>(Bi, g.pitch, g.W, g.H, y, x);
    }
    sB[idx] = v - K;
  }
  __syncthreads();
  // A statistics (of A - K)
  float sa, saa;
  {
    float p1 = 0.0f, p2 = 0.0f;
    for (int idx = t; idx < win * win; idx += kGenT) {
      const float v = sA[idx];
      p1 += v;
      p2 += v * v;
    }
    tree2(p1, p2, sa, saa);
  }
  const float n = (float)(win * win);
  const float mA = sa / n;
  const float varA = saa - sa * mA;
  const bool flatA = !(varA > kFlatRel * saa);

  // shift s, row part hp: rows [hp win / H, (hp + 1) win / H) of the window
  for (int item = t; item < S2 * H; item += kGenT) {
    const int hp = item / S2, sidx = item - hp * S2;
    const int sy = sidx / S - R, sx = sidx % S - R;
    float P = 0.0f, Sb = 0.0f, Q = 0.0f;
    if (!g.fixed || sx == 0 || sy == 0) {
      const int r0 = hp * win / H, r1 = (hp + 1) * win / H;
      for (int i = r0; i < r1; ++i) {
        const float* arow = sA + i * win;
        const float* brow = sB + (i + sy + R) * BWd + sx + R;
        // eight pixels' reads in flight together
        int j = 0;
        for (; j + 8 <= win; j += 8) {
          float av[8], bv[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            av[u] = arow[j + u];
            bv[u] = brow[j + u];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            P += av[u] * bv[u];
            Sb += bv[u];
            Q += bv[u] * bv[u];
          }
        }
        for (; j < win; ++j) {
          const float bv = brow[j];
          P += arow[j] * bv;
          Sb += bv;
          Q += bv * bv;
        }
      }
    }
    sPart[(0 * H + hp) * S2 + sidx] = P;
    sPart[(1 * H + hp) * S2 + sidx] = Sb;
    sPart[(2 * H + hp) * S2 + sidx] = Q;
  }
  __syncthreads();

  float best = -2.0f;
  int bkey = 1 << 30, nflat = 0;
  for (int sidx = t; sidx < S2; sidx += kGenT) {
    const int sy = sidx / S - R, sx = sidx % S - R;
    float r = 0.0f;
    const bool used = !g.fixed || sx == 0 || sy == 0;
    if (used) {
      float P = 0.0f, Sb = 0.0f, Q = 0.0f;
      for (int hp = 0; hp < H; ++hp) {
        P += sPart[(0 * H + hp) * S2 + sidx];
        Sb += sPart[(1 * H + hp) * S2 + sidx];
        Q += sPart[(2 * H + hp) * S2 + sidx];
      }
      float num = P - mA * Sb;
      float varB = Q - Sb * Sb / n;
      bool flat = flatA || !(varB > kFlatRel * Q);
      r = flat ? 0.0f : num * rsqrtf(varA * varB);
      nflat += flat;
      int key = tie_key(sy, sx);
      if (!g.fixed && better(r, key, best, bkey)) {
        best = r;
        bkey = key;
      }
    }
    sRho[sidx] = r;
  }
  s_red[t] = best;
  s_key[t] = bkey;
  __syncthreads();
  for (int o = kGenT / 2; o > 0; o >>= 1) {
    if (t < o && better(s_red[t + o], s_key[t + o], s_red[t], s_key[t])) {
      s_red[t] = s_red[t + o];
      s_key[t] = s_key[t + o];
    }
    __syncthreads();
  }
  // count flat shifts
  __shared__ int s_nflat;
  if (t == 0) s_nflat = 0;
  __syncthreads();
  if (nflat) atomicAdd(&s_nflat, nflat);
  __syncthreads();
  if (t == 0) {
    int sy = 0, sx = 0;
    if (!g.fixed) {
      int k = s_key[0];
      sx = (k & 63) - 32;
      sy = ((k >> 6) & 63) - 32;
    }
    // window mean of the interpolated predictor: per-axis node weights
    float pu = 0.0f, pv = 0.0f;
    if (Pn) {
      float* wx = sA;                     // A tile is no longer needed
      float* wy = sA + (win / g.step + 3);
      const float c = 0.5f * (float)(g.step - 1);
      int bxl, byl;
      {
        float tx = fminf(fmaxf(((float)ox - c) / g.step, 0.0f), (float)(g.nx - 1));
        float ty = fminf(fmaxf(((float)oy - c) / g.step, 0.0f), (float)(g.ny - 1));
        bxl = min((int)tx, max(g.nx - 2, 0));
        byl = min((int)ty, max(g.ny - 2, 0));
      }
      const int nw = win / g.step + 3;
      for (int q = 0; q < 2 * nw; ++q) sA[q] = 0.0f;
      for (int j = 0; j < win; ++j) {
        float tx = fminf(fmaxf(((float)(ox + j) - c) / g.step, 0.0f), (float)(g.nx - 1));
        int bx = min((int)tx, max(g.nx - 2, 0));
        float fx = tx - (float)bx;
        wx[bx - bxl] += 1.0f - fx;
        wx[(g.nx > 1 ? bx + 1 : bx) - bxl] += fx;
        float ty = fminf(fmaxf(((float)(oy + j) - c) / g.step, 0.0f), (float)(g.ny - 1));
        int by = min((int)ty, max(g.ny - 2, 0));
        float fy = ty - (float)by;
        wy[by - byl] += 1.0f - fy;
        wy[(g.ny > 1 ? by + 1 : by) - byl] += fy;
      }
      for (int i = 0; i < nw; ++i)
        for (int j = 0; j < nw; ++j) {
          float w = wy[i] * wx[j];
          if (w != 0.0f) {
            pu += w * node(0, byl + i, bxl + j);
            pv += w * node(1, byl + i, bxl + j);
          }
        }
      const float inv = 1.0f / ((float)win * (float)win);
      pu *= inv;
      pv *= inv;
    }
    const int nev = g.fixed ? 5 : S * S;
    auto rho = [&](int y, int x) { return sRho[(y + R) * S + x + R]; };
    finish_vector(g, pair, a, b, sy, sx, s_nflat == nev, pu, pv, rho);
  }
}

// ---------------------------------------------------------------------------
// Tiled, cell-shared (win = 2 step).
// ---------------------------------------------------------------------------
template <int STEP, int R, int SYG, int TW, int TH>
struct TileCfg {
  static constexpr int CW = TW + 1, CH = TH + 1, NC = CW * CH;
  static constexpr int NSY = 2 * R + 1, NS = NSY * NSY, NG = NSY / SYG;
  static constexpr int AW = CW * STEP, AH = CH * STEP;
  static constexpr int BW = AW + 2 * R, BH = AH + 2 * R;
  static constexpr int AP = AW + 4;   // LDS row pitches (floats)
  static constexpr int BP = (BW + 3) / 4 * 4 + 4;
  static constexpr int NNX = BW / STEP + 4, NNY = BH / STEP + 3;
  static constexpr int IN_FLOATS = AH * AP + BH * BP;
  // one shift band (SYG rows of NSY shifts) is split over the window's four
  // threads, PER shifts each, stored SLOTW apart (16-byte aligned chunks)
  static constexpr int NBS = SYG * NSY;
  static constexpr int PER = (NBS + 3) / 4;
  static constexpr int SLOTW = (PER + 3) / 4 * 4;
  static constexpr int BANDP = 4 * SLOTW;
  static constexpr int CSTR = BANDP + 4;                  // cell stride (spreads LDS banks)
  static constexpr int WSTR = NG * BANDP + 4;             // window stride of the coefficients
  static constexpr int XBUF = 3 * NC * CSTR;              // P, S, Q of one band, all cells
  static constexpr int RES_FLOATS = 2 * XBUF;             // two band buffers
  // room for the raw source tile of B behind the A and B' tiles: what the
  // result arrays leave free, else what fits a 71 KiB union (two
  // workgroups per CU with the small arrays), at least 16 KiB
  static constexpr int UNION_CAP = 71 * 1024 / 4;
  static constexpr int RAW_FIT = UNION_CAP - IN_FLOATS > 4096 ? UNION_CAP - IN_FLOATS : 4096;
  static constexpr int RAW_WORDS = RES_FLOATS - IN_FLOATS > RAW_FIT ? RES_FLOATS - IN_FLOATS : RAW_FIT;
  static constexpr int UNION = IN_FLOATS + RAW_WORDS > RES_FLOATS ? IN_FLOATS + RAW_WORDS : RES_FLOATS;
  static constexpr int NWIN = TW * TH;
  static_assert(NSY % SYG == 0, "shift rows must split evenly");
  static_assert(NWIN * WSTR <= XBUF, "window coefficients fit one band buffer");
  static_assert(STEP % 2 == 0, "50% overlap needs an even step");
  static_assert(STEP >= 4, "a group of four pixels spans at most two node columns");
};

template <typename T, int STEP, int R, int SYG, int TW, int TH, int NT>
__global__ __launch_bounds__(NT) void k_correct_tiled(CorrArgs g) {
  using C = TileCfg<STEP, R, SYG, TW, TH>;
  // workers: whole cell rows per wave (lane = row-in-wave * CW + column),
  // so that a cell's right-hand neighbour is the next lane of its wave
  constexpr int RPW = 64 / C::CW;
  static_assert((NT / 64) * RPW >= C::NG * C::CH, "one thread per (cell, shift band)");
  static_assert(4 * C::NWIN <= NT, "four threads per window");
  __shared__ __align__(16) float s_u[C::UNION];
  __shared__ float s_node[2][C::NNY][C::NNX];
  __shared__ float s_wsum[C::NWIN], s_wsq[C::NWIN];
  __shared__ float s_red[NT / 64];
  __shared__ float s_rng[NT / 64][5];
  __shared__ int s_rb[C::BH], s_cb[C::BW];
  __shared__ float s_rf[C::BH], s_cf[C::BW];
  __shared__ int s_tkey[C::NG * 4 * C::PER];   // tie key of (band, thread, shift), or kKeyNone

  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(g.mask, pair)) return;
  const int t = threadIdx.x;
  const int a0 = wg.y * TH, b0 = wg.x * TW;
  constexpr int h = STEP / 2;
  const int y0 = a0 * STEP - h, x0 = b0 * STEP - h;      // A tile origin
  const int yb = y0 - R, xb = x0 - R;                    // B' tile origin
  const uint8_t* Ai = g.A + (int64_t)pair * g.stride;
  const uint8_t* Bi = g.B + (int64_t)pair * g.stride;
  const int np = g.nx * g.ny;
  const float* Pn = g.pred ? g.pred + (int64_t)pair * 2 * np : nullptr;
  float* sA = s_u;                   // [AH][AP]
  float* sB = s_u + C::AH * C::AP;   // [BH][BP]

  constexpr int AQ = C::AW / 4;
  constexpr int NA = (C::AH * AQ + NT - 1) / NT;
  // plain A tile: when the tile origin is 4-byte aligned (STEP/2 pixels
  // are), its words are read here, all in flight together ahead of the node
  // cache, and unpacked after the first barrier
  constexpr bool kAlignedA = ((STEP / 2) * (int)sizeof(T)) % 4 == 0;
  constexpr int NWA = kAlignedA ? (int)sizeof(T) : 1;
  const bool plainA = !(g.central && Pn);
  uint32_t aw[NA][NWA], ak[NA][NWA];   // raw words and their keep masks
  if (kAlignedA && plainA) {
    const int rowbytes = g.W * (int)sizeof(T);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int idx0 = t + i * NT;
      const bool in = idx0 < C::AH * AQ;
      const int idx = in ? idx0 : 0;
      const int r = idx / AQ, q = 4 * (idx - (idx / AQ) * AQ);
      const int y = y0 + r;
      const uint32_t ok = (in && (unsigned)y < (unsigned)g.H) ? 0xffffffffu : 0u;
      const uint8_t* row = Ai + (int64_t)min(max(y, 0), g.H - 1) * g.pitch;
#pragma unroll
      for (int k = 0; k < NWA; ++k) {
        // masked_word, with the mask applied after the first barrier so that
        // nothing waits for these reads before the node cache is requested
        const int xa = (x0 + q) * (int)sizeof(T) + 4 * k;
        aw[i][k] = *reinterpret_cast<const uint32_t*>(row + min(max(xa, 0), (rowbytes - 1) & ~3));
        const int valid = rowbytes - xa;
        const uint32_t part = (1u << (8 * (valid & 3))) - 1u;
        ak[i][k] = ((xa < 0 || valid <= 0) ? 0u : (valid >= 4 ? 0xffffffffu : part)) & ok;
      }
    }
  }

  // tie keys of the shifts each window thread will see, per band
  for (int i = t; i < C::NG * 4 * C::PER; i += NT) {
    const int bnd = i / (4 * C::PER), o = i - bnd * 4 * C::PER;   // o = thread * PER + shift
    int key = kKeyNone;
    if (o < C::NBS) {
      const int sy = bnd * SYG + o / C::NSY - R, sx = o % C::NSY - R;
      if (!g.fixed || sx == 0 || sy == 0) key = tie_key(sy, sx);
    }
    s_tkey[i] = key;
  }
  // node cache covering the B' tile, and the range of the predictor over it
  // (every interpolated displacement is a convex combination of cached nodes)
  const float cen = 0.5f * (float)(STEP - 1);
  const int nlo_y = max(0, (int)floorf(((float)yb - cen) / STEP));
  const int nlo_x = max(0, (int)floorf(((float)xb - cen) / STEP));
  float umin = 0.0f, umax = 0.0f, vmin = 0.0f, vmax = 0.0f, bad = 0.0f;
  if (Pn) {
    umin = vmin = 3.0e38f;
    umax = vmax = -3.0e38f;
    for (int idx = t; idx < C::NNY * C::NNX; idx += NT) {
      int r = idx / C::NNX, q = idx % C::NNX;
      int ny_ = min(nlo_y + r, g.ny - 1), nx_ = min(nlo_x + q, g.nx - 1);
      float u = Pn[ny_ * g.nx + nx_], v = Pn[np + ny_ * g.nx + nx_];
      s_node[0][r][q] = u;
      s_node[1][r][q] = v;
      umin = fminf(umin, u);
      umax = fmaxf(umax, u);
      vmin = fminf(vmin, v);
      vmax = fmaxf(vmax, v);
      if (!(fabsf(u) < 1.0e6f && fabsf(v) < 1.0e6f)) bad = 1.0f;   // also NaN
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      bad = fmaxf(bad, __shfl_xor(bad, o));
      umin = fminf(umin, __shfl_xor(umin, o));
      umax = fmaxf(umax, __shfl_xor(umax, o));
      vmin = fminf(vmin, __shfl_xor(vmin, o));
      vmax = fmaxf(vmax, __shfl_xor(vmax, o));
    }
    if ((t & 63) == 0) {
      s_rng[t >> 6][0] = umin;
      s_rng[t >> 6][1] = umax;
      s_rng[t >> 6][2] = vmin;
      s_rng[t >> 6][3] = vmax;
      s_rng[t >> 6][4] = bad;
    }
  }
  // per-row / per-column interpolation tables of the B' tile (the A tile is
  // the same grid shifted by R): base node (cache index) and fraction, the
  // same arithmetic as interp_u
  for (int i = t; i < C::BH + C::BW; i += NT) {
    const bool row = i < C::BH;
    const int p = row ? yb + i : xb + (i - C::BH);
    const int n = row ? g.ny : g.nx;
    float tt = fminf(fmaxf(((float)p - cen) / (float)STEP, 0.0f), (float)(n - 1));
    int bb = min((int)tt, max(n - 2, 0));
    float ff = tt - (float)bb;
    if (row) { s_rb[i] = bb - nlo_y; s_rf[i] = ff; }
    else { s_cb[i - C::BH] = bb - nlo_x; s_cf[i - C::BH] = ff; }
  }
  __syncthreads();
  if (Pn) {
    umin = s_rng[0][0]; umax = s_rng[0][1]; vmin = s_rng[0][2]; vmax = s_rng[0][3]; bad = s_rng[0][4];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) {
      bad = fmaxf(bad, s_rng[i][4]);
      umin = fminf(umin, s_rng[i][0]);
      umax = fmaxf(umax, s_rng[i][1]);
      vmin = fminf(vmin, s_rng[i][2]);
      vmax = fmaxf(vmax, s_rng[i][3]);
    }
  }
  auto node = [&](int c, int y, int x) { return s_node[c][y - nlo_y][x - nlo_x]; };
  auto interp_tab = [&](int r, int q, float& u, float& v) {
    const int rb = s_rb[r], cb = s_cb[q];
    const float fy = s_rf[r], fx = s_cf[q];
    u = (1.0f - fy) * ((1.0f - fx) * s_node[0][rb][cb] + fx * s_node[0][rb][cb + 1]) +
        fy * ((1.0f - fx) * s_node[0][rb + 1][cb] + fx * s_node[0][rb + 1][cb + 1]);
    v = (1.0f - fy) * ((1.0f - fx) * s_node[1][rb][cb] + fx * s_node[1][rb][cb + 1]) +
        fy * ((1.0f - fx) * s_node[1][rb + 1][cb] + fx * s_node[1][rb + 1][cb + 1]);
  };

  // A tile in groups of four pixels (deformed by -u/2 in central mode), held
  // in registers until the tile offset K is known
  float av[NA][4];
#pragma unroll
  for (int i = 0; i < NA; ++i) av[i][0] = av[i][1] = av[i][2] = av[i][3] = 0.0f;
  float part = 0.0f;
  if (plainA) {
    if constexpr (kAlignedA) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const uint32_t w0 = aw[i][0] & ak[i][0], w1 = aw[i][NWA - 1] & ak[i][NWA - 1];
        if constexpr (sizeof(T) == 1) {
#pragma unroll
          for (int e = 0; e < 4; ++e) av[i][e] = (float)((w0 >> (8 * e)) & 0xffu);
        } else {
          av[i][0] = (float)(w0 & 0xffffu);
          av[i][1] = (float)(w0 >> 16);
          av[i][2] = (float)(w1 & 0xffffu);
          av[i][3] = (float)(w1 >> 16);
        }
      }
    } else {
      const int rowbytes = g.W * (int)sizeof(T);
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        const int idx0 = t + i * NT;
        const bool in = idx0 < C::AH * AQ;
        const int idx = in ? idx0 : 0;
        const int r = idx / AQ, q = 4 * (idx - (idx / AQ) * AQ);
        float v[4];
        load4<T>(Ai, g.pitch, g.H, rowbytes, y0 + r, x0 + q, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) av[i][e] = in ? v[e] : 0.0f;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int idx = t + i * NT;
      if (idx < C::AH * AQ) {
        const int r = idx / AQ, q = 4 * (idx - (idx / AQ) * AQ);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u, w;
          interp_tab(r + R, q + e + R, u, w);
          av[i][e] = bilin<T>(Ai, g.pitch, g.W, g.H, (x0 + q + e) - 0.5f * u, (y0 + r) - 0.5f * w);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) part += (av[i][0] + av[i][1]) + (av[i][2] + av[i][3]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
  if ((t & 63) == 0) s_red[t >> 6] = part;

  // raw source tile of B for the deformation, when its bounding box fits
  const float sgnB = g.central ? 0.5f : 1.0f;
  const int ix0 = (int)floorf((float)xb + sgnB * umin) - 1;
  const int ix1 = (int)floorf((float)(xb + C::BW - 1) + sgnB * umax) + 2;
  const int iy0 = (int)floorf((float)yb + sgnB * vmin) - 1;
  const int iy1 = (int)floorf((float)(yb + C::BH - 1) + sgnB * vmax) + 2;
  const int xw0 = (ix0 * (int)sizeof(T)) >> 2;
  const int nwords = ((ix1 * (int)sizeof(T) + (int)sizeof(T) - 1) >> 2) - xw0 + 1;
  const int nrows = iy1 - iy0 + 1;
  // (a displacement range that is not finite or wider than a window takes
  // the unstaged path, whose reads are checked one by one)
  const bool sane = bad == 0.0f && (umax - umin) < 64.0f && (vmax - vmin) < 64.0f;
  const bool staged = sane && nwords <= NT && nwords * nrows <= C::RAW_WORDS;
  uint32_t* sraw = reinterpret_cast<uint32_t*>(s_u + C::IN_FLOATS);
  if (staged) {
    // thread -> (word column, first row); rows advance by rstep, U reads in
    // flight per thread
    const int rowbytes = g.W * (int)sizeof(T);
    const int rstep = NT / nwords;
    const int r0 = t / nwords, w = t - r0 * nwords;
    constexpr int U = 8;
    if (r0 < rstep) {
      for (int rb = r0; rb < nrows; rb += U * rstep) {
        uint32_t val[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int y = iy0 + rb + u * rstep;
          const uint32_t ok = (unsigned)y < (unsigned)g.H ? 0xffffffffu : 0u;
          val[u] = masked_word(Bi + (int64_t)min(max(y, 0), g.H - 1) * g.pitch, rowbytes, 4 * (xw0 + w)) & ok;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (rb + u * rstep < nrows) sraw[(rb + u * rstep) * nwords + w] = val[u];
      }
    }
  }
  __syncthreads();
  // the tile offset K (every thread sums the per-wave partials itself)
  float ksum = 0.0f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) ksum += s_red[i];
  const float K = rintf(ksum / (float)(C::AH * C::AW));
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int idx = t + i * NT;
    if (idx < C::AH * AQ) {
      const int r = idx / AQ, q = 4 * (idx - (idx / AQ) * AQ);
      *reinterpret_cast<float4*>(sA + r * C::AP + q) =
          make_float4(av[i][0] - K, av[i][1] - K, av[i][2] - K, av[i][3] - K);
    }
  }
  // deformed B' tile
  if (staged) {
    // groups of four pixels of one row: the node row and its fraction are
    // shared, and the group spans at most two node columns (STEP > 4), so
    // the displacement is interpolated vertically at three node columns and
    // then horizontally per pixel.  The deformed coordinates stay inside the
    // raw box by its construction (a convex combination of cached nodes plus
    // a one-pixel margin); the clamps only keep the padding columns of a
    // ragged last group inside it.
    constexpr int BQ = (C::BW + 3) / 4;
    constexpr int RPI = NT / BQ;              // rows per pass
    // groups never straddle a node-column boundary when the tile origin and
    // the boundaries agree modulo 4
    constexpr bool kUniformCols = (STEP + R) % 4 == 0;
    const uint8_t* rawb = reinterpret_cast<const uint8_t*>(sraw);
    const int rowb = 4 * nwords, xoff = 4 * xw0;
    constexpr int ES = (int)sizeof(T);
    auto rawv = [&](const uint8_t* p) -> float { return (float)*reinterpret_cast<const T*>(p); };
    const int r_t = t / BQ, q = 4 * (t - (t / BQ) * BQ);
    const float fxlo = (float)ix0, fxhi = (float)(ix1 - 1), fylo = (float)iy0, fyhi = (float)(iy1 - 1);
    const int rbase = iy0 * rowb + xoff;
    const bool lane_on = t < RPI * BQ;
    const float xq = (float)(xb + q);
    for (int r = r_t; lane_on && r < C::BH; r += RPI) {
      float uu[4] = {0.0f, 0.0f, 0.0f, 0.0f}, vv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (Pn) {
        const int rb = s_rb[r];
        const float fy = s_rf[r];
        const int cb0 = s_cb[q];
        if constexpr (kUniformCols) {
          const float u0 = s_node[0][rb][cb0] + fy * (s_node[0][rb + 1][cb0] - s_node[0][rb][cb0]);
          const float u1 = s_node[0][rb][cb0 + 1] + fy * (s_node[0][rb + 1][cb0 + 1] - s_node[0][rb][cb0 + 1]);
          const float v0 = s_node[1][rb][cb0] + fy * (s_node[1][rb + 1][cb0] - s_node[1][rb][cb0]);
          const float v1 = s_node[1][rb][cb0 + 1] + fy * (s_node[1][rb + 1][cb0 + 1] - s_node[1][rb][cb0 + 1]);
          const float du = u1 - u0, dv = v1 - v0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float fx = s_cf[min(q + e, C::BW - 1)];
            uu[e] = u0 + fx * du;
            vv[e] = v0 + fx * dv;
          }
        } else {
          float Vu[3], Vv[3];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            Vu[j] = s_node[0][rb][cb0 + j] + fy * (s_node[0][rb + 1][cb0 + j] - s_node[0][rb][cb0 + j]);
            Vv[j] = s_node[1][rb][cb0 + j] + fy * (s_node[1][rb + 1][cb0 + j] - s_node[1][rb][cb0 + j]);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int qq = min(q + e, C::BW - 1);
            const bool nxt = s_cb[qq] != cb0;
            const float fx = s_cf[qq];
            const float ul = nxt ? Vu[1] : Vu[0], ur = nxt ? Vu[2] : Vu[1];
            const float vl = nxt ? Vv[1] : Vv[0], vr = nxt ? Vv[2] : Vv[1];
            uu[e] = ul + fx * (ur - ul);
            vv[e] = vl + fx * (vr - vl);
          }
        }
      }
      const float yr = (float)(yb + r);
      float out[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float qx = (xq + (float)e) + sgnB * uu[e], qy = yr + sgnB * vv[e];
        const float fx0 = floorf(qx), fy0 = floorf(qy);
        const float fx = qx - fx0, fy = qy - fy0;
        const int ix = (int)__builtin_amdgcn_fmed3f(fx0, fxlo, fxhi);
        const int iy = (int)__builtin_amdgcn_fmed3f(fy0, fylo, fyhi);
        const uint8_t* p0 = rawb + (iy * rowb + ix * ES) - rbase;
        const float p00 = rawv(p0), p01 = rawv(p0 + ES), p10 = rawv(p0 + rowb), p11 = rawv(p0 + rowb + ES);
        const float top = p00 + fx * (p01 - p00), bot = p10 + fx * (p11 - p10);
        out[e] = (top + fy * (bot - top)) - K;
      }
      *reinterpret_cast<float4*>(sB + r * C::BP + q) = make_float4(out[0], out[1], out[2], out[3]);
    }
  } else {
    for (int idx = t; idx < C::BH * C::BW; idx += NT) {
      int r = idx / C::BW, q = idx % C::BW;
      int y = yb + r, x = xb + q;
      float v;
      if (Pn) {
        float u, w;
        interp_tab(r, q, u, w);
        v = bilin<T>(Bi, g.pitch, g.W, g.H, x + sgnB * u, y + sgnB * w);
      } else {
        v = pixf<T>(Bi, g.pitch, g.W, g.H, y, x);
      }
      sB[r * C::BP + q] = v - K;
    }
  }
  __syncthreads();
  // A window statistics: four threads per window, four rows... of 2 STEP each
  if (t < 4 * C::NWIN) {
    int w = t >> 2, p = t & 3;
    int wi = w / TW, wj = w % TW;
    float s = 0.0f, ss = 0.0f;
    for (int r = p; r < 2 * STEP; r += 4) {
      const float* row = sA + (wi * STEP + r) * C::AP + wj * STEP;
#pragma unroll
      for (int q = 0; q < 2 * STEP; ++q) {
        float v = row[q];
        s += v;
        ss += v * v;
      }
    }
    s += __shfl_xor(s, 1);
    ss += __shfl_xor(ss, 1);
    s += __shfl_xor(s, 2);
    ss += __shfl_xor(ss, 2);
    if (p == 0) {
      s_wsum[w] = s;
      s_wsq[w] = ss;
    }
  }

  // ---- per cell and shift band: P = sum (A-K)(B'-K), S = sum (B'-K), Q = sum (B'-K)^2
  constexpr int BRW = STEP + 2 * R;   // B' columns one cell row needs
  float Pacc[SYG][C::NSY];
  float Sacc[SYG][C::NSY], Qacc[SYG][C::NSY];
  const int lrow = (t & 63) / C::CW;
  const int cj = (t & 63) - lrow * C::CW;
  const int grow = (t >> 6) * RPW + lrow;                // over (band, cell row)
  const bool worker = lrow < RPW && grow < C::NG * C::CH;
  const int grp = grow / C::CH, ci = grow - grp * C::CH;
  const int cell = ci * C::CW + cj;
  if (worker) {
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < C::NSY; ++j) Pacc[k][j] = 0.0f;
    float cs[BRW], cq[BRW];
#pragma unroll
    for (int x = 0; x < BRW; ++x) cs[x] = cq[x] = 0.0f;
    const float* abase = sA + (ci * STEP) * C::AP + cj * STEP;
    const float* bbase = sB + (ci * STEP + grp * SYG) * C::BP + cj * STEP;
    float br[SYG][BRW];
    // rows of the band for py = 0
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int x = 0; x < BRW; ++x) br[k][x] = bbase[k * C::BP + x];
#pragma unroll
    for (int py = 0; py < STEP; ++py) {
      float ar[STEP];
#pragma unroll
      for (int x = 0; x < STEP; ++x) ar[x] = abase[py * C::AP + x];
#pragma unroll
      for (int x = 0; x < BRW; ++x) {
        cs[x] += br[0][x];
        cq[x] += br[0][x] * br[0][x];
      }
#pragma unroll
      for (int k = 0; k < SYG; ++k)
#pragma unroll
        for (int j = 0; j < C::NSY; ++j) {
          float s = Pacc[k][j];
#pragma unroll
          for (int x = 0; x < STEP; ++x) s += ar[x] * br[k][x + j];
          Pacc[k][j] = s;
        }
      if (py + 1 < STEP) {
        // slide the band one row down
#pragma unroll
        for (int k = 0; k + 1 < SYG; ++k)
#pragma unroll
          for (int x = 0; x < BRW; ++x) br[k][x] = br[k + 1][x];
#pragma unroll
        for (int x = 0; x < BRW; ++x) br[SYG - 1][x] = bbase[(py + SYG) * C::BP + x];
      }
    }
    // column sums for the band's first row -> window-free cell box sums
#pragma unroll
    for (int k = 0; k < SYG; ++k) {
      if (k > 0) {
        const float* rin = bbase + (STEP + k - 1) * C::BP;
        const float* rout = bbase + (k - 1) * C::BP;
#pragma unroll
        for (int x = 0; x < BRW; ++x) {
          float vi = rin[x], vo = rout[x];
          cs[x] += vi - vo;
          cq[x] += vi * vi - vo * vo;
        }
      }
      float s = 0.0f, q = 0.0f;
#pragma unroll
      for (int x = 0; x < STEP; ++x) {
        s += cs[x];
        q += cq[x];
      }
      Sacc[k][0] = s;
      Qacc[k][0] = q;
#pragma unroll
      for (int j = 1; j < C::NSY; ++j) {
        s += cs[j + STEP - 1] - cs[j - 1];
        q += cq[j + STEP - 1] - cq[j - 1];
        Sacc[k][j] = s;
        Qacc[k][j] = q;
      }
    }
  }
  __syncthreads();   // everyone is done with the A and B' tiles
  // ---- windows, one shift band at a time.  Band b (shift rows
  // [b SYG, (b+1) SYG)) of every cell goes to LDS buffer X[b & 1] as three
  // arrays [cell][CSTR]; the window's four threads take PER consecutive
  // shifts each, stored at p*SLOTW so that every thread reads aligned
  // 16-byte chunks.  While band b is read, band b+1 is written to the other
  // buffer.
  constexpr int PER = C::PER, SLOTW = C::SLOTW, BANDP = C::BANDP, NB = C::NBS;
  constexpr int XB = C::XBUF, CSTR = C::CSTR, WSTR = C::WSTR;
  const int w = t >> 2, p = t & 3;
  const bool wact = t < 4 * C::NWIN;
  const int wi = w / TW, wj = w - (w / TW) * TW;
  const int c00 = wi * C::CW + wj, c10 = c00 + C::CW;
  // a cell plus its right-hand neighbour (the next lane: wave_shl:1 DPP);
  // the sum is garbage only in the last column, which no window uses
  auto hpair = [](float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, false));
  };
  auto write_band = [&](float* X) {
    // slot o of the band (row o / NSY, column o % NSY) sits at
    // (o / PER) * SLOTW + o % PER; what is stored is the sum over the cell
    // and its right-hand neighbour
#pragma unroll
    for (int v4 = 0; v4 < BANDP / 4; ++v4) {
      float p4[4], s4[4], q4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pos = 4 * v4 + e, th = pos / SLOTW, i = pos % SLOTW;
        const int o = th * PER + i;
        const bool real = i < PER && o < NB;
        const int k = real ? o / C::NSY : 0, j = real ? o % C::NSY : 0;
        p4[e] = real ? hpair(Pacc[k][j]) : 0.0f;
        s4[e] = real ? hpair(Sacc[k][j]) : 0.0f;
        q4[e] = real ? hpair(Qacc[k][j]) : 1.0f;
      }
      reinterpret_cast<float4*>(X + cell * CSTR)[v4] = make_float4(p4[0], p4[1], p4[2], p4[3]);
      reinterpret_cast<float4*>(X + XB / 3 + cell * CSTR)[v4] = make_float4(s4[0], s4[1], s4[2], s4[3]);
      reinterpret_cast<float4*>(X + 2 * (XB / 3) + cell * CSTR)[v4] = make_float4(q4[0], q4[1], q4[2], q4[3]);
    }
  };
  float* const X0 = s_u;
  float* const X1 = s_u + XB;
  if (worker && grp == 0) write_band(X0);
  __syncthreads();

  float rho[C::NG][PER];
  float best = -2.0f;
  int bkey = 1 << 30, nflat = 0;
  const float n = (float)(4 * STEP * STEP);
  float mA = 0.0f, varA = 0.0f;
  bool flatA = true;
  if (wact) {
    const float sa = s_wsum[w], saa = s_wsq[w];
    mA = sa / n;
    varA = saa - sa * mA;
    flatA = !(varA > kFlatRel * saa);
  }
#pragma unroll
  for (int bnd = 0; bnd < C::NG; ++bnd) {
    const float* X = (bnd & 1) ? X1 : X0;
    if (bnd + 1 < C::NG && worker && grp == bnd + 1) write_band((bnd & 1) ? X0 : X1);
#pragma unroll
    for (int i = 0; i < PER; ++i) rho[bnd][i] = 0.0f;
    if (wact) {
      float Pv[SLOTW], Sv[SLOTW], Qv[SLOTW];
#pragma unroll
      for (int v4 = 0; v4 < SLOTW / 4; ++v4) {
        auto ld = [&](int arr, int c) {
          return reinterpret_cast<const float4*>(X + arr * (XB / 3) + c * CSTR + p * SLOTW)[v4];
        };
        // stored values already hold (cell + right neighbour): the window
        // is its top pair plus its bottom pair
        const float4 P0 = ld(0, c00), P2 = ld(0, c10);
        const float4 S0 = ld(1, c00), S2 = ld(1, c10);
        const float4 Q0 = ld(2, c00), Q2 = ld(2, c10);
        Pv[4 * v4 + 0] = P0.x + P2.x;
        Pv[4 * v4 + 1] = P0.y + P2.y;
        Pv[4 * v4 + 2] = P0.z + P2.z;
        Pv[4 * v4 + 3] = P0.w + P2.w;
        Sv[4 * v4 + 0] = S0.x + S2.x;
        Sv[4 * v4 + 1] = S0.y + S2.y;
        Sv[4 * v4 + 2] = S0.z + S2.z;
        Sv[4 * v4 + 3] = S0.w + S2.w;
        Qv[4 * v4 + 0] = Q0.x + Q2.x;
        Qv[4 * v4 + 1] = Q0.y + Q2.y;
        Qv[4 * v4 + 2] = Q0.z + Q2.z;
        Qv[4 * v4 + 3] = Q0.w + Q2.w;
      }
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int key = s_tkey[(bnd * 4 + p) * PER + i];   // kKeyNone: not a used shift
        float num = Pv[i] - mA * Sv[i];
        float varB = Qv[i] - Sv[i] * Sv[i] / n;
        bool flat = flatA || !(varB > kFlatRel * Qv[i]);
        float r = flat ? 0.0f : num * rsqrtf(varA * varB);
        if (key != kKeyNone) {
          nflat += flat;
          if (!g.fixed && better(r, key, best, bkey)) {
            best = r;
            bkey = key;
          }
        }
        rho[bnd][i] = r;
      }
    }
    __syncthreads();
  }
  // reduce over the window's four lanes
#pragma unroll
  for (int o = 1; o <= 2; o <<= 1) {
    float ob = __shfl_xor(best, o);
    int ok = __shfl_xor(bkey, o);
    nflat += __shfl_xor(nflat, o);
    if (better(ob, ok, best, bkey)) {
      best = ob;
      bkey = ok;
    }
  }
  // coefficients of the window for the fit, in the buffer no round reads
  // any more: [window][band][thread][SLOTW], windows WSTR apart
  float* const rhoW = (C::NG & 1) ? X1 : X0;
  if (wact) {
#pragma unroll
    for (int bnd = 0; bnd < C::NG; ++bnd) {
      float* d = rhoW + w * WSTR + bnd * BANDP + p * SLOTW;
#pragma unroll
      for (int i = 0; i < PER; ++i) d[i] = rho[bnd][i];
    }
  }
  __syncthreads();
  if (wact && p == 0) {
    const int a = a0 + wi, b = b0 + wj;
    if (a < g.ny && b < g.nx) {
      int sy = 0, sx = 0;
      if (!g.fixed) {
        sx = (bkey & 63) - 32;
        sy = ((bkey >> 6) & 63) - 32;
      }
      const float* rr = rhoW + w * WSTR;
      auto rhof = [&](int y, int x) {
        const int yi = y + R, bnd = yi / SYG;
        const int o = (yi - bnd * SYG) * C::NSY + x + R;
        return rr[bnd * BANDP + (o / PER) * SLOTW + o % PER];
      };
      float pu = 0.0f, pv = 0.0f;
      if (Pn) window_mean_half_overlap(a, b, g.nx, g.ny, node, pu, pv);
      finish_vector(g, pair, a, b, sy, sx, nflat == (g.fixed ? 5 : C::NS), pu, pv, rhof);
    }
  }
}

// ---------------------------------------------------------------------------
// Band per wave (win = 2 step, frames deformed by the whole predictor): a
// workgroup owns TW x TH windows whose (TW+1)(TH+1) <= 64 cells map one to a
// lane, and wave g correlates every cell with shift band g (SYG rows of
// shifts).  Window sums are pair sums of lanes, the right-hand cell by DPP
// and the cell below by a lane permute, so that after the products the only
// LDS traffic is one coefficient per window and shift.  The A cell stays in
// registers as packed pixels.  Small LDS and register footprints give four
// workgroups per compute unit.
// ---------------------------------------------------------------------------
template <int STEP, int R, int SYG, int TW, int TH>
struct BandCfg {
  static constexpr int CW = TW + 1, CH = TH + 1, NC = CW * CH;
  static constexpr int NSY = 2 * R + 1, NS = NSY * NSY, NG = NSY / SYG;
  static constexpr int AW = CW * STEP, AH = CH * STEP;
  static constexpr int BW = AW + 2 * R, BH = AH + 2 * R;
  static constexpr int BP = (BW + 3) / 4 * 4 + 4;   // B' row pitch (floats)
  static constexpr int NNX = BW / STEP + 4, NNY = BH / STEP + 3;
  static constexpr int NWIN = TW * TH;
  // union after the B' tile: raw source box + interpolation tables while the
  // tile is deformed, then coefficients [window][shift] and the per-band
  // peaks [band][window] (value, key << 1 | all shifts flat)
  static constexpr int BW4 = (BW + 3) / 4 * 4;            // B' columns written (whole groups)
  static constexpr int TAB_WORDS = 2 * (BH + BW4);
  static constexpr int RES_WORDS = NWIN * NS + 2 * NG * NWIN;
  static constexpr int RAW_WORDS = 3888;   // raw source box of B
  static constexpr int UNION = RAW_WORDS + TAB_WORDS > RES_WORDS ? RAW_WORDS + TAB_WORDS : RES_WORDS;
  static_assert(NC <= 64, "a cell per lane");
  static_assert(NSY % SYG == 0, "shift rows must split evenly");
  static_assert(STEP % 2 == 0 && STEP > 4, "50% overlap; a group of four pixels spans two node columns");
};

template <typename T, int STEP, int R, int SYG, int TW, int TH>
__global__ __launch_bounds__(64 * ((2 * R + 1) / SYG)) __attribute__((amdgpu_waves_per_eu(3)))
void k_correct_bands(CorrArgs g) {
  using C = BandCfg<STEP, R, SYG, TW, TH>;
  constexpr int NT = 64 * C::NG;
  constexpr int ES = (int)sizeof(T);
  constexpr int NWR = STEP * ES / 4;   // words per cell row
  static_assert(((STEP / 2) * ES) % 4 == 0 && (STEP * ES) % 4 == 0, "cell rows are whole aligned words");
  __shared__ __align__(16) float sB[C::BH * C::BP];
  __shared__ __align__(16) float s_un[C::UNION];
  __shared__ float s_node[2][C::NNY][C::NNX];
  __shared__ float s_asum[2][ES == 1 ? 1 : C::NG][64];   // u16 cell sums, per wave

  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(g.mask, pair)) return;
  const int t = threadIdx.x, lane = t & 63;
  const int band = __builtin_amdgcn_readfirstlane(t >> 6);
  const int a0 = wg.y * TH, b0 = wg.x * TW;
  const int y0 = a0 * STEP - STEP / 2, x0 = b0 * STEP - STEP / 2;   // A tile origin
  const int yb = y0 - R, xb = x0 - R;                              // B' tile origin
  const uint8_t* Ai = g.A + (int64_t)pair * g.stride;
  const uint8_t* Bi = g.B + (int64_t)pair * g.stride;
  const int np = g.nx * g.ny;
  const float* Pn = g.pred ? g.pred + (int64_t)pair * 2 * np : nullptr;
  const bool cell_ok = lane < C::NC;
  const int ci = cell_ok ? lane / C::CW : 0, cj = cell_ok ? lane - (lane / C::CW) * C::CW : 0;

  // predictor nodes covering the B' tile: every wave reads all of them and
  // takes their range itself (no barrier before the raw box is requested)
  const float cen = 0.5f * (float)(STEP - 1);
  const int nlo_y = max(0, (int)floorf(((float)yb - cen) / STEP));
  const int nlo_x = max(0, (int)floorf(((float)xb - cen) / STEP));
  constexpr int NNODE = C::NNY * C::NNX, NL = (NNODE + 63) / 64;
  float nu[NL], nv[NL];
  if (Pn) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = min(lane + 64 * i, NNODE - 1);
      const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
      const int o = __umul24(min(nlo_y + r, g.ny - 1), g.nx) + min(nlo_x + q, g.nx - 1);
      nu[i] = Pn[(unsigned)o];
      nv[i] = Pn[(unsigned)(np + o)];
    }
  }
  // the A cell of this lane as packed pixels (zero outside the image)
  // a frame whose bytes fit 31 bits (pitch below 2^24) is addressed by 32-bit
  // offsets from its base, with 24-bit products
  const bool off32 = g.pitch < (1 << 24) && g.pitch * (int64_t)g.H <= 0x7fffffff;
  const unsigned pitch32 = (unsigned)g.pitch;
  uint32_t aw[STEP][NWR];
  {
    const int rowbytes = g.W * ES;
    const int xa0 = (x0 + cj * STEP) * ES;
    if (off32 && y0 >= 0 && y0 + C::AH <= g.H && x0 >= 0 && (x0 + C::AW) * ES <= rowbytes) {
      // the whole A tile lies inside the image
      const uint32_t ok = cell_ok ? 0xffffffffu : 0u;
      const unsigned o0 = __umul24((unsigned)(y0 + ci * STEP), pitch32) + (unsigned)xa0;
#pragma unroll
      for (int py = 0; py < STEP; ++py)
#pragma unroll
        for (int k = 0; k < NWR; ++k)
          aw[py][k] = *reinterpret_cast<const uint32_t*>(Ai + (size_t)(o0 + py * pitch32 + 4 * k)) & ok;
    } else {
#pragma unroll
      for (int py = 0; py < STEP; ++py) {
        const int y = y0 + ci * STEP + py;
        const uint32_t ok = (cell_ok && (unsigned)y < (unsigned)g.H) ? 0xffffffffu : 0u;
        const uint8_t* row = Ai + (int64_t)min(max(y, 0), g.H - 1) * g.pitch;
#pragma unroll
        for (int k = 0; k < NWR; ++k) aw[py][k] = masked_word(row, rowbytes, xa0 + 4 * k) & ok;
      }
    }
  }
  // range of the nodes as integer floors: the raw box only needs floor(u)
  // and floor(v) (the tile origin is an integer).  A node that is not finite
  // or not below 100 px marks the tile (range 255), which sends it to the
  // checked path.
  int flu = 0, fhu = 0, flv = 0, fhv = 0;
  if (Pn) {
    float lu = nu[0], hu = nu[0], lv = nv[0], hv = nv[0];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      lu = fminf(lu, nu[i]);
      hu = fmaxf(hu, nu[i]);
      lv = fminf(lv, nv[i]);
      hv = fmaxf(hv, nv[i]);
      ok = ok && fabsf(nu[i]) < 100.0f && fabsf(nv[i]) < 100.0f;   // false for NaN
    }
    // encoded so that a max serves every bound: 127 - floor(lo) and
    // floor(hi) + 128, two 16-bit fields per word, each reduced on its own
    const uint32_t el_u = ok ? 127 - (int)floorf(lu) : 255, eh_u = ok ? (int)floorf(hu) + 128 : 255;
    const uint32_t el_v = ok ? 127 - (int)floorf(lv) : 255, eh_v = ok ? (int)floorf(hv) + 128 : 255;
    const uint32_t ru = wave_max_pk16((el_u << 16) | eh_u), rv = wave_max_pk16((el_v << 16) | eh_v);
    flu = 127 - (int)(ru >> 16);
    fhu = (int)(ru & 0xffffu) - 128;
    flv = 127 - (int)(rv >> 16);
    fhv = (int)(rv & 0xffffu) - 128;
    if (band == 0) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int idx = lane + 64 * i;
        if (idx < NNODE) {
          const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
          s_node[0][r][q] = nu[i];
          s_node[1][r][q] = nv[i];
        }
      }
    }
  }

  // raw source box of B for the deformation, when it fits
  const int ix0 = xb + flu - 1;
  const int ix1 = xb + C::BW - 1 + fhu + 2;
  const int iy0 = yb + flv - 1;
  const int iy1 = yb + C::BH - 1 + fhv + 2;
  const int xw0 = (ix0 * ES) >> 2;
  const int nwords = ((ix1 * ES + ES - 1) >> 2) - xw0 + 1;
  const int nrows = iy1 - iy0 + 1;
  // (a displacement range that is marked or wider than a window takes the
  // unstaged path, whose reads are checked one by one)
  const bool sane = fhu - flu < 64 && fhv - flv < 64;
  const bool staged = sane && nwords <= NT && nwords * nrows <= C::RAW_WORDS;
  uint32_t* sraw = reinterpret_cast<uint32_t*>(s_un);
  int* s_rb = reinterpret_cast<int*>(s_un + C::RAW_WORDS);   // per B' row: base node, fraction
  float* s_rf = s_un + C::RAW_WORDS + C::BH;
  int* s_cb = reinterpret_cast<int*>(s_un + C::RAW_WORDS + 2 * C::BH);   // per B' column
  float* s_cf = s_un + C::RAW_WORDS + 2 * C::BH + C::BW4;
  if (staged) {
    // thread -> (word column, first row); U reads in flight per thread
    const int rowbytes = g.W * ES;
    const int rstep = NT / nwords;
    const int r0 = t / nwords, w = t - r0 * nwords;
    // reads in flight per thread: enough for the whole box in one round
    // (about 9 rows per thread for u8)
    constexpr int U = 12;
    const bool inside = off32 && iy0 >= 0 && iy0 + nrows <= g.H && xw0 >= 0 && 4 * (xw0 + nwords) <= rowbytes;
    if (r0 < rstep) {
      // slots past the box take its last row again (the same word is
      // written twice with the same value), so the stores need no branch
      for (int rb = r0; rb < nrows; rb += U * rstep) {
        uint32_t val[U];
        if (inside) {
          const unsigned col = 4u * (unsigned)(xw0 + w);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const unsigned y = (unsigned)(iy0 + min(rb + u * rstep, nrows - 1));
            val[u] = *reinterpret_cast<const uint32_t*>(Bi + (size_t)(__umul24(y, pitch32) + col));
          }
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int y = iy0 + min(rb + u * rstep, nrows - 1);
            const uint32_t ok = (unsigned)y < (unsigned)g.H ? 0xffffffffu : 0u;
            val[u] = masked_word(Bi + (int64_t)min(max(y, 0), g.H - 1) * g.pitch, rowbytes, 4 * (xw0 + w)) & ok;
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) sraw[min(rb + u * rstep, nrows - 1) * nwords + w] = val[u];
      }
    }
  }
  // interpolation tables of the B' tile (the same arithmetic as interp_u)
  // (columns past BW pad the last group: written to B', never correlated)
  for (int i = t; i < C::BH + C::BW4; i += NT) {
    const bool row = i < C::BH;
    const int p = row ? yb + i : xb + (i - C::BH);
    const int n = row ? g.ny : g.nx;
    float tt = fminf(fmaxf(((float)p - cen) / (float)STEP, 0.0f), (float)(n - 1));
    int bb = min((int)tt, max(n - 2, 0));
    float ff = tt - (float)bb;
    if (row) { s_rb[i] = bb - nlo_y; s_rf[i] = ff; }
    else { s_cb[i - C::BH] = bb - nlo_x; s_cf[i - C::BH] = ff; }
  }
  // the tile offset K: the rounded mean of the A tile (every wave holds all
  // of its cells and reduces them in the same order)
  int isum = 0;
#pragma unroll
  for (int py = 0; py < STEP; ++py)
#pragma unroll
    for (int k = 0; k < NWR; ++k) {
      if constexpr (ES == 1) isum = (int)__builtin_amdgcn_sad_u8(aw[py][k], 0u, (uint32_t)isum);
      else isum = (int)__builtin_amdgcn_sad_u16(aw[py][k], 0u, (uint32_t)isum);
    }
  isum = wave_sum(isum);
  const float K = (float)((isum + C::AH * C::AW / 2) / (C::AH * C::AW));   // (isum >= 0)
  // u16: the cell's sums of (A-K) and (A-K)^2 in FP32, rows dealt to the
  // waves (row py to wave py mod NG); the partial sums meet in LDS
  if constexpr (ES != 1) {
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int py = 0; py < STEP; ++py) {
      if (py % C::NG != band) continue;
#pragma unroll
      for (int x = 0; x < STEP; ++x) {
        const uint32_t wd = aw[py][(x * ES) >> 2];
        const float d = (float)((wd >> (16 * (x & 1))) & 0xffffu) - K;
        s1 += d;
        s2 += d * d;
      }
    }
    s_asum[0][band][lane] = s1;
    s_asum[1][band][lane] = s2;
  }
  __syncthreads();

  // deformed B' tile, in groups of four pixels of one row
  if (staged) {
    constexpr int BQ = (C::BW + 3) / 4;
    constexpr bool kUniformCols = (STEP + R) % 4 == 0;
    const uint8_t* rawb = reinterpret_cast<const uint8_t*>(sraw);
    const int rowb = 4 * nwords, xoff = 4 * xw0;
    auto rawv = [&](const uint8_t* p) -> float { return (float)*reinterpret_cast<const T*>(p); };
    // coordinates relative to the box: every real pixel lands at >= 1 (the
    // box has a one-pixel margin), so truncation is the floor; the clamps
    // only keep the padding columns of a ragged last group inside the box
    const int ixhi = ix1 - 1 - ix0, iyhi = iy1 - 1 - iy0;
    const int xadd = ix0 * ES - xoff;   // byte offset of box column 0 in a staged row
    const uint8_t* rawx = rawb + xadd;  // (folded into the base: one multiply-add per pixel)
    // one group of four pixels; two groups per pass, so that one group's
    // LDS round trips overlap the other's arithmetic
    auto group = [&](int idx) __attribute__((always_inline)) {
      const int r = idx / BQ, q = 4 * (idx - (idx / BQ) * BQ);
      float uu[4] = {0.0f, 0.0f, 0.0f, 0.0f}, vv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (Pn) {
        const int rb = s_rb[r];
        const float fy = s_rf[r];
        const int cb0 = s_cb[q];
        if constexpr (kUniformCols) {
          const float u0 = s_node[0][rb][cb0] + fy * (s_node[0][rb + 1][cb0] - s_node[0][rb][cb0]);
          const float u1 = s_node[0][rb][cb0 + 1] + fy * (s_node[0][rb + 1][cb0 + 1] - s_node[0][rb][cb0 + 1]);
          const float v0 = s_node[1][rb][cb0] + fy * (s_node[1][rb + 1][cb0] - s_node[1][rb][cb0]);
          const float v1 = s_node[1][rb][cb0 + 1] + fy * (s_node[1][rb + 1][cb0 + 1] - s_node[1][rb][cb0 + 1]);
          const float du = u1 - u0, dv = v1 - v0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float fx = s_cf[q + e];
            uu[e] = u0 + fx * du;
            vv[e] = v0 + fx * dv;
          }
        } else {
          float Vu[3], Vv[3];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            Vu[j] = s_node[0][rb][cb0 + j] + fy * (s_node[0][rb + 1][cb0 + j] - s_node[0][rb][cb0 + j]);
            Vv[j] = s_node[1][rb][cb0 + j] + fy * (s_node[1][rb + 1][cb0 + j] - s_node[1][rb][cb0 + j]);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool nxt = s_cb[q + e] != cb0;
            const float fx = s_cf[q + e];
            const float ul = nxt ? Vu[1] : Vu[0], ur = nxt ? Vu[2] : Vu[1];
            const float vl = nxt ? Vv[1] : Vv[0], vr = nxt ? Vv[2] : Vv[1];
            uu[e] = ul + fx * (ur - ul);
            vv[e] = vl + fx * (vr - vl);
          }
        }
      }
      const float yr = (float)(yb + r - iy0), xq = (float)(xb + q - ix0);
      float out[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float qx = (xq + (float)e) + uu[e], qy = yr + vv[e];
        const float fx = __builtin_amdgcn_fractf(qx), fy = __builtin_amdgcn_fractf(qy);
        // Without padding columns the box bounds every coordinate: qx lies in
        // [q + e + 1 - floor(lo) + lo, q + e + 1 - floor(lo) + hi] up to the
        // interpolation's rounding, so floor(qx) is in [0, ixhi] (and its
        // right-hand neighbour in the box), likewise in y; with padding
        // columns the clamps keep their reads inside the box.  (As unsigned,
        // a negative index would clamp to the top as well.)
        unsigned ix = (unsigned)(int)qx, iy = (unsigned)(int)qy;
        if constexpr (C::BW4 != C::BW) {
          ix = min(ix, (unsigned)ixhi);
          iy = min(iy, (unsigned)iyhi);
        }
        const uint8_t* p0 = rawx + (__umul24(iy, (unsigned)rowb) + ix * ES);
        const float p00 = rawv(p0), p01 = rawv(p0 + ES), p10 = rawv(p0 + rowb), p11 = rawv(p0 + rowb + ES);
        const float top = p00 + fx * (p01 - p00), bot = p10 + fx * (p11 - p10);
        out[e] = (top + fy * (bot - top)) - K;
      }
      *reinterpret_cast<float4*>(sB + r * C::BP + q) = make_float4(out[0], out[1], out[2], out[3]);
    };
    constexpr int NGR = C::BH * BQ;
    int idx = t;
    for (; idx + NT < NGR; idx += 2 * NT) {
      group(idx);
      group(idx + NT);
    }
    if (idx < NGR) group(idx);
  } else {
    for (int idx = t; idx < C::BH * C::BW; idx += NT) {
      const int r = idx / C::BW, q = idx - (idx / C::BW) * C::BW;
      const int y = yb + r, x = xb + q;
      float v;
      if (Pn) {
        const int rb = s_rb[r], cb = s_cb[q];
        const float fy = s_rf[r], fx = s_cf[q];
        const float u = (1.0f - fy) * ((1.0f - fx) * s_node[0][rb][cb] + fx * s_node[0][rb][cb + 1]) +
                        fy * ((1.0f - fx) * s_node[0][rb + 1][cb] + fx * s_node[0][rb + 1][cb + 1]);
        const float w = (1.0f - fy) * ((1.0f - fx) * s_node[1][rb][cb] + fx * s_node[1][rb][cb + 1]) +
                        fy * ((1.0f - fx) * s_node[1][rb + 1][cb] + fx * s_node[1][rb + 1][cb + 1]);
        v = bilin<T>(Bi, g.pitch, g.W, g.H, x + u, y + w);
      } else {
        v = pixf<T>(Bi, g.pitch, g.W, g.H, y, x);
      }
      sB[r * C::BP + q] = v - K;
    }
  }
  __syncthreads();

  // ---- this lane's cell against the wave's shift band: P = sum A (B'-K),
  // S = sum (B'-K), Q = sum (B'-K)^2, and the cell's own sum (A-K), (A-K)^2
  // (the covariance sum (A-K)(B'-K) - mean(A-K) S equals P - mean(A) S)
  constexpr int BRW = STEP + 2 * R;   // B' columns one cell row needs
  float Pacc[SYG][C::NSY], Sacc[SYG][C::NSY], Qacc[SYG][C::NSY];
  float sa = 0.0f, saa = 0.0f;
  if constexpr (ES == 1) {
    // the cell's sums of (A-K) and (A-K)^2 from exact integer sums of A, A^2
    uint32_t s1 = 0u, s2 = 0u;
#pragma unroll
    for (int py = 0; py < STEP; ++py)
#pragma unroll
      for (int k = 0; k < NWR; ++k) {
        s1 = __builtin_amdgcn_sad_u8(aw[py][k], 0u, s1);
        s2 = __builtin_amdgcn_udot4(aw[py][k], aw[py][k], s2, false);
      }
    const int Ki = (int)K;
    sa = (float)((int)s1 - STEP * STEP * Ki);
    saa = (float)((int)s2 - 2 * Ki * (int)s1 + STEP * STEP * Ki * Ki);
  } else {
#pragma unroll
    for (int q = 0; q < C::NG; ++q) {
      sa += s_asum[0][q][lane];
      saa += s_asum[1][q][lane];
    }
  }
  const float* bbase = sB + (ci * STEP + band * SYG) * C::BP + cj * STEP;
  float cs[BRW], cq[BRW];
  {
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < C::NSY; ++j) Pacc[k][j] = 0.0f;
#pragma unroll
    for (int x = 0; x < BRW; ++x) cs[x] = cq[x] = 0.0f;
    // stream the B' rows of the band once each; B' row rb meets A row
    // rb - k for shift row k, so the last SYG A rows are kept (converted)
    float ar[SYG][STEP];
#pragma unroll
    for (int rb = 0; rb < STEP + SYG - 1; ++rb) {
      float brow[BRW];
#pragma unroll
      for (int x = 0; x < BRW; ++x) brow[x] = bbase[rb * C::BP + x];
      if (rb < STEP) {
        float* an = ar[rb % SYG];
#pragma unroll
        for (int x = 0; x < STEP; ++x) {
          const uint32_t wd = aw[rb][(x * ES) >> 2];
          const uint32_t px = ES == 1 ? (wd >> (8 * (x & 3))) & 0xffu : (wd >> (16 * (x & 1))) & 0xffffu;
          an[x] = (float)px;   // raw A: the offset K enters through the mean below
        }
#pragma unroll
        for (int x = 0; x < BRW; ++x) {
          cs[x] += brow[x];
          cq[x] += brow[x] * brow[x];
        }
      }
#pragma unroll
      for (int k = 0; k < SYG; ++k) {
        const int py = rb - k;
        if (py >= 0 && py < STEP) {
          const float* ap = ar[py % SYG];
#pragma unroll
          for (int j = 0; j < C::NSY; ++j) {
            float s = Pacc[k][j];
#pragma unroll
            for (int x = 0; x < STEP; ++x) s += ap[x] * brow[x + j];
            Pacc[k][j] = s;
          }
        }
      }
    }
  }
  {
    // column sums of the band's first row, slid down for the other rows;
    // box sums over STEP columns for every shift column
#pragma unroll
    for (int k = 0; k < SYG; ++k) {
      if (k > 0) {
        const float* rin = bbase + (STEP + k - 1) * C::BP;
        const float* rout = bbase + (k - 1) * C::BP;
#pragma unroll
        for (int x = 0; x < BRW; ++x) {
          const float vi = rin[x], vo = rout[x];
          cs[x] += vi - vo;
          cq[x] += vi * vi - vo * vo;
        }
      }
      float s = 0.0f, q = 0.0f;
#pragma unroll
      for (int x = 0; x < STEP; ++x) {
        s += cs[x];
        q += cq[x];
      }
      Sacc[k][0] = s;
      Qacc[k][0] = q;
#pragma unroll
      for (int j = 1; j < C::NSY; ++j) {
        s += cs[j + STEP - 1] - cs[j - 1];
        q += cq[j + STEP - 1] - cq[j - 1];
        Sacc[k][j] = s;
        Qacc[k][j] = q;
      }
    }
  }
  // ---- window sums: (cell + right-hand neighbour) by DPP wave_shl:1, then
  // + the same pair one cell row down (lane + CW) by a lane permute.  Only
  // lanes of a window's top-left cell keep meaningful sums.
  auto quad = [&](float x) {
    const float h = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, false));
    return h + __int_as_float(__builtin_amdgcn_ds_bpermute((lane + C::CW) << 2, __float_as_int(h)));
  };
  sa = quad(sa);
  saa = quad(saa);
#pragma unroll
  for (int k = 0; k < SYG; ++k)
#pragma unroll
    for (int j = 0; j < C::NSY; ++j) {
      Pacc[k][j] = quad(Pacc[k][j]);
      Sacc[k][j] = quad(Sacc[k][j]);
      Qacc[k][j] = quad(Qacc[k][j]);
    }
  // ---- Pearson coefficient per shift, the band's peak by the tie key
  const bool wact = cell_ok && ci < TH && cj < TW;
  const int w = ci * TW + cj;
  float* const rhoW = s_un;                      // [window][shift]
  float* const s_best = s_un + C::NWIN * C::NS;  // [band][window]
  int* const s_pk = reinterpret_cast<int*>(s_best + C::NG * C::NWIN);
  {
    constexpr float kInvN = 1.0f / (float)(4 * STEP * STEP);
    const float mA = sa * kInvN;
    const float varA = saa - sa * mA;
    const float meanA = K + mA;
    const bool flatA = !(varA > kFlatRel * saa);
    // coefficients first (no control flow), then the band's peak
    float rv[SYG][C::NSY];
    bool allflat = true;   // every used shift of the band is flat
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < C::NSY; ++j) {
        const int sy = band * SYG + k - R, sx = j - R;
        const float num = Pacc[k][j] - meanA * Sacc[k][j];
        const float varB = Qacc[k][j] - Sacc[k][j] * Sacc[k][j] * kInvN;
        const bool flat = flatA || !(varB > kFlatRel * Qacc[k][j]);
        // (varA varB > 0 unless flat; the flat value replaces the quotient)
        const float r = num * __builtin_amdgcn_rsqf(varA * varB);
        rv[k][j] = flat ? 0.0f : r;
        const bool used = !g.fixed || sx == 0 || sy == 0;
        if (used) allflat = allflat && flat;
      }
    // the band's peak: the largest coefficient, then the smallest tie key
    // among the shifts that reach it
    float best = -2.0f;
    int bkey = 1 << 20;
    if (!g.fixed) {
#pragma unroll
      for (int k = 0; k < SYG; ++k)
#pragma unroll
        for (int j = 0; j < C::NSY; ++j) best = fmaxf(best, rv[k][j]);
#pragma unroll
      for (int k = 0; k < SYG; ++k)
#pragma unroll
        for (int j = 0; j < C::NSY; ++j)
          bkey = rv[k][j] == best ? min(bkey, tie_key(band * SYG + k - R, j - R)) : bkey;
    }
    if (wact) {
      float* d = rhoW + w * C::NS + band * SYG * C::NSY;
#pragma unroll
      for (int k = 0; k < SYG; ++k)
#pragma unroll
        for (int j = 0; j < C::NSY; ++j) d[k * C::NSY + j] = rv[k][j];
      s_best[band * C::NWIN + w] = best;
      s_pk[band * C::NWIN + w] = (bkey << 1) | (allflat ? 1 : 0);
    }
  }
  __syncthreads();
  // ---- peak over the bands, fit, composition with the predictor's window mean
  // (VALU issue bounds the kernel: one wave fits them all and the others end)
  const int wt = t;
  if (t < C::NWIN) {
    const int wi = wt / TW, wj = wt - (wt / TW) * TW;
    const int a = a0 + wi, b = b0 + wj;
    if (a < g.ny && b < g.nx) {
      float best = -2.0f;
      int bkey = 1 << 20;
      bool allflat = true;
#pragma unroll
      for (int q = 0; q < C::NG; ++q) {
        const float bq = s_best[q * C::NWIN + wt];
        const int pk = s_pk[q * C::NWIN + wt];
        allflat = allflat && (pk & 1);
        if (better(bq, pk >> 1, best, bkey)) {
          best = bq;
          bkey = pk >> 1;
        }
      }
      int sy = 0, sx = 0;
      if (!g.fixed) {
        sx = (bkey & 63) - 32;
        sy = ((bkey >> 6) & 63) - 32;
      }
      const float* rr = rhoW + wt * C::NS;
      auto rhof = [&](int y, int x) { return rr[(y + R) * C::NSY + x + R]; };
      auto node = [&](int c, int y, int x) { return s_node[c][y - nlo_y][x - nlo_x]; };
      float pu = 0.0f, pv = 0.0f;
      if (Pn) window_mean_half_overlap(a, b, g.nx, g.ny, node, pu, pv);
      finish_vector(g, pair, a, b, sy, sx, allflat, pu, pv, rhof);
    }
  }
}

// ---------------------------------------------------------------------------
// Two waves per shift band (win = 2 step, r 4): the band kernel above for
// 24 px windows, and for 16 px windows with both frames deformed (kCentral),
// whose LDS lets a CU hold two workgroups.  Three waves each would leave
// SIMDs with one wave.  The waves of a band share its shifts by columns (4
// and 5 of the 9), and of the box sums of B' one takes S and the other Q for
// all nine; what the other needs passes through LDS per window.  The packed
// A cells wait in LDS over the raw box (with kCentral A', as floats, in LDS
// of its own), so that a wave stays within 128 registers and four fit a
// SIMD.  Two more waves share the staging, the deformation and the fits:
// with six a SIMD would hold two waves of a workgroup or one, and a launch
// of 384 threads runs 15% (24 px) and 4% (central) longer.  What bounds it
// now is VALU issue (24 px: 450 of 524 us; central 131 of 175 us), beside it
// latency.  24 px windows: A as it is against B' - K, every sum in the band
// kernel's order; 8 x 4K u16 606 -> 524 us (three waves with the A cell in
// 72 of 256 registers, 9 spilled).  kCentral: A' is brought to K in LDS once
// the tile's sum is known, so that (A' - K)(B' - K) is summed as in
// k_correct_tiled, which served these windows (with A' as it is, bright
// frames were up to 3e-3 off in the coefficient, now 5e-6; 3,400 of 12 bits,
// particles of 150), and K is the mean of the tile's pixels inside the image,
// so that tiles over its edge lose no bits either (k_correct_tiled 2e-3);
// 16 x 1000 x 760 u8 215 -> 178 us (k_correct_tiled).
// ---------------------------------------------------------------------------
template <int N>
using Int = std::integral_constant<int, N>;

template <typename T, int STEP, int TW, int TH, bool kCentral>
struct HalvesCfg {
  static constexpr int ES = (int)sizeof(T), R = 4, SYG = 3;
  static constexpr int CW = TW + 1, CH = TH + 1, NC = CW * CH, NWIN = TW * TH;
  static constexpr int NSY = 2 * R + 1, NS = NSY * NSY, NG = NSY / SYG;
  static constexpr int H0 = 4, H1 = NSY - H0;             // shift columns of the two waves of a band
  static constexpr int NT = 512;
  static constexpr int AW = CW * STEP, AH = CH * STEP;
  static constexpr int BW = AW + 2 * R, BH = AH + 2 * R;
  static constexpr int BP = (BW + 3) / 4 * 4 + 4, AP = AW + 4;   // LDS row pitches (floats)
  static constexpr int NNX = BW / STEP + 4, NNY = BH / STEP + 3;
  static constexpr int TAB_WORDS = 2 * (BH + BW);
  // union: raw source box and interpolation tables while the tiles are
  // deformed; then what a wave of a band hands the other (S of H1 columns, Q
  // of H0 per window), and behind it the coefficients and the waves' peaks
  // (over the packed A cells, which the products read)
  static constexpr int XW = NG * NWIN * SYG * NSY;
  static constexpr int CP = STEP * (STEP * ES / 4) + 4;   // words per packed cell (rows of whole words)
  static constexpr int AW_WORDS = kCentral ? 0 : 64 * CP;
  static constexpr int RES0 = NWIN * NS + 4 * NG * NWIN;
  static constexpr int RES_WORDS = XW + (RES0 > AW_WORDS ? RES0 : AW_WORDS);
  static constexpr int RAW_WORDS = STEP == 8 ? 3888 : ((BW + 19) * 2 / 4 + 2) * (BH + 19);
  static constexpr int UNION = RAW_WORDS + TAB_WORDS > RES_WORDS ? RAW_WORDS + TAB_WORDS : RES_WORDS;
  static constexpr int A_WORDS = kCentral ? AH * AP : 0;
  static constexpr int LDS_WORDS = BH * BP + A_WORDS + UNION + 2 * NNY * NNX + 2 * NG * 64 + NT / 64;
  static_assert(NC <= 64 && BW % 4 == 0 && STEP % 4 == 0 && R % 4 == 0, "a cell per lane; whole groups of four pixels");
};

template <typename T, int STEP, int TW, int TH, bool kCentral>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
void k_correct_halves(CorrArgs g) {
  using C = HalvesCfg<T, STEP, TW, TH, kCentral>;
  constexpr int NT = C::NT, ES = C::ES, R = C::R, SYG = C::SYG, NSY = C::NSY;
  constexpr int NWR = STEP * ES / 4;   // words per cell row
  static_assert(NT == 512 && ((STEP / 2) * ES) % 4 == 0 && (STEP * ES) % 4 == 0, "cell rows are whole aligned words");
  // (all LDS is dynamic: told of 80 KB, the compiler reserves the registers
  // of the four waves a SIMD then holds as if no other workgroup fitted)
  extern __shared__ __align__(16) float s_dyn[];
  float* const sB = s_dyn;
  float* const sA = sB + C::BH * C::BP;
  float* const s_un = sA + C::A_WORDS;
  float(*const s_node)[C::NNY][C::NNX] = reinterpret_cast<float(*)[C::NNY][C::NNX]>(s_un + C::UNION);
  // cell sums of A - K and its square, rows dealt to the bands
  float(*const s_asum)[C::NG][64] = reinterpret_cast<float(*)[C::NG][64]>(s_un + C::UNION + 2 * C::NNY * C::NNX);
  float* const s_red = s_un + C::UNION + 2 * C::NNY * C::NNX + 2 * C::NG * 64;

  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(g.mask, pair)) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), band = wave >> 1;
  const int half = wave < 2 * C::NG ? wave & 1 : 2;   // 2: no shifts
  const int a0 = wg.y * TH, b0 = wg.x * TW;
  const int y0 = a0 * STEP - STEP / 2, x0 = b0 * STEP - STEP / 2;   // A tile origin
  const int yb = y0 - R, xb = x0 - R;                              // B' tile origin
  const uint8_t* Ai = g.A + (int64_t)pair * g.stride;
  const uint8_t* Bi = g.B + (int64_t)pair * g.stride;
  const int np = g.nx * g.ny, rowbytes = g.W * ES;
  const float* Pn = g.pred ? g.pred + (int64_t)pair * 2 * np : nullptr;
  const bool cell_ok = lane < C::NC;
  const int ci = cell_ok ? lane / C::CW : 0, cj = cell_ok ? lane - (lane / C::CW) * C::CW : 0;

  // predictor nodes covering the B' tile: every wave reads all of them and
  // takes their range itself (no barrier before the raw box is requested)
  const float cen = 0.5f * (float)(STEP - 1);
  const int nlo_y = max(0, (int)floorf(((float)yb - cen) / STEP));
  const int nlo_x = max(0, (int)floorf(((float)xb - cen) / STEP));
  constexpr int NNODE = C::NNY * C::NNX, NL = (NNODE + 63) / 64;
  float nu[NL], nv[NL];
  if (Pn) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = min(lane + 64 * i, NNODE - 1);
      const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
      const int o = __umul24(min(nlo_y + r, g.ny - 1), g.nx) + min(nlo_x + q, g.nx - 1);
      nu[i] = Pn[(unsigned)o];
      nv[i] = Pn[(unsigned)(np + o)];
    }
  }
  // a frame whose bytes fit 31 bits (pitch below 2^24) is addressed by 32-bit
  // offsets from its base, with 24-bit products
  const bool off32 = g.pitch < (1 << 24) && g.pitch * (int64_t)g.H <= 0x7fffffff;
  const unsigned pitch32 = (unsigned)g.pitch;
  // rows band, band + 3, .. of this lane's A cell as packed pixels (zero
  // outside the image), by the second wave of the band
  constexpr int NAR = kCentral ? 1 : STEP / C::NG;
  static_assert(kCentral || STEP % C::NG == 0, "cell rows split evenly over the bands");
  uint32_t aw[NAR][NWR];
  if (!kCentral && half == 1) {
    const int xa0 = (x0 + cj * STEP) * ES;
    const bool inside = off32 && y0 >= 0 && y0 + C::AH <= g.H && x0 >= 0 && (x0 + C::AW) * ES <= rowbytes;
#pragma unroll
    for (int i = 0; i < NAR; ++i) {
      const int y = y0 + ci * STEP + band + C::NG * i;
      if (inside) {
        const unsigned o = __umul24((unsigned)y, pitch32) + (unsigned)xa0;
#pragma unroll
        for (int k = 0; k < NWR; ++k)
          aw[i][k] = cell_ok ? *reinterpret_cast<const uint32_t*>(Ai + (size_t)(o + 4 * k)) : 0u;
      } else {
        const uint32_t ok = (cell_ok && (unsigned)y < (unsigned)g.H) ? 0xffffffffu : 0u;
        const uint8_t* row = Ai + (int64_t)min(max(y, 0), g.H - 1) * g.pitch;
#pragma unroll
        for (int k = 0; k < NWR; ++k) aw[i][k] = masked_word(row, rowbytes, xa0 + 4 * k) & ok;
      }
    }
  }
  // range of the (scaled) nodes as integer floors: see k_correct_bands
  float lu = 0.0f, hu = 0.0f, lv = 0.0f, hv = 0.0f;
  bool nodes_ok = true;
  if (Pn) {
    lu = hu = nu[0];
    lv = hv = nv[0];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      lu = fminf(lu, nu[i]);
      hu = fmaxf(hu, nu[i]);
      lv = fminf(lv, nv[i]);
      hv = fmaxf(hv, nv[i]);
      nodes_ok = nodes_ok && fabsf(nu[i]) < 100.0f && fabsf(nv[i]) < 100.0f;   // false for NaN
    }
    if (t < 64) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int idx = lane + 64 * i;
        if (idx < NNODE) {
          const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
          s_node[0][r][q] = nu[i];
          s_node[1][r][q] = nv[i];
        }
      }
    }
  }
  uint32_t* sraw = reinterpret_cast<uint32_t*>(s_un);
  int* s_rb = reinterpret_cast<int*>(s_un + C::RAW_WORDS);   // per B' row: base node, fraction
  float* s_rf = s_un + C::RAW_WORDS + C::BH;
  int* s_cb = reinterpret_cast<int*>(s_un + C::RAW_WORDS + 2 * C::BH);   // per B' column
  float* s_cf = s_un + C::RAW_WORDS + 2 * C::BH + C::BW;
  // stage the raw source box of a frame for its tile rows x cols at (ty, tx)
  // deformed by sgn * u, when it fits
  struct Box { int ix0, iy0, nwords; bool staged; };
  auto stage = [&](const uint8_t* img, int ty, int tx, int rows, int cols, float sgn) __attribute__((always_inline)) {
    int flu = 0, fhu = 0, flv = 0, fhv = 0;
    if (Pn) {
      const float xl = sgn < 0.0f ? sgn * hu : sgn * lu, xh = sgn < 0.0f ? sgn * lu : sgn * hu;
      const float yl = sgn < 0.0f ? sgn * hv : sgn * lv, yh = sgn < 0.0f ? sgn * lv : sgn * hv;
      // encoded so that a max serves every bound: 127 - floor(lo) and
      // floor(hi) + 128, two 16-bit fields per word, each reduced on its own;
      // 255 marks the tile
      const uint32_t el_u = nodes_ok ? 127 - (int)floorf(xl) : 255, eh_u = nodes_ok ? (int)floorf(xh) + 128 : 255;
      const uint32_t el_v = nodes_ok ? 127 - (int)floorf(yl) : 255, eh_v = nodes_ok ? (int)floorf(yh) + 128 : 255;
      const uint32_t ru = wave_max_pk16((el_u << 16) | eh_u), rv = wave_max_pk16((el_v << 16) | eh_v);
      flu = 127 - (int)(ru >> 16);
      fhu = (int)(ru & 0xffffu) - 128;
      flv = 127 - (int)(rv >> 16);
      fhv = (int)(rv & 0xffffu) - 128;
    }
    Box b;
    b.ix0 = tx + flu - 1;
    b.iy0 = ty + flv - 1;
    const int ix1 = tx + cols - 1 + fhu + 2, iy1 = ty + rows - 1 + fhv + 2;
    const int xw0 = (b.ix0 * ES) >> 2;
    b.nwords = ((ix1 * ES + ES - 1) >> 2) - xw0 + 1;
    const int nrows = iy1 - b.iy0 + 1;
    b.staged = fhu - flu < 64 && fhv - flv < 64 && b.nwords <= NT && b.nwords * nrows <= C::RAW_WORDS;
    if (b.staged) {
      // thread -> (word column, first row); U reads in flight per thread
      const int rstep = NT / b.nwords;
      const int r0 = t / b.nwords, w = t - r0 * b.nwords;
      constexpr int U = STEP == 8 ? 5 : 14;
      const bool inside = off32 && b.iy0 >= 0 && b.iy0 + nrows <= g.H && xw0 >= 0 && 4 * (xw0 + b.nwords) <= rowbytes;
      if (r0 < rstep) {
        // slots past the box take its last row again (the same word is
        // written twice with the same value), so the stores need no branch
        for (int rb = r0; rb < nrows; rb += U * rstep) {
          uint32_t val[U];
          if (inside) {
            const unsigned col = 4u * (unsigned)(xw0 + w);
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const unsigned y = (unsigned)(b.iy0 + min(rb + u * rstep, nrows - 1));
              val[u] = *reinterpret_cast<const uint32_t*>(img + (size_t)(__umul24(y, pitch32) + col));
            }
          } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int y = b.iy0 + min(rb + u * rstep, nrows - 1);
              const uint32_t ok = (unsigned)y < (unsigned)g.H ? 0xffffffffu : 0u;
              val[u] = masked_word(img + (int64_t)min(max(y, 0), g.H - 1) * g.pitch, rowbytes, 4 * (xw0 + w)) & ok;
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) sraw[min(rb + u * rstep, nrows - 1) * b.nwords + w] = val[u];
        }
      }
    }
    return b;
  };
  // deform the tile (ROWS x COLS at (ty, tx), tables from row / column TO)
  // by sgn * u, minus K, into dst (pitch DP); returns the thread's sum
  auto deform = [&](const uint8_t* img, const Box& b, int ty, int tx, auto rows_c, auto cols_c, auto to_c, auto dp_c,
                    float sgn, float K, float* dst) __attribute__((always_inline)) {
    constexpr int ROWS = decltype(rows_c)::value, COLS = decltype(cols_c)::value, TO = decltype(to_c)::value;
    constexpr int DP = decltype(dp_c)::value;
    float sum = 0.0f;
    if (b.staged) {
      // groups of four pixels of one row, two groups per pass, so that one
      // group's LDS round trips overlap the other's arithmetic; coordinates
      // relative to the box, where the floor is a truncation and every corner
      // lies inside (see k_correct_bands)
      constexpr int BQ = COLS / 4;
      const int rowb = 4 * b.nwords, xadd = b.ix0 * ES - 4 * ((b.ix0 * ES) >> 2);
      const uint8_t* rawx = reinterpret_cast<const uint8_t*>(sraw) + xadd;
      auto rawv = [&](const uint8_t* p) -> float { return (float)*reinterpret_cast<const T*>(p); };
      auto group = [&](int idx) __attribute__((always_inline)) {
        const int r = idx / BQ, q = 4 * (idx - (idx / BQ) * BQ);
        float uu[4] = {0.0f, 0.0f, 0.0f, 0.0f}, vv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (Pn) {
          // (no group straddles a node column: step and r are multiples of 4)
          const int rb = s_rb[TO + r];
          const float fy = s_rf[TO + r];
          const int cb0 = s_cb[TO + q];
          const float u0 = s_node[0][rb][cb0] + fy * (s_node[0][rb + 1][cb0] - s_node[0][rb][cb0]);
          const float u1 = s_node[0][rb][cb0 + 1] + fy * (s_node[0][rb + 1][cb0 + 1] - s_node[0][rb][cb0 + 1]);
          const float v0 = s_node[1][rb][cb0] + fy * (s_node[1][rb + 1][cb0] - s_node[1][rb][cb0]);
          const float v1 = s_node[1][rb][cb0 + 1] + fy * (s_node[1][rb + 1][cb0 + 1] - s_node[1][rb][cb0 + 1]);
          const float du = u1 - u0, dv = v1 - v0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float fx = s_cf[TO + q + e];
            uu[e] = u0 + fx * du;
            vv[e] = v0 + fx * dv;
            if constexpr (kCentral) {
              uu[e] *= sgn;
              vv[e] *= sgn;
            }
          }
        }
        const float yr = (float)(ty + r - b.iy0), xq = (float)(tx + q - b.ix0);
        float out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float qx = (xq + (float)e) + uu[e], qy = yr + vv[e];
          const float fx = __builtin_amdgcn_fractf(qx), fy = __builtin_amdgcn_fractf(qy);
          const unsigned ix = (unsigned)(int)qx, iy = (unsigned)(int)qy;
          const uint8_t* p0 = rawx + (__umul24(iy, (unsigned)rowb) + ix * ES);
          const float p00 = rawv(p0), p01 = rawv(p0 + ES), p10 = rawv(p0 + rowb), p11 = rawv(p0 + rowb + ES);
          const float top = p00 + fx * (p01 - p00), bot = p10 + fx * (p11 - p10);
          out[e] = (top + fy * (bot - top)) - K;
        }
        if constexpr (kCentral) sum += (out[0] + out[1]) + (out[2] + out[3]);
        *reinterpret_cast<float4*>(dst + r * DP + q) = make_float4(out[0], out[1], out[2], out[3]);
      };
      constexpr int NGR = ROWS * BQ;
      int idx = t;
      for (; idx + NT < NGR; idx += 2 * NT) {
        group(idx);
        group(idx + NT);
      }
      if (idx < NGR) group(idx);
    } else {
      for (int idx = t; idx < ROWS * COLS; idx += NT) {
        const int r = idx / COLS, q = idx - (idx / COLS) * COLS;
        const int y = ty + r, x = tx + q;
        float v;
        if (Pn) {
          const int rb = s_rb[TO + r], cb = s_cb[TO + q];
          const float fy = s_rf[TO + r], fx = s_cf[TO + q];
          const float u = (1.0f - fy) * ((1.0f - fx) * s_node[0][rb][cb] + fx * s_node[0][rb][cb + 1]) +
                          fy * ((1.0f - fx) * s_node[0][rb + 1][cb] + fx * s_node[0][rb + 1][cb + 1]);
          const float w = (1.0f - fy) * ((1.0f - fx) * s_node[1][rb][cb] + fx * s_node[1][rb][cb + 1]) +
                          fy * ((1.0f - fx) * s_node[1][rb + 1][cb] + fx * s_node[1][rb + 1][cb + 1]);
          v = bilin<T>(img, g.pitch, g.W, g.H, kCentral ? x + sgn * u : x + u, kCentral ? y + sgn * w : y + w);
        } else {
          v = pixf<T>(img, g.pitch, g.W, g.H, y, x);
        }
        sum += v == v ? v : 0.0f;   // (a node that is not finite leaves the other windows' K alone)
        dst[r * DP + q] = v - K;
      }
    }
    return sum;
  };
  // interpolation tables of the B' tile (the same arithmetic as interp_u)
  for (int i = t; i < C::BH + C::BW; i += NT) {
    const bool row = i < C::BH;
    const int p = row ? yb + i : xb + (i - C::BH);
    const int n = row ? g.ny : g.nx;
    float tt = fminf(fmaxf(((float)p - cen) / (float)STEP, 0.0f), (float)(n - 1));
    int bb = min((int)tt, max(n - 2, 0));
    float ff = tt - (float)bb;
    if (row) { s_rb[i] = bb - nlo_y; s_rf[i] = ff; }
    else { s_cb[i - C::BH] = bb - nlo_x; s_cf[i - C::BH] = ff; }
  }
  auto unpack = [](const uint32_t (&wd)[NWR], float (&an)[STEP]) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < STEP; ++x) {
      const uint32_t v = wd[(x * ES) >> 2];
      an[x] = (float)(ES == 1 ? (v >> (8 * (x & 3))) & 0xffu : (v >> (16 * (x & 1))) & 0xffffu);
    }
  };
  // pixel row py of this lane's A cell as floats
  uint32_t* const s_cell = reinterpret_cast<uint32_t*>(s_un + C::XW) + lane * C::CP;
  auto arow = [&](int py, float (&an)[STEP]) __attribute__((always_inline)) {
    if constexpr (kCentral) {
      const float* p = sA + (ci * STEP + py) * C::AP + cj * STEP;
#pragma unroll
      for (int x = 0; x < STEP; ++x) an[x] = p[x];
    } else {
      uint32_t wd[NWR];
#pragma unroll
      for (int k = 0; k < NWR; ++k) wd[k] = s_cell[py * NWR + k];
      unpack(wd, an);
    }
  };
  // K, the rounded mean of the A tile (kCentral: A' is held about it, too),
  // and the cells' sums of A - K and its square (rows dealt to the bands, by
  // the second wave of each)
  float K;
  auto cell_sums = [&]() __attribute__((always_inline)) {
    float s1 = 0.0f, s2 = 0.0f;
    auto add = [&](const float (&an)[STEP]) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < STEP; ++x) {
        const float d = kCentral ? an[x] : an[x] - K;
        s1 += d;
        s2 += d * d;
      }
    };
    float an[STEP];
    if constexpr (kCentral) {
#pragma unroll
      for (int py = 0; py < STEP; ++py) {
        if (py % C::NG != band) continue;
        arow(py, an);
        add(an);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NAR; ++i) {
        unpack(aw[i], an);
        add(an);
      }
    }
    s_asum[0][band][lane] = s1;
    s_asum[1][band][lane] = s2;
  };
  if constexpr (kCentral) {
    const Box ba = stage(Ai, y0, x0, C::AH, C::AW, -0.5f);
    __syncthreads();
    float part = deform(Ai, ba, y0, x0, Int<C::AH>(), Int<C::AW>(), Int<R>(), Int<C::AP>(), -0.5f, 0.0f, sA);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) s_red[t >> 6] = part;
    __syncthreads();
    K = 0.0f;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) K += s_red[i];
    // (of the pixels inside the image: the last tiles reach beyond it)
    const int nin = (min(y0 + C::AH, g.H) - max(y0, 0)) * (min(x0 + C::AW, g.W) - max(x0, 0));
    K = rintf(K / (float)nin);
    constexpr int AQ = C::AW / 4;
    for (int i = t; i < C::AH * AQ; i += NT) {
      float4* p = reinterpret_cast<float4*>(sA + (i / AQ) * C::AP) + (i - (i / AQ) * AQ);
      const float4 v = *p;
      *p = make_float4(v.x - K, v.y - K, v.z - K, v.w - K);
    }
  } else {
    // (integers: the waves' sums meet exactly)
    int isum = 0;
    if (half == 1) {
#pragma unroll
      for (int i = 0; i < NAR; ++i)
#pragma unroll
        for (int k = 0; k < NWR; ++k) {
          if constexpr (ES == 1) isum = (int)__builtin_amdgcn_sad_u8(aw[i][k], 0u, (uint32_t)isum);
          else isum = (int)__builtin_amdgcn_sad_u16(aw[i][k], 0u, (uint32_t)isum);
        }
    }
    isum = wave_sum(isum);
    if (lane == 0) s_red[t >> 6] = __int_as_float(isum);
  }
  const Box bb = stage(Bi, yb, xb, C::BH, C::BW, kCentral ? 0.5f : 1.0f);
  __syncthreads();
  if constexpr (!kCentral) {
    int isum = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) isum += __float_as_int(s_red[i]);
    K = (float)((isum + C::AH * C::AW / 2) / (C::AH * C::AW));   // (isum >= 0)
  }
  if (half == 1) cell_sums();
  deform(Bi, bb, yb, xb, Int<C::BH>(), Int<C::BW>(), Int<0>(), Int<C::BP>(), kCentral ? 0.5f : 1.0f, K, sB);
  if constexpr (!kCentral) {
    // the packed cells take the raw box's place
    __syncthreads();
    if (half == 1) {
#pragma unroll
      for (int i = 0; i < NAR; ++i)
#pragma unroll
        for (int k = 0; k < NWR; ++k) s_cell[(band + C::NG * i) * NWR + k] = aw[i][k];
    }
  }
  __syncthreads();

  // ---- this lane's cell against the wave's shifts
  constexpr int BRW = STEP + 2 * R;   // B' columns one cell row needs
  const float* bbase = sB + (ci * STEP + band * SYG) * C::BP + cj * STEP;
  // window sums: (cell + right-hand neighbour) by DPP wave_shl:1, then + the
  // same pair one cell row down (lane + CW) by a lane permute.  Only lanes of
  // a window's top-left cell keep meaningful sums.
  auto quad = [&](float x) {
    const float h = x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, false));
    return h + __int_as_float(__builtin_amdgcn_ds_bpermute((lane + C::CW) << 2, __float_as_int(h)));
  };
  // P = sum A (B' - K) (kCentral: of (A' - K) (B' - K)) of the shift columns
  // J0 .. J0 + NJ - 1: the B' rows of the band streamed once each; B' row rb
  // meets A row rb - k for shift row k, so the last SYG A rows are kept
  auto products = [&](auto j0_c, auto nj_c, float (&P)[SYG][C::H1]) __attribute__((always_inline)) {
    constexpr int J0 = decltype(j0_c)::value, NJ = decltype(nj_c)::value, NB = STEP + NJ - 1;
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < C::H1; ++j) P[k][j] = 0.0f;
    float ar[SYG][STEP];
#pragma unroll
    for (int rb = 0; rb < STEP + SYG - 1; ++rb) {
      float brow[NB];
#pragma unroll
      for (int x = 0; x < NB; ++x) brow[x] = bbase[rb * C::BP + J0 + x];
      if (rb < STEP) arow(rb, ar[rb % SYG]);
#pragma unroll
      for (int k = 0; k < SYG; ++k) {
        const int py = rb - k;
        if (py >= 0 && py < STEP) {
          const float* ap = ar[py % SYG];
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            float s = P[k][j];
#pragma unroll
            for (int x = 0; x < STEP; ++x) s += ap[x] * brow[x + j];
            P[k][j] = s;
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // (one row's reads ahead would not fit the registers)
    }
  };
  // box sums of B' - K (kSq: of its square) over STEP columns for every
  // shift: column sums of the band's first STEP rows, slid down for the
  // other rows
  auto boxes = [&](auto sq_c, float (&o)[SYG][NSY]) __attribute__((always_inline)) {
    constexpr bool kSq = decltype(sq_c)::value;
    float c[BRW];
#pragma unroll
    for (int x = 0; x < BRW; ++x) c[x] = 0.0f;
#pragma unroll
    for (int rb = 0; rb < STEP; ++rb) {
#pragma unroll
      for (int x = 0; x < BRW; ++x) {
        const float b = bbase[rb * C::BP + x];
        if constexpr (kSq) c[x] += b * b;
        else c[x] += b;
      }
    }
#pragma unroll
    for (int k = 0; k < SYG; ++k) {
      if (k > 0) {
        const float* rin = bbase + (STEP + k - 1) * C::BP;
        const float* rout = bbase + (k - 1) * C::BP;
#pragma unroll
        for (int x = 0; x < BRW; ++x) {
          const float vi = rin[x], vo = rout[x];
          if constexpr (kSq) c[x] += vi * vi - vo * vo;
          else c[x] += vi - vo;
        }
      }
      float s = 0.0f;
#pragma unroll
      for (int x = 0; x < STEP; ++x) s += c[x];
      o[k][0] = s;
#pragma unroll
      for (int j = 1; j < NSY; ++j) {
        s += c[j + STEP - 1] - c[j - 1];
        o[k][j] = s;
      }
    }
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < NSY; ++j) o[k][j] = quad(o[k][j]);
  };
  const bool wact = cell_ok && ci < TH && cj < TW;
  const int w = ci * TW + cj;
  float sa = 0.0f, saa = 0.0f;
#pragma unroll
  for (int q = 0; q < C::NG; ++q) {
    sa += s_asum[0][q][lane];
    saa += s_asum[1][q][lane];
  }
  sa = quad(sa);
  saa = quad(saa);
  float P[SYG][C::H1], SQ[SYG][NSY];   // SQ: S in the band's first wave, Q in its second
  // what the other wave needs: [band][shift row][column][window]
  float* const sx = s_un + band * (C::NWIN * SYG * NSY) + w;
  if (half == 0) {
    products(Int<0>(), Int<C::H0>(), P);
    boxes(std::false_type(), SQ);
  } else if (half == 1) {
    products(Int<C::H0>(), Int<C::H1>(), P);
    boxes(std::true_type(), SQ);
  }
  if (half < 2) {
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < C::H1; ++j) P[k][j] = quad(P[k][j]);
  }
  // (the raw box and the tables were last read before the barrier above)
  if (wact && half < 2) {
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < NSY; ++j)
        if ((j >= C::H0) == (half == 0)) sx[(k * NSY + j) * C::NWIN] = SQ[k][j];
  }
  __syncthreads();
  // ---- Pearson coefficient per shift, the wave's peak by the tie key
  float* const rhoW = s_un + C::XW;                    // [window][shift]
  float* const s_best = rhoW + C::NWIN * C::NS;        // [wave][window]
  int* const s_pk = reinterpret_cast<int*>(s_best + 2 * C::NG * C::NWIN);
  auto peak = [&](auto j0_c, auto nj_c) __attribute__((always_inline)) {
    constexpr int J0 = decltype(j0_c)::value, NJ = decltype(nj_c)::value;
    constexpr float kInvN = 1.0f / (float)(4 * STEP * STEP);
    const float mA = sa * kInvN;
    const float varA = saa - sa * mA;
    const float meanA = kCentral ? mA : K + mA;   // (of what the products took)
    const bool flatA = !(varA > kFlatRel * saa);
    float rv[SYG][NJ];
    bool allflat = true;   // every used shift of the wave is flat
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float other = wact ? sx[(k * NSY + J0 + j) * C::NWIN] : 1.0f;
        const float S = J0 == 0 ? SQ[k][J0 + j] : other, Q = J0 == 0 ? other : SQ[k][J0 + j];
        const float num = P[k][j] - meanA * S;
        const float varB = Q - S * S * kInvN;
        const bool flat = flatA || !(varB > kFlatRel * Q);
        // (varA varB > 0 unless flat; the flat value replaces the quotient)
        const float r = num * __builtin_amdgcn_rsqf(varA * varB);
        rv[k][j] = flat ? 0.0f : r;
        allflat = allflat && flat;
      }
    float best = -2.0f;
    int bkey = 1 << 20;
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < NJ; ++j) best = fmaxf(best, rv[k][j]);
#pragma unroll
    for (int k = 0; k < SYG; ++k)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        bkey = rv[k][j] == best ? min(bkey, tie_key(band * SYG + k - R, J0 + j - R)) : bkey;
    if (wact) {
      float* d = rhoW + w * C::NS + band * SYG * NSY + J0;
#pragma unroll
      for (int k = 0; k < SYG; ++k)
#pragma unroll
        for (int j = 0; j < NJ; ++j) d[k * NSY + j] = rv[k][j];
      s_best[wave * C::NWIN + w] = best;
      s_pk[wave * C::NWIN + w] = (bkey << 1) | (allflat ? 1 : 0);
    }
  };
  if (half == 0) peak(Int<0>(), Int<C::H0>());
  else if (half == 1) peak(Int<C::H0>(), Int<C::H1>());
  __syncthreads();
  // ---- peak over the waves, fit, composition with the predictor's window
  // mean; the windows are dealt to the waves
  constexpr int WPW = C::NWIN / (2 * C::NG);
  static_assert(WPW * 2 * C::NG == C::NWIN, "windows split evenly over the waves");
  const int wt = wave * WPW + lane;
  if (lane < WPW && half < 2) {
    const int wi = wt / TW, wj = wt - (wt / TW) * TW;
    const int a = a0 + wi, b = b0 + wj;
    if (a < g.ny && b < g.nx) {
      float best = -2.0f;
      int bkey = 1 << 20;
      bool allflat = true;
#pragma unroll
      for (int q = 0; q < 2 * C::NG; ++q) {
        const float bq = s_best[q * C::NWIN + wt];
        const int pk = s_pk[q * C::NWIN + wt];
        allflat = allflat && (pk & 1);
        if (better(bq, pk >> 1, best, bkey)) {
          best = bq;
          bkey = pk >> 1;
        }
      }
      const int sx_ = (bkey & 63) - 32, sy_ = ((bkey >> 6) & 63) - 32;
      const float* rr = rhoW + wt * C::NS;
      auto rhof = [&](int y, int x) { return rr[(y + R) * NSY + x + R]; };
      auto node = [&](int c, int y, int x) { return s_node[c][y - nlo_y][x - nlo_x]; };
      float pu = 0.0f, pv = 0.0f;
      if (Pn) window_mean_half_overlap(a, b, g.nx, g.ny, node, pu, pv);
      finish_vector(g, pair, a, b, sy_, sx_, allflat, pu, pv, rhof);
    }
  }
}

// ---------------------------------------------------------------------------
// Thread per (cell, shift row): 50%-overlap windows of large cells (win = 32,
// step 16).  A cell times its shifts is more work than a lane should hold
// and a tile of 63 cells more than a small frame has, so here a thread takes
// one cell, one row of shifts and one of PARTS interleaved parts of the
// cell's rows: it streams those rows of A and B' from LDS and keeps 2R+1
// sums of products, which PARTS neighbouring lanes add up by DPP.  The box
// sums S and Q of B' and its square are taken per cell, columns first (a
// thread per column and cell row), then along the row (a thread per cell,
// shift row and sum): sums over the rows (columns) that every shift shares,
// plus running sums at both ends, so that nothing is subtracted.  The cells'
// sums meet in LDS, where threads per window, shift row and a few columns
// form the coefficients.
// A cell's sums are taken about its own mean Kc, and a window's from its four
// cells' about the window's mean Kw: with d = Kc - Kw, n the pixels of a cell
// and P, S, s its sums of (A-Kc)(B'-Kc), B'-Kc and A-Kc,
//   sum (A-Kw)(B'-Kw) = sum over cells of P + d (S + s + n d),
// so light that differs from window to window costs no bits: 12-bit frames
// with particles of 300 under light of 3000 +- 600, error of the coefficient
// 0.8e-6 at most, as about each window's mean by itself; about the mean of a
// tile of windows, and with A as it is, 42e-6.  4 x 1024 x 512 u8 frames, r 4:
// 36.8 us, 22.6 of VALU issue beside 16.6 of LDS accesses (33.5 us about the
// tile's mean; k_correct_generic 454); one 256 x 256 pair, r 8: 13.8 us
// (generic 36), the latency of seven phases.
// Frames are deformed by the whole predictor (B only), or by half of it each
// (kCentral; A' is then held as floats, else the packed pixels are).
// ---------------------------------------------------------------------------
template <typename T, int STEP, int R, int TW, int TH, int PARTS, int NT, bool kCentral>
struct RowsCfg {
  static constexpr int ES = (int)sizeof(T);
  static constexpr int CW = TW + 1, CH = TH + 1, NC = CW * CH, NWIN = TW * TH;
  static constexpr int NSY = 2 * R + 1, WIN = 2 * STEP;
  static constexpr int AW = CW * STEP, AH = CH * STEP;
  static constexpr int BW = AW + 2 * R, BH = AH + 2 * R;
  static constexpr int odd4(int n) { return 4 * (((n + 3) / 4) | 1); }   // whole odd groups of four: rows spread over the banks
  static constexpr int BP = odd4(BW);
  static constexpr int AP = kCentral ? odd4(AW) : AW * ES / 4;           // words
  static constexpr int NNX = BW / STEP + 4, NNY = BH / STEP + 3;         // predictor nodes of the B' tile
  static constexpr int BRW = STEP + 2 * R;                               // B' columns of one cell
  static constexpr int NI = NC * NSY * PARTS;                            // items (threads) of the products
  // raw source box: the tile plus a predictor range of 17 px across it
  static constexpr int RAW = (BH + 20) * (((BW + 20) * ES + 3) / 4 + 2);
  // [raw box, then the column sums S and Q] [A] [B'], then the cells' sums
  // P, S, Q: [3][cell][shift row][shift column], and behind them the
  // coefficients [window][shift]
  static constexpr int VS = CH * NSY * BP, RES = 3 * NC * NSY * NSY;
  static constexpr int AWORDS = AH * AP;
  static constexpr int RV = kCentral ? (2 * VS > RAW + AWORDS ? 2 * VS - AWORDS : RAW) : (2 * VS > RAW ? 2 * VS : RAW);
  static constexpr int IN = (RV + 3) / 4 * 4 + AWORDS + BH * BP;
  static constexpr int OUT = RES + NWIN * NSY * NSY;
  static constexpr int TOTAL = IN > OUT ? IN : OUT;
  static_assert(NI <= NT, "one item per thread");
  static_assert(2 * NC * NSY <= NT, "a thread per cell, shift row and sum");
  // shift columns a thread turns into coefficients: as few as the threads allow
  static constexpr int JG = []() { int j = 1; while (NWIN * NSY * ((NSY + j - 1) / j) > NT) ++j; return j; }();
  static_assert(STEP == 16 && STEP % PARTS == 0 && (PARTS & (PARTS - 1)) == 0 && PARTS <= 16, "parts add up by DPP");
};

template <typename T, int STEP, int R, int TW, int TH, int PARTS, int NT, bool kCentral>
__global__ __launch_bounds__(NT) void k_correct_rows(CorrArgs g) {
  using C = RowsCfg<T, STEP, R, TW, TH, PARTS, NT, kCentral>;
  constexpr int ES = C::ES, NSY = C::NSY;
  __shared__ __align__(16) float s_mem[C::TOTAL];
  // per window: d of its cells, mean and variance of A - Kw, and what d adds
  // to P, S and Q by itself
  __shared__ __align__(16) float s_win[C::NWIN][12];
  __shared__ int s_sharp[C::NWIN];       // a used shift that is not flat
  __shared__ float s_node[2][C::NNY][C::NNX];
  __shared__ int s_rb[C::BH], s_cb[(C::BW + 3) / 4 * 4];
  __shared__ float s_rf[C::BH], s_cf[(C::BW + 3) / 4 * 4];
  __shared__ float s_cell[3][C::NC];     // per cell: Kc, sum of A - Kc and of its square
  __shared__ float s_red[NT / 64];
  float* const sV = s_mem;
  uint32_t* const sraw = reinterpret_cast<uint32_t*>(s_mem);
  float* const sA = s_mem + (C::RV + 3) / 4 * 4;
  uint32_t* const sAw = reinterpret_cast<uint32_t*>(sA);
  float* const sB = sA + C::AWORDS;
  float* const s_rho = s_mem + C::RES;

  const WgIdx wg = xcd_order();
  const int pair = wg.z;
  if (slot_off(g.mask, pair)) return;
  const int t = threadIdx.x, lane = t & 63;
  const int a0 = wg.y * TH, b0 = wg.x * TW;
  const int y0 = a0 * STEP - STEP / 2, x0 = b0 * STEP - STEP / 2;   // A tile origin
  const int yb = y0 - R, xb = x0 - R;                              // B' tile origin
  const uint8_t* Ai = g.A + (int64_t)pair * g.stride;
  const uint8_t* Bi = g.B + (int64_t)pair * g.stride;
  const int np = g.nx * g.ny, rowbytes = g.W * ES;
  const float* Pn = g.pred ? g.pred + (int64_t)pair * 2 * np : nullptr;

  // predictor nodes covering the B' tile: every wave reads all of them and
  // takes their range itself
  const float cen = 0.5f * (float)(STEP - 1);
  const int nlo_y = max(0, (int)floorf(((float)yb - cen) / STEP));
  const int nlo_x = max(0, (int)floorf(((float)xb - cen) / STEP));
  constexpr int NNODE = C::NNY * C::NNX, NL = (NNODE + 63) / 64;
  float nu[NL], nv[NL];
  if (Pn) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = min(lane + 64 * i, NNODE - 1);
      const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
      const int o = min(nlo_y + r, g.ny - 1) * g.nx + min(nlo_x + q, g.nx - 1);
      nu[i] = Pn[o];
      nv[i] = Pn[np + o];
    }
  }
  // the A tile as packed pixels (zero outside the image), and its sum
  float asum = 0.0f;
  if constexpr (!kCentral) {
    int isum = 0;
    constexpr int NA = (C::AWORDS + NT - 1) / NT;
    uint32_t w[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int idx = min(t + i * NT, C::AWORDS - 1);
      const int r = idx / C::AP, k = idx - (idx / C::AP) * C::AP;
      const int y = y0 + r;
      const uint32_t ok = (t + i * NT < C::AWORDS && (unsigned)y < (unsigned)g.H) ? 0xffffffffu : 0u;
      w[i] = masked_word(Ai + (int64_t)min(max(y, 0), g.H - 1) * g.pitch, rowbytes, x0 * ES + 4 * k) & ok;
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      if (t + i * NT < C::AWORDS) sAw[t + i * NT] = w[i];
      isum = ES == 1 ? (int)__builtin_amdgcn_sad_u8(w[i], 0u, (uint32_t)isum)
                     : (int)__builtin_amdgcn_sad_u16(w[i], 0u, (uint32_t)isum);
    }
    asum = (float)wave_sum(isum);
  }
  // interpolation tables of the B' tile (the same arithmetic as interp_u;
  // columns past BW pad the last group: written to B', never correlated)
  constexpr int BW4 = (C::BW + 3) / 4 * 4;
  for (int i = t; i < C::BH + BW4; i += NT) {
    const bool row = i < C::BH;
    const int p = row ? yb + i : xb + (i - C::BH);
    const int n = row ? g.ny : g.nx;
    const float tt = fminf(fmaxf(((float)p - cen) / (float)STEP, 0.0f), (float)(n - 1));
    const int bb = min((int)tt, max(n - 2, 0));
    const float ff = tt - (float)bb;
    if (row) { s_rb[i] = bb - nlo_y; s_rf[i] = ff; }
    else { s_cb[i - C::BH] = bb - nlo_x; s_cf[i - C::BH] = ff; }
  }
  // range of the nodes; a node that is not finite or not below 100 px marks
  // the tile, which sends it to the checked path
  float lu = 0.0f, hu = 0.0f, lv = 0.0f, hv = 0.0f;
  bool sane = true;
  if (Pn) {
    lu = hu = nu[0];
    lv = hv = nv[0];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      lu = fminf(lu, nu[i]);
      hu = fmaxf(hu, nu[i]);
      lv = fminf(lv, nv[i]);
      hv = fmaxf(hv, nv[i]);
      ok = ok && fabsf(nu[i]) < 100.0f && fabsf(nv[i]) < 100.0f;   // false for NaN
    }
    lu = wave_min(lu);
    hu = wave_max(hu);
    lv = wave_min(lv);
    hv = wave_max(hv);
    sane = __all(ok) && hu - lu < 64.0f && hv - lv < 64.0f;
    if (t < 64) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int idx = lane + 64 * i;
        if (idx < NNODE) {
          const int r = idx / C::NNX, q = idx - (idx / C::NNX) * C::NNX;
          s_node[0][r][q] = nu[i];
          s_node[1][r][q] = nv[i];
        }
      }
    }
  }
  // The raw source box of a frame for the deformation of the tile rows x
  // cols at (ty, tx) by s * u, staged when it fits: every real sample lands
  // at >= 1 and its right and lower neighbours in the box (a one-pixel
  // margin around the nodes' range).
  struct Box { int ix0, ix1, iy0, iy1, nwords; bool staged; };
  auto stage = [&](const uint8_t* img, int ty, int tx, int rows, int cols, float s) __attribute__((always_inline)) {
    const float xl = s < 0.0f ? s * hu : s * lu, xh = s < 0.0f ? s * lu : s * hu;
    const float yl = s < 0.0f ? s * hv : s * lv, yh = s < 0.0f ? s * lv : s * hv;
    Box b;
    b.ix0 = sane ? tx + (int)floorf(xl) - 1 : 0;
    b.ix1 = sane ? tx + cols - 1 + (int)floorf(xh) + 2 : 0;
    b.iy0 = sane ? ty + (int)floorf(yl) - 1 : 0;
    b.iy1 = sane ? ty + rows - 1 + (int)floorf(yh) + 2 : 0;
    const int xw0 = (b.ix0 * ES) >> 2;
    b.nwords = ((b.ix1 * ES + ES - 1) >> 2) - xw0 + 1;
    const int nrows = b.iy1 - b.iy0 + 1;
    b.staged = sane && b.nwords <= NT && b.nwords * nrows <= C::RAW;
    if (b.staged) {
      const int rstep = NT / b.nwords, r0 = t / b.nwords, w = t - r0 * b.nwords;
      constexpr int U = 8;   // reads in flight per thread
      if (r0 < rstep) {
        for (int rb = r0; rb < nrows; rb += U * rstep) {
          uint32_t val[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            // (slots past the box take its last row again: the same word is
            // written twice with the same value)
            const int y = b.iy0 + min(rb + u * rstep, nrows - 1);
            const uint32_t ok = (unsigned)y < (unsigned)g.H ? 0xffffffffu : 0u;
            val[u] = masked_word(img + (int64_t)min(max(y, 0), g.H - 1) * g.pitch, rowbytes, 4 * (xw0 + w)) & ok;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) sraw[min(rb + u * rstep, nrows - 1) * b.nwords + w] = val[u];
        }
      }
    }
    return b;
  };
  // deformed tile rows x cols4 (whole groups of four columns) at (ty, tx),
  // table rows / columns from (tr, tc), minus K, into dst; returns the
  // thread's sum
  auto deform = [&](const uint8_t* img, const Box& b, int ty, int tx, int rows, int cols4, int tr, int tc, float s,
                    float K, float* dst, int pitch, auto uniform) __attribute__((always_inline)) {
    // uniform: no group of four straddles a node column
    constexpr bool kUni = decltype(uniform)::value;
    const int nq = cols4 / 4;
    float sum = 0.0f;
    const uint8_t* rawb = reinterpret_cast<const uint8_t*>(sraw);
    const int rowb = 4 * b.nwords, xadd = b.ix0 * ES - 4 * ((b.ix0 * ES) >> 2);
    const unsigned ixhi = (unsigned)(b.ix1 - 1 - b.ix0), iyhi = (unsigned)(b.iy1 - 1 - b.iy0);
    for (int idx = t; idx < rows * nq; idx += NT) {
      const int r = idx / nq, q = 4 * (idx - (idx / nq) * nq);
      float out[4];
      if (b.staged) {
        float Vu[3] = {0.0f, 0.0f, 0.0f}, Vv[3] = {0.0f, 0.0f, 0.0f};
        int cb0 = 0;
        if (Pn) {
          const int rb = s_rb[tr + r];
          const float fy = s_rf[tr + r];
          cb0 = s_cb[tc + q];
          // (a group of four pixels spans at most two cells: three node columns)
#pragma unroll
          for (int j = 0; j < (kUni ? 2 : 3); ++j) {
            const float u0 = s_node[0][rb][cb0 + j], v0 = s_node[1][rb][cb0 + j];
            Vu[j] = u0 + fy * (s_node[0][rb + 1][cb0 + j] - u0);
            Vv[j] = v0 + fy * (s_node[1][rb + 1][cb0 + j] - v0);
          }
        }
        const float yr = (float)(ty + r - b.iy0), xq = (float)(tx + q - b.ix0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u = 0.0f, v = 0.0f;
          if (Pn) {
            const bool nxt = !kUni && s_cb[tc + q + e] != cb0;
            const float fx = s_cf[tc + q + e];
            const float ul = nxt ? Vu[1] : Vu[0], ur = nxt ? Vu[2] : Vu[1];
            const float vl = nxt ? Vv[1] : Vv[0], vr = nxt ? Vv[2] : Vv[1];
            u = s * (ul + fx * (ur - ul));
            v = s * (vl + fx * (vr - vl));
          }
          const float qx = (xq + (float)e) + u, qy = yr + v;
          const float fx = __builtin_amdgcn_fractf(qx), fy = __builtin_amdgcn_fractf(qy);
          // (the clamps only keep padding columns inside the box)
          const unsigned ix = min((unsigned)(int)qx, ixhi), iy = min((unsigned)(int)qy, iyhi);
          const uint8_t* p0 = rawb + (__umul24(iy, (unsigned)rowb) + ix * ES + xadd);
          auto px = [](const uint8_t* p) -> float { return (float)*reinterpret_cast<const T*>(p); };
          const float p00 = px(p0), p01 = px(p0 + ES), p10 = px(p0 + rowb), p11 = px(p0 + rowb + ES);
          const float top = p00 + fx * (p01 - p00), bot = p10 + fx * (p11 - p10);
          out[e] = (top + fy * (bot - top)) - K;
        }
      } else {
#pragma unroll 1
        for (int e = 0; e < 4; ++e) {
          const int y = ty + r, x = tx + q + e;
          float v;
          if (Pn) {
            const int rb = s_rb[tr + r], cb = s_cb[tc + q + e];
            const float fy = s_rf[tr + r], fx = s_cf[tc + q + e];
            const float u = (1.0f - fy) * ((1.0f - fx) * s_node[0][rb][cb] + fx * s_node[0][rb][cb + 1]) +
                            fy * ((1.0f - fx) * s_node[0][rb + 1][cb] + fx * s_node[0][rb + 1][cb + 1]);
            const float w = (1.0f - fy) * ((1.0f - fx) * s_node[1][rb][cb] + fx * s_node[1][rb][cb + 1]) +
                            fy * ((1.0f - fx) * s_node[1][rb + 1][cb] + fx * s_node[1][rb + 1][cb + 1]);
            v = bilin<T>(img, g.pitch, g.W, g.H, (float)x + s * u, (float)y + s * w);
          } else {
            v = pixf<T>(img, g.pitch, g.W, g.H, y, x);
          }
          out[e] = v - K;
        }
      }
      const float s4 = (out[0] + out[1]) + (out[2] + out[3]);
      sum += s4 == s4 ? s4 : 0.0f;   // (a node that is not finite leaves the other windows' K alone)
      *reinterpret_cast<float4*>(dst + r * pitch + q) = make_float4(out[0], out[1], out[2], out[3]);
    }
    return sum;
  };

  if constexpr (kCentral) {
    const Box ab = stage(Ai, y0, x0, C::AH, C::AW, -0.5f);
    __syncthreads();
    asum = deform(Ai, ab, y0, x0, C::AH, C::AW, R, R, -0.5f, 0.0f, sA, C::AP, std::true_type());
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) asum += __shfl_xor(asum, o);
    __syncthreads();   // the raw box of A is read
  }
  if (lane == 0) s_red[t >> 6] = asum;
  const Box bb = stage(Bi, yb, xb, C::BH, C::BW, kCentral ? 0.5f : 1.0f);
  __syncthreads();
  // K, the rounded mean of the A tile: what B' is held about
  float K = 0.0f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) K += s_red[i];
  K = rintf(K / (float)(C::AH * C::AW));
  deform(Bi, bb, yb, xb, C::BH, BW4, 0, 0, kCentral ? 0.5f : 1.0f, K, sB, C::BP,
         std::bool_constant<(STEP + R) % 4 == 0>());

  // pixel x of a cell row of A
  auto arow = [&](int cy, int cx, int py, float (&ar)[STEP]) __attribute__((always_inline)) {
    if constexpr (kCentral) {
      const float* p = sA + (cy * STEP + py) * C::AP + cx * STEP;
#pragma unroll
      for (int x = 0; x < STEP; ++x) ar[x] = p[x];
    } else {
      const uint32_t* p = sAw + (cy * STEP + py) * C::AP + cx * (STEP * ES / 4);
      uint32_t w[STEP * ES / 4];
#pragma unroll
      for (int k = 0; k < STEP * ES / 4; ++k) w[k] = p[k];
#pragma unroll
      for (int x = 0; x < STEP; ++x) {
        const uint32_t wd = w[(x * ES) >> 2];
        ar[x] = (float)(ES == 1 ? (wd >> (8 * (x & 3))) & 0xffu : (wd >> (16 * (x & 1))) & 0xffffu);
      }
    }
  };
  // sums over the lanes of one item (or the 16 rows of a cell): neighbouring
  // lanes by quad permutes, then the half-row and row mirrors
  auto lanes_sum = [](float v, int n) {
    auto dpp = [](float x, auto ctrl) {
      return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    if (n > 1) v += dpp(v, std::integral_constant<int, 0xB1>());
    if (n > 2) v += dpp(v, std::integral_constant<int, 0x4E>());
    if (n > 4) v += dpp(v, std::integral_constant<int, 0x141>());
    if (n > 8) v += dpp(v, std::integral_constant<int, 0x140>());
    return v;
  };
  // ---- per cell: Kc, the rounded mean of A, the sum of A - Kc and of its
  // square, a lane per cell row
  constexpr float kInvCell = 1.0f / (float)(STEP * STEP);
  for (int i = t; i < (16 * C::NC + 63) / 64 * 64; i += NT) {
    const int c = min(i >> 4, C::NC - 1), py = i & 15;
    float ar[STEP], s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
    arow(c / C::CW, c - (c / C::CW) * C::CW, py, ar);
#pragma unroll
    for (int x = 0; x < STEP; ++x) s0 += ar[x];
    const float Kc = rintf(lanes_sum(s0, 16) * kInvCell);
#pragma unroll
    for (int x = 0; x < STEP; ++x) {
      const float d = ar[x] - Kc;
      s1 += d;
      s2 += d * d;
    }
    s1 = lanes_sum(s1, 16);
    s2 = lanes_sum(s2, 16);
    if (py == 0) {
      s_cell[0][c] = Kc;
      s_cell[1][c] = s1;
      s_cell[2][c] = s2;
    }
  }
  __syncthreads();
  // ---- products: P = sum (A - Kc)(B' - Kc) over the thread's rows of its cell
  const int q = t / PARTS, part = t - q * PARTS;
  const int sy_i = q % NSY, cell = q / NSY;
  float P[NSY];
  if (t < C::NI) {
    const int ci = cell / C::CW, cj = cell - (cell / C::CW) * C::CW;
    const float Kc = s_cell[0][cell], kb = Kc - K;
#pragma unroll
    for (int j = 0; j < NSY; ++j) P[j] = 0.0f;
    const float* bbase = sB + (ci * STEP + sy_i) * C::BP + cj * STEP;
    // one row at a time in flight beside the one worked on (r 8: its rows do
    // not fit the registers of four waves a SIMD)
    constexpr int kRows = R > 4 ? 1 : 2;
#pragma unroll kRows
    for (int k = 0; k < STEP / PARTS; ++k) {
      const int py = part + PARTS * k;
      float ar[STEP], br[C::BRW];
      arow(ci, cj, py, ar);
#pragma unroll
      for (int x = 0; x < C::BRW; ++x) br[x] = bbase[py * C::BP + x];
#pragma unroll
      for (int x = 0; x < STEP; ++x) ar[x] -= Kc;
#pragma unroll
      for (int x = 0; x < C::BRW; ++x) br[x] -= kb;
#pragma unroll
      for (int x = 0; x < STEP; ++x)
#pragma unroll
        for (int j = 0; j < NSY; ++j) P[j] += ar[x] * br[x + j];
    }
#pragma unroll
    for (int j = 0; j < NSY; ++j) P[j] = lanes_sum(P[j], PARTS);
  }
  if constexpr (kCentral) __syncthreads();   // A' is read: the column sums take its place
  // ---- column sums of B' and its square over every cell row and row shift,
  // about the mean of the cell whose columns they are
  auto cell_of = [&](int ci, int x) { return ci * C::CW + min(max((x - R) >> 4, 0), C::CW - 1); };
  for (int i = t; i < C::CH * C::BW; i += NT) {
    const int ci = i / C::BW, x = i - (i / C::BW) * C::BW;
    const float* col = sB + ci * STEP * C::BP + x;
    float* vs = sV + ci * NSY * C::BP + x;
    float* vq = vs + C::VS;
    const float kb = s_cell[0][cell_of(ci, x)] - K;
    float v[STEP + 2 * R];
#pragma unroll
    for (int r = 0; r < STEP + 2 * R; ++r) v[r] = col[r * C::BP] - kb;
    float s = 0.0f, q2 = 0.0f;
#pragma unroll
    for (int r = 2 * R; r < STEP; ++r) {
      s += v[r];
      q2 += v[r] * v[r];
    }
    // rows the shift takes from the head, last row first, then the tail's
    float hs[NSY], hq[NSY];
    hs[2 * R] = hq[2 * R] = 0.0f;
#pragma unroll
    for (int r = 2 * R - 1; r >= 0; --r) {
      hs[r] = hs[r + 1] + v[r];
      hq[r] = hq[r + 1] + v[r] * v[r];
    }
    float ts = 0.0f, tq = 0.0f;
#pragma unroll
    for (int k = 0; k < NSY; ++k) {
      if (k > 0) {
        ts += v[STEP + k - 1];
        tq += v[STEP + k - 1] * v[STEP + k - 1];
      }
      vs[k * C::BP] = hs[k] + s + ts;
      vq[k * C::BP] = hq[k] + q2 + tq;
    }
  }
  __syncthreads();
  // ---- per cell and shift row: S, or Q, the sums of B' - Kc (and of its
  // square) along the row of column sums; the columns of the cells beside it
  // are brought to Kc first
  constexpr int kItems = C::NC * NSY, kArr = kItems * NSY;
  constexpr float n = (float)STEP, kInvN = 1.0f / (float)(C::WIN * C::WIN);
  float SQ[NSY];
  if (t < 2 * kItems) {
    const bool sq = t >= kItems;
    const int it = sq ? t - kItems : t, c = it / NSY, k = it - c * NSY, ci = c / C::CW, cj = c - ci * C::CW;
    const float* vs = sV + (ci * NSY + k) * C::BP + cj * STEP;
    const float Kc = s_cell[0][c];
    const float dl = s_cell[0][cell_of(ci, cj * STEP)] - Kc, dr = s_cell[0][cell_of(ci, cj * STEP + C::BRW - 1)] - Kc;
    float col[C::BRW];
    if (sq) {
#pragma unroll
      for (int x = 0; x < C::BRW; ++x) {
        const float d = x < R ? dl : dr;
        col[x] = vs[C::VS + x];
        if (x < R || x >= R + STEP) col[x] += d * (2.0f * vs[x] + n * d);
      }
    } else {
#pragma unroll
      for (int x = 0; x < C::BRW; ++x) {
        col[x] = vs[x];
        if (x < R || x >= R + STEP) col[x] += n * (x < R ? dl : dr);
      }
    }
    float head[NSY], mid = 0.0f, tail = 0.0f;
    head[2 * R] = 0.0f;
#pragma unroll
    for (int x = 2 * R - 1; x >= 0; --x) head[x] = head[x + 1] + col[x];
#pragma unroll
    for (int x = 2 * R; x < STEP; ++x) mid += col[x];
#pragma unroll
    for (int j = 0; j < NSY; ++j) {
      if (j > 0) tail += col[STEP + j - 1];
      SQ[j] = head[j] + mid + tail;
    }
  }
  // per window: its mean Kw, per cell d = Kc - Kw, and the sums of A - Kw and
  // its square
  auto cell_at = [](int w, int i) { return (w / TW + (i >> 1)) * C::CW + w - (w / TW) * TW + (i & 1); };
  if (t >= NT - C::NWIN) {
    const int w = NT - 1 - t;
    float Kw = 0.0f, s1 = 0.0f, sa = 0.0f, saa = 0.0f, cp = 0.0f, cs = 0.0f, cq = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      Kw += 0.25f * s_cell[0][cell_at(w, i)];
      s1 += s_cell[1][cell_at(w, i)];
    }
    Kw = rintf(Kw + s1 * kInvN);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = cell_at(w, i);
      const float d = s_cell[0][c] - Kw, e = n * n * d, f = s_cell[1][c] + e;
      s_win[w][i] = d;
      sa += f;
      saa += s_cell[2][c] + d * (s_cell[1][c] + f);
      cp += d * f;
      cs += e;
      cq += d * e;
    }
    const float mA = sa * kInvN, varA = saa - sa * mA;
    s_win[w][4] = mA;
    s_win[w][5] = varA > kFlatRel * saa ? varA : 0.0f;   // (0: flat)
    s_win[w][6] = cp;
    s_win[w][7] = cs;
    s_win[w][8] = cq;
    s_sharp[w] = 0;
  }
  __syncthreads();   // tiles and column sums are read: the cells' sums take their place
  if (t < C::NI && part == 0) {
#pragma unroll
    for (int j = 0; j < NSY; ++j) s_mem[q * NSY + j] = P[j];
  }
  if (t < 2 * kItems) {
#pragma unroll
    for (int j = 0; j < NSY; ++j) s_mem[kArr + t * NSY + j] = SQ[j];
  }
  __syncthreads();
  // ---- a thread per window, shift row and JG shift columns: the coefficients
  constexpr int NS = NSY * NSY, JG = C::JG, NJ = (NSY + JG - 1) / JG;
  if (t < C::NWIN * NSY * NJ) {
    const int wk = t / NJ, j0 = (t - wk * NJ) * JG, w = wk / NSY, k = wk - w * NSY;
    float v[12];
#pragma unroll
    for (int i = 0; i < 12; i += 4) *reinterpret_cast<float4*>(v + i) = *reinterpret_cast<const float4*>(&s_win[w][i]);
    const float mA = v[4], varA = v[5];
    const float* p = s_mem + cell_at(w, 0) * NS + k * NSY + j0;
    bool sharp = false;
#pragma unroll
    for (int j = 0; j < JG; ++j) {
      if (j0 + j >= NSY) break;
      float Pw = v[6], Sw = v[7], Qw = v[8], ds = 0.0f;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float* q = p + ((c >> 1) * C::CW + (c & 1)) * NS + j;
        const float Sc = q[kArr];
        Pw += q[0];
        Sw += Sc;
        Qw += q[2 * kArr];
        ds += v[c] * Sc;
      }
      Pw += ds;
      Qw += 2.0f * ds;
      const float num = Pw - mA * Sw;
      const float varB = Qw - Sw * Sw * kInvN;
      const bool flat = varA == 0.0f || !(varB > kFlatRel * Qw);
      s_rho[w * NS + k * NSY + j0 + j] = flat ? 0.0f : num * __builtin_amdgcn_rsqf(varA * varB);
      sharp = sharp || (!flat && (!g.fixed || k == R || j0 + j == R));
    }
    if (sharp) s_sharp[w] = 1;
  }
  __syncthreads();
  // ---- GL lanes per window (a wave each, or 16 where a tile has more windows
  // than waves): its peak; the first of them fits and composes
  constexpr int GL = C::NWIN <= NT / 64 ? 64 : 16;
  static_assert(C::NWIN * GL <= NT, "a group of lanes per window");
  const int gl = t & (GL - 1), w = t / GL, wi = w / TW, a = a0 + wi, b = b0 + w - wi * TW;
  float best = -2.0f;
  int bkey = 1 << 20;
  if (w < C::NWIN) {
#pragma unroll
    for (int i = 0; i < (NS + GL - 1) / GL; ++i) {
      const int s = gl + GL * i, k = s / NSY, key = tie_key(k - R, s - k * NSY - R);
      const float r = s_rho[w * NS + min(s, NS - 1)];
      if (s < NS && better(r, key, best, bkey)) {
        best = r;
        bkey = key;
      }
    }
  }
  // (keys are below 2^20: exact as floats)
  if constexpr (GL == 64) {
    const float top = wave_max(best);
    bkey = (int)wave_min(best == top ? (float)bkey : 1048576.0f);
  } else {
    auto rows = [](float x, auto op) __attribute__((always_inline)) {
      auto dpp = [](float v, auto ctrl) {
        const int i = __float_as_int(v);
        return __int_as_float(__builtin_amdgcn_update_dpp(i, i, decltype(ctrl)::value, 0xF, 0xF, false));
      };
      x = op(x, dpp(x, Int<0xB1>()));
      x = op(x, dpp(x, Int<0x4E>()));
      x = op(x, dpp(x, Int<0x141>()));
      return op(x, dpp(x, Int<0x140>()));
    };
    const float top = rows(best, [](float x, float y) { return fmaxf(x, y); });
    bkey = (int)rows(best == top ? (float)bkey : 1048576.0f, [](float x, float y) { return fminf(x, y); });
  }
  if (gl == 0 && w < C::NWIN && a < g.ny && b < g.nx) {
    int sy = 0, sx = 0;
    if (!g.fixed) {
      sx = (bkey & 63) - 32;
      sy = ((bkey >> 6) & 63) - 32;
    }
    const float* rr = s_rho + w * NS;
    auto rhof = [&](int y, int x) { return rr[(y + R) * NSY + x + R]; };
    auto node = [&](int c, int y, int x) { return s_node[c][y - nlo_y][x - nlo_x]; };
    float pu = 0.0f, pv = 0.0f;
    if (Pn) window_mean_half_overlap(a, b, g.nx, g.ny, node, pu, pv);
    finish_vector(g, pair, a, b, sy, sx, s_sharp[w] == 0, pu, pv, rhof);
  }
}

template <typename T, int STEP, int R, int SYG, int TW, int TH, int NT>
hipError_t launch_tiled(const CorrArgs& g, int n, hipStream_t s) {
  dim3 grid((g.nx + TW - 1) / TW, (g.ny + TH - 1) / TH, n);
  hipLaunchKernelGGL((k_correct_tiled<T, STEP, R, SYG, TW, TH, NT>), grid, dim3(NT), 0, s, g);
  return hipGetLastError();
}

template <typename T, int STEP, int R, int SYG, int TW, int TH>
hipError_t launch_bands(const CorrArgs& g, int n, hipStream_t s) {
  dim3 grid((g.nx + TW - 1) / TW, (g.ny + TH - 1) / TH, n);
  hipLaunchKernelGGL((k_correct_bands<T, STEP, R, SYG, TW, TH>), grid, dim3(64 * ((2 * R + 1) / SYG)), 0, s, g);
  return hipGetLastError();
}

template <typename T, int STEP, int R, int TW, int TH, int PARTS, int NT>
hipError_t launch_rows(const CorrArgs& g, int n, hipStream_t s) {
  dim3 grid((g.nx + TW - 1) / TW, (g.ny + TH - 1) / TH, n);
  // (without a predictor the symmetric deformation moves nothing)
  if (g.central && g.pred)
    hipLaunchKernelGGL((k_correct_rows<T, STEP, R, TW, TH, PARTS, NT, true>), grid, dim3(NT), 0, s, g);
  else
    hipLaunchKernelGGL((k_correct_rows<T, STEP, R, TW, TH, PARTS, NT, false>), grid, dim3(NT), 0, s, g);
  return hipGetLastError();
}

template <typename T, int STEP, bool kCentral>
hipError_t launch_halves(const CorrArgs& g, int n, hipStream_t s) {
  constexpr int TW = 8, TH = 6;
  constexpr size_t lds = sizeof(float) * HalvesCfg<T, STEP, TW, TH, kCentral>::LDS_WORDS;
  dim3 grid((g.nx + TW - 1) / TW, (g.ny + TH - 1) / TH, n);
  hipLaunchKernelGGL((k_correct_halves<T, STEP, TW, TH, kCentral>), grid, dim3(512), lds, s, g);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tiled_t(const CorrArgs& g, int n, hipStream_t s) {
  if (!g.central && g.step == 8 && g.R == 4) return launch_bands<T, 8, 4, 3, 8, 6>(g, n, s);
  if (!g.central && g.step == 8 && g.R == 1) return launch_bands<T, 8, 1, 1, 8, 6>(g, n, s);
  if constexpr (sizeof(T) == 2) {   // (u8 cells of 12 px are not whole words at half a cell)
    if (!g.central && g.step == 12 && g.R == 4) return launch_halves<T, 12, false>(g, n, s);
  }
  if (g.step == 8 && g.R == 4) return launch_halves<T, 8, true>(g, n, s);
  // The others stay with the tiled kernel: with both 24 px frames deformed,
  // A' as floats would take two waves per band to 118 KB of LDS, one
  // workgroup a CU; the nine shifts of r 1 make no bands to share.
  if (g.step == 8 && g.R == 1) return launch_tiled<T, 8, 1, 1, 8, 8, 256>(g, n, s);
  if (g.step == 12 && g.R == 4) return launch_tiled<T, 12, 4, 3, 5, 5, 128>(g, n, s);
  if (g.step == 12 && g.R == 1) return launch_tiled<T, 12, 1, 1, 5, 5, 128>(g, n, s);
  if (g.step == 16) {
    // Small frames take a workgroup per window with its cells' rows in many
    // parts (latency), larger ones share cells in a tile.  For one u8 pair
    // both take as long at about 1,100 windows for r 4 (18 and 20 us at
    // 1,024; 26 and 20 at 1,600) and 400 for r 8 (15 and 21 us at 256; 28
    // and 22 at 576), but a batch gains from the tile earlier (r 4, 4 x
    // 2,048 windows: 97 and 33 us), so the line is 400.  It goes by the frame
    // and not by the batch: the two sum in another order, and a pair's
    // result must not depend on the batch it is in.
    const bool tile = g.nx * g.ny > 400;
    if (g.R == 4) return tile ? launch_rows<T, 16, 4, 4, 4, 2, 512>(g, n, s) : launch_rows<T, 16, 4, 1, 1, 8, 320>(g, n, s);
    if (g.R == 8) return tile ? launch_rows<T, 16, 8, 4, 2, 2, 512>(g, n, s) : launch_rows<T, 16, 8, 1, 1, 8, 576>(g, n, s);
    if (g.R == 1) return tile ? launch_rows<T, 16, 1, 4, 4, 4, 320>(g, n, s) : launch_rows<T, 16, 1, 1, 1, 16, 192>(g, n, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int correct_impl(const Plan& P) {
  const int R = P.p.peak == PIV_PEAK_FIXED_CENTER ? 1 : P.p.radius;
  if (P.p.dtype == PIV_F32) return 0;
  if (P.p.win != 2 * P.p.step) return 0;
  if ((P.p.step == 8 || P.p.step == 12) && (R == 4 || R == 1)) return 1;
  if (P.p.step == 16 && (R == 8 || R == 4 || R == 1)) return 1;
  return 0;
}

hipError_t launch_correct(const Plan& P, const void* A, const void* B, int64_t pitch, int n,
                          const float* pred, float* disp, float* peak, uint8_t* flags, hipStream_t s,
                          int64_t disp_stride) {
  CorrArgs g;
  g.A = (const uint8_t*)A;
  g.B = (const uint8_t*)B;
  g.pitch = pitch;
  g.stride = pitch * P.p.height;
  g.W = P.p.width;
  g.H = P.p.height;
  g.nx = P.nx;
  g.ny = P.ny;
  g.win = P.p.win;
  g.step = P.p.step;
  g.fixed = P.p.peak == PIV_PEAK_FIXED_CENTER;
  g.R = g.fixed ? 1 : P.p.radius;
  g.central = P.p.warp == PIV_WARP_CENTRAL;
  g.pred = pred;
  g.disp = disp;
  g.dstride = disp_stride ? disp_stride : 2 * (int64_t)P.nx * P.ny;
  g.peak = peak;
  g.flags = flags;
  g.mask = P.slot_mask;
  if (correct_impl(P) == 1) {
    return P.p.dtype == PIV_U8 ? launch_tiled_t<uint8_t>(g, n, s) : launch_tiled_t<uint16_t>(g, n, s);
  }
  const int BWd = g.win + 2 * g.R, S = 2 * g.R + 1, S2 = S * S;
  const int H = std::max(1, std::min(g.win, kGenT / S2));   // (as in the kernel)
  size_t lds = sizeof(float) * ((size_t)g.win * g.win + (size_t)BWd * BWd + (size_t)S2 + 3 * (size_t)H * S2);
  dim3 grid(P.nx, P.ny, n);
  switch (P.p.dtype) {
    case PIV_U8: hipLaunchKernelGGL(k_correct_generic<uint8_t>, grid, dim3(kGenT), lds, s, g); break;
    case PIV_U16: hipLaunchKernelGGL(k_correct_generic<uint16_t>, grid, dim3(kGenT), lds, s, g); break;
    default: hipLaunchKernelGGL(k_correct_generic<float>, grid, dim3(kGenT), lds, s, g); break;
  }
  return hipGetLastError();
}

}  // namespace piv
