// Pre-processing of the frames (Sec. 2: a high-pass filter removes the
// static background, then contrast-limited adaptive histogram equalisation
// brightens the image; Sec. 3.1 uses both to match the intensities of
// stitched images).  Integer arithmetic throughout, so the results are
// exact.  Both passes stream the frames once (reads and writes coalesced by
// rows); the tile halos of the high-pass come from L2.
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "piv_internal.h"

namespace piv {
namespace {

// ---------------------------------------------------------------------------
// High-pass: out = max(0, I - floor(sum / count)) over the image part of the
// (2r+1)^2 box around each pixel.  One wave owns a strip of columns and a
// band of rows and walks down it: a lane holds the vertical box sums of four
// pixels (u8: as two pairs of 16-bit fields, a sum is at most 33 x 255),
// updated per row by the row entering and the row leaving the box.  The sums of the columns around the lane's
// pixels come from the neighbouring lanes by DPP wave shifts, so rows need no
// barrier and several are in flight; a lane's last 2r+1 rows wait in its own
// LDS column for the row's turn at the centre and at leaving, so that every
// row is read once per band.  Bound by VALU issue (about 45 instructions per
// four pixels and row, u8) and, at an eighth of the waves a SIMD can hold,
// latency.  64 x 1 MP u8, r 7: 103 -> 54 us (with word strips, sums through
// LDS and the leaving and centre rows read again from memory, 3.5 times the
// frame's bytes); 8 x 4K u16, r 5: 121 -> 68 us.  The strip's first and last
// h = ceil(r / 4) lanes only supply sums, so strips overlap by 2h lanes.  The
// pixel count of the clipped box is a product of two clipped spans; the
// quotient comes from a float reciprocal, corrected to the exact floor.
// ---------------------------------------------------------------------------
// Rows of a band: more bands hide latency, each adds 2r rows to read.  Full
// chips, calls of 64 x 1 MP u8 with 16, 32 and 64 rows: r 3 43.5, 44.1 and
// 45.0 us, r 7 49.8, 48.9 and 49.6, r 12 65.5, 63.6 and 58.5, r 16 78.8, 75.1
// and 81.5; 8 x 4K u16 with 32, 64 and 128: r 3 57.0, 58.2 and 72.5, r 5
// 62.1, 61.5 and 70.1, r 12 81.9, 82.1 and 83.3, r 16 100.3, 99.7 and 118.5.
// (One frame alone would gain from shorter bands: one of 4K u16, r 5, 28 us
// with 64 rows and 14 with 16.)
template <typename T>
constexpr int hp_band() { return sizeof(T) == 1 ? 32 : 64; }

// floor(s / c) for quotients below 2^16 (s < 2^27, 1 <= c < 2^11): the
// float estimate is then within one of the quotient, and integer
// corrections make it exact
__device__ __forceinline__ uint32_t udiv_small(uint32_t s, uint32_t c) {
  int q = (int)((float)s * __builtin_amdgcn_rcpf((float)c));
  int r = (int)s - q * (int)c;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    q += r < 0 ? -1 : (r >= (int)c ? 1 : 0);
    r = (int)s - q * (int)c;
  }
  return (uint32_t)q;
}

// floor(s / D) for the whole box, D = (2R+1)^2, s <= D * maxval.
// u16 (s < 2^27): the product with M = ceil(2^(32+k) / D), k = ceil(log2 D) - 1
// (so that M < 2^32), keeps its error s (M D - 2^(32+k)) / D below
// 2^(32+k) / D > 2^31 > s, hence exact.  u8 (s < 2^19): the same with a
// 32-bit product of 24-bit factors at full rate, floor(s M / 2^K) with
// M = ceil(2^K / D), exact while s (M D - 2^K) < 2^K and s M < 2^32 (tested
// here at compile time; radii 9, 10 and 12 to 16 have no such K and take the
// u16 product).
template <int D, bool kByte>
struct BoxDiv {
  static constexpr int K = []() { int k = 0; while ((1 << (k + 1)) < D) ++k; return k; }();
  static constexpr uint32_t M = (uint32_t)((((uint64_t)1 << (32 + K)) + D - 1) / D);
  static_assert((1ull << K) < (unsigned long long)D && (((uint64_t)1 << (32 + K)) / D) > (1u << 27), "magic range");
  static constexpr uint64_t SMAX = 255ull * D;
  static constexpr bool ok(int k) {
    const uint64_t m = (((uint64_t)1 << k) + D - 1) / D;
    return SMAX * m < (1ull << 32) && SMAX * (m * D - ((uint64_t)1 << k)) < ((uint64_t)1 << k) && m < (1u << 24);
  }
  static constexpr int K8 = []() { int k = 31; while (k > 0 && !ok(k)) --k; return k; }();
  static constexpr uint32_t M8 = (uint32_t)((((uint64_t)1 << K8) + D - 1) / D);
  static __device__ __forceinline__ uint32_t div(uint32_t s) {
    if constexpr (kByte && K8 > 0) return (uint32_t)__umul24(s, M8) >> K8;   // (declared to return int)
    else return __umulhi(s, M) >> K;
  }
};

// the value of the lane to the right / left (0 past the wave's ends)
__device__ __forceinline__ uint32_t from_right(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t from_left(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);
}

constexpr int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// Horizontal box sums of a lane's four pixels from the vertical sums V of
// its columns: NF columns per word of V (2: 16-bit fields, 1: 32 bits).
// Words of the columns -R .. R + 3 around the lane's first are fetched from
// the lanes around; the columns that all four boxes share are summed once.
template <int R, int NF>
__device__ __forceinline__ void box_rows(const uint32_t (&V)[4 / NF], uint32_t (&hs)[4]) {
  constexpr int NV = 4 / NF;
  constexpr int lo = floor_div(-R, NF), hi = floor_div(R + 3, NF);   // word range, own words 0 .. NV - 1
  uint32_t w[hi - lo + 1];
#pragma unroll
  for (int m = 0; m < NV && m <= hi; ++m) w[m - lo] = V[m];
#pragma unroll
  for (int m = NV; m <= hi; ++m) w[m - lo] = from_right(w[m - NV - lo]);
#pragma unroll
  for (int m = -1; m >= lo; --m) w[m - lo] = from_left(m + NV >= 0 ? V[m + NV] : w[m + NV - lo]);
  auto add = [](uint32_t acc, uint32_t word, bool f0, bool f1) __attribute__((always_inline)) {
    if constexpr (NF == 1) {
      return acc + word;
    } else {
      typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
      const uint32_t sel = (f0 ? 1u : 0u) | (f1 ? 0x10000u : 0u);
      return (uint32_t)__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, word), __builtin_bit_cast(u16x2, sel), acc, false);
    }
  };
  uint32_t common = 0u;
#pragma unroll
  for (int m = lo; m <= hi; ++m)
    if (NF * m >= 3 - R && NF * m + NF - 1 <= R) common = add(common, w[m - lo], true, true);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t s = common;
#pragma unroll
    for (int m = lo; m <= hi; ++m) {
      if (NF * m >= 3 - R && NF * m + NF - 1 <= R) continue;
      const bool f0 = NF * m >= e - R && NF * m <= e + R, f1 = NF == 2 && 2 * m + 1 >= e - R && 2 * m + 1 <= e + R;
      if (f0 || f1) s = add(s, w[m - lo], f0, f1);
    }
    hs[e] = s;
  }
}

template <typename T, int R>
__global__ __launch_bounds__(64) void k_highpass(const uint8_t* __restrict__ in, uint8_t* __restrict__ out,
                                                 int64_t pitch, int64_t stride, int W, int H,
                                                 const uint8_t* mask) {
  constexpr int ES = (int)sizeof(T), NW = ES, PX = 4;   // a lane's words of a row, its pixels
  constexpr int NF = ES == 1 ? 2 : 1, NV = 4 / NF;
  constexpr int r = R;
  using Div = BoxDiv<(2 * R + 1) * (2 * R + 1), ES == 1>;
  constexpr int G = 4;                                // rows per group
  constexpr int N = 2 * R + 1 + G;                   // rows of the ring
  __shared__ uint32_t ring[N * 64 * NW];
  const int pair = blockIdx.z;
  if (slot_off(mask, pair)) return;
  const int L = threadIdx.x;
  constexpr int h = (r + PX - 1) / PX, nout = 64 - 2 * h;
  const int x0 = PX * (blockIdx.x * nout + L - h);   // this lane's first pixel (may lie off the image)
  const int xa = x0 * ES;                            // its byte offset in a row
  const int rowbytes = W * ES;
  const uint8_t* src = in + (int64_t)pair * stride;
  struct RowWords { uint32_t w[NW]; };
  struct __attribute__((aligned(4))) Wide { uint32_t w[NW]; };
  // the lane's words of a row, zero outside the image: a strip inside the
  // row reads them together, one at an edge word by word through masks
  const bool whole = __all(xa >= 0 && xa + 4 * NW <= rowbytes);
  const int y_first = blockIdx.y * hp_band<T>(), y_end = min(y_first + hp_band<T>(), H);
  const bool outl = L >= h && L < 64 - h;            // lanes whose pixels are written
  uint32_t cx[PX];
  bool fx = true;
#pragma unroll
  for (int e = 0; e < PX; ++e) {
    cx[e] = (uint32_t)(min(x0 + e + r, W - 1) - max(x0 + e - r, 0) + 1);
    fx = fx && cx[e] == 2 * r + 1;
  }
  // (every written pixel of the strip has its box's full width)
  const bool full_x = __all(fx || !outl);
  // divisors c = cx (2r + 1) of rows that are not clipped, as a product:
  // floor(s / c) = floor(s M / 2^(32 + k)), M and k as in BoxDiv (c >= 3)
  uint32_t lm[PX];
  int lk[PX];
  if (!full_x) {
#pragma unroll
    for (int e = 0; e < PX; ++e) {
      const uint32_t c = (uint32_t)max((int)cx[e], 1) * (2 * r + 1);
      lk[e] = 31 - __builtin_clz(c - 1);
      lm[e] = (uint32_t)((((uint64_t)1 << (32 + lk[e])) + c - 1) / c);
    }
  }
  uint8_t* dst = out + (int64_t)pair * stride;

  auto strip = [&](auto whole_c) __attribute__((always_inline)) {
    constexpr bool kWhole = decltype(whole_c)::value;
    auto row_words = [&](int y) __attribute__((always_inline)) {
      RowWords o;
      const uint32_t ok = (unsigned)y < (unsigned)H ? 0xffffffffu : 0u;
      const uint8_t* row = src + (int64_t)min(max(y, 0), H - 1) * pitch;
      if constexpr (kWhole) {
        const Wide v = *reinterpret_cast<const Wide*>(row + xa);
#pragma unroll
        for (int k = 0; k < NW; ++k) o.w[k] = v.w[k] & ok;
      } else {
#pragma unroll
        for (int k = 0; k < NW; ++k) o.w[k] = masked_word(row, rowbytes, xa + 4 * k) & ok;
      }
      return o;
    };
    auto px = [](const RowWords& w, int e) -> uint32_t {
      return ES == 1 ? (w.w[0] >> (8 * e)) & 0xffu : (w.w[(e * ES) >> 2] >> (16 * (e & 1))) & 0xffffu;
    };
    // the lane's pixels in the layout of V
    auto fields = [&](const RowWords& w, int m) -> uint32_t {
      if constexpr (ES == 1) return __builtin_amdgcn_perm(0u, w.w[0], m == 0 ? 0x0c010c00u : 0x0c030c02u);
      else return px(w, m);
    };
    // ring of the lane's words of the last rows (its own LDS column, so the
    // accesses of a wave need no barrier): row y sits in slot (y - first) mod N
    auto put = [&](int slot, const RowWords& w) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NW; ++k) ring[(slot * 64 + L) * NW + k] = w.w[k];
    };
    auto get = [&](int slot) __attribute__((always_inline)) {
      RowWords w;
#pragma unroll
      for (int k = 0; k < NW; ++k) w.w[k] = ring[(slot * 64 + L) * NW + k];
      return w;
    };
    auto wrap = [](int slot) { return slot >= N ? slot - N : slot; };
    // slot 0 holds row y_first - r - 1 (which no box of the band takes)
    uint32_t V[NV];
#pragma unroll
    for (int m = 0; m < NV; ++m) V[m] = 0u;
    RowWords ci[G], co[G], cc[G], ni[G];
    constexpr int INIT = 2 * R;   // rows y_first - r .. y_first + r - 1
#pragma unroll
    for (int d0 = 0; d0 < INIT; d0 += 8) {
      RowWords w[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (d0 + k < INIT) w[k] = row_words(y_first - r + d0 + k);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (d0 + k < INIT) {
          put(1 + d0 + k, w[k]);
#pragma unroll
          for (int m = 0; m < NV; ++m) V[m] += fields(w[k], m);
        }
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) ring[L * NW + k] = 0u;
    auto fetch = [&](int yg, RowWords (&wi)[G]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < G; ++k) wi[k] = row_words(yg + k + r);
    };
    fetch(y_first, ci);
    int base = 0;   // slot of row yg - r - 1
    for (int yg = y_first; yg < y_end; yg += G) {
      if (yg + G < y_end) fetch(yg + G, ni);
      // (the ring holds rows yg - r - 1 .. yg + G - 1 + r)
#pragma unroll
      for (int k = 0; k < G; ++k) put(wrap(base + 2 * R + 1 + k), ci[k]);
#pragma unroll
      for (int k = 0; k < G; ++k) co[k] = get(wrap(base + k));
#pragma unroll
      for (int k = 0; k < G; ++k) cc[k] = get(wrap(base + R + 1 + k));
      base = wrap(base + G);
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const int y = yg + k;
        if (y >= y_end) break;
        // (every field ends in range, so the fields' sums do not mix)
#pragma unroll
        for (int m = 0; m < NV; ++m) V[m] = V[m] + fields(ci[k], m) - fields(co[k], m);
        uint32_t hs[PX], o[PX];
        box_rows<R, NF>(V, hs);
        const uint32_t cy = (uint32_t)(min(y + r, H - 1) - max(y - r, 0) + 1);
        if (cy == 2 * r + 1 && !full_x) {
          // boxes clipped at the left or right: the lane's own divisors
#pragma unroll
          for (int e = 0; e < PX; ++e)
            o[e] = __builtin_elementwise_sub_sat(px(cc[k], e), __umulhi(hs[e], lm[e]) >> lk[e]);
        } else if (cy == 2 * r + 1) {
          // the whole box inside the image (the usual case, taken by the
          // whole wave): the constant divisor's product
#pragma unroll
          for (int e = 0; e < PX; ++e) o[e] = __builtin_elementwise_sub_sat(px(cc[k], e), Div::div(hs[e]));
        } else {
#pragma unroll
          for (int e = 0; e < PX; ++e) o[e] = __builtin_elementwise_sub_sat(px(cc[k], e), udiv_small(hs[e], max(cx[e], 1u) * cy));
        }
        if (outl) {
          T* orow = reinterpret_cast<T*>(dst + (int64_t)y * pitch);
          if (kWhole || (x0 >= 0 && x0 + PX <= W)) {
            Wide v;
            if constexpr (ES == 1) {
              v.w[0] = o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24);
            } else {
              v.w[0] = o[0] | (o[1] << 16);
              v.w[NW - 1] = o[2] | (o[3] << 16);
            }
            *reinterpret_cast<Wide*>(orow + x0) = v;
          } else {
#pragma unroll
            for (int e = 0; e < PX; ++e)
              if (x0 + e >= 0 && x0 + e < W) orow[x0 + e] = (T)o[e];
          }
        }
      }
#pragma unroll
      for (int k = 0; k < G; ++k) ci[k] = ni[k];
    }
  };
  if (whole) strip(std::true_type());
  else strip(std::false_type());
}

// ---------------------------------------------------------------------------
// CLAHE, pass 1: one workgroup per tile.  Histogram in LDS with integer
// atomics (the order of the adds does not matter): NH copies of every bin
// lie side by side and a lane takes copy lane mod NH, so that neighbouring
// pixels of one value go to different banks; zeros (the bulk of a particle
// image's background) are what the other bins leave of the tile's pixels.
// Reads take 16 bytes a lane, several in flight.  What a tile costs is the
// instructions per pixel (about 4 and an LDS atomic), so u16 tiles, few and
// large, get 1,024 threads: 8 frames of 4K u16 on 7 x 5 tiles 224 -> 43 us
// (one word per thread and step, a division each, 256 threads; the number of
// copies, 1 to 4, changes nothing), 64 x 1 MP u8 on 8 x 8 tiles 44 -> 21 us.
// Then the clip at max(1, floor(clip * npix / nbins)) (the same double
// arithmetic as the host), the clipped excess spread evenly
// (excess / nbins to every bin, one more to the first `rest` bins at a
// stride of max(nbins / rest, 1)), a prefix sum and
// lut[b] = (cdf * maxval + npix / 2) / npix.
// ---------------------------------------------------------------------------
// (j L < 2^31: frames are at most 32767 px and grids 64 tiles)
__device__ __forceinline__ int tile_edge(int j, int L, int n) { return (j * L) / n; }

// sum over the workgroup (every thread gets it); red: one word per wave
template <int NT>
__device__ __forceinline__ uint32_t group_sum(uint32_t v, uint32_t* red) {
  const uint32_t s = (uint32_t)wave_sum((int)v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  uint32_t t = 0u;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += red[i];
  __syncthreads();
  return t;
}

template <typename T, int NT, int NH, int HB, int SH>
__global__ __launch_bounds__(NT) void k_clahe_lut(const uint8_t* __restrict__ in, int64_t pitch, int64_t stride,
                                                  int W, int H, int tx, int ty, int nbins, int maxval,
                                                  double clip_factor, uint16_t* lut, const uint8_t* mask) {
  constexpr int ES = (int)sizeof(T), PW = 4 / ES, NWAVE = NT / 64;
  __shared__ uint32_t hist[NH * HB];                // [bin][copy], then the merged bins
  __shared__ uint32_t red[NWAVE];
  const int pair = blockIdx.z;
  if (slot_off(mask, pair)) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int i = blockIdx.x, j = blockIdx.y;
  const int xa = tile_edge(i, W, tx), xb = tile_edge(i + 1, W, tx);
  const int ya = tile_edge(j, H, ty), yb = tile_edge(j + 1, H, ty);
  const int tw = xb - xa, th = yb - ya;
  const uint32_t npix = (uint32_t)tw * (uint32_t)th;   // (frames are at most 32767 x 32767)
  for (int b = t; b < NH * nbins; b += NT) hist[b] = 0u;
  __syncthreads();
  uint32_t* hc = hist + (lane & (NH - 1));
  const uint8_t* src = in + (int64_t)pair * stride;
  auto count = [&](uint32_t v) __attribute__((always_inline)) {
    if (v) atomicAdd(&hc[(v >> SH) * NH], 1u);
  };
  // Items of four words that lie in the tile: nc per row, dealt to the
  // threads in order, U of a thread's items requested together.
  const int wa = (xa * ES + 3) >> 2, nc = max(((xb * ES) >> 2) - wa, 0) >> 2, items = nc * th;
  constexpr int U = 4;
  struct __attribute__((aligned(4))) Four { uint32_t w[4]; };
  const int srow = NT / max(nc, 1), scol = NT - srow * nc;   // one step of NT items
  int ry = t / max(nc, 1), rc = t - ry * nc;                 // the thread's next item
  for (int p0 = t; p0 < items; p0 += U * NT) {
    Four v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = *reinterpret_cast<const Four*>(src + (int64_t)(ya + min(ry, th - 1)) * pitch + 4 * (wa + 4 * rc));
      ry += srow;
      rc += scol;
      if (rc >= nc) {
        rc -= nc;
        ++ry;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p0 + u * NT >= items) break;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int e = 0; e < PW; ++e) count(ES == 1 ? (v[u].w[k] >> (8 * e)) & 0xffu : (v[u].w[k] >> (16 * e)) & 0xffffu);
    }
  }
  // The words left at the sides of a row, the first and last of them partly
  // the tile's, word by word and pixel by pixel (as lanes of the loop above
  // they cost every wave their steps: 16 u8 frames of 1000 x 760, a tile
  // each, 351 us both passes, now 103)
  const int w0 = (xa * ES) >> 2, nl = wa - w0, ns = nl + ((xb * ES + 3) >> 2) - (wa + 4 * nc);
  for (int p = t; p < th * ns; p += NT) {
    const int r = p / ns, k = p - r * ns, w = k < nl ? w0 + k : wa + 4 * nc + k - nl;
    const uint32_t wd = masked_word(src + (int64_t)(ya + r) * pitch, W * ES, 4 * w);
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      const int px = PW * w + e;
      if (px >= xa && px < xb) count(ES == 1 ? (wd >> (8 * e)) & 0xffu : (wd >> (16 * e)) & 0xffffu);
    }
  }
  __syncthreads();
  // merge the copies: a thread owns a contiguous chunk of bins from here on;
  // bin 0 takes the pixels that no bin counted, the zeros
  constexpr int PER = HB / NT > 0 ? HB / NT : 1;
  const int per = nbins / NT > 0 ? nbins / NT : 1;   // (bins are a power of two; per <= PER)
  const int b0 = t * per;
  const double cd = floor(clip_factor * (double)npix / (double)nbins);
  const uint32_t clip = cd < 1.0 ? 1u : cd >= (double)npix ? npix : (uint32_t)cd;
  uint32_t hb[PER], counted = 0u, ex = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    hb[k] = 0u;
    if (k < per && b0 + k < nbins) {
#pragma unroll
      for (int c = 0; c < NH; ++c) hb[k] += hist[(b0 + k) * NH + c];
      counted += hb[k];
    }
  }
  const uint32_t all = group_sum<NT>(counted, red);
  if (t == 0) hb[0] += npix - all;
#pragma unroll
  for (int k = 0; k < PER; ++k) {   // (a limit at or above npix clips nothing)
    if (hb[k] > clip) {
      ex += hb[k] - clip;
      hb[k] = clip;
    }
  }
  const uint32_t excess = group_sum<NT>(ex, red);
  const uint32_t each = excess / (uint32_t)nbins, rest = excess - each * (uint32_t)nbins;
  const uint32_t sstep = rest ? max((uint32_t)nbins / rest, 1u) : 1u;
  uint32_t local = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t b = (uint32_t)(b0 + k);
    if (k < per && b < (uint32_t)nbins) {
      const uint32_t extra = (rest && b % sstep == 0u && b / sstep < rest) ? 1u : 0u;
      hb[k] += each + extra;
      local += hb[k];
    }
  }
  // inclusive scan of the threads' totals: within the wave by lane shuffles,
  // then the waves before this one
  uint32_t inc = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)inc, o);
    if (lane >= o) inc += up;
  }
  if (lane == 63) red[wave] = inc;
  __syncthreads();
  uint32_t cdf = inc - local;
#pragma unroll
  for (int q = 0; q < NWAVE; ++q) cdf += q < wave ? red[q] : 0u;
  uint16_t* L = lut + (((int64_t)pair * ty + j) * tx + i) * nbins;
  const bool fits32 = (uint64_t)npix * (uint32_t)maxval + npix / 2 < ((uint64_t)1 << 32);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k < per && b0 + k < nbins) {
      cdf += hb[k];
      L[b0 + k] = (uint16_t)(fits32 ? (cdf * (uint32_t)maxval + npix / 2) / npix
                                    : (uint32_t)(((uint64_t)cdf * (uint32_t)maxval + npix / 2) / npix));
    }
  }
}

// CLAHE, pass 2 for small u8 tiles and blends beyond 32 bits (the other
// cases: k_clahe_cells below): every pixel blends the mappings of the (up to) four tiles
// whose centres surround it.  In doubled coordinates (centres may be
// half-integers) the tile holding x is k = ceil((x+1) tx / W) - 1 and the
// centre at or left of 2x is k or k - 1; before the first centre or after
// the last a single tile is used.
struct Axis {
  int a, b;
  int w, d;
};
__device__ __forceinline__ Axis clahe_axis(int x, int L, int n) {
  const int X = 2 * x;
  const int k = ((x + 1) * n + L - 1) / L - 1;
  const int ck = tile_edge(k, L, n) + tile_edge(k + 1, L, n) - 1;
  const int a = ck <= X ? k : k - 1;
  Axis r;
  if (a < 0 || a >= n - 1) {
    r.a = r.b = a < 0 ? 0 : n - 1;
    r.w = 0;
    r.d = 1;
  } else {
    const int ca = tile_edge(a, L, n) + tile_edge(a + 1, L, n) - 1;
    const int cb = tile_edge(a + 1, L, n) + tile_edge(a + 2, L, n) - 1;
    r.a = a;
    r.b = a + 1;
    r.w = X - ca;
    r.d = cb - ca;
  }
  return r;
}

// A workgroup covers MQ columns (four per thread) and MR rows.  The column
// blend data (tile pair and weights) is tabulated once per workgroup in LDS;
// when the mappings the block touches fit (u8), they are staged in LDS too,
// otherwise they are read from memory (L1/L2).  Every thread reads its four
// pixels, then writes them, so the pass may run in place.
constexpr int MQ = 1024, MR = 16;

// floor((num + den / 2) / den) for 0 <= num < 2^52, 1 <= den < 2^32: the
// double quotient is within one of the result, then an integer correction
// makes it exact (cheaper than a 64-bit integer division)
__device__ __forceinline__ int64_t round_div(int64_t num, int64_t den) {
  const int64_t n2 = num + den / 2;
  int64_t q = (int64_t)((double)n2 / (double)den);
  int64_t r = n2 - q * den;
  q += r < 0 ? -1 : (r >= den ? 1 : 0);
  return q;
}
constexpr int kStageWords = 6144;   // LDS words for staged mappings (24 KB)

template <typename T, bool kStaged, bool kNarrow>
__global__ __launch_bounds__(256) void k_clahe_map(const uint8_t* in, uint8_t* out, int64_t pitch, int64_t stride,
                                                   int W, int H, int tx, int ty, int nbins, int shift,
                                                   const uint16_t* __restrict__ lut, const uint8_t* mask) {
  constexpr int ES = (int)sizeof(T);
  __shared__ uint32_t s_ax[MQ];          // per column: a | b << 8 | w << 16 (w < 2^16, d in s_ad)
  __shared__ uint16_t s_ad[MQ];
  __shared__ Axis s_ay[MR];
  __shared__ uint32_t s_lut[kStaged ? kStageWords : 1];
  const int pair = blockIdx.z;
  if (slot_off(mask, pair)) return;
  const int t = threadIdx.x;
  const int x0 = blockIdx.x * MQ, y0 = blockIdx.y * MR;
  const int nq = min(MQ, W - x0);
  for (int c = t; c < nq; c += 256) {
    const Axis a = clahe_axis(x0 + c, W, tx);
    s_ax[c] = (uint32_t)a.a | ((uint32_t)a.b << 8) | ((uint32_t)a.w << 16);
    s_ad[c] = (uint16_t)a.d;
  }
  if (t < MR && y0 + t < H) s_ay[t] = clahe_axis(y0 + t, H, ty);
  const uint16_t* Lp = lut + (int64_t)pair * ty * tx * nbins;
  // tiles the block can touch: columns of its first and last pixel, rows of
  // its first and last row
  const Axis axl = clahe_axis(x0, W, tx), axr = clahe_axis(x0 + nq - 1, W, tx);
  const int yl = min(y0 + MR, H) - 1;
  const Axis ayt = clahe_axis(y0, H, ty), ayb = clahe_axis(yl, H, ty);
  const int i0 = axl.a, i1 = axr.b, j0 = ayt.a, j1 = ayb.b;
  const int ni = i1 - i0 + 1;
  if constexpr (kStaged) {
    const int words = (j1 - j0 + 1) * ni * nbins / 2;
    for (int k = t; k < words; k += 256) {
      const int e = 2 * k;
      const int tile = e / nbins, b = e - tile * nbins;
      const int jj = j0 + tile / ni, ii = i0 + tile - (tile / ni) * ni;
      s_lut[k] = *reinterpret_cast<const uint32_t*>(Lp + ((int64_t)jj * tx + ii) * nbins + b);
    }
  }
  __syncthreads();
  const uint16_t* sl = reinterpret_cast<const uint16_t*>(s_lut);
  // a mapping entry at (row part, column part, bin): the staged copy or the
  // global one, with the parts of the offset formed once per row and column
  auto L = [&](int rpart, int cpart, int b) -> int {
    if constexpr (kStaged) return sl[rpart + cpart + b];
    else return Lp[(int64_t)rpart + cpart + b];
  };
  auto rpart_of = [&](int jj) { return kStaged ? (jj - j0) * ni * nbins : jj * tx * nbins; };
  auto cpart_of = [&](int ii) { return kStaged ? (ii - i0) * nbins : ii * nbins; };
  const int c0 = 4 * t;
  if (c0 >= nq) return;
  const int xq = x0 + c0;
  const bool full = c0 + 4 <= nq;
  // this thread's four columns: tiles, weights and mapping offsets (the
  // same on every row)
  int ca[4], cb[4], cwx[4], cdx[4], kdx[4];
  float rdx[4];   // 1 / dx (the quotient's estimate is corrected exactly below)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = min(c0 + e, nq - 1);
    const uint32_t ax = s_ax[c];
    ca[e] = cpart_of((int)(ax & 0xff));
    cb[e] = cpart_of((int)((ax >> 8) & 0xff));
    cwx[e] = (int)(ax >> 16);
    cdx[e] = s_ad[c];
    rdx[e] = __builtin_amdgcn_rcpf((float)cdx[e]);
    kdx[e] = (cdx[e] & (cdx[e] - 1)) == 0 ? __builtin_ctz((unsigned)cdx[e]) : -1;   // log2 dx, or -1
  }
  for (int k = 0; k < MR; ++k) {
    const int y = y0 + k;
    if (y >= H) break;
    const Axis ay = s_ay[k];
    const int ra = rpart_of(ay.a), rb = rpart_of(ay.b);
    const float rdy = __builtin_amdgcn_rcpf((float)ay.d);
    const int kdy = (ay.d & (ay.d - 1)) == 0 ? __builtin_ctz((unsigned)ay.d) : -1;
    const T* row = reinterpret_cast<const T*>(in + (int64_t)pair * stride + (int64_t)y * pitch);
    T* orow = reinterpret_cast<T*>(out + (int64_t)pair * stride + (int64_t)y * pitch);
    uint32_t v[4];
    if (full) {
      if constexpr (ES == 1) {
        const uint32_t wd = *reinterpret_cast<const uint32_t*>(row + xq);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (wd >> (8 * e)) & 0xffu;
      } else {
        const uint32_t w0 = *reinterpret_cast<const uint32_t*>(row + xq);
        const uint32_t w1 = *reinterpret_cast<const uint32_t*>(row + xq + 2);
        v[0] = w0 & 0xffffu; v[1] = w0 >> 16; v[2] = w1 & 0xffffu; v[3] = w1 >> 16;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = c0 + e < nq ? (uint32_t)row[xq + e] : 0u;
    }
    uint32_t o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int wx = cwx[e], dx = cdx[e];
      const int b = (int)(v[e] >> shift);
      if constexpr (kNarrow) {
        // every numerator and denominator below 2^24 (checked on the host):
        // float estimate of the rounded quotient, then an exact correction
        const int l00 = L(ra, ca[e], b), l01 = L(ra, cb[e], b), l10 = L(rb, ca[e], b), l11 = L(rb, cb[e], b);
        const int num = (ay.d - ay.w) * ((dx - wx) * l00 + wx * l01) + ay.w * ((dx - wx) * l10 + wx * l11);
        const int den = dx * ay.d;
        const int n2 = num + den / 2;
        int q;
        if (kdx[e] >= 0 && kdy >= 0) {
          // a power-of-two denominator (tile spans of 2^k px): the floor by a shift
          q = n2 >> (kdx[e] + kdy);
        } else {
          // (the rounded quotient is below 2^16, so the estimate from the two
          // reciprocals is within one of it)
          q = (int)((float)n2 * rdx[e] * rdy);
          const int rr = n2 - q * den;
          q += rr < 0 ? -1 : (rr >= den ? 1 : 0);
        }
        o[e] = (uint32_t)q;
      } else {
        const int64_t l00 = L(ra, ca[e], b), l01 = L(ra, cb[e], b), l10 = L(rb, ca[e], b), l11 = L(rb, cb[e], b);
        const int64_t num = (int64_t)(ay.d - ay.w) * ((dx - wx) * l00 + wx * l01) +
                            (int64_t)ay.w * ((dx - wx) * l10 + wx * l11);
        const int64_t den = (int64_t)dx * ay.d;
        o[e] = (uint32_t)round_div(num, den);
      }
    }
    if (full) {
      if constexpr (ES == 1) {
        *reinterpret_cast<uint32_t*>(orow + xq) = o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24);
      } else {
        *reinterpret_cast<uint32_t*>(orow + xq) = o[0] | (o[1] << 16);
        *reinterpret_cast<uint32_t*>(orow + xq + 2) = o[2] | (o[3] << 16);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c0 + e < nq) orow[xq + e] = (T)o[e];
    }
  }
}

// CLAHE, pass 2, by cells: the frame falls into (tx + 1) x (ty + 1) cells
// bounded by the tile centres, and all pixels of a cell blend the same four
// mappings over the same denominators.  A workgroup takes a band of rows of
// one cell: it lays the four mappings in LDS as one 8-byte entry per bin
// (one read per pixel), its threads take groups of four pixels in order, U
// of them requested together, and the division by the cell's constant is a
// shift or a product.  The weights are linear in x and y, both of a pair in
// one word.  Every pixel is read and written by one thread, bytes of another
// cell in a group are left alone, so the pass may run in place.
// kTop16: the horizontal blends fit 16 bits, so both halves of the blend are
// 16-bit dot products; otherwise they are products of 24-bit factors (both
// checked on the host, as is that the numerator fits 32 bits).
// 64 x 1 MP u8 on 8 x 8 tiles: 85 -> 45 us, 8 x 4K u16 on 7 x 5 tiles: 187
// -> 72 us (the kernel above: a table of column constants per thread, four reads per pixel
// from the staged (u8) or global (u16) mappings, full 32- or 64-bit products).
struct CellAxis {
  int lo, hi;   // pixels [lo, hi)
  int ta, tb;   // the two tiles
  int w0, d;    // weight of tb at pixel x: (2 x - w0) / d
};
// cell k of an axis: between the centres of tiles k - 1 and k
__device__ __forceinline__ CellAxis clahe_cell(int k, int L, int n) {
  CellAxis r;
  // the first pixel at or right of tile a's centre (e(a) + e(a+1) - 1) / 2
  auto start = [&](int a) { return (tile_edge(a, L, n) + tile_edge(a + 1, L, n)) >> 1; };
  r.lo = k == 0 ? 0 : start(k - 1);
  r.hi = k == n ? L : start(k);
  if (k == 0 || k == n) {
    r.ta = r.tb = k == 0 ? 0 : n - 1;
    r.w0 = 0;
    r.d = 0;   // (one tile: the weights are constant, see below)
  } else {
    r.ta = k - 1;
    r.tb = k;
    r.w0 = tile_edge(k - 1, L, n) + tile_edge(k, L, n) - 1;
    r.d = tile_edge(k + 1, L, n) - tile_edge(k - 1, L, n);
  }
  return r;
}

template <typename T, int NT, int NB, int SH, bool kTop16>
__global__ __launch_bounds__(NT) void k_clahe_cells(const uint8_t* in, uint8_t* out, int64_t pitch, int64_t stride,
                                                    int W, int H, int tx, int ty, int bands, int band_rows,
                                                    const uint16_t* __restrict__ lut, const uint8_t* mask) {
  constexpr int ES = (int)sizeof(T), NW = ES;   // words of a group of four pixels
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  __shared__ __align__(16) uint2 s_lut[NB];     // {top left | top right << 16, bottom left | bottom right << 16}
  const int pair = blockIdx.z;
  if (slot_off(mask, pair)) return;
  const int t = threadIdx.x;
  const int ky = blockIdx.y / bands, band = blockIdx.y - ky * bands;
  const CellAxis cx = clahe_cell(blockIdx.x, W, tx), cy = clahe_cell(ky, H, ty);
  const int y_lo = cy.lo + band * band_rows, y_hi = min(y_lo + band_rows, cy.hi);
  if (cx.lo >= cx.hi || y_lo >= y_hi) return;   // (the whole workgroup)
  {
    const uint16_t* Lp = lut + (int64_t)pair * ty * tx * NB;
    const uint32_t* q00 = reinterpret_cast<const uint32_t*>(Lp + ((int64_t)cy.ta * tx + cx.ta) * NB);
    const uint32_t* q01 = reinterpret_cast<const uint32_t*>(Lp + ((int64_t)cy.ta * tx + cx.tb) * NB);
    const uint32_t* q10 = reinterpret_cast<const uint32_t*>(Lp + ((int64_t)cy.tb * tx + cx.ta) * NB);
    const uint32_t* q11 = reinterpret_cast<const uint32_t*>(Lp + ((int64_t)cy.tb * tx + cx.tb) * NB);
    for (int k = t; k < NB / 2; k += NT) {   // two bins of each mapping a word
      const uint32_t a = q00[k], b = q01[k], c = q10[k], d = q11[k];
      s_lut[2 * k] = make_uint2((a & 0xffffu) | (b << 16), (c & 0xffffu) | (d << 16));
      s_lut[2 * k + 1] = make_uint2((a >> 16) | (b & 0xffff0000u), (c >> 16) | (d & 0xffff0000u));
    }
  }
  // weights as (d - w) | w << 16 with w = 2 x - w0; an edge cell's are 1 | 0,
  // and 2 | 0 across where that leaves the denominator 1 (the rounded
  // quotient of twice numerator and denominator is the same)
  const int dy = cy.d ? cy.d : 1, dx = cx.d ? cx.d : (dy == 1 ? 2 : 1);
  const uint32_t wx_c = cx.d ? (uint32_t)(cx.d + cx.w0) - ((uint32_t)cx.w0 << 16) : (uint32_t)dx;
  const uint32_t wy_c = cy.d ? (uint32_t)(cy.d + cy.w0) - ((uint32_t)cy.w0 << 16) : 1u;
  const uint32_t wstep = 0x20000u - 2u;                  // per pixel
  const uint32_t wx_s = cx.d ? wstep : 0u, wy_s = cy.d ? wstep : 0u;
  const uint32_t den = (uint32_t)dx * (uint32_t)dy, half = den / 2;
  // floor(n2 / den), den >= 2: n2 M / 2^(32 + k), M = ceil(2^(32 + k) / den),
  // k = ceil(log2 den) - 1, is exact for n2 < 2^31 (its error n2 (M den -
  // 2^(32+k)) / den stays below 2^(32+k) / den) and else at most one too large
  const int kd = 31 - __builtin_clz(den - 1);
  const uint32_t md = (uint32_t)((((uint64_t)1 << (32 + kd)) + den - 1) / den);
  const bool pow2 = (den & (den - 1)) == 0;
  __syncthreads();

  const uint8_t* src = in + (int64_t)pair * stride;
  uint8_t* dst = out + (int64_t)pair * stride;
  const int g0 = cx.lo >> 2, ng = ((cx.hi + 3) >> 2) - g0, items = ng * (y_hi - y_lo);
  const int srow = NT / ng, scol = NT - srow * ng;   // one step of NT groups
  int ry = t / ng, rc = t - ry * ng;                 // the thread's next group
  constexpr int U = 4;
  struct __attribute__((aligned(4))) Group { uint32_t w[NW]; };
  auto cell = [&](auto pow2_c) __attribute__((always_inline)) {
    for (int p0 = t; p0 < items; p0 += U * NT) {
      Group v[U];
      int gx[U], gy[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        gx[u] = 4 * (g0 + rc);
        gy[u] = min(y_lo + ry, y_hi - 1);
        const uint8_t* row = src + (int64_t)gy[u] * pitch;
        if (gx[u] + 4 <= W) {
          v[u] = *reinterpret_cast<const Group*>(row + gx[u] * ES);
        } else {
#pragma unroll
          for (int k = 0; k < NW; ++k) v[u].w[k] = masked_word(row, W * ES, gx[u] * ES + 4 * k);
        }
        ry += srow;
        rc += scol;
        if (rc >= ng) {
          rc -= ng;
          ++ry;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (p0 + u * NT >= items) break;
        const uint32_t wy = wy_c + (uint32_t)gy[u] * wy_s;
        uint32_t wx = wx_c + (uint32_t)gx[u] * wx_s;
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t px = ES == 1 ? (v[u].w[0] >> (8 * e)) & 0xffu : (v[u].w[(e * ES) >> 2] >> (16 * (e & 1))) & 0xffffu;
          const uint2 l = s_lut[(px >> SH) & (NB - 1)];
          const uint32_t top = (uint32_t)__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, l.x),
                                                                __builtin_bit_cast(u16x2, wx), 0u, false);
          const uint32_t bot = (uint32_t)__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, l.y),
                                                                __builtin_bit_cast(u16x2, wx), 0u, false);
          uint32_t n2;
          if constexpr (kTop16)
            n2 = (uint32_t)__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, top | (bot << 16)),
                                                  __builtin_bit_cast(u16x2, wy), half, false);
          else
            n2 = (uint32_t)__umul24(top, wy & 0xffffu) + (uint32_t)__umul24(bot, wy >> 16) + half;
          if constexpr (decltype(pow2_c)::value) {
            o[e] = n2 >> (kd + 1);
          } else {
            o[e] = __umulhi(n2, md) >> kd;
            if constexpr (!kTop16) o[e] -= o[e] * den > n2 ? 1u : 0u;
          }
          wx += wx_s;
        }
        T* orow = reinterpret_cast<T*>(dst + (int64_t)gy[u] * pitch);
        if (gx[u] >= cx.lo && gx[u] + 4 <= cx.hi) {
          Group w;
          if constexpr (ES == 1) {
            w.w[0] = o[0] | (o[1] << 8) | (o[2] << 16) | (o[3] << 24);
          } else {
            w.w[0] = o[0] | (o[1] << 16);
            w.w[NW - 1] = o[2] | (o[3] << 16);
          }
          *reinterpret_cast<Group*>(orow + gx[u]) = w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (gx[u] + e >= cx.lo && gx[u] + e < cx.hi) orow[gx[u] + e] = (T)o[e];
        }
      }
    }
  };
  if (pow2) cell(std::true_type());
  else cell(std::false_type());
}

}  // namespace

int clahe_bins(const Plan& P) {
  const int bits = P.p.dtype == PIV_U8 ? 8 : P.p.bit_depth;
  return 1 << (bits < 12 ? bits : 12);
}

hipError_t launch_highpass(const Plan& P, const void* in, void* out, int64_t pitch, int n, int r, hipStream_t s) {
  const int nout = 64 - 2 * ((r + 3) / 4);             // groups of four pixels written per strip
  const int words = (P.p.width + 3) / 4;
  const int band = P.es == 1 ? hp_band<uint8_t>() : hp_band<uint16_t>();
  dim3 grid((words + nout - 1) / nout, (P.p.height + band - 1) / band, n);
  const int64_t stride = pitch * P.p.height;
  const uint8_t* i8 = (const uint8_t*)in;
  uint8_t* o8 = (uint8_t*)out;
  switch (r) {
#define PIV_HP(R_)                                                                                               \
  case R_:                                                                                                     \
    if (P.es == 1)                                                                                             \
      hipLaunchKernelGGL((k_highpass<uint8_t, R_>), grid, dim3(64), 0, s, i8, o8, pitch, stride, P.p.width,   \
                         P.p.height, P.slot_mask);                                                              \
    else                                                                                                       \
      hipLaunchKernelGGL((k_highpass<uint16_t, R_>), grid, dim3(64), 0, s, i8, o8, pitch, stride, P.p.width,  \
                         P.p.height, P.slot_mask);                                                              \
    break;
    PIV_HP(1) PIV_HP(2) PIV_HP(3) PIV_HP(4) PIV_HP(5) PIV_HP(6) PIV_HP(7) PIV_HP(8)
    PIV_HP(9) PIV_HP(10) PIV_HP(11) PIV_HP(12) PIV_HP(13) PIV_HP(14) PIV_HP(15) PIV_HP(16)
#undef PIV_HP
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The staged map kernel holds the mappings of every tile a block can touch:
// at most (columns of MQ pixels' tiles + 2) x (rows of MR rows' tiles + 2).
static bool clahe_stage_fits(const Plan& P, int tx, int ty, int nbins) {
  const int tw = P.p.width / tx, th = P.p.height / ty;   // smallest tile sizes
  if (tw < 1 || th < 1) return false;
  const int ncol = MQ / tw + 3, nrow = MR / th + 3;
  return (int64_t)ncol * nrow * nbins / 2 <= kStageWords;
}

hipError_t launch_clahe(const Plan& P, const void* in, void* out, int64_t pitch, int n, int tx, int ty,
                        double clip_factor, uint16_t* lut, hipStream_t s) {
  const int bits = P.p.dtype == PIV_U8 ? 8 : P.p.bit_depth;
  const int nbins = clahe_bins(P), shift = bits - (bits < 12 ? bits : 12), maxval = (1 << bits) - 1;
  const int64_t stride = pitch * P.p.height;
  const uint8_t* i8 = (const uint8_t*)in;
  uint8_t* o8 = (uint8_t*)out;
  dim3 g1(tx, ty, n);
#define PIV_LUT(T_, NT_, NH_, HB_, SH_)                                                                                \
  hipLaunchKernelGGL((k_clahe_lut<T_, NT_, NH_, HB_, SH_>), g1, dim3(NT_), 0, s, i8, pitch, stride, P.p.width, P.p.height, \
                     tx, ty, nbins, maxval, clip_factor, lut, P.slot_mask)
  if (P.es == 1) PIV_LUT(uint8_t, 256, 8, 256, 0);
  else if (shift == 0) PIV_LUT(uint16_t, 1024, 2, 4096, 0);
  else PIV_LUT(uint16_t, 1024, 2, 4096, 4);   // 16 bits in 4096 bins
#undef PIV_LUT
  if (hipError_t e = hipGetLastError()) return e;
  // the blend denominator per axis is a centre distance in doubled
  // coordinates, e(a+2) - e(a)
  auto dmax = [](int L, int n) {
    int64_t m = 2;
    for (int a = 0; a + 2 <= n; ++a) m = std::max<int64_t>(m, (int64_t)(a + 2) * L / n - (int64_t)a * L / n);
    return m;
  };
  const int64_t dxm = dmax(P.p.width, tx), dd = dxm * dmax(P.p.height, ty);
  // By cells where numerators, and the quotient times its denominator, fit 32
  // bits, and for u8 while a tile has 1,024 pixels or more: a cell lays all
  // bins of its mappings in LDS whatever its size (16 x 1 MP u8, both passes:
  // 28 against 38 us at tiles of 128 x 128, 41 and 70 at 64 x 64, 109 and 107
  // at 32 x 32, 392 and 239 at 16 x 16; u16 is faster by cells down to 30 x
  // 17, 439 and 500 us).
  if ((maxval + 2) * dd < (int64_t(1) << 32) && maxval * dxm < (1 << 24) &&
      (P.es == 2 || (int64_t)P.p.width * P.p.height >= (int64_t)1024 * tx * ty)) {
    const bool top16 = maxval * dxm < 65536 && (maxval + 1) * dd < (int64_t(1) << 31);
    auto cell_max = [](int L, int n) {   // the largest extent of a cell
      auto start = [&](int a) { return (int)(((int64_t)a * L / n + (int64_t)(a + 1) * L / n) >> 1); };
      int m = std::max(start(0), L - start(n - 1));
      for (int a = 1; a < n; ++a) m = std::max(m, start(a) - start(a - 1));
      return m;
    };
    // pixels of a workgroup: enough to pay for its mappings (2 and 32 KB);
    // half as many u8, or twice as many u16, take 17% and 7% longer
    const int rows = cell_max(P.p.height, ty), target = P.es == 1 ? 16384 : 32768;
    const int band_rows = std::min(rows, std::max(8, target / cell_max(P.p.width, tx)));
    const int bands = (rows + band_rows - 1) / band_rows;
    dim3 gc(tx + 1, (ty + 1) * bands, n);
#define PIV_CELLS(T_, NT_, NB_, SH_, TOP_)                                                                              \
  hipLaunchKernelGGL((k_clahe_cells<T_, NT_, NB_, SH_, TOP_>), gc, dim3(NT_), 0, s, i8, o8, pitch, stride, P.p.width,     \
                     P.p.height, tx, ty, bands, band_rows, (const uint16_t*)lut, P.slot_mask)
    if (P.es == 1) {
      if (top16) PIV_CELLS(uint8_t, 256, 256, 0, true);
      else PIV_CELLS(uint8_t, 256, 256, 0, false);
    } else if (shift == 0) {
      if (top16) PIV_CELLS(uint16_t, 512, 4096, 0, true);
      else PIV_CELLS(uint16_t, 512, 4096, 0, false);
    } else {   // (16-bit values: a blend over two pixels or more leaves 16 bits)
      PIV_CELLS(uint16_t, 512, 4096, 4, false);
    }
#undef PIV_CELLS
    return hipGetLastError();
  }
  dim3 g2((P.p.width + MQ - 1) / MQ, (P.p.height + MR - 1) / MR, n);
  // small u8 tiles (their numerators stay below 2^24), and blends beyond 32 bits
  const bool staged = clahe_stage_fits(P, tx, ty, nbins), narrow = maxval * dd + dd / 2 < (int64_t(1) << 24);
#define PIV_MAP(T_, ST_, NA_)                                                                                           \
  hipLaunchKernelGGL((k_clahe_map<T_, ST_, NA_>), g2, dim3(256), 0, s, i8, o8, pitch, stride, P.p.width, P.p.height, tx, \
                     ty, nbins, shift, (const uint16_t*)lut, P.slot_mask)
  if (P.es == 2) PIV_MAP(uint16_t, false, false);
  else if (staged && narrow) PIV_MAP(uint8_t, true, true);
  else if (narrow) PIV_MAP(uint8_t, false, true);
  else if (staged) PIV_MAP(uint8_t, true, false);
  else PIV_MAP(uint8_t, false, false);
#undef PIV_MAP
  return hipGetLastError();
}

}  // namespace piv
