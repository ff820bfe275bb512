// Frame pre-processing: letterbox-resize + normalise (uint8 HWC frame -> NHWC
// tensor of the model's type) and ROI crop-resize (a variable number of source
// boxes -> fixed-size crops).  Both are bilinear with half-pixel centres, taps
// clamped to the frame, no antialias filter, one rounding to the output type.
//
// Each lane produces PX neighbouring output pixels of one row and writes them
// with 8/16-byte stores; a wavefront therefore covers a contiguous output span
// and a contiguous span of each tapped source row.
#include "octo_internal.h"

namespace octo {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// PX pixels, contiguous; C4: every pixel is written as 4 values (RGB + 0)
template <typename T, int PX, bool C4>
__device__ __forceinline__ void store_pixels(T* dst, const float* v) {
  if (C4) {
    typedef T t4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const t4 o = {(T)v[3 * p], (T)v[3 * p + 1], (T)v[3 * p + 2], (T)0.0f};
      *(t4*)(dst + 4 * p) = o;
    }
  } else if (PX == 4) {
    alignas(16) T o[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) o[i] = (T)v[i];
    if (sizeof(T) == 2) {
      uint2* d = (uint2*)dst; const uint2* s = (const uint2*)o;
      d[0] = s[0]; d[1] = s[1]; d[2] = s[2];
    } else {
      float4* d = (float4*)dst; const float4* s = (const float4*)o;
      d[0] = s[0]; d[1] = s[1]; d[2] = s[2];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 3 * PX; ++i) dst[i] = (T)v[i];
  }
}

// Frame addresses come out of a table in memory, where the compiler cannot see that they are global memory: it would load with instructions
// that count as LDS accesses too, and wait for all of them before it reads LDS.
typedef const __attribute__((address_space(1))) uint8_t* Src;
__device__ __forceinline__ Src frame_of(const ResizeArgs& a, int i) { return (Src)(uintptr_t)a.frames[i]; }

// 12 source bytes (4 RGB pixels) starting at pixel ws of a row, fetched with one unaligned 3-dword load
struct __attribute__((packed)) Win12 { uint32_t d0, d1, d2; };
__device__ __forceinline__ Win12 load_window(Src row, int ws) {
  const auto* p = (const __attribute__((address_space(1))) Win12*)(row + 3 * ws);
  return {p->d0, p->d1, p->d2};
}
// the three channels of the pixel that starts at byte `off` (0, 3, 6 or 9) of the window
__device__ __forceinline__ void window_pixel(const Win12& w, int off, float* rgb) {
  const unsigned long long lo = (unsigned long long)w.d0 | ((unsigned long long)w.d1 << 32);
  const unsigned long long hi = (unsigned long long)w.d1 | ((unsigned long long)w.d2 << 32);
  const unsigned v = off < 4 ? (unsigned)(lo >> (8 * off)) : (unsigned)(hi >> (8 * (off - 4)));
  rgb[0] = (float)(v & 0xFFu); rgb[1] = (float)((v >> 8) & 0xFFu); rgb[2] = (float)((v >> 16) & 0xFFu);
}

// Bilinear sample of taps (xa, xb) x (row_a, row_b); xb is xa or xa + 1 (clamping), so both taps of a row come from
// one window.  Needs src_w >= 4.
__device__ __forceinline__ void bilinear_rgb(Src row_a, Src row_b, int xa, int xb, int src_w, float fx, float fy,
                                             const float* scale, const float* bias, float* out) {
  const int ws = xa < src_w - 4 ? xa : src_w - 4;
  const Win12 wa = load_window(row_a, ws), wb = load_window(row_b, ws);
  float p00[3], p01[3], p10[3], p11[3];
  window_pixel(wa, 3 * (xa - ws), p00); window_pixel(wa, 3 * (xb - ws), p01);
  window_pixel(wb, 3 * (xa - ws), p10); window_pixel(wb, 3 * (xb - ws), p11);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    float top = (1.0f - fx) * p00[c] + fx * p01[c];
    float bot = (1.0f - fx) * p10[c] + fx * p11[c];
    out[c] = ((1.0f - fy) * top + fy * bot) * scale[c] + bias[c];
  }
}

struct LetterboxGeom { int nw, nh, left, top; };

// EXACT: the source / resized size ratio is an odd integer in both directions, so every output pixel is exactly one
// source pixel (1080p -> 640x360 and 2160p -> 1280x720 are ratio 3): one window load per pixel, no interpolation.
//
// Four pixels at ratio 3 are 36 consecutive bytes of the source row; where those are aligned to 4 they are loaded as words, and a value
// is a byte of a word at a place known at compile time (byte windows : words, frames from memory, us: 8 frames 1080p to 640 x 640 x 4 17.9 :
// 15.3, 32 50 : 37, 32 of 2160p to 1280 x 1280 x 4 with the rows in groups 204 : 129, 3.7 TB/s).  R rows per lane: a lane's time is two dependent trips to memory, the frame's
// address and then its pixels, and the rows' words are loaded beside each other.  letterbox_p says when.  Frames whose addresses turn
// out not to be aligned take their rows one after the other.
// BEGIN: the launch is also the batch's first, begin_kernel's work included, and takes the frames from its arguments instead of the table that it writes for the later ones.
struct NoBegin {};
template <typename T, int PX, bool C4, bool EXACT, int R, bool BEGIN>
__global__ void letterbox_kernel(const ResizeArgs a, const LetterboxGeom g, const std::conditional_t<BEGIN, BeginArgs, NoBegin> b) {
  if constexpr (BEGIN) begin_batch(b, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
  const int wq = a.dst_w / PX;
  int n_items = a.n;
  if (a.n_dyn) { int d = *a.n_dyn; n_items = d < a.n ? d : a.n; }
  const unsigned groups = (unsigned)(a.dst_h + R - 1) / R;                             // of rows; a.div_h divides by this
  const unsigned total = (unsigned)n_items * groups * (unsigned)wq;                  // < 2^31 (checked by the launcher)
  T* dst = (T*)a.dst;
  const int rx = a.src_w / g.nw, ry = a.src_h / g.nh;      // only meaningful when EXACT
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const unsigned t = fast_div(i, a.div_wq);
    const int xq = (int)(i - t * (unsigned)wq);
    const int img = (int)fast_div(t, a.div_h);
    const int y0 = (int)(t - (unsigned)img * groups) * R;
    Src base;
    size_t pitch;
    if constexpr (BEGIN) { base = (Src)b.ptr[img]; pitch = b.pitch[img]; }
    else { base = frame_of(a, img); pitch = a.pitches[img]; }
    T* out = dst + (((size_t)img * a.dst_h + y0) * a.dst_w + (size_t)xq * PX) * (C4 ? 4 : 3);
    const size_t out_pitch = (size_t)a.dst_w * (C4 ? 4 : 3);
    if constexpr (EXACT && PX == 4) {
      const int xi0 = xq * 4 - g.left;
      if (rx == 3 && xi0 >= 0 && xi0 + 4 <= g.nw && (((uintptr_t)base | pitch | (unsigned)(9 * xi0)) & 3) == 0) {
        uint32_t w[R][9];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int yi = y0 + r - g.top;
          if ((unsigned)yi >= (unsigned)g.nh) continue;
          const auto* p = (const __attribute__((address_space(1))) uint32_t*)(base + (size_t)(ry * yi + (ry - 1) / 2) * pitch + 9 * xi0);
#pragma unroll
          for (int k = 0; k < 9; ++k) w[r][k] = p[k];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (y0 + r >= a.dst_h) break;
          const bool row_in = (unsigned)(y0 + r - g.top) < (unsigned)g.nh;
          float v[12];
#pragma unroll
          for (int px = 0; px < 4; ++px)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              constexpr int CENTRE = 3;      // byte of the middle pixel of three
              const int at = 9 * px + CENTRE + c;
              v[3 * px + c] = (row_in ? (float)((w[r][at / 4] >> (at % 4 * 8)) & 0xFFu) : (float)a.pad_value) * a.scale[c] + a.bias[c];
            }
          store_pixels<T, PX, C4>(out + r * out_pitch, v);
        }
        continue;
      }
    }
#pragma unroll 1
    for (int y = y0; y < y0 + R && y < a.dst_h; ++y) {
      float v[3 * PX];
      const int yi = y - g.top;
      const bool row_in = (unsigned)yi < (unsigned)g.nh;
      int ya = 0, yb = 0; float fy = 0.f;
      if (row_in) {
        if (EXACT) {
          ya = yb = ry * yi + (ry - 1) / 2;
        } else {
          // source y = (yi + 0.5) * Hs / nh - 0.5 = ((2 yi + 1) Hs - nh) / (2 nh), split exactly into floor and fraction
          const int num = (2 * yi + 1) * a.src_h - g.nh, den = 2 * g.nh;
          int ys = num >= 0 ? num / den : -((-num + den - 1) / den);
          fy = (float)(num - ys * den) / (float)den;
          ya = clampi(ys, 0, a.src_h - 1); yb = clampi(ys + 1, 0, a.src_h - 1);
        }
      }
#pragma unroll
      for (int px = 0; px < PX; ++px) {
        const int xi = xq * PX + px - g.left;
        if (row_in && (unsigned)xi < (unsigned)g.nw) {
          if (EXACT) {
            const int xs = rx * xi + (rx - 1) / 2;
            const int ws = xs < a.src_w - 4 ? xs : a.src_w - 4;
            float rgb[3];
            window_pixel(load_window(base + (size_t)ya * pitch, ws), 3 * (xs - ws), rgb);
#pragma unroll
            for (int c = 0; c < 3; ++c) v[3 * px + c] = rgb[c] * a.scale[c] + a.bias[c];
          } else {
            const int num = (2 * xi + 1) * a.src_w - g.nw, den = 2 * g.nw;
            int x0 = num >= 0 ? num / den : -((-num + den - 1) / den);
            const float fx = (float)(num - x0 * den) / (float)den;
            const int xa = clampi(x0, 0, a.src_w - 1), xb = clampi(x0 + 1, 0, a.src_w - 1);
            bilinear_rgb(base + (size_t)ya * pitch, base + (size_t)yb * pitch, xa, xb, a.src_w, fx, fy, a.scale, a.bias, v + 3 * px);
          }
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c) v[3 * px + c] = (float)a.pad_value * a.scale[c] + a.bias[c];
        }
      }
      store_pixels<T, PX, C4>(out + (y - y0) * out_pitch, v);
    }
  }
}

template <typename T, int PX, bool C4>
__global__ void crop_resize_kernel(const ResizeArgs a) {
  const int wq = a.dst_w / PX;
  int n_items = a.n;
  if (a.n_dyn) { int d = *a.n_dyn; n_items = d < a.n ? (d < 0 ? 0 : d) : a.n; }
  const unsigned total = (unsigned)n_items * (unsigned)a.dst_h * (unsigned)wq;       // < 2^31 (checked by the launcher)
  T* dst = (T*)a.dst;
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const unsigned t = fast_div(i, a.div_wq);
    const int xq = (int)(i - t * (unsigned)wq);
    const int roi = (int)fast_div(t, a.div_h);
    const int y = (int)(t - (unsigned)roi * (unsigned)a.dst_h);
    const octo_roi r = a.rois[roi];
    const int fr = clampi(r.frame, 0, a.n_frames - 1);
    const Src base = frame_of(a, fr);
    const size_t pitch = a.pitches[fr];
    const float sy = r.y1 + ((float)y + 0.5f) * ((r.y2 - r.y1) / (float)a.dst_h) - 0.5f;
    const float y0f = floorf(sy);
    const float fy = sy - y0f;
    const int ya = clampi((int)y0f, 0, a.src_h - 1), yb = clampi((int)y0f + 1, 0, a.src_h - 1);
    const float step = (r.x2 - r.x1) / (float)a.dst_w;
    float v[3 * PX];
#pragma unroll
    for (int px = 0; px < PX; ++px) {
      const float sx = r.x1 + ((float)(xq * PX + px) + 0.5f) * step - 0.5f;
      const float x0f = floorf(sx);
      const float fx = sx - x0f;
      const int xa = clampi((int)x0f, 0, a.src_w - 1), xb = clampi((int)x0f + 1, 0, a.src_w - 1);
      bilinear_rgb(base + (size_t)ya * pitch, base + (size_t)yb * pitch, xa, xb, a.src_w, fx, fy, a.scale, a.bias, v + 3 * px);
    }
    store_pixels<T, PX, C4>(dst + (((size_t)roi * a.dst_h + y) * a.dst_w + (size_t)xq * PX) * (C4 ? 4 : 3), v);
  }
}

// Crop-resize with the source rows staged in LDS.  One wavefront (a 64-thread workgroup) produces a few consecutive output rows of
// one ROI, 4 pixels per lane.  A source row is copied into LDS - only the span of pixels this part of the output row needs, with
// aligned 16-byte loads -, every lane picks its taps from there and keeps the 12 horizontally interpolated values in registers
// for as long as output rows tap that source row.  Sampling straight from global memory costs two 12-byte loads at arbitrary
// addresses per output pixel; for crops that are enlarged or mildly reduced (the usual case: objects of 24-360 pixels to 224)
// neighbouring lanes hit the same few cache lines over and over, and the kernel runs at the rate the L1 can look lines up.  With
// the rows in LDS it is bound by vector arithmetic, about 100 instructions per pixel with both source rows of every output row
// interpolated anew; an enlarged crop needs less than one new source row per output row (3617 crops to 224 x 224: 776 -> 449 us).
// A span too long for the buffer (strong reduction: taps of neighbouring pixels share no lines anyway) is sampled
// directly, as in the kernel above.  Same arithmetic, so the results are identical.
constexpr int CROP_ROWBUF = 2048;     // bytes of LDS for the staged source row
constexpr int CROP_ROWS = 8;          // most output rows of one ROI per wavefront

template <typename T, bool C4>
__global__ __launch_bounds__(64) void crop_resize_rows_kernel(const ResizeArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t srow[CROP_ROWBUF];
  const int wq = a.dst_w / 4;
  int n_items = a.n;
  if (a.n_dyn) { int d = *a.n_dyn; n_items = d < a.n ? (d < 0 ? 0 : d) : a.n; }
  const int lane = threadIdx.x;
  T* dst = (T*)a.dst;
  // Workgroup b runs on die b % 8, and each die has its own L2.  The rows of one ROI tap the same source lines again
  // and again (an enlarged crop reads every source row several times), so all rows of ROI r are given to die r % 8:
  // spread over the dies, each of the eight L2s fetched the ROI's pixels from memory for itself.  Within a die the
  // workgroups take consecutive rows, so the rows of one ROI are in flight together.  The grid is a multiple of 8.
  const unsigned die = blockIdx.x & 7u, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
  const unsigned die_rois = (unsigned)n_items > die ? ((unsigned)n_items - die + 7u) >> 3 : 0u;
  // rows per wavefront: as many as leave every workgroup something to do
  unsigned rows = die_rois * (unsigned)a.dst_h / slots;                    // < 2^31 (checked by the launcher)
  rows = rows < 1u ? 1u : (rows > (unsigned)CROP_ROWS ? (unsigned)CROP_ROWS : rows);
  const unsigned per_roi = ((unsigned)a.dst_h + rows - 1u) / rows;
  for (unsigned u = slot; u < die_rois * per_roi; u += slots) {
    const unsigned nth = u / per_roi;
    const int roi = (int)(die + 8u * nth);
    const int y0 = (int)((u - nth * per_roi) * rows), y1 = y0 + (int)rows < a.dst_h ? y0 + (int)rows : a.dst_h;
    const octo_roi r = a.rois[roi];
    const int fr = clampi(r.frame, 0, a.n_frames - 1);
    const Src base = frame_of(a, fr);
    const size_t pitch = a.pitches[fr];
    const float ystep = (r.y2 - r.y1) / (float)a.dst_h, step = (r.x2 - r.x1) / (float)a.dst_w;
    for (int xq0 = 0; xq0 < wq; xq0 += 64) {
      // source pixels this chunk of the row taps: the coordinate is monotonic in the output pixel, so the ends bound it
      const int pa = xq0 * 4, pb = (xq0 + 64 < wq ? xq0 + 64 : wq) * 4 - 1;
      const float sa = r.x1 + ((float)pa + 0.5f) * step - 0.5f, sb = r.x1 + ((float)pb + 0.5f) * step - 0.5f;
      const int xlo = clampi((int)floorf(fminf(sa, sb)), 0, a.src_w - 1);
      const int xhi = clampi((int)floorf(fmaxf(sa, sb)) + 1, 0, a.src_w - 1);
      const int span = (xhi - xlo + 1) * 3;
      const bool staged = span > 0 && span + 32 <= CROP_ROWBUF;
      const int xq = xq0 + lane;
      int xa[4], xb[4];
      float fx[4];
#pragma unroll
      for (int px = 0; px < 4; ++px) {
        const float sx = r.x1 + ((float)(xq * 4 + px) + 0.5f) * step - 0.5f;
        const float x0f = floorf(sx);
        fx[px] = sx - x0f;
        xa[px] = clampi((int)x0f, 0, a.src_w - 1); xb[px] = clampi((int)x0f + 1, 0, a.src_w - 1);
      }
      // source row ys: staged, and interpolated at this lane's four pixels
      auto interpolate = [&](int ys, float (&h)[12]) __attribute__((always_inline)) {
        const Src rowp = base + (size_t)ys * pitch;
        const Src p0 = rowp + 3 * xlo;
        const Src a0 = (Src)((uintptr_t)p0 & ~(uintptr_t)15);
        const int nvec = (int)((p0 + span - a0 + 15) >> 4);
        const Src row_end = rowp + (size_t)a.src_w * 3;
        __syncthreads();                   // the row before has been read
        for (int v = lane; v < nvec; v += 64) {
          const Src va = a0 + 16 * v;
          u32x4 q;
          if (va >= rowp && va + 16 <= row_end) {
            q = *(const __attribute__((address_space(1))) u32x4*)va;
          } else {
            // first or last vector of the row: never touch bytes outside the row
            alignas(16) uint8_t b[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) b[e] = (va + e >= rowp && va + e < row_end) ? va[e] : (uint8_t)0;
            q = *(const u32x4*)b;
          }
          *(u32x4*)&srow[16 * v] = q;
        }
        __syncthreads();
        const int koff = (int)(p0 - a0) - 3 * xlo;     // LDS byte index of source pixel x: koff + 3 * x
#pragma unroll
        for (int px = 0; px < 4; ++px) {
          int k = koff + 3 * xa[px];
          k = k < 0 ? 0 : (k > CROP_ROWBUF - 12 ? CROP_ROWBUF - 12 : k);      // taps lie inside the span; non-finite boxes must not index outside the buffer
          const uint32_t* w = (const uint32_t*)&srow[k & ~3];
          const unsigned lo = __builtin_amdgcn_alignbyte(w[1], w[0], k & 3), hi = __builtin_amdgcn_alignbyte(w[2], w[1], k & 3);
          const unsigned nx = xb[px] == xa[px] ? lo : __builtin_amdgcn_alignbyte(hi, lo, 3);
#pragma unroll
          for (int c = 0; c < 3; ++c)
            h[3 * px + c] = (1.0f - fx[px]) * (float)((lo >> (8 * c)) & 0xFFu) + fx[px] * (float)((nx >> (8 * c)) & 0xFFu);
        }
      };
      int ra = -1, rb = -1;                // source rows behind ha and hb
      float ha[12], hb[12];
      for (int y = y0; y < y1; ++y) {
        const float sy = r.y1 + ((float)y + 0.5f) * ystep - 0.5f;
        const float y0f = floorf(sy);
        const float fy = sy - y0f;
        const int ya = clampi((int)y0f, 0, a.src_h - 1), yb = clampi((int)y0f + 1, 0, a.src_h - 1);
        float v[12];
        if (staged) {
          if (ya != ra) {
            if (ya == rb) {
#pragma unroll
              for (int i = 0; i < 12; ++i) ha[i] = hb[i];
            } else {
              interpolate(ya, ha);
            }
            ra = ya;
          }
          if (yb != rb) {
            if (yb == ra) {
#pragma unroll
              for (int i = 0; i < 12; ++i) hb[i] = ha[i];
            } else {
              interpolate(yb, hb);
            }
            rb = yb;
          }
#pragma unroll
          for (int i = 0; i < 12; ++i) v[i] = ((1.0f - fy) * ha[i] + fy * hb[i]) * a.scale[i % 3] + a.bias[i % 3];
        } else if (xq < wq) {
#pragma unroll
          for (int px = 0; px < 4; ++px)
            bilinear_rgb(base + (size_t)ya * pitch, base + (size_t)yb * pitch, xa[px], xb[px], a.src_w, fx[px], fy, a.scale, a.bias, v + 3 * px);
        }
        if (xq < wq) store_pixels<T, 4, C4>(dst + (((size_t)roi * a.dst_h + y) * a.dst_w + (size_t)xq * 4) * (C4 ? 4 : 3), v);
      }
    }
  }
}

static inline unsigned resize_grid(long long work) {
  long long g = (work + 255) / 256;
  if (g < 1) g = 1;
  if (g > 256 * 32) g = 256 * 32;
  return (unsigned)g;
}

static LetterboxGeom letterbox_geom(int src_h, int src_w, int dst_h, int dst_w) {
  // scale r = min(dst_w/src_w, dst_h/src_h); resized size rounded half-up; centred with floor
  double r = (double)dst_w / src_w;
  if ((double)dst_h / src_h < r) r = (double)dst_h / src_h;
  LetterboxGeom g;
  g.nw = (int)(src_w * r + 0.5);
  g.nh = (int)(src_h * r + 0.5);
  if (g.nw < 1) g.nw = 1;
  if (g.nh < 1) g.nh = 1;
  g.left = (dst_w - g.nw) / 2;
  g.top = (dst_h - g.nh) / 2;
  return g;
}

void letterbox_geometry(int src_h, int src_w, int dst_h, int dst_w, int* nw, int* nh, int* left, int* top) {
  LetterboxGeom g = letterbox_geom(src_h, src_w, dst_h, dst_w);
  *nw = g.nw; *nh = g.nh; *left = g.left; *top = g.top;
}

// lanes per output row for the pixel-group width the dispatch below will pick
static bool resize_prepare(ResizeArgs& a) {
  const bool px4 = a.dst_w % 4 == 0 && ((uintptr_t)a.dst & 15) == 0;
  const int wq = px4 ? a.dst_w / 4 : a.dst_w;
  if ((long long)a.n * a.dst_h * wq >= 0x7FFFFFFFLL || a.dst_h < 1 || wq < 1) return false;
  a.div_wq = make_fastdiv((unsigned)wq);
  a.div_h = make_fastdiv((unsigned)a.dst_h);
  return true;
}

constexpr int LETTERBOX_ROWS = 4;
template <typename T, int PX, bool C4, bool EXACT> static hipError_t letterbox_p(const ResizeArgs& a, const LetterboxGeom& g, int num_cu, const BeginArgs* begin, hipStream_t s) {
  auto go = [&](auto with, auto without, long long lanes, const ResizeArgs& b) {
    if (begin) hipLaunchKernelGGL(with, dim3(resize_grid(lanes)), dim3(256), 0, s, b, g, *begin);
    else hipLaunchKernelGGL(without, dim3(resize_grid(lanes)), dim3(256), 0, s, b, g, NoBegin{});
    return hipGetLastError();
  };
  if constexpr (EXACT && PX == 4) {
    // Rows in groups where they are loaded as words (ratio 3, the left border a multiple of four pixels) and the launch is three rounds of
    // 32 wavefronts per compute unit even so: with fewer, the groups' uneven end costs more than the loads beside each other save.  One
    // row : four, frames from memory, us: 1080p to 640 x 640 x 4, 8 frames 15.3 : 15.5, 16 21.8 : 24.3, 32 36.7 : 37.9, 64 69.7 : 68.1; 2160p to
    // 1280 x 1280 x 4, 8 frames 36.9 : 38.1, 16 70.1 : 68.3, 32 138 : 129.  Rows one after the other lose with any number of frames: ratio 5, 32
    // frames 62.0 : 71.6, a border of 142 pixels 50.9 : 61.9, ratio 1, 64 frames 46 : 57.
    const long long lanes = (long long)a.n * ((a.dst_h + LETTERBOX_ROWS - 1) / LETTERBOX_ROWS) * (a.dst_w / PX);
    if (a.src_w / g.nw == 3 && g.left % 4 == 0 && lanes >= 3LL * 32 * 64 * num_cu) {
      ResizeArgs b = a;
      b.div_h = make_fastdiv((unsigned)((a.dst_h + LETTERBOX_ROWS - 1) / LETTERBOX_ROWS));
      return go(letterbox_kernel<T, PX, C4, EXACT, LETTERBOX_ROWS, true>, letterbox_kernel<T, PX, C4, EXACT, LETTERBOX_ROWS, false>, lanes, b);
    }
  }
  return go(letterbox_kernel<T, PX, C4, EXACT, 1, true>, letterbox_kernel<T, PX, C4, EXACT, 1, false>, (long long)a.n * a.dst_h * (a.dst_w / PX), a);
}
template <typename T, bool EXACT> static hipError_t letterbox_e(const ResizeArgs& a, const LetterboxGeom& g, int num_cu, const BeginArgs* begin, hipStream_t s) {
  const bool px4 = a.dst_w % 4 == 0 && ((uintptr_t)a.dst & 15) == 0;
  if (a.dst_c == 4) return px4 ? letterbox_p<T, 4, true, EXACT>(a, g, num_cu, begin, s) : letterbox_p<T, 1, true, EXACT>(a, g, num_cu, begin, s);
  return px4 ? letterbox_p<T, 4, false, EXACT>(a, g, num_cu, begin, s) : letterbox_p<T, 1, false, EXACT>(a, g, num_cu, begin, s);
}
template <typename T> static hipError_t letterbox_t(const ResizeArgs& a, int num_cu, const BeginArgs* begin, hipStream_t s) {
  const LetterboxGeom g = letterbox_geom(a.src_h, a.src_w, a.dst_h, a.dst_w);
  const bool exact = a.src_w % g.nw == 0 && a.src_h % g.nh == 0 && ((a.src_w / g.nw) & 1) && ((a.src_h / g.nh) & 1);
  return exact ? letterbox_e<T, true>(a, g, num_cu, begin, s) : letterbox_e<T, false>(a, g, num_cu, begin, s);
}
template <typename T> static hipError_t crop_t(const ResizeArgs& a, hipStream_t s) {
  // one 64-thread workgroup per output row, at most 32 per compute unit at a time; each die strides over the rows of
  // its own ROIs (every eighth), so the grid is 8 x the workgroups one die gets
  const long long die_rows = (long long)((a.n + 7) / 8) * a.dst_h;
  const unsigned row_grid = 8u * (unsigned)(die_rows < 32 * 32 ? (die_rows < 1 ? 1 : die_rows) : 32 * 32);
  if (a.dst_c == 4 && ((uintptr_t)a.dst & 15) == 0 && a.dst_w % 4 == 0) {
    hipLaunchKernelGGL((crop_resize_rows_kernel<T, true>), dim3(row_grid), dim3(64), 0, s, a);
  } else if (a.dst_c == 4) {
    hipLaunchKernelGGL((crop_resize_kernel<T, 1, true>), dim3(resize_grid((long long)a.n * a.dst_h * a.dst_w)), dim3(256), 0, s, a);
  } else if (a.dst_w % 4 == 0 && ((uintptr_t)a.dst & 15) == 0) {
    hipLaunchKernelGGL((crop_resize_rows_kernel<T, false>), dim3(row_grid), dim3(64), 0, s, a);
  } else {
    hipLaunchKernelGGL((crop_resize_kernel<T, 1, false>), dim3(resize_grid((long long)a.n * a.dst_h * a.dst_w)), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_letterbox(int dtype, const ResizeArgs& a0, int num_cu, hipStream_t s, const BeginArgs* begin) {
  if (a0.n <= 0) return hipSuccess;
  if (begin && a0.n > begin->n) return hipErrorInvalidValue;          // every item's frame is in the arguments
  ResizeArgs a = a0;
  if ((a.dst_c != 3 && a.dst_c != 4) || a.src_w < 4 || !resize_prepare(a)) return hipErrorInvalidValue;
  switch (dtype) {
    case OCTO_F32: return letterbox_t<float>(a, num_cu, begin, s);
    case OCTO_F16: return letterbox_t<_Float16>(a, num_cu, begin, s);
    case OCTO_BF16: return letterbox_t<__bf16>(a, num_cu, begin, s);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_crop_resize(int dtype, const ResizeArgs& a0, hipStream_t s) {
  if (a0.n <= 0) return hipSuccess;
  ResizeArgs a = a0;
  if ((a.dst_c != 3 && a.dst_c != 4) || a.src_w < 4 || !resize_prepare(a)) return hipErrorInvalidValue;
  switch (dtype) {
    case OCTO_F32: return crop_t<float>(a, s);
    case OCTO_F16: return crop_t<_Float16>(a, s);
    case OCTO_BF16: return crop_t<__bf16>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace octo
