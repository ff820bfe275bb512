// HBM-bound glue layers on NHWC tensors: max-pool, nearest 2x upsample, channel
// copy (concatenation fallback), element-wise add, global average pool, argmax.
// Every kernel is a grid-stride loop over (pixel, channel-vector) work items so
// that an item count held in device memory can bound the work.
#include "octo_internal.h"

namespace octo {

template <typename T> __device__ __forceinline__ float ld_f32(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void st_f32(T* p, float v) { *p = (T)v; }

__device__ __forceinline__ int dyn_items(const int* n_dyn, int n) {
  if (!n_dyn) return n;
  int d = *n_dyn;
  return d < n ? (d < 0 ? 0 : d) : n;
}

static inline unsigned grid_for(long long work, int block) {
  long long g = (work + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 256 * 16) g = 256 * 16;
  return (unsigned)g;
}

// V = channels handled per work item (1, or 16 bytes worth)
template <typename T, int V>
__global__ void maxpool_kernel(const PoolArgs a) {
  const int cv = a.C / V;
  const long long total = (long long)dyn_items(a.n_dyn, a.n) * a.Ho * a.Wo * cv;
  const T* x = (const T*)a.x;
  T* y = (T*)a.y;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    int c = (int)(i % cv) * V;
    long long pix = i / cv;
    int wo = (int)(pix % a.Wo);
    long long t = pix / a.Wo;
    int ho = (int)(t % a.Ho);
    long long img = t / a.Ho;
    float m[V];
#pragma unroll
    for (int e = 0; e < V; ++e) m[e] = -INFINITY;
    for (int r = 0; r < a.k; ++r) {
      int hi = ho * a.stride - a.pad + r;
      if ((unsigned)hi >= (unsigned)a.H) continue;
      for (int s = 0; s < a.k; ++s) {
        int wi = wo * a.stride - a.pad + s;
        if ((unsigned)wi >= (unsigned)a.W) continue;
        const T* p = x + ((size_t)(img * a.H + hi) * a.W + wi) * a.x_ld + a.x_coff + c;
        alignas(16) T v[V];
        if (V > 1) *(uint4*)v = *(const uint4*)p; else v[0] = *p;
#pragma unroll
        for (int e = 0; e < V; ++e) m[e] = fmaxf(m[e], (float)v[e]);
      }
    }
    alignas(16) T o[V];
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = (T)m[e];
    T* q = y + (size_t)pix * a.y_ld + a.y_coff + c;
    if (V > 1) *(uint4*)q = *(const uint4*)o; else *q = o[0];
  }
}

// Stride-1 "same" max-pool (window K, padding K / 2: the chained 5x5 pools of a spatial-pyramid block).  A work item
// owns one (image, row segment, column, 16-byte channel vector) and walks down the rows: of every input row it takes
// the maximum over the K columns of its window once and keeps the last K of those row maxima in registers, so an
// output costs K loads instead of K x K.  The row loop is unrolled K times so that the ring of row maxima is indexed
// statically.  Same result as maxpool_kernel: a maximum does not depend on the order it is taken in.
template <typename T, int K>
__global__ __launch_bounds__(256) void maxpool_rows_kernel(const PoolArgs a, int seg_rows, int n_seg) {
  constexpr int V = 16 / (int)sizeof(T), P = K / 2;
  const int cv = a.C / V;
  const long long total = (long long)dyn_items(a.n_dyn, a.n) * n_seg * a.W * cv;
  const T* x = (const T*)a.x;
  T* y = (T*)a.y;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    const int c = (int)(i % cv) * V;
    long long t = i / cv;
    const int wo = (int)(t % a.W); t /= a.W;
    const int seg = (int)(t % n_seg);
    const long long img = t / n_seg;
    const int r0 = seg * seg_rows, r1 = r0 + seg_rows < a.H ? r0 + seg_rows : a.H;
    const int s_lo = wo - P < 0 ? 0 : wo - P, s_hi = wo + P > a.W - 1 ? a.W - 1 : wo + P;
    float ring[K][V];
    // maximum of input row r over this item's window columns (a row outside the image contributes nothing)
    auto row_max = [&](int r, float (&m)[V]) {
#pragma unroll
      for (int e = 0; e < V; ++e) m[e] = -INFINITY;
      if ((unsigned)r >= (unsigned)a.H) return;
      const T* p = x + ((size_t)(img * a.H + r) * a.W) * a.x_ld + a.x_coff + c;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int wi = s_lo + j;
        if (wi > s_hi) break;
        alignas(16) T v[V];
        *(uint4*)v = *(const uint4*)(p + (size_t)wi * a.x_ld);
#pragma unroll
        for (int e = 0; e < V; ++e) m[e] = fmaxf(m[e], (float)v[e]);
      }
    };
#pragma unroll
    for (int j = 0; j < K - 1; ++j) row_max(r0 - P + j, ring[j]);
    for (int ho = r0; ho < r1; ho += K) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (ho + j >= r1) break;
        row_max(ho + j + P, ring[(j + K - 1) % K]);        // replaces the row that left the window
        alignas(16) T o[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          float m = ring[0][e];
#pragma unroll
          for (int q = 1; q < K; ++q) m = fmaxf(m, ring[q][e]);
          o[e] = (T)m;
        }
        *(uint4*)(y + ((size_t)(img * a.H + ho + j) * a.W + wo) * a.y_ld + a.y_coff + c) = *(const uint4*)o;
      }
    }
  }
}

// Three chained stride-1 "same" max-pools of one size (a spatial-pyramid block): a workgroup holds the whole map of NV
// 16-byte channel vectors of one item in LDS and pools it three times, rows first, then columns, writing the result of
// every stage; the map is read once and no stage waits for another launch.  A maximum does not depend on the order it is
// taken in, so the results are those of three separate pools.  Bound by vector arithmetic and LDS: values of 16-bit types are
// held as integers of the same order, so that a vector of eight takes four packed instructions per maximum (with
// conversions to and from fp32 64 x 20 x 20 x 256 took 40 us).
// Order-preserving integer of a 16-bit float: the magnitude bits of negative values are inverted; the inverse is the same
// function.  NaN takes the place of -inf (whose integer is ~inf) in all types, as in the separate pools, whose running maximum
// starts at -inf and ignores NaN: a window of nothing but NaN gives -inf.
typedef short short8v __attribute__((ext_vector_type(8)));
__device__ __forceinline__ short8v order_flip(short8v x) { return x ^ ((x >> 15) & (short)0x7FFF); }
template <typename T> __device__ __forceinline__ uint4 pool_key(uint4 q) {
  if constexpr (sizeof(T) == 4) {
    const float4 x = __builtin_bit_cast(float4, q);
    return __builtin_bit_cast(uint4, make_float4(fmaxf(x.x, -INFINITY), fmaxf(x.y, -INFINITY), fmaxf(x.z, -INFINITY), fmaxf(x.w, -INFINITY)));
  }
  const short inf = std::is_same<T, _Float16>::value ? 0x7C00 : 0x7F80;
  short8v x = __builtin_bit_cast(short8v, q);
  const short8v k = order_flip(x);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = (short)(x[e] & 0x7FFF) > inf ? (short)~inf : k[e];
  return __builtin_bit_cast(uint4, x);
}
template <typename T> __device__ __forceinline__ uint4 pool_value(uint4 q) {
  if constexpr (sizeof(T) == 4) return q;
  return __builtin_bit_cast(uint4, order_flip(__builtin_bit_cast(short8v, q)));
}
template <typename T> __device__ __forceinline__ uint4 pool_max(uint4 p, uint4 q) {
  if constexpr (sizeof(T) == 4) {
    const float4 x = __builtin_bit_cast(float4, p), y = __builtin_bit_cast(float4, q);
    return __builtin_bit_cast(uint4, make_float4(fmaxf(x.x, y.x), fmaxf(x.y, y.y), fmaxf(x.z, y.z), fmaxf(x.w, y.w)));
  }
  return __builtin_bit_cast(uint4, __builtin_elementwise_max(__builtin_bit_cast(short8v, p), __builtin_bit_cast(short8v, q)));
}

// nv_log: log2 of the channel vectors a workgroup holds; div_w: division by the map width
template <typename T>
__global__ __launch_bounds__(512) void maxpool_chain_kernel(const PoolArgs a, PoolChain ch, int nv_log, FastDiv div_w) {
  constexpr int V = 16 / (int)sizeof(T);
  extern __shared__ __attribute__((aligned(16))) unsigned char chain_lds[];
  uint4* m0 = (uint4*)chain_lds;
  const int nv = 1 << nv_log;
  const int hw = a.H * a.W, work = hw * nv, P = a.k / 2;
  uint4* m1 = m0 + work;
  const int groups = a.C / V / nv;                       // channel groups per item
  const int total = dyn_items(a.n_dyn, a.n) * groups;
  // the channel groups of one item share cache lines: they run on one die (workgroup b runs on die b % 8)
  const int per_die = (total + 7) >> 3;
  for (int b = blockIdx.x; b < per_die * 8; b += gridDim.x) {
    const int u = (b & 7) * per_die + (b >> 3);
    if (u >= total) continue;
    const int img = u / groups, c0 = (u - img * groups) * nv * V;
    const T* x = (const T*)a.x + (size_t)img * hw * a.x_ld + a.x_coff + c0;
    for (int i = threadIdx.x; i < work; i += blockDim.x)
      m0[i] = pool_key<T>(*(const uint4*)(x + (size_t)(i >> nv_log) * a.x_ld + (i & (nv - 1)) * V));
    __syncthreads();
    for (int st = 0; st < 3; ++st) {
      for (int i = threadIdx.x; i < work; i += blockDim.x) {
        const int pix = i >> nv_log, col = pix - (int)fast_div((unsigned)pix, div_w) * a.W;
        uint4 m = m0[i];
        for (int d = 1; d <= P; ++d) {
          if (col - d >= 0) m = pool_max<T>(m, m0[i - d * nv]);
          if (col + d < a.W) m = pool_max<T>(m, m0[i + d * nv]);
        }
        m1[i] = m;
      }
      __syncthreads();
      T* y = (T*)ch.y[st] + (size_t)img * hw * ch.ld[st] + ch.coff[st] + c0;
      for (int i = threadIdx.x; i < work; i += blockDim.x) {
        const int pix = i >> nv_log, row = (int)fast_div((unsigned)pix, div_w);
        uint4 m = m1[i];
        for (int d = 1; d <= P; ++d) {
          if (row - d >= 0) m = pool_max<T>(m, m1[i - d * a.W * nv]);
          if (row + d < a.H) m = pool_max<T>(m, m1[i + d * a.W * nv]);
        }
        m0[i] = m;
        *(uint4*)(y + (size_t)pix * ch.ld[st] + (i & (nv - 1)) * V) = pool_value<T>(m);
      }
      __syncthreads();
    }
  }
}

// mode 0: nearest 2x upsample (y is 2H x 2W); mode 1: plain copy (y is H x W)
template <typename T, int V, int MODE>
__global__ void copy_kernel(const PoolArgs a) {
  const int cv = a.C / V;
  const int Ho = MODE == 0 ? 2 * a.H : a.H, Wo = MODE == 0 ? 2 * a.W : a.W;
  const long long total = (long long)dyn_items(a.n_dyn, a.n) * Ho * Wo * cv;
  const T* x = (const T*)a.x;
  T* y = (T*)a.y;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    int c = (int)(i % cv) * V;
    long long pix = i / cv;
    int wo = (int)(pix % Wo);
    long long t = pix / Wo;
    int ho = (int)(t % Ho);
    long long img = t / Ho;
    int hi = MODE == 0 ? ho >> 1 : ho, wi = MODE == 0 ? wo >> 1 : wo;
    const T* p = x + ((size_t)(img * a.H + hi) * a.W + wi) * a.x_ld + a.x_coff + c;
    T* q = y + (size_t)pix * a.y_ld + a.y_coff + c;
    if (V > 1) *(uint4*)q = *(const uint4*)p; else *q = *p;
  }
}

template <typename T>
__global__ void add_kernel(const AddArgs a) {
  const long long total = (long long)dyn_items(a.n_dyn, a.n) * a.H * a.W * a.C;
  const T* pa = (const T*)a.a;
  const T* pb = (const T*)a.b;
  T* y = (T*)a.y;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    int c = (int)(i % a.C);
    long long pix = i / a.C;
    float v = (float)pa[(size_t)pix * a.a_ld + a.a_coff + c] + (float)pb[(size_t)pix * a.b_ld + a.b_coff + c];
    if (a.act == OCTO_ACT_RELU) v = fmaxf(v, 0.0f);
    else if (a.act == OCTO_ACT_SILU) v = v / (1.0f + __expf(-v));
    y[(size_t)pix * a.y_ld + a.y_coff + c] = (T)v;
  }
}

// Global average pool, one workgroup per (item, 64 V channels): VL lanes take neighbouring 16-byte channel vectors of a
// pixel, the workgroup's 256 / VL lane groups every (256 / VL)-th pixel, and the groups' sums meet in LDS.  A thread per
// channel that walked all pixels alone was one chain of loads: 14 us for 11 items of 7 x 7 x 512 and 2.0 TB/s for 3617.
template <typename T, typename Out>
__device__ __forceinline__ void gap_chunk(const PoolArgs& a, int img, int chunk, int vl, float (*part)[16 / sizeof(T) + 1], Out&& out) {
  constexpr int V = 16 / (int)sizeof(T);
  const int cv = a.C / V, hw = a.H * a.W;
  const int lane = threadIdx.x & (vl - 1), group = threadIdx.x / vl, groups = 256 / vl, v = chunk * vl + lane;
  float s[V];
#pragma unroll
  for (int e = 0; e < V; ++e) s[e] = 0.0f;
  if (v < cv) {
    const T* p = (const T*)a.x + (size_t)img * hw * a.x_ld + a.x_coff + v * V;
#pragma unroll 4
    for (int j = group; j < hw; j += groups) {
      alignas(16) T q[V];
      *(uint4*)q = *(const uint4*)(p + (size_t)j * a.x_ld);
#pragma unroll
      for (int e = 0; e < V; ++e) s[e] += (float)q[e];
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) part[threadIdx.x][e] = s[e];
  __syncthreads();
  for (int o = threadIdx.x; o < vl * V; o += 256) {
    const int l = o / V, e = o - l * V, c = (chunk * vl + l) * V + e;
    if (c < a.C) {
      float t = 0.0f;
      for (int g = 0; g < groups; ++g) t += part[g * vl + l][e];
      out(c, (T)(t / (float)hw));
    }
  }
  __syncthreads();
}
template <typename T>
__global__ __launch_bounds__(256) void gap_kernel(const PoolArgs a, int vl) {
  constexpr int V = 16 / (int)sizeof(T);
  __shared__ float part[256][V + 1];
  const int items = dyn_items(a.n_dyn, a.n), chunks = (a.C / V + vl - 1) / vl;
  for (int u = blockIdx.x; u < items * chunks; u += gridDim.x) {
    const int img = u / chunks;
    gap_chunk<T>(a, img, u - img * chunks, vl, part, [&](int c, T m) { ((T*)a.y)[(size_t)img * a.y_ld + a.y_coff + c] = m; });
  }
}
// channel counts or pitches that are no whole vectors: one thread per (item, channel)
template <typename T>
__global__ void gap_scalar_kernel(const PoolArgs a) {
  const long long total = (long long)dyn_items(a.n_dyn, a.n) * a.C;
  const T* x = (const T*)a.x;
  T* y = (T*)a.y;
  const int hw = a.H * a.W;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    int c = (int)(i % a.C);
    long long img = i / a.C;
    const T* p = x + (size_t)img * hw * a.x_ld + a.x_coff + c;
    float s = 0.0f;
    for (int j = 0; j < hw; ++j) s += (float)p[(size_t)j * a.x_ld];
    y[(size_t)img * a.y_ld + a.y_coff + c] = (T)(s / (float)hw);
  }
}

// Index of the largest of a row's values for a wavefront; ties resolve to the lowest index, 0 if there is no number.  Eight loads per lane
// are in flight at a time.
__device__ __forceinline__ int wave_argmax(const float* row, int n_out, int lane) {
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int j0 = lane; j0 < n_out; j0 += 512) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = j0 + 64 * q < n_out ? row[j0 + 64 * q] : -INFINITY;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (j0 + 64 * q < n_out && (v[q] > best || (v[q] == best && j0 + 64 * q < bi))) { best = v[q]; bi = j0 + 64 * q; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    float ob = __shfl_xor(best, off);
    int oi = __shfl_xor(bi, off);
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  }
  return bi == 0x7fffffff ? 0 : bi;
}
// The label of a row; with d.boxes it is also written to the result record of the box the row was cropped from.
__device__ __forceinline__ void put_label(int* labels, const LabelDest& d, int r, int label) {
  labels[r] = label;
  if (d.boxes) d.boxes[(size_t)d.rois[r].frame * d.max_det + d.rois[r].rank].child_label[d.slot] = label;
}
// one wavefront per row
__global__ __launch_bounds__(256) void argmax_kernel(const float* logits, int ld, int n_out, const int* n_dyn, int n, int* labels, const LabelDest d) {
  const int rows = dyn_items(n_dyn, n);
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int n_waves = (gridDim.x * blockDim.x) >> 6;
  for (int r = wave; r < rows; r += n_waves) {
    const int label = wave_argmax(logits + (size_t)r * ld, n_out, lane);
    if (lane == 0) put_label(labels, d, r, label);
  }
}

// The end of a classifier - global average pool, fully connected layer, label - with a workgroup per item, which keeps the means in LDS and
// reads the whole weight matrix: three launches of a chain in one.  The means are rounded to the tensor's type as the pool kernel does; a logit
// is summed in fp32, 64 lanes' parts and then their sum.  Bound by latency, for many items by reading the map.  Measured in us with a copy of
// the input, separate : fused, 16-bit: 64 channels to 10 outputs 13.2 : 7.6 for 2 items, 19.0 : 18.0 for 2048; 512 channels to 16 outputs
// (16 KB of weights) 15.5 : 10.6 and 54.9 : 53.3; to 32 15.2 : 11.7 and 54.9 : 56.9; to 128 16.0 : 18.6; 2048 channels to 8 15.8 : 20.6 (a workgroup
// takes them in four turns).  Hence the lines: one turn of 64 channel vectors, 16 KB.
constexpr int CLASSIFY_W_BYTES = 16 * 1024, CLASSIFY_OUT = CLASSIFY_W_BYTES / 128;       // (rows are padded to 128 bytes)
template <typename T>
__global__ __launch_bounds__(256) void classify_kernel(const ClassifyArgs a, int vl) {
  constexpr int V = 16 / (int)sizeof(T), OUTS = 4;     // outputs that a wavefront sums at a time
  __shared__ float part[256][V + 1];
  __shared__ __attribute__((aligned(16))) float mean[64 * V];
  __shared__ float logit[CLASSIFY_OUT];
  const PoolArgs& g = a.pool;
  const int items = dyn_items(g.n_dyn, g.n);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int img = blockIdx.x; img < items; img += gridDim.x) {
    gap_chunk<T>(g, img, 0, vl, part, [&](int c, T m) { ((T*)g.y)[(size_t)img * g.y_ld + g.y_coff + c] = m; mean[c] = (float)m; });
    for (int o0 = wave * OUTS; o0 < a.n_out; o0 += 4 * OUTS) {
      float s[OUTS];
#pragma unroll
      for (int q = 0; q < OUTS; ++q) s[q] = 0.0f;
      if (const int k = lane * V; k < g.C) {
        alignas(16) T w[OUTS][V];
#pragma unroll
        for (int q = 0; q < OUTS; ++q)       // (an output past the last one repeats it)
          *(uint4*)w[q] = *(const uint4*)((const T*)a.w + (size_t)(o0 + q < a.n_out ? o0 + q : a.n_out - 1) * a.kp + k);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const float m = mean[k + e];
#pragma unroll
          for (int q = 0; q < OUTS; ++q) s[q] = fmaf((float)w[q][e], m, s[q]);
        }
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int q = 0; q < OUTS; ++q) s[q] += __shfl_xor(s[q], off);
#pragma unroll
      for (int q = 0; q < OUTS; ++q)
        if (lane == q && o0 + q < a.n_out) {
          const float v = s[q] + a.bias[o0 + q];
          logit[o0 + q] = v;
          a.logits[(size_t)img * a.ld + o0 + q] = v;
        }
    }
    __syncthreads();
    if (wave == 0) {
      const int label = wave_argmax(logit, a.n_out, lane);
      if (lane == 0) put_label(a.labels, a.dest, img, label);
    }
    __syncthreads();                         // the logits have been read
  }
}

__global__ void fill_i32_kernel(int* p, int value, int count) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) p[i] = value;
}

template <typename T> static bool vec_ok(const void* x, int x_ld, int x_coff, const void* y, int y_ld, int y_coff, int C) {
  constexpr int V = 16 / sizeof(T);
  return C % V == 0 && x_ld % V == 0 && x_coff % V == 0 && y_ld % V == 0 && y_coff % V == 0 &&
         ((uintptr_t)x & 15) == 0 && ((uintptr_t)y & 15) == 0;
}

template <typename T> static hipError_t maxpool_t(const PoolArgs& a, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  if (vec_ok<T>(a.x, a.x_ld, a.x_coff, a.y, a.y_ld, a.y_coff, a.C)) {
    // Stride-1 "same" pools with enough columns to give every SIMD a wavefront: the row-walking kernel.  (With fewer
    // its serial walk down the rows is slower than the general kernel's k x k loads per output: 8 x 20 x 20 x 256 took
    // 25 us against 14.)  Row segments: several windows long, since each re-reads k - 1 rows.
    const long long columns = (long long)a.n * a.W * (a.C / V);
    long long n_seg = (262144 + columns - 1) / columns;
    if (n_seg > a.H / (2 * a.k)) n_seg = a.H / (2 * a.k);
    if (n_seg < 1) n_seg = 1;
    if (a.stride == 1 && (a.k == 5 || a.k == 3) && a.pad == a.k / 2 && a.Ho == a.H && a.Wo == a.W && a.H >= 2 * a.k && columns * n_seg >= 65536) {
      const int seg_rows = (int)((a.H + n_seg - 1) / n_seg);
      n_seg = (a.H + seg_rows - 1) / seg_rows;
      const unsigned grid = grid_for(columns * n_seg, 256);
      if (a.k == 5) hipLaunchKernelGGL((maxpool_rows_kernel<T, 5>), dim3(grid), dim3(256), 0, s, a, seg_rows, (int)n_seg);
      else hipLaunchKernelGGL((maxpool_rows_kernel<T, 3>), dim3(grid), dim3(256), 0, s, a, seg_rows, (int)n_seg);
      return hipGetLastError();
    }
    long long work = (long long)a.n * a.Ho * a.Wo * (a.C / V);
    hipLaunchKernelGGL((maxpool_kernel<T, V>), dim3(grid_for(work, 256)), dim3(256), 0, s, a);
  } else {
    long long work = (long long)a.n * a.Ho * a.Wo * a.C;
    hipLaunchKernelGGL((maxpool_kernel<T, 1>), dim3(grid_for(work, 256)), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}
template <typename T> static hipError_t maxpool_chain_t(const PoolArgs& a, const PoolChain& ch, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  for (int st = 0; st < 3; ++st)
    if (!vec_ok<T>(a.x, a.x_ld, a.x_coff, ch.y[st], ch.ld[st], ch.coff[st], a.C)) return hipErrorNotSupported;
  // as many channel vectors per workgroup as keep two maps within 52 KB (three workgroups per compute unit), so that a
  // workgroup reads 64 contiguous bytes of a pixel where the map is small and there are workgroups enough
  // (8 workgroups on one 20 x 20 x 256 map: 22 us)
  int nv = 4;
  while (nv > 1 && (a.C / V % nv || (long long)a.H * a.W * nv * 32 > 52 * 1024 || (long long)a.n * (a.C / V / nv) < 512)) nv /= 2;
  const long long lds = (long long)a.H * a.W * nv * 32;
  if (lds > 64 * 1024 || (long long)a.n * (a.C / V) >= 0x7FFFFFF0LL) return hipErrorNotSupported;
  const long long units = ((long long)a.n * (a.C / V / nv) + 7) / 8 * 8;
  hipLaunchKernelGGL((maxpool_chain_kernel<T>), dim3((unsigned)(units < 256 * 4 ? units : 256 * 4)), dim3(512), (unsigned)lds, s, a, ch, nv == 4 ? 2 : nv == 2 ? 1 : 0, make_fastdiv((unsigned)a.W));
  return hipGetLastError();
}
template <typename T, int MODE> static hipError_t copy_t(const PoolArgs& a, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  const int mul = MODE == 0 ? 4 : 1;
  if (vec_ok<T>(a.x, a.x_ld, a.x_coff, a.y, a.y_ld, a.y_coff, a.C)) {
    long long work = (long long)a.n * a.H * a.W * mul * (a.C / V);
    hipLaunchKernelGGL((copy_kernel<T, V, MODE>), dim3(grid_for(work, 256)), dim3(256), 0, s, a);
  } else {
    long long work = (long long)a.n * a.H * a.W * mul * a.C;
    hipLaunchKernelGGL((copy_kernel<T, 1, MODE>), dim3(grid_for(work, 256)), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

#define DISPATCH_T(dtype, EXPR_F32, EXPR_F16, EXPR_BF16) \
  switch (dtype) { case OCTO_F32: return EXPR_F32; case OCTO_F16: return EXPR_F16; case OCTO_BF16: return EXPR_BF16; } \
  return hipErrorInvalidValue;

hipError_t launch_maxpool(int dtype, const PoolArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, maxpool_t<float>(a, s), maxpool_t<_Float16>(a, s), maxpool_t<__bf16>(a, s))
}
hipError_t launch_maxpool_chain(int dtype, const PoolArgs& a, const PoolChain& ch, hipStream_t s) {
  DISPATCH_T(dtype, maxpool_chain_t<float>(a, ch, s), maxpool_chain_t<_Float16>(a, ch, s), maxpool_chain_t<__bf16>(a, ch, s))
}
hipError_t launch_upsample2x(int dtype, const PoolArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, (copy_t<float, 0>(a, s)), (copy_t<_Float16, 0>(a, s)), (copy_t<__bf16, 0>(a, s)))
}
hipError_t launch_copy_channels(int dtype, const PoolArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, (copy_t<float, 1>(a, s)), (copy_t<_Float16, 1>(a, s)), (copy_t<__bf16, 1>(a, s)))
}
template <typename T> static hipError_t add_t(const AddArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((add_kernel<T>), dim3(grid_for((long long)a.n * a.H * a.W * a.C, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_add(int dtype, const AddArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, add_t<float>(a, s), add_t<_Float16>(a, s), add_t<__bf16>(a, s))
}
// lanes over channel vectors in a workgroup of the pool kernel; 0: no whole vectors
template <typename T> static int gap_lanes(const PoolArgs& a) {
  constexpr int V = 16 / sizeof(T);
  if (a.C % V != 0 || a.x_ld % V != 0 || a.x_coff % V != 0 || ((uintptr_t)a.x & 15) != 0) return 0;
  int vl = 4;
  while (vl < 64 && vl < a.C / V) vl *= 2;
  return vl;
}
template <typename T> static hipError_t gap_t(const PoolArgs& a, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  if (const int vl = gap_lanes<T>(a)) {
    const long long units = (long long)a.n * ((a.C / V + vl - 1) / vl);
    if (units < 0x7FFFFFFFLL) {
      hipLaunchKernelGGL((gap_kernel<T>), dim3((unsigned)(units < 256 * 8 ? units : 256 * 8)), dim3(256), 0, s, a, vl);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((gap_scalar_kernel<T>), dim3(grid_for((long long)a.n * a.C, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_gap(int dtype, const PoolArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, gap_t<float>(a, s), gap_t<_Float16>(a, s), gap_t<__bf16>(a, s))
}
template <typename T> static hipError_t classify_t(const ClassifyArgs& a, hipStream_t s) {
  const int vl = gap_lanes<T>(a.pool);
  if (!vl || a.pool.C > 1024 / (int)sizeof(T) || a.n_out < 1 || a.n_out > CLASSIFY_OUT || (long long)a.n_out * a.kp * (int)sizeof(T) > CLASSIFY_W_BYTES ||
      a.kp < a.pool.C || a.kp * sizeof(T) % 16 != 0 || ((uintptr_t)a.w & 15) != 0)
    return hipErrorNotSupported;
  if (a.pool.n <= 0) return hipSuccess;
  hipLaunchKernelGGL((classify_kernel<T>), dim3((unsigned)(a.pool.n < 256 * 8 ? a.pool.n : 256 * 8)), dim3(256), 0, s, a, vl);
  return hipGetLastError();
}
hipError_t launch_classify(int dtype, const ClassifyArgs& a, hipStream_t s) {
  DISPATCH_T(dtype, classify_t<float>(a, s), classify_t<_Float16>(a, s), classify_t<__bf16>(a, s))
}
hipError_t launch_argmax(const float* logits, int ld, int n_out, const int* n_dyn, int n, int* labels, const LabelDest& d, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(argmax_kernel, dim3(grid_for((long long)n * 64, 256)), dim3(256), 0, s, logits, ld, n_out, n_dyn, n, labels, d);
  return hipGetLastError();
}
hipError_t launch_fill_i32(int* p, int value, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(count, 256)), dim3(256), 0, s, p, value, count);
  return hipGetLastError();
}

}  // namespace octo
