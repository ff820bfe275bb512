// Internal declarations shared by the HIP translation units of libocto.
// Nothing here is part of the public C ABI (that is include/octo.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/octo.h"
#include "kernel_ids.h"

namespace octo {

// A view of an NHWC activation tensor.  `ld` is the element distance between two
// pixels and `coff` the first channel inside that pitch, so a tensor can be a
// channel slice of a wider (concatenation) buffer.
struct TensorView {
  void* ptr = nullptr;
  int h = 0, w = 0, c = 0;
  int ld = 0, coff = 0;
};

struct HeldPlan;
struct SmallGroup;
struct ConvKernelArgs {
  const void* x;
  const void* w;        // packed weights [cout_pad][kp]
  const float* bias;    // [cout]
  const void* res;      // optional residual (same h, w, cout as y)
  void* y;
  const int* n_dyn;     // optional: number of items actually present (device), clamped to n
  int n;                // item capacity
  int H, W, Cin, x_ld, x_coff;
  int Ho, Wo, Cout, y_ld, y_coff;
  int res_ld, res_coff;
  int kh, kw, stride_h, stride_w, pad_h, pad_w;
  int K, Kp;
  int w_rows;                     // rows of the packed weight matrix (cout padded to a multiple of 128)
  unsigned magic_howo, shift_howo, magic_wo, shift_wo; int HoWo_is_one;   // pixel index -> (image, row, column)
  unsigned magic_cin, magic_kw;   // floor(2^32 / d) + 1 for d = Cin, kw (set by launch_conv)
  int act, res_mode;
  int out_f32;          // write fp32 instead of the storage type
  int n_hint;           // host only: expected item count when it is taken on the device (0: assume n); picks the tile shape
  int n_split;          // host only: item count the choice between orders of summation is made for (0: n)
  int pair_view;        // the layer is a 3-channel first layer run on pixel pairs of a 4-channel-padded input
  // Fused 3x3 / stride-2 / pad-1 max-pool (first-layer kernel only): when pool_y is set, only the pooled tensor is
  // written and y is not touched; launch_conv returns hipErrorNotSupported if no kernel can do that for the layer.
  void* pool_y;
  int pool_ho, pool_wo, pool_ld, pool_coff;
  int stem_seg;                   // output rows per segment of a strip (set by launch_stem)
  // Two layers in one launch (general, flowing, split-K and streaming 1x1 kernels, 16-bit types, no residual): output channels below `split` go to y as
  // usual, channels split .. Cout - 1 to y2 as its channels 0 ..; split is a multiple of 8 and 0 when unused.
  void* y2;
  int y2_ld, y2_coff, split;
  // Nearest 2x upsampling of the output, written beside y (16-bit types, whole 16-byte vectors, no second output): pixel
  // (i, j) also goes to pixels (2 i .. 2 i + 1, 2 j .. 2 j + 1) of up_y.  Unused when null.
  void* up_y;
  int up_next;                    // host only: an upsampling of the output follows; the split-K kernel is chosen as if it were to write it
  int up_ld, up_coff;
  int in_place;                   // host only: one launch of many; its input was written by the launch before and comes from beyond the L2s
  // 8-bit floating point storage only: y = act(acc * scale[c] + bias[c] (+ res * res_scale)), stored as
  // E4M3(y * y_inv_scale) unless out_f32.  scale: device, one factor per output channel, padded like the bias.
  const float* scale;
  float res_scale, y_inv_scale;
};
// A launch: what the kernels above take, and what only the host reads.  Apart, so that a kernel's arguments are no longer than they need be: with the two pointers among them the short calls on
// kernels that take this struct were 0.15 - 0.4 us slower (E4M3 256 -> 200, 3x3 / stride 2 on 32 x 17 x 18 10.3 : 10.7, bf16 56 -> 56, 3x3 on 18 x 26 x 18 6.1 : 6.25).
struct ConvArgs : ConvKernelArgs {
  SmallGroup* group;              // conv_small_kernel's launch is collected here instead (conv_small_choice.h); null: launched
  const HeldPlan* held;           // what a model keeps for a 3x3 layer that may run on conv3x3_held_kernel (conv3x3_held_choice.h), or null
};

// element size of a storage type
inline __host__ __device__ int dtype_size(int dt) { return dt == OCTO_F32 ? 4 : (dt == OCTO_F8 ? 1 : 2); }

// ---- launchers (each enqueues on `s`, never synchronises) -------------------
// Optional pair of events attached to the convolution's own dispatch (start and end of the kernel on the device).
struct ConvTiming { hipEvent_t start = nullptr, stop = nullptr; };
hipError_t launch_conv(int dtype, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id = nullptr, ConvTiming tm = ConvTiming());
// first-layer kernel for pixel-pair layers; hipErrorNotSupported when the layer does not fit it
hipError_t launch_stem(int dtype, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm);
// 1x1 layers of large maps with resident weights; hipErrorNotSupported when the layer does not fit it
hipError_t launch_conv1x1_stream(int dtype, const ConvArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm);
// The weights of a 3x3 layer, 16-bit types, from rows of kp values into the order that conv3x3_held_kernel reads them (held_weight_bytes, conv3x3_held_choice.h)
hipError_t launch_held_pack(const void* w, int kp, int cin, int cout, void* out, hipStream_t s);
// The first layers of a detector in one launch (16-bit types, SiLU): 3 -> 32, 6x6 / stride 2 / pad 2 on the pixel-pair view; 32 -> 64, 3x3 / stride 2 / pad 1; two 1x1
// layers 64 -> 32 whose weights are stacked.  w, bias, kp: of those three.  hipErrorNotSupported when a tensor does not fit.
struct EntryArgs {
  const void* x; int n, H, W;
  const void* w[3]; const float* bias[3]; int kp[3];
  void* y[2]; int y_ld[2], y_coff[2];
};
hipError_t launch_entry(int dtype, const EntryArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm);
// A cross-stage block of 32 channels behind its entry convolutions in one launch (16-bit types, SiLU): 1x1 32 -> 32 of x, 3x3 / pad 1 32 -> 32 of that (plus x with a
// shortcut), 1x1 64 -> 64 of the concatenation of that and z.  w, bias, kp: of those three.  hipErrorNotSupported when a tensor does not fit.
struct BlockArgs {
  const void* x; int x_ld, x_coff;
  const void* z; int z_ld, z_coff;
  void* y; int y_ld, y_coff;
  int n, H, W, shortcut;
  const void* w[3]; const float* bias[3]; int kp[3];
};
// The two entry 1x1 layers of a cross-stage block (a, b; weights stacked) and a 1x1 layer on the first one's output (h), SiLU; a.a may be null: not written.
struct LeadArgs {
  const void* x; int x_ld, x_coff;
  void* a; int a_ld, a_coff;
  void* b; int b_ld, b_coff;
  void* h; int h_ld, h_coff;
  long long pixels; int Cin, C;
  const void* w[2]; const float* bias[2]; int kp[2];
};
bool lead_fits(int c, int cin);
hipError_t launch_lead(int dtype, const LeadArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm);
hipError_t launch_block(int dtype, const BlockArgs& a, int num_cu, hipStream_t s, int* kernel_id, ConvTiming tm);
enum { KID_NONE = 0, KID_MAXPOOL = 1, KID_UPSAMPLE = 2, KID_COPY = 3, KID_ADD = 4, KID_GAP = 5 };
size_t conv_packed_weight_elems(int cout, int kh, int kw, int cin, int dtype, int* kp_out, int* cout_pad_out);

struct PoolArgs {
  const void* x; void* y; const int* n_dyn; int n;
  int H, W, C, x_ld, x_coff, Ho, Wo, y_ld, y_coff, k, stride, pad;
};
hipError_t launch_maxpool(int dtype, const PoolArgs& a, hipStream_t s);
// Three chained stride-1 "same" pools (window a.k) of a.x, every stage's result written; a.y is not used.
// hipErrorNotSupported when the map does not fit LDS or a tensor is not in whole 16-byte vectors.
struct PoolChain { void* y[3]; int ld[3], coff[3]; };
hipError_t launch_maxpool_chain(int dtype, const PoolArgs& a, const PoolChain& ch, hipStream_t s);
hipError_t launch_upsample2x(int dtype, const PoolArgs& a, hipStream_t s);       // uses H, W, C, lds/coffs
hipError_t launch_copy_channels(int dtype, const PoolArgs& a, hipStream_t s);    // y[:, :, :, coff:coff+C] = x
struct AddArgs {
  const void* a; const void* b; void* y; const int* n_dyn; int n;
  int H, W, C, a_ld, a_coff, b_ld, b_coff, y_ld, y_coff, act;
};
hipError_t launch_add(int dtype, const AddArgs& a, hipStream_t s);
hipError_t launch_gap(int dtype, const PoolArgs& a, hipStream_t s);              // y [n][C] mean over H*W
// Where the labels of a child's items go besides its own label array: child_label[slot] of the box that item r was cropped
// from (rois[r]: frame, rank).  boxes == nullptr: nowhere.
struct LabelDest { octo_box* boxes = nullptr; const octo_roi* rois = nullptr; int max_det = 0, slot = 0; };
// Global average pool, fully connected layer without activation and label in one launch; every tensor is written.  kp: values per row of w.
// hipErrorNotSupported: the matrix is too large for a workgroup per item, or the pool's input is not in whole 16-byte vectors.
struct ClassifyArgs { PoolArgs pool; const void* w; const float* bias; int kp, n_out; float* logits; int ld; int* labels; LabelDest dest; };
hipError_t launch_classify(int dtype, const ClassifyArgs& a, hipStream_t s);
hipError_t launch_argmax(const float* logits, int ld, int n_out, const int* n_dyn, int n, int* labels, const LabelDest& d, hipStream_t s);
hipError_t launch_fill_i32(int* p, int value, int count, hipStream_t s);

// floor(n / d) for n < 2^31 by multiply-high and shift; built on the host
struct FastDiv { unsigned mul, shift; int is_one; };
inline FastDiv make_fastdiv(unsigned d) {
  FastDiv f{0u, 0u, d <= 1u ? 1 : 0};
  if (f.is_one) return f;
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  const unsigned long long m = ((1ull << (32 + s)) + d - 1) / d;
  if (m >> 32) { f.mul = (unsigned)(((1ull << (31 + s)) + d - 1) / d); f.shift = s - 1; }
  else { f.mul = (unsigned)m; f.shift = s; }
  return f;
}
#ifdef __HIPCC__
__device__ __forceinline__ unsigned fast_div(unsigned n, const FastDiv& f) { return f.is_one ? n : __umulhi(n, f.mul) >> f.shift; }
#endif

// First launch of a batch: the frame table (passed by value, at most MAX frames per launch) and cleared counters.
struct BeginArgs {
  static constexpr int MAX = 64, REGIONS = 4;
  const uint8_t* ptr[MAX]; size_t pitch[MAX];
  int n;                                   // frames of this launch
  const uint8_t** d_ptr; size_t* d_pitch;
  int* clear[REGIONS]; int clear_count[REGIONS];      // ranges of ints to zero (nullptr / 0: unused)
};
#ifdef __HIPCC__
__device__ __forceinline__ void begin_batch(const BeginArgs& a, int i0, int step) {      // thread i0 of step
  if (i0 < a.n) { a.d_ptr[i0] = a.ptr[i0]; a.d_pitch[i0] = a.pitch[i0]; }
#pragma unroll
  for (int r = 0; r < BeginArgs::REGIONS; ++r)
    for (int i = i0; i < a.clear_count[r]; i += step) a.clear[r][i] = 0;
}
#endif

struct ResizeArgs {
  const uint8_t* const* frames;   // device table of frame base pointers
  const size_t* pitches;          // device table of row pitches in bytes
  int src_h, src_w;
  void* dst; int dst_h, dst_w;
  int dst_c;                      // 3, or 4: a zero fourth channel so that two neighbouring pixels form one 16-byte vector
  float scale[3], bias[3];
  int pad_value;
  int n; const int* n_dyn;
  // crop mode only
  const octo_roi* rois;
  int n_frames;                   // frames behind `frames` (ROI frame indices are clamped to it)
  FastDiv div_wq, div_h;          // set by the launchers: lanes per output row, rows per item
};
void letterbox_geometry(int src_h, int src_w, int dst_h, int dst_w, int* nw, int* nh, int* left, int* top);
hipError_t launch_letterbox(int dtype, const ResizeArgs& a, int num_cu, hipStream_t s, const BeginArgs* begin = nullptr);      // begin: the launch does that too
hipError_t launch_crop_resize(int dtype, const ResizeArgs& a, hipStream_t s);

struct DecodeArgs {
  const void* head[3]; int head_ld[3];
  int n_levels; int gh[3], gw[3], stride[3]; float anchors[3][3][2];
  int n_anchors, n_classes; float score_thr;
  int n; const int* n_dyn;
  octo_cand* cand; int* count; int cap;      // per item: cand[item*cap ...], count[item*count_stride]
  int count_stride;                          // >= 1; 32 puts every item's counter on its own 128-byte line
  int* overflow;
};
hipError_t launch_decode(int dtype, const DecodeArgs& a, hipStream_t s);

struct TopkArgs {
  const octo_cand* in; const int* in_count; int in_cap;
  int in_count_stride;
  octo_cand* out; int* out_count; int k;     // out stride = k_cap
  int k_cap;
  int n; const int* n_dyn;
};
hipError_t launch_topk(const TopkArgs& a, hipStream_t s);

struct NmsArgs {
  const octo_cand* top; const int* top_count; int k_cap;     // k_cap multiple of 64
  float iou_thr; int max_det;
  unsigned long long* mask;                                  // [n][k_cap][k_cap/64]
  int* keep; int* n_keep;                                    // keep[item*max_det ...]
  int n; const int* n_dyn;
  LabelDest dest;                                            // child detectors: the number of kept boxes is the item's label
};
hipError_t launch_nms(const NmsArgs& a, hipStream_t s);
size_t nms_mask_bytes(int n, int k_cap);

struct CompactArgs {
  const octo_cand* top; int k_cap;
  const int* keep; const int* n_keep; int max_det;
  int n; const int* n_dyn;
  // geometry of the letterbox that produced the boxes (identity for child detectors)
  float left, top_pad, rx, ry, src_w, src_h;
  int n_edges; uint64_t class_mask[OCTO_MAX_EDGES][2];
  octo_roi* rois[OCTO_MAX_EDGES]; int* n_roi[OCTO_MAX_EDGES]; int roi_cap[OCTO_MAX_EDGES];
  int* roi_of[OCTO_MAX_EDGES];             // [n][max_det] -> roi id or -1 (required)
  int* roi_cnt[OCTO_MAX_EDGES];            // [n] scratch: ROIs per item (required)
  octo_box* boxes;                         // [n][max_det] final boxes in source pixels
  int* flags;                              // [n]
  int dense;                               // step 1 on its own: roi_of past an item's last kept box becomes -1 (else it is left alone)
};
hipError_t launch_compact(const CompactArgs& a, hipStream_t s, bool counted = false);     // counted: step 1 has run (launch_select)
// Top-k, NMS and (with ca) step 1 of the compaction in one launch; m.mask is not used.
constexpr int SELECT_MAX = 1024;           // boxes per item, at most
bool select_fits(const TopkArgs& a);
hipError_t launch_select(const TopkArgs& a, const NmsArgs& m, const CompactArgs* ca, hipStream_t s);

hipError_t launch_begin(const BeginArgs& a, hipStream_t s);

// Last launch of a batch: the result block's header and the boxes in use go straight to pinned host memory.
struct PublishArgs {
  const char* src; char* dst;              // result block on the device, its mirror in host memory
  int header_bytes;                        // counters in front of the boxes (a multiple of 16)
  const int* n_keep; int max_det; int n;
  unsigned* done; unsigned number;         // host memory: the number of the batch is written there
};
hipError_t launch_publish(const PublishArgs& a, hipStream_t s);

// ---- host-side scheduling (no GPU) ------------------------------------------
int cwd_search(octo_sched_pipeline* p);
int coral_schedule(octo_sched_pipeline* ps, int n_pipelines, double mem, double util_max, int n_streams,
                   octo_placement* out);

}  // namespace octo
