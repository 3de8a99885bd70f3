// Host side of the C ABI declared in include/evconv.h: description checking, workspace
// layout, weight re-layout, and the per-step launch sequence.  No computation of the method
// happens on the host; every step of the path is a kernel launch on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/evconv.h"
#include "evconv_kernels.h"

using namespace evk;

namespace {

thread_local std::string g_create_error;

// Workspace of evconv_create_static: one array per GPU, part of the loaded code object, so a net
// built in it needs no device allocation by anybody.  In host code the array's name is only a
// handle for hipGetSymbolAddress; the device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[EVCONV_STATIC_WORKSPACE_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
void* g_scratch_ptr[kMaxDevices] = {};       // device address of `scratch` on each device
evconv_net* g_static_owner[kMaxDevices] = {};  // the live net that occupies it, if any

enum KernelKind { kKernConvValu = 0, kKernConvMfmaF32, kKernElementwise, kKernGap, kKernPool, kKernConvMfmaBf16,
                  kKernConvNarrow, kKernConvMfmaSplit, kKernConvPointwise, kKernDelay };
const char* const kKernelNames[] = {"conv_valu_f32", "conv_mfma_f32", "elementwise", "global_avgpool",
                                    "maxpool", "conv_mfma_bf16", "conv_narrow_mfma_f32", "conv_mfma_f32_split_bf16x3", "conv_pointwise_f32",
                                    "delay"};

// fp32 -> bf16 bits, round to nearest even
uint16_t to_bf16(float x) {
  uint32_t u;
  memcpy(&u, &x, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Eight weights, each as the sum of `parts` bf16 values (matrix-core kernels): a part is the
// rounding of what the ones before it leave, so three of them hold an fp32 value exactly; part q
// of the eight goes to at[q * plane ..].  Three parts are for finite values only: one that would
// round to an infinite bf16 is cut off instead.  (Loops without branches: a net has millions of
// weights and this is most of the time that create takes.)
void weight_parts8(const float* v, int parts, uint16_t* at, size_t plane) {
  float rest[8];
  memcpy(rest, v, sizeof rest);
  for (int q = 0; q < parts; ++q) {
    uint16_t h[8];
    for (int e = 0; e < 8; ++e) {
      uint32_t u;
      memcpy(&u, &rest[e], 4);
      uint32_t b = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
      b = (u & 0x7fffffffu) > 0x7f800000u ? 0x7fc0u : b;
      b -= parts == 3 && (b & 0x7fffu) == 0x7f80u ? 1u : 0u;
      h[e] = (uint16_t)b;
      const uint32_t back = b << 16;
      float f;
      memcpy(&f, &back, 4);
      rest[e] -= f;
    }
    memcpy(at + q * plane, h, sizeof h);
  }
}
// Power of two that a conv's fp32 weights are multiplied with so that three bf16 parts hold them: a bf16
// has no bits below 2^-133, and weights of less than about 2^-110 have bits there (those below 2^-134
// would even become zero, and an infinite increment times them NaN).  With 2^16 every one of them
// is exact; the sums are then finite up to 2^112 instead of 2^128, so weights that do not need it are
// taken as they are, with one exception: the high parts of two operands may be up to 2^-8 larger
// than the operands, so a product just below the largest fp32 value would overflow on its way.  It
// needs a weight of nearly 1 or more; such weights are halved (exactly, if no weight has a bit at
// 2^-133).  `fits` becomes false for weights that are not finite or lie too far apart: those go to
// the vector kernel.
constexpr int kTinyWeightExponent = 16;
constexpr uint32_t kHalvedFrom = 0x3f7d70a4u;  // 0.99: below it a weight's high part is 0.9922 at most, an increment's 3.39e38: 3.37e38
float weight_scale(const float* w, size_t n, bool* fits) {
  uint32_t special = 0, small = 0, largest = 0;
  for (size_t i = 0; i < n; ++i) {
    uint32_t u;
    memcpy(&u, &w[i], 4);
    u &= 0x7fffffffu;
    special |= u >= 0x7f800000u ? 1u : 0u;
    small |= u - 1u < (18u << 23) - 1u ? 1u : 0u;  // nonzero, below 2^-109
    largest = std::max(largest, u);
  }
  *fits = !special;
  const float scale = largest >= kHalvedFrom ? 0.5f : 1.0f;
  if (special || !small) return scale;
  bool exact = true;
  for (size_t i = 0; i < n && exact; ++i)
    if (fabsf(w[i]) < 0x1p-109f) {
      const float up = ldexpf(w[i], 133) * scale;  // its integer part is what a bf16 can hold
      exact = up == truncf(up);
    }
  if (exact) return scale;
  *fits = largest < (uint32_t)(127 + 112) << 23;
  return ldexpf(1.0f, kTinyWeightExponent);
}
int weight_part_count(int wdtype) { return wdtype == EVCONV_F32 ? 3 : wdtype == EVCONV_F32_SPLIT ? 2 : 1; }

// Whether a 5 x 5 conv (stride 1, padding 2) behind a bilinear x2 up-sampling of lo_h x lo_w stored sites has the
// up-sampling folded into its weights: where some 8 x 8 tile of stored sites lies wholly two sites or more away
// from the border (smaller maps, half of whose taps would be those of a border, keep the interpolating gather).
bool fold_pays(int lo_h, int lo_w) { return lo_h >= 18 && lo_w >= 18; }

struct NodePlan {
  evconv_node_desc d;
  Geo ga, gb, go;
  bool keeps_z = false, structural = false;
  int kernel = 0;
  int c_out_pad = 0;
  int tail_units = 0;       // ConvParams::tail_units
  float w_scale = 1.0f, w_fold_scale = 1.0f;  // fp32 matrix-core weights (and folded ones) are stored times these
  int fused_into = -1;      // ADD or SPARSIFY node executed in the epilogue of that conv node
  int fused_sp = -1;        // conv node: the SPARSIFY node it executes behind its last epilogue stage
  int n_fused = 0;          // conv node: ADD nodes it executes, in order
  int fused_nodes[kMaxFusedAdds] = {-1, -1};
  int head_batch = -1;      // prediction head: the head whose launch it runs in (the last one of its batch)
  int mates[kMaxConvBatch - 1] = {-1, -1, -1};  // conv node: later convs of the same input that run in its launch
  int n_mates = 0;
  bool mates_batch = false;  // ... as a batch of one variant (otherwise a shortcut conv)
  int paired_into = -1;      // such a later conv: the node whose launch it runs in
  int gather_fused_into = -1;  // UPSAMPLE node computed inside the gather of that conv node, never stored
  int upsampled_from = -2;     // conv node: the node (-1: network input) whose x2 up-sampling it reads through
                               // its gather, its in0 being the folded UPSAMPLE node; -2: none
  // conv node reading through an up-sampling that is folded into per-phase weights
  // (ConvParams::fold_list); room is reserved where fold_set_bytes says so
  bool folds = false;
  size_t off_w_fold = 0, off_fold_list = 0;
  void* w_fold = nullptr;
  int* fold_list = nullptr;
  // workspace offsets (bytes); resolved to pointers at create
  size_t off_step = 0;      // SPARSIFY: device scalar k
  size_t off_z2 = 0;        // MUL: accumulated second factor
  float* z2 = nullptr;
  size_t off_occ_saved = 0;  // DELAY: S_out words of the delayed node as the previous step left them
  uint64_t* occ_saved = nullptr;
  bool integrates = false;      // output node whose kernel keeps the public tensors itself
  bool saved_in_lists = false;  // DELAY: its words are copied by the compaction kernel
  float* step = nullptr;
  float step_fixed = -1.0f; // >= 0: k supplied by the description
  size_t off_z = 0, off_out = 0, off_pool = 0, off_occ = 0, off_touched = 0, off_idx = 0, off_count = 0,
         off_bitmap = 0, off_w = 0, off_bias = 0, off_y = 0, off_dy = 0;
  float *z = nullptr, *out = nullptr, *pool_in = nullptr, *bias = nullptr, *y = nullptr, *dy = nullptr;
  void* w = nullptr;
  uint64_t *occ = nullptr, *touched = nullptr, *bitmap = nullptr;
  int32_t *idx = nullptr, *count = nullptr;
};

struct Layout {
  std::vector<NodePlan> nodes;
  Geo gin;
  size_t off_x_prev = 0, off_dx = 0, off_occ_in = 0, off_idx_in = 0, off_count_in = 0, off_bitmap_in = 0;
  size_t off_occ_nodes = 0, n_occ_words = 0;  // contiguous occupancy region of all nodes
  size_t off_sets = 0, off_rms = 0, off_int = 0;
  size_t off_row_or = 0;  // scratch of the increment builder (wide inputs)
  size_t off_ks_part = 0, off_ks_count = 0;  // scratch of convs whose channels are split over workgroups
  size_t stride = 0;   // bytes of one stream's state; what several streams share (weights, descriptors) lies behind the last one
  int n_streams = 1;
  size_t total = 0;
  int max_ty = 0;
};

size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

struct Bump {
  size_t cur = 0;
  size_t take(size_t bytes) {
    size_t o = cur;
    cur = align_up(cur + bytes);
    return o;
  }
};

// Nodes that read each node.
std::vector<int> consumer_counts(const std::vector<NodePlan>& nodes) {
  std::vector<int> n(nodes.size(), 0);
  for (const NodePlan& x : nodes) {
    const evconv_node_desc& d = x.d;
    if (d.in0 >= 0) ++n[d.in0];
    const bool two = d.op == EVCONV_OP_ADD || d.op == EVCONV_OP_CONCAT || d.op == EVCONV_OP_MUL;
    if (two && d.in1 >= 0 && d.in1 != d.in0) ++n[d.in1];
  }
  return n;
}

// Bytes of the weight sets that hold the up-sampling in front of conv node n (four phases of taps, see prepare_fold, x
// input channels padded to 32); 0 where it is not folded: bf16-declared weights (they would be rounded a second
// time), maps on which it does not pay, sets in which the kernel's byte offsets do not fit 31 bits, an up-sampling that
// something else reads or applies to, flags.
size_t fold_set_bytes(const std::vector<NodePlan>& nodes, const std::vector<int>& consumers, const NodePlan& n, uint32_t flags, int n_streams) {
  const evconv_node_desc& d = n.d;
  if (d.op != EVCONV_OP_CONV2D || d.kh != 5 || d.stride != 1 || d.pad != 2 || d.in0 < 0 || d.wdtype == EVCONV_BF16) return 0;
  if (flags & (EVCONV_FLAG_NO_FUSION | EVCONV_FLAG_NO_FOLD | EVCONV_FLAG_FORCE_VALU)) return 0;
  const evconv_node_desc& u = nodes[d.in0].d;
  if (u.op != EVCONV_OP_UPSAMPLE_BILINEAR2X || u.act != EVCONV_ACT_NONE || u.is_output || consumers[d.in0] != 1) return 0;
  ConvParams probe = {};
  probe.gi = n.ga; probe.go = n.go; probe.k = d.kh; probe.stride = d.stride; probe.pad = d.pad; probe.c_out_pad = n.c_out_pad;
  probe.st = Streams{0, n_streams}; probe.fp32 = d.wdtype == EVCONV_F32;
  if (!conv_mfma_upsample_supported(probe) || !fold_pays(n.ga.h / 2, n.ga.w / 2)) return 0;
  const size_t phase = (size_t)kFoldVectors * kFoldVectors * ((d.c_in + 31) / 32 * 32) * n.c_out_pad * 2 * weight_part_count(d.wdtype);
  return phase < (size_t)1 << 31 ? 4 * phase : 0;
}

evconv_status fail(std::string* err, evconv_status st, const std::string& msg) {
  if (err) *err = msg;
  return st;
}

// Checks the description and lays the workspace out.  Pure host arithmetic.
evconv_status make_layout(const evconv_net_desc* desc, size_t weight_bytes, bool check_weights, Layout* L,
                          std::string* err) {
  if (!desc || !desc->nodes) return fail(err, EVCONV_ERR_INVALID_ARG, "null description");
  if (desc->abi_version != EVCONV_ABI_VERSION) return fail(err, EVCONV_ERR_BAD_DESC, "abi_version mismatch");
  if (desc->n_nodes <= 0) return fail(err, EVCONV_ERR_BAD_DESC, "n_nodes must be positive");
  if (desc->in_c <= 0 || desc->in_h <= 0 || desc->in_w <= 0) return fail(err, EVCONV_ERR_SHAPE, "bad input shape");
  if (desc->flags & ~(EVCONV_FLAG_NO_FUSION | EVCONV_FLAG_NO_FOLD | EVCONV_FLAG_FORCE_VALU))
    return fail(err, EVCONV_ERR_INVALID_ARG, "unknown bits in flags");
  if (!(desc->sparsify_tp >= 0.0f)) return fail(err, EVCONV_ERR_INVALID_ARG, "sparsify_tp must be >= 0");
  if (desc->n_streams < 0 || desc->n_streams > 256) return fail(err, EVCONV_ERR_INVALID_ARG, "n_streams must be in [0, 256]");
  if ((long long)desc->in_h * desc->in_w > (1ll << 30)) return fail(err, EVCONV_ERR_SHAPE, "input too large");

  L->gin = make_geo(desc->in_c, desc->in_h, desc->in_w);
  L->nodes.resize(desc->n_nodes);
  L->max_ty = L->gin.ty;
  Bump b;
  // occupancy words of all nodes first, contiguous: cleared in one sweep at the start of a step
  L->off_occ_nodes = b.cur;
  std::vector<size_t> occ_word_off(desc->n_nodes);
  size_t words = 0;
  for (int i = 0; i < desc->n_nodes; ++i) {
    const evconv_node_desc& d = desc->nodes[i];
    NodePlan& n = L->nodes[i];
    n.d = d;
    char where[64];
    snprintf(where, sizeof where, "node %d: ", i);
    if (d.op < 0 || d.op > EVCONV_OP_DELAY) return fail(err, EVCONV_ERR_INVALID_ARG, std::string(where) + "bad op");
    if (d.act < 0 || d.act > EVCONV_ACT_ONE_MINUS) return fail(err, EVCONV_ERR_INVALID_ARG, std::string(where) + "bad act");
    const bool delay = d.op == EVCONV_OP_DELAY;
    if (delay) {
      // in0: the later node whose previous-step value this is; in1: an earlier node of its size
      if (d.in0 <= i || d.in0 >= desc->n_nodes) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "DELAY: in0 must be a later node");
      if (d.in1 < -1 || d.in1 >= i) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "DELAY: in1 is not an earlier node");
      if (d.act != EVCONV_ACT_NONE) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "DELAY takes no activation");
      if (d.c_out <= 0) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "c_out must be positive");
    } else if (d.in0 < -1 || d.in0 >= i) {
      return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "in0 is not an earlier node");
    }
    const bool two = d.op == EVCONV_OP_ADD || d.op == EVCONV_OP_CONCAT || d.op == EVCONV_OP_MUL;
    if (two && (d.in1 < -1 || d.in1 >= i)) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "in1 is not an earlier node");
    if (!two && !delay) n.d.in1 = -1;  // (ignored, and not an index: the description may hold anything there)
    if (delay) {
      n.ga = d.in1 < 0 ? L->gin : L->nodes[d.in1].go;
      n.ga = make_geo(d.c_out, n.ga.h, n.ga.w);
    } else {
      n.ga = d.in0 < 0 ? L->gin : L->nodes[d.in0].go;
    }
    n.gb = two ? (d.in1 < 0 ? L->gin : L->nodes[d.in1].go) : n.ga;
    int c = n.ga.c, h = n.ga.h, w = n.ga.w;
    switch (d.op) {
      case EVCONV_OP_CONV2D:
      case EVCONV_OP_LINEAR:
      case EVCONV_OP_MAXPOOL: {
        int k = d.kh, s = d.stride, pad = d.pad;
        if (d.op == EVCONV_OP_LINEAR) {
          if (h != 1 || w != 1) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "LINEAR needs a 1 x 1 input");
          k = 1; s = 1; pad = 0;
          n.d.kh = n.d.kw = 1; n.d.stride = 1; n.d.pad = 0;
        } else {
          if (d.kh != d.kw || k < 1 || k > 7) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "kernel must be square, 1..7");
          if (s < 1 || s > 2) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "stride must be 1 or 2");
          if (pad < 0 || pad >= k) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "pad must be in [0, k)");
        }
        if (d.op == EVCONV_OP_MAXPOOL) {
          if (d.act != EVCONV_ACT_NONE) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "MAXPOOL takes no activation");
        } else {
          if (d.c_in != c) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "c_in does not match the input node");
          if (d.c_out <= 0) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "c_out must be positive");
          if (d.wdtype != EVCONV_F32 && d.wdtype != EVCONV_BF16 && d.wdtype != EVCONV_F32_SPLIT) return fail(err, EVCONV_ERR_INVALID_ARG, std::string(where) + "bad wdtype");
          const size_t wb = (size_t)d.c_out * d.c_in * k * k * sizeof(float);
          if (d.weight_off < 0 || (d.weight_off & 3)) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "bad weight_off");
          if (check_weights && (size_t)d.weight_off + wb > weight_bytes) return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "weights out of range");
          if (d.bias_off >= 0 && ((d.bias_off & 3) || (check_weights && (size_t)d.bias_off + d.c_out * sizeof(float) > weight_bytes)))
            return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "bias out of range");
          c = d.c_out;
        }
        const int ho = (h + 2 * pad - k) / s + 1, wo = (w + 2 * pad - k) / s + 1;
        if (h + 2 * pad < k || w + 2 * pad < k || ho <= 0 || wo <= 0) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "empty output");
        h = ho; w = wo;
        break;
      }
      case EVCONV_OP_ADD:
        if (n.gb.c != c || n.gb.h != h || n.gb.w != w) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "ADD inputs differ in shape");
        break;
      case EVCONV_OP_MUL:
        if (n.gb.c != c || n.gb.h != h || n.gb.w != w) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "MUL inputs differ in shape");
        if (d.act != EVCONV_ACT_NONE) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "MUL takes no activation");
        break;
      case EVCONV_OP_CONCAT:
        if (n.gb.h != h || n.gb.w != w) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "CONCAT inputs differ in size");
        c += n.gb.c;
        break;
      case EVCONV_OP_UPSAMPLE_BILINEAR2X: h *= 2; w *= 2; break;
      case EVCONV_OP_GLOBAL_AVGPOOL: h = 1; w = 1; break;
      case EVCONV_OP_ACT: break;
      case EVCONV_OP_DELAY: break;  // shape of in1 with c_out channels; checked against in0 below
      case EVCONV_OP_SPARSIFY:
        if (d.act != EVCONV_ACT_NONE) return fail(err, EVCONV_ERR_UNSUPPORTED, std::string(where) + "SPARSIFY takes no activation");
        if (d.weight_off >= 0 && ((d.weight_off & 3) || (check_weights && (size_t)d.weight_off + 4 > weight_bytes)))
          return fail(err, EVCONV_ERR_BAD_DESC, std::string(where) + "step value out of range");
        break;
    }
    if ((long long)h * w > (1ll << 30)) return fail(err, EVCONV_ERR_SHAPE, std::string(where) + "output too large");
    n.go = make_geo(c, h, w);
    if (n.go.ty > L->max_ty) L->max_ty = n.go.ty;
    const bool lin = d.op == EVCONV_OP_CONV2D || d.op == EVCONV_OP_LINEAR;
    n.keeps_z = (lin || d.op == EVCONV_OP_GLOBAL_AVGPOOL || d.op == EVCONV_OP_ACT ||
                 d.op == EVCONV_OP_SPARSIFY || d.op == EVCONV_OP_MUL || d.op == EVCONV_OP_DELAY ||
                 d.act != EVCONV_ACT_NONE) &&
                d.op != EVCONV_OP_MAXPOOL;
    n.structural = (d.op == EVCONV_OP_ADD || d.op == EVCONV_OP_CONCAT || d.op == EVCONV_OP_UPSAMPLE_BILINEAR2X ||
                    d.op == EVCONV_OP_GLOBAL_AVGPOOL || d.op == EVCONV_OP_MUL || d.op == EVCONV_OP_DELAY) &&
                   d.act == EVCONV_ACT_NONE;
    if (lin) {
      n.kernel = kKernConvValu;
      n.c_out_pad = (d.c_out + 31) / 32 * 32;
    } else if (d.op == EVCONV_OP_GLOBAL_AVGPOOL) n.kernel = kKernGap;
    else if (d.op == EVCONV_OP_MAXPOOL) n.kernel = kKernPool;
    else if (d.op == EVCONV_OP_DELAY) n.kernel = kKernDelay;
    else n.kernel = kKernElementwise;
    occ_word_off[i] = words;
    words += 2 * (size_t)n.go.tiles();
  }
  for (int i = 0; i < desc->n_nodes; ++i) {
    const NodePlan& n = L->nodes[i];
    if (n.d.op != EVCONV_OP_DELAY) continue;
    const Geo& x = L->nodes[n.d.in0].go;
    if (x.c != n.go.c || x.h != n.go.h || x.w != n.go.w) {
      char where[96];
      snprintf(where, sizeof where, "node %d: DELAY shape differs from that of node %d", i, n.d.in0);
      return fail(err, EVCONV_ERR_SHAPE, where);
    }
  }
  size_t ks_floats = 0, ks_counters = 0;  // (the layers run one after the other: one scratch for all)
  for (int i = 0; i < desc->n_nodes; ++i) {
    const NodePlan& n = L->nodes[i];
    if (n.d.op != EVCONV_OP_CONV2D && n.d.op != EVCONV_OP_LINEAR) continue;
    ConvParams probe;
    probe.gi = n.ga; probe.go = n.go; probe.k = n.d.kh; probe.stride = n.d.stride; probe.c_out_pad = n.c_out_pad;
    probe.n_fused = 0; probe.pad = n.d.pad; probe.st = Streams{0, desc->n_streams > 0 ? desc->n_streams : 1};
    probe.fp32 = n.d.wdtype == EVCONV_F32;
    size_t f = 0, c = 0;
    if (conv_mfma_f32_supported(probe)) conv_mfma_split_scratch(probe, &f, &c);
    ks_floats = std::max(ks_floats, f);
    ks_counters = std::max(ks_counters, c);
  }
  // the arrival counters lie behind the occupancy words and are cleared with them at the start of a pass
  // (every launch leaves them zero; a pass that did not run to its end need not have)
  L->off_ks_count = L->off_occ_nodes + words * sizeof(uint64_t);
  words += (ks_counters * sizeof(unsigned) + 7) / 8;
  L->n_occ_words = words;
  b.take(words * sizeof(uint64_t));
  for (int i = 0; i < desc->n_nodes; ++i) {
    NodePlan& n = L->nodes[i];
    n.off_occ = L->off_occ_nodes + occ_word_off[i] * sizeof(uint64_t);
    n.off_touched = n.off_occ + (size_t)n.go.tiles() * sizeof(uint64_t);
  }
  const std::vector<int> consumers = consumer_counts(L->nodes);
  // What the streams share: with several, offsets behind their states until these are known.  With one, every layer's
  // weights beside its state (depth net in split mode 243.8 us, with all weights behind the states 245.4; flow net 271.8 / 272.6).
  L->n_streams = desc->n_streams > 0 ? desc->n_streams : 1;
  Bump behind;
  Bump& shared = L->n_streams > 1 ? behind : b;
  // input stage
  const size_t in_elems = (size_t)L->gin.c * L->gin.sites();
  L->off_x_prev = b.take(in_elems * 4);
  L->off_dx = b.take(in_elems * 4);
  L->off_occ_in = b.take((size_t)L->gin.tiles() * 8);
  L->off_idx_in = b.take((size_t)L->gin.sites() * 4);
  L->off_count_in = b.take(4);
  L->off_bitmap_in = b.take(((size_t)L->gin.tiles() + 63) / 64 * 8);
  for (int i = 0; i < desc->n_nodes; ++i) {
    NodePlan& n = L->nodes[i];
    const size_t elems = (size_t)n.go.c * n.go.sites();
    if (n.keeps_z || n.d.op == EVCONV_OP_MAXPOOL) n.off_z = b.take(elems * 4);
    if (n.d.op == EVCONV_OP_SPARSIFY) n.off_step = b.take(4);
    if (n.d.op == EVCONV_OP_MUL) n.off_z2 = b.take(elems * 4);
    if (n.d.op == EVCONV_OP_DELAY) n.off_occ_saved = b.take((size_t)n.go.tiles() * 8);
    if (n.d.op == EVCONV_OP_MAXPOOL) n.off_pool = b.take((size_t)n.ga.c * n.ga.sites() * 4);
    n.off_out = b.take(elems * 4);
    n.off_idx = b.take((size_t)n.go.sites() * 4);
    n.off_count = b.take(4);
    n.off_bitmap = b.take(((size_t)n.go.tiles() + 63) / 64 * 8);
    if (n.d.op == EVCONV_OP_CONV2D || n.d.op == EVCONV_OP_LINEAR) {
      const int k = n.d.kh;
      // room for input channels padded to whole chunks (at most 64), three bf16 parts each at most,
      // or a padded flattened contraction (the narrow-input kernel's per-lane layout)
      n.off_w = shared.take(std::max(((size_t)k * k * ((n.d.c_in + 63) / 64 * 64) + 16) * n.c_out_pad *
                                    (n.d.wdtype == EVCONV_F32 ? 6 : 4),
                                conv_narrow_weight_floats(n.c_out_pad) * 4));
      if (n.d.bias_off >= 0) n.off_bias = shared.take((size_t)n.d.c_out * 4);
      if (const size_t fold = fold_set_bytes(L->nodes, consumers, n, desc->flags, L->n_streams)) {
        n.folds = true;
        n.off_w_fold = shared.take(fold);
        n.off_fold_list = shared.take((size_t)((n.ga.h / 2 + 7) / 8) * ((n.ga.w / 2 + 7) / 8) * 3 * sizeof(int));
      }
    }
    if (n.d.is_output) {
      n.off_y = b.take(elems * 4);
      n.off_dy = b.take(elems * 4);
    }
  }
  L->off_row_or = b.take(builder_scratch_words(L->gin) * sizeof(uint64_t));
  L->off_rms = b.take(sizeof(float) * kRmsBlocks);
  L->off_ks_part = b.take(ks_floats * sizeof(float));
  L->off_int = shared.take(sizeof(IntegrateDesc) * (size_t)desc->n_nodes);
  L->off_sets = shared.take(sizeof(SetDesc) * (size_t)(desc->n_nodes + 1));
  L->stride = b.cur;
  const size_t states = L->n_streams > 1 ? L->stride * (size_t)L->n_streams : 0;
  for (NodePlan& n : L->nodes)
    for (size_t* off : {&n.off_w, &n.off_bias, &n.off_w_fold, &n.off_fold_list}) *off += states;
  L->off_int += states;
  L->off_sets += states;
  L->total = states + shared.cur;
  return EVCONV_OK;
}

}  // namespace

struct evconv_net {
  Layout L;
  float sparsify_tp = 0.0f;
  float* rms_partial = nullptr;
  std::vector<evconv_node_desc> desc_nodes;
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  int mode = EVCONV_MODE_INCREMENTAL;
  uint32_t flags = 0;
  bool has_sparsify = false;  // some SPARSIFY node has a nonzero rounding step
  // AUTO mode: windows of kAutoProbe steps are timed in each mode with an event pair; the faster
  // mode then runs for kAutoHold steps
  int auto_choice = EVCONV_MODE_INCREMENTAL;
  int auto_phase = 0;         // 0: timing incremental, 1: timing dense recompute, 2: holding auto_choice
  int auto_count = 0;         // steps done in the current phase
  bool auto_pending = false;  // both windows are recorded, their events may not have completed yet
  hipEvent_t auto_ev[4] = {nullptr, nullptr, nullptr, nullptr};
  int refresh_period = 0, since_refresh = 0;
  bool has_state = false;
  int static_device = -1;   // >= 0: the net lives in that device's static workspace
  bool last_dense = true;   // the previous pass was a regular forward pass (DELAY nodes)
  bool zero_state = false;  // the pass being enqueued starts from the zero recurrent state (reset)
  Streams st{0, 1};
  size_t in_stride = 0;
  std::string err;
  std::vector<int> outputs;
  float *x_prev = nullptr, *dx = nullptr;
  uint64_t *occ_in = nullptr, *bitmap_in = nullptr, *occ_nodes = nullptr;
  int32_t *idx_in = nullptr, *count_in = nullptr;
  SetDesc* sets_dev = nullptr;
  IntegrateDesc* int_dev = nullptr;  // outputs integrated at the end of a pass
  int n_int = 0, int_blocks = 0, int_large = 0;
  // optional per-node timing with HIP events on the net's stream
  bool prof = false;
  std::vector<hipEvent_t> prof_ev;
  std::vector<int> prof_node;
  std::vector<double> node_ms;
  std::vector<long long> node_launches;
};

namespace {

evconv_status hip_fail(evconv_net* net, hipError_t e, const char* what) {
  net->err = std::string(what) + ": " + hipGetErrorString(e);
  return EVCONV_ERR_HIP;
}

// kPassRefresh: the refresh step of "Drift Errors" in mid-stream: a reset that keeps the recurrent
// state and returns dy = y(n) - y(n-1), so that Eq.2 holds across it
enum PassKind { kPassStep = 0, kPassReset = 1, kPassRecompute = 2, kPassRefresh = 3 };
constexpr int kAutoProbe = 4, kAutoHold = 256;

// Enqueues one pass of the whole network.
evconv_status run_pass(evconv_net* net, const float* input, int builder_mode, PassKind pass) {
  hipStream_t s = net->stream;
  const int dense = pass != kPassStep;
  const bool reinit = pass == kPassReset || pass == kPassRefresh;  // sparsification residuals and steps restart
  const int int_mode = pass == kPassStep ? kIntStep : pass == kPassReset ? kIntReset : kIntRecompute;
  BuilderParams bp;
  bp.in = input; bp.x_prev = net->x_prev; bp.dx = net->dx; bp.occ = net->occ_in;
  bp.row_or = (uint64_t*)(net->ws + net->L.off_row_or);
  bp.clear = net->occ_nodes; bp.n_clear = (unsigned)net->L.n_occ_words;
  bp.g = net->L.gin; bp.mode = builder_mode;
  bp.st = net->st; bp.in_stride = net->in_stride;
  // per-launch timing (evconv_profile_begin): record r is an event pair around the launches of
  // prof_node[r]; -1 stands for the increment builder, n_nodes for the list compaction
  auto timed_begin = [&]() {
    const bool timed = net->prof && 2 * (net->prof_node.size() + 1) <= net->prof_ev.size();
    if (timed) (void)hipEventRecord(net->prof_ev[2 * net->prof_node.size()], s);
    return timed;
  };
  auto timed_end = [&](bool timed, int node) {
    if (!timed) return;
    (void)hipEventRecord(net->prof_ev[2 * net->prof_node.size() + 1], s);
    net->prof_node.push_back(node);
  };
  {
    const bool timed = timed_begin();
    launch_builder(bp, s);
    timed_end(timed, -1);
  }

  // arguments of conv node i's launch
  auto conv_params = [&](int i) {
    const NodePlan& n = net->L.nodes[i];
    const evconv_node_desc& d = n.d;
    const float* a = d.in0 < 0 ? net->dx : net->L.nodes[d.in0].out;
    const uint64_t* occ_a = d.in0 < 0 ? net->occ_in : net->L.nodes[d.in0].occ;
    ConvParams p;
    p.in = a; p.occ_in = occ_a; p.w = n.w; p.bias = n.bias; p.z = n.z; p.out = n.out;
    p.occ_out = n.occ; p.occ_touched = n.touched; p.gi = n.ga; p.go = n.go; p.c_out_pad = n.c_out_pad;
    p.k = d.kh; p.stride = d.stride; p.pad = d.pad; p.act = d.act; p.dense = dense;
    p.n_fused = n.n_fused;
    p.st = net->st;
    p.upsample = 0; p.lo_h = 0; p.lo_w = 0;
    p.tail_units = n.tail_units; p.fp32 = d.wdtype == EVCONV_F32;
    p.w_unscale = 1.0f / n.w_scale; p.w_fold_unscale = 1.0f / n.w_fold_scale;
    p.ks = 0; p.ks_chunks = 0;
    p.ks_part = (float*)(net->ws + net->L.off_ks_part);
    p.ks_count = (unsigned*)(net->ws + net->L.off_ks_count);
    p.y = nullptr; p.dy = nullptr; p.int_mode = 0;
    p.fold_list = n.fold_list; p.w_fold = n.w_fold; p.wg_swap = 0;
    if (n.upsampled_from != -2) {
      // read the stored low-resolution tensor; p.gi stays the up-sampled geometry
      const int src = n.upsampled_from;
      p.in = src < 0 ? net->dx : net->L.nodes[src].out;
      p.occ_in = src < 0 ? net->occ_in : net->L.nodes[src].occ;
      const Geo& gl = src < 0 ? net->L.gin : net->L.nodes[src].go;
      p.upsample = 1; p.lo_h = gl.h; p.lo_w = gl.w;
    }
    p.sp = FusedSparsify{};
    if (n.fused_sp >= 0) {
      const NodePlan& sp = net->L.nodes[n.fused_sp];
      p.sp.delta = sp.z; p.sp.out = sp.out; p.sp.occ_out = sp.occ; p.sp.occ_touched = sp.touched; p.sp.step = sp.step;
    }
    for (int f = 0; f < kMaxFusedAdds; ++f) p.fused[f] = FusedAdd{};
    for (int f = 0; f < n.n_fused; ++f) {
      const NodePlan& a_node = net->L.nodes[n.fused_nodes[f]];
      // the ADD's other input: the one that is not the previous stage
      const int prev = f == 0 ? i : n.fused_nodes[f - 1];
      const int other = a_node.d.in0 == prev ? a_node.d.in1 : a_node.d.in0;
      FusedAdd& fa = p.fused[f];
      fa.skip = other < 0 ? net->dx : net->L.nodes[other].out;
      fa.occ_skip = other < 0 ? net->occ_in : net->L.nodes[other].occ;
      fa.z = a_node.z; fa.out = a_node.out; fa.occ_out = a_node.occ; fa.occ_touched = a_node.touched;
      fa.act = a_node.d.act; fa.keeps_z = a_node.keeps_z; fa.structural = a_node.structural;
    }
    if (n.integrates) {
      p.y = n.y; p.dy = n.dy;
      p.int_mode = int_mode;
    }
    return p;
  };

  for (size_t i = 0; i < net->L.nodes.size(); ++i) {
    NodePlan& n = net->L.nodes[i];
    const evconv_node_desc& d = n.d;
    const float* a = d.in0 < 0 ? net->dx : net->L.nodes[d.in0].out;
    const uint64_t* occ_a = d.in0 < 0 ? net->occ_in : net->L.nodes[d.in0].occ;
    const bool two = d.op == EVCONV_OP_ADD || d.op == EVCONV_OP_CONCAT || d.op == EVCONV_OP_MUL;
    const float* bptr = two ? (d.in1 < 0 ? net->dx : net->L.nodes[d.in1].out) : nullptr;
    const uint64_t* occ_b = two ? (d.in1 < 0 ? net->occ_in : net->L.nodes[d.in1].occ) : nullptr;
    if (n.gather_fused_into >= 0) continue;  // exists only inside the consuming conv's gather
    if (n.paired_into >= 0) continue;        // has run in an earlier conv's launch
    if (n.head_batch >= 0 && n.head_batch != (int)i) continue;  // runs in a later head's launch
    if (n.kernel == kKernDelay) {
      const NodePlan& x = net->L.nodes[d.in0];  // not yet visited in this pass: holds the previous pass's results
      DelayParams p;
      p.src_out = x.out; p.occ_saved = n.occ_saved; p.z = n.z; p.out = n.out;
      p.occ_out = n.occ; p.occ_touched = n.touched; p.g = n.go;
      p.dense = dense; p.last_dense = net->last_dense; p.zero_state = net->zero_state;
      p.st = net->st;
      launch_delay(p, s);
      continue;
    }
    if (n.fused_into >= 0) {  // computed by the producing conv's epilogue
      if (d.op == EVCONV_OP_SPARSIFY && reinit && n.step_fixed < 0.0f)
        // refresh: k = t_p * RMS of the layer input, which the producer has just written in full
        launch_rms_step(a, (size_t)n.ga.c * n.ga.sites(), net->sparsify_tp, net->rms_partial, n.step, net->st, s);
      continue;
    }
    const bool timed = timed_begin();
    switch (n.kernel) {
      case kKernConvValu:
      case kKernConvNarrow:
      case kKernConvPointwise:
      case kKernConvMfmaSplit:
      case kKernConvMfmaBf16:
      case kKernConvMfmaF32: {
        if (n.head_batch == (int)i) {  // the last head of a batch runs all of them
          ConvParams heads[kMaxHeadBatch];
          int n_heads = 0;
          for (int h = 0; h <= (int)i; ++h)
            if (net->L.nodes[h].head_batch == (int)i) heads[n_heads++] = conv_params(h);
          launch_conv_pointwise_batch(heads, n_heads, s);
          break;
        }
        const ConvParams p = conv_params((int)i);
        if (n.mates_batch) {
          ConvParams convs[kMaxConvBatch] = {p};
          for (int m = 0; m < n.n_mates; ++m) convs[1 + m] = conv_params(n.mates[m]);
          if (n.kernel == kKernConvMfmaF32) launch_conv_mfma_f32_batch(convs, 1 + n.n_mates, s);
          else if (n.kernel == kKernConvMfmaBf16) launch_conv_mfma_bf16_batch(convs, 1 + n.n_mates, s);
          else launch_conv_mfma_split_batch(convs, 1 + n.n_mates, s);
          break;
        }
        if (n.n_mates) {
          const ConvParams p2 = conv_params(n.mates[0]);
          if (n.kernel == kKernConvMfmaF32) launch_conv_mfma_f32_pair(p, p2, s);
          else if (n.kernel == kKernConvMfmaBf16) launch_conv_mfma_bf16_pair(p, p2, s);
          else launch_conv_mfma_split_pair(p, p2, s);
          break;
        }
        if (n.kernel == kKernConvMfmaF32) launch_conv_mfma_f32(p, s);
        else if (n.kernel == kKernConvMfmaBf16) launch_conv_mfma_bf16(p, s);
        else if (n.kernel == kKernConvNarrow) launch_conv_narrow(p, s);
        else if (n.kernel == kKernConvPointwise) launch_conv_pointwise(p, s);
        else if (n.kernel == kKernConvMfmaSplit) launch_conv_mfma_split(p, s);
        else launch_conv_valu(p, s);
        break;
      }
      case kKernElementwise: {
        EwParams p;
        p.op = d.op == EVCONV_OP_ADD ? kEwAdd : d.op == EVCONV_OP_CONCAT ? kEwConcat : d.op == EVCONV_OP_MUL ? kEwMul :
               d.op == EVCONV_OP_UPSAMPLE_BILINEAR2X ? kEwUp2x : d.op == EVCONV_OP_SPARSIFY ? kEwSparsify : kEwAct;
        p.step = n.step;
        p.st = net->st;
        if (d.op == EVCONV_OP_SPARSIFY && reinit && n.step_fixed < 0.0f)
          // refresh: k = t_p * RMS of the layer input, which the producer has just written in full
          launch_rms_step(a, (size_t)n.ga.c * n.ga.sites(), net->sparsify_tp, net->rms_partial, n.step, net->st, s);
        p.act = d.act; p.dense = dense; p.keeps_z = n.keeps_z; p.structural = n.structural;
        p.ga = n.ga; p.gb = n.gb; p.go = n.go; p.a = a; p.occ_a = occ_a; p.b = bptr; p.occ_b = occ_b;
        if (d.op == EVCONV_OP_CONCAT && n.upsampled_from != -2) {
          // the first operand is an up-sampling that is never stored: read its stored source
          const int src = n.upsampled_from;
          p.op = kEwConcatUp;
          p.a = src < 0 ? net->dx : net->L.nodes[src].out;
          p.occ_a = src < 0 ? net->occ_in : net->L.nodes[src].occ;
          p.ga = src < 0 ? net->L.gin : net->L.nodes[src].go;
        }
        p.z = n.z; p.z2 = n.z2; p.out = n.out; p.occ_out = n.occ; p.occ_touched = n.touched;
        p.k = 1; p.stride = 1; p.pad = 0;
        launch_elementwise(p, s);
        break;
      }
      case kKernPool: {
        EwParams p;
        p.st = net->st; p.z2 = nullptr; p.step = nullptr;
        p.act = kActNone; p.dense = dense; p.keeps_z = 0; p.structural = 0;
        p.ga = n.ga; p.gb = n.ga; p.a = a; p.occ_a = occ_a; p.b = nullptr; p.occ_b = nullptr;
        p.out = nullptr; p.occ_out = nullptr; p.occ_touched = nullptr;
        p.k = d.kh; p.stride = d.stride; p.pad = d.pad;
        p.op = kEwPoolAcc; p.go = n.ga; p.z = n.pool_in;  // a_acc += x_inc on S_in
        launch_elementwise(p, s);
        p.op = kEwPoolMax; p.go = n.go; p.a = n.pool_in; p.z = n.z; p.out = n.out;
        p.occ_out = n.occ; p.occ_touched = n.touched;
        launch_elementwise(p, s);
        break;
      }
      case kKernGap: {
        GapParams p;
        p.a = a; p.occ_a = occ_a; p.ga = n.ga; p.z = n.z; p.out = n.out; p.occ_out = n.occ;
        p.occ_touched = n.touched; p.act = d.act; p.dense = dense;
        p.st = net->st;
        launch_gap(p, s);
        break;
      }
    }
    timed_end(timed, (int)i);
  }
  // recurrent state: keep the delayed nodes' active sets for the next pass (the occupancy words
  // are cleared when it starts).  The compaction of the masks does that on its way, except where
  // the words are cleared before it runs or a node is delayed a second time.
  const bool save_in_lists = !reinit;
  for (size_t i = 0; i < net->L.nodes.size(); ++i) {
    const NodePlan& n = net->L.nodes[i];
    if (n.kernel == kKernDelay && !(save_in_lists && n.saved_in_lists)) launch_copy_u64(n.occ_saved, net->L.nodes[n.d.in0].occ, (size_t)n.go.tiles(), net->st, s);
  }
  net->last_dense = dense != 0;
  if (pass == kPassRefresh) {
    // the nodes' buffers hold values, not increments: every set is emptied, except the active sets of
    // the output nodes, whose dy = y(n) - y(n-1) is a genuine increment at every site
    size_t from = 0;
    for (size_t i = 0; i <= net->L.nodes.size(); ++i) {
      const bool last = i == net->L.nodes.size();
      if (!last && !net->L.nodes[i].d.is_output) continue;
      const size_t to = last ? net->L.n_occ_words : (size_t)(net->L.nodes[i].occ - net->occ_nodes);
      if (to > from) launch_fill_u64(net->occ_nodes + from, to - from, 0, net->st, s);
      if (!last) from = to + (size_t)net->L.nodes[i].go.tiles();  // skip the S words, clear the T words behind them
    }
  }
  {
    const bool timed = timed_begin();
    FinishParams fp;
    fp.sets = net->sets_dev; fp.n_sets = (int)net->L.nodes.size() + 1; fp.max_ty = net->L.max_ty;
    fp.save = save_in_lists;
    fp.empty = pass == kPassReset;  // (the nodes' buffers hold values, not increments)
    fp.outputs = net->int_dev; fp.n_outputs = net->n_int; fp.int_blocks = net->int_blocks; fp.int_mode = int_mode;
    fp.int_large = net->int_large;
    fp.st = net->st;
    launch_finish(fp, s);
    timed_end(timed, (int)net->L.nodes.size());
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(net, e, "kernel launch");
  return EVCONV_OK;
}

void fill_outputs(evconv_net* net, evconv_out* out) {
  if (!out) return;
  for (size_t j = 0; j < net->outputs.size(); ++j) {
    const NodePlan& n = net->L.nodes[net->outputs[j]];
    out[j].node = net->outputs[j];
    out[j].c = n.go.c; out[j].h = n.go.h; out[j].w = n.go.w;
    out[j].y = n.y; out[j].dy = n.dy; out[j].dy_idx = n.idx; out[j].dy_count = n.count;
  }
}

// The weight sets of the four phases and the list of tiles (conv_fold_impl.h), into the workspace.  `lo` is the
// stored tensor's geometry.
hipError_t prepare_fold(evconv_net* net, NodePlan& n, const void* weights, const Geo& lo) {
  constexpr int k = 5, taps = kFoldVectors * kFoldVectors;
  const int ci_n = n.d.c_in, co_n = n.d.c_out, cop = n.c_out_pad;
  // vec[parity][vector][kernel row]: what the up-sampled row under a kernel row contributes to the vector's stored
  // row (columns likewise).  Half-pixel centres: row 2q of the up-sampled tensor is 0.75 * stored row q + 0.25 * row q -
  // 1, row 2q + 1 is 0.75 * row q + 0.25 * row q + 1.  On the first stored row up-sampled rows from 0 on exist, and
  // their sources before row 0 are row 0 (the last row: mirrored).
  double vec[2][kFoldVectors][k] = {};
  for (int par = 0; par < 2; ++par)
    for (int ky = 0; ky < k; ++ky) {
      const int r = par + ky - 2;                      // up-sampled row relative to 2 * (stored row)
      const int q = r >= 0 ? r / 2 : -((1 - r) / 2);   // floor(r / 2)
      const int src[2] = {q, (r - 2 * q) ? q + 1 : q - 1};
      for (int e = 0; e < 2; ++e) {
        const double coef = e ? 0.25 : 0.75;
        vec[par][src[e] + 2 - par][ky] += coef;
        if (r >= 0 && src[e] <= 0) vec[par][kFoldTop][ky] += coef;
        if (r <= 1 && src[e] >= 0) vec[par][kFoldBottom][ky] += coef;
      }
    }
  std::vector<double> folded((size_t)4 * taps * ci_n * co_n, 0.0);
  const float* src = (const float*)((const char*)weights + n.d.weight_off);
  std::vector<double> w((size_t)k * k * ci_n * co_n);  // [tap][ci][co]
  for (int co = 0; co < co_n; ++co)
    for (int ci = 0; ci < ci_n; ++ci)
      for (int t = 0; t < k * k; ++t) w[((size_t)t * ci_n + ci) * co_n + co] = src[((size_t)co * ci_n + ci) * k * k + t];
  for (int ph = 0; ph < 4; ++ph)
    for (int t = 0; t < taps; ++t) {
      double* dst = &folded[((size_t)ph * taps + t) * ci_n * co_n];
      for (int ky = 0; ky < k; ++ky)
        for (int kx = 0; kx < k; ++kx) {
          const double coef = vec[ph >> 1][t / kFoldVectors][ky] * vec[ph & 1][t % kFoldVectors][kx];
          const double* from = &w[(size_t)(ky * k + kx) * ci_n * co_n];
          if (coef != 0.0)
            for (size_t e = 0; e < (size_t)ci_n * co_n; ++e) dst[e] += coef * from[e];
        }
    }
  const std::vector<float> values(folded.begin(), folded.end());
  const int parts = weight_part_count(n.d.wdtype);
  bool fits = true;
  const float scale = weight_scale(values.data(), values.size(), &fits);
  if (!fits) return hipSuccess;  // (a sum of finite weights can overflow: not folded then)
  if (parts == 3) n.w_fold_scale = scale;
  const int ci_p = (ci_n + 31) / 32 * 32;
  const size_t plane = (size_t)taps * ci_p * cop;  // values per part and phase; a phase's planes follow each other
  std::vector<uint16_t> staging(4 * parts * plane, 0);
  for (int ph = 0; ph < 4; ++ph)
    for (int t = 0; t < taps; ++t)
      for (int c8 = 0; c8 < ci_n; c8 += 8) {
        // (fp32 mode: every second group of 16 channels negated, those of the odd partial sums; see conv_mfma_negated)
        const float factor = parts == 3 && (c8 / 16) % 2 ? -n.w_fold_scale : n.w_fold_scale;
        for (int co = 0; co < co_n; ++co) {
          float v[8];
          for (int e = 0; e < 8; ++e)
            v[e] = c8 + e < ci_n ? factor * values[(((size_t)ph * taps + t) * ci_n + c8 + e) * co_n + co] : 0.0f;
          weight_parts8(v, parts, staging.data() + ph * parts * plane + (((size_t)t * (ci_p / 8) + c8 / 8) * cop + co) * 8, plane);
        }
      }
  // Tiles of the border first: their workgroups contract more taps.
  std::vector<int> list, inner;
  for (int ty = 0; ty < lo.ty; ++ty)
    for (int tx = 0; tx < lo.tx; ++tx)
      (ty == 0 || tx == 0 || ty == lo.ty - 1 || tx == lo.tx - 1 ? list : inner).push_back(ty * lo.tx + tx);
  list.insert(list.end(), inner.begin(), inner.end());
  // Behind the tiles the halves of them that hold sites, 2 * tile + half (a workgroup for an empty one still takes a
  // place: 128 -> 64 channels behind 18 x 18, two streams, fp32 20.9 us, now 17.6).  Upper and lower halves in turn, so that an
  // XCD reads the taps of the border for one of the two kinds only (lists without that order: +3 % on 8 us).
  std::vector<int> halves[2];
  for (int t : list)
    for (int half = 0; half < 2; ++half)
      if (t / lo.tx * 8 + half * 4 < lo.h) halves[half].push_back(2 * t + half);
  std::stable_partition(halves[0].begin(), halves[0].end(), [&](int e) { const int ty = e / 2 / lo.tx; return ty == 0 || ty == lo.ty - 1; });
  for (size_t i = 0; i < halves[0].size(); ++i) {
    list.push_back(halves[0][i]);
    if (i < halves[1].size()) list.push_back(halves[1][i]);
  }
  n.w_fold = net->ws + n.off_w_fold;
  n.fold_list = (int*)(net->ws + n.off_fold_list);
  hipError_t e = hipMemcpy(n.w_fold, staging.data(), staging.size() * 2, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(n.fold_list, list.data(), list.size() * 4, hipMemcpyHostToDevice);
  return e;
}

}  // namespace

extern "C" {

evconv_status evconv_query_workspace(const evconv_net_desc* desc, size_t* bytes) {
  if (!bytes) return EVCONV_ERR_INVALID_ARG;
  Layout L;
  evconv_status st = make_layout(desc, 0, false, &L, &g_create_error);
  if (st != EVCONV_OK) return st;
  *bytes = L.total;
  return EVCONV_OK;
}

}  // extern "C"

namespace {
bool is_mfma(const NodePlan& n) {
  return n.kernel == kKernConvMfmaF32 || n.kernel == kKernConvMfmaBf16 || n.kernel == kKernConvMfmaSplit;
}

// Folds ADD and SPARSIFY nodes into the epilogues of matrix-core convs.  Returns how many.
int plan_epilogues(std::vector<NodePlan>& nodes) {
  int folded = 0;
  // where in a pass a node is computed
  auto pos = [&](int i) { return i >= 0 && nodes[i].paired_into >= 0 ? nodes[i].paired_into : i; };
  // A DELAY of node i that stands between the conv and i reads i's buffers as the previous step left
  // them; computed in the conv's epilogue they would already hold this step's values.
  auto delayed_between = [&](int host, int i) {
    for (int dn = pos(host) + 1; dn < i; ++dn)
      if (nodes[dn].d.op == EVCONV_OP_DELAY && nodes[dn].d.in0 == i) return true;
    return false;
  };
  // An ADD goes to the conv that produces the later one of its inputs (residual add + activation, skip
  // adds).  Every buffer of the ADD node is still written.
  for (int i = 0; i < (int)nodes.size(); ++i) {
    NodePlan& a_node = nodes[i];
    if (a_node.d.op != EVCONV_OP_ADD) continue;
    const bool in0_later = pos(a_node.d.in0) > pos(a_node.d.in1);
    const int later = in0_later ? a_node.d.in0 : a_node.d.in1;
    const int other = in0_later ? a_node.d.in1 : a_node.d.in0;
    if (later < 0 || later == other) continue;
    const int host = nodes[later].fused_into >= 0 ? nodes[later].fused_into : later;
    NodePlan& c_node = nodes[host];
    if (!is_mfma(c_node) || c_node.n_fused >= kMaxFusedAdds) continue;
    if (host != later && c_node.fused_nodes[c_node.n_fused - 1] != later) continue;  // chain must be contiguous
    if (pos(other) >= pos(host)) continue;  // the other input must exist before the conv runs
    if (delayed_between(host, i)) continue;
    c_node.fused_nodes[c_node.n_fused++] = i;
    a_node.fused_into = host;
    ++folded;
  }
  // A sparsification layer goes to the matrix-core conv that produces its input, directly or through the
  // last ADD folded into that conv: the layer then reads the increment where it is made (no launch, no
  // re-read).  One layer per conv; every buffer of the layer is still written.
  for (int i = 0; i < (int)nodes.size(); ++i) {
    NodePlan& s_node = nodes[i];
    if (s_node.d.op != EVCONV_OP_SPARSIFY || s_node.d.in0 < 0 || s_node.d.is_output) continue;
    const NodePlan& x = nodes[s_node.d.in0];
    int host = -1;
    if (x.fused_into >= 0) {
      const NodePlan& h = nodes[x.fused_into];
      if (x.d.op == EVCONV_OP_ADD && h.n_fused > 0 && h.fused_nodes[h.n_fused - 1] == s_node.d.in0) host = x.fused_into;
    } else if (x.n_fused == 0 && is_mfma(x)) {
      host = s_node.d.in0;
    }
    if (host < 0 || nodes[host].fused_sp >= 0 || delayed_between(host, i)) continue;
    nodes[host].fused_sp = i;
    s_node.fused_into = host;
    ++folded;
  }
  return folded;
}

evconv_status create_impl(const evconv_net_desc* desc, const void* weights, size_t weight_bytes,
                          void* workspace, size_t workspace_bytes, void* hip_stream, evconv_net** out) {
  if (!out || !workspace || (!weights && weight_bytes)) {
    g_create_error = "null argument";
    return EVCONV_ERR_INVALID_ARG;
  }
  evconv_net* net = new evconv_net();
  evconv_status st = make_layout(desc, weight_bytes, true, &net->L, &g_create_error);
  if (st != EVCONV_OK) { delete net; return st; }
  if (((uintptr_t)workspace & 255) || workspace_bytes < net->L.total) {
    g_create_error = "workspace too small or not 256-byte aligned";
    delete net;
    return EVCONV_ERR_WORKSPACE;
  }
  Layout& L = net->L;
  net->ws = (char*)workspace;
  net->stream = (hipStream_t)hip_stream;
  net->desc_nodes.assign(desc->nodes, desc->nodes + desc->n_nodes);
  char* ws = net->ws;
  net->x_prev = (float*)(ws + L.off_x_prev);
  net->dx = (float*)(ws + L.off_dx);
  net->occ_in = (uint64_t*)(ws + L.off_occ_in);
  net->idx_in = (int32_t*)(ws + L.off_idx_in);
  net->count_in = (int32_t*)(ws + L.off_count_in);
  net->bitmap_in = (uint64_t*)(ws + L.off_bitmap_in);
  net->occ_nodes = (uint64_t*)(ws + L.off_occ_nodes);
  net->sets_dev = (SetDesc*)(ws + L.off_sets);
  net->rms_partial = (float*)(ws + L.off_rms);
  net->sparsify_tp = desc->sparsify_tp;
  net->flags = desc->flags;
  net->st = Streams{L.stride, L.n_streams};
  net->in_stride = (size_t)L.gin.c * L.gin.sites() * sizeof(float);

  // (the uploads below are blocking copies that are not ordered with a non-blocking caller stream:
  // the clearing has to be complete before the first of them)
  hipError_t e = hipMemsetAsync(ws, 0, L.total, net->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
  if (e != hipSuccess) { g_create_error = std::string("clearing the workspace: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }

  std::vector<SetDesc> sets(L.nodes.size() + 1);
  sets[0] = SetDesc{net->occ_in, net->idx_in, net->count_in, net->bitmap_in, L.gin.h, L.gin.w, L.gin.tx, L.gin.ty, nullptr, nullptr};
  std::vector<float> staging;
  for (size_t i = 0; i < L.nodes.size(); ++i) {
    NodePlan& n = L.nodes[i];
    const size_t elems = (size_t)n.go.c * n.go.sites();
    (void)elems;
    n.z = (n.keeps_z || n.d.op == EVCONV_OP_MAXPOOL) ? (float*)(ws + n.off_z) : nullptr;
    if (n.d.op == EVCONV_OP_SPARSIFY) {
      n.step = (float*)(ws + n.off_step);
      if (n.d.weight_off < 0 && desc->sparsify_tp > 0.0f) net->has_sparsify = true;
      if (n.d.weight_off >= 0) {
        memcpy(&n.step_fixed, (const char*)weights + n.d.weight_off, 4);
        if (!(n.step_fixed >= 0.0f)) { g_create_error = "negative sparsification step"; delete net; return EVCONV_ERR_BAD_DESC; }
        if (n.step_fixed > 0.0f) net->has_sparsify = true;
        for (int sidx = 0; sidx < L.n_streams && e == hipSuccess; ++sidx)
          e = hipMemcpy((char*)n.step + (size_t)sidx * L.stride, &n.step_fixed, 4, hipMemcpyHostToDevice);
        if (e != hipSuccess) { g_create_error = std::string("upload: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }
      }
    }
    n.pool_in = n.d.op == EVCONV_OP_MAXPOOL ? (float*)(ws + n.off_pool) : nullptr;
    n.z2 = n.d.op == EVCONV_OP_MUL ? (float*)(ws + n.off_z2) : nullptr;
    n.occ_saved = n.d.op == EVCONV_OP_DELAY ? (uint64_t*)(ws + n.off_occ_saved) : nullptr;
    n.out = (float*)(ws + n.off_out);
    n.occ = (uint64_t*)(ws + n.off_occ);
    n.touched = (uint64_t*)(ws + n.off_touched);
    n.idx = (int32_t*)(ws + n.off_idx);
    n.count = (int32_t*)(ws + n.off_count);
    n.bitmap = (uint64_t*)(ws + n.off_bitmap);
    if (n.d.is_output) {
      n.y = (float*)(ws + n.off_y);
      n.dy = (float*)(ws + n.off_dy);
      net->outputs.push_back((int)i);
    }
    sets[i + 1] = SetDesc{n.occ, n.idx, n.count, n.bitmap, n.go.h, n.go.w, n.go.tx, n.go.ty, nullptr, n.occ};
    if (n.d.op == EVCONV_OP_CONV2D || n.d.op == EVCONV_OP_LINEAR) {
      const int k = n.d.kh, ci_n = n.d.c_in, co_n = n.d.c_out, cop = n.c_out_pad;
      ConvParams probe;
      probe.gi = n.ga; probe.go = n.go; probe.k = k; probe.stride = n.d.stride; probe.c_out_pad = cop;
      probe.n_fused = 0; probe.pad = n.d.pad; probe.st = Streams{L.stride, L.n_streams};
      probe.fp32 = n.d.wdtype == EVCONV_F32;
      n.tail_units = n.d.in0 < 0 || L.nodes[n.d.in0].d.op != EVCONV_OP_UPSAMPLE_BILINEAR2X;
      probe.tail_units = n.tail_units;
      const bool force_valu = (net->flags & EVCONV_FLAG_FORCE_VALU) != 0;
      // (a weight that is infinite or NaN: the vector kernel, which multiplies it as it is)
      if (!force_valu && n.d.wdtype == EVCONV_F32 && conv_mfma_f32_supported(probe)) {
        bool fits = true;
        n.w_scale = weight_scale((const float*)((const char*)weights + n.d.weight_off), (size_t)k * k * ci_n * co_n, &fits);
        if (fits) n.kernel = kKernConvMfmaF32;
      }
      if (!force_valu && n.d.wdtype == EVCONV_BF16 && conv_mfma_bf16_supported(probe)) n.kernel = kKernConvMfmaBf16;
      if (!force_valu && n.d.wdtype == EVCONV_F32_SPLIT && conv_mfma_split_supported(probe)) n.kernel = kKernConvMfmaSplit;
      if (!force_valu && n.kernel == kKernConvValu && conv_narrow_supported(probe)) n.kernel = kKernConvNarrow;
      if (!force_valu && conv_pointwise_supported(probe)) n.kernel = kKernConvPointwise;
      n.integrates = n.kernel == kKernConvPointwise && n.d.is_output && conv_pointwise_integrates(probe);
      const float* src = (const float*)((const char*)weights + n.d.weight_off);
      staging.assign(((size_t)k * k * ((ci_n + 63) / 64 * 64) + 16) * cop, 0.0f);
      const int ci_p = conv_mfma_padded_cin(probe);  // matrix-core kinds: channels padded with zero rows
      if (n.kernel == kKernConvPointwise) {
        // 1 x 1 taps: [c_out][c_in] as supplied; bf16-declared weights are rounded and widened again
        staging.resize((size_t)co_n * ci_n);
        for (size_t e = 0; e < staging.size(); ++e) {
          float w = src[e];
          if (n.d.wdtype == EVCONV_BF16) {
            const uint32_t u = (uint32_t)to_bf16(w) << 16;
            memcpy(&w, &u, 4);
          }
          staging[e] = w;
        }
      } else if (n.kernel == kKernConvNarrow) {
        // flattened contraction k = tap * c_in + ci, laid out per matrix-core lane, zeros beyond
        // taps * c_in and beyond c_out; bf16-declared weights are rounded to bf16 and widened again
        staging.assign(conv_narrow_weight_floats(cop), 0.0f);
        for (int co = 0; co < co_n; ++co)
          for (int ci = 0; ci < ci_n; ++ci)
            for (int t = 0; t < k * k; ++t) {
              float w = src[((size_t)co * ci_n + ci) * k * k + t];
              if (n.d.wdtype == EVCONV_BF16) {
                const uint32_t u = (uint32_t)to_bf16(w) << 16;
                memcpy(&w, &u, 4);
              }
              staging[conv_narrow_weight_index(t * ci_n + ci, co)] = w;
            }
      } else if (n.kernel != kKernConvValu) {
        // matrix-core layout, one plane [tap][c_in/8][c_out][8] of bf16 per part: a lane's 8 input
        // channels are 16 bytes
        const int parts = weight_part_count(n.d.wdtype);
        const size_t plane = (size_t)k * k * ci_p * cop;
        staging.assign((parts * plane + 1) / 2, 0.0f);
        uint16_t* h16 = (uint16_t*)staging.data();
        const int groups = (ci_n + 15) / 16;
        std::vector<float> sign((size_t)k * k * groups, 1.0f);  // [tap][group of 16 channels]
        for (int t = 0; t < k * k && parts == 3; ++t)
          for (int g = 0; g < groups; ++g) sign[(size_t)t * groups + g] = conv_mfma_negated(probe, t, 16 * g) ? -1.0f : 1.0f;
        for (int co = 0; co < co_n; ++co)
          for (int c8 = 0; c8 < ci_n; c8 += 8)
            for (int t = 0; t < k * k; ++t) {
              float v[8];
              const float sg = sign[(size_t)t * groups + c8 / 16] * (parts == 3 ? n.w_scale : 1.0f);
              for (int e = 0; e < 8; ++e) v[e] = c8 + e < ci_n ? sg * src[((size_t)co * ci_n + c8 + e) * k * k + t] : 0.0f;
              weight_parts8(v, parts, h16 + (((size_t)t * (ci_p / 8) + c8 / 8) * cop + co) * 8, plane);
            }
      } else {
        // vector-ALU layout [tap][c_in][c_out_pad] (zero padded output channels)
        for (int co = 0; co < co_n; ++co)
          for (int ci = 0; ci < ci_n; ++ci)
            for (int t = 0; t < k * k; ++t)
              staging[((size_t)t * ci_n + ci) * cop + co] = src[((size_t)co * ci_n + ci) * k * k + t];
      }
      n.w = ws + n.off_w;
      e = hipMemcpyAsync(n.w, staging.data(), staging.size() * 4, hipMemcpyHostToDevice, net->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(net->stream);  // staging is reused
      if (e == hipSuccess && n.d.bias_off >= 0) {
        n.bias = (float*)(ws + n.off_bias);
        e = hipMemcpy(n.bias, (const char*)weights + n.d.bias_off, (size_t)co_n * 4, hipMemcpyHostToDevice);
      }
      if (e != hipSuccess) { g_create_error = std::string("weight upload: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }
    }
  }
  std::vector<IntegrateDesc> ints;
  for (int i : net->outputs) {
    const NodePlan& n = L.nodes[i];
    if (n.integrates) continue;
    ints.push_back(IntegrateDesc{n.out, n.occ, n.y, n.dy, n.go.h, n.go.w, n.go.c, n.go.tx, net->int_blocks});
    net->int_blocks += integrate_blocks(n.go.c, n.go.sites());
    if (integrate_large(n.go.c, n.go.sites())) net->int_large = 1;
  }
  net->n_int = (int)ints.size();
  net->int_dev = (IntegrateDesc*)(ws + L.off_int);
  if (e == hipSuccess && !ints.empty()) e = hipMemcpy(net->int_dev, ints.data(), ints.size() * sizeof(IntegrateDesc), hipMemcpyHostToDevice);
  if (e != hipSuccess) { g_create_error = std::string("upload: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }
  for (NodePlan& n : L.nodes) {
    if (n.d.op != EVCONV_OP_DELAY || sets[n.d.in0 + 1].save) continue;
    sets[n.d.in0 + 1].save = n.occ_saved;
    n.saved_in_lists = true;
  }
  e = hipMemcpyAsync(net->sets_dev, sets.data(), sets.size() * sizeof(SetDesc), hipMemcpyHostToDevice, net->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
  if (e != hipSuccess) { g_create_error = std::string("upload: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }
  if (net->outputs.empty()) { g_create_error = "no output node"; delete net; return EVCONV_ERR_BAD_DESC; }
  const bool fuse = !(net->flags & EVCONV_FLAG_NO_FUSION);
  // A block's shortcut conv runs in the launch of the block's first conv, which reads the same tensor, and
  // the gate convs of a cell in one launch (pair_supported and batchable say where; the sums stay as they
  // are).
  if (fuse) {
    // (a conv that runs earlier may no longer host an ADD whose other input is computed in between, or an ADD
    // of two convs of its launch: such a conv stays where it is)
    auto folds = [&](int late, int into) {
      std::vector<NodePlan> plan = L.nodes;
      if (into >= 0) plan[late].paired_into = into;
      return plan_epilogues(plan);
    };
    auto probe_of = [&](const NodePlan& n) {
      ConvParams p = {};
      p.gi = n.ga; p.go = n.go; p.c_out_pad = n.c_out_pad; p.k = n.d.kh; p.stride = n.d.stride; p.pad = n.d.pad;
      p.st = net->st; p.tail_units = n.tail_units; p.fp32 = n.d.wdtype == EVCONV_F32;
      return p;
    };
    for (int j = 0; j < (int)L.nodes.size(); ++j) {
      NodePlan& late = L.nodes[j];
      if (!is_mfma(late)) continue;
      for (int i = 0; i < j && late.paired_into < 0; ++i) {
        NodePlan& first = L.nodes[i];
        if (first.kernel != late.kernel || first.d.in0 != late.d.in0 || first.paired_into >= 0) continue;
        const ConvParams p = probe_of(first), q = probe_of(late);
        const bool shortcut = late.d.kh == 1 && first.n_mates == 0 && conv_mfma_pair_supported(p, q);
        const bool batch = (first.n_mates == 0 || first.mates_batch) && first.n_mates < kMaxConvBatch - 1 &&
                           conv_mfma_batch_supported(p, q);
        if (!shortcut && !batch) continue;
        bool delayed_between = false;  // (a DELAY of the later one in between must see last step's buffers)
        for (int dn = i + 1; dn < j; ++dn)
          if (L.nodes[dn].d.op == EVCONV_OP_DELAY && L.nodes[dn].d.in0 == j) delayed_between = true;
        if (delayed_between || folds(j, i) < folds(j, -1)) continue;
        first.mates[first.n_mates++] = j;
        first.mates_batch = !shortcut;
        late.paired_into = i;
      }
    }
  }
  // Prediction heads whose results nothing in the net reads run together, where the last one of them
  // stands: their launches need not come between the layers.
  if (fuse) {
    std::vector<char> read(L.nodes.size(), 0);
    for (const NodePlan& n : L.nodes) {
      if (n.d.in0 >= 0) read[n.d.in0] = 1;
      if (n.d.in1 >= 0) read[n.d.in1] = 1;
    }
    auto variant = [&](const NodePlan& n) {
      ConvParams p = {};
      p.go = n.go; p.st = net->st;
      return conv_pointwise_variant(p);
    };
    auto open = [&](int i) {
      return L.nodes[i].kernel == kKernConvPointwise && L.nodes[i].integrates && !read[i] && L.nodes[i].head_batch < 0;
    };
    for (int i = 0; i < (int)L.nodes.size(); ++i) {
      if (!open(i)) continue;
      int members[kMaxHeadBatch] = {i}, n = 1;
      long long tiles = L.nodes[i].go.tiles();
      for (int j = i + 1; j < (int)L.nodes.size() && n < kMaxHeadBatch; ++j) {
        if (!open(j) || variant(L.nodes[j]) != variant(L.nodes[i]) || tiles + L.nodes[j].go.tiles() > (1ll << 23)) continue;
        tiles += L.nodes[j].go.tiles();
        members[n++] = j;
      }
      for (int k = 0; k < n && n > 1; ++k) L.nodes[members[k]].head_batch = members[n - 1];
    }
  }
  if (fuse) plan_epilogues(L.nodes);
  // Fold a bilinear x2 up-sampling into the gather of the matrix-core conv that is its only
  // consumer: the up-sampled tensor is then never written (its node keeps no state).
  if (fuse) {
    const std::vector<int> n_consumers = consumer_counts(L.nodes);
    for (size_t i = 0; i < L.nodes.size(); ++i) {
      NodePlan& c_node = L.nodes[i];
      if (c_node.d.op != EVCONV_OP_CONV2D || c_node.d.in0 < 0) continue;
      NodePlan& u_node = L.nodes[c_node.d.in0];
      if (u_node.d.op != EVCONV_OP_UPSAMPLE_BILINEAR2X || u_node.d.act != EVCONV_ACT_NONE || u_node.d.is_output ||
          n_consumers[c_node.d.in0] != 1 || u_node.fused_into >= 0) continue;
      if (c_node.kernel != kKernConvMfmaF32 && c_node.kernel != kKernConvMfmaBf16 && c_node.kernel != kKernConvMfmaSplit)
        continue;
      ConvParams probe;
      probe.gi = c_node.ga; probe.go = c_node.go; probe.k = c_node.d.kh; probe.stride = c_node.d.stride;
      probe.c_out_pad = c_node.c_out_pad; probe.n_fused = 0; probe.pad = c_node.d.pad;
      probe.st = Streams{L.stride, L.n_streams};
      probe.fp32 = c_node.d.wdtype == EVCONV_F32;
      if (!conv_mfma_upsample_supported(probe)) continue;
      u_node.gather_fused_into = (int)i;
      c_node.upsampled_from = u_node.d.in0;
      // where that pays the up-sampling goes into the weights instead
      if (c_node.folds) {
        const Geo& lo = u_node.d.in0 < 0 ? L.gin : L.nodes[u_node.d.in0].go;
        e = prepare_fold(net, c_node, weights, lo);
        if (e != hipSuccess) { g_create_error = std::string("folded weights upload: ") + hipGetErrorString(e); delete net; return EVCONV_ERR_HIP; }
      }
    }
    // the same for a CONCAT whose first operand is an up-sampling nobody else reads: one kernel
    // interpolates that operand's channels and copies the other's
    for (size_t i = 0; i < L.nodes.size(); ++i) {
      NodePlan& c_node = L.nodes[i];
      if (c_node.d.op != EVCONV_OP_CONCAT || c_node.d.in0 < 0 || c_node.d.in0 == c_node.d.in1) continue;
      NodePlan& u_node = L.nodes[c_node.d.in0];
      if (u_node.d.op != EVCONV_OP_UPSAMPLE_BILINEAR2X || u_node.d.act != EVCONV_ACT_NONE || u_node.d.is_output ||
          n_consumers[c_node.d.in0] != 1 || u_node.fused_into >= 0 || u_node.gather_fused_into >= 0) continue;
      u_node.gather_fused_into = (int)i;
      c_node.upsampled_from = u_node.d.in0;
    }
  }
  *out = net;
  return EVCONV_OK;
}
}  // namespace

extern "C" {

evconv_status evconv_create(const evconv_net_desc* desc, const void* weights, size_t weight_bytes,
                            void* workspace, size_t workspace_bytes, void* hip_stream, evconv_net** out) {
  return create_impl(desc, weights, weight_bytes, workspace, workspace_bytes, hip_stream, out);
}

evconv_status evconv_create_static(const evconv_net_desc* desc, const void* weights, size_t weight_bytes,
                                   void* hip_stream, evconv_net** out) {
  if (!out) { g_create_error = "null argument"; return EVCONV_ERR_INVALID_ARG; }
  Layout L;
  evconv_status st = make_layout(desc, weight_bytes, true, &L, &g_create_error);
  if (st != EVCONV_OK) return st;
  if (L.total > (size_t)EVCONV_STATIC_WORKSPACE_BYTES) {
    g_create_error = "this description needs " + std::to_string(L.total) + " bytes of workspace, the static workspace holds " +
                     std::to_string((size_t)EVCONV_STATIC_WORKSPACE_BYTES);
    return EVCONV_ERR_WORKSPACE;
  }
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    g_create_error = e != hipSuccess ? std::string("hipGetDevice: ") + hipGetErrorString(e) : "device index out of range";
    return EVCONV_ERR_HIP;
  }
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (g_static_owner[dev]) {
    g_create_error = "the static workspace of this device is in use by a net that has not been destroyed";
    return EVCONV_ERR_STATE;
  }
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      g_create_error = std::string("hipGetSymbolAddress: ") + hipGetErrorString(e);
      return EVCONV_ERR_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  // (create_impl clears the part of the array it lays the net out in: the array keeps whatever the
  // previous net left there)
  evconv_net* net = nullptr;
  st = create_impl(desc, weights, weight_bytes, g_scratch_ptr[dev], (size_t)EVCONV_STATIC_WORKSPACE_BYTES, hip_stream, &net);
  if (st != EVCONV_OK) return st;
  net->static_device = dev;
  g_static_owner[dev] = net;
  *out = net;
  return EVCONV_OK;
}

int32_t evconv_num_outputs(const evconv_net* net) { return net ? (int32_t)net->outputs.size() : 0; }

evconv_status evconv_reset(evconv_net* net, const float* x0, evconv_out* out) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (!x0) { net->err = "null x0"; return EVCONV_ERR_INVALID_ARG; }
  net->zero_state = true;
  evconv_status st = run_pass(net, x0, kBuildReset, kPassReset);
  net->zero_state = false;
  if (st != EVCONV_OK) return st;
  net->has_state = true;
  net->since_refresh = 0;
  fill_outputs(net, out);
  return EVCONV_OK;
}

static evconv_status step_common(evconv_net* net, const float* in, int builder_mode, evconv_out* out) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (!in) { net->err = "null input"; return EVCONV_ERR_INVALID_ARG; }
  if (!net->has_state) { net->err = "step before reset"; return EVCONV_ERR_STATE; }
  evconv_status st;
  const bool refresh = net->refresh_period > 0 && net->since_refresh + 1 >= net->refresh_period;
  int mode = net->mode;
  hipEvent_t ev_after = nullptr;
  if (mode == EVCONV_MODE_AUTO) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    (void)hipStreamIsCapturing(net->stream, &cap);
    if (net->has_sparsify || cap != hipStreamCaptureStatusNone || refresh) {
      mode = net->has_sparsify ? EVCONV_MODE_INCREMENTAL : net->auto_choice;
      if (refresh && net->auto_phase < 2) net->auto_count = 0;  // a window holding a refresh is timed again
    } else {
      if (net->auto_pending && hipEventQuery(net->auto_ev[3]) == hipSuccess) {
        float t_inc = 0.f, t_dense = 0.f;
        if (hipEventElapsedTime(&t_inc, net->auto_ev[0], net->auto_ev[1]) == hipSuccess &&
            hipEventElapsedTime(&t_dense, net->auto_ev[2], net->auto_ev[3]) == hipSuccess)
          net->auto_choice = t_dense < t_inc ? EVCONV_MODE_DENSE_RECOMPUTE : EVCONV_MODE_INCREMENTAL;
        net->auto_pending = false;
      }
      (void)hipGetLastError();  // (hipErrorNotReady of the query is not an error of this net)
      if (net->auto_phase == 2 && net->auto_count >= kAutoHold && !net->auto_pending) {
        net->auto_phase = 0;
        net->auto_count = 0;
      }
      mode = net->auto_phase == 0 ? EVCONV_MODE_INCREMENTAL : net->auto_phase == 1 ? EVCONV_MODE_DENSE_RECOMPUTE : net->auto_choice;
      if (net->auto_phase < 2) {
        if (net->auto_count == 0) (void)hipEventRecord(net->auto_ev[2 * net->auto_phase], net->stream);
        if (net->auto_count == kAutoProbe - 1) ev_after = net->auto_ev[2 * net->auto_phase + 1];
      }
      if (++net->auto_count >= kAutoProbe && net->auto_phase < 2) {
        if (net->auto_phase == 1) net->auto_pending = true;
        ++net->auto_phase;
        net->auto_count = 0;
      }
    }
  }
  if (refresh) {
    // "Drift Errors": every N-th step is a regular forward pass of x(n) that re-initialises every
    // accumulated tensor (and the sparsification residuals and step sizes)
    st = run_pass(net, in, builder_mode == kBuildFrame ? kBuildReset : kBuildIncrementDense, kPassRefresh);
    net->since_refresh = 0;
  } else if (mode == EVCONV_MODE_DENSE_RECOMPUTE) {
    // regular forward pass of x(n): the builder first folds the input into x_prev (and, for a
    // supplied increment, adds it), then the dense pass reads the updated frame
    st = run_pass(net, in, builder_mode == kBuildFrame ? kBuildReset : kBuildIncrementDense, kPassRecompute);
  } else {
    st = run_pass(net, in, builder_mode, kPassStep);
    ++net->since_refresh;
  }
  if (ev_after) (void)hipEventRecord(ev_after, net->stream);
  if (st != EVCONV_OK) return st;
  fill_outputs(net, out);
  return EVCONV_OK;
}

evconv_status evconv_step(evconv_net* net, const float* increment, evconv_out* out) {
  return step_common(net, increment, kBuildIncrement, out);
}

evconv_status evconv_step_frame(evconv_net* net, const float* x_t, evconv_out* out) {
  return step_common(net, x_t, kBuildFrame, out);
}

evconv_status evconv_destroy(evconv_net* net) {
  if (!net) return EVCONV_OK;
  (void)hipStreamSynchronize(net->stream);
  for (hipEvent_t e : net->prof_ev) (void)hipEventDestroy(e);
  for (hipEvent_t e : net->auto_ev)
    if (e) (void)hipEventDestroy(e);
  if (net->static_device >= 0) {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (g_static_owner[net->static_device] == net) g_static_owner[net->static_device] = nullptr;
  }
  delete net;
  return EVCONV_OK;
}

evconv_status evconv_set_mode(evconv_net* net, int32_t mode) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (mode != EVCONV_MODE_INCREMENTAL && mode != EVCONV_MODE_DENSE_RECOMPUTE && mode != EVCONV_MODE_AUTO) {
    net->err = "bad mode";
    return EVCONV_ERR_INVALID_ARG;
  }
  if (mode == EVCONV_MODE_AUTO) {
    for (hipEvent_t& e : net->auto_ev)
      if (!e) {
        hipError_t err = hipEventCreate(&e);
        if (err != hipSuccess) return hip_fail(net, err, "hipEventCreate");
      }
    net->auto_phase = 0;
    net->auto_count = 0;
    net->auto_pending = false;
    net->auto_choice = EVCONV_MODE_INCREMENTAL;
  }
  net->mode = mode;
  return EVCONV_OK;
}

int32_t evconv_current_mode(const evconv_net* net) {
  if (!net) return -1;
  if (net->mode != EVCONV_MODE_AUTO) return net->mode;
  if (net->has_sparsify) return EVCONV_MODE_INCREMENTAL;
  return net->auto_phase == 0 ? EVCONV_MODE_INCREMENTAL : net->auto_phase == 1 ? EVCONV_MODE_DENSE_RECOMPUTE : net->auto_choice;
}

evconv_status evconv_set_refresh_period(evconv_net* net, int32_t period) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (period < 0) { net->err = "refresh period must be >= 0"; return EVCONV_ERR_INVALID_ARG; }
  net->refresh_period = period;
  net->since_refresh = 0;
  return EVCONV_OK;
}

evconv_status evconv_node_shape(const evconv_net* net, int32_t node, int32_t* chw) {
  if (!net || !chw || node < -1 || node >= (int)net->L.nodes.size()) return EVCONV_ERR_INVALID_ARG;
  const Geo& g = node < 0 ? net->L.gin : net->L.nodes[node].go;
  chw[0] = g.c; chw[1] = g.h; chw[2] = g.w;
  return EVCONV_OK;
}

evconv_status evconv_get_state(evconv_net* net, int32_t node, int32_t kind, void* dst, size_t bytes) {
  return evconv_get_state_stream(net, 0, node, kind, dst, bytes);
}

evconv_status evconv_stream_stride(const evconv_net* net, size_t* bytes, int32_t* n_streams) {
  if (!net || !bytes) return EVCONV_ERR_INVALID_ARG;
  *bytes = net->L.stride;
  if (n_streams) *n_streams = net->L.n_streams;
  return EVCONV_OK;
}

evconv_status evconv_get_state_stream(evconv_net* net, int32_t stream, int32_t node, int32_t kind, void* dst,
                                      size_t bytes) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (stream < 0 || stream >= net->L.n_streams) { net->err = "no such stream"; return EVCONV_ERR_INVALID_ARG; }
  if (!dst || node < -1 || node >= (int)net->L.nodes.size()) { net->err = "bad node or null dst"; return EVCONV_ERR_INVALID_ARG; }
  if (node >= 0 && net->L.nodes[node].gather_fused_into >= 0) {
    net->err = "this node is computed inside its consumer and keeps no state";
    return EVCONV_ERR_INVALID_ARG;
  }
  const Geo& g = node < 0 ? net->L.gin : net->L.nodes[node].go;
  const NodePlan* n = node < 0 ? nullptr : &net->L.nodes[node];
  const void* src = nullptr;
  size_t need = 0;
  const size_t elems = (size_t)g.c * g.sites();
  switch (kind) {
    case EVCONV_STATE_Z: src = n ? n->z : nullptr; need = elems * 4; break;
    case EVCONV_STATE_DY: src = n ? (const void*)n->out : (const void*)net->dx; need = elems * 4; break;
    case EVCONV_STATE_IDX: src = n ? n->idx : net->idx_in; need = (size_t)g.sites() * 4; break;
    case EVCONV_STATE_COUNT: src = n ? n->count : net->count_in; need = 4; break;
    case EVCONV_STATE_BITMAP: src = n ? n->bitmap : net->bitmap_in; need = ((size_t)g.tiles() + 63) / 64 * 8; break;
    case EVCONV_STATE_OCC: src = n ? n->occ : net->occ_in; need = (size_t)g.tiles() * 8; break;
    case EVCONV_STATE_OCC_TOUCHED: src = n ? n->touched : net->occ_in; need = (size_t)g.tiles() * 8; break;
    case EVCONV_STATE_X_PREV: src = n ? nullptr : net->x_prev; need = elems * 4; break;
    case EVCONV_STATE_STEP: src = n ? n->step : nullptr; need = 4; break;
    case EVCONV_STATE_Z2: src = n ? n->z2 : nullptr; need = elems * 4; break;
    default: net->err = "bad state kind"; return EVCONV_ERR_INVALID_ARG;
  }
  if (!src) { net->err = "this node keeps no such state"; return EVCONV_ERR_INVALID_ARG; }
  if (bytes != need) { net->err = "size mismatch: expected " + std::to_string(need) + " bytes"; return EVCONV_ERR_INVALID_ARG; }
  hipError_t e = hipStreamSynchronize(net->stream);
  if (e == hipSuccess)
    e = hipMemcpy(dst, (const char*)src + (size_t)stream * net->L.stride, need, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(net, e, "get_state");
  return EVCONV_OK;
}

evconv_status evconv_get_stats(evconv_net* net, int32_t node, evconv_layer_stats* out) {
  if (!net || !out || node < 0 || node >= (int)net->L.nodes.size()) return EVCONV_ERR_INVALID_ARG;
  const NodePlan& n = net->L.nodes[node];
  const int tiles = n.go.tiles();
  std::vector<uint64_t> words(2 * (size_t)tiles);
  hipError_t e = hipStreamSynchronize(net->stream);
  if (e == hipSuccess) e = hipMemcpy(words.data(), n.occ, words.size() * 8, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_fail(net, e, "get_stats");
  memset(out, 0, sizeof *out);
  out->n_sites = n.go.sites();
  out->n_tiles = tiles;
  for (int t = 0; t < tiles; ++t) {
    out->n_active += __builtin_popcountll(words[t]);
    out->n_touched += __builtin_popcountll(words[tiles + t]);
    out->n_touched_tiles += words[tiles + t] != 0;
  }
  if (n.d.op == EVCONV_OP_CONV2D || n.d.op == EVCONV_OP_LINEAR) {
    const double per_site = 2.0 * n.d.kh * n.d.kh * n.d.c_in * n.d.c_out;
    out->flops_dense = per_site * n.go.sites();
    out->flops_executed = per_site * 64.0 * out->n_touched_tiles;
  }
  return EVCONV_OK;
}

evconv_status evconv_profile_begin(evconv_net* net, int32_t max_records) {
  if (!net || max_records <= 0) return EVCONV_ERR_INVALID_ARG;
  for (hipEvent_t e : net->prof_ev) (void)hipEventDestroy(e);
  net->prof_ev.assign(2 * (size_t)max_records, nullptr);
  for (hipEvent_t& e : net->prof_ev) {
    hipError_t err = hipEventCreate(&e);
    if (err != hipSuccess) return hip_fail(net, err, "hipEventCreate");
  }
  net->prof_node.clear();
  net->node_ms.assign(net->L.nodes.size() + 2, 0.0);  // [node + 1]
  net->node_launches.assign(net->L.nodes.size() + 2, 0);
  net->prof = true;
  return EVCONV_OK;
}

evconv_status evconv_profile_end(evconv_net* net) {
  if (!net) return EVCONV_ERR_INVALID_ARG;
  if (!net->prof) { net->err = "profiling was not started"; return EVCONV_ERR_STATE; }
  net->prof = false;
  hipError_t e = hipStreamSynchronize(net->stream);
  if (e != hipSuccess) return hip_fail(net, e, "profile_end");
  for (size_t r = 0; r < net->prof_node.size(); ++r) {
    float ms = 0.f;
    e = hipEventElapsedTime(&ms, net->prof_ev[2 * r], net->prof_ev[2 * r + 1]);
    if (e != hipSuccess) return hip_fail(net, e, "hipEventElapsedTime");
    net->node_ms[net->prof_node[r] + 1] += ms;
    net->node_launches[net->prof_node[r] + 1] += 1;
  }
  for (hipEvent_t ev : net->prof_ev) (void)hipEventDestroy(ev);
  net->prof_ev.clear();
  net->prof_node.clear();
  return EVCONV_OK;
}

evconv_status evconv_get_node_time(const evconv_net* net, int32_t node, double* ms_total, int64_t* launches) {
  if (!net || !ms_total || !launches || node < -1 || node > (int)net->L.nodes.size()) return EVCONV_ERR_INVALID_ARG;
  if (net->node_ms.empty()) { *ms_total = 0; *launches = 0; return EVCONV_OK; }
  *ms_total = net->node_ms[node + 1];
  *launches = net->node_launches[node + 1];
  return EVCONV_OK;
}

const char* evconv_node_kernel(const evconv_net* net, int32_t node) {
  if (!net || node < 0 || node >= (int)net->L.nodes.size()) return "";
  if (net->L.nodes[node].fused_into >= 0) return "fused_into_conv_epilogue";
  if (net->L.nodes[node].gather_fused_into >= 0) {
    const NodePlan& consumer = net->L.nodes[net->L.nodes[node].gather_fused_into];
    if (consumer.d.op == EVCONV_OP_CONCAT) return "fused_into_concat_gather";
    return consumer.fold_list ? "fused_into_conv_weights" : "fused_into_conv_gather";
  }
  return kKernelNames[net->L.nodes[node].kernel];
}

evconv_status evconv_debug_phase_stamps(int32_t operand_mode, uint64_t* out, int32_t max_records, int32_t reset,
                                        int32_t* n_records) {
  if (!n_records || max_records < 0 || (max_records > 0 && !out)) return EVCONV_ERR_INVALID_ARG;
  int n;
  unsigned long long* dst = (unsigned long long*)out;
  if (operand_mode == EVCONV_F32) n = evk::conv_mfma_f32_phase_stamps(dst, max_records, reset != 0);
  else if (operand_mode == EVCONV_BF16) n = evk::conv_mfma_bf16_phase_stamps(dst, max_records, reset != 0);
  else if (operand_mode == EVCONV_F32_SPLIT) n = evk::conv_mfma_split_phase_stamps(dst, max_records, reset != 0);
  else return EVCONV_ERR_INVALID_ARG;
  if (n == -1) return EVCONV_ERR_UNSUPPORTED;
  if (n < 0) return EVCONV_ERR_HIP;
  *n_records = n;
  return EVCONV_OK;
}

evconv_status evconv_debug_chip_probes(void* scratch, size_t scratch_bytes, void* hip_stream, float* out, int32_t n_out) {
  if (!scratch || !out || scratch_bytes < EVCONV_CHIP_PROBE_SCRATCH_BYTES || n_out < EVCONV_CHIP_PROBE_VALUES)
    return EVCONV_ERR_INVALID_ARG;
  static_assert(EVCONV_CHIP_PROBE_VALUES == evk::kChipProbeValues && EVCONV_CHIP_PROBE_SCRATCH_BYTES == evk::kChipProbeScratch,
                "header and probes disagree");
  return evk::chip_probes(scratch, scratch_bytes, (hipStream_t)hip_stream, out, n_out) == evk::kChipProbeValues ? EVCONV_OK
                                                                                                                 : EVCONV_ERR_HIP;
}

const char* evconv_last_error(const evconv_net* net) { return net ? net->err.c_str() : g_create_error.c_str(); }

}  // extern "C"
