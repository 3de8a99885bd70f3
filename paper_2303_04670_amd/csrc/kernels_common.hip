// gfx950 kernels: increment builder, elementwise / structural increment operators, global
// average pool, output integration, ordered list compaction.
//
// Conventions: tensors are H x W x C fp32; a tile is 8 x 8 sites and its occupancy word has
// bit (y%8)*8 + x%8 set for an active site; tiles are row-major.  Nothing here uses
// floating-point atomics: every accumulated element has exactly one writer, so results are
// run-to-run bit-reproducible.
#include <algorithm>

#include "evconv_kernels.h"

namespace evk {

namespace {

// pointers read from memory are generic ones to the compiler (see at_stream)
template <class T>
__device__ __forceinline__ T __attribute__((address_space(1)))* as_global(T* q) {
  return (T __attribute__((address_space(1)))*)q;
}

// inclusive sum over the lanes of a wave (all of them active), by lane shifts in the vector ALU: the
// same through __shfl_up is six round trips through the LDS
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8 inside rows of 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

template <class WORDS>
__device__ __forceinline__ bool occ_bit(WORDS occ, int tx, int y, int x) {
  uint64_t w = occ[(y >> 3) * tx + (x >> 3)];
  return (w >> (((y & 7) << 3) | (x & 7))) & 1ull;
}

__device__ __forceinline__ float apply_act(int act, float v) {
  if (act == kActRelu) return fmaxf(v, 0.0f);
  if (act == kActSigmoid) return 1.0f / (1.0f + expf(-v));
  if (act == kActTanh) return tanhf(v);
  if (act == kActOneMinus) return 1.0f - v;
  return v;
}

// in-bounds mask of tile (tile_y, tile_x) of an h x w grid, bit layout as the occupancy words
__device__ __forceinline__ uint64_t inbounds_word(int h, int w, int tile_y, int tile_x) {
  int rows = min(8, h - tile_y * 8), cols = min(8, w - tile_x * 8);
  uint64_t row = (cols >= 8) ? 0xffull : ((1ull << cols) - 1);
  uint64_t m = 0;
  for (int r = 0; r < rows; ++r) m |= row << (8 * r);
  return m;
}

}  // namespace

// =============================================================================== builder
// N elements of a thread, element j at ok[j] ? e[j] : nowhere (d[j] = 0).  All loads are requested before
// the first store: a store to the cached frame between two loads of it would keep them in order,
// one round trip per channel.
template <int N>
__device__ __forceinline__ void build_elements(const BuilderParams& p, const int* e, const bool* ok, float* d) {
  float in[N], prev[N];
  const bool needs_prev = p.mode != kBuildReset;
#pragma unroll
  for (int j = 0; j < N; ++j) in[j] = ok[j] ? p.in[e[j]] : 0.0f;
#pragma unroll
  for (int j = 0; j < N; ++j) prev[j] = (ok[j] && needs_prev) ? p.x_prev[e[j]] : 0.0f;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    // Eq.1: one binary32 subtraction; a supplied increment advances the cached frame (dense
    // recompute emits the new frame); a reset emits the frame
    const float sum = prev[j] + in[j];
    const float x = (p.mode == kBuildIncrement || p.mode == kBuildIncrementDense) ? sum : in[j];
    d[j] = p.mode == kBuildFrame ? in[j] - prev[j] : p.mode == kBuildIncrementDense ? sum : in[j];
    if (ok[j]) p.x_prev[e[j]] = x;
  }
}

// clear the per-node occupancy words that the layer kernels OR into
__device__ __forceinline__ void clear_words(const BuilderParams& p) {
  if (!p.clear) return;
  const ClearShare mine = clear_share(gridDim.x, gridDim.y, blockDim.x, blockIdx.x, blockIdx.y, threadIdx.x);
  for (long long i = mine.first; i < (long long)p.n_clear; i += mine.step) p.clear[i] = 0;
}

// Strips: one workgroup = 8 wavefronts = an 8-row x 64-column strip (8 tiles).  Wave r reads row r with
// 256-byte coalesced loads per channel, all N in flight; its ballot is the 64-column activity of
// that row.  The eight ballots are transposed through LDS into eight tile occupancy words.
template <int N>
__global__ __launch_bounds__(512) void builder_kernel(BuilderParams p) {
  touch_params<BuilderParams>();
  {
    const size_t so = (size_t)blockIdx.z * p.st.stride;
    p.in = at_stream(p.in, (size_t)blockIdx.z * p.in_stride);
    p.x_prev = at_stream(p.x_prev, so); p.dx = at_stream(p.dx, so);
    p.occ = at_stream(p.occ, so); p.clear = at_stream(p.clear, so);
  }
  __shared__ uint64_t s_rows[8];
  const int lane = threadIdx.x & 63;
  const int r = threadIdx.x >> 6;
  const int y = blockIdx.y * 8 + r;
  const int x = blockIdx.x * 64 + lane;
  const int hw = p.g.h * p.g.w;
  const bool inb = (y < p.g.h) && (x < p.g.w);
  bool any = false;
  if (inb) {
    const int site = y * p.g.w + x;
    int e[N];
    bool ok[N];
    float d[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      ok[j] = true;
      e[j] = j * hw + site;
    }
    build_elements<N>(p, e, ok, d);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      p.dx[(size_t)site * N + j] = d[j];
      any |= d[j] != 0.0f;
    }
  }
  const uint64_t row_mask = __ballot(any);
  if (lane == 0) s_rows[r] = row_mask;
  __syncthreads();
  if (threadIdx.x < 8) {
    const int j = threadIdx.x;
    const int tile_x = blockIdx.x * 8 + j;
    if (tile_x < p.g.tx) {
      uint64_t word = 0;
      for (int rr = 0; rr < 8; ++rr) word |= ((s_rows[rr] >> (8 * j)) & 0xffull) << (8 * rr);
      if (p.mode >= kBuildReset) word = 0;
      p.occ[blockIdx.y * p.g.tx + tile_x] = word;
    }
  }
  clear_words(p);
}

// Wide inputs (a network that starts inside another one): workgroup = 64 sites, 2^LS columns x 64 / 2^LS
// rows, x 8 N channels, lane = site, the channels dealt to the 8 waves, so that the channel-major input is read in
// runs of up to 256 bytes.  The increments are turned through LDS and written in runs of the workgroup's
// channels.  The sites' activity is the OR over their channel blocks: 32 sites and a bit per block that has
// arrived share a scratch word (p.row_or), so that one atomic both adds a block's share and tells the last one
// that it is the last; that one writes the tile rows' bytes and leaves the word zero for the next launch.
constexpr int kWideBlocks = 32;  // channel blocks at most: arrival bits of a scratch word
template <int N, int LS>
__global__ __launch_bounds__(512) void builder_wide_kernel(BuilderParams p) {
  touch_params<BuilderParams>();
  {
    const size_t so = (size_t)blockIdx.z * p.st.stride;
    p.in = at_stream(p.in, (size_t)blockIdx.z * p.in_stride);
    p.x_prev = at_stream(p.x_prev, so); p.dx = at_stream(p.dx, so);
    p.occ = at_stream(p.occ, so); p.clear = at_stream(p.clear, so);
    p.row_or = at_stream(p.row_or, so);
  }
  constexpr int CB = 8 * N, COLS = 1 << LS;
  // (pitch 66: the reads below are of eight sites x eight channel groups, 8 banks apart)
  __shared__ float s_d[CB][66];
  __shared__ uint64_t s_any[8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int strips = (p.g.w + COLS - 1) >> LS;
  const int group = blockIdx.x / strips, strip = blockIdx.x - group * strips;
  const int y0 = group * (64 >> LS), x0 = strip * COLS, hw = p.g.h * p.g.w, C = p.g.c;
  auto exists = [&](int site) { return y0 + (site >> LS) < p.g.h && x0 + (site & (COLS - 1)) < p.g.w; };
  auto index = [&](int site) { return (y0 + (site >> LS)) * p.g.w + x0 + (site & (COLS - 1)); };
  const bool inb = exists(lane);  // (the rows of the last tiles that lie below the image: bytes of zeros)
  const int own = index(lane);
  bool any = false;
  for (int c0 = blockIdx.y * CB; c0 < C; c0 += gridDim.y * CB) {
    if (c0 != (int)blockIdx.y * CB) __syncthreads();
    const int nc = min(CB, C - c0);
    int e[N];
    bool ok[N];
    float d[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int c = wave * N + j;
      ok[j] = inb && c < nc;
      e[j] = (c0 + c) * hw + own;
    }
    build_elements<N>(p, e, ok, d);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      s_d[wave * N + j][lane] = d[j];
      any |= ok[j] && d[j] != 0.0f;
    }
    __syncthreads();
    if (LS < 6 || y0 < p.g.h) {  // (uniform; rows of 64 columns lie below the image as a whole)
      if ((C & 3) == 0) {
#pragma unroll
        for (int i = tid; i < 64 * (CB / 4); i += 512) {
          const int q = i / (CB / 4), c = i % (CB / 4) * 4;
          if (exists(q) && c < nc)
            *(float4*)&p.dx[(size_t)index(q) * C + c0 + c] = make_float4(s_d[c][q], s_d[c + 1][q], s_d[c + 2][q], s_d[c + 3][q]);
        }
      } else {
#pragma unroll
        for (int i = tid; i < 64 * CB; i += 512) {
          const int q = i / CB, c = i % CB;
          if (exists(q) && c < nc) p.dx[(size_t)index(q) * C + c0 + c] = s_d[c][q];
        }
      }
    }
  }
  const uint64_t b = __ballot(any);
  if (lane == 0) s_any[wave] = b;
  __syncthreads();
  if (tid < 2) {  // lane h: sites 32 h on
    uint64_t word = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) word |= s_any[i];
    unsigned bits = (unsigned)(word >> (32 * tid));
    bool last = true;
    uint64_t* const acc = p.row_or + (size_t)blockIdx.x * 2 + tid;
    if (p.mode >= kBuildReset) {  // no active set; scratch as a launch of another kind expects it
      bits = 0;
      if (blockIdx.y == 0) *acc = 0;
    } else if (gridDim.y > 1) {
      const unsigned long long mine = bits | (1ull << (32 + blockIdx.y));
      const unsigned long long all = mine | __hip_atomic_fetch_or((unsigned long long*)acc, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = (unsigned)(all >> 32) == (unsigned)((1ull << gridDim.y) - 1ull);
      bits = (unsigned)all;
      if (last) __hip_atomic_store(acc, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (last) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // eight sites: a row of a tile
        const int site = (4 * tid + j) * 8, y = y0 + (site >> LS), tx = (x0 + (site & (COLS - 1))) >> 3;
        if (tx < p.g.tx) ((unsigned char*)(p.occ + (size_t)(y >> 3) * p.g.tx + tx))[y & 7] = (unsigned char)(bits >> (8 * j));
      }
    }
  }
  clear_words(p);
}
size_t builder_scratch_words(const Geo& g) { return (size_t)builder_wide_groups(g.h, g.w) * 2; }

template <int N>
void launch_builder_wide(const BuilderParams& p, hipStream_t s) {
  const dim3 grid((unsigned)builder_wide_groups(p.g.h, p.g.w), std::min((p.g.c + 8 * N - 1) / (8 * N), kWideBlocks), p.st.n);
  switch (builder_wide_ls(p.g.w)) {
    case 6: hipLaunchKernelGGL((builder_wide_kernel<N, 6>), grid, dim3(512), 0, s, p); return;
    case 5: hipLaunchKernelGGL((builder_wide_kernel<N, 5>), grid, dim3(512), 0, s, p); return;
    case 4: hipLaunchKernelGGL((builder_wide_kernel<N, 4>), grid, dim3(512), 0, s, p); return;
    default: hipLaunchKernelGGL((builder_wide_kernel<N, 3>), grid, dim3(512), 0, s, p); return;
  }
}

void launch_builder(const BuilderParams& p, hipStream_t s) {
  dim3 grid((p.g.w + 63) / 64, (p.g.h + 7) / 8, p.st.n);
  // Strips for up to 8 channels, all of them in flight (with rows, whose waves are mostly idle there, 5 on 256 x
  // 352 3.7 / 7.1 us, 8 on 480 x 640 9.1 / 13.9), and for up to 12 from 32768 sites on, where there are waves
  // enough beside a thread's longer chain (rows / strips: 9 on 480 x 640 16.2 / 9.8, eight streams 117 / 63; 12 there 15.9 / 12.2;
  // 12 on 260 x 346 8.7 / 6.8, on 200 x 200 5.8 / 5.2, on 100 x 100 3.6 / 3.8; 9 on 64 x 64 3.2 / 3.5).
  // Rows for more.  Before, strips that walked the channels 8 at a time or tiles x 64 channels, read in pieces of
  // 32 bytes (12 on 64 x 64 6.0, now 3.4 us; 24 on 480 x 640 47.8 / 21.7; 64 on 91 x 121 11.4 / 6.1; 256 on 32 x 44
  // 8.4 / 5.0; 256 on 260 x 346 186 / 78.5, 4.7 TB/s).
  // Several rows to a workgroup on narrow images (eight streams: 64 channels on 2000 x 6 in rows of 64 columns,
  // mostly idle, 114 us, in tiles x 64 channels 20.0, now 22.1; 32 on 300 x 20 13.5 / 17.8 / 8.9, on 400 x 14 15.9 / 15.5 / 7.8;
  // beyond 32 columns 64 are best: 32 on 64 x 36 5.7, in rows of 32 5.9, on 300 x 40 14.8 / 16.7, on 400 x 60 22.4 / 26.9).
  // 16 channels a workgroup up to 16 channels, else 32, a line of 128 bytes (24 on 480 x 640 in blocks of 16, 32
  // and 64: 28.8 / 21.7 / 35.2; 256 on 260 x 346 97 / 78 / 86; 16 on 480 x 640 16.6 / 19.4).
  if (p.g.c > 12 || (p.g.c > 8 && (long long)p.g.sites() * p.st.n < 32768)) {
    if (p.g.c <= 16) launch_builder_wide<2>(p, s);
    else launch_builder_wide<4>(p, s);
    return;
  }
  switch (p.g.c) {
    case 1: hipLaunchKernelGGL((builder_kernel<1>), grid, dim3(512), 0, s, p); return;
    case 2: hipLaunchKernelGGL((builder_kernel<2>), grid, dim3(512), 0, s, p); return;
    case 3: hipLaunchKernelGGL((builder_kernel<3>), grid, dim3(512), 0, s, p); return;
    case 4: hipLaunchKernelGGL((builder_kernel<4>), grid, dim3(512), 0, s, p); return;
    case 5: hipLaunchKernelGGL((builder_kernel<5>), grid, dim3(512), 0, s, p); return;
    case 6: hipLaunchKernelGGL((builder_kernel<6>), grid, dim3(512), 0, s, p); return;
    case 7: hipLaunchKernelGGL((builder_kernel<7>), grid, dim3(512), 0, s, p); return;
    case 8: hipLaunchKernelGGL((builder_kernel<8>), grid, dim3(512), 0, s, p); return;
    case 9: hipLaunchKernelGGL((builder_kernel<9>), grid, dim3(512), 0, s, p); return;
    case 10: hipLaunchKernelGGL((builder_kernel<10>), grid, dim3(512), 0, s, p); return;
    case 11: hipLaunchKernelGGL((builder_kernel<11>), grid, dim3(512), 0, s, p); return;
    case 12: hipLaunchKernelGGL((builder_kernel<12>), grid, dim3(512), 0, s, p); return;
  }
}

// =============================================================================== elementwise
// One workgroup per output tile and slice of the channels.  Every wave derives the tile's touched word;
// the 256 threads take (site, channel vector) pairs with the channel index fastest, so global accesses
// are contiguous runs of C floats per site.
constexpr int kEwVecPerBlock = 16;  // channel vectors per workgroup at most: wide layers split over blockIdx.y

template <int VEC> struct VecT { float v[VEC]; };
template <int VEC> __device__ __forceinline__ VecT<VEC> ldv(const float* ptr) {
  VecT<VEC> r;
  if (VEC == 4) {
    const float4 t = *(const float4*)ptr;  // channel counts are multiples of 4 and buffers 256-byte aligned
    r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) r.v[i] = ptr[i];
  }
  return r;
}
template <int VEC> __device__ __forceinline__ void stv(float* ptr, const VecT<VEC>& x) {
  if (VEC == 4) {
    *(float4*)ptr = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) ptr[i] = x.v[i];
  }
}
template <int VEC> __device__ __forceinline__ VecT<VEC> zerov() {
  VecT<VEC> r;
#pragma unroll
  for (int i = 0; i < VEC; ++i) r.v[i] = 0.0f;
  return r;
}

// One row of bits per lane: bit x of lane y's row is site (y0 + y, x0 + x) of a tensor with these words,
// n_rows <= 24 rows of n_cols <= 24 columns; sites outside the image are zero bits.  A row is a byte of
// each of at most four words (for a tile beyond the left or right border a neighbour's byte is read,
// and cut off with the columns outside the image).
__device__ __forceinline__ unsigned occ_rows(const uint64_t* occ, const Geo& g, int y0, int x0, int n_rows, int n_cols) {
  const int lane = threadIdx.x & 63, y = y0 + lane, tx0 = x0 >> 3;
  const bool row_ok = lane < n_rows && (unsigned)y < (unsigned)g.h;
  const unsigned char* const bytes = (const unsigned char*)occ + (row_ok ? (size_t)(y >> 3) * g.tx * 8 + (y & 7) : 0);
  unsigned b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = bytes[min(max(tx0 + i, 0), g.tx - 1) * 8];
  const int lo = max(0, -x0), hi = min(n_cols, g.w - x0);
  const unsigned inside = ((1u << max(hi, 0)) - 1u) & ~((1u << lo) - 1u);
  return row_ok ? ((b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24)) >> (x0 - tx0 * 8)) & inside : 0u;
}
__device__ __forceinline__ unsigned row_of_lane(unsigned rows, int lane) {
  return (unsigned)__builtin_amdgcn_ds_bpermute(lane * 4, (int)rows);
}

// Four elements of a thread in flight, where that leaves the registers of six waves per SIMD: sums, products,
// maxima and up-samplings of whole vectors take two at a time (sum with an activation, 64 channels on 256 x
// 352, every site active: 30.6 us with four, 25.0 with two; product, 2 % of the sites active, 7.8 and 6.3).
constexpr int ew_in_flight(int op, int vec) {
  return vec == 4 && (op == kEwAdd || op == kEwMul || op == kEwPoolMax || op == kEwUp2x) ? 2 : 4;
}

// The operator and the elements that a thread has in flight (N) are known at compile time: their loads go
// out together, and no wave waits for another before its last step.  With the operator looked up per element
// and a list of the touched sites in LDS, a tile was a chain of up to four round trips (concatenation of an
// up-sampled tensor, 16 x 16 to 256 x 256: 5.8 / 7.4 / 8.4 / 9.8 us, now 5.0 / 6.0 / 6.8 / 9.0; 5 + 64 channels on
// 256 x 352 15.4, now 10.2; max-pool of ResNet-18, two launches, 10.9, now 7.7).
// Element e is vector e % cv of touched site number e / cv: where few sites are touched, few waves have
// work (64 channels on 256 x 352, 2 % of the sites active, tanh / product: 11.4 / 7.6 us with an element
// for each of the 64 sites, now 7.5 / 6.3).
// ACT: a concatenation or an up-sampling with an activation (Eq.12-14 behind Eq.11 or Eq.10), which keeps state.
template <int OP, int VEC, int N, bool ACT = false>
__global__ __launch_bounds__(256) void elementwise_kernel(EwParams p) {
  touch_params<EwParams>();
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  const float* const pa = at_stream(p.a, so);
  const float* const pb = at_stream(p.b, so);
  float* const pz = at_stream(p.z, so);
  float* const pz2 = at_stream(p.z2, so);
  float* const pout = at_stream(p.out, so);
  const bool dense = p.dense != 0;
  constexpr bool TWO = OP == kEwAdd || OP == kEwConcat || OP == kEwMul;
  constexpr bool UP = OP == kEwUp2x || OP == kEwConcatUp;
  const int tid = threadIdx.x, lane = tid & 63;
  const int tile = blockIdx.x;
  const int tile_y = p.tx_magic ? (int)__umulhi((unsigned)tile, p.tx_magic) : tile / p.go.tx, tile_x = tile - tile_y * p.go.tx;

  // the tile's touched word and the operands' active sites, in every wave
  const int rows = min(8, p.go.h - tile_y * 8), cols = min(8, p.go.w - tile_x * 8);
  const uint64_t inb = ((cols >= 8 ? 0xffull : ((1ull << cols) - 1ull)) * 0x0101010101010101ull) &
                       (rows >= 8 ? ~0ull : ((1ull << (8 * rows)) - 1ull));
  uint64_t word, wa = ~0ull, wb = ~0ull;
  unsigned src_rows = 0;  // UP: activity of the stored sites under the tile, from (tile_y * 4 - 1, tile_x * 4 - 1) on
  if (TWO) {
    if (!dense) {
      wa = at_stream(p.occ_a, so)[tile];
      wb = at_stream(p.occ_b, so)[tile];
    }
    word = dense ? inb : wa | wb;
  } else if (UP) {
    if (OP == kEwConcatUp && !dense) wb = at_stream(p.occ_b, so)[tile];
    src_rows = occ_rows(at_stream(p.occ_a, so), p.ga, tile_y * 4 - 1, tile_x * 4 - 1, 6, 6);
    const int ly = lane >> 3, lx = lane & 7;
    const int y0 = (ly + 1) >> 1, x0 = (lx + 1) >> 1;  // (rows and columns y0 and y0 + 1 of the region; outside the image: zero bits)
    const unsigned r = row_of_lane(src_rows, y0) | row_of_lane(src_rows, y0 + 1);
    word = __ballot(((r >> x0) & 3u) != 0);
    if (OP == kEwConcatUp) word |= wb;
    word = dense ? inb : word & inb;
  } else if (OP == kEwPoolMax) {  // windows that contain an active input site
    const int P = 7 * p.stride + p.k;
    const unsigned in_rows = occ_rows(at_stream(p.occ_a, so), p.ga, tile_y * 8 * p.stride - p.pad, tile_x * 8 * p.stride - p.pad, P, P);
    const int ly = lane >> 3, lx = lane & 7;
    unsigned r = 0;
#pragma unroll
    for (int ky = 0; ky < 7; ++ky) {
      const unsigned v = row_of_lane(in_rows, ly * p.stride + ky);
      r |= ky < p.k ? v : 0u;
    }
    word = __ballot(((r >> (lx * p.stride)) & ((1u << p.k) - 1u)) != 0);
    word = dense ? inb : word & inb;
  } else {
    word = dense ? inb : at_stream(p.occ_a, so)[tile];
  }
  if (word == 0) return;

  const int C = p.go.c;
  // channel vectors [v0, v0 + cv) of every touched site belong to this workgroup
  const int v0 = blockIdx.y * p.vec_per_block, cv = min(p.vec_per_block, C / VEC - v0);
  const int cv_magic = (65536 + cv - 1) / cv;  // e / cv == (e * cv_magic) >> 16 for e < 1024 (cv <= 16)
  // (a concatenation of an up-sampling, whose tiles are mostly full, takes all 64 sites as they are: 64 + 64
  // channels on 64 x 64 6.0 us, 6.4 with the list)
  constexpr bool LISTED = OP != kEwConcatUp;
  const int n_sites = LISTED ? __popcll(word) : 64, total = n_sites * cv;
  uint64_t nz_sites = 0;  // sites at which this thread produced a nonzero element
  const int first = __builtin_amdgcn_readfirstlane(tid >> 6) * 64;  // of this wave
  int nth = 0;
  if (LISTED && first < total) {
    // lane r: the r-th touched site (the sites that are not touched follow: a permutation of the lanes)
    const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(word >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)word, 0u));
    nth = __builtin_amdgcn_ds_permute((((word >> lane) & 1ull) ? below : n_sites + lane - below) * 4, lane);
  }
  for (int e0 = first; e0 < total; e0 += N * 256) {
    int site[N], c[N];
    size_t q[N];
    bool on[N];
#pragma unroll
    for (int it = 0; it < N; ++it) {
      const int e = e0 + lane + it * 256, r = __umul24(e, cv_magic) >> 16;
      site[it] = LISTED ? __builtin_amdgcn_ds_bpermute(r * 4, nth) : r & 63;  // (r counts modulo 64)
      c[it] = (v0 + (e - __umul24(r, cv))) * VEC;
      on[it] = r < n_sites && (LISTED || ((word >> site[it]) & 1ull));
      q[it] = (size_t)(tile_y * 8 + (site[it] >> 3)) * p.go.w + (tile_x * 8 + (site[it] & 7));
    }

    // ---- loads: the operands' increments (full values in a regular forward pass) and the old state
    VecT<VEC> lin[N], lin_b[N], z_old[N], z2_old[N];
#pragma unroll
    for (int it = 0; it < N; ++it) {
      const bool on_a = on[it] && ((wa >> site[it]) & 1ull), on_b = on[it] && ((wb >> site[it]) & 1ull);
      lin_b[it] = zerov<VEC>();
      if (OP == kEwMul || OP == kEwAdd) {
        lin[it] = on_a ? ldv<VEC>(&pa[q[it] * C + c[it]]) : zerov<VEC>();
        lin_b[it] = on_b ? ldv<VEC>(&pb[q[it] * C + c[it]]) : zerov<VEC>();
      } else if (OP == kEwConcat) {
        const int ca = p.ga.c, cb = p.gb.c;  // (VEC 4: c_a % 4 == 0, a vector never straddles the two inputs)
        const bool of_a = c[it] < ca;
        lin[it] = (of_a ? on_a : on_b) ? ldv<VEC>(of_a ? &pa[q[it] * ca + c[it]] : &pb[q[it] * cb + c[it] - ca]) : zerov<VEC>();
      } else if (OP == kEwAct || OP == kEwPoolAcc || OP == kEwSparsify) {
        lin[it] = on[it] ? ldv<VEC>(&pa[q[it] * C + c[it]]) : zerov<VEC>();
      }
    }
    constexpr bool STATE = OP == kEwMul || OP == kEwPoolMax || OP == kEwPoolAcc || OP == kEwAdd || OP == kEwAct || ACT;
    const float sp_k = OP == kEwSparsify && !dense ? *at_stream(p.step, so) : 0.0f;
    const bool reads_z = OP == kEwPoolMax || (OP == kEwSparsify ? sp_k > 0.0f : STATE && !dense && (OP == kEwMul || OP == kEwPoolAcc || p.keeps_z));
    if (STATE || OP == kEwSparsify) {
#pragma unroll
      for (int it = 0; it < N; ++it) z_old[it] = on[it] && reads_z ? ldv<VEC>(&pz[q[it] * C + c[it]]) : zerov<VEC>();
    }
    if (OP == kEwMul) {
#pragma unroll
      for (int it = 0; it < N; ++it) z2_old[it] = on[it] && !dense ? ldv<VEC>(&pz2[q[it] * C + c[it]]) : zerov<VEC>();
    }
    if (UP) {
      // bilinear x2 of the stored tensor (half-pixel centres, clamped borders): the four sources of a site
      const int CA = p.ga.c;  // channels of the stored tensor (== C for a bare up-sampling)
#pragma unroll
      for (int it = 0; it < N; ++it) {
        const int ly = site[it] >> 3, lx = site[it] & 7;
        const int oy = tile_y * 8 + ly, ox = tile_x * 8 + lx;
        const int iy = oy >> 1, ix = ox >> 1;
        const int y0 = (oy & 1) ? iy : max(iy - 1, 0), y1 = (oy & 1) ? min(iy + 1, p.ga.h - 1) : iy;
        const int x0 = (ox & 1) ? ix : max(ix - 1, 0), x1 = (ox & 1) ? min(ix + 1, p.ga.w - 1) : ix;
        const float wy0 = (oy & 1) ? 0.75f : 0.25f, wy1 = 1.0f - wy0;
        const float wx0 = (ox & 1) ? 0.75f : 0.25f, wx1 = 1.0f - wx0;
        const int by = tile_y * 4 - 1, bx = tile_x * 4 - 1;
        // (the exchange between lanes stands before the branch: it needs all of them)
        const unsigned s0 = row_of_lane(src_rows, y0 - by), s1 = row_of_lane(src_rows, y1 - by);
        const unsigned r0 = dense ? ~0u : s0, r1 = dense ? ~0u : s1;
        if (OP == kEwConcatUp && c[it] >= CA) {  // the second operand's channels (VEC 4: c_a % 4 == 0, a vector is on one side)
          const bool on_b = on[it] && ((wb >> site[it]) & 1ull);
          lin[it] = on_b ? ldv<VEC>(&pb[q[it] * p.gb.c + c[it] - CA]) : zerov<VEC>();
          continue;
        }
        auto source = [&](unsigned row, int y, int x) {
          return on[it] && ((row >> (x - bx)) & 1u) ? ldv<VEC>(&pa[((size_t)y * p.ga.w + x) * CA + c[it]]) : zerov<VEC>();
        };
        const VecT<VEC> v00 = source(r0, y0, x0), v01 = source(r0, y0, x1), v10 = source(r1, y1, x0), v11 = source(r1, y1, x1);
#pragma unroll
        for (int i = 0; i < VEC; ++i)
          lin[it].v[i] = wy0 * (wx0 * v00.v[i] + wx1 * v01.v[i]) + wy1 * (wx0 * v10.v[i] + wx1 * v11.v[i]);
      }
    }
    if (OP == kEwPoolMax) {  // pa is the accumulated pool input, pz the cached window maximum
#pragma unroll
      for (int it = 0; it < N; ++it) {
        const int oy = tile_y * 8 + (site[it] >> 3), ox = tile_x * 8 + (site[it] & 7);
#pragma unroll
        for (int i = 0; i < VEC; ++i) lin[it].v[i] = -INFINITY;
        if (!on[it] || p.k != 3) continue;
        // the usual window: nine loads requested together (an out-of-image tap reads the window's
        // centre instead and is left out of the maximum), then the maxima in the same order
        const int cy = min(max(oy * p.stride - p.pad + 1, 0), p.ga.h - 1), cx = min(max(ox * p.stride - p.pad + 1, 0), p.ga.w - 1);
        VecT<VEC> t[9];
        bool ok[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) {
          const int iy = oy * p.stride - p.pad + j / 3, ix = ox * p.stride - p.pad + j % 3;
          ok[j] = (unsigned)iy < (unsigned)p.ga.h && (unsigned)ix < (unsigned)p.ga.w;
          t[j] = ldv<VEC>(&pa[((size_t)(ok[j] ? iy : cy) * p.ga.w + (ok[j] ? ix : cx)) * C + c[it]]);
        }
#pragma unroll
        for (int j = 0; j < 9; ++j)
#pragma unroll
          for (int i = 0; i < VEC; ++i) lin[it].v[i] = ok[j] ? fmaxf(lin[it].v[i], t[j].v[i]) : lin[it].v[i];
      }
      // other windows: tap by tap, the elements of a thread together
      if (p.k != 3) {
        for (int ky = 0; ky < p.k; ++ky)
          for (int kx = 0; kx < p.k; ++kx) {
            VecT<VEC> t[N];
            bool ok[N];
#pragma unroll
            for (int it = 0; it < N; ++it) {
              const int iy = (tile_y * 8 + (site[it] >> 3)) * p.stride - p.pad + ky, ix = (tile_x * 8 + (site[it] & 7)) * p.stride - p.pad + kx;
              ok[it] = on[it] && (unsigned)iy < (unsigned)p.ga.h && (unsigned)ix < (unsigned)p.ga.w;
              t[it] = ok[it] ? ldv<VEC>(&pa[((size_t)iy * p.ga.w + ix) * C + c[it]]) : zerov<VEC>();
            }
#pragma unroll
            for (int it = 0; it < N; ++it)
#pragma unroll
              for (int i = 0; i < VEC; ++i) lin[it].v[i] = ok[it] ? fmaxf(lin[it].v[i], t[it].v[i]) : lin[it].v[i];
          }
      }
    }

    // ---- results, state, and the sites at which this thread produced a nonzero element
#pragma unroll
    for (int it = 0; it < N; ++it) {
      if (!on[it]) continue;
      float* const zq = &pz[q[it] * C + c[it]];
      VecT<VEC> o = lin[it];
      if (OP == kEwAdd) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) o.v[i] = lin[it].v[i] + lin_b[it].v[i];
      }
      if (OP == kEwPoolAcc) {
        // (a regular pass stores the value as it is: x + 0 is not x for x = -0)
#pragma unroll
        for (int i = 0; i < VEC; ++i) o.v[i] = dense ? lin[it].v[i] : z_old[it].v[i] + lin[it].v[i];
        stv<VEC>(zq, o);
        continue;
      }
      if (OP == kEwMul) {
        // Eq.15-17: y_inc = (x1acc + x1_inc) * x2_inc + x2acc * x1_inc, then both accumulators
        // advance.  Explicitly rounded operations: no fused multiply-add, so the result is the
        // same single-rounded sequence on any implementation.
#pragma clang fp contract(off)
        VecT<VEC> n1 = lin[it], n2 = lin_b[it];
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          if (dense) {
            o.v[i] = lin[it].v[i] * lin_b[it].v[i];
          } else {
            n1.v[i] = z_old[it].v[i] + lin[it].v[i];
            n2.v[i] = z2_old[it].v[i] + lin_b[it].v[i];
            const float t1 = n1.v[i] * lin_b[it].v[i], t2 = z2_old[it].v[i] * lin[it].v[i];
            o.v[i] = t1 + t2;
          }
        }
        stv<VEC>(zq, n1);
        stv<VEC>(&pz2[q[it] * C + c[it]], n2);
      } else if (OP == kEwSparsify) {
        // Eq.3-8: x_corr = delta + x_inc; y_inc = k floor(0.5 + x_corr / k); delta = x_corr - y_inc
        VecT<VEC> d_new = zerov<VEC>();
        if (sp_k > 0.0f) {
#pragma clang fp contract(off)  // the residual is x_corr minus the rounded product, not a fused form
#pragma unroll
          for (int i = 0; i < VEC; ++i) {
            // (an element with a zero increment emits nothing and keeps its residual: |delta| <= k/2)
            const float x_corr = z_old[it].v[i] + lin[it].v[i];
            const bool moved = lin[it].v[i] != 0.0f;
            o.v[i] = moved ? sp_k * floorf(0.5f + x_corr / sp_k) : 0.0f;
            d_new.v[i] = moved ? x_corr - o.v[i] : z_old[it].v[i];
          }
        }
        if (dense || sp_k > 0.0f) stv<VEC>(zq, d_new);  // a refresh clears the residual
      } else if (OP == kEwPoolMax) {
        stv<VEC>(zq, lin[it]);
#pragma unroll
        for (int i = 0; i < VEC; ++i) o.v[i] = dense ? lin[it].v[i] : lin[it].v[i] - z_old[it].v[i];
      } else if (ACT || ((OP == kEwAdd || OP == kEwAct) && p.keeps_z)) {
        VecT<VEC> z_new = o;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          const float x = o.v[i];
          if (dense) {
            o.v[i] = apply_act(p.act, x);
          } else {
            z_new.v[i] = z_old[it].v[i] + x;
            o.v[i] = (p.act == kActNone) ? x : apply_act(p.act, z_new.v[i]) - apply_act(p.act, z_old[it].v[i]);
          }
        }
        stv<VEC>(zq, z_new);
      }
      stv<VEC>(&pout[q[it] * C + c[it]], o);
      bool nz = false;
#pragma unroll
      for (int i = 0; i < VEC; ++i) nz |= (o.v[i] != 0.0f);
      if (nz) nz_sites |= 1ull << site[it];
    }
    if (N != 2 || ew_in_flight(OP, VEC) != 2) break;  // (a workgroup has no more)
  }
  if (OP == kEwPoolAcc) return;
  if (p.structural || dense) {
    if (tid == 0 && blockIdx.y == 0) {
      at_stream(p.occ_out, so)[tile] = word;
      at_stream(p.occ_touched, so)[tile] = word;
    }
    return;
  }
  // the waves' ORs meet in LDS (one LDS atomic per element would be served lane by lane where the lanes
  // share a site)
  __shared__ uint64_t s_nz[4];
  unsigned lo = (unsigned)nz_sites, hi = (unsigned)(nz_sites >> 32);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    lo |= __shfl_xor(lo, m);
    hi |= __shfl_xor(hi, m);
  }
  if (lane == 0) s_nz[tid >> 6] = (uint64_t)lo | ((uint64_t)hi << 32);
  __syncthreads();
  if (tid == 0) {
    const uint64_t flags = (s_nz[0] | s_nz[1]) | (s_nz[2] | s_nz[3]);
    if (flags) atomicOr((unsigned long long*)&at_stream(p.occ_out, so)[tile], (unsigned long long)flags);  // pre-zeroed word
    if (blockIdx.y == 0) at_stream(p.occ_touched, so)[tile] = word;
  }
}

// Concatenation, without an activation, of operands whose channel counts are not multiples of four (Eq.11: the
// structural OR of the two active sets).  An operand's channels are taken four at a time all the same: 16-byte
// accesses need dword alignment only, and the last one to three channels of a site go singly.  A site's run of floats is
// one workgroup's, up to kConcatItems pieces.  Bound by HBM; with single floats, in runs of 16 channels that begin
// anywhere in a line, 5 + 64 channels on 256 x 352, every site active, 18.5 us, now 10.8 (4.6 TB/s; in a ConvLSTM's
// step 12.8).
constexpr int kConcatItems = 32;
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void concat_ragged_kernel(EwParams p) {
  touch_params<EwParams>();
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  const float* const pa = at_stream(p.a, so);
  const float* const pb = at_stream(p.b, so);
  float* const pout = at_stream(p.out, so);
  const bool dense = p.dense != 0;
  const int tid = threadIdx.x, lane = tid & 63, tile = blockIdx.x;
  const int tile_y = p.tx_magic ? (int)__umulhi((unsigned)tile, p.tx_magic) : tile / p.go.tx, tile_x = tile - tile_y * p.go.tx;
  const uint64_t inb = inbounds_word(p.go.h, p.go.w, tile_y, tile_x);
  const uint64_t wa = dense ? ~0ull : at_stream(p.occ_a, so)[tile], wb = dense ? ~0ull : at_stream(p.occ_b, so)[tile];
  const uint64_t word = dense ? inb : wa | wb;
  if (word == 0) return;
  const int ca = p.ga.c, cb = p.gb.c, C = p.go.c, na = (ca + 3) >> 2;
  // pieces [i0, i0 + ni) of every touched site belong to this workgroup
  const int i0 = blockIdx.y * p.vec_per_block, ni = min(p.vec_per_block, na + ((cb + 3) >> 2) - i0);
  const int ni_magic = (65536 + ni - 1) / ni;  // e / ni == (e * ni_magic) >> 16 for e < 2048 (ni <= 32)
  const int n_sites = __popcll(word), total = n_sites * ni;
  // lane r: the r-th touched site
  const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(word >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)word, 0u));
  const int nth = __builtin_amdgcn_ds_permute((((word >> lane) & 1ull) ? below : n_sites + lane - below) * 4, lane);
  constexpr int N = 4;
  for (int e0 = __builtin_amdgcn_readfirstlane(tid >> 6) * 64; e0 < total; e0 += N * 256) {
    float4 v[N];
    float* to[N];
    int n[N];  // floats of the piece, 0: none
#pragma unroll
    for (int it = 0; it < N; ++it) {
      const int e = e0 + lane + it * 256, r = (int)(__umul24(e, ni_magic) >> 16);
      const int site = __builtin_amdgcn_ds_bpermute(r * 4, nth);  // (r counts modulo 64)
      const int i = i0 + e - __umul24(r, ni), q = (tile_y * 8 + (site >> 3)) * p.go.w + tile_x * 8 + (site & 7);
      const bool of_a = i < na;
      const int c = (of_a ? i : i - na) * 4, cn = of_a ? ca : cb;
      const float* const from = (of_a ? pa : pb) + ((size_t)q * cn + c);
      const bool on = e < total && (((of_a ? wa : wb) >> site) & 1ull);
      n[it] = e < total ? min(4, cn - c) : 0;
      to[it] = pout + ((size_t)q * C + (of_a ? c : ca + c));
      v[it] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (on && n[it] == 4) {
        const floatx4u x = *(const floatx4u*)from;
        v[it] = make_float4(x.x, x.y, x.z, x.w);
      } else if (on) {
        v[it].x = from[0];
        if (n[it] > 1) v[it].y = from[1];
        if (n[it] > 2) v[it].z = from[2];
      }
    }
#pragma unroll
    for (int it = 0; it < N; ++it) {
      if (n[it] == 4) {
        *(floatx4u*)to[it] = floatx4u{v[it].x, v[it].y, v[it].z, v[it].w};
      } else {
        if (n[it] > 0) to[it][0] = v[it].x;
        if (n[it] > 1) to[it][1] = v[it].y;
        if (n[it] > 2) to[it][2] = v[it].z;
      }
    }
  }
  if (tid == 0 && blockIdx.y == 0) {
    at_stream(p.occ_out, so)[tile] = word;
    at_stream(p.occ_touched, so)[tile] = word;
  }
}

template <int OP, int VEC>
void launch_ew(const EwParams& q, const dim3& grid, hipStream_t s) {
  constexpr int kMax = ew_in_flight(OP, VEC);
  const int n = std::min((std::min(q.vec_per_block, q.go.c / VEC) * 64 + 255) / 256, kMax);  // elements of a thread
  if (n <= 1) hipLaunchKernelGGL((elementwise_kernel<OP, VEC, 1>), grid, dim3(256), 0, s, q);
  else if (n <= 2) hipLaunchKernelGGL((elementwise_kernel<OP, VEC, 2>), grid, dim3(256), 0, s, q);
  else hipLaunchKernelGGL((elementwise_kernel<OP, VEC, kMax>), grid, dim3(256), 0, s, q);
}

template <int OP, int VEC>
void launch_ew_act(const EwParams& q, const dim3& grid, hipStream_t s) {
  hipLaunchKernelGGL((elementwise_kernel<OP, VEC, ew_in_flight(OP, VEC), true>), grid, dim3(256), 0, s, q);
}

void launch_elementwise(const EwParams& p, hipStream_t s) {
  bool vec4 = (p.go.c % 4) == 0;
  if (p.op == kEwConcat || p.op == kEwConcatUp) vec4 = vec4 && (p.ga.c % 4) == 0;
  // Maps of few tiles are split over the channels, down to one pass of the 256 threads over a full tile
  // (4 vectors of 64 sites), until there are 384 workgroups: ResNet-18's 56 x 56 x 64 max-pool, 49
  // workgroups of four passes in sequence, 11.8 -> 6.8 us.  More cost sparse steps more than they give
  // dense ones (three nodes on 32 x 44 x 512 with 5 % of the sites active: 21.5 us in 192 workgroups, 22.8 in 384,
  // 26.8 in 768; on 64 x 88 x 128, all sites: 37.5 in 176, 28.9 in 352, 25.8 in 704).
  EwParams q = p;
  const bool act = (p.op == kEwConcat || p.op == kEwConcatUp || p.op == kEwUp2x) && p.act != kActNone;
  // Ragged concatenations in pieces of four channels from 2 Mi values on: below that the latency of a workgroup
  // counts, which is longer (single floats / pieces, every site active and 2 % of them: 5 + 64 channels on 256 x 352
  // 18.5 / 10.8 and 6.4 / 4.2 us, 33 + 31 14.8 / 12.2 and 5.7 / 4.6; 6 + 10 there 5.6 / 6.2 and 3.7 / 4.3, 3 + 3 4.6 / 5.5 and 3.4 / 4.8,
  // 255 + 2 on 64 x 88 5.9 / 6.0 and 4.0 / 4.0, 33 + 31 3.6 / 4.1 and 3.0 / 3.7).
  const bool ragged_concat = p.op == kEwConcat && !vec4 && !act && (long long)p.go.sites() * p.st.n * p.go.c >= 2 << 20;
  const int cv_all = ragged_concat ? (p.ga.c + 3) / 4 + (p.gb.c + 3) / 4 : p.go.c / (vec4 ? 4 : 1);
  q.vec_per_block = ragged_concat ? kConcatItems : kEwVecPerBlock;
  while (q.vec_per_block > kEwVecPerBlock / 4 &&
         (long long)p.go.tiles() * ((cv_all + q.vec_per_block - 1) / q.vec_per_block) * p.st.n < 384)
    q.vec_per_block /= 2;
  dim3 grid(p.go.tiles(), (cv_all + q.vec_per_block - 1) / q.vec_per_block, p.st.n);
  q.tx_magic = p.go.tx == 1 || (long long)p.go.tiles() * p.go.tx >= (1ll << 32)
                   ? 0u : (unsigned)((0x100000000ull + (unsigned)p.go.tx - 1) / (unsigned)p.go.tx);
  if (ragged_concat) {
    hipLaunchKernelGGL(concat_ragged_kernel, grid, dim3(256), 0, s, q);
    return;
  }
  if (act) {
    // (one variant each: such nodes are rare)
#define EVK_EW_ACT(OP) case OP: if (vec4) launch_ew_act<OP, 4>(q, grid, s); else launch_ew_act<OP, 1>(q, grid, s); break;
    switch (p.op) { EVK_EW_ACT(kEwConcat) EVK_EW_ACT(kEwConcatUp) EVK_EW_ACT(kEwUp2x) }
#undef EVK_EW_ACT
    return;
  }
#define EVK_EW(OP) case OP: if (vec4) launch_ew<OP, 4>(q, grid, s); else launch_ew<OP, 1>(q, grid, s); break;
  switch (p.op) {
    EVK_EW(kEwAdd) EVK_EW(kEwAct) EVK_EW(kEwConcat) EVK_EW(kEwUp2x) EVK_EW(kEwPoolAcc) EVK_EW(kEwPoolMax) EVK_EW(kEwSparsify)
    EVK_EW(kEwMul) EVK_EW(kEwConcatUp)
  }
#undef EVK_EW
}

// =============================================================================== global avg pool
// Workgroup = 64 channels x 4 row slices: slice s sums the active sites of tile rows s and s + 4
// of every tile, a row's eight loads in flight together; the four partial sums are added in a
// fixed order.  Sites are visited in a fixed order throughout, so the fp32 sum is reproducible.
__global__ __launch_bounds__(256) void gap_kernel(GapParams p) {
  touch_params<GapParams>();
  {
    const size_t so = (size_t)blockIdx.z * p.st.stride;
    p.a = at_stream(p.a, so); p.occ_a = at_stream(p.occ_a, so); p.z = at_stream(p.z, so);
    p.out = at_stream(p.out, so); p.occ_out = at_stream(p.occ_out, so); p.occ_touched = at_stream(p.occ_touched, so);
  }
  __shared__ float s_part[4][64];
  const int cl = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + cl;
  const int C = p.ga.c;
  const bool c_ok = c < C;
  bool any = false;
  float sum = 0.0f;
  for (int t = 0; t < p.ga.tiles(); ++t) {
    const int tile_y = t / p.ga.tx, tile_x = t - tile_y * p.ga.tx;
    const uint64_t w = p.dense ? inbounds_word(p.ga.h, p.ga.w, tile_y, tile_x) : p.occ_a[t];
    any |= (w != 0);
    for (int r = slice; r < 8; r += 4) {
      const unsigned bits = (unsigned)(w >> (8 * r)) & 0xffu;
      if (bits == 0) continue;
      const int y = tile_y * 8 + r;
      float v[8];
#pragma unroll
      for (int x = 0; x < 8; ++x)
        v[x] = (((bits >> x) & 1u) && c_ok) ? p.a[((size_t)y * p.ga.w + tile_x * 8 + x) * C + c] : 0.0f;
#pragma unroll
      for (int x = 0; x < 8; ++x) sum += v[x];
    }
  }
  if (!any) return;  // (the same for every thread)
  s_part[slice][cl] = sum;
  __syncthreads();
  if (slice != 0) return;
  bool nz = false;
  if (c_ok) {
    const float lin = ((s_part[0][cl] + s_part[1][cl]) + (s_part[2][cl] + s_part[3][cl])) / (float)(p.ga.h * p.ga.w);
    float o;
    if (p.dense) {
      p.z[c] = lin;
      o = apply_act(p.act, lin);
    } else {
      const float z_old = p.z[c], z_new = z_old + lin;
      p.z[c] = z_new;
      o = (p.act == kActNone) ? lin : apply_act(p.act, z_new) - apply_act(p.act, z_old);
    }
    p.out[c] = o;
    nz = (o != 0.0f);
  }
  const bool structural = (p.act == kActNone) || p.dense;
  const uint64_t b = __ballot(nz);
  if (cl == 0) {
    if (structural) { if (c == 0) p.occ_out[0] = 1ull; }
    else if (b) atomicOr((unsigned long long*)p.occ_out, 1ull);
    if (c == 0) p.occ_touched[0] = 1ull;
  }
}

void launch_gap(const GapParams& p, hipStream_t s) {
  hipLaunchKernelGGL(gap_kernel, dim3((p.ga.c + 63) / 64, 1, p.st.n), dim3(256), 0, s, p);
}

// =============================================================================== recurrent state
// Workgroup = one 8 x 8 tile; thread = (site, channel vector) pairs strided over the tile's active
// sites.  Bound by HBM (reads the delayed increment and the state, writes both).
template <int VEC>
__global__ __launch_bounds__(256) void delay_kernel(DelayParams p) {
  touch_params<DelayParams>();
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  const float* src = at_stream(p.src_out, so);
  float* z = at_stream(p.z, so);
  float* out = at_stream(p.out, so);
  const int tile = blockIdx.x;
  const int tile_y = tile / p.g.tx, tile_x = tile - tile_y * p.g.tx;
  const uint64_t inb = inbounds_word(p.g.h, p.g.w, tile_y, tile_x);
  const uint64_t saved = at_stream(p.occ_saved, so)[tile] & inb;
  // sites visited: all of the tile in or after a regular pass, the delayed node's active set otherwise
  const uint64_t word = (p.dense || p.last_dense) ? inb : saved;
  if (threadIdx.x == 0) {  // this workgroup is the tile's only writer
    at_stream(p.occ_out, so)[tile] = word;
    at_stream(p.occ_touched, so)[tile] = word;
  }
  const int C = p.g.c, cv = C / VEC;
  const int n_active = __popcll(word);
  __shared__ unsigned char s_site[64];  // the visited sites in ascending order
  if (threadIdx.x < 64 && ((word >> threadIdx.x) & 1ull))
    s_site[__popcll(word & ((1ull << threadIdx.x) - 1ull))] = (unsigned char)threadIdx.x;
  __syncthreads();
  for (int e = threadIdx.x; e < n_active * cv; e += 256) {
    const int k = p.cv_magic ? (int)__umulhi((unsigned)e, p.cv_magic) : e / cv, c = (e - k * cv) * VEC;
    const int site = s_site[k];
    const int oy = tile_y * 8 + (site >> 3), ox = tile_x * 8 + (site & 7);
    const size_t q = ((size_t)oy * p.g.w + ox) * C + c;
    VecT<VEC> o, n;
    if (p.dense) {
      o = zerov<VEC>();
      if (!p.zero_state) {
        if (p.last_dense) {
          o = ldv<VEC>(&src[q]);
        } else {
          const VecT<VEC> zo = ldv<VEC>(&z[q]);
          const VecT<VEC> d = ((saved >> site) & 1ull) ? ldv<VEC>(&src[q]) : zerov<VEC>();
#pragma unroll
          for (int i = 0; i < VEC; ++i) o.v[i] = zo.v[i] + d.v[i];
        }
      }
      n = o;
    } else {
      const VecT<VEC> zo = ldv<VEC>(&z[q]), x = ldv<VEC>(&src[q]);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        o.v[i] = p.last_dense ? x.v[i] - zo.v[i] : x.v[i];
        n.v[i] = zo.v[i] + o.v[i];
      }
    }
    stv<VEC>(&out[q], o);
    stv<VEC>(&z[q], n);
  }
}

void launch_delay(const DelayParams& p, hipStream_t s) {
  const dim3 grid(p.g.tiles(), 1, p.st.n);
  const bool vec4 = p.g.c % 4 == 0;
  const int cv = p.g.c / (vec4 ? 4 : 1);
  DelayParams q = p;
  // e / cv by a factor, exact while e * cv < 2^32 (e < 64 * cv)
  q.cv_magic = cv > 1 && cv < 8192 ? (unsigned)((0x100000000ull + (unsigned)cv - 1) / (unsigned)cv) : 0u;
  if (vec4) hipLaunchKernelGGL(delay_kernel<4>, grid, dim3(256), 0, s, q);
  else hipLaunchKernelGGL(delay_kernel<1>, grid, dim3(256), 0, s, q);
}

__global__ __launch_bounds__(256) void copy_u64_kernel(uint64_t* dst, const uint64_t* src, size_t n, size_t stride) {
  const size_t so = (size_t)blockIdx.y * stride;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) at_stream(dst, so)[i] = at_stream(src, so)[i];
}

void launch_copy_u64(uint64_t* dst, const uint64_t* src, size_t n, Streams st, hipStream_t s) {
  hipLaunchKernelGGL(copy_u64_kernel, dim3((unsigned)((n + 255) / 256), st.n), dim3(256), 0, s, dst, src, n, st.stride);
}

// =============================================================================== end of a pass
// One launch at the end of a pass: the output integrations (Eq.2) and the ordered lists of all
// sets.  They depend on the nodes' results only, not on each other, and as launches of their own
// they were 4 us each with about 2 us between them.

// One element of the public tensors; on: the site is in the active set.
struct IntegrateAt {
  const float __attribute__((address_space(1)))* delta;
  const uint64_t __attribute__((address_space(1)))* occ;
  float __attribute__((address_space(1)))* y;
  float __attribute__((address_space(1)))* dy;
  int h, w, c, tx;
};
__device__ __forceinline__ void integrate_element(const IntegrateAt& p, int mode, int e, float v, bool on) {
  if (mode == kIntStep) {
    if (on) p.y[e] += v;
    p.dy[e] = v;
  } else if (mode == kIntReset) {
    p.y[e] = v;
    p.dy[e] = 0.0f;
  } else {
    p.dy[e] = v - p.y[e];
    p.y[e] = v;
  }
}

// Block `b` of an output's integration.  Up to 4 channels: 512 sites, a thread each; more: 64 sites x
// 32 channels, read in runs of a site's channels and turned through LDS to be written in runs of
// sites.  (One thread per site walked the channels one round trip after the other: 101 channels
// on one site 35 us.)
constexpr int kIntFew = 4, kIntChannels = 32;
constexpr long long kIntSparseReads = 12ll << 20;  // elements
template <bool LARGE>
__device__ __forceinline__ void integrate_block(const IntegrateAt& p, int mode, int b) {
  __shared__ float s_v[64][kIntChannels + 1];
  const int hw = p.h * p.w, C = p.c, tid = threadIdx.x;
  if (C <= kIntFew) {
    const int site = b * 512 + tid;
    if (site >= hw) return;
    const int y = site / p.w, x = site - y * p.w;
    const bool on = mode != kIntStep || occ_bit(p.occ, p.tx, y, x);
    float v[kIntFew];
#pragma unroll
    for (int c = 0; c < kIntFew; ++c) v[c] = on && c < C ? p.delta[(size_t)site * C + c] : 0.0f;
#pragma unroll
    for (int c = 0; c < kIntFew; ++c)
      if (c < C) integrate_element(p, mode, c * hw + site, v[c], on);
    return;
  }
  const int cb = (C + kIntChannels - 1) / kIntChannels;
  const int s0 = b / cb * 64, c0 = b % cb * kIntChannels;
  const int q = tid & 63, site = s0 + q;
  auto active = [&]() {
    const int y = site / p.w, x = site - y * p.w;
    return site < hw && (mode != kIntStep || occ_bit(p.occ, p.tx, y, x));
  };
  // A step needs the increments of the active sites only.  Waiting for the occupancy words before they
  // are requested pays where the increments come from HBM; smaller tensors lie in the caches and are
  // read alongside the words (2 % of the sites active, a step of one conv: 64 channels on 480 x 640, 79 MB, 224 us
  // reading all, 182 reading the active ones; on 260 x 346, 23 MB, 65.9 and 69.6).
  // LARGE: the net has such an output (a variant of its own: the test alone costs 0.2 us)
  const bool sparse_reads = LARGE && (long long)hw * C >= kIntSparseReads;
  const uint64_t wanted = sparse_reads ? __ballot(active()) : ~0ull;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = tid & (kIntChannels - 1), r = (tid >> 5) + 16 * i;
    s_v[r][c] = (s0 + r < hw && c0 + c < C && ((wanted >> r) & 1ull)) ? p.delta[(size_t)(s0 + r) * C + c0 + c] : 0.0f;
  }
  __syncthreads();
  const bool on = sparse_reads ? ((wanted >> q) & 1ull) != 0 : active();
  if (site >= hw) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = (tid >> 6) + 8 * i;
    if (c0 + c < C) integrate_element(p, mode, (c0 + c) * hw + site, on ? s_v[q][c] : 0.0f, on);
  }
}

bool integrate_large(int c, int sites) { return c > kIntFew && (long long)c * sites >= kIntSparseReads; }
int integrate_blocks(int c, int sites) {
  return c <= kIntFew ? (sites + 511) / 512 : (sites + 63) / 64 * ((c + kIntChannels - 1) / kIntChannels);
}

// Workgroup (strip, set): strip = one row of tiles = 8 image rows.  Its first list position is
// the number of active sites in all earlier strips (a reduction over their occupancy words);
// inside the strip wave r owns image row r and scans the per-tile byte popcounts with a
// wave-wide prefix sum, so indices come out strictly ascending in y*W + x.
// A recurrent net's delayed nodes have their words copied to SetDesc::save on the way.
// empty: the strip's words, and the set's count and bitmap become zeros.
__device__ __forceinline__ void lists_block(const SetDesc& d, int strip, size_t so, int save, int empty) {
  __shared__ int s_part[8];
  __shared__ int s_rowcnt[8];
  if (strip >= d.ty) return;
  const auto occ = as_global(at_stream(d.occ, so));
  const auto idx = as_global(at_stream(d.idx, so));
  const int tid = threadIdx.x, lane = tid & 63, r = tid >> 6;
  if (empty) {
    const int n_tiles = d.tx * d.ty;
    if (d.words) {
      const auto words = as_global(at_stream(d.words, so));
      for (int t = tid; t < d.tx; t += 512) words[strip * d.tx + t] = words[n_tiles + strip * d.tx + t] = 0;
    }
    if (strip == 0) {
      const auto bitmap = as_global(at_stream(d.bitmap, so));
      for (int t = tid; t < (n_tiles + 63) >> 6; t += 512) bitmap[t] = 0;
      if (tid == 0) *as_global(at_stream(d.count, so)) = 0;
    }
    return;
  }
  if (save && d.save) {
    const auto copy = as_global(at_stream(d.save, so));
    for (int t = tid; t < d.tx; t += 512) copy[strip * d.tx + t] = occ[strip * d.tx + t];
  }

  // active sites of the earlier strips, four words of a thread in flight
  int cnt = 0;
  const int before = strip * d.tx;
  for (int t = tid; t < before; t += 4 * 512) {
    uint64_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = t + i * 512 < before ? occ[t + i * 512] : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) cnt += __popcll(w[i]);
  }
  // row r of this strip: per-tile 8-bit masks (bytes of the words)
  const auto row_bytes = (const unsigned char __attribute__((address_space(1)))*)(occ + before) + r;
  unsigned byte = lane < d.tx ? row_bytes[lane * 8] : 0u;
  int incl = wave_scan(__popc(byte));
  int row_total = __builtin_amdgcn_readlane(incl, 63);
  for (int j0 = 64; j0 < d.tx; j0 += 64) {
    const int j = j0 + lane;
    row_total += __builtin_amdgcn_readlane(wave_scan(j < d.tx ? __popc((unsigned)row_bytes[j * 8]) : 0), 63);
  }
  cnt = __builtin_amdgcn_readlane(wave_scan(cnt), 63);
  if (lane == 0) { s_part[r] = cnt; s_rowcnt[r] = row_total; }
  __syncthreads();

  int base = 0;
  for (int i = 0; i < 8; ++i) base += s_part[i];
  int strip_total = 0;
  for (int i = 0; i < 8; ++i) {
    if (i < r) base += s_rowcnt[i];
    strip_total += s_rowcnt[i];
  }
  int running = base;  // list position of the first active site of row r
  const int y = strip * 8 + r;
  for (int j0 = 0;;) {
    int pos = running + incl - __popc(byte);
    const int at = y * d.w + (j0 + lane) * 8;
    while (byte) {
      const int bit = __ffs(byte) - 1;
      byte &= byte - 1;
      idx[pos++] = at + bit;
    }
    running += __builtin_amdgcn_readlane(incl, 63);
    j0 += 64;
    if (j0 >= d.tx) break;
    byte = j0 + lane < d.tx ? row_bytes[(j0 + lane) * 8] : 0u;
    incl = wave_scan(__popc(byte));
  }
  if (strip == d.ty - 1 && tid == 0) {
    int s = 0;
    for (int i = 0; i < 8; ++i) s += s_part[i];
    *as_global(at_stream(d.count, so)) = s + strip_total;
  }
  if (strip == 0) {  // tile bitmap: one ballot per 64 tiles
    const int n_tiles = d.tx * d.ty;
    const auto bitmap = as_global(at_stream(d.bitmap, so));
    for (int w0 = r * 64; w0 < n_tiles; w0 += 512) {
      const int t = w0 + lane;
      const uint64_t b = __ballot(t < n_tiles && occ[t] != 0);
      if (lane == 0) bitmap[w0 >> 6] = b;
    }
  }
}

template <bool LARGE>
__global__ __launch_bounds__(512) void finish_kernel(FinishParams p) {
  touch_params<FinishParams>();
  const size_t so = (size_t)blockIdx.y * p.st.stride;  // the descriptors hold stream 0's pointers
  const int total = p.int_blocks + p.n_sets * p.max_ty;
  for (int blk = blockIdx.x; blk < total; blk += gridDim.x) {
    if (blk < p.int_blocks) {
      int i = 0;
      while (i + 1 < p.n_outputs && blk >= p.outputs[i + 1].first_block) ++i;
      const IntegrateDesc& d = p.outputs[i];
      const IntegrateAt at = {as_global(at_stream(d.delta, so)), as_global(at_stream(d.occ, so)), as_global(at_stream(d.y, so)),
                              as_global(at_stream(d.dy, so)), d.h, d.w, d.c, d.tx};
      integrate_block<LARGE>(at, p.int_mode, blk - d.first_block);
    } else {
      const int b = blk - p.int_blocks, set = b / p.max_ty;
      lists_block(p.sets[set], b - set * p.max_ty, so, p.save, p.empty);
    }
    __syncthreads();  // (the next block reuses the shared memory)
  }
}

// The lists alone, for nets whose outputs are all integrated by their own kernels: 31 sets of 32
// strips 7.2 us, against 8.2 through the kernel above.
__global__ __launch_bounds__(512) void build_lists_kernel(const SetDesc* sets, size_t stream_stride, int save, int empty) {
  lists_block(sets[blockIdx.y], blockIdx.x, (size_t)blockIdx.z * stream_stride, save, empty);
}

void launch_finish(const FinishParams& p, hipStream_t s) {
  if (p.int_blocks == 0) {
    hipLaunchKernelGGL(build_lists_kernel, dim3(p.max_ty, p.n_sets, p.st.n), dim3(512), 0, s, p.sets, p.st.stride, p.save, p.empty);
    return;
  }
  // (a launch holds less than 2^32 threads; the loop takes what is left of a very tall input)
  const int blocks = std::min(p.int_blocks + p.n_sets * p.max_ty, 1 << 22);
  if (p.int_large) hipLaunchKernelGGL(finish_kernel<true>, dim3(blocks, p.st.n), dim3(512), 0, s, p);
  else hipLaunchKernelGGL(finish_kernel<false>, dim3(blocks, p.st.n), dim3(512), 0, s, p);
}

// =============================================================================== rounding step
// stage 1: block b sums the squares of its contiguous slice in a fixed order (thread-strided
// partials, then a shared-memory tree); stage 2: one block adds the kRmsBlocks partials the same
// way and writes k = tp * sqrt(sum / n) kept to 8 fraction bits.
__global__ __launch_bounds__(256) void rms_stage1_kernel(const float* x, size_t n, float* partial, size_t stream_stride) {
  x = at_stream(x, (size_t)blockIdx.y * stream_stride);
  partial = at_stream(partial, (size_t)blockIdx.y * stream_stride);
  __shared__ float s_sum[256];
  const size_t per = (n + kRmsBlocks - 1) / kRmsBlocks;
  const size_t lo = blockIdx.x * per, hi = min(n, lo + per);
  float acc = 0.0f;
  for (size_t i = lo + threadIdx.x; i < hi; i += 256) acc += x[i] * x[i];
  s_sum[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s_sum[threadIdx.x] += s_sum[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = s_sum[0];
}
__global__ __launch_bounds__(256) void rms_stage2_kernel(const float* partial, size_t n, float tp, float* step_out,
                                                        size_t stream_stride) {
  partial = at_stream(partial, (size_t)blockIdx.y * stream_stride);
  step_out = at_stream(step_out, (size_t)blockIdx.y * stream_stride);
  __shared__ float s_sum[256];
  s_sum[threadIdx.x] = threadIdx.x < kRmsBlocks ? partial[threadIdx.x] : 0.0f;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s_sum[threadIdx.x] += s_sum[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float k = tp * sqrtf(s_sum[0] / (float)n);
    unsigned u = __float_as_uint(k);
    u = (u + 0x4000u) & 0xffff8000u;
    *step_out = __uint_as_float(u);
  }
}
void launch_rms_step(const float* x, size_t n, float tp, float* partial, float* step_out, Streams st, hipStream_t s) {
  static_assert(kRmsBlocks == 256, "stage 2 adds one partial per thread");
  hipLaunchKernelGGL(rms_stage1_kernel, dim3(kRmsBlocks, st.n), dim3(256), 0, s, x, n, partial, st.stride);
  hipLaunchKernelGGL(rms_stage2_kernel, dim3(1, st.n), dim3(256), 0, s, partial, n, tp, step_out, st.stride);
}

__global__ void fill_u64_kernel(uint64_t* p, size_t n, uint64_t v, size_t stream_stride) {
  p = at_stream(p, (size_t)blockIdx.y * stream_stride);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
void launch_fill_u64(uint64_t* p, size_t n, uint64_t v, Streams st, hipStream_t s) {
  if (!n) return;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks, st.n), dim3(256), 0, s, p, n, v, st.stride);
}

}  // namespace evk
