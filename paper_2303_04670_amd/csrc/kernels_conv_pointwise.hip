// 1 x 1 convolutions with few output channels (prediction heads: c_out <= 8, stride 1, no
// padding) and LINEAR on a 1 x 1 grid (classifier).  Both are dot products per site, bound by
// reading the input increment: the matrix-core tiling (32 output channels per block) and the
// general vector kernel (a halo patch through LDS) would waste nearly all of their work here.
//
// conv_pointwise_few_kernel: workgroup = one 8 x 8 tile, four lanes per site.  Lane q of a site
//   reads the float4 channel groups q, q+4, q+8, ... of its site (the four lanes of a site read
//   64 contiguous bytes per step), multiplies by the matching weights [c_out][c_in] and the four
//   partial sums are added with two lane shuffles, in a fixed order.  T = S_in (Eq.13: a 1 x 1
//   window has no footprint); z read-modify-write, activation increment (Eq.12-14), occupancy
//   words as in the other convolution kernels.
// linear_site_kernel: one wavefront per output channel of the single site.
#include <cstddef>
#include <type_traits>

#include "evconv_kernels.h"

namespace evk {

namespace {

constexpr int kMaxFew = 8;  // output channels of the few-channel kernel

__device__ __forceinline__ float act_p(int act, float v) {
  if (act == kActRelu) return fmaxf(v, 0.0f);
  if (act == kActSigmoid) return 1.0f / (1.0f + expf(-v));
  if (act == kActTanh) return tanhf(v);
  if (act == kActOneMinus) return 1.0f - v;
  return v;
}

// z read-modify-write and output increment of one (site, channel) element
// (old_z: returns the old z)
template <class P, class F>
__device__ __forceinline__ float finish_element(const P& p, float* z, float* out, size_t q, int co, float v, F&& old_z) {
  float o;
  if (p.dense) {
    const float zn = v + (p.bias ? p.bias[co] : 0.0f);
    z[q] = zn;
    o = act_p(p.act, zn);
  } else {
    const float z_old = old_z(), z_new = z_old + v;
    z[q] = z_new;
    o = (p.act == kActNone) ? v : act_p(p.act, z_new) - act_p(p.act, z_old);
  }
  out[q] = o;
  return o;
}

// NOUT: output channels rounded up to 1, 2, 4 or 8 (rows beyond c_out repeat the last one and are not
// used), so that the loads of several channel pieces are in flight together: with a loop over c_out
// inside, a site's channels were a chain of round trips (256 channels on 32 x 32: 11.6 us, now 7.4).
// UNROLL pieces are in flight: four with eight rows take the registers of half the waves, which
// launches that fill the chip (more than 1024 tiles) need more; those take two, and exactly c_out
// rows (256 x 352: 16 -> 8 channels 17.9 us before, 25.2 with four pieces, 17.5 with two; 256 -> 5
// channels 34.6, 38.9, 30.4; 64 x 88, 88 tiles: 512 -> 8 channels 53.7, 25.6, 27.5).
// EARLY: the old values are requested before the dot products.  That keeps two more registers per row (four
// rows: 60 against 76, eight: 62 against 120), so it is not for regular passes, which read none
// (64 -> 8 channels on 512 x 700: 60.2 us early, 50.8 late), nor, on many tiles, for short dot products of
// more than two rows (30 -> 8 channels on 512 x 700, 2 % of the sites active: 40.1 and 33.5; 64 -> 8: 40.0
// early, 43.7 late).
template <int NOUT, int UNROLL, bool EARLY, class P>
__device__ __forceinline__ void few_tile(const P& p, const int tile) {
  asm volatile("" ::"s"(p.go.h), "s"(p.go.w), "s"(p.go.c), "s"(p.go.tx), "s"(p.gi.c), "s"(p.dense), "s"(p.occ_in), "s"(p.in), "s"(p.w), "s"(p.z),
               "s"(p.out), "s"(p.y), "s"(p.dy), "s"(p.int_mode), "s"(p.act), "s"(p.bias), "s"(p.st.stride), "s"(p.tx_magic));
  __shared__ unsigned s_nz[4];
  const size_t so = (size_t)blockIdx.z * p.st.stride;  // this workgroup's stream
  const int tid = threadIdx.x;
  const bool dense = p.dense != 0;
  // same geometry in and out: the touched word is the input's occupancy word
  const uint64_t word = dense ? ~0ull : at_stream(p.occ_in, so)[tile];
  const int tile_y = p.tx_magic ? (int)__umulhi((unsigned)tile, p.tx_magic) : tile / p.go.tx, tile_x = tile - tile_y * p.go.tx;
  const int site = tid >> 2, q4 = tid & 3;  // site inside the tile, lane inside the site's group of four
  const int oy = tile_y * 8 + (site >> 3), ox = tile_x * 8 + (site & 7);
  const bool inb = oy < p.go.h && ox < p.go.w;
  const int Cin = p.gi.c, Cout = p.go.c;
  // in-bounds mask of the tile, so that dense mode and ragged borders agree with `on`
  const int rows = min(8, p.go.h - tile_y * 8), cols = min(8, p.go.w - tile_x * 8);
  const uint64_t rowbits = cols >= 8 ? 0xffull : ((1ull << cols) - 1ull);
  const uint64_t touched_word = word & (rowbits * 0x0101010101010101ull) & (rows >= 8 ? ~0ull : ((1ull << (8 * rows)) - 1ull));
  const bool on = (touched_word >> site) & 1ull;
  // output node kept by this kernel: public tensors are C x H x W
  const int hw = p.go.h * p.go.w;
  float* const pub_y = p.y ? at_stream(p.y, so) : nullptr;
  float* const pub_dy = p.dy ? at_stream(p.dy, so) : nullptr;
  if (touched_word == 0) {
    // nothing changed under this tile: the increment of its sites is zero
    if (pub_dy && inb && q4 == 0)
      for (int j = 0; j < Cout; ++j) pub_dy[(size_t)j * hw + oy * p.go.w + ox] = 0.0f;
    return;
  }

  // old values of the elements this thread finishes, requested before the dot products (EARLY)
  const bool mine = inb && q4 == 0;
  float* const z = at_stream(p.z, so);
  float* const out = at_stream(p.out, so);
  const size_t q0 = ((size_t)oy * p.go.w + ox) * Cout, e0 = (size_t)oy * p.go.w + ox;
  const bool reads_y = pub_y && (p.int_mode == kIntStep ? on : p.int_mode != kIntReset);
  float z_early[NOUT], y_early[NOUT];
#pragma unroll
  for (int j = 0; j < NOUT; ++j) {
    z_early[j] = EARLY && mine && on && !dense && j < Cout ? z[q0 + j] : 0.0f;
    y_early[j] = EARLY && mine && reads_y && j < Cout ? pub_y[(size_t)j * hw + e0] : 0.0f;
  }

  float acc[NOUT];
#pragma unroll
  for (int j = 0; j < NOUT; ++j) acc[j] = 0.0f;
  if (on) {
    const float* __restrict__ x = at_stream(p.in, so) + ((size_t)oy * p.gi.w + ox) * Cin;
    const float* __restrict__ w = (const float*)p.w;  // [c_out][c_in]
    if ((Cin & 3) == 0) {
#pragma unroll UNROLL
      for (int c = q4 * 4; c < Cin; c += 16) {
        const float4 xv = *(const float4*)&x[c];
#pragma unroll
        for (int j = 0; j < NOUT; ++j) {
          const float4 wv = *(const float4*)&w[(size_t)min(j, Cout - 1) * Cin + c];
          acc[j] = fmaf(xv.x, wv.x, acc[j]);
          acc[j] = fmaf(xv.y, wv.y, acc[j]);
          acc[j] = fmaf(xv.z, wv.z, acc[j]);
          acc[j] = fmaf(xv.w, wv.w, acc[j]);
        }
      }
    } else {
      for (int c = q4; c < Cin; c += 4) {
        const float xv = x[c];
#pragma unroll
        for (int j = 0; j < NOUT; ++j) {
          acc[j] = fmaf(xv, w[(size_t)min(j, Cout - 1) * Cin + c], acc[j]);
        }
      }
    }
  }
  // add the four lanes of a site: (0 + 1) + (2 + 3), every lane ends with the full sum
#pragma unroll
  for (int j = 0; j < NOUT; ++j) {
    acc[j] += __shfl_xor(acc[j], 1);
    acc[j] += __shfl_xor(acc[j], 2);
  }
  bool nz = false;
  if (mine) {
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
      if (j >= Cout) break;
      float o = 0.0f;
      if (on) {
        o = finish_element(p, z, out, q0 + j, j, acc[j], [&] { return EARLY ? z_early[j] : z[q0 + j]; });
        nz |= o != 0.0f;
      }
      if (pub_y) {  // the step's output and its increment, as the stand-alone integration writes them
        const size_t e = (size_t)j * hw + e0;
        auto old_y = [&] { return EARLY ? y_early[j] : pub_y[e]; };
        if (p.int_mode == kIntStep) {
          if (on) pub_y[e] = old_y() + o;
          pub_dy[e] = o;
        } else if (p.int_mode == kIntReset) {
          pub_y[e] = o;
          pub_dy[e] = 0.0f;
        } else {
          pub_dy[e] = o - old_y();
          pub_y[e] = o;
        }
      }
    }
  }
  // a site's bit is that of the first of its four lanes: the wave's 16 bits, four apart, closed up
  uint64_t b = __ballot(nz) & 0x1111111111111111ull;
  b = (b | (b >> 3)) & 0x0303030303030303ull;
  b = (b | (b >> 6)) & 0x000f000f000f000full;
  b = (b | (b >> 12)) & 0x000000ff000000ffull;
  if ((tid & 63) == 0) s_nz[tid >> 6] = (unsigned)(b | (b >> 24)) & 0xffffu;
  __syncthreads();
  if (tid == 0) {
    const uint64_t s_out = dense ? touched_word : (s_nz[0] | (s_nz[1] << 16)) | ((uint64_t)(s_nz[2] | (s_nz[3] << 16)) << 32);
    at_stream(p.occ_out, so)[tile] = s_out;       // this workgroup is the tile's only writer
    at_stream(p.occ_touched, so)[tile] = touched_word;
  }
}

template <int NOUT, int UNROLL, bool EARLY>
__global__ __launch_bounds__(256) void conv_pointwise_few_kernel(ConvParams p) {
  touch_params<ConvParams>();
  few_tile<NOUT, UNROLL, EARLY>(p, blockIdx.x);
}

// Several heads in one launch: workgroups first[i] .. first[i + 1] - 1 are head i's tiles.  Nothing reads a
// prediction, so the heads of an encoder-decoder's scales need not stand between its layers: four
// launches of 6.2, 5.2, 5.0 and 6.2 us (32 x 32 to 256 x 256), in one 9.0.
struct HeadBatch { ConvParams p[kMaxHeadBatch]; int first[kMaxHeadBatch]; int n; };
template <int NOUT, int UNROLL, bool EARLY>
__global__ __launch_bounds__(256) void conv_pointwise_batch_kernel(HeadBatch q) {
  int i = 0;
#pragma unroll
  for (int j = 1; j < kMaxHeadBatch; ++j)
    if (j < q.n && (int)blockIdx.x >= q.first[j]) i = j;
  const unsigned args = (unsigned)(offsetof(HeadBatch, p) + i * sizeof(ConvParams));
  touch_params<ConvParams>(args);
  typedef const char __attribute__((address_space(4))) Byte;
  Byte* const base = (Byte*)__builtin_amdgcn_kernarg_segment_ptr();
  const int first = *(const int __attribute__((address_space(4)))*)(base + offsetof(HeadBatch, first) + i * sizeof(int));
  few_tile<NOUT, UNROLL, EARLY>(*(const ConvParams __attribute__((address_space(4)))*)(base + args), (int)blockIdx.x - first);
}

// one wavefront per output channel: the lanes stride through c_in (coalesced weight row), then a
// butterfly adds the 64 partial sums in a fixed order
__global__ __launch_bounds__(256) void linear_site_kernel(ConvParams p) {
  touch_params<ConvParams>();
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  const int lane = threadIdx.x & 63;
  const int co = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int Cin = p.gi.c, Cout = p.go.c;
  const bool active = p.dense || (at_stream(p.occ_in, so)[0] & 1ull);
  if (!active || co >= Cout) return;  // uniform per wavefront
  const float* __restrict__ x = at_stream(p.in, so);
  const float* __restrict__ w = (const float*)p.w + (size_t)co * Cin;  // [c_out][c_in]
  const float z_old = lane == 0 && !p.dense ? at_stream(p.z, so)[co] : 0.0f;  // (requested before the dot product)
  float acc = 0.0f;
  for (int c = lane; c < Cin; c += 8 * 64) {  // eight pieces in flight (beyond c_in: the last one again, not added)
    float xv[8], wv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ci = min(c + 64 * i, Cin - 1);
      xv[i] = x[ci];
      wv[i] = w[ci];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (c + 64 * i < Cin) acc = fmaf(xv[i], wv[i], acc);
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) acc += __shfl_xor(acc, m);
  if (lane == 0) {
    const bool nz = finish_element(p, at_stream(p.z, so), at_stream(p.out, so), (size_t)co, co, acc, [&] { return z_old; }) != 0.0f;
    // pre-zeroed words; the wavefronts of one launch OR their share in
    if (p.dense || nz) atomicOr((unsigned long long*)at_stream(p.occ_out, so), 1ull);
    if (co == 0) at_stream(p.occ_touched, so)[0] = 1ull;
  }
}

}  // namespace

bool conv_pointwise_integrates(const ConvParams& p) { return !(p.go.h == 1 && p.go.w == 1 && p.go.c > kMaxFew); }

bool conv_pointwise_supported(const ConvParams& p) {
  if (p.k != 1 || p.stride != 1 || p.pad != 0 || p.n_fused != 0) return false;
  if (p.gi.h != p.go.h || p.gi.w != p.go.w) return false;
  return p.go.c <= kMaxFew || (p.go.h == 1 && p.go.w == 1);
}

namespace {

// tiles per row as a factor (exact while the product fits 32 bits)
ConvParams with_magic(ConvParams p) {
  p.tx_magic = p.go.tx == 1 || (long long)p.go.tiles() * p.go.tx >= (1ll << 32)
                   ? 0u : (unsigned)((0x100000000ull + (unsigned)p.go.tx - 1) / (unsigned)p.go.tx);
  return p;
}

// calls f(rows, pieces in flight, old values early) with the variant that takes p, as compile-time values
// (the first two are the same in every pass of a net)
template <class F>
void with_few_variant(const ConvParams& p, F&& f) {
  using std::integral_constant;
  const bool many = (long long)p.go.tiles() * p.st.n > 1024;
  auto variant = [&](auto rows, auto pieces) {
    if (p.dense || (many && p.go.c > 2 && (p.gi.c % 4 != 0 || p.gi.c < 32))) f(rows, pieces, std::false_type{});
    else f(rows, pieces, std::true_type{});
  };
  if (p.go.c == 1) variant(integral_constant<int, 1>{}, integral_constant<int, 4>{});
  else if (p.go.c == 2) variant(integral_constant<int, 2>{}, integral_constant<int, 4>{});
  else if (!many && p.go.c <= 4) variant(integral_constant<int, 4>{}, integral_constant<int, 4>{});
  else if (!many) variant(integral_constant<int, 8>{}, integral_constant<int, 4>{});
  else if (p.go.c == 3) variant(integral_constant<int, 3>{}, integral_constant<int, 2>{});
  else if (p.go.c == 4) variant(integral_constant<int, 4>{}, integral_constant<int, 2>{});
  else if (p.go.c == 5) variant(integral_constant<int, 5>{}, integral_constant<int, 2>{});
  else if (p.go.c == 6) variant(integral_constant<int, 6>{}, integral_constant<int, 2>{});
  else if (p.go.c == 7) variant(integral_constant<int, 7>{}, integral_constant<int, 2>{});
  else variant(integral_constant<int, 8>{}, integral_constant<int, 2>{});
}

}  // namespace

void launch_conv_pointwise(const ConvParams& q, hipStream_t s) {
  const ConvParams p = with_magic(q);
  if (p.go.h == 1 && p.go.w == 1 && p.go.c > kMaxFew) {
    hipLaunchKernelGGL(linear_site_kernel, dim3((p.go.c + 3) / 4, 1, p.st.n), dim3(256), 0, s, p);
    return;
  }
  with_few_variant(p, [&](auto rows, auto pieces, auto early) {
    hipLaunchKernelGGL((conv_pointwise_few_kernel<decltype(rows)::value, decltype(pieces)::value, decltype(early)::value>),
                       dim3(p.go.tiles(), 1, p.st.n), dim3(256), 0, s, p);
  });
}

int conv_pointwise_variant(const ConvParams& p) {
  int v = 0;
  with_few_variant(p, [&](auto rows, auto pieces, auto) { v = rows() * 16 + pieces(); });
  return v;
}

void launch_conv_pointwise_batch(const ConvParams* heads, int n, hipStream_t s) {
  HeadBatch q = {};
  int blocks = 0;
  for (int i = 0; i < n; ++i) {
    q.p[i] = with_magic(heads[i]);
    q.first[i] = blocks;
    blocks += heads[i].go.tiles();
  }
  q.n = n;
  with_few_variant(heads[0], [&](auto rows, auto pieces, auto early) {
    hipLaunchKernelGGL((conv_pointwise_batch_kernel<decltype(rows)::value, decltype(pieces)::value, decltype(early)::value>),
                       dim3(blocks, 1, heads[0].st.n), dim3(256), 0, s, q);
  });
}

}  // namespace evk
