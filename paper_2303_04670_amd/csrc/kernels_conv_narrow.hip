// Sparse incremental convolution for narrow inputs, on the matrix cores.
//
// For layers whose whole contraction K = taps x c_in is at most 128 and whose c_out is at least 16
// (the last block of 32 output channels is zero-padded): the first convolution on the event tensor
// (c_in = 2..8 channels).  With so few input channels a per-tap channel contraction is too thin
// for an MFMA, so the contraction runs over the flattened index k = tap * c_in + ci (im2col by
// addressing, nothing is materialised):
//   A[m][k] = patch[site(m) + tap offset(k)][ci(k)]   one ds_read_b32 at a per-lane offset that is
//             worked out once per workgroup and kept in registers (one register per MFMA step)
//   B[k][n] = the weights, re-laid on the host so that a lane's values for all steps are
//             contiguous; a wave keeps its whole share in registers while it walks tiles
// v_mfma_f32_16x16x4_f32, fp32 operands and accumulation (bf16-declared weights are widened, which
// is at least as accurate as the bf16 path).
//
// Workgroup = 4 waves = one 8 x 8 output tile x 32 output channels; wave = a half tile (four
// rows, 32 sites) x 16 channels as two 16 x 16 accumulator blocks that share the weight operand:
// no partial sums, and the epilogue goes straight from the accumulator registers to memory.
// Workgroups walk tiles with the grid's stride.
//
// A tile is one chain of dependent memory round trips, so they are made as few as possible: the
// occupancy bytes (one row of bits per lane, in every wave) and the whole halo patch are requested together at the start (the patch
// unconditionally: it is a few KB; inactive and out-of-image sites are zeroed from the masks on
// the way into LDS), old z values and - once per workgroup - the weights as soon as the tile is
// known to be touched.  Masks, z read-modify-write, activation increment (Eq.12-14) and
// occupancy words as in the other convolution kernels.
#include <algorithm>

#include "evconv_kernels.h"

namespace evk {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kMaxK = 128;             // largest contraction length
constexpr int kMaxSteps = kMaxK / 4;   // MFMA steps of four k each
constexpr int kMaxPatchPerThread = 10; // patch elements per thread (256 threads)

__device__ __forceinline__ float act_n(int act, float v) {
  if (act == kActRelu) return fmaxf(v, 0.0f);
  if (act == kActSigmoid) return 1.0f / (1.0f + expf(-v));
  if (act == kActTanh) return tanhf(v);
  if (act == kActOneMinus) return 1.0f - v;
  return v;
}

template <int MAXE>  // patch elements per thread
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAXE <= 3 ? 4 : 3))) void conv_narrow_kernel(ConvParams p) {
  touch_params<ConvParams>();
  asm volatile("" ::"s"(p.gi.h), "s"(p.gi.w), "s"(p.gi.c), "s"(p.gi.tx), "s"(p.gi.ty), "s"(p.go.h), "s"(p.go.w), "s"(p.go.c), "s"(p.go.tx),
               "s"(p.go.ty), "s"(p.k), "s"(p.stride), "s"(p.pad), "s"(p.dense), "s"(p.occ_in), "s"(p.in), "s"(p.z), "s"(p.out), "s"(p.w),
               "s"(p.st.stride), "s"(p.tx_magic), "s"(p.k_magic), "s"(p.co_magic), "s"(p.gw_magic[0]));
  const size_t so = (size_t)blockIdx.z * p.st.stride;  // this workgroup's stream
  constexpr int NT = 256;
  extern __shared__ __align__(16) float s_patch[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave & 1, cb = wave >> 1;  // this wave: tile rows 4 * half .. + 3, output channels 16 * cb .. + 15
  const int kq = lane >> 4, n16 = lane & 15;               // MFMA operand lane: k = 4 * step + kq; row / column n16
  const int s = p.stride, K = p.k;
  const int H = p.gi.h, W = p.gi.w, Cin = p.gi.c, Cout = p.go.c;
  const bool dense = p.dense != 0;
  const int P = 7 * s + K;  // patch edge, <= 21
  const int CS = Cin | 1;   // odd LDS site stride
  const int k_tot = K * K * Cin, n_steps = (k_tot + 3) >> 2;
  const int cin_magic = (int)p.co_magic;  // e / Cin == (e * cin_magic) >> 16 for e < 3600 (Cin <= 8)
  const int p_magic = p.gw_magic[0];   // site / P likewise for site < 441
  const int k_magic = p.k_magic;    // tap / K likewise for tap < 49
  __shared__ __align__(16) int s_koff[4][kMaxSteps];  // [k % 4][step]

  // once per workgroup: the LDS position of the patch element that operand k multiplies, relative to the
  // patch origin of the site (the second row block's lies `blk1` further on).  Beyond taps x c_in it is the
  // position of a zero kept behind the patch: the operand is then an explicit zero, not a patch
  // element times a zero weight (the element may be infinite or NaN).
  const int zero_at = P * P * CS;
  const int blk1 = 2 * s * P * CS;
  const int site0 = ((4 * half + (n16 >> 3)) * s * P + (n16 & 7) * s) * CS;
  if (tid == 0) s_patch[zero_at] = s_patch[zero_at + blk1] = 0.0f;  // (never overwritten: the patch ends before them)
  if (tid < kMaxK) {
    const int k = tid;
    const int tap = (k * cin_magic) >> 16, ci = k - tap * Cin;
    const int ky = (tap * k_magic) >> 16, kx = tap - ky * K;
    s_koff[k & 3][k >> 2] = k < k_tot ? (ky * P + kx) * CS + ci : zero_at;
  }
  // per patch element of this thread: where it goes in LDS, its place in the rows of bits and its
  // offset in the input relative to the patch origin (the same for every tile)
  int e_lds[MAXE], e_row[MAXE], e_px[MAXE], e_goff[MAXE];
  const int total = P * P * Cin;
#pragma unroll
  for (int j = 0; j < MAXE; ++j) {
    const int e = tid + j * NT;
    const int site = (e * cin_magic) >> 16, c = e - site * Cin;
    const int py = (site * p_magic) >> 16, px = site - py * P;
    e_lds[j] = e < total ? site * CS + c : -1;
    e_row[j] = py * 4;
    e_px[j] = px;
    e_goff[j] = (py * (W * Cin) + px * Cin + c) * 4;
  }
  // the weights of this wave's lane, one per step, fetched when the first touched tile is met
  // (a workgroup without one leaves without reading them)
  float wreg[kMaxSteps];
  bool staged = false;
  const int co = blockIdx.y * 32 + cb * 16 + n16;
  const unsigned site_bytes = (unsigned)Cout * 4u;
  constexpr unsigned kNowhere = 0x80000000u;  // out of range: loads return 0, stores are dropped

  bool first = true;
  for (int tile = blockIdx.x; tile < p.go.tiles(); tile += gridDim.x) {
    const int tile_y = p.tx_magic ? (int)__umulhi((unsigned)tile, p.tx_magic) : tile / p.go.tx, tile_x = tile - tile_y * p.go.tx;
    const int iy0 = tile_y * 8 * s - p.pad, ix0 = tile_x * 8 * s - p.pad;
    // Requests first: the activity of the region, one row of bits per lane (a byte of each of at most four
    // occupancy words; for a tile beyond the left or right border a neighbour's byte is read, which is
    // cut off with the columns outside the image), and every element of the patch.
    const int rtx0 = ix0 >> 3, iy = iy0 + lane;
    const bool row_ok = lane < P && (unsigned)iy < (unsigned)H;
    unsigned row_byte[4];
    {
      const __amdgpu_buffer_rsrc_t occ_rsrc =
          __builtin_amdgcn_make_buffer_rsrc((void*)at_stream(p.occ_in, so), 0, p.gi.ty * p.gi.tx * 8, 0x00020000);
      const unsigned off = row_ok ? (unsigned)(__mul24(iy >> 3, p.gi.tx) * 8 + (iy & 7)) : kNowhere;
#pragma unroll
      for (int rx = 0; rx < 4; ++rx)
        row_byte[rx] = (unsigned char)__builtin_amdgcn_raw_buffer_load_b8(occ_rsrc, off, min(max(rtx0 + rx, 0), p.gi.tx - 1) * 8, 0);
    }
    const __amdgpu_buffer_rsrc_t in_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)at_stream(p.in, so), 0, H * W * Cin * 4, 0x00020000);
    // (rows outside the image give an out-of-range offset: the load returns 0; columns outside it
    // read a neighbouring row's site, which the mask below discards; a thread without a j-th
    // element gets an out-of-range offset as well)
    const int origin = (iy0 * W + ix0) * Cin * 4;
    float pre[MAXE];
#pragma unroll
    for (int j = 0; j < MAXE; ++j) {
      const unsigned off = e_lds[j] >= 0 ? (unsigned)(origin + e_goff[j]) : kNowhere;
      pre[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(in_rsrc, off, 0, 0));
    }
    const int lo = max(0, -ix0), hi = min(P, W - ix0);  // valid columns in [lo, hi)
    const unsigned inside = ((1u << max(hi, 0)) - 1u) & ~((1u << lo) - 1u);  // (lo <= pad, hi <= 21)
    const unsigned span = row_byte[0] | (row_byte[1] << 8) | (row_byte[2] << 16) | (row_byte[3] << 24);
    const unsigned bits = (dense ? ~0u : span >> (ix0 - rtx0 * 8)) & (row_ok ? inside : 0u);

    uint64_t touched_word;  // whole tile, identical in all waves
    {
      const int ly = lane >> 3, lx = lane & 7;
      const int oy = tile_y * 8 + ly, ox = tile_x * 8 + lx;
      unsigned rows = 0;
#pragma unroll
      for (int ky = 0; ky < 7; ++ky) {
        const unsigned row = (unsigned)__builtin_amdgcn_ds_bpermute((ly * s + ky) * 4, (int)bits);
        rows |= ky < K ? row : 0u;
      }
      touched_word = __ballot((oy < p.go.h) & (ox < p.go.w) & (dense | (((rows >> (lx * s)) & ((1u << K) - 1u)) != 0)));
    }
    if (touched_word == 0) continue;
    const unsigned my_touched = (unsigned)(touched_word >> (32 * half));  // this wave's 32 sites

    // accumulator element (block r, register i, lane) = local site 16 * r + 4 * kq + i of the half
    // tile, channel n16 of this wave's 16
    const unsigned site_bits = co < Cout ? my_touched >> (4 * kq) : 0u;  // bit 16 * r + i
    // (offsets from the tile's first row, so that outputs of more than 2 GiB are in reach)
    const size_t row0 = (size_t)(tile_y * 8) * p.go.w * Cout;
    const int row_bytes = min(8, p.go.h - tile_y * 8) * p.go.w * Cout * 4;
    const __amdgpu_buffer_rsrc_t z_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(at_stream(p.z, so) + row0), 0, row_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(at_stream(p.out, so) + row0), 0, row_bytes, 0x00020000);
    const unsigned out_off = ((unsigned)((4 * half + (kq >> 1)) * p.go.w + tile_x * 8 + 4 * (kq & 1)) * (unsigned)Cout + (unsigned)co) * 4u;
    const unsigned block_step = 2u * (unsigned)p.go.w * site_bytes;  // two tile rows
    unsigned at[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) at[r][i] = ((site_bits >> (16 * r + i)) & 1u) ? out_off + (r ? block_step : 0u) + i * site_bytes : kNowhere;
    float z_old[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        z_old[r][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(z_rsrc, dense ? kNowhere : at[r][i], 0, 0));
    if (!staged) {
      // re-laid weights: [32-channel group][block of 16][lane][step]: a lane's share is 128 bytes
      const float4* wsrc = (const float4*)((const float*)p.w + (((size_t)blockIdx.y * 2 + cb) * 64 + lane) * kMaxSteps);
#pragma unroll
      for (int v = 0; v < kMaxSteps / 4; ++v) {
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        if (4 * v < n_steps) t = wsrc[v];
        wreg[4 * v] = t.x; wreg[4 * v + 1] = t.y; wreg[4 * v + 2] = t.z; wreg[4 * v + 3] = t.w;
      }
      staged = true;
    }
    if (!first) __syncthreads();  // the previous tile's patch is no longer in use
    first = false;
    // patch into LDS: inactive and out-of-image sites become zeros
#pragma unroll
    for (int j = 0; j < MAXE; ++j) {
      const unsigned row = (unsigned)__builtin_amdgcn_ds_bpermute(e_row[j], (int)bits);
      if (e_lds[j] >= 0) s_patch[e_lds[j]] = ((row >> e_px[j]) & 1u) ? pre[j] : 0.0f;
    }
    __syncthreads();
    if (my_touched == 0) continue;  // (uniform per wave; the barriers of the next tile are met by all waves)

    floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    {
      // the two row blocks of the half tile: rows 4 * half + (n16 >> 3) and two rows further down
      // (the distance is re-materialised per tile so that the second block's 32 addresses are
      // formed at their use instead of living in registers across the tile loop)
      int blk1_v = blk1, site0_v = site0;
      asm volatile("" : "+v"(blk1_v), "+v"(site0_v));
      // in batches of eight steps: the operand reads of a batch, then its matrix instructions
#pragma unroll
      for (int s0 = 0; s0 < kMaxSteps; s0 += 8) {
        if (s0 >= n_steps) break;
        const int4 k0 = *(const int4*)&s_koff[kq][s0], k1 = *(const int4*)&s_koff[kq][s0 + 4];
        const int ko[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
        float a0[8], a1[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          // (the zero behind the patch is addressed absolutely: site0 is taken off again)
          const int at = ko[j] >= zero_at ? ko[j] : ko[j] + site0_v;
          a0[j] = s_patch[at];
          a1[j] = s_patch[at + blk1_v];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j], wreg[s0 + j], acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[j], wreg[s0 + j], acc1, 0, 0, 0);
        }
      }
    }

    // epilogue straight from the accumulator registers
    unsigned nz = 0;  // nonzero output sites of this wave (bits of its 32-site half)
    const float bias = (dense && p.bias && co < Cout) ? p.bias[co] : 0.0f;
    auto epilogue = [&](auto&& increment) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = r == 0 ? acc0[i] : acc1[i];
          const float z_new = (dense ? bias : z_old[r][i]) + v;
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(z_new), z_rsrc, at[r][i], 0, 0);
          const float o = increment(v, z_new, z_old[r][i]);
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), o_rsrc, at[r][i], 0, 0);
          const uint64_t bal = __ballot(at[r][i] != kNowhere && o != 0.0f);  // 16 lanes (channels) per site: sites 16 * r + 4 * g + i
#pragma unroll
          for (int g = 0; g < 4; ++g) nz |= ((bal >> (16 * g)) & 0xffffull) ? 1u << (16 * r + 4 * g + i) : 0u;
        }
    };
    // regular pass: z = v + bias, o = act(z); incremental: z += v, o = act(z_new) - act(z_old) (z_old reads
    // as 0 in a regular pass, so ReLU's difference serves both)
    if (p.act == kActRelu) epilogue([](float, float z1, float z0) { return fmaxf(z1, 0.0f) - fmaxf(z0, 0.0f); });
    else if (p.act == kActNone) epilogue([&](float v, float z1, float) { return dense ? z1 : v; });
    else epilogue([&](float, float z1, float z0) { return dense ? act_n(p.act, z1) : act_n(p.act, z1) - act_n(p.act, z0); });
    if (lane == 0) {
      const uint64_t mine = (uint64_t)(dense ? my_touched : nz) << (32 * half);
      if (mine) atomicOr((unsigned long long*)&at_stream(p.occ_out, so)[tile], (unsigned long long)mine);  // pre-zeroed word
      if (blockIdx.y == 0 && cb == 0) {
        const uint64_t t = (uint64_t)my_touched << (32 * half);
        if (t) atomicOr((unsigned long long*)&at_stream(p.occ_touched, so)[tile], (unsigned long long)t);
      }
    }
  }  // tiles
}

}  // namespace

bool conv_narrow_supported(const ConvParams& p) {
  const int k_tot = p.k * p.k * p.gi.c;
  const int P = 7 * p.stride + p.k;
  return k_tot <= kMaxK && p.gi.c <= 8 && p.go.c >= 16 && p.c_out_pad == (p.go.c + 31) / 32 * 32 && p.n_fused == 0 &&
         P * P * p.gi.c <= kMaxPatchPerThread * 256 &&
         (long long)p.gi.h * p.gi.w * p.gi.c * 4 < (1ll << 31) &&  // byte offsets of the gather fit 31 bits,
         8ll * p.go.w * p.go.c * 4 < (1ll << 31);                  // and those inside a row of output tiles
}

// re-laid weights: floats for c_out_pad output channels, and the position of W[k][co]
// (k = tap * c_in + ci): [co / 32][(co % 32) / 16][lane = (k % 4) * 16 + co % 16][step = k / 4]
size_t conv_narrow_weight_floats(int c_out_pad) { return (size_t)(c_out_pad / 32) * 2 * 64 * kMaxSteps; }
size_t conv_narrow_weight_index(int k, int co) {
  return ((size_t)((co >> 5) * 2 + ((co & 31) >> 4)) * 64 + (size_t)(k & 3) * 16 + (co & 15)) * kMaxSteps + (k >> 2);
}

void launch_conv_narrow(const ConvParams& p, hipStream_t s) {
  const int P = 7 * p.stride + p.k;
  const int cs = p.gi.c | 1;
  // the patch, then room for the two zeros that stand in for operands beyond taps x c_in
  const size_t lds = ((size_t)P * P * cs + 2 * p.stride * P * cs + 1) * sizeof(float);
  // workgroups walk the tiles with the grid's stride; enough of them to fill the chip's resident
  // slots (a tile is one chain of dependent memory round trips, so few long walks are slow).  A regular
  // pass, in which every tile is touched, takes as many as are resident: 256 x 352, 1408 tiles, 18.4 us with
  // a workgroup per tile, 16.5 with 1024 workgroups; a step with 2 % of the sites active 12.6 and 13.0.
  dim3 grid(std::min(p.go.tiles(), std::max((p.dense ? 1024 : 4096) / p.st.n, 256)), p.c_out_pad / 32, p.st.n);
  // divisors of the kernel's index arithmetic (tiles per row: exact while the product fits 32 bits)
  ConvParams q = p;
  q.tx_magic = p.go.tx == 1 || (long long)p.go.tiles() * p.go.tx >= (1ll << 32) ? 0u : (unsigned)((0x100000000ull + (unsigned)p.go.tx - 1) / (unsigned)p.go.tx);
  q.k_magic = (65536 + p.k - 1) / p.k;
  q.co_magic = (65536 + p.gi.c - 1) / p.gi.c;
  q.gw_magic[0] = (65536 + P - 1) / P;
  if (P * P * p.gi.c <= 3 * 256) hipLaunchKernelGGL(conv_narrow_kernel<3>, grid, dim3(256), lds, s, q);
  else hipLaunchKernelGGL(conv_narrow_kernel<kMaxPatchPerThread>, grid, dim3(256), lds, s, q);
}

}  // namespace evk
