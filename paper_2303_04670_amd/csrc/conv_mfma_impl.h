// Sparse incremental convolution on the matrix cores.
//
// Used where the per-tile channel contraction is a dense GEMM: c_in >= 9 (any count: the last
// channel chunk is zero-padded), c_out >= 16 (any count: the last block of 32 is zero-padded).
// Implicit GEMM per touched output tile (8 x 8 sites): M = 32 * MB sites (MB = 2: the whole
// tile as two 32-row MFMA blocks, rows 0-3 and 4-7; MB = 1: one workgroup per half tile),
// N = 32 output channels per workgroup, K = taps x c_in.
//
//   bf16 mode : the gather rounds increments to bf16 on their way into LDS, weights are bf16,
//               v_mfma_f32_32x32x16_bf16 with fp32 accumulation; a unit = one tap x 16 channels
//               (one MFMA per block); lanes 0-31 hold channels 0-7, lanes 32-63 channels 8-15.
//   fp32 mode : the same instruction on operands written as the sum of three bf16 parts (Henry, Tang,
//               Heinecke: "Leveraging the bfloat16 Artificial Intelligence Datatype For
//               Higher-Precision Computations", 2019): x = hi + mid + lo with hi = bf16(x), mid =
//               bf16(x - hi), lo = x - hi - mid.  3 x 8 signed significant bits hold the 24 of an
//               fp32 value, as long as it has no bits below 2^-133, where bf16 ends: every value of
//               2^-110 and more.  The gather does that for the increments (smaller ones are rounded
//               to multiples of 2^-133), the host for the weights (if some are smaller, all of a
//               conv's are stored times 2^16).  A product is the six partial products down to 2^-16
//               of it (lo*hi, mid*mid, hi*lo, mid*hi, hi*mid, hi*hi); the three left out add up to
//               less than 2^-24 of it, the largest rounding error of one fp32 product.  Six MFMAs at
//               16 times the rate of the chip's fp32 matrix instruction, which besides runs on the
//               vector pipeline and takes its time from every address and epilogue instruction.
//   split mode: two parts and three products (lo*hi, hi*lo, hi*hi): 16 significant bits, relative
//               error of a product about 2^-16, against 2^-8 in bf16 mode.
//
// Workgroup = NW (4 or 8) wavefronts that split K: the units of every channel chunk are dealt
// round-robin to the waves; each wave keeps the MB accumulators and the partial sums are added
// through LDS at the end.  K-splitting (rather than N-splitting), 8 waves and half tiles are what
// spread the low-resolution layers (24-88 tiles) over 256 CUs; the launcher picks MB and NW from
// the number of workgroups a layer yields.
//   Masks: every wave has one bit row per patch row, in the lane of that number (a byte of each of at
//     most four occupancy words); the touched word of the tile and the gather predicates come from
//     rows fetched from other lanes (ds_bpermute).  Nothing before the first patch goes through LDS or
//     waits at a barrier.
//   A operand: the input halo patch of the current chunk, gathered once per workgroup into LDS
//     with buffer loads whose offset is pushed out of range for inactive / out-of-image sites:
//     the hardware bounds check returns zeros without a memory access (conditioned fetch).  The
//     next chunk's patch is fetched into registers while the current one is being contracted.
//     A lane reads its fragment with one ds_read_b128; the LDS site stride keeps that
//     conflict-free for stride-1 layers.
//   B operand: weights re-laid as one plane [tap][c_in/8][c_out][8] of bf16 per part, so that a
//     lane's fragment is one 16-byte buffer load per part (L2-resident), held in a three-fragment
//     ring two units ahead, across chunk boundaries.
// Epilogue: lane = output channel, so every z / increment access is a 128-byte row segment; the
// old z values are requested before the contraction starts.  ADD nodes that consume the conv
// output (residual add + activation, skip adds) run here as well, writing their own buffers.
//
// A bilinear x2 up-sampling in front of the conv (Eq.9-10: both linear) never exists in memory: the patch is
// interpolated from the stored tensor on its way into LDS (UPS variants), or the up-sampling is folded into the
// weights (5 x 5, fp32 and split modes: conv_fold_impl.h).
//
// Vector instructions are kept few throughout: per-lane parts of an address are computed once and
// kept, per-unit / per-row parts live in scalar registers (buffer instructions with a scalar
// offset), masks are tested where their bits sit.
// (This header holds the kernels and their launchers, conv_mfma_body.h the body of a workgroup; one
// translation unit per operand mode instantiates them, so that the three modes compile in parallel.)
#pragma once
#include <algorithm>
#include <type_traits>

#include <cstddef>

#include "evconv_kernels.h"

namespace evk {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
// Phase stamps.  In a build with -DEVCONV_PHASE_STAMPS (never the product build) one lane per
// workgroup writes the 100 MHz wall clock at the boundaries of the kernel's phases into a device
// array of the translation unit; evconv_debug_phase_stamps copies the records out.  Without the
// define EVK_PHASE expands to nothing.  A record is 32 x u64:
enum PhaseField {
  kPhStart = 0,            // first instruction of the workgroup
  kPhOccInLds = 1,         // occupancy bytes arrived (the gather addressing is worked out meanwhile)
  kPhBitRows = 2,          // bit rows of the patch built
  kPhAddressed = 3,        // first patch chunk requested, touched words, old z requested
  kPhFirstIssued = 4,      // first weight fragments requested
  kPhFirstPatchInLds = 5,  // first chunk arrived, in LDS (and interpolated), next chunk requested
  kPhChunksDone = 6,       // end of the chunk loop
  kPhFusedRequested = 10,  // operands of the fused stages requested
  kPhReduced = 7,          // partial sums of the waves in LDS
  kPhArrived = 14,         // everything requested so far has arrived
  kPhEpilogueDone = 8,     // all passes of the epilogue issued
  kPhFlagsBallot = 11,     // (start of the nonzero-flag collection)
  kPhFlagsInLds = 12,      // the waves' flag words written
  kPhFlagsBarrier = 13,    // ... and visible to the workgroup
  kPhEnd = 9,              // tile words OR-ed into memory
  kPhContractionTicks = 20,  // ticks inside the contraction loops, all chunks
  kPhChunkChangeTicks = 21,  // ticks in barriers, LDS stores and interpolation between them
  kPhGrid = 24, kPhBlock = 25, kPhHwId = 26,  // workgroups of the launch, this one's index, HW_ID | XCC_ID << 32
  kPhLayer = 27,           // output height | c_in << 16 | k << 32 | c_out << 40
};
#ifdef EVCONV_PHASE_STAMPS
constexpr unsigned kPhaseRecords = 1u << 15;
static __device__ unsigned long long g_phase[kPhaseRecords][32];
// (a counter for each of 64 classes of workgroups, in lines of their own: with one for all of them 704 workgroups
// started 8 us apart, a queue at the counter)
constexpr unsigned kPhaseClasses = 64, kPhaseClassRecords = kPhaseRecords / kPhaseClasses;
static __device__ unsigned g_phase_n[kPhaseClasses][32];
#define EVK_PHASE_OPEN() const unsigned ph_slot = tid == 0 ? phase_record(p) : 0xffffffffu
#define EVK_PHASE(i) do { if (tid == 0 && ph_slot < kPhaseRecords) g_phase[ph_slot][i] = wall_clock64(); } while (0)
template <class P>
static __device__ unsigned phase_record(const P& p) {  // a record for this workgroup
  const unsigned long long now = wall_clock64();
  const unsigned cls = (blockIdx.x + blockIdx.y * gridDim.x) % kPhaseClasses, nth = atomicAdd(&g_phase_n[cls][0], 1u);
  const unsigned slot = nth < kPhaseClassRecords ? cls * kPhaseClassRecords + nth : kPhaseRecords;
  if (slot < kPhaseRecords) {
    unsigned long long* r = g_phase[slot];
    for (int i = 1; i < 24; ++i) r[i] = 0;
    r[kPhStart] = now;
    r[kPhGrid] = (unsigned long long)gridDim.x * gridDim.y;
    r[kPhBlock] = blockIdx.x + (unsigned long long)blockIdx.y * gridDim.x;
    r[kPhHwId] = __builtin_amdgcn_s_getreg(4 | (31 << 11)) | ((unsigned long long)__builtin_amdgcn_s_getreg(20 | (31 << 11)) << 32);
    r[kPhLayer] = (unsigned long long)p.go.h | ((unsigned long long)p.gi.c << 16) | ((unsigned long long)p.k << 32) |
                  ((unsigned long long)p.go.c << 40);
  }
  return slot;
}
#else
#define EVK_PHASE_OPEN() do {} while (0)
#define EVK_PHASE(i) do {} while (0)
#endif
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// operand modes of the contraction
constexpr int kOpF32 = 0;    // fp32 operands, each written exactly as three bf16 parts, six bf16 MFMAs per product
constexpr int kOpBf16 = 1;   // bf16 operands (increments rounded in the gather), v_mfma_f32_32x32x16_bf16
constexpr int kOpSplit = 2;  // fp32 operands split into bf16 high + low parts, three bf16 MFMAs per product

// one weight fragment of a lane: the high, (fp32 mode) middle and (fp32, split mode) low parts
struct BFrag { float4 h, m, l; };
// one patch fragment of a lane: the parts of both 32-row blocks (second block: two-block workgroups only)
struct AFrag { float4 h0, h1, m0, m1, l0, l1; };

__device__ __forceinline__ float act_m(int act, float v) {
  if (act == kActRelu) return fmaxf(v, 0.0f);
  if (act == kActSigmoid) return 1.0f / (1.0f + expf(-v));
  if (act == kActTanh) return tanhf(v);
  if (act == kActOneMinus) return 1.0f - v;
  return v;
}

// fp32 -> bf16, round to nearest even, two values packed low/high: one v_cvt_pk_bf16_f32
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
  floatx2 v;
  v.x = lo;
  v.y = hi;
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// Largest halo patch (sites) a variant can meet: 64- and 128-channel chunks are used with stride 1
// and taps <= 3, 32-channel chunks with stride 1 (taps <= 7), 16-channel chunks also with stride 2.
// (s2k: 0, or the largest kernel of a variant for stride 2, or minus that of one for stride 1)
constexpr int max_patch_sites(int chunk, int mb, int s2k) {
  const int rows = 4 * mb - 1;
  if (s2k > 0) return (rows * 2 + s2k) * (14 + s2k);
  if (s2k < 0) return (rows - s2k) * (7 - s2k);
  return chunk >= 64 ? (rows + 3) * 10 : chunk == 32 ? (rows + 7) * 14 : (rows * 2 + 7) * 21;
}

// n / d with magic = ceil(2^32 / d): exact while n * d < 2^32 (the launcher passes 0 where that may
// not hold, and for d == 1)
__device__ __forceinline__ int fast_div(int n, int d, unsigned magic) {
  return magic ? (int)__umulhi((unsigned)n, magic) : n / d;
}

constexpr int op_parts(int opm) { return opm == kOpF32 ? 3 : opm == kOpSplit ? 2 : 1; }
// 4-byte words of a patch site in LDS
constexpr int patch_site_words(int chunk, int opm) { return chunk / 2 * op_parts(opm) + 4; }

// The three parts of a value beyond the bf16 rounding range, into bits [shift, shift + 16) of h, m,
// l.  A finite one: the high part is cut off instead of rounded up to infinity.  An infinity goes
// into the low part alone: the low part is multiplied with the weight's high part only, which is
// zero for zero weights only (weights too small for a bf16 are stored times a power of two), so the
// product is the IEEE one (inf * 0 of a weight's zero low parts would be NaN).
constexpr float kBf16Overflow = 3.3961775e38f;  // 0x7f7f8000: the smallest value that rounds to an infinite bf16
__device__ __forceinline__ void split3_large(float x, int shift, unsigned& h, unsigned& m, unsigned& l) {
  if (!(fabsf(x) >= kBf16Overflow)) return;
  unsigned ph = 0, pm = 0, pl = __float_as_uint(x) >> 16;
  if (fabsf(x) != INFINITY) {
    ph = __float_as_uint(x) >> 16;
    const float r = x - __uint_as_float(ph << 16);
    pm = __float_as_uint(r) >> 16;
    pl = __float_as_uint(r - __uint_as_float(pm << 16)) >> 16;
  }
  const unsigned keep = ~(0xffffu << shift);
  h = (h & keep) | (ph << shift);
  m = (m & keep) | (pm << shift);
  l = (l & keep) | (pl << shift);
}

// The register budget is held to 4 (half tiles) or 3 (whole tiles) waves per SIMD: the bf16 and
// split modes are bound by latencies, not by the matrix cores, and lose a third of their speed
// when one workgroup fewer fits on a CU.
//
// UPS: the conv's input is the bilinear x2 up-sampling of p.in (half-pixel centres, weights
// 0.25 / 0.75, clamped borders), which is never written to memory: the low-resolution sites under
// the halo are gathered into a second LDS buffer and every patch element is interpolated from
// four of them on its way into the patch buffer.  p.gi describes the up-sampled tensor, p.lo_h x
// p.lo_w the stored one; p.occ_in are the stored tensor's occupancy words, and an up-sampled
// site is active where one of its four sources is.
//
// KSP: the channels are split over p.ks workgroups as well (chunk ranges of p.ks_chunks chunks).
// S2K: the largest kernel of a variant for stride 2, minus that of one for stride 1, or 0: any (launch_shape).
// What a workgroup gathers:
constexpr int kPlain = 0;        // the stored tensor
constexpr int kInterpolate = 1;  // UPS: the up-sampled tensor, interpolated from the stored one

// Waves per SIMD that the registers of a variant are held to.  Five where the plain four-wave half tiles reach
// them (bf16, and split mode in chunks of 64 channels: 88 to 96 registers): launches of 1024 to 1280 and of
// 2048 to 2560 workgroups are then one round on the chip less.
constexpr int min_waves(int chunk, int nw, int opm, int mb, int mode, bool ksp, int s2k) {
  if (mb == 2 || (mode != kPlain && nw == 4)) return 3;
  if (mode == kPlain && !ksp && s2k <= 0 && nw == 4 && (opm == kOpBf16 || (opm == kOpSplit && chunk == 64))) return 5;
  return 4;
}

// The body of a workgroup is text that is included twice: into the kernel of the plain convs, whose
// arguments the compiler knows where they are (through a reference it keeps more of them in scalar
// registers than there are, 0.2-0.5 us a layer), and into a function for the kernels that choose between
// bodies.
template <int CHUNK, int NW, int OPM, int MB, int MODE, bool KSP, int S2K>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(min_waves(CHUNK, NW, OPM, MB, MODE, KSP, S2K))))
void conv_mfma_kernel(ConvParams p) {
  touch_params<ConvParams>();
  // (what the prologue needs is loaded together, too: on demand it was a dozen loads, each waited for)
  if (MODE == kPlain) asm volatile("" ::"s"(p.gi.h), "s"(p.gi.w), "s"(p.gi.c), "s"(p.go.h), "s"(p.go.w), "s"(p.go.c), "s"(p.go.tx), "s"(p.k),
               "s"(p.stride), "s"(p.pad), "s"(p.dense), "s"(p.n_fused), "s"(p.c_out_pad), "s"(p.occ_in), "s"(p.in), "s"(p.z),
               "s"(p.w), "s"(p.st.stride), "s"(p.wg_swap), "s"(p.tx_magic), "s"(p.gw_magic[0]), "s"(p.k_magic));
  // this workgroup's stream: every state pointer of p is used through at_stream(.., so); p itself
  // stays untouched so that it remains in the kernel-argument segment
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  // Consecutive workgroups (x fastest) go to the chip's 8 XCDs in turn, each with an L2 of its own.
  // x over tiles: an XCD sees every eighth tile and all of the weights; x over the blocks of
  // output channels (wg_swap): an XCD sees all tiles and one in eight (four, two) of the weight
  // blocks.  The launcher picks whichever of the two operands is larger to be split.
  const int wg_tile = p.wg_swap ? blockIdx.y : blockIdx.x, wg_ck = p.wg_swap ? blockIdx.x : blockIdx.y;
  constexpr bool UPS = MODE != kPlain, PAIR = false, LATE = false;
#include "conv_mfma_body.h"
}

// args: byte offset of this workgroup's ConvParams in the kernel arguments
// LATE: old z values are requested after the contraction, which leaves registers for one more wave per SIMD
template <int CHUNK, int NW, int OPM, int MB, int MODE, bool KSP, int S2K, bool PAIR, bool LATE = false>
__device__ __forceinline__ void conv_workgroup(const unsigned args, const int wg_tile, const int wg_ck) {
  typedef const char __attribute__((address_space(4))) Byte;
  const auto& p = *(const ConvParams __attribute__((address_space(4)))*)((Byte*)__builtin_amdgcn_kernarg_segment_ptr() + args);
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  constexpr bool UPS = MODE != kPlain;
#include "conv_mfma_body.h"
}

// Two convs that read the same tensor, in one launch (see launch_pair): the first n_first workgroups
// are a's.
struct ConvPair { ConvParams a, b; int n_first; };
template <int OPM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void conv_mfma_pair_kernel(ConvPair q) {
  const bool second = (int)blockIdx.x >= q.n_first;
  const unsigned args = second ? (unsigned)offsetof(ConvPair, b) : 0u;
  touch_params<ConvParams>(args);
  typedef const char __attribute__((address_space(4))) Byte;
  const auto& p = *(const ConvParams __attribute__((address_space(4)))*)((Byte*)__builtin_amdgcn_kernarg_segment_ptr() + args);
  const int wg = (int)blockIdx.x - (second ? q.n_first : 0);
  const int y = wg / p.grid_x, x = wg - y * p.grid_x;
  conv_workgroup<64, 8, OPM, 1, kPlain, true, 3, true>(args, p.wg_swap ? y : x, p.wg_swap ? x : y);
}

// Up to four convs of the same tensor and one variant in one launch (see launch_batch): workgroup
// first[i] is the first of conv i.
struct ConvBatch { ConvParams p[kMaxConvBatch]; int first[kMaxConvBatch]; int n; };
template <int OPM, int S2K>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OPM == kOpBf16 ? 5 : 4))) void conv_mfma_batch_kernel(ConvBatch q) {
  int i = 0;
#pragma unroll
  for (int j = 1; j < kMaxConvBatch; ++j)
    if (j < q.n && (int)blockIdx.x >= q.first[j]) i = j;
  const unsigned args = (unsigned)(offsetof(ConvBatch, p) + i * sizeof(ConvParams));
  touch_params<ConvParams>(args);
  typedef const char __attribute__((address_space(4))) Byte;
  Byte* const base = (Byte*)__builtin_amdgcn_kernarg_segment_ptr();
  const auto& p = *(const ConvParams __attribute__((address_space(4)))*)(base + args);
  const int wg = (int)blockIdx.x - *(const int __attribute__((address_space(4)))*)(base + offsetof(ConvBatch, first) + i * sizeof(int));
  const int y = wg / p.grid_x, x = wg - y * p.grid_x;
  conv_workgroup<32, 4, OPM, 1, kPlain, false, S2K, false, OPM == kOpBf16>(args, p.wg_swap ? y : x, p.wg_swap ? x : y);
}

inline int chunk_for(const ConvParams& p) {
  // low-resolution layers (few workgroups, always 8 waves): 128-channel chunks halve the number of
  // gather round trips, which is what these latency-bound launches consist of
  if (p.stride == 1 && p.k <= 3 && p.gi.c % 128 == 0 &&
      (long long)p.go.tiles() * (p.c_out_pad / 32) * p.st.n * 2 < 512) return 128;
  // Stride-2 layers of few half-tile workgroups: a patch of 64 (3 x 3) or 32 (5 x 5) channels still fits
  // the gather registers and saves chunk changes; where the chip is full several times over the
  // smaller patch's extra workgroups per CU win.  Measured in fp32 mode, chunks of 16 -> larger:
  // 128 -> 256 on 32 x 44 (384 workgroups) 31.5 -> 28.3 us, 64 -> 128 on 64 x 88 (704) 23.7 -> 22.9, 32 ->
  // 64 on 128 x 176 (1408) 27.1 -> 27.7; ResNet-18's 64 -> 128 on 28 x 28 (128) 13.2 -> 11.5; with 16
  // streams (6144 to 22528) 218 -> 252, 215 -> 250 and 294 -> 325.
  // (1 x 1: the patch is small whatever the chunk, and a chunk of 16 channels is a single unit: chunks of 32
  // there too; 128 -> 256 on 192 x 192 35.6 -> 30.3 us, 256 -> 512 on 256 x 256 155 -> 127)
  const long long n_half = (long long)p.go.tiles() * (p.c_out_pad / 32) * p.st.n * 2;
  if (p.stride == 2 && p.k == 1 && n_half > 1024 && p.gi.c % 32 == 0) return 32;
  if (p.stride == 2 && n_half <= 1024) {
    if (p.k <= 3 && p.gi.c % 64 == 0 && n_half < 512) return 64;
    if (p.k <= 5 && p.gi.c % 32 == 0) return 32;
  }
  if (p.stride == 1 && p.k <= 3 && p.gi.c % 64 == 0) return 64;
  if (p.stride == 1 && (p.gi.c % 32 == 0 || (p.gi.c % 16 != 0 && p.gi.c > 32))) return 32;  // ragged: fewer, padded chunks
  return 16;
}

// divisors of the kernels' index arithmetic
inline unsigned magic32(long long n, int d) {  // for dividends below n
  return d == 1 || n * d >= (1ll << 32) ? 0u : (unsigned)((0x100000000ull + (unsigned)d - 1) / (unsigned)d);
}
inline int magic16(int d) { return (65536 + d - 1) / d; }

// A variant's launch: its arguments, grid and dynamic LDS
struct ConvLaunch { ConvParams q; dim3 grid; size_t lds; };
template <int CHUNK, int NW, int OPM, int MB, bool KSP>
ConvLaunch variant_launch(const ConvParams& p) {
  const int PH = (4 * MB - 1) * p.stride + p.k, PW = 7 * p.stride + p.k;
  // (rows of the patch are padded to a pitch of 32 modulo 64 words: at most 64 more per row)
  size_t lds = (size_t)PH * (PW * patch_site_words(CHUNK, OPM) + 64) * sizeof(float);
  const size_t part = (size_t)NW * MB * 16 * 64 * sizeof(float);  // partial sums reuse the patch
  // The operand that is read by every XCD in full should be the smaller one: the weights of the
  // high-resolution layers, the input of the low-resolution ones (k * k * c_out weights per input
  // channel against one value per stored site per input channel).  Measured on the 32 x 44 -> 64 x
  // 88 up-sampling conv (256 -> 128 channels, 5 x 5): 95 -> 86 us; neutral on the other layers.
  ConvParams q = p;
  const long long in_sites = p.upsample ? (long long)p.lo_h * p.lo_w : (long long)p.gi.h * p.gi.w;
  q.wg_swap = (long long)p.k * p.k * p.go.c > in_sites && p.go.tiles() * (2 / MB) <= 65535;
  const int n_ck = p.c_out_pad / 32 * (KSP ? p.ks : 1);
  q.tx_magic = magic32(p.go.tiles(), p.go.tx);
  q.co_magic = magic32(n_ck, p.c_out_pad / 32);
  q.k_magic = magic16(p.k);
  q.gw_magic[0] = magic16(PW);
  q.gw_magic[1] = magic16(PW / 2 + 3);
  q.nbx_magic = magic16(((PW - p.pad - 2) >> 1) - ((-p.pad - 1) >> 1) + 1);  // (a tile's first column is even)
  dim3 grid(p.go.tiles() * (2 / MB), n_ck, p.st.n);
  if (q.wg_swap) grid = dim3(n_ck, p.go.tiles() * (2 / MB), p.st.n);
  q.grid_x = (int)grid.x;
  if (CHUNK == 32 && p.upsample)  // the low-resolution source region behind the patch buffer
    lds += (size_t)(PH / 2 + 3) * (PW / 2 + 3) * (CHUNK + 4) * sizeof(float);
  return ConvLaunch{q, grid, std::max(lds, part)};
}

template <int CHUNK, int NW, int OPM, int MB, bool KSP = false, int S2K = 0>
void launch_variant(const ConvParams& p, hipStream_t s) {
  const ConvLaunch l = variant_launch<CHUNK, NW, OPM, MB, KSP>(p);
  if constexpr (CHUNK == 32 && !KSP && S2K == 0) {
    if (p.upsample) {
      hipLaunchKernelGGL((conv_mfma_kernel<CHUNK, NW, OPM, MB, kInterpolate, false, 0>), l.grid, dim3(NW * 64), l.lds, s, l.q);
      return;
    }
  }
  hipLaunchKernelGGL((conv_mfma_kernel<CHUNK, NW, OPM, MB, kPlain, KSP, S2K>), l.grid, dim3(NW * 64), l.lds, s, l.q);
}

// share of the chip's 256 CUs kept busy when n equally long workgroups run at once
inline double fill(long long n) { return (double)n / 256.0 / (double)((n + 255) / 256); }

// The variant that a conv takes which does not split its channels: channels per chunk, half or whole tiles, four
// or eight waves.
struct Shape { int chunk; bool halves, eight; };
inline Shape shape_for(const ConvParams& p) {
  const int chunk = chunk_for(p);
  const long long n2 = (long long)p.go.tiles() * (p.c_out_pad / 32) * p.st.n;  // workgroups with whole tiles
  if (chunk == 128) return {chunk, true, true};  // chosen only for few workgroups
  if (p.stride == 2 && chunk != 16) return {chunk, true, 2 * n2 < 512};
  // Whole tiles (two accumulators per wave, every weight fragment used twice) pay off only when
  // the launch fills the chip several times over and a workgroup has a long contraction; measured
  // on the layers of the evaluation networks, half tiles win everywhere else (more, shorter
  // workgroups: shorter prologues and patches, better balance)
  const bool halves = !(n2 >= 512 && p.k * p.k * p.gi.c >= 1600) || fill(2 * n2) > fill(n2) + 0.1;
  return {chunk, halves, halves && 2 * n2 < 512};  // few workgroups: 8 waves each split K further
}

// Variants for the small kernels: what a thread gathers of a patch is then as many registers and conversions as
// the patch needs.  In the variants for any kernel a thread takes its items in pairs, also where it has one
// (1 x 1) or three (3 x 3 at stride 2), and holds the registers of a 7 x 7 patch.  us, in those / in these, fp32: 1 x 1,
// 288 -> 288 on 256 x 352 322 / 244, 160 -> 64 on 128 x 128 15.2 / 13.3; 3 x 3 at stride 2, 128 -> 128 on 256 x 352 61.7 /
// 56.4; 3 x 3, 69 -> 64 on 64 x 88 13.9 / 13.0.
template <int CHUNK, int OPM, int S2K>
void launch_bound(const ConvParams& p, const Shape& shape, hipStream_t s) {
  if (shape.eight) launch_variant<CHUNK, 8, OPM, 1, false, S2K>(p, s);
  else if constexpr (CHUNK < 128) {
    if (shape.halves) launch_variant<CHUNK, 4, OPM, 1, false, S2K>(p, s);
    else launch_variant<CHUNK, 4, OPM, 2, false, S2K>(p, s);
  }
}
template <int CHUNK, int OPM>
void launch_shape(const ConvParams& p, const Shape& shape, hipStream_t s) {
  if constexpr (CHUNK == 32 || CHUNK == 64) {
    if (p.stride == 2) {
      constexpr int K2 = CHUNK == 32 ? 5 : 3;
      if (shape.eight) {
        if (p.k == 1) launch_variant<CHUNK, 8, OPM, 1, false, 1>(p, s);
        else if (p.k <= 3) launch_variant<CHUNK, 8, OPM, 1, false, 3>(p, s);
        else launch_variant<CHUNK, 8, OPM, 1, false, K2>(p, s);
      } else {
        if (p.k == 1) launch_variant<32, 4, OPM, 1, false, 1>(p, s);
        else if (p.k <= 3) launch_variant<32, 4, OPM, 1, false, 3>(p, s);
        else launch_variant<32, 4, OPM, 1, false, 5>(p, s);
      }
      return;
    }
  }
  if constexpr (CHUNK == 16) {
    if (p.stride == 2 && p.k <= 3 && shape.halves && !shape.eight) {
      launch_variant<16, 4, OPM, 1, false, 3>(p, s);
      return;
    }
  }
  const bool stride1 = p.stride == 1 && !p.upsample;
  if (stride1 && p.k == 1) launch_bound<CHUNK, OPM, -1>(p, shape, s);
  else if (CHUNK <= 32 && stride1 && p.k <= 3) launch_bound<CHUNK, OPM, CHUNK <= 32 ? -3 : 0>(p, shape, s);
  else launch_bound<CHUNK, OPM, 0>(p, shape, s);
}

// Launches with few workgroups (maps of a few tiles) are bound by what one workgroup does in
// sequence: a round trip per channel chunk, and weights that only the occupied CUs stream in (a 7 x 7
// x 512 layer: 32 workgroups, 0.9 MB of fp32-mode weights through each CU's L1).  Splitting the
// channels over workgroups too turns the chunks into parallel round trips and spreads the weights;
// it costs the exchange of the shares, about 3 us at the end of the workgroup.  The split fills the
// chip's 512 resident 8-wave workgroups and stops there: beyond them it only adds exchanges
// (measured, us per layer in fp32 mode, not split / 512 / 768 workgroups: 512 channels on 7 x 7
// 22.2 / 14.4 / 14.3; 512 on 16 x 16 23.9 / 18.7 / 18.5; 256 on 14 x 14 15.2 / 13.0 / 13.2; 768 -> 256 on 32 x
// 32 33.2 / 31.4 / 38.8; 256 on 32 x 44 20.4 / not split / 27.3; four waves per workgroup are slower
// on all of them).  Chunks of 64 channels (5 x 5 at stride 2 and, in fp32 mode, larger kernels at
// stride 1: 32; fp32, not split / split: 288 -> 96, 5 x 5 on 20 x 20 31.9 / 16.3, 512 -> 256 on 28 x 28 56 / 45).
// What a workgroup saves, channels times taps, has to be worth the exchange: 512 in fp32 mode (256 in
// launches of up to 16 workgroups), 1024 (640 up to 64) in the modes whose contraction is shorter.
// Measured, not split / split: 1 x 1 in fp32 mode, 128 -> 128 on 14 x 14 8.9 / 10.3, 512 -> 128 on 14 x 14 11.7 /
// 12.5 and on 7 x 7 11.9 / 11.1, 768 -> 128 on 7 x 7 14.1 / 11.8; bf16, 128 -> 128, 3 x 3 on 20 x 20 10.0 / 10.4, 64 -> 64, 5 x
// 5 at stride 2 on 112 x 112 11.3 / 12.4, 128 -> 256 on 48 x 48 14.9 / 13.8.
struct KSplit { int chunk = 0, chunks_each = 0, ks = 0; };  // ks == 0: not split
inline KSplit ksplit_for(const ConvParams& p) {
  KSplit r;
  const long long n = 2ll * p.go.tiles() * (p.c_out_pad / 32) * p.st.n;  // half-tile workgroups
  if (p.k <= 3 && p.gi.c % 64 == 0) r.chunk = 64;
  else if (p.stride == 2 && p.k <= 5 && p.gi.c % 32 == 0) r.chunk = 32;
  else if (p.fp32 && p.stride == 1 && p.k > 3 && p.gi.c % 32 == 0) r.chunk = 32;
  else return r;
  const int chunks = p.gi.c / r.chunk;
  const int want = (int)std::min<long long>(chunks, 512 / n);
  if (want < 2) return r;
  r.chunks_each = (chunks + want - 1) / want;
  const int saved = (chunks - r.chunks_each) * r.chunk * p.k * p.k;
  if (saved < (p.fp32 ? (n <= 16 ? 256 : 512) : (n <= 64 ? 640 : 1024))) return r;
  r.ks = (chunks + r.chunks_each - 1) / r.chunks_each;
  return r;
}

#include "conv_fold_impl.h"

template <int OPM>
void launch_any(const ConvParams& p, hipStream_t s) {
  if constexpr (OPM != kOpBf16) {  // (weights declared as bf16 are not folded)
    if (p.upsample && p.fold_list) {
      launch_fold<OPM>(p, s);
      return;
    }
  }
  const KSplit r = p.upsample ? KSplit() : ksplit_for(p);
  if (r.ks) {
    ConvParams q = p;
    q.ks = r.ks; q.ks_chunks = r.chunks_each;
    if (r.chunk == 64 && p.stride == 1 && p.k == 1) launch_variant<64, 8, OPM, 1, true, -1>(q, s);
    else if (r.chunk == 64 && p.stride == 1) launch_variant<64, 8, OPM, 1, true, 0>(q, s);
    else if (r.chunk == 64) launch_variant<64, 8, OPM, 1, true, 3>(q, s);
    else if (p.stride == 1) launch_variant<32, 8, OPM, 1, true, OPM == kOpF32 ? 0 : 5>(q, s);  // (fp32 mode only)
    else launch_variant<32, 8, OPM, 1, true, 5>(q, s);
    return;
  }
  const Shape shape = shape_for(p);
  switch (shape.chunk) {
    case 128: launch_shape<128, OPM>(p, shape, s); break;
    case 64: launch_shape<64, OPM>(p, shape, s); break;
    case 32: launch_shape<32, OPM>(p, shape, s); break;
    default: launch_shape<16, OPM>(p, shape, s); break;
  }
}

// A block's first conv (3 x 3, stride 2) and its shortcut (1 x 1, stride 2) read the same tensor and need
// nothing of each other.  As launches of their own each is a few microseconds of fixed latency with
// most of the chip idle (ResNet-18, 64 -> 128 channels on 56 x 56 8.3 and 6.8 us, in one launch 8.1; 128 ->
// 256 on 28 x 28 10.1 and 7.8, now 9.1; 256 -> 512 on 14 x 14 9.6 and 10.8, now 9.8).  Only where both take the
// eight-wave half-tile variant with 64-channel chunks anyway, so that neither's sums change, and at
// most one splits its channels over workgroups (they would share the scratch).
inline bool pairable(const ConvParams& p) {
  if (p.stride != 2 || p.upsample) return false;
  const KSplit r = ksplit_for(p);
  if (r.ks) return r.chunk == 64;
  const Shape shape = shape_for(p);
  return shape.chunk == 64 && shape.eight;
}
inline bool pair_supported(const ConvParams& a, const ConvParams& b) {
  return pairable(a) && pairable(b) && !(ksplit_for(a).ks && ksplit_for(b).ks) && a.st.n == b.st.n;
}
template <int OPM>
void launch_pair(const ConvParams& a, const ConvParams& b, hipStream_t s) {
  auto prepare = [](const ConvParams& p) {
    ConvParams q = p;
    const KSplit r = ksplit_for(p);
    q.ks = r.ks ? r.ks : 1;
    q.ks_chunks = r.ks ? r.chunks_each : (p.gi.c + 63) / 64;
    return variant_launch<64, 8, OPM, 1, true>(q);
  };
  const ConvLaunch la = prepare(a), lb = prepare(b);
  const int na = (int)(la.grid.x * la.grid.y), nb = (int)(lb.grid.x * lb.grid.y);
  ConvPair q{la.q, lb.q, na};
  hipLaunchKernelGGL(conv_mfma_pair_kernel<OPM>, dim3(na + nb, 1, a.st.n), dim3(512), std::max(la.lds, lb.lds), s, q);
}

// The gate convs of a recurrent cell read one tensor.  In one launch the last, partly filled round of
// workgroups and the start of the next launch come once instead of four times (the four convs of a
// ConvLSTM cell, 69 -> 64 channels on 256 x 352, fp32: 192 -> 168 us).  For the variant of four-wave half
// tiles with 32-channel chunks, the one such layers take, and kernels of one size: a launch takes the variant and
// the LDS of its largest (3 x 3 beside 1 x 1, 33 -> 40 channels on 480 x 640, fp32: 311 us apart, 331 together).
// 1 x 1 kernels up to 4096 workgroups each (96 -> 96 on 480 x 640, split: 498 / 531).  A launch each / one launch, over
// 824 cells of two to four convs, 64 x 72 to 480 x 640, ms in all: fp32 131.1 / 129.0, split 111.1 / 109.0, bf16 97.6 /
// 96.0; none is slower by more than the spread.  (bf16 takes old z late here and holds five waves per SIMD.)
inline bool batchable(const ConvParams& p) {
  if (p.stride != 1 || p.upsample || ksplit_for(p).ks) return false;
  const Shape shape = shape_for(p);
  const long long n = 2ll * p.go.tiles() * (p.c_out_pad / 32) * p.st.n;
  return shape.chunk == 32 && shape.halves && !shape.eight && (p.k > 1 || n <= 4096);
}
inline bool batch_supported(const ConvParams& a, const ConvParams& b) { return batchable(a) && batchable(b) && a.k == b.k; }
template <int OPM>
void launch_batch(const ConvParams* convs, int n, hipStream_t s) {
  ConvBatch q = {};
  unsigned blocks = 0;
  size_t lds = 0;
  for (int i = 0; i < n; ++i) {
    const ConvLaunch l = variant_launch<32, 4, OPM, 1, false>(convs[i]);
    q.p[i] = l.q;
    q.first[i] = (int)blocks;
    blocks += l.grid.x * l.grid.y;
    lds = std::max(lds, l.lds);
  }
  q.n = n;
  const dim3 grid(blocks, 1, convs[0].st.n);
  if (convs[0].k == 1) hipLaunchKernelGGL((conv_mfma_batch_kernel<OPM, -1>), grid, dim3(256), lds, s, q);
  else if (convs[0].k <= 3) hipLaunchKernelGGL((conv_mfma_batch_kernel<OPM, -3>), grid, dim3(256), lds, s, q);
  else hipLaunchKernelGGL((conv_mfma_batch_kernel<OPM, 0>), grid, dim3(256), lds, s, q);
}

// Copies the phase records of this translation unit's kernels to `host` (32 x u64 each, at most
// max_records); returns how many workgroups have written one since the last reset, or -1 in a
// build without phase stamps.
inline int phase_stamps_read(unsigned long long* host, int max_records, bool reset) {
#ifdef EVCONV_PHASE_STAMPS
  static unsigned counts[kPhaseClasses][32];
  if (hipDeviceSynchronize() != hipSuccess) return -2;
  if (hipMemcpyFromSymbol(counts, HIP_SYMBOL(g_phase_n), sizeof(counts)) != hipSuccess) return -2;
  unsigned n = 0, taken = 0;
  for (unsigned c = 0; c < kPhaseClasses; ++c) {
    const unsigned take = std::min(std::min(counts[c][0], kPhaseClassRecords), (unsigned)std::max(max_records, 0) - taken);
    if (host && take &&
        hipMemcpyFromSymbol(host + (size_t)taken * 32, HIP_SYMBOL(g_phase), sizeof(unsigned long long) * 32 * take,
                            sizeof(unsigned long long) * 32 * kPhaseClassRecords * c) != hipSuccess) return -2;
    n += counts[c][0];
    taken += take;
  }
  if (reset) {
    static const unsigned zero[kPhaseClasses][32] = {};
    if (hipMemcpyToSymbol(HIP_SYMBOL(g_phase_n), zero, sizeof(zero)) != hipSuccess) return -2;
  }
  return (int)n;
#else
  (void)host; (void)max_records; (void)reset;
  return -1;
#endif
}

}  // namespace

}  // namespace evk
