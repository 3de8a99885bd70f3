// Matrix-core convolution, fp32 operands as three exact bf16 parts (six bf16 MFMAs per product, fp32
// accumulation; weights are [3 planes][tap][c_in/8][c_out][8] bf16), and the shape predicates shared
// by all operand modes.  The kernel itself is in conv_mfma_impl.h.
#include "conv_mfma_impl.h"

namespace evk {

bool conv_mfma_f32_supported(const ConvParams& p) {
  return p.gi.c >= 9 && p.go.c >= 16 && p.c_out_pad == (p.go.c + 31) / 32 * 32 &&  // (fewer input channels: the narrow-input kernel)
         (long long)p.gi.h * p.gi.w * p.gi.c * 4 < (1ll << 31) &&  // byte offsets of the gather fit 31 bits
         (long long)(p.go.h + 8) * p.go.w * p.go.c * 4 < (1ll << 31) &&  // those of the epilogue too
         (long long)p.k * p.k * ((p.gi.c + 127) / 128 * 128) * p.c_out_pad * 8 < (1ll << 31);  // and those of all weight planes
}
// a bilinear x2 up-sampling in front of this conv can be folded into its gather
bool conv_mfma_upsample_supported(const ConvParams& p) {
  return conv_mfma_f32_supported(p) && chunk_for(p) == 32 && p.stride == 1 && p.k <= 7;
}
// input channels of the re-laid weights: c_in rounded up to whole chunks of the variant that runs
int conv_mfma_padded_cin(const ConvParams& p) {
  const int chunk = chunk_for(p);
  return (p.gi.c + chunk - 1) / chunk * chunk;  // (c_in itself where the channels are split over workgroups)
}
// fp32 mode: whether the weights of (tap, input channel) are stored negated.  The bf16 matrix
// instruction does not round its sums symmetrically (measured: every layer's sums come out low by
// 0.3 to 0.8e-7 of their mean magnitude, with a random error of 1.4e-7), and an error of one sign
// survives where random ones average out, as in a global mean: ResNet-18's logits were off by 4.0e-7
// against 64 bits, 1.2e-7 with the chip's fp32 instruction.  So the units of the odd waves
// contract negated weights and their sums are negated again where the waves' sums meet.  A unit is
// 16 channels of one tap, dealt round-robin to an even number of waves: the parity of its number
// inside its chunk, tap * (groups of 16 channels in the chunk) + group, is its wave's.  Where a chunk
// is one unit (1 x 1 taps, chunks of 16 channels) there is nothing to alternate: two waves contract
// every unit, one of them with the weights negated in registers, and half of the difference is taken
// (48 -> 32 channels on 96 x 96: mean error against 64 bits -1.1e-8 of the mean magnitude with one
// wave, 1e-10 now; the second wave was idle).
bool conv_mfma_negated(const ConvParams& p, int tap, int ci) {
  const KSplit r = ksplit_for(p);
  const int chunk = r.ks ? r.chunk : chunk_for(p), c0 = ci / chunk * chunk;
  if (p.k == 1 && chunk == 16) return false;
  const int groups = p.tail_units ? std::min(chunk, (p.gi.c - c0 + 15) / 16 * 16) / 16 : chunk / 16;
  return (tap * groups + (ci - c0) / 16) & 1;
}
// per stream: shares of the sums and arrival counters of a conv whose channels are split over workgroups
void conv_mfma_split_scratch(const ConvParams& p, size_t* part_floats, size_t* counters) {
  const KSplit r = ksplit_for(p);
  const size_t blocks = (size_t)p.go.tiles() * 2 * (p.c_out_pad / 32);
  *part_floats = r.ks ? blocks * r.ks * 32 * 32 : 0;
  *counters = r.ks ? blocks : 0;
}
bool conv_mfma_batch_supported(const ConvParams& a, const ConvParams& b) { return batch_supported(a, b); }
bool conv_mfma_pair_supported(const ConvParams& a, const ConvParams& b) { return pair_supported(a, b); }
void launch_conv_mfma_f32(const ConvParams& p, hipStream_t s) { launch_any<kOpF32>(p, s); }
void launch_conv_mfma_f32_batch(const ConvParams* convs, int n, hipStream_t s) { launch_batch<kOpF32>(convs, n, s); }
void launch_conv_mfma_f32_pair(const ConvParams& a, const ConvParams& b, hipStream_t s) { launch_pair<kOpF32>(a, b, s); }
int conv_mfma_f32_phase_stamps(unsigned long long* host, int max_records, bool reset) {
  return phase_stamps_read(host, max_records, reset);
}

}  // namespace evk
