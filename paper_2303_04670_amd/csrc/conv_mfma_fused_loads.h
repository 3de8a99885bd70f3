// Operands of the ADDs and of the sparsification layer that are folded into a matrix-core conv's epilogue (text, see
// conv_mfma_epilogue.h).
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f) {
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) f_skip[f][it] = f_zold[f][it] = 0.0f;
    if (f >= p.n_fused) continue;
    const uint64_t skip_mine = mine(skip_word[f]);
    const __amdgpu_buffer_rsrc_t skip_rsrc = out_rsrc(at_stream(p.fused[f].skip, so));
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) f_skip[f][it] = ep_load(skip_rsrc, has(skip_mine, it), it);
    if (p.fused[f].keeps_z && !dense) {
      const __amdgpu_buffer_rsrc_t fz_rsrc = out_rsrc(at_stream(p.fused[f].z, so));
#pragma unroll
      for (int it = 0; it < EP_ITERS; ++it) f_zold[f][it] = ep_load(fz_rsrc, has(site_mine, it), it);
    }
  }

#pragma unroll
  for (int it = 0; it < EP_ITERS; ++it) sp_delta[it] = 0.0f;
  if (p.sp.delta && !dense) {
    sp_k = *at_stream(p.sp.step, so);
    const __amdgpu_buffer_rsrc_t d_rsrc = out_rsrc(at_stream(p.sp.delta, so));
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) sp_delta[it] = ep_load(d_rsrc, sp_k > 0.0f && has(site_mine, it), it);
  }
