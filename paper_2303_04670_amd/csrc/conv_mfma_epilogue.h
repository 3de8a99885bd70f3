// The epilogue of a matrix-core conv, text that conv_mfma_body.h and conv_fold_impl.h include into a workgroup's
// body (no include guard): the accumulated tensor, the activation increment, folded ADDs and a folded
// sparsification layer, at the EP_ITERS sites of one output channel that a thread owns.  What the including
// code declares: p, so, dense, bias; v_sum (the contraction), z_old, f_skip, f_zold, sp_delta, sp_k (operands); has(word, it),
// ep_bit(it) (site `it` in touched_mine, site_mine and the nz words below), ep_voff + ep_at(it) (its byte offset), z_rsrc,
// o_rsrc, out_rsrc, kSkipAccess.  It leaves the nonzero sites in nz_mine, nz_fused_mine and nz_sp_mine.
  auto ep_store_at = [&](const __amdgpu_buffer_rsrc_t& r, unsigned voff, int it, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, ep_at(it), 0);
  };
  // Activations other than none / ReLU need branches (exp, tanh); nets made of the two simple
  // ones, the usual case, take a loop without any: every decision that is the same for the whole
  // workgroup becomes a select, so that the passes can be interleaved freely (a branch per
  // decision and pass made each pass a chain of kernel-argument loads and waits).
  bool simple_acts = p.act == kActNone || p.act == kActRelu;
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f)
    if (f < p.n_fused && p.fused[f].keeps_z && !(p.fused[f].act == kActNone || p.fused[f].act == kActRelu))
      simple_acts = false;
  // (one copy per number of fused ADDs, for one ADD with and without an accumulated tensor: a stage
  // that does not exist would still issue its stores)
  auto epilogue_simple = [&](auto sp_tag, auto nf_tag, auto kz_tag) {
    constexpr bool HAS_SP = decltype(sp_tag)::value;
    constexpr int NF = decltype(nf_tag)::value;   // fused ADDs
    constexpr int KZ = decltype(kz_tag)::value;   // they keep a z: 0 no, 1 yes, 2 looked up
    const bool relu0 = p.act == kActRelu;
    bool f_kz[kMaxFusedAdds], f_relu[kMaxFusedAdds];
    __amdgpu_buffer_rsrc_t f_out_r[kMaxFusedAdds], f_z_r[kMaxFusedAdds];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      f_kz[f] = KZ == 2 ? p.fused[f].keeps_z != 0 : KZ == 1;
      f_relu[f] = f_kz[f] && p.fused[f].act == kActRelu;
      // (a z that does not exist is stored nowhere: its offsets are out of range)
      f_out_r[f] = out_rsrc(at_stream(p.fused[f].out, so));
      f_z_r[f] = out_rsrc(at_stream(f_kz[f] ? p.fused[f].z : p.out, so));
    }
    const __amdgpu_buffer_rsrc_t sp_delta_r = out_rsrc(at_stream(HAS_SP ? p.sp.delta : p.out, so));
    const __amdgpu_buffer_rsrc_t sp_out_r = out_rsrc(at_stream(HAS_SP ? p.sp.out : p.out, so));
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) {
      const bool on_site = has(site_mine, it), on_conv = has(touched_mine, it);
      const unsigned at_site = on_site ? ep_voff : kSkipAccess, at_conv = on_conv ? ep_voff : kSkipAccess;
      // regular pass: z = v + bias, o = act(z); incremental: z += v, o = act(z_new) - act(z_old)
      // (z_old reads as 0 in a regular pass, so ReLU's difference form serves both)
      const float v = v_sum[it];
      const float z_new = (dense ? bias : z_old[it]) + v;
      ep_store_at(z_rsrc, at_conv, it, z_new);
      float o = relu0 ? fmaxf(z_new, 0.0f) - fmaxf(z_old[it], 0.0f) : (dense ? z_new : v);
      o = on_conv ? o : 0.0f;
      ep_store_at(o_rsrc, at_conv, it, o);
      if (o != 0.0f) nz_mine |= 1ull << ep_bit(it);
      // fused ADD nodes (Eq.11 followed by Eq.12-14): a = the value just produced, b = skip input
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const float lin = o + f_skip[f][it];
        float o2 = lin;
        if (KZ != 0) {
          const float z2_new = dense ? lin : f_zold[f][it] + lin;
          ep_store_at(f_z_r[f], f_kz[f] ? at_site : kSkipAccess, it, z2_new);
          o2 = f_relu[f] ? fmaxf(z2_new, 0.0f) - fmaxf(f_zold[f][it], 0.0f) : lin;
        }
        o2 = on_site ? o2 : 0.0f;
        ep_store_at(f_out_r[f], at_site, it, o2);
        if (o2 != 0.0f) nz_fused_mine[f] |= 1ull << ep_bit(it);
        o = o2;
      }
      // fused sparsification layer on the last stage's increment (Eq.3-8): x_corr = delta + x_inc,
      // y_inc = k floor(0.5 + x_corr / k), delta = x_corr - y_inc where x_inc is nonzero; elsewhere
      // y_inc = 0 and the residual stays.  A regular pass: identity, residual cleared.
      if (HAS_SP) {
#pragma clang fp contract(off)  // the residual is x_corr minus the rounded product, not a fused form
        const bool sp_on = sp_k > 0.0f, moved = o != 0.0f;   // (sp_k is 0 in a regular pass)
        const float x_corr = sp_delta[it] + o;
        const float q = sp_k * floorf(0.5f + x_corr / sp_k);
        const float y = sp_on ? (moved ? q : 0.0f) : o;
        ep_store_at(sp_delta_r, (dense || (sp_on && moved)) ? at_site : kSkipAccess, it, dense ? 0.0f : x_corr - y);
        ep_store_at(sp_out_r, at_site, it, y);
        if (y != 0.0f) nz_sp_mine |= 1ull << ep_bit(it);
      }
    }
  };
  if (simple_acts) {
    using std::integral_constant;
    if (p.sp.delta) {
      if (p.n_fused == 0) epilogue_simple(std::true_type{}, integral_constant<int, 0>{}, integral_constant<int, 0>{});
      else if (p.n_fused == 1) epilogue_simple(std::true_type{}, integral_constant<int, 1>{}, integral_constant<int, 2>{});
      else epilogue_simple(std::true_type{}, integral_constant<int, 2>{}, integral_constant<int, 2>{});
    } else {
      if (p.n_fused == 0) epilogue_simple(std::false_type{}, integral_constant<int, 0>{}, integral_constant<int, 0>{});
      else if (p.n_fused == 1 && !p.fused[0].keeps_z) epilogue_simple(std::false_type{}, integral_constant<int, 1>{}, integral_constant<int, 0>{});
      else if (p.n_fused == 1) epilogue_simple(std::false_type{}, integral_constant<int, 1>{}, integral_constant<int, 1>{});
      else epilogue_simple(std::false_type{}, integral_constant<int, 2>{}, integral_constant<int, 2>{});
    }
  } else {
#pragma unroll
  for (int it = 0; it < EP_ITERS; ++it) {
    const bool on_site = has(site_mine, it), on_conv = has(touched_mine, it);
    const unsigned at_site = on_site ? ep_voff : kSkipAccess, at_conv = on_conv ? ep_voff : kSkipAccess;
    float o;
    {
      const float v = v_sum[it];
      if (dense) {
        const float z = v + bias;
        ep_store_at(z_rsrc, at_conv, it, z);
        o = act_m(p.act, z);
      } else {
        const float z_new = z_old[it] + v;
        ep_store_at(z_rsrc, at_conv, it, z_new);
        o = (p.act == kActNone) ? v : act_m(p.act, z_new) - act_m(p.act, z_old[it]);
      }
      o = on_conv ? o : 0.0f;
      ep_store_at(o_rsrc, at_conv, it, o);
      if (o != 0.0f) nz_mine |= 1ull << ep_bit(it);
    }
    // fused ADD nodes (Eq.11 followed by Eq.12-14): a = the value just produced, b = skip input
#pragma unroll
    for (int f = 0; f < kMaxFusedAdds; ++f) {
      if (f >= p.n_fused) break;
      const auto& fa = p.fused[f];
      const float lin = o + f_skip[f][it];
      if (fa.keeps_z) {
        const __amdgpu_buffer_rsrc_t fz_rsrc = out_rsrc(at_stream(fa.z, so));
        if (dense) {
          ep_store_at(fz_rsrc, at_site, it, lin);
          o = act_m(fa.act, lin);
        } else {
          const float z2_old = f_zold[f][it];
          const float z2_new = z2_old + lin;
          ep_store_at(fz_rsrc, at_site, it, z2_new);
          o = (fa.act == kActNone) ? lin : act_m(fa.act, z2_new) - act_m(fa.act, z2_old);
        }
      } else {
        o = lin;
      }
      o = on_site ? o : 0.0f;
      ep_store_at(out_rsrc(at_stream(fa.out, so)), at_site, it, o);
      if (o != 0.0f) nz_fused_mine[f] |= 1ull << ep_bit(it);
    }
    // fused sparsification layer on the last stage's increment (Eq.3-8): x_corr = delta + x_inc,
    // y_inc = k floor(0.5 + x_corr / k), delta = x_corr - y_inc where x_inc is nonzero; elsewhere
    // y_inc = 0 and the residual stays.  A regular pass: identity, residual cleared.
    if (p.sp.delta) {
#pragma clang fp contract(off)  // the residual is x_corr minus the rounded product, not a fused form
      float y = o;
      if (dense) {
        ep_store_at(out_rsrc(at_stream(p.sp.delta, so)), at_site, it, 0.0f);
      } else if (sp_k > 0.0f) {
        const float x_corr = sp_delta[it] + o;
        y = (o != 0.0f) ? sp_k * floorf(0.5f + x_corr / sp_k) : 0.0f;
        ep_store_at(out_rsrc(at_stream(p.sp.delta, so)), (o != 0.0f) ? at_site : kSkipAccess, it, x_corr - y);
      }
      ep_store_at(out_rsrc(at_stream(p.sp.out, so)), at_site, it, y);
      if (y != 0.0f) nz_sp_mine |= 1ull << ep_bit(it);
    }
  }
  }
