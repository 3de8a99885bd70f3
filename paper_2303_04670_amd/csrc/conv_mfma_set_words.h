    // Site bits of a matrix-core conv workgroup for set number `set` of up to 4 + 2 * (fused ADDs) (text, see
    // conv_mfma_epilogue.h): S and T of the conv, then T and S of each fused ADD (Eq.11b), then T and S of a fused
    // sparsification layer (its T is the active set of the stage it reads).  All words of those sets are
    // pre-zeroed and the other workgroups of a tile OR their share in.
    // S of the producer as seen by this workgroup's rows and channels
    uint64_t s_prev = dense ? touched_word : nz_word(0);
    uint64_t bits = set == 0 ? s_prev : (set == 1 && wg_co == 0) ? touched_word : 0ull;
    uint64_t* words = set == 0 ? p.occ_out : set == 1 ? p.occ_touched : nullptr;
#pragma unroll
    for (int f = 0; f < kMaxFusedAdds; ++f) {
      if (f >= p.n_fused) break;
      const auto& fa = p.fused[f];
      const uint64_t t_f = s_prev | skip_word[f];  // Eq.11b
      const uint64_t nz_f = nz_word(1 + f);
      const uint64_t s_f = (fa.structural || dense) ? t_f : nz_f;
      if (set == 2 + 2 * f) { bits = t_f; words = fa.occ_touched; }
      if (set == 3 + 2 * f) { bits = s_f; words = fa.occ_out; }
      s_prev = s_f;
    }
    if (p.sp.delta) {
      const uint64_t nz_sp = nz_word(1 + kMaxFusedAdds);
      if (set == 2 + 2 * kMaxFusedAdds) { bits = s_prev; words = p.sp.occ_touched; }
      if (set == 3 + 2 * kMaxFusedAdds) { bits = dense ? s_prev : nz_sp; words = p.sp.occ_out; }
    }
