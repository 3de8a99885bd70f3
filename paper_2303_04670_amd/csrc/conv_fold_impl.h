// A 5 x 5 conv (stride 1, padding 2) that reads a bilinear x2 up-sampling, with the up-sampling folded into its
// weights (fp32 and split modes; conv_mfma_impl.h includes this into its namespace).
//
// Both are linear (Eq.9-10), so the outputs of one phase (row parity, column parity) are a conv of the stored
// tensor with four taps per dimension instead of five: 16 products where the up-sampled tensor takes 25.  The
// four rows under an output of stored row q start at row q - 2 (even outputs) or q - 1 (odd ones).  Stored rows
// outside the image read as the first or last row, as the operator clamps them.  What remains is the conv's
// zero padding, which concerns the outputs of the first and of the last stored row only: up-sampled rows that
// do not exist must not count.  Those rows that lie on the near side of the output then come down to one vector of
// taps on the stored row itself (kFoldTop, kFoldBottom), and the same holds for columns.  So a phase has
// kFoldVectors x kFoldVectors weight taps, pairs of a row and a column vector; a workgroup away from the
// border contracts the 4 x 4 of the middle, one that holds sites of a border 5 x 4 or 5 x 5 of them, and a
// lane whose site a pair does not concern contracts a zero (no tap is taken off again: an infinity stays
// what it is, and nothing cancels).
//
// Workgroup = one phase of a tile of stored sites (MB 2: two blocks of 32 sites) or of half a tile (MB 1), 32
// output channels.  Its four waves split the contraction as in conv_mfma_body.h: the units of a chunk (a tap x 16
// channels) are dealt round-robin to them and their sums meet in LDS; in fp32 mode the units of the odd waves have negated
// weights (conv_mfma_negated).  A tile of which the image holds four rows or four columns at most is one
// block: the upper rows, or eight rows of four columns.
//
// Bound by the matrix pipe in large launches (with 16 streams busy 0.72 / 0.71 / 0.56 of the cycles in which a CU holds
// waves in the depth net's three decoders, at 1.9 to 2.0 GHz) and, in small ones, by the phases of a workgroup.  Before, tiles with border
// sites interpolated the up-sampled tensor and contracted all 25 taps: the decoders in fp32 57.0 / 47.9 / 47.2
// us, now 47.4 / 42.1 / 43.7; split 39.3 / 31.6 / 35.3, now 32.7 / 27.5 / 32.8; 16 streams 609 / 564 / 603, now 538 / 497 / 560; 128
// -> 64 behind 30 x 40 20.7, now 17.5.  (All four phases of half a tile in one workgroup, which gathers once for them,
// are slower than a workgroup each: 85 / 55 / 44 us, the fragments of four weight sets pass through one L1.)
template <int CHUNK, int MB, int OPM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, MB == 2 ? 3 : 8))) void conv_fold_kernel(ConvParams p) {
  touch_params<ConvParams>();
  asm volatile("" ::"s"(p.go.h), "s"(p.go.w), "s"(p.go.c), "s"(p.go.tx), "s"(p.gi.c), "s"(p.dense), "s"(p.n_fused), "s"(p.c_out_pad),
               "s"(p.occ_in), "s"(p.in), "s"(p.z), "s"(p.w_fold), "s"(p.fold_list), "s"(p.lo_h), "s"(p.lo_w), "s"(p.st.stride),
               "s"(p.wg_swap), "s"(p.tx_magic));
  const size_t so = (size_t)blockIdx.z * p.st.stride;
  constexpr int PARTS = op_parts(OPM), NB = 32, NT = 256;
  constexpr int NW = 4, NROWS = 4 * MB;  // waves; rows of stored sites
  constexpr int PH = NROWS + 3, PW = 11;               // patch
  constexpr int CS = patch_site_words(CHUNK, OPM), LO = CHUNK / 2;
  constexpr int RP = ((PW * CS + 31) / 64) * 64 + 32;  // row pitch, see conv_mfma_body.h
  constexpr int NV = CHUNK / 4;
  constexpr int MAXG = (PH * PW * NV + NT - 1) / NT;   // gathered float4 per thread
  constexpr int PATCH = CS;                            // a site of zeros stands before the patch
  constexpr int SUB = 32;                              // channels whose units are dealt together
  extern __shared__ __align__(16) float s_mem[];
  __shared__ uint64_t s_nz[(2 + kMaxFusedAdds) * 4];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  EVK_PHASE_OPEN();
  const bool dense = p.dense != 0;
  const int H = p.lo_h, W = p.lo_w, Cin = p.gi.c, Cout = p.go.c;
  // workgroup -> list entry (a tile, or a tile and which half of it), phase; phases vary fastest, so that an XCD
  // (every eighth workgroup) reads one of the four weight sets
  const int wg_tile = p.wg_swap ? blockIdx.y : blockIdx.x, wg_co = p.wg_swap ? blockIdx.x : blockIdx.y;
  const int phase = wg_tile & 3, entry = p.fold_list[wg_tile >> 2];
  const int tile = MB == 1 ? entry >> 1 : entry, r0 = MB == 1 ? (entry & 1) * 4 : 0;
  const int s_tx = (W + 7) >> 3;
  const int tile_y = fast_div(tile, s_tx, p.tx_magic), tile_x = tile - tile_y * s_tx;
  const int y0 = tile_y * 8 + r0, x0 = tile_x * 8;
  const int fpy = phase >> 1, fpx = phase & 1;
  const int iy0 = y0 - 2 + fpy, ix0 = x0 - 2 + fpx;
  const bool flat = MB == 1 || y0 + 4 >= H;      // the first block holds all rows
  const bool narrow = MB == 2 && x0 + 4 >= W;    // it holds all columns, as eight rows of four

  // activity: one row of bits per lane, rows and columns clamped to the image
  auto clamped = [](int v, int n) { return min(max(v, 0), n - 1); };
  unsigned row_byte[3];
  const int rtx0 = ix0 >> 3;
  {
    const __amdgpu_buffer_rsrc_t occ_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)at_stream(p.occ_in, so), 0, ((H + 7) >> 3) * s_tx * 8, 0x00020000);
    const int gy = clamped(iy0 + min(lane, PH - 1), H);
    const unsigned off = (unsigned)(__mul24(gy >> 3, s_tx) * 8 + (gy & 7));
#pragma unroll
    for (int i = 0; i < 3; ++i)
      row_byte[i] = (unsigned char)__builtin_amdgcn_raw_buffer_load_b8(occ_rsrc, off, clamped(rtx0 + i, s_tx) * 8, 0);
  }
  // lane = site of the stored tile; its output's occupancy in the fused ADDs' other inputs
  const int ly = lane >> 3, lx = lane & 7;
  const bool exists = (unsigned)(ly - r0) < (unsigned)NROWS && tile_y * 8 + ly < H && x0 + lx < W;
  uint64_t skip_raw[kMaxFusedAdds];
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f) {
    skip_raw[f] = 0;
    if (f >= p.n_fused || dense) continue;
    if (exists) skip_raw[f] = at_stream(p.fused[f].occ_skip, so)[(2 * tile_y + (ly >> 2)) * p.go.tx + 2 * tile_x + (lx >> 2)];
  }

  // ---- patch gather: per thread a fixed list of (LDS offset, byte offset into the input)
  constexpr unsigned kOob = 0x80000000u;
  constexpr int kSites = PH * PW;
  const int v4 = tid % NV;
  int lds_off[MAXG];  // (until the occupancy is known: patch row and column in bits 16-23 and 24-31)
  unsigned g_off[MAXG];
#pragma unroll
  for (int j = 0; j < MAXG; ++j) {
    // (a thread whose j-th item lies beyond the region repeats the last site's: the same value to the same place)
    const int site = min(tid / NV + j * (NT / NV), kSites - 1);
    const int py = __umul24(site, (65536 + PW - 1) / PW) >> 16, px = site - __umul24(py, PW);
    lds_off[j] = (PATCH + __umul24(py, RP) + px * CS + v4 * 2) | (py << 16) | (px << 24);
    g_off[j] = (unsigned)(clamped(iy0 + py, H) * W + clamped(ix0 + px, W)) * (unsigned)Cin * 4u + v4 * 16u;
  }
  static_assert(PATCH + PH * RP < 65536, "LDS offsets of the gather fit 16 bits");

  auto of_lane = [](int i, unsigned v) { return (unsigned)__builtin_amdgcn_ds_bpermute(i * 4, (int)v); };
  unsigned bits;
  EVK_PHASE(kPhOccInLds);
  {
    const int lo = max(0, -ix0), hi = min(PW, W - ix0);  // columns inside the image
    const unsigned span = (row_byte[0] | (row_byte[1] << 8) | (row_byte[2] << 16)) >> (ix0 - rtx0 * 8);
    const unsigned inside = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    const unsigned left = (span >> lo) & 1u ? (1u << lo) - 1u : 0u;
    const unsigned right = (span >> (hi - 1)) & 1u ? ((1u << PW) - 1u) & ~((1u << hi) - 1u) : 0u;
    bits = lane < PH ? (dense ? (1u << PW) - 1u : (span & inside) | left | right) : 0u;
  }
  EVK_PHASE(kPhBitRows);
#pragma unroll
  for (int j = 0; j < MAXG; ++j) {
    const int py = (lds_off[j] >> 16) & 0xff, px = lds_off[j] >> 24;
    lds_off[j] &= 0xffff;
    const unsigned row = of_lane(py, bits);
    if (!((row >> px) & 1u)) g_off[j] = kOob;
  }
  // (c_in: see conv_mfma_body.h)
  const int tail = Cin & 3;
  const bool ragged = (Cin % CHUNK) != 0;
  const __amdgpu_buffer_rsrc_t in_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)at_stream(p.in, so), 0, H * W * Cin * 4 + (tail ? 12 : 0), 0x00020000);
  float4 pre[MAXG];
  auto fetch = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
      unsigned off = g_off[j];
      if (ragged && c0 + v4 * 4 >= Cin) off = kOob;
      pre[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, off, c0 * 4, 0));
    }
  };
  fetch(0);
  // touched word: any of the 4 x 4 stored sites under an output
  uint64_t touched_word;
  {
    unsigned rows = 0;
#pragma unroll
    for (int ky = 0; ky < 4; ++ky) rows |= of_lane(ly - r0 + ky, bits);
    touched_word = __ballot(exists & (dense | (((rows >> lx) & 0xfu) != 0)));
  }
  uint64_t skip_word[kMaxFusedAdds];
  uint64_t site_word = touched_word;  // sites this workgroup has to visit in the epilogue
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f) {
    skip_word[f] = 0;
    if (f >= p.n_fused) continue;
    skip_word[f] = dense ? touched_word
                         : __ballot(((skip_raw[f] >> ((2 * (ly & 3) + fpy) * 8 + 2 * (lx & 3) + fpx)) & 1ull) != 0);
    site_word |= skip_word[f];
  }
  if (site_word == 0) return;
  const bool conv_on = touched_word != 0;

  // Epilogue addressing: lane = output channel co0 + lane % 32; its sites are those of accumulator registers
  // i = wave * EP_ITERS + it (of all blocks): row i / 4, column 4 * half + i % 4; where a block is eight rows of four
  // columns, row 2 * (i / 4) + half and column i % 4.
  constexpr int EP_ITERS = 16 * MB / NW, EP_ROWS = EP_ITERS / 4;
  const int co = lane & 31, co0 = wg_co * NB;
  const int ey = y0 + (narrow ? 2 * wave * EP_ROWS + half : wave * EP_ROWS), ex = x0 + (narrow ? 0 : 4 * half);
  const unsigned ep_voff = (unsigned)(((2 * ey + fpy) * p.go.w + 2 * ex + fpx) * Cout + co0 + co) * 4u;
  const unsigned ep_col = 8u * (unsigned)Cout, ep_row = (unsigned)(narrow ? 2 * p.go.w : p.go.w) * ep_col;
  auto ep_at = [&](int it) { return (unsigned)(it >> 2) * ep_row + (unsigned)(it & 3) * ep_col; };
  auto ep_bit = [](int it) { return (it >> 2) * 8 + (it & 3); };
  const int out_bytes = p.go.h * p.go.w * Cout * 4;
  constexpr unsigned kSkipAccess = 0x80000000u;
  const bool co_ok = co0 + co < Cout;
  // (a lane's rows of a word, closed up where they are every second one; beyond the first block: none)
  auto mine = [&](uint64_t w) {
    uint64_t v = w >> ((r0 + wave * EP_ROWS) * 8 + 4 * half);
    if (narrow) {
      v = (w >> (8 * half)) & 0x00ff00ff00ff00ffull;
      v = (v | (v >> 8)) & 0x0000ffff0000ffffull;
      v = ((v | (v >> 16)) & 0xffffffffull) >> (wave * EP_ROWS * 8);
    }
    return co_ok ? v : 0ull;
  };
  auto has = [&](uint64_t sp, int it) { return ((sp >> ep_bit(it)) & 1ull) != 0; };
  auto out_rsrc = [&](const void* ptr) { return __builtin_amdgcn_make_buffer_rsrc((void*)ptr, 0, out_bytes, 0x00020000); };
  auto ep_load = [&](const __amdgpu_buffer_rsrc_t& r, bool on, int it) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, on ? ep_voff : kSkipAccess, ep_at(it), 0));
  };
  const uint64_t touched_mine = mine(touched_word), site_mine = mine(site_word);

  // one float4 of patch channels into the patch buffer, as bf16 parts (see conv_mfma_body.h)
  auto put = [&](int off, const float4& x, bool large) __attribute__((always_inline)) {
    uint2 h, m, l;
    h.x = pack_bf16x2(x.x, x.y);
    h.y = pack_bf16x2(x.z, x.w);
    float4 r = make_float4(x.x - __uint_as_float(h.x << 16), x.y - __uint_as_float(h.x & 0xffff0000u),
                           x.z - __uint_as_float(h.y << 16), x.w - __uint_as_float(h.y & 0xffff0000u));
    m.x = pack_bf16x2(r.x, r.y);
    m.y = pack_bf16x2(r.z, r.w);
    if (PARTS == 3) {
      l.x = pack_bf16x2(r.x - __uint_as_float(m.x << 16), r.y - __uint_as_float(m.x & 0xffff0000u));
      l.y = pack_bf16x2(r.z - __uint_as_float(m.y << 16), r.w - __uint_as_float(m.y & 0xffff0000u));
      if (large) {
        split3_large(x.x, 0, h.x, m.x, l.x);
        split3_large(x.y, 16, h.x, m.x, l.x);
        split3_large(x.z, 0, h.y, m.y, l.y);
        split3_large(x.w, 16, h.y, m.y, l.y);
      }
      *(uint2*)&s_mem[off + 2 * LO] = l;
    }
    *(uint2*)&s_mem[off] = h;
    *(uint2*)&s_mem[off + LO] = m;
  };
  auto stash = [&](int c0) __attribute__((always_inline)) {
    if (tail) {
      const int left = Cin - (c0 + v4 * 4);
      if (left > 0 && left < 4) {
#pragma unroll
        for (int j = 0; j < MAXG; ++j) {
          if (left < 2) pre[j].y = 0.0f;
          if (left < 3) pre[j].z = 0.0f;
          pre[j].w = 0.0f;
        }
      }
    }
    float largest = 0.0f;
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
      put(lds_off[j], pre[j], false);
      if (PARTS == 3)
        largest = fmaxf(fmaxf(fmaxf(fabsf(pre[j].x), fabsf(pre[j].y)), fmaxf(fabsf(pre[j].z), fabsf(pre[j].w))), largest);
    }
    if (PARTS == 3 && __builtin_expect(largest >= kBf16Overflow, 0)) {
#pragma unroll
      for (int j = 0; j < MAXG; ++j) put(lds_off[j], pre[j], true);
    }
  };

  // ---- contraction
  floatx16 acc[MB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[a][i] = 0.0f;
  const int m = lane & 31, cop = p.c_out_pad;
  const int cin_rows = (Cin + 31) / 32 * 4;  // 16-byte weight rows per tap: 8 bf16
  const int my = narrow ? m >> 2 : m >> 3, mx = narrow ? m & 3 : m & 7;  // site of this lane in the first block
  const int a_lane = PATCH + my * RP + mx * CS + half * 4;
  const unsigned w_plane = (unsigned)(kFoldVectors * kFoldVectors * cin_rows * cop) * 16u, w_set = w_plane * PARTS;
  const __amdgpu_buffer_rsrc_t w_rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p.w_fold + (size_t)phase * w_set), 0, (int)w_set, 0x00020000);
  const unsigned w_lane = (unsigned)(half * cop + co0 + m) * 16u;
  // Taps of this workgroup: row vectors 0-3 (and the top's or the bottom's) x column vectors likewise.  Lane j of
  // the tables: this wave's j-th unit of 32 channels.
  const bool top = y0 == 0, bottom = y0 + NROWS >= H, left_edge = x0 == 0, right_edge = x0 + 8 >= W;
  int n_mine;
  unsigned w_table;
  int a_table;
  const int nr = 4 + (top | bottom), nc = 4 + (left_edge | right_edge);
  {
    const int n_units = nr * nc * 2;
    n_mine = (n_units - wave + NW - 1) / NW;
    const int u = min(wave + lane * NW, n_units - 1);
    const int tap = u >> 1, kg = u & 1;
    const int rv = __umul24(tap, nc == 5 ? 13108 : 16384) >> 16, cv = tap - rv * nc;
    const int row = rv < 4 ? rv : top ? kFoldTop : kFoldBottom, col = cv < 4 ? cv : left_edge ? kFoldTop : kFoldBottom;
    const int ky = rv < 4 ? rv : 2 - fpy, kx = cv < 4 ? cv : 2 - fpx;  // (the border's vectors: the stored row, column itself)
    a_table = __umul24(ky, RP) + kx * CS + kg * 8;
    w_table = (unsigned)((row * kFoldVectors + col) * cin_rows + kg * 2) * (unsigned)(cop * 16);
  }
  // Which taps concern this lane's site (bit r * nc + c: row vector r, column vector c): on the first row (column) the
  // stored row itself and what lies before it are replaced by the top's vector, on the last one itself and
  // what lies behind it by the bottom's.  The others read the zeros.
  auto vectors = [](int at, int n, int par) {  // of a site in row (column) `at` of n; vector 4 is the border's
    return at == 0 ? (0xfu & ~((2u << (2 - par)) - 1u)) | 16u : at == n - 1 ? ((1u << (2 - par)) - 1u) | 16u : 0xfu;
  };
  unsigned concerns[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const unsigned rows = vectors(y0 + 4 * b + my, H, fpy), cols = vectors(x0 + mx, W, fpx) & ((1u << nc) - 1u);
    concerns[b] = 0;
#pragma unroll
    for (int r = 0; r < 5; ++r) concerns[b] |= (rows >> r) & 1u ? cols << (r * nc) : 0u;
  }

  struct BF { float4 h, m, l; };
  auto b_load = [&](int c0, int j) __attribute__((always_inline)) {
    const unsigned soff = __builtin_amdgcn_readlane(w_table, j) + (unsigned)((c0 >> 3) * (cop * 16));
    BF f;
    f.h = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff, 0));
    f.m = f.l = f.h;
    if (PARTS == 3) f.m = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff + w_plane, 0));
    f.l = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff + (PARTS - 1) * w_plane, 0));
    return f;
  };
  // A ring of two weight fragments: the next unit's is requested before a unit is contracted.  (A ring of four and
  // patch fragments a unit ahead cost the registers of a fourth wave: slower wherever waves are many.)
  BF ring[2];
  // the patch fragment of unit j of the 32 channels that start at LDS word `at` of a site
  auto a_load = [&](int j, int at, int b) __attribute__((always_inline)) {
    const int concerned = __builtin_amdgcn_sbfe((int)concerns[b], (unsigned)((wave + j * NW) >> 1), 1);  // -1 or 0
    const float* const ap = &s_mem[(a_lane + at + b * 4 * RP + __builtin_amdgcn_readlane(a_table, j)) & concerned];
    BF f;
    f.h = *(const float4*)ap;
    f.m = PARTS == 3 ? *(const float4*)(ap + LO) : f.h;
    f.l = *(const float4*)(ap + (PARTS - 1) * LO);
    return f;
  };
  auto mm = [](floatx16& c, const float4& a, const float4& b) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  };
  auto unit = [&](floatx16& c, const BF& a, const BF& b) __attribute__((always_inline)) {
    if (PARTS == 3) {
      mm(c, a.l, b.h);
      mm(c, a.m, b.m);
      mm(c, a.h, b.l);
      mm(c, a.m, b.h);
      mm(c, a.h, b.m);
    } else {
      mm(c, a.l, b.h);
      mm(c, a.h, b.l);
    }
    mm(c, a.h, b.h);
  };

  EVK_PHASE(kPhAddressed);
  if (tid < CS / 4) *(float4*)&s_mem[tid * 4] = make_float4(0.f, 0.f, 0.f, 0.f);
  static_assert(CS % 4 == 0, "16-byte pieces");
  const bool two = !flat && !narrow;  // (uniform)
  ring[0].h = ring[0].m = ring[0].l = make_float4(0.f, 0.f, 0.f, 0.f);
  if (conv_on) ring[0] = b_load(0, 0);
  EVK_PHASE(kPhFirstIssued);
#ifdef EVCONV_PHASE_STAMPS
  unsigned long long ph_contract = 0, ph_change = 0;
#endif
  auto contract = [&](auto two_tag) __attribute__((always_inline)) {
    constexpr bool TWO = decltype(two_tag)::value;
    for (int c0 = 0; c0 < Cin; c0 += CHUNK) {
#ifdef EVCONV_PHASE_STAMPS
      const unsigned long long ph_a = wall_clock64();
#endif
      if (c0) __syncthreads();
      stash(c0);
      __syncthreads();
      if (c0 + CHUNK < Cin) fetch(c0 + CHUNK);
#ifdef EVCONV_PHASE_STAMPS
      const unsigned long long ph_b = wall_clock64();
      ph_change += ph_b - ph_a;
      if (c0 == 0) EVK_PHASE(kPhFirstPatchInLds);
#endif
#pragma unroll
      for (int sub = 0; sub < CHUNK / SUB; ++sub) {
        const int cs = c0 + sub * SUB, at = sub * (SUB / 2);
        int j = 0;
        auto step = [&](int i) __attribute__((always_inline)) {  // unit j + i; i is known at compile time
          // (after the last unit of these channels the next ones' first: the ring starts at 0 again)
          ring[1 - i] = b_load(cs, j + i + 1);
          // (left to itself the compiler requests it among the unit's last MFMAs: half tiles 10-20 % slower)
          __builtin_amdgcn_sched_barrier(0);
          const BF a0 = a_load(j + i, at, 0), a1 = TWO ? a_load(j + i, at, MB - 1) : a0;
          __builtin_amdgcn_sched_barrier(0);
          unit(acc[0], a0, ring[i]);
          if (TWO) unit(acc[MB - 1], a1, ring[i]);
        };
        for (; j + 2 <= n_mine; j += 2) {
          step(0);
          step(1);
        }
        if (j < n_mine) step(0);
        if (cs + SUB < Cin) ring[0] = b_load(cs + SUB, 0);
      }
#ifdef EVCONV_PHASE_STAMPS
      ph_contract += wall_clock64() - ph_b;
#endif
    }
  };
  // (a copy of the loop each: with a test for the second block in it, 3 % slower)
  if (conv_on) {
    if (MB == 2 && two) contract(std::bool_constant<MB == 2>{});
    else contract(std::false_type{});
  }
  EVK_PHASE(kPhChunksDone);
#ifdef EVCONV_PHASE_STAMPS
  if (tid == 0 && ph_slot < kPhaseRecords) {
    g_phase[ph_slot][kPhContractionTicks] = ph_contract;
    g_phase[ph_slot][kPhChunkChangeTicks] = ph_change;
  }
#endif

  // ---- epilogue: its operands are requested before the waves' sums meet
  const __amdgpu_buffer_rsrc_t z_rsrc = out_rsrc(at_stream(p.z, so)), o_rsrc = out_rsrc(at_stream(p.out, so));
  float z_old[EP_ITERS], f_skip[kMaxFusedAdds][EP_ITERS], f_zold[kMaxFusedAdds][EP_ITERS], sp_delta[EP_ITERS];
  float sp_k = 0.0f;
#pragma unroll
  for (int it = 0; it < EP_ITERS; ++it) z_old[it] = ep_load(z_rsrc, !dense && has(touched_mine, it), it);
  {
#include "conv_mfma_fused_loads.h"
  }
  EVK_PHASE(kPhFusedRequested);
  float v_sum[EP_ITERS];
  // (fp32 mode: the weights are stored times a power of two, those of the odd units negated)
  const float unscale = p.w_fold_unscale;
  // the waves' sums meet in LDS: [wave][register][lane]
  constexpr int SLOT = MB * 1024;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16 * MB; ++i)
    s_mem[wave * SLOT + i * 64 + lane] = PARTS == 3 ? acc[i / 16][i % 16] * (wave & 1 ? -unscale : unscale) : acc[i / 16][i % 16];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < EP_ITERS; ++it) {
    const float* const q = &s_mem[(wave * EP_ITERS + it) * 64 + lane];
    v_sum[it] = (q[0] + q[SLOT]) + (q[2 * SLOT] + q[3 * SLOT]);
  }

  EVK_PHASE(kPhReduced);
#ifdef EVCONV_PHASE_STAMPS
  __builtin_amdgcn_s_waitcnt(0);
  EVK_PHASE(kPhArrived);
#endif
  const float bias = (dense && p.bias && co_ok) ? p.bias[co0 + co] : 0.0f;
  uint64_t nz_mine = 0, nz_fused_mine[kMaxFusedAdds] = {0, 0}, nz_sp_mine = 0;
#include "conv_mfma_epilogue.h"
  EVK_PHASE(kPhEpilogueDone);
  EVK_PHASE(kPhFlagsBallot);

  // A site is nonzero where one of its 32 channels is: lanes 0-31 hold a site, lanes 32-63 the one four columns
  // further right (one row further down).
  auto collect = [&](int slot, uint64_t mine_bits) {
    uint64_t w = 0;
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) {
      const uint64_t b = __ballot(((mine_bits >> ep_bit(it)) & 1ull) != 0);
      const unsigned lo = (unsigned)b != 0 ? 1u : 0u, hi = (unsigned)(b >> 32) != 0 ? 1u : 0u;
      w |= (uint64_t)(lo | (narrow ? hi << 8 : hi << 4)) << ((it >> 2) * (narrow ? 16 : 8) + (it & 3));
    }
    if (lane == 0) s_nz[slot * NW + wave] = w << ((r0 + wave * EP_ROWS * (narrow ? 2 : 1)) * 8 & 63);
  };
  collect(0, nz_mine);
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f)
    if (f < p.n_fused) collect(1 + f, nz_fused_mine[f]);
  if (p.sp.delta) collect(1 + kMaxFusedAdds, nz_sp_mine);
  EVK_PHASE(kPhFlagsInLds);
  __syncthreads();
  EVK_PHASE(kPhFlagsBarrier);
  auto nz_word = [&](int slot) {
    uint64_t w = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) w |= s_nz[slot * NW + i];
    return w;
  };
  if (tid < 4 * (4 + 2 * kMaxFusedAdds)) {
    // Four lanes per set: the phase's bits go to the words of the four up-sampled tiles over the stored tile,
    // one per lane; site (y, x) is bit (2 * (y % 4) + fpy, 2 * (x % 4) + fpx) of tile (y / 4, x / 4).
    const int set = tid >> 2;
#include "conv_mfma_set_words.h"
    if (bits && words) {
      const int a = (tid >> 1) & 1, b = tid & 1;
      uint64_t spread = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned nib = (unsigned)(bits >> ((4 * a + r) * 8 + 4 * b)) & 0xfu;
        const unsigned wide = (nib & 1u) | ((nib & 2u) << 1) | ((nib & 4u) << 2) | ((nib & 8u) << 3);
        spread |= (uint64_t)wide << ((2 * r + fpy) * 8 + fpx);
      }
      if (spread)
        atomicOr((unsigned long long*)&at_stream(words, so)[(2 * tile_y + a) * p.go.tx + 2 * tile_x + b], (unsigned long long)spread);
    }
  }
  EVK_PHASE(kPhEnd);
}

template <int CHUNK, int MB, int OPM>
void launch_fold_variant(const ConvParams& p, hipStream_t s) {
  constexpr int PH = 4 * MB + 3, PW = 11, CS = patch_site_words(CHUNK, OPM);
  constexpr size_t patch = (size_t)PH * (((PW * CS + 31) / 64) * 64 + 32) + CS, sums = MB * 4096;
  const int tiles = ((p.lo_h + 7) >> 3) * ((p.lo_w + 7) >> 3), n_co = p.c_out_pad / 32;
  const int wgs = (MB == 1 ? ((p.lo_h + 3) >> 2) * ((p.lo_w + 7) >> 3) : tiles) * 4;
  ConvParams q = p;
  if (MB == 1) q.fold_list += tiles;  // (the half tiles stand behind the tiles)
  q.tx_magic = magic32(tiles, (p.lo_w + 7) >> 3);
  // (which operand every XCD reads in full: see variant_launch)
  q.wg_swap = (long long)p.k * p.k * p.go.c > (long long)p.lo_h * p.lo_w && wgs <= 65535;
  const dim3 grid = q.wg_swap ? dim3(n_co, wgs, p.st.n) : dim3(wgs, n_co, p.st.n);
  hipLaunchKernelGGL((conv_fold_kernel<CHUNK, MB, OPM>), grid, dim3(256), std::max(patch, sums) * sizeof(float), s, q);
}

// Whole tiles use a weight fragment twice; half tiles are twice the workgroups.  Measured, whole / half tiles, us, fp32 and
// split mode (workgroups in whole tiles): 128 -> 64 channels behind 30 x 40 23.0 / 17.5, 16.9 / 12.9 (160); 256 -> 128 behind
// 32 x 44 49.8 / 46.3, 31.7 / 30.7 (384); 64 -> 32 behind 80 x 92 18.7 / 18.6, 14.0 / 14.0 (480); 128 -> 64 behind 57 x 66 36.6 /
// 37.9, 23.9 / 25.7 (576); 256 -> 128 behind 45 x 45 70.8 / 68.9, 41.7 / 44.4 (576); 128 -> 64 behind 64 x 88 41.5 / 42.8, 26.3 / 31.0
// (704); 64 -> 32 behind 91 x 121 25.0 / 27.9, 17.7 / 21.5 (768); 256 -> 128 behind 32 x 44, four streams 153 / 166, 87 / 104 (1536); 16
// streams 609 / 686, 373 / 449.  Half tiles are bound by round trips: chunks of 64 channels where there are any (64 / 32: 46.3 /
// 46.5, 30.7 / 31.5 behind 32 x 44, 29.1 / 30.2, 20.6 / 21.9 behind 20 x 23).
template <int OPM>
void launch_fold(const ConvParams& p, hipStream_t s) {
  const long long whole = 4ll * ((p.lo_h + 7) >> 3) * ((p.lo_w + 7) >> 3) * (p.c_out_pad / 32) * p.st.n;
  if (whole >= kFoldWholeTiles) launch_fold_variant<32, 2, OPM>(p, s);
  else if (p.gi.c % 64 == 0) launch_fold_variant<64, 1, OPM>(p, s);
  else launch_fold_variant<32, 1, OPM>(p, s);
}
