// The body of a matrix-core conv workgroup (conv_mfma_impl.h includes it into functions; no include
// guard).  What the including function declares: the template parameters CHUNK, NW, OPM, MB, MODE, UPS, KSP,
// S2K, PAIR and LATE, the arguments p, this workgroup's stream offset so, its tile (or list entry) and channel
// block wg_tile and wg_ck.
  const bool dense = p.dense != 0;
  constexpr int PARTS = op_parts(OPM);     // bf16 parts of an operand
  constexpr int NB = 32;                   // output channels per workgroup
  constexpr int NT = NW * 64;
  static_assert(MB == 1 || NW == 4, "whole tiles are for launches that fill the chip with four waves each");
  // LDS site stride in 4-byte words; stride / 4 is odd (the eight sites of a patch row fall into
  // eight distinct 16-byte slots of the banks).  A site holds one plane of CHUNK bf16 per part.
  constexpr int CS = patch_site_words(CHUNK, OPM);
  constexpr int LO = CHUNK / 2;  // word offset between the planes of a site
  constexpr int UCH = 16;        // channels per unit
  constexpr int KG = CHUNK / UCH;     // units per tap and chunk
  constexpr int NV = CHUNK / 4;       // float4 per patch site
  constexpr int MAXV = (max_patch_sites(CHUNK, MB, S2K) * NV + NT - 1) / NT;  // patch float4 per thread
  constexpr int SUBS = 2 / MB;        // workgroups per tile
  constexpr int NROWS = 4 * MB;       // output rows of this workgroup
  constexpr int NSITES = 32 * MB;
  constexpr int EP_SITES = NT / NB;   // sites per epilogue pass
  constexpr int EP_ITERS = NSITES / EP_SITES;
  static_assert(EP_ITERS >= 1 && EP_SITES <= 32, "epilogue mapping");
  constexpr int NACC = MB * 16;  // accumulator registers of a lane
  constexpr int SLOT = NACC * 64;     // floats per partial-sum slot
  constexpr int CSL = CHUNK + 4;      // UPS: site stride of the low-resolution fp32 buffer
  constexpr int LPMAX = 10;           // UPS: a 14-row patch has sources in at most 14 / 2 + 3 rows
  // gathered float4 per thread
  constexpr int MAXG = MODE == kInterpolate ? (LPMAX * LPMAX * NV + NT - 1) / NT : MAXV;
  extern __shared__ __align__(16) float s_mem[];
  __shared__ unsigned s_arrived;  // KSP: shares of the block that were there before this one
  __shared__ uint64_t s_nz[(2 + kMaxFusedAdds) * NW];  // nonzero-site bits per wave: conv, each fused ADD, fused sparsification
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  EVK_PHASE_OPEN();
  const int n_co = p.c_out_pad / NB;
  const int ks = KSP ? fast_div(wg_ck, n_co, p.co_magic) : 0, wg_co = KSP ? wg_ck - ks * n_co : wg_ck;
  const int sub = wg_tile % SUBS;
  const int tile = wg_tile / SUBS;
  constexpr bool ups = MODE == kInterpolate;  // this workgroup interpolates its patch
  const int r0 = sub * NROWS;  // first tile row of this workgroup
  const uint64_t row_mask = MB == 2 ? ~0ull : (0xffffffffull << (32 * sub));
  const int tile_y = fast_div(tile, p.go.tx, p.tx_magic), tile_x = tile - tile_y * p.go.tx;
  const int s = p.stride, K = p.k;
  const int H = p.gi.h, W = p.gi.w, Cin = p.gi.c, Cout = p.go.c;
  const int iy0 = (tile_y * 8 + r0) * s - p.pad, ix0 = tile_x * 8 * s - p.pad;
  const int PH = (NROWS - 1) * s + K, PW = 7 * s + K;
  // The region whose stored occupancy is read: the patch itself, or (UPS) the low-resolution
  // sources of the patch: rows (iy0 >> 1) - 1 .. and columns likewise, PH / 2 + 3 by PW / 2 + 3
  // sites (a source index is i/2 - 1, i/2 or i/2 + 1 before clamping to the image).
  const int SH = UPS ? p.lo_h : H, SW = UPS ? p.lo_w : W;  // stored tensor
  const int s_ty = (SH + 7) >> 3, s_tx = (SW + 7) >> 3;
  const int gy0 = ups ? (iy0 >> 1) - 1 : iy0, gx0 = ups ? (ix0 >> 1) - 1 : ix0;
  const int GH = ups ? PH / 2 + 3 : PH, GW = ups ? PW / 2 + 3 : PW;

  // Activity of the region as one row of bits per lane: bit x of lane y's `bits` is site (y, x).  A row
  // is a byte of each of at most four occupancy words, so every wave reads the bytes of its lanes' rows
  // itself and nothing before the first patch goes through LDS or a barrier.  (For a tile beyond the left
  // or right border a neighbour's byte is read; it is cut off with the columns outside the image.)
  const int rtx0 = gx0 >> 3, gy = gy0 + lane;
  const bool row_ok = lane < GH && (unsigned)gy < (unsigned)SH;
  // (read in a regular pass too, where they are not used: without a branch the loads are in flight while
  // the addresses below are worked out)
  unsigned row_byte[4];
  {
    const __amdgpu_buffer_rsrc_t occ_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)at_stream(p.occ_in, so), 0, s_ty * s_tx * 8, 0x00020000);
    const unsigned off = row_ok ? (unsigned)(__mul24(gy >> 3, s_tx) * 8 + (gy & 7)) : 0x80000000u;
#pragma unroll
    for (int rx = 0; rx < 4; ++rx)
      row_byte[rx] = (unsigned char)__builtin_amdgcn_raw_buffer_load_b8(occ_rsrc, off, min(max(rtx0 + rx, 0), s_tx - 1) * 8, 0);
  }

  // occupancy words of the fused ADD nodes' other inputs: requested first, so that their latency
  // runs alongside that of the input's occupancy words instead of after it
  uint64_t skip_raw[kMaxFusedAdds];
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f) {
    skip_raw[f] = 0;
    if (f >= p.n_fused || dense) continue;
    skip_raw[f] = at_stream(p.fused[f].occ_skip, so)[tile];
  }
  // While the occupancy words are on their way: everything about the gather that depends on the
  // tile's position only.
  // ---- patch gather: per thread a fixed list of (LDS offset, byte offset into the input)
  // The gathered region is the patch itself, or (UPS) its low-resolution source region, which
  // goes to a second fp32 buffer behind the patch buffer.
  constexpr unsigned kOob = 0x80000000u;
  // Row pitch of the patch in LDS (4-byte words).  The LDS serves a 16-byte read per lane in
  // groups of 16 lanes over 64 banks; the 16 lanes of an A-fragment read are two rows of eight
  // sites.  The site stride (an odd number of 16-byte slots) spreads a row's eight sites over
  // eight distinct slots; a row pitch of 128 bytes modulo 256 puts the next row's sites on the
  // other eight.  (Stride-2 layers read every other site and row: no pitch frees them of
  // conflicts, they keep the dense pitch.)
  const int RP = s == 1 ? ((PW * CS + 31) / 64) * 64 + 32 : PW * CS;
  float* const s_low = s_mem + PH * RP;  // UPS only
  const int last_site = GH * GW - 1;
  const int gw_magic = p.gw_magic[ups ? 1 : 0];  // site / GW == (site * gw_magic) >> 16 for site < 441
  const unsigned row_bytes = (unsigned)(SW * Cin) * 4u, g_origin = (unsigned)gy0 * row_bytes + (unsigned)(gx0 * Cin) * 4u;
  // (a thread whose j-th item lies beyond the region repeats the last site's: the same value goes to
  // the same place twice, and no item needs a test of its own, only one that is the same for the
  // whole workgroup where no thread has a j-th item)
  static_assert(NT % NV == 0, "a thread's items are of one channel group");
  const int v4 = tid % NV;  // channel group of this thread's items
  // (items go in pairs, so that the work of two of them overlaps)
  auto has_pair = [&](int j) { return j == 0 || (UPS && PARTS != 1) || j * (NT / NV) <= last_site; };
  int lds_off[MAXG];     // (until the occupancy is known: patch row and column in bits 16-23 and 24-31)
  unsigned g_off[MAXG];
#pragma unroll
  for (int j = 0; j < MAXG; ++j) {
    const int site = min(tid / NV + j * (NT / NV), last_site);
    // (24-bit products: full rate, unlike 32-bit ones)
    const int py = __umul24(site, gw_magic) >> 16, px = site - __umul24(py, GW);
    lds_off[j] = (ups ? site * CSL + v4 * 4 : __umul24(py, RP) + px * CS + v4 * 2) | (py << 16) | (px << 24);
    g_off[j] = g_origin + (unsigned)py * row_bytes + __umul24(px, Cin) * 4u + v4 * 16u;
  }
  // UPS: every patch element from its four sources in the low-resolution buffer, with the
  // weights and the summation order of the stand-alone up-sampling operator
  //
  // Work item = one 2 x 2 block of up-sampled sites (rows 2i+1, 2i+2, columns 2j+1, 2j+2) x four
  // channels: its four values come from the same four stored sites (rows i, i+1, columns j, j+1,
  // clamped to the image), so the four reads and the two horizontal sums per stored row are
  // shared; a site without an active source comes out as zero because inactive sources are
  // stored as zeros.  The items of a thread are the same for every chunk: offsets and masks are
  // worked out once.
  constexpr int MAXB = MODE == kInterpolate ? (8 * (MB == 2 ? 8 : 6) * NV + NT - 1) / NT : 1;  // <= 8 x 8 blocks (K <= 7)
  // per item two packed words: ib_src = source offset (12 bits) | row step (10) | column step (6);
  // ib_dst = patch offset + 4096 (16 bits) | write mask (4) | inside-the-image mask (4)
  int ib_src[MAXB], ib_dst[MAXB];
#pragma unroll
  for (int b = 0; b < MAXB; ++b) ib_src[b] = ib_dst[b] = 0;
  if (ups) {
    const int by0 = (iy0 - 1) >> 1, bx0 = (ix0 - 1) >> 1;
    const int nby = ((iy0 + PH - 2) >> 1) - by0 + 1, nbx = ((ix0 + PW - 2) >> 1) - bx0 + 1;
    const int nbx_magic = p.nbx_magic;  // blk / nbx == (blk * nbx_magic) >> 16 for blk < 64
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
      const int e = tid + b * NT;
      const int blk = e / NV, v = e - blk * NV;
      ib_src[b] = ib_dst[b] = 0;
      if (blk < nby * nbx) {
        const int bi = __umul24(blk, nbx_magic) >> 16, bj = blk - __umul24(bi, nbx);
        const int i = by0 + bi, j = bx0 + bj;
        const int cy0 = min(max(i, 0), SH - 1), cy1 = min(max(i + 1, 0), SH - 1);
        const int cx0 = min(max(j, 0), SW - 1), cx1 = min(max(j + 1, 0), SW - 1);
        ib_src[b] = (((cy0 - gy0) * GW + (cx0 - gx0)) * CSL + v * 4) | (((cy1 - cy0) * GW * CSL) << 12) |
                    (((cx1 - cx0) * CSL) << 22);
        const int py = 2 * i + 1 - iy0, px = 2 * j + 1 - ix0;  // patch coordinates of the block, -1 at least
        const int dst = py * RP + px * CS + v * 2 + 4096;
        int mask = 0;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const bool in_patch = py + r >= 0 && py + r < PH && px + c >= 0 && px + c < PW;
            const bool in_image = (unsigned)(iy0 + py + r) < (unsigned)H && (unsigned)(ix0 + px + c) < (unsigned)W;
            if (in_patch) mask |= 1 << (r * 2 + c);
            if (in_patch && in_image) mask |= 16 << (r * 2 + c);
          }
        ib_dst[b] = dst | (mask << 16);
      }
    }
  }

  // columns [lo, hi) of a region whose first one is image column x0, as a mask
  auto inside = [](int x0, int n, int width) {
    const int lo = max(0, -x0), hi = min(n, width - x0);
    return (hi >= 32 ? ~0u : ((1u << max(hi, 0)) - 1u)) & ~((1u << min(lo, 31)) - 1u);
  };
  auto of_lane = [](int i, unsigned v) { return (unsigned)__builtin_amdgcn_ds_bpermute(i * 4, (int)v); };
  const unsigned span = row_byte[0] | (row_byte[1] << 8) | (row_byte[2] << 16) | (row_byte[3] << 24);
  const unsigned src_bits = (dense ? ~0u : span >> (gx0 - rtx0 * 8)) & (row_ok ? inside(gx0, GW, SW) : 0u);  // the gathered region's
  EVK_PHASE(kPhOccInLds);
  unsigned bits = src_bits;  // the patch's
  if (ups) {
    // an up-sampled site is active where one of its four sources is: OR of two source rows, then of two
    // source columns (column 2b: stored columns b - 1 and b; column 2b + 1: b and b + 1; a column that
    // the clamped border replaces is the other one, and out of image it is a zero bit), interleaved
    const int iy = iy0 + lane, hy = iy >> 1;
    const int y0 = (iy & 1) ? hy : max(hy - 1, 0), y1 = (iy & 1) ? min(hy + 1, SH - 1) : hy;
    const unsigned src = of_lane(y0 - gy0, src_bits) | of_lane(y1 - gy0, src_bits);
    auto spread = [](unsigned v) {
      v = (v | (v << 8)) & 0x00ff00ffu;
      v = (v | (v << 4)) & 0x0f0f0f0fu;
      v = (v | (v << 2)) & 0x33333333u;
      return (v | (v << 1)) & 0x55555555u;
    };
    const unsigned up = spread((src | (src << 1)) & 0xffffu) | (spread((src | (src >> 1)) & 0xffffu) << 1);
    bits = lane < PH && (unsigned)iy < (unsigned)H ? (up >> (ix0 - 2 * gx0)) & inside(ix0, PW, W) : 0u;
  }

  EVK_PHASE(kPhBitRows);
  const int c_lo = KSP ? ks * p.ks_chunks * CHUNK : 0;
  // the gather's offsets, now conditioned on the occupancy (out of range where the site is inactive)
#pragma unroll
  for (int j = 0; j < MAXG; ++j) {
    const int py = (lds_off[j] >> 16) & 0xff, px = lds_off[j] >> 24;
    lds_off[j] &= 0xffff;
    const unsigned row = of_lane(py, src_bits);
    if (!((row >> px) & 1u)) g_off[j] = kOob;
  }
  // c_in need not be a multiple of four: the 16-byte load of a site's last channel group then
  // runs into the next site (buffer loads of dwords need dword alignment only); the foreign
  // components are zeroed on the way into LDS.  The range is extended by those 12 bytes so that
  // the last site's group is not rejected as a whole (every tensor of the workspace is followed
  // by padding or by another buffer of the workspace).
  const int tail = Cin & 3;
  const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)at_stream(p.in, so), 0, SH * SW * Cin * 4 + (tail ? 12 : 0), 0x00020000);
  float4 pre[MAXG];
  // c_in need not be a multiple of the chunk: channel groups beyond c_in read as zeros (their
  // weight rows are zero padding as well)
  const bool ragged = (Cin % CHUNK) != 0;
  auto fetch = [&](int c0) {
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
      if (!has_pair(j & ~1)) continue;
      unsigned off = g_off[j];
      if (ragged && c0 + v4 * 4 >= Cin) off = kOob;
      pre[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, off, c0 * 4, 0));
    }
  };
  // (requested before the touched set is worked out: where no site of the patch is active, nothing is read)
  fetch(c_lo);
  // touched word of this workgroup's rows (identical in all waves): OR of the K bit rows under a
  // site, then any of the K columns
  uint64_t touched_word;
  {
    const int ly = lane >> 3, lx = lane & 7;
    const int oy = tile_y * 8 + ly, ox = tile_x * 8 + lx;
    const int lr = ly - r0;
    unsigned rows = 0;
#pragma unroll
    for (int ky = 0; ky < 7; ++ky) {
      const unsigned row = of_lane(lr * s + ky, bits);
      rows |= ky < K ? row : 0u;
    }
    // (no short circuits: they would become branches)
    const bool exists = ((unsigned)lr < (unsigned)NROWS) & (oy < p.go.h) & (ox < p.go.w);
    const bool touched = exists & (dense | (((rows >> (lx * s)) & ((1u << K) - 1u)) != 0));
    touched_word = __ballot(touched);
  }
  // fused ADD nodes: their other input may be active where the conv is not
  uint64_t skip_word[kMaxFusedAdds];
  uint64_t site_word = touched_word;  // sites this workgroup has to visit in the epilogue
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f) {
    skip_word[f] = 0;
    if (f < p.n_fused) skip_word[f] = dense ? touched_word : (skip_raw[f] & row_mask);
    site_word |= skip_word[f];
  }
  if (site_word == 0) return;
  const bool conv_on = touched_word != 0;
  if (KSP && ks != 0 && !conv_on) return;  // nothing to contract: the first workgroup runs the epilogue alone
  const int c_hi = KSP ? min(p.gi.c, c_lo + p.ks_chunks * CHUNK) : p.gi.c;

  // Epilogue addressing.  Thread = output channel co0 + tid % 32 at the EP_ITERS sites
  // r0 * 8 + it * EP_SITES + tid / 32 (EP_SITES = 8 or 16: consecutive `it` are one or two tile rows
  // apart).  Every tensor of the output geometry is reached as buffer + the byte offset of the
  // thread's first site (one vector register for the whole kernel) + a scalar offset per `it`;
  // an access that must not happen gets an out-of-range vector offset (loads return 0, stores are
  // dropped).  The bits of a thread's sites are kept where they are in the 64-bit words, EP_SITES
  // bits apart: no per-site shifts, no 64-bit address arithmetic on the vector ALU.
  const int co = tid & (NB - 1);
  const int co0 = wg_co * NB;
  const int es = tid / NB;
  const int ey = tile_y * 8 + r0 + (es >> 3), ex = tile_x * 8 + (es & 7);
  const unsigned ep_voff =
      (unsigned)(((ey * p.go.w + ex) * Cout + co0 + co) * 4);
  const unsigned ep_step = (unsigned)((EP_SITES / 8) * p.go.w * Cout * 4);
  auto ep_at = [&](int it) { return (unsigned)it * ep_step; };
  auto ep_bit = [](int it) { return it * EP_SITES; };
  const int out_bytes = p.go.h * p.go.w * Cout * 4;
  constexpr unsigned kSkipAccess = 0x80000000u;
  constexpr uint64_t kMine = EP_SITES == 8 ? 0x0101010101010101ull : EP_SITES == 16 ? 0x0001000100010001ull : 0x1ull;
  // c_out need not be a multiple of 32: the last block's weights are zero-padded and the threads
  // of the channels that do not exist own no sites (they take no part in the epilogue)
  const bool co_ok = co0 + co < Cout;
  auto mine = [&](uint64_t w) { return co_ok ? (w >> (r0 * 8 + es)) & kMine : 0ull; };   // bit it * EP_SITES: site `it`
  auto has = [&](uint64_t sp, int it) { return ((sp >> (it * EP_SITES)) & 1ull) != 0; };
  auto out_rsrc = [&](const void* ptr) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)ptr, 0, out_bytes, 0x00020000);
  };
  auto ep_load = [&](const __amdgpu_buffer_rsrc_t& r, bool on, int it) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, on ? ep_voff : kSkipAccess, ep_at(it), 0));
  };
  const uint64_t touched_mine = mine(touched_word), site_mine = mine(site_word);
  const __amdgpu_buffer_rsrc_t z_rsrc = out_rsrc(at_stream(p.z, so));

  // old z values of the epilogue, requested now so that they arrive during the contraction
  // (KSP: by the one workgroup that runs the epilogue, when it knows that it does)
  float z_old[EP_ITERS];
  auto request_z = [&]() {
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) z_old[it] = ep_load(z_rsrc, !dense && has(touched_mine, it), it);
  };
  // (variants without registers to spare: after it)
  constexpr bool LATE_Z = LATE || (PARTS == 3 && NW == 4 && S2K == 5);
  if (!KSP && !LATE_Z) request_z();

  // one float4 of patch channels into the patch buffer, as the operand mode's bf16 parts
  // (large: some of the values a bf16 cannot round without overflow, or are infinite; a NaN makes every part NaN)
  auto put = [&](int off, const float4& x, bool large) __attribute__((always_inline)) {
    uint2 h, m, l;
    h.x = pack_bf16x2(x.x, x.y);
    h.y = pack_bf16x2(x.z, x.w);
    if (PARTS == 1) {
      *(uint2*)&s_mem[off] = h;
      return;
    }
    // x = hi + mid (+ lo): each part the bf16 rounding of what the parts before it leave (the
    // subtractions are exact); three parts hold all 24 bits of an fp32 value of 2^-110 and more
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
  auto max4 = [](const float4& x, float m) {
    return fmaxf(fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))), m);
  };
  auto stash = [&](int c0) {
    if (tail) {  // (uniform; nets with c_in % 4 == 0 pay nothing)
      const int left = Cin - (c0 + v4 * 4);  // channels of this thread's group inside c_in
      if (left > 0 && left < 4) {
#pragma unroll
        for (int j = 0; j < MAXG; ++j) {
          if (left < 2) pre[j].y = 0.0f;
          if (left < 3) pre[j].z = 0.0f;
          pre[j].w = 0.0f;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < MAXG; ++j) {
      if (!has_pair(j & ~1)) continue;
      if (ups) *(float4*)&s_low[lds_off[j]] = pre[j];
      else put(lds_off[j], pre[j], false);
    }
    // the rare large values are looked for once for all items: a branch per item would keep the items'
    // work apart
    if (PARTS == 3 && !ups) {
      float largest = 0.0f;
#pragma unroll
      for (int j = 0; j < MAXG; ++j)
        if (has_pair(j & ~1)) largest = max4(pre[j], largest);
      if (__builtin_expect(largest >= kBf16Overflow, 0)) {
#pragma unroll
        for (int j = 0; j < MAXG; ++j)
          if (has_pair(j & ~1)) put(lds_off[j], pre[j], true);
      }
    }
  };
  auto interpolate = [&]() {
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
      // (fp32 mode, whole tiles: unpacked here and not once before the chunk loop, where the unpacked
      // values, kept across the contraction, do not fit the registers)
      if (PARTS == 3 && MB == 2) asm volatile("" : "+v"(ib_src[b]), "+v"(ib_dst[b]));
      const int mask = ib_dst[b] >> 16;
      if (mask == 0) continue;
      const float* q = &s_low[ib_src[b] & 0xfff];
      const int dy = (ib_src[b] >> 12) & 0x3ff, dx = ib_src[b] >> 22;
      const float4 v00 = *(const float4*)q, v01 = *(const float4*)(q + dx);
      const float4 v10 = *(const float4*)(q + dy), v11 = *(const float4*)(q + dy + dx);
      // horizontal sums of the two stored rows for the odd (a) and the even (b) column, then the
      // vertical ones: the same products and order as wy0 * (wx0 * v00 + wx1 * v01) + wy1 * (...)
      auto hsum = [](float w0, const float4& l, float w1, const float4& r) {
        return make_float4(w0 * l.x + w1 * r.x, w0 * l.y + w1 * r.y, w0 * l.z + w1 * r.z, w0 * l.w + w1 * r.w);
      };
      const float4 a0 = hsum(0.75f, v00, 0.25f, v01), b0 = hsum(0.25f, v00, 0.75f, v01);
      const float4 a1 = hsum(0.75f, v10, 0.25f, v11), b1 = hsum(0.25f, v10, 0.75f, v11);
      const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
      const int dst = (ib_dst[b] & 0xffff) - 4096;
      auto block = [&](bool large) __attribute__((always_inline)) {
        if (mask & 1) put(dst, (mask & 16) ? hsum(0.75f, a0, 0.25f, a1) : zero, large);
        if (mask & 2) put(dst + CS, (mask & 32) ? hsum(0.75f, b0, 0.25f, b1) : zero, large);
        if (mask & 4) put(dst + RP, (mask & 64) ? hsum(0.25f, a0, 0.75f, a1) : zero, large);
        if (mask & 8) put(dst + RP + CS, (mask & 128) ? hsum(0.25f, b0, 0.75f, b1) : zero, large);
      };
      block(false);
      // (an interpolated value is no larger than its sources)
      if (PARTS == 3 && __builtin_expect(max4(v00, max4(v01, max4(v10, max4(v11, 0.0f)))) >= kBf16Overflow, 0)) block(true);
    }
  };

  floatx16 acc0, acc1;
#pragma unroll
  for (int i = 0; i < 16; ++i) { acc0[i] = 0.0f; acc1[i] = 0.0f; }
  // operand lane: k-group `half` (two groups of 32 lanes), row / column m of the block
  const int half = lane >> 5, m = lane & 31;
  const int mly = m >> 3, mlx = m & 7;  // site of this lane inside a block
  const int cop = p.c_out_pad;
  const int cin_pad = (Cin + CHUNK - 1) / CHUNK * CHUNK;    // the weights are zero-padded to whole chunks
  const int cin_rows = cin_pad >> 3;                        // 16-byte weight rows per tap: 8 bf16
  const int a_lane_off = mly * s * RP + mlx * s * CS + half * 4;
  const int a_blk1 = 4 * s * RP;  // the second block starts four tile rows further down
  // Units of a chunk: (tap u / kgn, channel group u % kgn), kgn = KG groups of 16 channels or, with
  // p.tail_units in a last chunk that c_in does not fill, as many as hold channels; unit
  // u_j = wave + j * NW is this wave's j-th.
  constexpr bool TAIL = !UPS && !KSP && S2K <= 0 && CHUNK == 32;  // the other variants' chunks are full or one group
  // bf16 and split modes, stride 2: the order of the sums is that of chunks of 16 channels (the taps
  // dealt to the waves, one group of 16 channels after the other), whichever chunk the launcher
  // takes.  The rounding of the next layer's operands turns a last-bit difference of an fp32 sum
  // into one of 16 (8) bits, so a launch shape that reordered them would show: the depth net in bf16
  // by 3.5e-3.
  const bool groups_in_order = S2K > 0 && PARTS != 3 && (!KSP || (PAIR && p.ks == 1));
  // fp32 mode, chunks of one unit (1 x 1 taps, 16 channels): waves 0 and 1 contract all of them, wave 1
  // with the weights negated in registers, and half of their difference is the sum (conv_mfma_negated)
  const bool pair = PARTS == 3 && CHUNK == 16 && K == 1;
  int n_mine = 0;
  // Both fragment addresses are a per-lane constant plus a per-unit part that is the same in all
  // lanes.  Lane j of a table register holds unit j's part (beyond the last unit: the last one's, so
  // that look-ahead loads stay unconditional and in bounds) and a readlane brings it into a scalar
  // register: worked out per unit in scalar arithmetic, the two parts were 20 scalar instructions a
  // unit, in a kernel whose vector and scalar units are both more than half busy.
  // B: buffer load with the lane part as vector offset and the unit part as scalar offset
  // (bytes; the launcher checks that the re-laid weights stay below 2 GiB).
  const unsigned w_plane = (unsigned)(K * K * cin_rows * cop) * 16u;  // the planes of the parts follow each other
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)(w_plane * PARTS), 0x00020000);
  const unsigned w_lane = (unsigned)(half * cop + co0 + m) * 16u;
  unsigned w_table = 0;  // byte offset of unit `lane`'s weight rows in a chunk that starts at channel 0
  int a_table = 0;       // offset of its patch sites, words
  auto set_units = [&](int c0) {  // for the chunk starting at channel c0
    const int kgn = TAIL && p.tail_units ? min(KG, (Cin - c0 + UCH - 1) / UCH) : KG;
    const int n_units = K * K * kgn;
    const int u = min(wave + lane * NW, n_units - 1);
    static_assert(!TAIL || KG == 2, "one or two groups per chunk");
    int tap = kgn == KG ? u / KG : u, kg = kgn == KG ? u % KG : 0;
    n_mine = max(0, (n_units - wave + NW - 1) / NW);
    if (groups_in_order) {
      const int n_taps = max(0, (K * K - wave + NW - 1) / NW);
      kg = 0;
#pragma unroll
      for (int g = 1; g < KG; ++g) kg += lane >= g * n_taps ? 1 : 0;
      tap = min(wave + (lane - kg * n_taps) * NW, K * K - 1);
      n_mine = n_taps * KG;
    }
    if (pair) n_mine = wave < 2 ? 1 : 0;
    const int ky = __umul24(tap, p.k_magic) >> 16, kx = tap - __umul24(ky, K);  // tap < 49
    a_table = __umul24(ky, RP) + kx * CS + kg * 8;  // a unit's 16 bf16 are 8 words
    w_table = (__umul24(tap, cin_rows) + kg * (UCH / 8)) * (unsigned)(cop * 16);  // 16-byte rows of 8 bf16
  };
  set_units(c_lo);
  // fragments of unit j of the chunk starting at channel c0
  auto b_load = [&](int c0, int j) {
    const unsigned soff = __builtin_amdgcn_readlane(w_table, j) + (unsigned)((c0 >> 3) * (cop * 16));
    BFrag f;
    f.h = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff, 0));
    f.m = f.l = f.h;
    if (PARTS == 3) f.m = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff + w_plane, 0));
    if (PARTS >= 2)
      f.l = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, w_lane, soff + (PARTS - 1) * w_plane, 0));
    return f;
  };
  // A fragment of unit j: the parts of this lane's site in both
  // 32-row blocks; unused members cost nothing
  auto a_load = [&](int j) {
    AFrag f;
    const float* ap = &s_mem[a_lane_off + __builtin_amdgcn_readlane(a_table, j)];
    f.h0 = *(const float4*)ap;
    f.h1 = MB == 2 ? *(const float4*)(ap + a_blk1) : f.h0;
    f.m0 = PARTS == 3 ? *(const float4*)(ap + LO) : f.h0;
    f.m1 = (PARTS == 3 && MB == 2) ? *(const float4*)(ap + a_blk1 + LO) : f.h0;
    f.l0 = PARTS >= 2 ? *(const float4*)(ap + (PARTS - 1) * LO) : f.h0;
    f.l1 = (PARTS >= 2 && MB == 2) ? *(const float4*)(ap + a_blk1 + (PARTS - 1) * LO) : f.h0;
    return f;
  };
  auto mm = [](floatx16& acc, const float4& a, const float4& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  };
  // products of one unit, the smallest terms first; what is left out is 2^-16 (split) or less than 2^-24
  // (fp32 mode: the largest rounding error of an fp32 product) of the product
  auto unit = [&](const AFrag& a, const BFrag& b) {
    if (PARTS == 3) {
      mm(acc0, a.l0, b.h);
      if (MB == 2) mm(acc1, a.l1, b.h);
      mm(acc0, a.m0, b.m);
      if (MB == 2) mm(acc1, a.m1, b.m);
      mm(acc0, a.h0, b.l);
      if (MB == 2) mm(acc1, a.h1, b.l);
      mm(acc0, a.m0, b.h);
      if (MB == 2) mm(acc1, a.m1, b.h);
      mm(acc0, a.h0, b.m);
      if (MB == 2) mm(acc1, a.h1, b.m);
    }
    if (PARTS == 2) {
      mm(acc0, a.l0, b.h);
      mm(acc0, a.h0, b.l);
      mm(acc0, a.h0, b.h);
      if (MB == 2) {
        mm(acc1, a.l1, b.h);
        mm(acc1, a.h1, b.l);
        mm(acc1, a.h1, b.h);
      }
      return;
    }
    mm(acc0, a.h0, b.h);
    if (MB == 2) mm(acc1, a.h1, b.h);
  };

  // Ring of three weight fragments, two units of look-ahead, no register copies: vector loads
  // complete in order, so each wait only covers loads issued two units earlier.  The first two
  // fragments of a chunk are requested before the barriers that precede it.
  BFrag bq0, bq1, bq2;
  bq0.h = bq0.m = bq0.l = make_float4(0.f, 0.f, 0.f, 0.f);
  bq1 = bq0;
  bq2 = bq0;
  EVK_PHASE(kPhAddressed);
  if (conv_on && n_mine > 0) {
    bq0 = b_load(c_lo, 0);
    bq1 = b_load(c_lo, 1);
  }
  EVK_PHASE(kPhFirstIssued);
#ifdef EVCONV_PHASE_STAMPS
  unsigned long long ph_contract = 0, ph_change = 0;
#endif
  for (int c0 = c_lo; conv_on && c0 < c_hi; c0 += CHUNK) {
#ifdef EVCONV_PHASE_STAMPS
    const unsigned long long ph_a = wall_clock64();
#endif
    if (c0 != c_lo) __syncthreads();  // all waves are done reading the previous chunk
    stash(c0);
    __syncthreads();
    if (ups) {
      interpolate();
      __syncthreads();
    }
    const bool more = c0 + CHUNK < c_hi;
    if (more) fetch(c0 + CHUNK);  // next chunk's patch, in flight during the contraction
#ifdef EVCONV_PHASE_STAMPS
    const unsigned long long ph_b = wall_clock64();
    ph_change += ph_b - ph_a;
    if (c0 == c_lo) EVK_PHASE(kPhFirstPatchInLds);
#endif
    if (n_mine <= 0) continue;    // more waves than units (1 x 1 taps): only help with the gather
    // bf16 mode: the A fragments run one unit ahead of their use (three names, two alive at a time),
    // so that an LDS read is in flight during the matrix instructions of the unit before it.  The
    // modes with several parts have no registers to spare for that and read each fragment at its use.
    constexpr bool APIPE = PARTS == 1;
    int j = 0;
    AFrag aq0 = a_load(0), aq1 = aq0, aq2 = aq0;
    // Requests first, then the unit's matrix instructions: left to itself the compiler moves the weight loads of a unit
    // among its last MFMAs and the patch reads next to their uses, and the wave waits for both (depth net
    // in bf16 206 -> 202 us, flow net 280 -> 272).  Not in the variants for any kernel that are held to five waves, whose
    // registers it takes.  Nor where a wave has few units of a chunk (a four-wave half tile's 1 x 1 kernels, 3 x 3 in
    // chunks of 16 channels) or short ones (3 x 3 in bf16), so that it holds up the way to the next chunk, nor in
    // fp32 convs split over workgroups in chunks of 32: barrier / none, 1 x 1, 16 -> 32 on 180 x 240, split 10.9 / 9.8 us;
    // 3 x 3, 96 -> 33 there, bf16 25.8 / 23.4 (where these have a single chunk it costs a little: 31 -> 26 on 82 x 260 8.6 /
    // 8.8); 7 x 7, 320 -> 320 on 14 x 14, fp32 34.1 / 31.8.
    constexpr bool FEW = NW == 4 && MB == 1 && !KSP &&
                         (S2K == 1 || (S2K == -1 && CHUNK <= 32) || (S2K == -3 && (CHUNK == 16 || OPM == kOpBf16)));
    constexpr bool SPLIT32 = KSP && OPM == kOpF32 && CHUNK == 32 && S2K == 0;
    constexpr bool FRONT = !FEW && !SPLIT32 && !(min_waves(CHUNK, NW, OPM, MB, MODE, KSP, S2K) == 5 && S2K == 0);
    auto in_front = []() __attribute__((always_inline)) { if (FRONT) __builtin_amdgcn_sched_barrier(0); };
    auto step = [&](AFrag& cur, AFrag& nxt, int jj, const BFrag& b) {
      if (APIPE) nxt = a_load(jj + 1); else cur = a_load(jj);
      in_front();
      unit(cur, b);
    };
    for (; j + 3 <= n_mine; j += 3) {
      bq2 = b_load(c0, j + 2);
      in_front();
      step(aq0, aq1, j, bq0);
      bq0 = b_load(c0, j + 3);
      in_front();
      step(aq1, aq2, j + 1, bq1);
      bq1 = b_load(c0, j + 4);
      in_front();
      step(aq2, aq0, j + 2, bq2);
    }
    if (pair && wave == 1) {  // (uniform; its only unit)
      auto flip = [](float4& v) {  // the signs of eight bf16
        uint4 u = __builtin_bit_cast(uint4, v);
        u.x ^= 0x80008000u; u.y ^= 0x80008000u; u.z ^= 0x80008000u; u.w ^= 0x80008000u;
        v = __builtin_bit_cast(float4, u);
      };
      flip(bq0.h); flip(bq0.m); flip(bq0.l);
    }
    if (j < n_mine) step(aq0, aq1, j, bq0);
    if (j + 1 < n_mine) step(aq1, aq2, j + 1, bq1);
    if (more) {
      if (TAIL && p.tail_units && c0 + 2 * CHUNK > Cin) set_units(c0 + CHUNK);  // (uniform; the next chunk is not full)
      bq0 = b_load(c0 + CHUNK, 0);
      bq1 = b_load(c0 + CHUNK, 1);
    }
#ifdef EVCONV_PHASE_STAMPS
    ph_contract += wall_clock64() - ph_b;
#endif
  }
  EVK_PHASE(kPhChunksDone);
#ifdef EVCONV_PHASE_STAMPS
  if (tid == 0 && ph_slot < kPhaseRecords) {
    g_phase[ph_slot][kPhContractionTicks] = ph_contract;
    g_phase[ph_slot][kPhChunkChangeTicks] = ph_change;
  }
#endif

  // operands of the fused ADD stages, requested together now so that one memory latency covers
  // all of them and the reduction below hides part of it
  float f_skip[kMaxFusedAdds][EP_ITERS], f_zold[kMaxFusedAdds][EP_ITERS];
  float sp_delta[EP_ITERS];  // residuals and rounding step of a fused sparsification layer
  float sp_k = 0.0f;
  auto request_fused = [&]() {
#include "conv_mfma_fused_loads.h"
  };
  // (the arguments of the epilogue, loaded together)
  asm volatile("" ::"s"(p.out), "s"(p.bias), "s"(p.act), "s"(p.occ_out), "s"(p.occ_touched), "s"(p.sp.delta), "s"(p.fused[0].skip),
               "s"(p.fused[0].z), "s"(p.fused[0].out), "s"(p.fused[0].occ_out), "s"(p.fused[0].occ_touched), "s"(p.fused[0].act),
               "s"(p.fused[0].keeps_z), "s"(p.fused[0].structural), "s"(p.fused[1].keeps_z), "s"(p.w_unscale));
  if (!KSP && LATE_Z) request_z();
  if (!KSP) request_fused();
  EVK_PHASE(kPhFusedRequested);
  // ---- reduce the NW partial sums through LDS: slots [NW][block*16 + reg][lane]
  // (fp32 mode: the weights are stored times a power of two, those of the odd waves' units negated;
  // see conv_mfma_negated and ConvParams::w_unscale)
  const float unscale = p.w_unscale * (pair ? 0.5f : 1.0f);
  auto spill = [&](float* part, float factor) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      part[i * 64 + lane] = PARTS == 3 ? acc0[i] * factor : acc0[i];
      if (MB == 2) part[(16 + i) * 64 + lane] = PARTS == 3 ? acc1[i] * factor : acc1[i];
    }
  };
  __syncthreads();
  spill(s_mem + wave * SLOT, wave & 1 ? -unscale : unscale);
  __syncthreads();
  EVK_PHASE(kPhReduced);
#ifdef EVCONV_PHASE_STAMPS
  __builtin_amdgcn_s_waitcnt(0);  // (separates waiting for the operands from the epilogue's own time)
  EVK_PHASE(kPhArrived);
#endif

  // epilogue: thread -> (output channel = tid % 32, EP_ITERS sites); accumulator element
  // (block b, register i, lane l) is local site b*32 + 8*(i/4) + 4*(l/32) + i%4, channel l%32
  // (nonzero bits are collected where the thread's sites are, EP_SITES bits apart, and shifted to
  // their place in the tile word once)
  uint64_t nz_mine = 0;
  uint64_t nz_fused_mine[kMaxFusedAdds] = {0, 0};
  uint64_t nz_sp_mine = 0;
  const __amdgpu_buffer_rsrc_t o_rsrc = out_rsrc(at_stream(p.out, so));
  // partial sum of local site ls = it * EP_SITES + es: the part of the LDS offset that depends on
  // the thread (es < 16), the rest is a constant per `it`
  const int off_mine = ((es >> 3) * 4 + (es & 3)) * 64 + ((es >> 2) & 1) * 32 + co;
  const float bias = (dense && p.bias && co_ok) ? p.bias[co0 + co] : 0.0f;
  // Straight-line code: a site this thread does not own gets an out-of-range offset (its stores
  // are dropped) instead of a branch around it, and the partial sums of all passes are read from
  // LDS up front, so that the passes are not a chain of LDS round trips.
  float v_sum[EP_ITERS];
#pragma unroll
  for (int it = 0; it < EP_ITERS; ++it) {
    constexpr int kRow = EP_SITES / 8;  // tile rows per `it`
    const int off = off_mine + (((it * kRow) >> 2) * 16 + ((it * kRow) & 3) * 4) * 64;
    float part[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) part[q] = NW == 8 ? s_mem[off + q * SLOT] + s_mem[off + (q + 4) * SLOT] : s_mem[off + q * SLOT];
    v_sum[it] = (part[0] + part[1]) + (part[2] + part[3]);
  }
  if (KSP) {
    if (conv_on && !(PAIR && p.ks == 1)) {
      // This workgroup's share of the sums goes to memory; the last of the p.ks workgroups to arrive
      // (a counter that it resets) adds all shares in the order of the channels, whatever the order
      // of arrival, and runs the epilogue; nobody waits for anybody.  Shares and counter are
      // written and read with device-scope accesses, which go past the XCDs' own L2s, and a share
      // is complete (s_waitcnt, all waves) before the counter is touched.  A fence would instead
      // write back and invalidate a whole L2, weights included.
      const size_t out_blk = (size_t)wg_tile * n_co + wg_co;
      float* const share = at_stream(p.ks_part, so) + out_blk * p.ks * (NSITES * NB) + tid;
#pragma unroll
      for (int it = 0; it < EP_ITERS; ++it)
        __hip_atomic_store(share + (size_t)ks * (NSITES * NB) + it * NT, v_sum[it], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) {
        unsigned* const cnt = at_stream(p.ks_count, so) + out_blk;
        const unsigned before = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == (unsigned)p.ks - 1u) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_arrived = before;
      }
      __syncthreads();
      if (s_arrived != (unsigned)p.ks - 1u) return;
      request_z();
      request_fused();
      asm volatile("" ::: "memory");
      // (all shares in flight, eight at a time: one round trip to memory instead of one per two shares;
      // those that do not exist are the last one again and not added)
#pragma unroll
      for (int it = 0; it < EP_ITERS; ++it) v_sum[it] = 0.0f;
      auto add_shares = [&](int q0, auto n_tag) {
        constexpr int N = decltype(n_tag)::value;
        float add[N][EP_ITERS];
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
          for (int it = 0; it < EP_ITERS; ++it)
            add[q][it] = __hip_atomic_load(share + (size_t)min(q0 + q, p.ks - 1) * (NSITES * NB) + it * NT, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
          for (int it = 0; it < EP_ITERS; ++it)
            if (q0 + q < p.ks) v_sum[it] += add[q][it];
      };
      if (p.ks == 2) add_shares(0, std::integral_constant<int, 2>{});
      else if (p.ks <= 4) add_shares(0, std::integral_constant<int, 4>{});
      else for (int q0 = 0; q0 < p.ks; q0 += 8) add_shares(q0, std::integral_constant<int, 8>{});
    } else {
      request_z();
      request_fused();
    }
  }
#include "conv_mfma_epilogue.h"
  EVK_PHASE(kPhEpilogueDone);
  // A site is nonzero where one of its 32 channels is: lanes 0-31 of a wave hold site es = 2 * wave
  // of every pass, lanes 32-63 site 2 * wave + 1, so one ballot per pass gives the wave's two site
  // bits; the waves' words meet in LDS (no atomics: 64 lanes hitting one LDS word are served one
  // after the other, about 2 us per instruction).
  auto lds_or = [&](int slot, uint64_t mine_bits) {
    uint64_t w = 0;
#pragma unroll
    for (int it = 0; it < EP_ITERS; ++it) {
      const uint64_t b = __ballot(((mine_bits >> (it * EP_SITES)) & 1ull) != 0);
      w |= (uint64_t)(((unsigned)b != 0 ? 1u : 0u) | ((unsigned)(b >> 32) != 0 ? 2u : 0u)) << (it * EP_SITES);
    }
    if (lane == 0) s_nz[slot * NW + wave] = w << (r0 * 8 + (64 / NB) * wave);
  };
  auto nz_word = [&](int slot) {
    uint64_t w = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) w |= s_nz[slot * NW + i];
    return w;
  };
  EVK_PHASE(kPhFlagsBallot);
  lds_or(0, nz_mine);
#pragma unroll
  for (int f = 0; f < kMaxFusedAdds; ++f)
    if (f < p.n_fused) lds_or(1 + f, nz_fused_mine[f]);
  if (p.sp.delta) lds_or(1 + kMaxFusedAdds, nz_sp_mine);
  EVK_PHASE(kPhFlagsInLds);
  __syncthreads();
  EVK_PHASE(kPhFlagsBarrier);
  if (tid < 4 + 2 * kMaxFusedAdds) {  // a lane per set
    const int set = tid;
#include "conv_mfma_set_words.h"
    if (bits && words) atomicOr((unsigned long long*)&at_stream(words, so)[tile], (unsigned long long)bits);
  }
  EVK_PHASE(kPhEnd);
