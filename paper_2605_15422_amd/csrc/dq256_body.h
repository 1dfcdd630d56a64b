// Body of the dQ workgroup in dq256.h and dq256.hip: workgroup `bid` of `nblk`, 512 threads; STATS: it may have to form the row statistics
// (p.make_stats()).  Text and not a function: called from the kernel its main loop is laid out otherwise and takes 1 to 3 % longer.
  using C = Cfg<D>;
  constexpr int KS = C::KS, RB = C::RB, CPR = C::CPR, TILE_BYTES = C::TILE_BYTES, STAGE_BYTES = C::STAGE_BYTES;
  constexpr int XCH_OFF = C::XCH_OFF, OUT_RS = C::OUT_RS, IPT = C::IPT, RPI = C::RPI, NRO = C::NRO, EBLK = C::EBLK;
  constexpr bool LOADER = C::LOADER;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  QBlock b;
  if (!decode_qblock<BN>(p, b, bid, nblk)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int P = b.P, R = b.R, W = p.window;
  const int n_ctx_run = b.n_ctx - b.c0;
  const int n_tiles = b.n_tiles;

  if (wave < 4) {
    // ================================= producer ==============================================
    const float c = p.scale_log2;
    const int head = b.hk * p.G + b.hc * p.GP + wave / p.RSH;
    const int row0 = b.blk_row0 + (wave % p.RSH) * 32;
    const int row = row0 + l32;
    const bool wave_valid = row0 < R;

    bf16x8 qf[KS], dof[KS];
    float lse2, negd;
    {
      const int64_t grow = b.row_begin + min(row, R - 1);
      const u16* qp = p.q.ptr + grow * p.q.ts + (int64_t)head * p.q.hs + hi * 8;
      const u16* dop = p.dout.ptr + grow * p.dout.ts + (int64_t)head * p.dout.hs + hi * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
        dof[ks] = *reinterpret_cast<const bf16x8*>(dop + ks * 16);
      }
      lse2 = p.lse[(int64_t)head * p.total + grow] * LOG2E;
      if (STATS && p.make_stats()) {
        const u16* op = p.o.ptr + grow * p.o.ts + (int64_t)head * p.o.hs + hi * 8;
        float t[KS];
        constexpr int GRP = 4;   // (at most GRP operands of O next to the Q and dO fragments)
#pragma unroll
        for (int k0 = 0; k0 < KS; k0 += GRP) {
          bf16x8 of[GRP];
#pragma unroll
          for (int q = 0; q < GRP; ++q) of[q] = *reinterpret_cast<const bf16x8*>(op + (k0 + q) * 16);
#pragma unroll
          for (int q = 0; q < GRP; ++q) t[k0 + q] = dot8_bf16(dof[k0 + q], of[q]);
        }
        negd = -xor32_sum(butterfly_sum(t));
      } else {
        negd = -p.dvec[(int64_t)head * p.total + grow];
      }
      // consumed (and therefore waited for) here: no compiler-placed vector-memory wait inside the main loop
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : : "v"(qf[ks]), "v"(dof[ks]));
      asm volatile("" : : "v"(lse2), "v"(negd));
    }
    // 16-byte row operand of k-step ks: row l32, chunk 2 ks + hi
    int roff[NRO];
#pragma unroll
    for (int j = 0; j < NRO; ++j) roff[j] = tile_off<D>(l32, 2 * j + hi);
    unsigned char* xw = smem + XCH_OFF + wave * 2048 + lane * 16;

    const bool never_plain = LOCAL || !wave_valid;
    const int ctx_masked = (P % BN) ? b.n_ctx - 1 : -1;   // the partial last prompt tile
    const int dec_masked = min(row0 + 1, R) / BN;         // response tiles from the diagonal (or the sequence end) on

    __syncthreads();   // tile 0 is in LDS
    for (int it = 0; it < n_tiles; ++it) {
      const unsigned char* kh = smem + (it & (NSTAGE - 1)) * STAGE_BYTES;
      const unsigned char* vh = kh + TILE_BYTES;
      const bool is_ctx = it < n_ctx_run;
      const int kt = is_ctx ? b.c0 + it : b.d0 + it - n_ctx_run;
      const int key0 = kt * BN;
      // most tiles are entirely visible to the 32 rows of this wave: no tests for them
      const bool plain = !never_plain && (is_ctx ? kt != ctx_masked : kt < dec_masked);
      const bool active = plain || (wave_valid && tile_active<LOCAL, 32>(is_ctx, key0, row0, row0 + 31, P, W) &&
                                    key0 < (is_ctx ? P : R));
      unsigned char* xo = xw + (it & 1) * XCH_BYTES;
      if (__builtin_expect(active, 1)) {
        // operands in groups of four, the next group requested before the MFMAs of the current one
        constexpr int GRP = 4, NG = 2 * KS / GRP;
        bf16x8 op[2][GRP];
        auto request = [&](int gi, bf16x8* out) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < GRP; ++q) {
            const int ks = (gi * GRP + q) % KS;
            const unsigned char* base = gi * GRP < KS ? kh : vh;
            out[q] = *reinterpret_cast<const bf16x8*>(base + roff[ks % NRO] + ks / NRO * (NRO * 32));
          }
        };
        request(0, op[0]);
        f32x16 s, dpt;
        float ev[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          s[r] = 0.f;
          dpt[r] = negd;
        }
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
          if (gi + 1 < NG) request(gi + 1, op[(gi + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = 0; q < GRP; ++q) {
            const int i = gi * GRP + q;
            if (i < KS) {
              // S^T = K Q^T, complete before the dP chain starts ...
              s = mfma32(op[gi & 1][q], qf[i], s);
            } else {
              // ... so that its exponentials issue in the shadow of the dP^T - D = V dO^T - D MFMAs
              const int ks = i - KS;
              dpt = mfma32(op[gi & 1][q], dof[ks], dpt);
#pragma unroll
              for (int j = 0; j < (16 + KS - 1) / KS; ++j) {
                const int e = 16 * ks / KS + j;   // the sixteen exponentials spread evenly over the KS MFMAs
                if (e >= 16 * (ks + 1) / KS) continue;
                ev[e] = __builtin_amdgcn_exp2f(s[e] * c - lse2);
                asm volatile("" : "+v"(ev[e]));
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        const bool need = !plain && tile_needs_mask<LOCAL, 32>(is_ctx, key0, row0, P, R, W);
        if (__builtin_expect(need, 0)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = key0 + crow(r, hi);
            if (!visible<LOCAL>(is_ctx, key, row, P, R, W)) ev[r] = 0.f;
          }
        }
        float dsv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) dsv[r] = ev[r] * dpt[r];   // dS^T
        *reinterpret_cast<bf16x8*>(xo) = pack8_bf16(dsv);
        *reinterpret_cast<bf16x8*>(xo + 1024) = pack8_bf16(dsv + 8);
      } else {
        // nothing visible: the consumers do not branch, they add a product with dS = 0
        const u32x4 z = {0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(xo) = z;
        *reinterpret_cast<u32x4*>(xo + 1024) = z;
      }
      __syncthreads();
    }
    if (STATS && p.make_stats() && hi == 0 && row < R) {
      const int64_t at = (int64_t)head * p.total + b.row_begin + row;
      p.dvec[at] = -negd;
      p.lse2[at] = lse2;
    }
    __syncthreads();   // the consumers' last interval
  } else {
    // ================================= consumer ==============================================
    const int jb = wave - 4;
    const u16* kc_base = p.kc.ptr + (int64_t)b.ctx_off * p.kc.ts + (int64_t)b.hk * p.kc.hs;
    const u16* vc_base = p.vc.ptr + (int64_t)b.ctx_off * p.vc.ts + (int64_t)b.hk * p.vc.hs;
    const u16* kd_base = p.kd.ptr + (int64_t)b.row_begin * p.kd.ts + (int64_t)b.hk * p.kd.hs;
    const u16* vd_base = p.vd.ptr + (int64_t)b.row_begin * p.vd.ts + (int64_t)b.hk * p.vd.hs;
    // global -> LDS tile loads: instruction i = jb + 4 t of a tile covers RPI key rows; lane l lands at LDS chunk
    // position l % CPR of row l / CPR of the instruction and fetches the chunk the swizzle stores there.  The
    // swizzle has a period of 16 rows and the instructions of a wave are 8 rows apart: odd t flip bit 1 of the
    // chunk index.  Keys past the end of the region re-read the last key: their scores are masked like any
    // invisible key.
    const uint32_t smem_addr = (uint32_t)reinterpret_cast<uintptr_t>(smem);
    const int ld_row0 = jb * RPI + lane / CPR;
    const int ld_coff = ((lane % CPR) ^ swz<D>(ld_row0)) * 16;
    // (loader: its twelve instructions per tensor are consecutive; t and t + 3 are 8 rows apart)
    int sp_row[3], sp_coff[3];
    if constexpr (LOADER) {
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        sp_row[t] = split_row<D>(t, lane);
        sp_coff[t] = (split_pos<D>(t, lane) ^ swz<D>(sp_row[t])) * 16;
      }
    }
    const int ktsb_c = (int)p.kc.ts * 2, ktsb_d = (int)p.kd.ts * 2, vtsb_c = (int)p.vc.ts * 2, vtsb_d = (int)p.vd.ts * 2;
    auto issue_loads = [&](int it) __attribute__((always_inline)) {
      const bool is_ctx = it < n_ctx_run;
      const int key0 = is_ctx ? (b.c0 + it) * BN : (b.d0 + it - n_ctx_run) * BN;
      const int ktsb = is_ctx ? ktsb_c : ktsb_d, vtsb = is_ctx ? vtsb_c : vtsb_d;
      const u16* kb = uniform_ptr(reinterpret_cast<const u16*>(
          reinterpret_cast<const unsigned char*>(is_ctx ? kc_base : kd_base) + (int64_t)key0 * ktsb));
      const u16* vb = uniform_ptr(reinterpret_cast<const u16*>(
          reinterpret_cast<const unsigned char*>(is_ctx ? vc_base : vd_base) + (int64_t)key0 * vtsb));
      const int last = (is_ctx ? P : R) - key0 - 1;
      const uint32_t stage_addr = smem_addr + (it & (NSTAGE - 1)) * STAGE_BYTES;
      if constexpr (LOADER) {
        static_for<IPT>([&](auto Tc) __attribute__((always_inline)) {
          constexpr int t = decltype(Tc)::value;
          const unsigned row = (unsigned)min(sp_row[t % 3] + t / 3 * kSplitRows<D>, last);
          const uint32_t coff = (uint32_t)(sp_coff[t % 3] ^ ((t / 3 & 1) * 32));
          dma16_at<t * 1024>(kb, __umul24(row, (unsigned)ktsb) + coff, stage_addr);
          dma16_at<TILE_BYTES + t * 1024>(vb, __umul24(row, (unsigned)vtsb) + coff, stage_addr);
        });
        return;
      }
      const uint32_t dst = stage_addr + jb * 1024;
#pragma unroll
      for (int t = 0; t < IPT; ++t) {
        const unsigned row = (unsigned)min(ld_row0 + t * 4 * RPI, last);
        const uint32_t coff = (uint32_t)(ld_coff ^ ((t & 1) * 32));
        dma16(kb, __umul24(row, (unsigned)ktsb) + coff, dst + t * 4096);
        dma16(vb, __umul24(row, (unsigned)vtsb) + coff, dst + TILE_BYTES + t * 4096);
      }
    };
    // tile it+1 must have landed before the barrier; tiles it+2 and it+3 may stay in flight
    auto wait_loads = [&](int it) __attribute__((always_inline)) {
      if (it + 3 < n_tiles) wait_vm<4 * IPT>();
      else if (it + 2 < n_tiles) wait_vm<2 * IPT>();
      else wait_vm<0>();
    };
    if (!LOADER || jb == 3) {
#pragma unroll 1
      for (int it = 0; it < min(n_tiles, 3); ++it) issue_loads(it);
      wait_loads(-1);   // tile 0
    }
    if (LOADER && jb == 3) {
      // The loader: every request of the workgroup, in intervals of their own (LDS stages as below).
      __syncthreads();   // tile 0 is in LDS
      for (int it = 0; it <= n_tiles; ++it) {
        if (it + 3 < n_tiles) issue_loads(it + 3);
        wait_loads(it);
        __syncthreads();
      }
    } else {
    f32x16 dq[NSUB][2];
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[s][e][r] = 0.f;
    // transpose reads: rows 4 hi + (lane % 16) / 4 and + 8 of a 16-key group, head-dim blocks jb and jb + EBLK (at head
    // dim 256 the second lies 256 bytes further: bit 4 of the chunk index)
    int toff0[2], toff1[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      toff0[e] = LOADER ? tr_off<D>(lane, hi * 4, (jb + e * EBLK) * 32) : tr_off<D>(lane, hi * 4, jb * 32) + e * 256;
      toff1[e] = LOADER ? tr_off<D>(lane, hi * 4 + 8, (jb + e * EBLK) * 32) : tr_off<D>(lane, hi * 4 + 8, jb * 32) + e * 256;
    }
    const unsigned char* xr = smem + XCH_OFF + lane * 16;
    bf16x8 kt[2][2];   // [16-key group][head-dim block]: K^T operands of the tile accumulated next interval

    __syncthreads();   // tile 0 is in LDS
    for (int it = 0; it <= n_tiles; ++it) {
      // tile it+3 goes into the stage of tile it-1: the producers read it during the last interval, and its
      // K^T operands are in this wave's registers since then
      if (!LOADER && it + 3 < n_tiles) issue_loads(it + 3);
      if (it > 0) {
        const unsigned char* xi = xr + ((it - 1) & 1) * XCH_BYTES;
        bf16x8 ds[2][NSUB];
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int s = 0; s < NSUB; ++s) ds[t2][s] = *reinterpret_cast<const bf16x8*>(xi + s * 2048 + t2 * 1024);
        __builtin_amdgcn_sched_barrier(0);
        // dQ^T += K^T dS^T
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int s = 0; s < NSUB; ++s) dq[s][e] = mfma32(kt[t2][e], ds[t2][s], dq[s][e]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (it < n_tiles) {
        const unsigned char* kh = smem + (it & (NSTAGE - 1)) * STAGE_BYTES;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int e = 0; e < 2; ++e)
            kt[t2][e] = tr_pair(kh + t2 * 16 * RB + toff0[e], kh + t2 * 16 * RB + toff1[e]);
      }
      if (!LOADER) wait_loads(it);
      __syncthreads();
    }

    // ---- epilogue: lane owns a query row, register r the head-dim column crow(r) of a block.  Stored from here a
    // row would leave in 16-byte pieces, 32 rows per instruction; the scaled tile goes through LDS instead (the stages
    // are free now) and leaves as whole 512-byte rows, written by all eight waves.
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      unsigned char* orow = smem + (s * 32 + l32) * OUT_RS;
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          u32x2 w;
          w.x = pack2_bf16(dq[s][e][r4 * 4 + 0] * p.scale, dq[s][e][r4 * 4 + 1] * p.scale);
          w.y = pack2_bf16(dq[s][e][r4 * 4 + 2] * p.scale, dq[s][e][r4 * 4 + 3] * p.scale);
          *reinterpret_cast<u32x2*>(orow + ((jb + EBLK * e) * 32 + r4 * 8 + hi * 4) * 2) = w;
        }
    }
    }
  }
  __syncthreads();   // the scaled tile is in LDS
  {
    // 16-byte piece n % CPR of tile row n / CPR, n = thread, + 512, ...
#pragma unroll
    for (int i = 0; i < NSUB * 32 * CPR / 512; ++i) {
      const unsigned n = (unsigned)(i * 512 + tid);
      const int tr = n / CPR, piece = n % CPR, s = tr >> 5;
      const int head = b.hk * p.G + b.hc * p.GP + s / p.RSH;
      const int row = b.blk_row0 + (s % p.RSH) * 32 + (tr & 31);
      if (row >= R) continue;
      const u32x4 w = *reinterpret_cast<const u32x4*>(smem + tr * OUT_RS + piece * 16);
      u16* op = p.dq.ptr + (int64_t)(b.row_begin + row) * p.dq.ts + (int64_t)head * p.dq.hs;
      *reinterpret_cast<u32x4*>(op + piece * 8) = w;
    }
  }
