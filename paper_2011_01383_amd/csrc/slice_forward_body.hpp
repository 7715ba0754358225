// The body of slice_forward_kernel and of slice_forward, included by forward.hip in
// both.  In scope: CELL, H, J, kCached, kWeightsFromMemory and kFused; the arguments
// a, the node groups Q and the LDS arrays W_s, C_s, Z_s, bias_s, chunk and cache.
  using D = Dims<CELL, H, J>;
  constexpr int GJ = D::GJ, MPAD = D::MPAD, NT = D::NT, LDW = D::LDW, KW = D::KW, NB = D::NB, KA = D::KA;
  constexpr bool kLeafInputs = CELL == CORTEX_TREE_RNN || CELL == CORTEX_NARY_TREELSTM;
  constexpr bool kLstm = CELL == CORTEX_NARY_TREELSTM;
  constexpr int EPI = kTileM * J;          // (row, unit) pairs of a tile
  // Gate rows beyond the last full 16-row MFMA tile: when only four remain
  // (N-ary TreeLSTM, J = 4: the u gate), an MFMA tile would be three-quarters
  // padding, so they are contracted on the vector ALU, from the same operand
  // registers, while the matrix cores run the full tiles.
  constexpr bool kVecTail = GJ % 16 == 4 && NT >= 2;
  constexpr int NTM = kVecTail ? NT - 1 : NT;    // MFMA tiles of gate rows
  constexpr int SEGS = SrcCfg<CELL>::SEGS;
  // A block's 16 columns never straddle two operand segments (H is a
  // multiple of 16), so the segment of block b is the same for the whole
  // wave; a wave's range touches at most two segments (KW <= H).
  static_assert(KA == SEGS * H && KA <= kFwdWaves * KW && KW <= H && H % 16 == 0, "block layout");

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g4 = lane >> 4;
  // node group q's slices are workgroups q, q + Q, q + 2Q, ..., which
  // round-robin dispatch puts on the XCDs congruent to q modulo gcd(Q, 8)
  // (two XCDs for Q = 4) instead of spreading a group over all eight
  const int slice = blockIdx.x / Q, group = blockIdx.x % Q;
  const int hbase = slice * J;
  const int N = a.N;
  const uint32_t tag = launch_tag(a.sync);     // read with the status: one round trip
  const TagBuf hs(a.hs, (uint32_t)N * H * 8);
  const TagBuf cs(a.cs, kLstm ? (uint32_t)N * H * 8 : 0u);
  // plain operand rows: the input table (leaf children) or the DAG inputs
  const InBuf xin(CELL == CELL_DAG ? (const void *)a.x : (const void *)a.x_table,
                  CELL == CELL_DAG ? (a.x ? (uint32_t)N * H * 4 : 0u)
                                   : (kLeafInputs && a.x_table ? (uint32_t)a.x_rows * H * 4 : 0u));
  // this wave's columns: segment sgA from column o0 within it, crossing into
  // segment sgA + 1 at block cross_b (NB when it does not)
  const int kw = wave * KW;
  const int sgA = kw / H, o0 = kw % H;
  const int cross_b = (H - o0) / 16 < NB ? (H - o0) / 16 : NB;

  CORTEX_TRACE_KERNEL(0);
  // the status, the weight slice and the cached linearization are requested
  // together: one memory round trip for all of them
  const int status0 = load_status(a.status);
  int L;
  const int *off, *codes, *xrow;
  if constexpr (kFused) {
    // the weight loads share their round trip with the children and input
    // rows the linearizer requests
    static_assert(kCached && !kWeightsFromMemory, "fused launches cache the structure");
    WeightRegs<CELL, H, J> wr;
    issue_weight_slice<CELL, H, J>(a, hbase, wr);
    const bool ok = fused_setup<CELL>(a, cache, L, off, codes, xrow);
    commit_weight_slice<CELL, H, J>(wr, W_s, bias_s);
    if (!ok || status0 != 0) return;
    __syncthreads();                  // the weight slice is in LDS before any tile reads it
    CORTEX_TRACE_KERNEL(1);
  } else {
    SrcRegs pf;
    {
      WeightRegs<CELL, H, J> wr;
      issue_weight_slice<CELL, H, J>(a, hbase, wr);
      prefetch_sources<CELL, kCached>(a, pf);
      commit_weight_slice<CELL, H, J>(wr, W_s, bias_s);
    }
    if (status0 != 0) return;
    CORTEX_TRACE_KERNEL(1);
    if (!setup_sources<CELL, kCached>(a, pf, cache, L, off, codes, xrow)) return;
  }
  CORTEX_TRACE_KERNEL(2);
  if (!mark_entered(a.sync, tag, a.status)) return;
  const int off1 = off[1];
  int gave_up = 0;

  for (int l = a.level_lo; l < L && l < a.level_hi; ++l) {
    CORTEX_TRACE_POINT(l, 0);
    const int r0 = off[l], r1 = off[l + 1];
    if (!kCached && (r1 < r0 || r1 > N || (l == 0 && r0 != 0))) {
      raise_status(a.status, CORTEX_ST_BAD_LINEARIZATION);
      return;
    }
    if (kLeafInputs && l == 0) {
      write_leaf_outputs<H, kLstm>(a, kCached ? xrow : nullptr, r1, hs, cs, tag);
      continue;
    }
    const int ntile = (r1 - r0 + kTileM - 1) / kTileM;
    int u0 = ((group - l) % Q + Q) % Q;            // first tile of the current chunk

    // source code of tile u, row i, segment sg (cached, or the staged chunk)
    auto code_of = [&](int u, int i, int sg) __attribute__((always_inline)) -> int {
      if (kCached) return codes[(r0 + u * kTileM + i) * SEGS + sg];
      return chunk.code[(u - u0) / Q][i][sg];
    };
    auto code_b = [&](const int (&cd)[2], int b) __attribute__((always_inline)) -> int {
      return b >= cross_b ? cd[1] : cd[0];
    };
    auto col_b = [&](int b) __attribute__((always_inline)) -> int {   // this lane's first column in block b
      return (b >= cross_b ? o0 + 16 * b - H : o0 + 16 * b) + 4 * g4;
    };

    // Operands of tile u for this lane: fragments f, the row's source codes
    // cd (this lane's segment and the next), and (N-ary) the staged memory
    // cells cc of pair tid's non-leaf children (elements ce).
    auto issue = [&](int u, Frag (&f)[NB], int (&cd)[2], u32x2 (&cc)[2], int (&ce)[2]) __attribute__((always_inline)) {
      const int row = r0 + u * kTileM + i16;
      cd[0] = cd[1] = -1;
      if (row < r1 && sgA < SEGS) {
        cd[0] = code_of(u, i16, sgA);
        if (cross_b < NB && sgA + 1 < SEGS) cd[1] = code_of(u, i16, sgA + 1);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int c = code_b(cd, b), o = col_b(b);
        if (c >= 0) {
          const uint32_t so = (uint32_t)(c * H + o) * 8u;
          f[b].lo = hs.load2_at(so);
          f[b].hi = hs.load2_at(so + 16u);
        } else {
          // both halves written on both paths: a store to a selected half
          // would force the fragments out of registers
          f[b].lo = xin.load4(c <= -2 ? (uint32_t)(((-2 - c) * H + o) * 4) : kNoSource);
          f[b].hi = u32x4{0u, 0u, 0u, 0u};
        }
      }
      if (kLstm) {
        const int prow = r0 + u * kTileM + tid / J;
        const bool live = tid < EPI && prow < r1;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int c = live ? code_of(u, tid / J, s) : -1;
          ce[s] = c >= 0 ? c * H + hbase + tid % J : -1;
          cc[s] = cs.load1_at(ce[s] >= 0 ? (uint32_t)ce[s] * 8u : kNoSource);
        }
      }
    };
    auto all_ready = [&](const Frag (&f)[NB], const int (&cd)[2], const u32x2 (&cc)[2],
                         const int (&ce)[2]) __attribute__((always_inline)) -> bool {
      bool r = true;
#pragma unroll
      for (int b = 0; b < NB; ++b) r = r && (code_b(cd, b) < 0 || f[b].ready(tag));
      if (kLstm) {
#pragma unroll
        for (int s = 0; s < 2; ++s) r = r && (ce[s] < 0 || cc[s].y == tag);
      }
      return r;
    };

    // One tile: wait for its staged operands, request the next tile's, contract,
    // apply the gates, write the states.
    auto process = [&](int u, Frag (&f)[NB], int (&cd)[2], u32x2 (&cc)[2], int (&ce)[2], bool more,
                       Frag (&fn)[NB], int (&cdn)[2], u32x2 (&ccn)[2], int (&cen)[2]) __attribute__((always_inline)) {
      CORTEX_TRACE_POINT(l, 1);
      if (!gave_up && !all_ready(f, cd, cc, ce)) {
        const uint64_t t0 = wall_clock64();
        for (;;) {
          __builtin_amdgcn_s_sleep(1);
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const int c = code_b(cd, b);
            if (c >= 0 && !f[b].ready(tag)) {
              const uint32_t so = (uint32_t)(c * H + col_b(b)) * 8u;
              f[b].lo = hs.load2_at(so);
              f[b].hi = hs.load2_at(so + 16u);
            }
          }
          if (kLstm) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
              if (ce[s] >= 0 && cc[s].y != tag) cc[s] = cs.load1_at((uint32_t)ce[s] * 8u);
          }
          const int stv = load_status(a.status);
          if (all_ready(f, cd, cc, ce)) break;
          if (stv != 0) {
            gave_up = 1;
            break;
          }
          if (wall_clock64() - t0 > a.timeout) {
            raise_status(a.status, CORTEX_ST_BARRIER_TIMEOUT);
            gave_up = 1;
            break;
          }
        }
      }
      CORTEX_TRACE_POINT(l, 2);
      if (more) issue(u + Q, fn, cdn, ccn, cen);   // in flight during this tile's contraction
      // ---- contraction: partial sums of this wave's k range ----
      floatx4 acc0[NT], acc1[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc0[nt] = acc1[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
      // vector-ALU rows: this lane's row i16 over its 4 NB columns, for the
      // four gate rows 16 NTM .. +3
      float tail[4] = {0.f, 0.f, 0.f, 0.f};
      if constexpr (!kWeightsFromMemory) {
        const float *brow = &W_s[i16 * LDW + kw + 4 * g4];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const float4 av = f[b].value(code_b(cd, b) >= 0);
#pragma unroll
          for (int nt = 0; nt < NTM; ++nt) {
            const float4 bv = *(const float4 *)(brow + nt * 16 * LDW + 16 * b);
            if (b & 1) acc1[nt] = mfma_k16(av, bv, acc1[nt]);
            else acc0[nt] = mfma_k16(av, bv, acc0[nt]);
          }
          if constexpr (kVecTail) {
            const float *trow = &W_s[16 * NTM * LDW + kw + 16 * b + 4 * g4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 w = *(const float4 *)(trow + q * LDW);
              tail[q] = fmaf(av.x, w.x, fmaf(av.y, w.y, fmaf(av.z, w.z, fmaf(av.w, w.w, tail[q]))));
            }
          }
        }
      } else {
        // ablation: no model persistence; the same weight-slice values,
        // read from the weight tensors at every tile
        float4 bw[NB][NTM];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int nt = 0; nt < NTM; ++nt) bw[b][nt] = weight_slice_at<CELL, H, J>(a, hbase, nt * 16 + i16, kw + 16 * b + 4 * g4);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const float4 av = f[b].value(code_b(cd, b) >= 0);
#pragma unroll
          for (int nt = 0; nt < NTM; ++nt) {
            if (b & 1) acc1[nt] = mfma_k16(av, bw[b][nt], acc1[nt]);
            else acc0[nt] = mfma_k16(av, bw[b][nt], acc0[nt]);
          }
          if constexpr (kVecTail) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 w = weight_slice_at<CELL, H, J>(a, hbase, 16 * NTM + q, kw + 16 * b + 4 * g4);
              tail[q] = fmaf(av.x, w.x, fmaf(av.y, w.y, fmaf(av.z, w.z, fmaf(av.w, w.w, tail[q]))));
            }
          }
        }
      }
      CORTEX_TRACE_WAVE(l);
      // The next tile's loads stay in flight through this tile's epilogue
      // (vector memory operations retire in order, so their first use
      // waits for them alone).
#pragma unroll
      for (int nt = 0; nt < NTM; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          C_s[(wave * kTileM + 4 * g4 + v) * MPAD + nt * 16 + i16] = acc0[nt][v] + acc1[nt][v];
      if constexpr (kVecTail) {
        // the four lanes of row i16 (lane groups g4) hold disjoint column sets
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          tail[q] += __shfl_xor(tail[q], 16);
          tail[q] += __shfl_xor(tail[q], 32);
        }
        if (g4 == 0)
          *(float4 *)&C_s[(wave * kTileM + i16) * MPAD + 16 * NTM] = make_float4(tail[0], tail[1], tail[2], tail[3]);
      }
      __syncthreads();
      CORTEX_TRACE_POINT(l, 3);
      // ---- gates: one thread per (row, gate row) sums the wave partials
      //      and applies the nonlinearity; TreeRNN / DAG-RNN rows are done
      //      here, N-ary TreeLSTM combines the gates below ----
      for (int p = tid; p < kTileM * GJ; p += kFwdThreads) {
        const int i = p / GJ, m = p % GJ;
        float sum = bias_s[m];
#pragma unroll
        for (int w = 0; w < kFwdWaves; ++w) sum += C_s[(w * kTileM + i) * MPAD + m];
        if constexpr (kLstm) {
          Z_s[p] = m >= 4 * J ? tanh_f(sum) : sigmoidf(sum);      // gates (i, f_l, f_r, o | u)
        } else {
          const int row = r0 + u * kTileM + i;
          if (row < r1) {
            const uint32_t el = (uint32_t)(row * H + hbase + m);
            const float hv = tanh_f(sum);
            hs.store1(el, hv, tag);
            a.h[el] = hv;
          }
        }
      }
      if constexpr (kLstm) {
        __syncthreads();
        const int row = r0 + u * kTileM + tid / J;
        if (tid < EPI && row < r1) {
          const int j = tid % J;
          const float *z = &Z_s[(tid / J) * GJ];
          const float cn = z[j] * z[4 * J + j] + z[J + j] * as_float(cc[0].x) + z[2 * J + j] * as_float(cc[1].x);
          const float hv = z[3 * J + j] * tanh_f(cn);
          const uint32_t el = (uint32_t)(row * H + hbase + j);
          cs.store1(el, cn, tag);
          hs.store1(el, hv, tag);
          a.c[el] = cn;
          a.h[el] = hv;
        }
      }
      __syncthreads();
      CORTEX_TRACE_POINT(l, 4);
    };

    // Two operand sets in turn: the next tile's loads are in flight while
    // the current tile is computed, with no register copies between tiles.
    Frag fa[NB], fb[NB];
    int cda[2], cdb[2], cea[2] = {-1, -1}, ceb[2] = {-1, -1};
    u32x2 cca[2], ccb[2];
    for (; u0 < ntile; u0 += Q * kChunkTiles) {
      const int u_last = min(ntile - 1, u0 + Q * (kChunkTiles - 1));
      if (!kCached) {
        __syncthreads();                // the previous chunk's codes are no longer read
        stage_chunk_codes<CELL>(a, chunk, u0, (u_last - u0) / Q + 1, Q, r0, r1, off1);
        __syncthreads();
      }
      issue(u0, fa, cda, cca, cea);
      CORTEX_TRACE_POINT(l, 6);
      for (int u = u0;;) {
        bool more = u + Q <= u_last;
        process(u, fa, cda, cca, cea, more, fb, cdb, ccb, ceb);
        u += Q;
        if (!more) break;
        more = u + Q <= u_last;
        process(u, fb, cdb, ccb, ceb, more, fa, cda, cca, cea);
        u += Q;
        if (!more) break;
      }
    }
    CORTEX_TRACE_POINT(l, 5);
    if (__syncthreads_or(gave_up)) return;
    if (a.level_barrier && !grid_sync<false>(SyncWords{a.sync}, a.status, a.timeout)) return;
  }
  CORTEX_TRACE_KERNEL(3);
  if (a.retire) retire_tag(a.sync, tag, a.status, a.timeout);
