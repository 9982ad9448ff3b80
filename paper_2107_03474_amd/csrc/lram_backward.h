// lram_backward.h -- part of liblram (included by lram.hip only).
//
// Backward: the value-gradient atomic scatter, the query gradient (and the
// activation layer's chain), and the backward kernel of the atomic and sorted
// scatters.

#pragma once

namespace {

// The merged scatter pays off when lookups share their closest lattice point
// (their neighbour lists then overlap): it is chosen when at least a tenth of
// the lookups share theirs with another lookup of the batch.
__device__ __forceinline__ bool merge_chosen(uint32_t shared, int64_t L) { return 10 * (int64_t)shared >= L; }

// Backward, fused with the query gradient: per lookup, read the 32 rows once
// for <G, v_j> and form dq from the coordinate errors.

// Value-gradient scatter of one lookup: M consecutive lanes own one gradient
// row, so each atomic instruction covers 64/M whole rows.
template <int M, int KS, int NBUF, int WBUF>
__device__ __forceinline__ void scatter_atomic(const WaveLds<KS, NBUF, WBUF>& W, int buf, int count,
                                               const float* __restrict__ gout, int64_t l, float* __restrict__ gtab,
                                               int lane) {
  constexpr int RA = WAVE / M;
  const int col = lane % M;
  const float gc = gout[(size_t)l * M + col];
  const int kend = KS == NB ? NB / RA : (min(count, KS) + RA - 1) / RA;
#pragma unroll 4
  for (int k = 0; k < kend; ++k) {
    const int j = k * RA + lane / M;
    const int32_t s = W.nbr[buf][j].slot;
    if (s >= 0) unsafeAtomicAdd(gtab + (size_t)s * M + col, W.wgt[buf][j] * gc);
  }
}

// dq_i = sum_j -2 u_j^3 (x_i - k_{j,i}) <G, v_j> of one lookup (zero without
// neighbours), written to gq[l][8].
// TH (activation layer): also dL/ds = sum_j w_j <G, v_j> = <G, phi>, and the
// chain through q_i = c_i arg z_i and s = (sum 1/|z_i|)^-1 (Sec. 2.3), with
// dL/dq = s dq:
//   dL/da_i = dL/ds s^2 a_i / r_i^3 - dL/dq_i c_i b_i / r_i^2,
//   dL/db_i = dL/ds s^2 b_i / r_i^3 + dL/dq_i c_i a_i / r_i^2,
// written to gq[l][16] (zero where s = 0) by theta_chain for a whole tile:
// grad_query leaves dq and dL/ds of tile position t in LDS.
//
// <G, v_j> and the sums over j are formed in fp64 (fp32 x fp32 products are
// exact there).  Next to a lattice point one term carries all of dq (and
// behind the activation layer dL/ds is sum_j w_j <G, v_j>), so a cancelling
// fp32 dot product would become the relative error of the whole gradient.
//
// What bounds it is VALU issue: with up to 16 lanes to a row, every row's dot
// product crossed four fp64 shuffle steps and every lane repeated its row's
// coefficient (about 330 VALU instructions per lookup at m = 64 fp32).  Four
// lanes to a row instead (each reads its 16 bytes of every 64): the two
// passes' dot products are reduced together by one exchange of halves and
// one sum, after which two lanes hold each row's coefficient and take four
// coordinates each; the sum over the 32 rows halves the number of coordinates
// per lane at its first two steps.  Measured at 262,144 lookups (m = 64 fp32,
// 2^20 rows): merged backward behind the activation layer 1,606 -> 1,368 us;
// untruncated backward of 29,997 lookups (m = 32 fp32) 322 -> 247 us; 4,096
// lookups at K = 4 21.3 -> 19.6 us.
template <int DT, int M, int TH, int KS, int NBUF, int WBUF>
__device__ __forceinline__ void grad_query(Frame& F, WaveLds<KS, NBUF, WBUF>& W, int buf, const Tables& T, int t,
                                           int count, const char* __restrict__ tb, const float* __restrict__ gout, int64_t l,
                                           int lane, float* gq) {
  constexpr int R = chunk_rows<KS>();  // rows per chunk of the row loop
  using G = RowGeom<DT, M, R>;
  constexpr int LE = G::LPR / G::NP;   // lanes that share a row's dot product in the end (2, or 4 for chunks of 16)
  constexpr int IC = 8 / LE;           // query coordinates per lane
  const int rsub = lane / G::LPR, ch = lane % G::LPR;
  const int e = lane % LE;
  const int pass = ch / LE;            // the pass whose row this lane ends up with
  double dq[IC];
  double dls = 0.0;  // dL/ds (TH)
#pragma unroll
  for (int k = 0; k < IC; ++k) dq[k] = 0.0;
  if (count > 0) {
    double g[G::NC * G::EPC];
#pragma unroll
    for (int c = 0; c < G::NC; ++c) {
      const float* gp = gout + (size_t)l * M + (c * G::LPR + ch) * G::EPC;
#pragma unroll
      for (int k = 0; k < G::EPC; k += 4) {
        const float4 gv = *reinterpret_cast<const float4*>(gp + k);
        g[c * G::EPC + k] = gv.x; g[c * G::EPC + k + 1] = gv.y;
        g[c * G::EPC + k + 2] = gv.z; g[c * G::EPC + k + 3] = gv.w;
      }
    }
    // selectors of the query coordinates e*IC .. this lane accumulates
    uint32_t lsel[IC];
#pragma unroll
    for (int k = 0; k < IC; ++k) lsel[k] = F.sel[e * IC + k];
    for (int r0 = 0; r0 < (KS == NB ? 1 : count); r0 += R) {
      // rows of padding entries read row 0; their coefficient is zeroed below
      uint4 v[G::NP][G::NC];
#pragma unroll
      for (int p = 0; p < G::NP; ++p) {
        const int32_t s = max(W.nbr[buf][r0 + p * G::RPP + rsub].slot, 0);
        const char* src = tb + (size_t)s * G::RB + ch * 16;
#pragma unroll
        for (int c = 0; c < G::NC; ++c) v[p][c] = *reinterpret_cast<const uint4*>(src + c * (G::LPR * 16));
      }
      double pd[G::NP];
#pragma unroll
      for (int p = 0; p < G::NP; ++p) {
        pd[p] = 0.0;
#pragma unroll
        for (int c = 0; c < G::NC; ++c) {
          float f[G::EPC];
          unpack16<DT, G::EPC>(v[p][c], f);
#pragma unroll
          for (int k = 0; k < G::EPC; ++k) pd[p] = fma(g[c * G::EPC + k], (double)f[k], pd[p]);
        }
      }
      // over the row's four lanes: two passes exchange halves (lane bit 1),
      // then one sum (bit 0); a single pass is summed over both bits
      double dot;
      if constexpr (G::NP == 2) {
        const bool up = (ch & 2) != 0;
        dot = up ? pd[1] : pd[0];
        dot += dpp_f64<DPP_XOR2>(up ? pd[0] : pd[1]);
      } else {
        static_assert(G::NP == 1, "one or two passes");
        dot = pd[0] + dpp_f64<DPP_XOR2>(pd[0]);
      }
      dot += dpp_f64<DPP_XOR1>(dot);
      const Nbr n = W.nbr[buf][r0 + pass * G::RPP + rsub];
      const bool real = n.slot >= 0;
      const float u = 1.0f - __uint_as_float(n.dbits) * 0.125f;
      const double a = real ? -2.0 * (double)(u * u * u) * dot : 0.0;
      if constexpr (TH) {
        const float u2 = u * u;
        dls += real ? (double)(u2 * u2) * dot : 0.0;
      }
#pragma unroll
      for (int k = 0; k < IC; ++k) {
        const uint32_t ab = __builtin_amdgcn_perm(n.hi, n.lo, lsel[k]);
        // (padding entries carry no candidate: an entry of the wave's own tables, built
        // where count > 0 and so finite, times zero)
        dq[k] = fma(a, (double)lds_f32(T.et, ab + 256u * (e * IC + k)), dq[k]);
      }
    }  // chunks of R rows
  }
  // over the rows (lane bits 5 .. log2(LE)); bits 5 and 4 halve the
  // coordinates per lane as long as there are two
  int i = e * IC;
#pragma unroll
  for (int k = 0; k < IC / 2; ++k) dq[k] = add_halves_f64<32>(dq[k], dq[k + IC / 2]);
  i += (lane & 32) ? IC / 2 : 0;
  if constexpr (IC == 4) {
    dq[0] = add_halves_f64<16>(dq[0], dq[1]);
    i += (lane & 16) ? 1 : 0;
  } else {
    dq[0] = add_halves_f64<16>(dq[0], dq[0]);
  }
  dq[0] = sum_row_f64<LE>(dq[0]);
  if constexpr (TH) {
    dls = add_halves_f64<32>(dls, dls);
    dls = add_halves_f64<16>(dls, dls);
    dls = sum_row_f64<LE>(dls);
  }
  // one lane per coordinate writes it
  if ((lane & (IC == 4 ? 14 : 28)) == 0) {
    if constexpr (TH == IN_QUERY)
      gq[l * 8 + i] = (float)dq[0];
    else
      W.dq[t][i] = dq[0];
  }
  if constexpr (TH != IN_QUERY)
    if (lane == 0) *reinterpret_cast<double*>(&F.r2) = dls;
}

// The activation layer's chain for the nt lookups of a tile, one coordinate to
// a lane: its fp64 divisions and square roots run for eight lookups at once
// rather than lookup by lookup on eight of 64 lanes (262,144 lookups, m = 64 fp32:
// the backward's search and gradient 443 -> 400 us).  lookup: the lookup at a
// tile position, negative where nothing is written.
template <typename WL, typename Lookup>
__device__ __forceinline__ void theta_chain(const Frame* FR, const WL& W, int nt, int lane, Lookup lookup, float* gq,
                                            const float* __restrict__ z, const Params& P) {
  const int i = lane & 7;
  double ci = P.cK[0];
#pragma unroll
  for (int k = 1; k < 8; ++k) ci = i == k ? P.cK[k] : ci;
  wave_lds_sync();
#pragma unroll 1
  for (int t = lane >> 3; t < TILE; t += 8) {
    const int64_t l = lookup(t);
    if (t < nt && l >= 0) {
      const double sc = FR[t].s, dls = *reinterpret_cast<const double*>(&FR[t].r2);
      double ga = 0.0, gb = 0.0;
      if (sc > 0.0) {
        const float2 ab = *reinterpret_cast<const float2*>(z + l * 16 + 2 * i);
        const double a = ab.x, b = ab.y;
        const double r2 = a * a + b * b;
        const double ir2 = 1.0 / r2, ir3 = ir2 / sqrt(r2);  // 1/r^2, 1/r^3
        const double ds = dls * sc * sc, dqs = W.dq[t][i] * sc * ci;
        ga = ds * a * ir3 - dqs * b * ir2;
        gb = ds * b * ir3 + dqs * a * ir2;
      }
      *reinterpret_cast<float2*>(gq + l * 16 + 2 * i) = make_float2((float)ga, (float)gb);
    }
  }
  wave_lds_sync();
}

// Waves per SIMD of the backward that emits pairs.  Rows of 64 columns spill three
// registers at four (bf16, a whole backward by sorted runs, 2^18 rows, four / three: 262,144
// lookups 722 / 711 us, 524,288 1,440 / 1,407); rows of 32 are as fast or faster at four
// (540 / 549, 1,059 / 1,085; three spilled), and so are those behind the staged activation
// layer, nine spilled registers included (m = 64 bf16 760 / 778, 1,476 / 1,521).
template <int DT, int M, int TH>
constexpr int pair_waves() { return TH == IN_QUERY && M == 64 ? 3 : kernel_waves<DT, M, TH>(); }

// The value gradient is either added straight into grad_table with fp32
// atomics (EMIT = false), or emitted as (location, (lookup, w_j)) pairs for
// the location sort (EMIT = true; padding gets the key N, which sorts last),
// whose digits are counted here into ghist (the counts hide behind the row
// loads; a kernel of their own took 37 us for 8.4 M pairs).
// gate (nullable): the merged scatter's device-side choice -- this kernel does
// nothing when the batch is merged instead (see merge_chosen).
// TH: the lookups' input; z the activation layer's own input, for its chain.
// IN_STAGED: q is grad_in itself, lookup l's record at the start of its row,
// read by the wave that writes the row afterwards.
// ORD: visit the lookups in the order perm (as k_forward).
// SAVED: the forward's lists (NbrList saved) replace the search.
template <int DT, int M, bool EMIT, int TH, int KS = NB, bool ORD = false, bool SAVED = false>
__global__ void __launch_bounds__(THREADS, (EMIT ? pair_waves<DT, M, TH>() : kernel_waves<DT, M, TH>())) k_backward(const float* q, const float* __restrict__ z, Params P,
                                                      const void* __restrict__ table,
                                                      const float* __restrict__ gout, float* __restrict__ gtab,
                                                      float* gq, uint32_t* __restrict__ pair_key,
                                                      uint2* __restrict__ pair_val, const uint32_t* __restrict__ gate,
                                                      const uint32_t* __restrict__ perm, NbrList saved,
                                                      uint32_t* __restrict__ ghist) {
  static_assert(!EMIT || KS == NB, "the sorted scatter takes lists of 32");
  static_assert(!(SAVED || ORD) || (KS == NB && !TH), "orders and saved lists serve the k = 32 lookup");
  __shared__ ListLds<KS, SAVED> S;
  __shared__ uint32_t digits[EMIT ? SORT_PASSES_MAX : 1][EMIT ? RADIX : 1];
  if (gate && merge_chosen(*gate, P.L)) return;
  if constexpr (EMIT) {
#pragma unroll
    for (int p = 0; p < SORT_PASSES_MAX; ++p) digits[p][threadIdx.x] = 0u;
  }
  WaveCtx c;
  wave_ctx(P, c, ORD);
  const int lane = c.lane;
  const char* tb = reinterpret_cast<const char*>(table);
  auto& W = S.wave[c.wave];
  // Lists of 16 leave the row atomics less to overlap with: the query gradient's
  // row loads come back behind the lookup's own atomics when those go first, unless
  // the wave has one or two lookups, whose last atomics would only end later.
  // 2^24 rows, uniform, m = 32 bf16, atomics first / last: 32,768 lookups 68 / 60 us, 262,144 519 / 449;
  // 2,048 8.8 / 9.5.  Lists of 32 overlap better with the atomics first (4,096 lookups 20.9 / 22.6),
  // longer ones alike.
  const bool late = KS < NB && P.lpw >= 4;
  // scatter and query gradient of list buf, which is lookup l's (ok: inside the batch)
  auto finish = [&](Frame& F, int buf, int t, int count, int64_t l, bool ok) {
    if (!EMIT && gtab && count > 0 && !late) scatter_atomic<M, KS>(W, buf, count, gout, l, gtab, lane);
    if (gq && ok) grad_query<DT, M, TH, KS>(F, W, buf, S.tab, t, count, tb, gout, l, lane, gq);
    if (!EMIT && gtab && count > 0 && late) scatter_atomic<M, KS>(W, buf, count, gout, l, gtab, lane);
    if (EMIT && gtab && lane < NB && ok) {
      const int32_t s = W.nbr[buf][lane].slot;
      const uint32_t key = s >= 0 ? (uint32_t)s : P.N;
      pair_key[l * NB + lane] = key;
#pragma unroll
      for (int p = 0; p < SORT_PASSES_MAX; ++p)
        if (p < P.passes) atomicAdd(&digits[p][(key >> (p * RADIX_BITS)) & (RADIX - 1)], 1u);
      pair_val[l * NB + lane] = make_uint2((uint32_t)l, __float_as_uint(W.wgt[buf][lane]));
    }
  };
  if constexpr (KS == NB) {
    TileInput<TH, ORD> in(q, perm, c.base, c.nl, P, lane);
    TileSearch<TH, SAVED ? 1 : 2, !SAVED> ts(P, S, c.wave, lane);
    if constexpr (EMIT && SAVED) __syncthreads();  // (the digits' counters; a search's own barrier otherwise)
    for (int t0 = 0; t0 < c.nl; t0 += TILE) {
      const int nt = min(TILE, c.nl - t0);
      ts.frames(in.v, in.have, nt);
      in.advance(t0, P);
      if constexpr (SAVED) {
        for (int t = 0; t < nt; ++t) {
          bool ok;
          const int64_t l = in.lookup(t0, t, P, ok);
          const int count = ts.one.load(ts.FR[t], read_sel(ts.FR[t]), 0, saved, l, P.N);
          finish(ts.FR[t], 0, t, count, l, ok);
          wave_lds_sync();
        }
      } else {
        for (int p = 0; 2 * p < nt; ++p) {
          ts.pair(p, 0);
          bool ok;
          const int64_t l0 = in.lookup(t0, 2 * p, P, ok);
          finish(ts.FR[2 * p], 0, 2 * p, ts.count0, l0, ok);
          const int64_t l1 = in.lookup(t0, 2 * p + 1, P, ok);
          if (2 * p + 1 < nt) finish(ts.FR[2 * p + 1], 1, 2 * p + 1, ts.count1, l1, ok);
          wave_lds_sync();
        }
      }
      if constexpr (TH != IN_QUERY)
        if (gq) theta_chain(ts.FR, W, nt, lane, [&](int t) { return c.base + t0 + t; }, gq, z, P);
    }
    if constexpr (EMIT) {
      __syncthreads();
      uint32_t* g = ghist + (blockIdx.x % SORT_HIST_COPIES) * (SORT_PASSES_MAX * RADIX);
      for (int p = 0; p < P.passes; ++p) {
        const uint32_t n = digits[p][threadIdx.x];
        if (gtab && n) atomicAdd(&g[p * RADIX + threadIdx.x], n);
      }
    }
  } else {
    static_assert(KS == NB || (!TH && !ORD && !SAVED && !EMIT), "other lists serve the plain lookup");
    Search<KS> srch(P, S.tab, W, S.tile, c.wave, lane);
    const QuadCtx<IN_QUERY> Q(P, lane);
    Frame* FR = S.frames[c.wave];
    for (int t0 = 0; t0 < c.nl; t0 += TILE) {
      const int nt = min(TILE, c.nl - t0);
      tile_frames(q, c.base + t0, nt, P, FR, Q, lane);
      for (int t = 0; t < nt; ++t) {
        const int count = srch.run(FR[t], read_sel(FR[t]), 0);
        finish(FR[t], 0, t, count, c.base + t0 + t, true);
        wave_lds_sync();
      }
    }
  }
}

}  // namespace
