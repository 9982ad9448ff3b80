// lram_lookup.h -- part of liblram (included by lram.hip only).
//
// Lookup kernels: neighbour lists, the forward gather-reduce (pipelined for k
// = 32, chunked for other k).

#pragma once

namespace {

// ---------------------------------------------------------------------------
// Kernels.

struct WaveCtx {
  int wave, lane;
  int64_t base;
  int nl;
};

// xcd: take the workgroups' ranges XCD-contiguously (for lookups visited in a
// locality order, so that neighbouring ranges share an L2).
__device__ __forceinline__ bool wave_ctx(const Params P, WaveCtx& c, bool xcd = false) {
  c.wave = (int)uniform(threadIdx.x / WAVE);  // scalar: loop bounds and LDS bases stay out of vector registers
  c.lane = threadIdx.x % WAVE;
  const int64_t blk = xcd ? xcd_block() : (int64_t)blockIdx.x;
  c.base = (blk * WAVES + c.wave) * P.lpw;
  c.nl = (int)max<int64_t>(0, min<int64_t>(P.lpw, P.L - c.base));
  return c.nl > 0;
}

// Writes one list of a lookup (entries in LDS, count real ones) ordered by
// (distance bits, location, lattice point); half: the lanes of one half wave
// (32 entries), otherwise all lanes.
template <int KS, int NBUF, int WBUF>
__device__ __forceinline__ void store_list(const WaveLds<KS, NBUF, WBUF>& W, int buf, int wb, int first, int step,
                                           int count, const Frame& F, const Sel& sel, int64_t l, int32_t* slot_out,
                                           float* w_out, float* d2_out) {
  for (int me_i = first; me_i < KS; me_i += step) {
    const Nbr me = W.nbr[buf][me_i];
    int rank = me_i;
    if (me_i < count) {
      // (distance bits, location) as one key; equal keys (the same location
      // twice, which takes a torus side of 2) are ordered by the point itself
      const uint64_t mk = (uint64_t)me.dbits << 32 | (uint32_t)me.slot;
      rank = 0;
      int same = 0;
      for (int e = 0; e < count; ++e) {
        const uint2 o = *reinterpret_cast<const uint2*>(&W.nbr[buf][e].dbits);
        const uint64_t ok = (uint64_t)o.x << 32 | o.y;
        rank += ok < mk ? 1 : 0;
        same += ok == mk ? 1 : 0;
      }
      if (same > 1) {
        const uint32_t lk = cand_liftkey(me.lo, me.hi, sel, F);
        for (int e = 0; e < count; ++e) {
          const Nbr o = W.nbr[buf][e];
          if (o.dbits == me.dbits && o.slot == me.slot && e != me_i)
            rank += cand_liftkey(o.lo, o.hi, sel, F) < lk ? 1 : 0;
        }
      }
    }
    slot_out[l * KS + rank] = me.slot;
    w_out[l * KS + rank] = W.wgt[wb][me_i];
    if (d2_out) d2_out[l * KS + rank] = __uint_as_float(me.dbits);
  }
}

// Neighbour lists of width KS (NB = 32: Sec. 2.6; KALL: the whole support).
template <int KS>
__global__ void __launch_bounds__(THREADS, 4) k_neighbors(const float* __restrict__ q, Params P,
                                                       int32_t* __restrict__ slot_out, float* __restrict__ w_out,
                                                       float* __restrict__ d2_out) {
  __shared__ SearchLds<KS> S;
  WaveCtx c;
  if constexpr (KS == NB) {
    wave_ctx(P, c);
    TileInput<IN_QUERY, false> in(q, nullptr, c.base, c.nl, P, c.lane);
    TileSearch<IN_QUERY, 2> ts(P, S, c.wave, c.lane);
    for (int t0 = 0; t0 < c.nl; t0 += TILE) {
      const int nt = min(TILE, c.nl - t0);
      ts.frames(in.v, in.have, nt);
      in.advance(t0, P);
      for (int p = 0; 2 * p < nt; ++p) {
        ts.pair(p, 0);
        // a half wave orders each list of the pair
        const int h = c.lane >> 5, t = 2 * p + h;
        const Frame& F = ts.FR[t];
        Sel sel;
#pragma unroll
        for (int i = 0; i < 8; ++i) sel.s[i] = F.sel[i];
        if (t < nt)
          store_list<NB, 2, 2>(ts.W, h, h, c.lane & 31, NB, h ? ts.count1 : ts.count0, F, sel, c.base + t0 + t, slot_out,
                               w_out, d2_out);
        wave_lds_sync();
      }
    }
  } else {
    if (!wave_ctx(P, c)) return;
    Search<KS> srch(P, S.tab, S.wave[c.wave], S.tile, c.wave, c.lane);
    const QuadCtx<IN_QUERY> Q(P, c.lane);
    Frame* FR = S.frames[c.wave];
    for (int t0 = 0; t0 < c.nl; t0 += TILE) {
      const int nt = min(TILE, c.nl - t0);
      tile_frames(q, c.base + t0, nt, P, FR, Q, c.lane);
      for (int t = 0; t < nt; ++t) {
        const Sel sel = read_sel(FR[t]);
        const int count = srch.run(FR[t], sel, 0);
        store_list<KS, 1, 1>(S.wave[c.wave], 0, 0, c.lane, WAVE, count, FR[t], sel, c.base + t0 + t, slot_out, w_out,
                             d2_out);
        wave_lds_sync();
      }
    }
  }
}

// Row geometry of the backward's table reads for chunks of R rows: four lanes
// to a row, 16 bytes each, NC loads per row (the four lanes cover 64 bytes).
template <int DT, int M, int R = NB>
struct RowGeom {
  static constexpr int ES = DT == LRAM_F32 ? 4 : 2;      // table element bytes
  static constexpr int RB = M * ES;                       // row bytes
  static constexpr int LPR = 4;                           // lanes per row
  static constexpr int NC = RB / (16 * LPR);              // 16-byte chunks per lane and row
  static constexpr int RPP = WAVE / LPR;                  // rows per pass
  static constexpr int NP = R / RPP;                      // passes
  static constexpr int EPC = 16 / ES;                     // elements per 16-byte chunk
  static_assert(RB % (16 * LPR) == 0 && R % RPP == 0 && LPR % NP == 0, "row geometry");
};

// Rows handled together by the gathers of a list of KS neighbours.
template <int KS>
constexpr int chunk_rows() { return KS < NB ? KS : NB; }

template <int DT, int EPC>
__device__ __forceinline__ void unpack16(const uint4 v, float (&f)[EPC]) {
  if constexpr (DT == LRAM_F32) {
    f[0] = __uint_as_float(v.x);
    f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z);
    f[3] = __uint_as_float(v.w);
  } else {
    f[0] = bf16_lo(v.x); f[1] = bf16_hi(v.x);
    f[2] = bf16_lo(v.y); f[3] = bf16_hi(v.y);
    f[4] = bf16_lo(v.z); f[5] = bf16_hi(v.z);
    f[6] = bf16_lo(v.w); f[7] = bf16_hi(v.w);
  }
}

// Gather geometry of the forward: each lane reads 16 contiguous bytes of a row,
// LPR lanes cover a row, one load instruction covers RPI rows, NI instructions
// cover R rows; a lane accumulates EPL output elements over its NI rows, and
// the RPI row groups are summed across lanes.
template <int DT, int M, int R = NB>
struct FwdGeom {
  static constexpr int ES = DT == LRAM_F32 ? 4 : 2;
  static constexpr int RB = M * ES;
  static constexpr int LPR = RB / 16;
  static constexpr int RPI = WAVE / LPR;
  static constexpr int NI = R / RPI;
  static constexpr int EPL = 16 / ES;
  static_assert(LPR >= 4 && LPR <= 16 && R % RPI == 0, "forward gather geometry");
};

// Loads the rows r0 .. r0 + R of list `buf` (R = the geometry's chunk).
// full: every entry is real, so the loads need no condition; padding entries
// (location -1) are not read and give zeros.
template <int DT, int M, int KS, int R = NB, int NBUF, int WBUF>
__device__ __forceinline__ void fwd_issue(const char* __restrict__ tb, const WaveLds<KS, NBUF, WBUF>& W, int buf, int lane,
                                          bool full, uint4 (&v)[FwdGeom<DT, M, R>::NI], int r0 = 0) {
  using G = FwdGeom<DT, M, R>;
  const int rsub = lane / G::LPR, col = lane % G::LPR;
  if (full) {
#pragma unroll
    for (int p = 0; p < G::NI; ++p) {
      const uint32_t s = (uint32_t)W.nbr[buf][r0 + p * G::RPI + rsub].slot;
      v[p] = *reinterpret_cast<const uint4*>(tb + (size_t)s * G::RB + col * 16);
    }
  } else {
#pragma unroll
    for (int p = 0; p < G::NI; ++p) {
      const int32_t s = W.nbr[buf][r0 + p * G::RPI + rsub].slot;
      v[p] = make_uint4(0, 0, 0, 0);
      if (s >= 0) v[p] = *reinterpret_cast<const uint4*>(tb + (size_t)s * G::RB + col * 16);
    }
  }
}

// acc += sum over the rows r0 .. r0 + R of w_j * v_j (this lane's columns),
// weight list wb.
template <int DT, int M, int KS, int R = NB, int NBUF, int WBUF>
__device__ __forceinline__ void fwd_accumulate(const WaveLds<KS, NBUF, WBUF>& W, int wb, int lane,
                                               const uint4 (&v)[FwdGeom<DT, M, R>::NI],
                                               float (&acc)[FwdGeom<DT, M, R>::EPL], int r0 = 0) {
  using G = FwdGeom<DT, M, R>;
  const int rsub = lane / G::LPR;
#pragma unroll
  for (int p = 0; p < G::NI; ++p) {
    const float w = W.wgt[wb][r0 + p * G::RPI + rsub];
    float f[G::EPL];
    unpack16<DT, G::EPL>(v[p], f);
#pragma unroll
    for (int e = 0; e < G::EPL; ++e) acc[e] = fmaf(w, f[e], acc[e]);
  }
}

// Sums the row groups of the wave and writes out[l] once (nothing when !ok).
// Lane bits 5 and 4 always tell row groups apart: there the lanes exchange
// halves of their columns while they add, so a lane ends with a quarter of
// its columns (one fp32, two bf16); the bits below are plain sums.
template <int DT, int M>
__device__ __forceinline__ void fwd_store(int lane, int64_t l, float (&acc)[FwdGeom<DT, M>::EPL],
                                          void* out, bool ok = true) {
  using G = FwdGeom<DT, M>;
  constexpr int Q = G::EPL / 4;
#pragma unroll
  for (int e = 0; e < 2 * Q; ++e) acc[e] = add_halves_f32<32>(acc[e], acc[e + 2 * Q]);
#pragma unroll
  for (int e = 0; e < Q; ++e) {
    acc[e] = add_halves_f32<16>(acc[e], acc[e + Q]);
    if constexpr (G::LPR <= 8) acc[e] += dpp_f32<DPP_ROR8>(acc[e]);
    if constexpr (G::LPR <= 4) acc[e] += dpp_f32<DPP_ROR4>(acc[e]);
  }
  if ((lane & 15) < G::LPR && ok) {
    const int piece = (lane & 15) * 4 + ((lane & 32) ? 2 : 0) + ((lane & 16) ? 1 : 0);
    char* ob = reinterpret_cast<char*>(out) + (size_t)l * G::RB + piece * 4;
    if constexpr (DT == LRAM_F32)
      *reinterpret_cast<float*>(ob) = acc[0];
    else
      *reinterpret_cast<uint32_t*>(ob) = pack_bf16x2(acc[0], acc[1]);
  }
}

template <int DT, int M>
__device__ __forceinline__ void fwd_consume(const WaveLds<NB, 2, 4>& W, int wb, int lane, int64_t l,
                                            const uint4 (&v)[FwdGeom<DT, M>::NI], void* out,
                                            bool ok = true) {
  float acc[FwdGeom<DT, M>::EPL];
#pragma unroll
  for (int e = 0; e < FwdGeom<DT, M>::EPL; ++e) acc[e] = 0.0f;
  fwd_accumulate<DT, M, NB>(W, wb, lane, v, acc);
  fwd_store<DT, M>(lane, l, acc, out, ok);
}

// Waves per SIMD that the forward and the backward are built for: 256-byte fp32
// rows need more registers than four leave, and the activation layer's inline fp64
// arguments (small batches only) more than three: held to three they spilled up
// to 36 registers (m = 64 fp32, three / two, forward of 32 lookups 9.2 / 7.5 us, of 6,000
// 17.7 / 14.7, backward 16.4 / 14.6, 65.2 / 63.2).
template <int DT, int M, int TH>
constexpr int kernel_waves() { return TH == IN_THETA ? 2 : (DT == LRAM_F32 && M == 64 ? 3 : 4); }

// TH: the lookups' input; the activation layer's scale s is folded into the
// weights by the search.  IN_STAGED: q is the output itself, lookup l's record
// at the start of its row, read by the wave that writes the row afterwards.
// ORD: visit the lookups in the order perm (position -> lookup, e.g. sorted
// by closest lattice point, so that lookups sharing rows run close together
// in time and on the same XCD); outputs still go to the lookup's row.
// SAVE: write every lookup's list for the backward (NbrList).
template <int DT, int M, int TH, bool ORD = false, bool SAVE = false>
__global__ void __launch_bounds__(THREADS, (kernel_waves<DT, M, TH>())) k_forward(const float* q, Params P,
                                                     const void* __restrict__ table, void* out,
                                                     const uint32_t* __restrict__ perm, NbrList save) {
  using G = FwdGeom<DT, M>;
  __shared__ SearchLds<NB, 2, 4> S;
  WaveCtx c;
  wave_ctx(P, c, ORD);
  TileInput<TH, ORD> in(q, perm, c.base, c.nl, P, c.lane);
  TileSearch<TH, 4> ts(P, S, c.wave, c.lane);
  const char* tb = reinterpret_cast<const char*>(table);
  for (int t0 = 0; t0 < c.nl; t0 += TILE) {
    const int nt = min(TILE, c.nl - t0), np = (nt + 1) / 2;
    ts.frames(in.v, in.have, nt);
    in.advance(t0, P);
    uint4 v0[G::NI], v1[G::NI];
    // pair p is searched while the rows of pair p - 1 are in flight
#pragma unroll 1
    for (int p = 0; p <= np; ++p) {
      bool ok;
      if (p < np) {
        ts.pair(p, 2 * (p & 1));
        if constexpr (SAVE) {
          const int64_t l0 = in.lookup(t0, 2 * p, P, ok);
          ts.one.save(0, 2 * (p & 1), save, l0, ok);
          const int64_t l1 = in.lookup(t0, 2 * p + 1, P, ok);
          ts.one.save(1, 2 * (p & 1) + 1, save, l1, ok);
        }
      }
      if (p > 0) {
        const int wb = 2 * ((p - 1) & 1);
        const int64_t l0 = in.lookup(t0, 2 * p - 2, P, ok);
        fwd_consume<DT, M>(ts.W, wb, c.lane, l0, v0, out, ok);
        const int64_t l1 = in.lookup(t0, 2 * p - 1, P, ok);
        fwd_consume<DT, M>(ts.W, wb + 1, c.lane, l1, v1, out, ok);
      }
      if (p < np) {
        fwd_issue<DT, M, NB>(tb, ts.W, 0, c.lane, ts.count0 == NB, v0);
        fwd_issue<DT, M, NB>(tb, ts.W, 1, c.lane, ts.count1 == NB, v1);
      }
    }
    wave_lds_sync();
  }
}

// Forward with lists of KS != 32 neighbours (the variable-k and untruncated
// lookups): per lookup, the rows are gathered in chunks of up to 32, only as
// many chunks as the lookup has neighbours.
template <int DT, int M, int KS>
__global__ void __launch_bounds__(THREADS) k_forward_k(const float* __restrict__ q, Params P,
                                                       const void* __restrict__ table, void* __restrict__ out) {
  constexpr int R = chunk_rows<KS>();
  using G = FwdGeom<DT, M, R>;
  __shared__ SearchLds<KS> S;
  WaveCtx c;
  if (!wave_ctx(P, c)) return;
  Search<KS> srch(P, S.tab, S.wave[c.wave], S.tile, c.wave, c.lane);
  WaveLds<KS>& W = S.wave[c.wave];
  const QuadCtx<IN_QUERY> Q(P, c.lane);
  Frame* FR = S.frames[c.wave];
  const char* tb = reinterpret_cast<const char*>(table);
  for (int t0 = 0; t0 < c.nl; t0 += TILE) {
    const int nt = min(TILE, c.nl - t0);
    tile_frames(q, c.base + t0, nt, P, FR, Q, c.lane);
    for (int t = 0; t < nt; ++t) {
      const int count = srch.run(FR[t], read_sel(FR[t]), 0);
      float acc[G::EPL];
#pragma unroll
      for (int e = 0; e < G::EPL; ++e) acc[e] = 0.0f;
      for (int r0 = 0; r0 < count; r0 += R) {
        uint4 v[G::NI];
        fwd_issue<DT, M, KS, R>(tb, W, 0, c.lane, r0 + R <= count, v, r0);
        fwd_accumulate<DT, M, KS, R>(W, 0, c.lane, v, acc, r0);
      }
      fwd_store<DT, M>(c.lane, c.base + t0 + t, acc, out);
      wave_lds_sync();
    }
  }
}

}  // namespace
