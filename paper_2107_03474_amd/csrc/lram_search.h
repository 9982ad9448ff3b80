// lram_search.h -- part of liblram (included by lram.hip only).
//
// The neighbour search (Sec. 2.6): phase A (wrap, closest point of Lambda, the
// signed permutation into F), the general search of one lookup by a wave
// (per-query tables, candidate scan, selection of the closest k, locations and
// weights), and the tile search of 16 lookups by a wave for k = 32.

#pragma once

namespace {

// ---------------------------------------------------------------------------
// Phase A: closest point of Lambda and the reduction into F (Sec. 2.6).

// Nearest point of D8 = {r in Z^8 : sum r even} to y: round every coordinate,
// and if the sum is odd re-round the coordinate that was worst rounded.
__device__ __forceinline__ void d8_round(const float (&y)[8], int (&r)[8]) {
  float dmax = -1.0f;
  int jmax = 0, s = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float ri = rintf(y[i]);
    r[i] = (int)ri;
    float d = fabsf(y[i] - ri);
    if (d > dmax) {
      dmax = d;
      jmax = i;
    }
    s += r[i];
  }
  if (s & 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i == jmax) r[i] += (y[i] > (float)r[i]) ? 1 : -1;
  }
}

// The lookups' input (the template parameter TH of everything that reads it):
// q [L][8]; z [L][16] of the activation layer (Sec. 2.3), turned into q where
// it is read; or q and the output scale s of the activation layer as
// k_theta_coords left them, in records of Params::stage floats (q in the first
// 8, s in the 9th).  The arguments of z take 8 fp64 atan2 and square roots per
// lookup: in front of a tile's search no row loads cover that latency, and
// their registers cost a wave per SIMD, so large batches have them formed by a
// kernel of their own, in rows of the output that the lookups write last
// (forward of 262,144 lookups, m = 64 fp32: 338 -> 281 us, of 524,288, m = 64
// bf16: 505 -> 454 us, k_theta_coords' 17 and 25 us included).
enum : int { IN_QUERY = 0, IN_THETA = 1, IN_STAGED = 2 };

// Input float4s per lookup.
template <int TH>
constexpr int in_vec4() { return TH == IN_THETA ? 4 : 2; }

// The query of one lookup and its output scale, from the lookup's input
// vectors v.  IN_QUERY: q itself (8 floats), scale 1.  IN_THETA, the
// activation layer of Sec. 2.3: z_i = in[2i] + i in[2i+1], q_i = (K_i / 2 pi)
// arg z_i formed in fp64 and rounded once to fp32, scale (sum_i 1/|z_i|)^-1 (0
// when some z_i = 0); a non-finite input gives a NaN query (empty neighbour
// list) and scale 0.
template <int TH>
__device__ __forceinline__ void query_from(const float4 (&v)[in_vec4<TH>()], const Params P, float (&qq)[8],
                                           float& scale) {
  if constexpr (TH != IN_THETA) {
    qq[0] = v[0].x; qq[1] = v[0].y; qq[2] = v[0].z; qq[3] = v[0].w;
    qq[4] = v[1].x; qq[5] = v[1].y; qq[6] = v[1].z; qq[7] = v[1].w;
    scale = 1.0f;
  } else {
    float z[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      z[4 * k] = v[k].x; z[4 * k + 1] = v[k].y; z[4 * k + 2] = v[k].z; z[4 * k + 3] = v[k].w;
    }
    bool finite = true;
    double inv = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double a = z[2 * i], b = z[2 * i + 1];
      finite = finite && isfinite(z[2 * i]) && isfinite(z[2 * i + 1]);
      inv += 1.0 / sqrt(a * a + b * b);
      qq[i] = (float)(atan2(b, a) * P.cK[i]);
    }
    if (!finite) qq[0] = __builtin_nanf("");
    scale = finite ? (float)(1.0 / inv) : 0.0f;
  }
}

template <int TH>
__device__ __forceinline__ void load_input(const float* __restrict__ in, float4 (&v)[in_vec4<TH>()]) {
#pragma unroll
  for (int k = 0; k < in_vec4<TH>(); ++k) v[k] = reinterpret_cast<const float4*>(in)[k];
}

template <int TH>
__device__ __forceinline__ void load_query(const float* __restrict__ in, const Params P, float (&qq)[8],
                                           float& scale) {
  float4 v[in_vec4<TH>()];
  load_input<TH>(in, v);
  query_from<TH>(v, P, qq, scale);
}

// Wrapped Lambda-scale query x and the closest point c of Lambda (either coset);
// false for a non-finite query (x = 0 then).
__device__ __forceinline__ bool closest_point(const float (&qq)[8], bool have, const Params P, float (&x)[8],
                                              int (&c)[8]) {
  bool valid = have;
  if (have) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float xi = 2.0f * qq[i];
      if (!(xi >= 0.0f && xi < P.twoK[i])) xi = fmodf(xi, P.twoK[i]);
      valid = valid && isfinite(xi);
      x[i] = xi;
    }
  }
  if (!valid) {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = 0.0f;
  }
  // Lambda = 2 D8  u  (2 D8 + 1): decode both cosets at half scale.
  float y0[8], y1[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    y0[i] = x[i] * 0.5f;
    y1[i] = (x[i] - 1.0f) * 0.5f;
  }
  int r0[8], r1[8];
  d8_round(y0, r0);
  d8_round(y1, r1);
  float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float e0 = x[i] - (float)(2 * r0[i]);
    float e1 = x[i] - (float)(2 * r1[i] + 1);
    d0 += e0 * e0;
    d1 += e1 * e1;
  }
  const bool odd = d1 < d0;
#pragma unroll
  for (int i = 0; i < 8; ++i) c[i] = odd ? 2 * r1[i] + 1 : 2 * r0[i];
  return valid;
}

// Lane constants of phase A: lane = 4 * (lookup of the tile) + quarter; a
// quarter holds the original coordinates 2 * quarter and 2 * quarter + 1.
template <int TH>
struct QuadCtx {
  int n, kq;
  float tk0, tk1;    // torus sides at the Lambda scale
  double ck0, ck1;   // K_i / (2 pi) (TH)
  __device__ QuadCtx(const Params P, int lane) : n(lane >> 2), kq(lane & 3) {
    tk0 = P.twoK[0];
    tk1 = P.twoK[1];
    ck0 = P.cK[0];
    ck1 = P.cK[1];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      tk0 = kq == k ? P.twoK[2 * k] : tk0;
      tk1 = kq == k ? P.twoK[2 * k + 1] : tk1;
      if constexpr (TH == IN_THETA) {
        ck0 = kq == k ? P.cK[2 * k] : ck0;
        ck1 = kq == k ? P.cK[2 * k + 1] : ck1;
      }
    }
  }
};

// Input values of one quarter of a lookup: q_{2k}, q_{2k+1}, or z_{2k}, z_{2k+1}
// as (Re, Im, Re, Im).
template <int TH>
struct QuadIn {
  float v[TH == IN_THETA ? 4 : 2];
  float s;  // IN_STAGED: the output scale
};

template <int TH>
__device__ __forceinline__ QuadIn<TH> load_quad(const float* in, size_t l, int kq, int stage) {
  QuadIn<TH> o;
  o.s = 1.0f;
  if constexpr (TH == IN_THETA) {
    const float4 a = reinterpret_cast<const float4*>(in + l * 16)[kq];
    o.v[0] = a.x; o.v[1] = a.y; o.v[2] = a.z; o.v[3] = a.w;
  } else {
    const float* r = in + l * (size_t)(TH == IN_STAGED ? stage : 8);
    const float2 a = reinterpret_cast<const float2*>(r)[kq];
    o.v[0] = a.x; o.v[1] = a.y;
    if constexpr (TH == IN_STAGED) o.s = r[8];
  }
  return o;
}

__device__ __forceinline__ float quad_sum(float x) {
  x += dpp_f32<DPP_XOR1>(x);
  return x + dpp_f32<DPP_XOR2>(x);
}
__device__ __forceinline__ uint32_t quad_xor(uint32_t x) {
  x ^= dpp_u32<DPP_XOR1>(x);
  return x ^ dpp_u32<DPP_XOR2>(x);
}
__device__ __forceinline__ uint32_t quad_max(uint32_t x) {
  x = max(x, dpp_u32<DPP_XOR1>(x));
  return max(x, dpp_u32<DPP_XOR2>(x));
}
// Non-negative a with the coordinate index in its last three bits: keys of the
// eight coordinates are distinct and order like a (equal but for those bits:
// the lower index first).
__device__ __forceinline__ uint32_t coord_key(float a, int i) { return (__float_as_uint(a) & ~7u) | (uint32_t)(7 - i); }

// Nearest point of D8 to y, two coordinates to a lane: round every
// coordinate, and if the sum is odd re-round the one that was worst rounded
// (to within 2^-20 relative of the worst: where two are that close, either
// choice is a closest point to within the same).
__device__ __forceinline__ void d8_round_quad(float y0, float y1, int kq, int& r0, int& r1) {
  const float f0 = rintf(y0), f1 = rintf(y1);
  r0 = (int)f0;
  r1 = (int)f1;
  const uint32_t k0 = coord_key(fabsf(y0 - f0), 2 * kq), k1 = coord_key(fabsf(y1 - f1), 2 * kq + 1);
  const uint32_t worst = quad_max(max(k0, k1));
  const bool odd = quad_xor((uint32_t)(r0 + r1)) & 1u;
  if (odd && k0 == worst) r0 += y0 > f0 ? 1 : -1;
  if (odd && k1 == worst) r1 += y1 > f1 ? 1 : -1;
}

// Phase A of a tile: the frames of its 16 lookups, four lanes each (in: this
// lane's quarter; have: the lookup exists).  The frames' sel words hold -z_r/2
// afterwards; returns this lane's two v_perm selectors, which finish_frames
// puts there once the selection has read z.
template <int TH>
__device__ __forceinline__ uint2 make_frames(const QuadIn<TH>& in, bool have, const QuadCtx<TH>& Q, Frame* fr) {
  const int kq = opaque(Q.kq), n = opaque(Q.n), i0 = 2 * kq, i1 = i0 + 1;  // (opaque: as in tile_select)
  const int quad0 = 4 * n;
  float q0, q1, scale = in.s;
  bool fin = have;
  if constexpr (TH == IN_THETA) {
    const double a0 = in.v[0], b0 = in.v[1], a1 = in.v[2], b1 = in.v[3];
    fin = fin && isfinite(in.v[0]) && isfinite(in.v[1]) && isfinite(in.v[2]) && isfinite(in.v[3]);
    double inv = 1.0 / sqrt(a0 * a0 + b0 * b0) + 1.0 / sqrt(a1 * a1 + b1 * b1);
    inv += dpp_f64<DPP_XOR1>(inv);
    inv += dpp_f64<DPP_XOR2>(inv);
    q0 = (float)(atan2(b0, a0) * Q.ck0);
    q1 = (float)(atan2(b1, a1) * Q.ck1);
    scale = (float)(1.0 / inv);
  } else {
    q0 = in.v[0];
    q1 = in.v[1];
  }
  float x0 = 2.0f * q0, x1 = 2.0f * q1;
  if (!(x0 >= 0.0f && x0 < Q.tk0)) x0 = fmodf(x0, opaque(Q.tk0));
  if (!(x1 >= 0.0f && x1 < Q.tk1)) x1 = fmodf(x1, opaque(Q.tk1));
  fin = fin && isfinite(x0) && isfinite(x1);
  const bool valid = ((__ballot(fin) >> quad0) & 15u) == 15u;
  if (!valid) x0 = x1 = 0.0f;
  // Lambda = 2 D8  u  (2 D8 + 1): decode both cosets at half scale
  int e0, e1, o0, o1;
  d8_round_quad(x0 * 0.5f, x1 * 0.5f, kq, e0, e1);
  d8_round_quad((x0 - 1.0f) * 0.5f, (x1 - 1.0f) * 0.5f, kq, o0, o1);
  e0 *= 2;
  e1 *= 2;
  o0 = 2 * o0 + 1;
  o1 = 2 * o1 + 1;
  const float ye0 = x0 - (float)e0, ye1 = x1 - (float)e1, yo0 = x0 - (float)o0, yo1 = x1 - (float)o1;
  const float de = quad_sum(ye0 * ye0 + ye1 * ye1), dd = quad_sum(yo0 * yo0 + yo1 * yo1);
  const bool odd = dd < de;  // the same in the quad's lanes: their sums commute
  const int c0 = odd ? o0 : e0, c1 = odd ? o1 : e1;
  const float y0 = odd ? yo0 : ye0, y1 = odd ? yo1 : ye1;
  const float a0 = fabsf(y0), a1 = fabsf(y1);
  uint32_t n0 = y0 < 0.0f ? 1u : 0u, n1 = y1 < 0.0f ? 1u : 0u;
  // rank of |y_i| in descending order: F position of coordinate i
  const uint32_t k0 = coord_key(a0, i0), k1 = coord_key(a1, i1);
  int r0 = k1 > k0 ? 1 : 0, r1 = 1 - r0;
  auto other = [&](uint32_t k) {
    r0 += k > k0 ? 1 : 0;
    r1 += k > k1 ? 1 : 0;
  };
  other(dpp_u32<DPP_XOR1>(k0));
  other(dpp_u32<DPP_XOR1>(k1));
  other(dpp_u32<DPP_XOR2>(k0));
  other(dpp_u32<DPP_XOR2>(k1));
  other(dpp_u32<DPP_XOR3>(k0));
  other(dpp_u32<DPP_XOR3>(k1));
  // only even numbers of sign changes are isometries of Lambda: fix the parity
  // on the coordinate that lands last (smallest |y|); its z is negative then
  const uint32_t par = quad_xor(n0 ^ n1);
  const bool f0 = par && r0 == 7, f1 = par && r1 == 7;
  n0 ^= f0 ? 1u : 0u;
  n1 ^= f1 ? 1u : 0u;
  Frame& F = fr[n];
  reinterpret_cast<uint4*>(F.rec)[kq] = make_uint4(__float_as_uint(x0), 2u * (uint32_t)c0 | n0, __float_as_uint(x1),
                                                   2u * (uint32_t)c1 | n1);
  F.sel[r0] = __float_as_uint(f0 ? 0.5f * a0 : -0.5f * a0);
  F.sel[r1] = __float_as_uint(f1 ? 0.5f * a1 : -0.5f * a1);
  if (kq == 0)
    reinterpret_cast<uint4*>(&F.valid)[0] =
        make_uint4(valid ? 1u : 0u, __float_as_uint(valid ? scale : 0.0f), __float_as_uint(odd ? dd : de), 0u);
  return make_uint2(0x0C0C0C00u | (uint32_t)r0, 0x0C0C0C00u | (uint32_t)r1);
}

__device__ __forceinline__ void finish_frames(uint2 sel, int lane, Frame* fr) {
  reinterpret_cast<uint2*>(fr[lane >> 2].sel)[lane & 3] = sel;
}

// ---------------------------------------------------------------------------
// The neighbour search of one lookup by a wave.

// Packed candidate bytes: byte j = 4*(p_j - CMIN) + 64*w (the LDS byte offset of
// table entry (., w, p_j) within a coordinate's 256-byte block).  Strict list,
// then boundary list; the words hold w = 0.
struct PackedCandidates {
  uint32_t w[E8_NSTRICT + E8_NBOUNDARY][2];
};
constexpr PackedCandidates pack_candidates() {
  constexpr signed char strict[E8_NSTRICT][8] = E8_STRICT_INIT;
  constexpr signed char boundary[E8_NBOUNDARY][8] = E8_BOUNDARY_INIT;
  PackedCandidates o{};
  for (int i = 0; i < E8_NSTRICT + E8_NBOUNDARY; ++i)
    for (int r = 0; r < 8; ++r) {
      const int p = i < E8_NSTRICT ? strict[i][r] : boundary[i - E8_NSTRICT][r];
      o.w[i][r / 4] |= (uint32_t)(4 * (p - CMIN)) << (8 * (r % 4));
    }
  return o;
}
__constant__ __align__(16) PackedCandidates c_packed = pack_candidates();

template <int LIST>
__device__ __forceinline__ bool load_candidate(int idx, uint32_t wbyte, uint32_t& lo, uint32_t& hi) {
  constexpr int n = LIST == 0 ? E8_NSTRICT : E8_NBOUNDARY;
  const bool in = idx < n;
  const uint2 c = *reinterpret_cast<const uint2*>(c_packed.w[(LIST == 0 ? 0 : E8_NSTRICT) + (in ? idx : 0)]);
  lo = in ? c.x + wbyte * 0x01010101u : 0u;
  hi = in ? c.y + wbyte * 0x01010101u : 0u;
  return in;
}

struct Sel {
  uint32_t s[8];  // v_perm selectors (uniform): byte r_i of the candidate into byte 0
  bool valid;
};

__device__ __forceinline__ Sel read_sel(const Frame& F) {
  Sel o;
  const uint4 a = reinterpret_cast<const uint4*>(F.sel)[0];
  const uint4 b = reinterpret_cast<const uint4*>(F.sel)[1];
  o.s[0] = uniform(a.x); o.s[1] = uniform(a.y); o.s[2] = uniform(a.z); o.s[3] = uniform(a.w);
  o.s[4] = uniform(b.x); o.s[5] = uniform(b.y); o.s[6] = uniform(b.z); o.s[7] = uniform(b.w);
  o.valid = uniform(F.valid) != 0u;
  return o;
}

// Recipe distance^2 of candidate (lo,hi): sum over original coordinates i, in
// order, of the per-query table entry (x_i - k_i)^2 (already fp32-rounded).
__device__ __forceinline__ float cand_d2(const float* qt, uint32_t lo, uint32_t hi, const Sel& sel) {
  float d = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float v = lds_f32(qt, __builtin_amdgcn_perm(hi, lo, sel.s[i]) + 256u * i);
    d = (i == 0) ? v : d + v;
  }
  return d;
}

__device__ __forceinline__ int32_t cand_slot(const uint32_t* st, uint32_t lo, uint32_t hi, const Sel& sel) {
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) m += lds_u32(st, __builtin_amdgcn_perm(hi, lo, sel.s[i]) + 256u * i);
  return (int32_t)(m >> 1);
}

// Lexicographic key of the lattice point itself (only consulted between equal
// (distance, location) pairs, which requires a torus side of 2).
__device__ __forceinline__ uint32_t cand_liftkey(uint32_t lo, uint32_t hi, const Sel& sel, const Frame& F) {
  uint32_t key = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t a = __builtin_amdgcn_perm(hi, lo, sel.s[i]);
    const int p = (int)((a & 31u) >> 2) + CMIN;
    const int rc = (int)F.rec[i].y;
    const int k = (rc & 1) ? (rc >> 1) - p : (rc >> 1) + p;
    key |= ((uint32_t)(k + 8) & 15u) << (4 * (7 - i));
  }
  return key;
}

template <int NS>
__device__ __forceinline__ int count_below(const uint32_t (&key)[NS], uint32_t t) {
  int c = 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) c += __popcll(__ballot(key[s] < t));
  return c;
}

// Threshold selection of the closest ks (Sec. 2.6: ks = 32) over NS candidate
// slots per lane.  Returns the number selected; a slot is selected iff key < thr, or
// key == tie_key and it is among the `need` first of those in (location,
// lattice point) order (tie_key = KEY_INF when there is no tie).  *suspect is
// set when a point of the boundary list could enter the selection (the ks-th
// distance is within 1e-3 of the support edge, or fewer than ks points are in
// the support).
template <int NS>
__device__ __forceinline__ int threshold_k(const uint32_t (&key)[NS], const int ks, uint32_t& thr, uint32_t& tie_key,
                                           int& need, bool& suspect) {
  tie_key = KEY_INF;
  need = 0;
  const int n8 = count_below(key, KEY_8);
  if (n8 <= ks) {
    thr = KEY_8;
    suspect = true;
    return n8;
  }
  // bisection on the (monotone) bit patterns of non-negative floats:
  // invariant count(< lo) < ks < count(< hi)
  uint32_t lo_k = KEY_4, hi_k = KEY_8;
  int c = count_below(key, lo_k);
  if (c == ks) {
    thr = lo_k;
    suspect = false;
    return ks;
  }
  if (c > ks) {
    hi_k = lo_k;
    lo_k = 0;
  }
  while (hi_k - lo_k > 1) {
    const uint32_t mid = lo_k + ((hi_k - lo_k) >> 1);
    c = count_below(key, mid);
    if (c == ks) {
      thr = mid;
      suspect = mid > KEY_SUSPECT;
      return ks;
    }
    if (c < ks)
      lo_k = mid;
    else
      hi_k = mid;
  }
  // several candidates share the distance bits lo_k at the 32nd place
  thr = lo_k;
  tie_key = lo_k;
  need = ks - count_below(key, lo_k);
  suspect = lo_k > KEY_SUSPECT;
  return ks;
}

// Inclusive prefix sum across the 64 lanes of a wave (DPP row shifts, then row
// broadcasts to carry the row totals).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false); // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false); // row_bcast:31
  return x;
}

// Threshold selection of the closest ks through a 64-bucket histogram of the
// distance bits on [4, 8) (bucket = top six mantissa bits): one LDS atomic per
// candidate, a wave prefix sum and one ballot locate the bucket of the ks-th
// point; the bisection then only runs inside that bucket.  Same contract as
// threshold_k.
template <int NS>
__device__ __forceinline__ int threshold_k_hist(const uint32_t (&key)[NS], uint32_t* hist, int lane, const int ks,
                                                uint32_t& thr, uint32_t& tie_key, int& need, bool& suspect) {
  const int clow = count_below(key, KEY_4);
  if (clow >= ks) return threshold_k<NS>(key, ks, thr, tie_key, need, suspect);  // never expected
  hist[lane] = 0;
  wave_lds_sync();
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (key[s] >= KEY_4 && key[s] < KEY_8) atomicAdd(&hist[(key[s] - KEY_4) >> 17], 1u);
  wave_lds_sync();
  const uint32_t h = hist[lane];
  const uint32_t pre = wave_inclusive_scan(h);
  const int n8 = clow + (int)__builtin_amdgcn_readlane(pre, 63);
  tie_key = KEY_INF;
  need = 0;
  if (n8 <= ks) {
    thr = KEY_8;
    suspect = true;
    return n8;
  }
  const uint64_t m = __ballot(clow + (int)pre >= ks);
  const int b = (int)__builtin_ctzll(m);
  const int below = clow + (int)__builtin_amdgcn_readlane(pre, b) - (int)__builtin_amdgcn_readlane(h, b);
  const int inb = (int)__builtin_amdgcn_readlane(h, b);
  uint32_t lo_k = KEY_4 + ((uint32_t)b << 17), hi_k = lo_k + (1u << 17);
  if (below + inb == ks) {
    thr = hi_k;
    suspect = hi_k > KEY_SUSPECT;
    return ks;
  }
  // invariant count(< lo) = below < ks < count(< hi)
  while (hi_k - lo_k > 1) {
    const uint32_t mid = lo_k + ((hi_k - lo_k) >> 1);
    const int c = count_below(key, mid);
    if (c == ks) {
      thr = mid;
      suspect = mid > KEY_SUSPECT;
      return ks;
    }
    if (c < ks)
      lo_k = mid;
    else
      hi_k = mid;
  }
  thr = lo_k;
  tie_key = lo_k;
  need = ks - count_below(key, lo_k);
  suspect = lo_k > KEY_SUSPECT;
  return ks;
}

// Lists other than the closest 32 keep the packed strict candidates in
// registers; the closest 32 come here only where the tile search cannot decide
// and take all of them from the tile search's LDS.
template <int KS, int NBUF = (KS == NB ? 2 : 1), int WBUF = NBUF, bool SELECT = true>
struct Search {
  Tables& S;
  WaveLds<KS, NBUF, WBUF>& W;
  TileLds<KS == NB && SELECT>& T;
  int lane;
  uint32_t wbyte;
  static constexpr int NC_REG = KS == NB ? 1 : NS_STRICT;
  uint32_t lo[NC_REG], hi[NC_REG];
  // lists of 64 and the untruncated lookup scan the boundary candidates often
  // (whenever the support holds fewer than 64 points) or always: they stay in
  // registers too (lists of 16 read them from constant memory on the rare
  // path that needs them)
  static constexpr int NB_REG = KS >= 64 ? NS_BOUND : 1;
  uint32_t blo[NB_REG], bhi[NB_REG];
  // lane constants of the table build: coordinate i = lane/8, value v = lane%8
  int ti, tp, tK;
  uint32_t tS, tN0;
  uint32_t toff;  // byte offset of entry (i, w, v)

  // (the kernel argument is read field by field: holding a reference to it
  // would force the argument block into private memory)
  __device__ Search(const Params P, Tables& s, WaveLds<KS, NBUF, WBUF>& wv, TileLds<KS == NB && SELECT>& tl, int w, int l)
      : S(s), W(wv), T(tl), lane(l), wbyte(64u * (uint32_t)w) {
    if constexpr (NC_REG == NS_STRICT) {
#pragma unroll
      for (int k = 0; k < NS_STRICT; ++k) load_candidate<0>(lane + WAVE * k, wbyte, lo[k], hi[k]);
    }
    if constexpr (NB_REG == NS_BOUND) {
#pragma unroll
      for (int k = 0; k < NS_BOUND; ++k) load_candidate<1>(lane + WAVE * k, wbyte, blo[k], bhi[k]);
    }
    ti = lane >> 3;
    tp = (lane & 7) + CMIN;
    tK = P.K[0];
    tS = P.S[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) {
      tK = ti == i ? P.K[i] : tK;
      tS = ti == i ? P.S[i] : tS;
    }
    tN0 = ti == 0 ? P.N : 0u;
    toff = 256u * ti + wbyte + 4u * (lane & 7);
  }

  // Candidate (lo, hi) of lane-slot s; false where the slot has none.
  __device__ __forceinline__ bool cand(int s, uint32_t& l, uint32_t& h) const {
    const bool strict = s < NS_STRICT;
    const int i = strict ? lane + WAVE * s : lane + WAVE * (s - NS_STRICT);
    const bool in = i < (strict ? E8_NSTRICT : E8_NBOUNDARY);
    if constexpr (KS == NB) {
      const uint2 c = T.cand[in ? (strict ? i : E8_NSTRICT + i) : 0];
      l = c.x + wbyte * 0x01010101u;
      h = c.y + wbyte * 0x01010101u;
    } else if (strict) {
      l = lo[s];
      h = hi[s];
    } else if constexpr (NB_REG == NS_BOUND) {
      l = blo[s - NS_STRICT];
      h = bhi[s - NS_STRICT];
    } else {
      load_candidate<1>(opaque(i), wbyte, l, h);
    }
    return in;
  }

  // Per-query tables for frame F: entry (i, v) describes the lattice
  // coordinate k_i = c_i + s'_i (v + CMIN); list h of a pair.
  __device__ __forceinline__ void build_tables(const Frame& F, int h = 0) {
    const uint2 r = F.rec[ti];
    const int neg = -(int)(r.y & 1u);
    const int k = ((int)r.y >> 1) + ((tp ^ neg) - neg);
    const float e = __uint_as_float(r.x) - (float)k;
    const float e2 = e * e;
    // floor(k / 2) mod K: |x_i| < 2K, |x_i - c_i| <= 2 and |p| <= 4 put floor(k / 2) within [-K-3, K+3]
    const uint32_t Y = torus_coord((uint32_t)(k >> 1), (uint32_t)tK);
    const uint32_t sl = Y * tS + (tN0 & (uint32_t)-(k & 1));
    const uint32_t o = toff + 32u * (uint32_t)h;
    *reinterpret_cast<float*>(reinterpret_cast<char*>(S.qt) + o) = e2;
    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(S.st) + o) = sl;
    *reinterpret_cast<float*>(reinterpret_cast<char*>(S.et) + o) = e;
  }

  // Writes the selected candidates into W.nbr[buf][0..count), or their indices
  // into lookup buf's list of the tile for the closest 32 (slot-major, then
  // lane order); ties at the ks-th place are broken by (location, lattice point).
  template <int NS>
  __device__ __forceinline__ void emit(const uint32_t (&key)[NS], uint32_t thr, uint32_t tie_key, int need,
                                       const Sel& sel, const Frame& F, int buf) {
    int nt = 0;
    if (tie_key != KEY_INF) {
      // rare: list the tied candidates' (location, lattice point) keys (unrolled:
      // a runtime index into the candidate registers would spill them)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bool tied = key[s] == tie_key;
        const uint64_t m = __ballot(tied);
        if (m) {
          uint32_t l, h;
          cand(s, l, h);
          const int pos = nt + prefix_count(m);
          if (tied && pos < tie_max<KS>()) {
            W.tie[pos][0] = (uint32_t)cand_slot(S.st, l, h, sel);
            W.tie[pos][1] = cand_liftkey(l, h, sel, F);
          }
          nt += __popcll(m);
        }
      }
      nt = min(nt, tie_max<KS>());
      wave_lds_sync();
    }
    int base = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      bool p = key[s] < thr;
      if (tie_key != KEY_INF && key[s] == tie_key) {
        uint32_t l, h;
        cand(s, l, h);
        const uint32_t ms = (uint32_t)cand_slot(S.st, l, h, sel);
        const uint32_t mk = cand_liftkey(l, h, sel, F);
        int rank = 0;
#pragma unroll 1
        for (int e = 0; e < nt; ++e) {
          const uint32_t es = W.tie[e][0], ek = W.tie[e][1];
          rank += (es < ms || (es == ms && ek < mk)) ? 1 : 0;
        }
        p = rank < need;
      }
      const uint64_t m = __ballot(p);
      const int pos = base + prefix_count(m);
      if (p && pos < KS) {
        if constexpr (KS == NB) {
          T.idx[wbyte / 64][buf][pos] =
              (uint16_t)(s < NS_STRICT ? lane + WAVE * s : E8_NSTRICT + lane + WAVE * (s - NS_STRICT));
        } else {
          uint32_t l, h;
          cand(s, l, h);
          Nbr& n = W.nbr[buf][pos];
          n.lo = l;
          n.hi = h;
          n.dbits = key[s];
        }
      }
      base += __popcll(m);
    }
  }

  // Full neighbour search of frame F into buffer `buf`: W.nbr[buf][0..KS) with
  // (lo, hi, dbits, slot) and W.wgt[buf] with the fp32 recipe weights, padded
  // with slot -1 / weight 0 -- for the closest 32 only the candidates' indices,
  // into lookup buf's list of the tile.  Returns the number of real neighbours.
  __device__ __forceinline__ int run(const Frame& F, const Sel& sel, int buf) {
    int count = 0;
    if (sel.valid) {
      build_tables(F);
      wave_lds_sync();
      uint32_t thr = KEY_8, tie_key = KEY_INF;
      int need = 0;
      bool suspect = true;
      bool fast = false;
      // lists of 16: scan the E8_FAST2 candidates nearest to F first,
      // then the E8_FAST nearest; when the ks-th closest of a set is below
      // its bound none of the others can be among the closest ks
      uint32_t key3[NS_FAST];
      if constexpr (KS < NB) {
        uint32_t key2[NS_FAST2];
#pragma unroll
        for (int k = 0; k < NS_FAST2; ++k) key2[k] = key3[k] = __float_as_uint(cand_d2(S.qt, lo[k], hi[k], sel));
        count = threshold_k_hist<NS_FAST2>(key2, W.hist, lane, KS, thr, tie_key, need, suspect);
        fast = count == KS && !suspect && (tie_key != KEY_INF ? tie_key < KEY_FAST2 : thr <= KEY_FAST2);
        if (fast) {
          emit<NS_FAST2>(key2, thr, tie_key, need, sel, F, buf);
        } else {
#pragma unroll
          for (int k = NS_FAST2; k < NS_FAST; ++k) key3[k] = __float_as_uint(cand_d2(S.qt, lo[k], hi[k], sel));
          thr = KEY_8;
          tie_key = KEY_INF;
          need = 0;
          suspect = true;
          count = threshold_k_hist<NS_FAST>(key3, W.hist, lane, KS, thr, tie_key, need, suspect);
          fast = count == KS && !suspect && (tie_key != KEY_INF ? tie_key < KEY_FAST : thr <= KEY_FAST);
          if (fast) emit<NS_FAST>(key3, thr, tie_key, need, sel, F, buf);
        }
      }
      if (!fast) {
        uint32_t key[NS_STRICT];
#pragma unroll
        for (int k = 0; k < NS_STRICT; ++k) {
          if (KS < NB && k < NS_FAST) {
            key[k] = key3[k];
          } else {
            uint32_t l, h;
            const bool in = cand(k, l, h);
            key[k] = in ? __float_as_uint(cand_d2(S.qt, l, h, sel)) : KEY_INF;
          }
        }
        thr = KEY_8;
        tie_key = KEY_INF;
        need = 0;
        suspect = true;
        if constexpr (KS != KALL)
          count = threshold_k_hist<NS_STRICT>(key, W.hist, lane, KS, thr, tie_key, need, suspect);
        if (!suspect) {
          emit<NS_STRICT>(key, thr, tie_key, need, sel, F, buf);
        } else {
          // rare: rescan together with the points at distance exactly sqrt(8) from F
          uint32_t key7[NS_ALL];
#pragma unroll
          for (int k = 0; k < NS_STRICT; ++k) key7[k] = key[k];
#pragma unroll
          for (int k = NS_STRICT; k < NS_ALL; ++k) {
            uint32_t l, h;
            const bool in = cand(k, l, h);
            key7[k] = in ? __float_as_uint(cand_d2(S.qt, l, h, sel)) : KEY_INF;
          }
          if constexpr (KS == KALL) {
            // untruncated: every candidate whose recipe distance is below 8
            count = min(count_below(key7, KEY_8), KS);
            emit<NS_ALL>(key7, KEY_8, KEY_INF, 0, sel, F, buf);
          } else {
            bool suspect7;
            count = threshold_k<NS_ALL>(key7, KS, thr, tie_key, need, suspect7);
            emit<NS_ALL>(key7, thr, tie_key, need, sel, F, buf);
          }
        }
      }
      wave_lds_sync();
    }
    if constexpr (KS == NB) return count;
    // locations and weights, one neighbour per lane
#pragma unroll
    for (int r = 0; r < (KS + WAVE - 1) / WAVE; ++r) {
      const int e = lane + WAVE * r;
      if (e < KS) {
        Nbr& n = W.nbr[buf][e];
        if (e < count) {
          n.slot = cand_slot(S.st, n.lo, n.hi, sel);
          const float u = 1.0f - __uint_as_float(n.dbits) * 0.125f;
          const float u2 = u * u;
          W.wgt[buf][e] = (u2 * u2) * F.s;  // exact for plain lookups (s = 1)
        } else {
          n.lo = n.hi = wbyte * 0x01010101u;  // an entry of this wave's own tables (grad_query reads it, times zero)
          n.dbits = KEY_INF;
          n.slot = -1;
          W.wgt[buf][e] = 0.0f;
        }
      }
    }
    wave_lds_sync();
    return count;
  }

  // The list of lookup l saved by the forward (NbrList), in place of run():
  // the per-query tables are rebuilt from the frame (the coordinate errors for
  // dq) and each entry's recipe distance is recomputed from its code exactly
  // as run() formed it.  Entries whose slot lies outside [0, N) count as
  // padding, so no list content can address outside the value table.
  __device__ __forceinline__ int load(const Frame& F, const Sel& sel, int buf, const NbrList nl, int64_t l, uint32_t N) {
    static_assert(KS == NB, "saved lists hold the closest 32");
    const bool valid = sel.valid;
    if (valid) {
      build_tables(F);
      wave_lds_sync();
    }
    bool real = false;
    if (lane < KS) {
      const size_t o = (size_t)l * KS + lane;
      const int32_t s = valid ? nl.slot[o] : -1;
      real = s >= 0 && (uint32_t)s < N;
      Nbr& n = W.nbr[buf][lane];
      if (real) {
        uint32_t l8, h8;
        bytes_of(nl.code[o] & 0xFFFFFFu, wbyte, l8, h8);
        n.lo = l8;
        n.hi = h8;
        n.dbits = __float_as_uint(cand_d2(S.qt, l8, h8, sel));
        n.slot = s;
        W.wgt[buf][lane] = nl.w[o];
      } else {
        n.lo = n.hi = wbyte * 0x01010101u;  // (as in run)
        n.dbits = KEY_INF;
        n.slot = -1;
        W.wgt[buf][lane] = 0.0f;
      }
    }
    wave_lds_sync();
    return __popcll(__ballot(real));
  }

  // Writes list `buf` of lookup l to the saved lists (lanes 0..KS-1; nothing when !ok).
  __device__ __forceinline__ void save(int buf, int wb, const NbrList nl, int64_t l, bool ok) const {
    static_assert(KS == NB, "saved lists hold the closest 32");
    if (lane < KS && ok) {
      const size_t o = (size_t)l * KS + lane;
      const Nbr n = W.nbr[buf][lane];
      nl.slot[o] = n.slot;
      nl.w[o] = W.wgt[wb][lane];
      nl.code[o] = n.slot >= 0 ? code_of(n.lo, n.hi) : 0u;
    }
  }
};

// ---------------------------------------------------------------------------
// The tile search: the closest 32 of 16 lookups by one wave.
//
// With a whole wave to a lookup the search was bound by VALU issue: 228
// instructions per lookup, most of them the distances of 128 to 192 candidates
// (v_perm, LDS read and add for every coordinate) and the selection's
// histogram and bisection.  Only 77 of the 232 candidates are ever among the 32
// closest of a random query, and ten always are, so the selection is a choice
// of 22 out of 64, and it does not need the recipe's distances:
//   1. distances of the candidates to the 16 queries in F come from the matrix
//      cores, |p|^2/4 - z.p/2 (quarter units, |z|^2/4 left out): a lane holds 16
//      of its lookup's 64 candidates in registers.  The points' coordinates are
//      exact in bf16 and z is the sum of three bf16 numbers (8 bits of its
//      mantissa each), so one v_mfma_f32_16x16x32_bf16 forms 16 x 16 distances
//      with exact products and fp32 sums (the third of its depth times zero is
//      idle); two v_mfma_f32_16x16x4_f32 took four times its cycles and
//      2,150 clocks of a tile's latency;
//   2. a threshold with 22 of the 64 below it is found by interpolation on the
//      count (about four rounds, all 16 lookups at once, no LDS);
//   3. the choice is accepted if no candidate -- of the 64, of the ten (all
//      below) or of the remaining 158 (all above) -- lies within TILE_EPS of
//      the threshold and the threshold is clear of the support's edge: the
//      recipe's order of the two sides is then the same.  In quarter units: a
//      distance is 24 additions of sums below 8, each within one unit of
//      2^-21 whether the matrix cores round to nearest or truncate (1.15e-5
//      together; 1e-6 observed), z moves it by 2.4e-7 and the recipe's own
//      rounding by 7.8e-7: 1.25e-5 in all.  Otherwise the lookup
//      takes the general search (about 1 in 700 random queries, and queries
//      next to a lattice point or hole);
//   4. the recipe's distances, locations and weights of the chosen 32 alone are
//      formed two lookups at a time, one neighbour to a lane.
// About 75 VALU instructions per lookup.  Measured before and after: lists of
// 100,003 lookups 173 -> 65 us; flags of 262,144 lookups 132 -> 59 us; forward of
// 262,144 lookups (2^18 rows, m = 64 fp32) 328 -> 249 us, of 131,072 (m = 64 bf16)
// 114 -> 69 us, of 4,194,304 (1e8 rows, m = 32 bf16, ordered) 2,538 -> 2,039 us.
// The rows of the product: blocks 0-3 the 64, block 4 the ten (rows 0-9) and
// six others, blocks 5-14 the others.

constexpr int TILE_PICK = NB - TILE_ALWAYS;
constexpr float TILE_EPS = 1.5e-5f;  // quarter units: 6e-5 in distance^2
constexpr float TILE_STEP = 2e-5f;   // a threshold placed next to a candidate keeps this far from it
constexpr float TILE_EDGE = 7.999f;  // as KEY_SUSPECT
constexpr int TILE_ROUNDS = 7;

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

struct TileOps {
  uint32_t rows[E8_TILE_BLOCKS * TILE][4];  // F coordinates of the rows' points, eight bf16
  float c[2][16];                           // |p|^2 / 4 of the rows of blocks 3 and 4 (mixed norms)
  uint32_t cand[CANDS + 1][2];       // packed bytes 4 (p_r - CMIN)
};

constexpr TileOps make_tile_ops() {
  constexpr int rows[E8_TILE_BLOCKS][16] = E8_TILE_INIT;
  constexpr signed char pts[E8_NSTRICT][8] = E8_STRICT_INIT;
  constexpr signed char edge[E8_NBOUNDARY][8] = E8_BOUNDARY_INIT;
  TileOps o{};
  auto pack = [&o](int at, const signed char* p) {
    for (int r = 0; r < 8; ++r) o.cand[at][r / 4] |= (uint32_t)(4 * (p[r] - E8_CAND_MIN)) << (8 * (r % 4));
  };
  bool placed[E8_NSTRICT] = {};
  for (int b = 0; b < E8_TILE_BLOCKS; ++b)
    for (int m = 0; m < 16; ++m) {
      const signed char* p = pts[rows[b][m]];
      float n2 = 0.0f;
      for (int r = 0; r < 8; ++r) {
        // |p_r| <= 4: exact in the upper half of its fp32 bits
        o.rows[16 * b + m][r / 2] |= (__builtin_bit_cast(uint32_t, (float)p[r]) >> 16) << (16 * (r % 2));
        n2 += (float)(p[r] * p[r]);
      }
      if (b == 3 || b == 4) o.c[b - 3][m] = 0.25f * n2;
      // lane group m / 4 shifts its 16 candidates' signs into a word, block by
      // block: candidate (b, m) ends at bit 15 - (4 b + m % 4)
      if (b < 4) pack((m / 4) * 16 + 15 - (4 * b + m % 4), p);
      if (b == 4 && m < TILE_ALWAYS) pack(TILE_VAR + m, p);
      if (b < 4 || (b == 4 && m < TILE_ALWAYS)) placed[rows[b][m]] = true;
    }
  int at = TILE_VAR + TILE_ALWAYS;
  for (int i = 0; i < E8_NSTRICT; ++i)
    if (!placed[i]) pack(at++, pts[i]);
  for (int i = 0; i < E8_NBOUNDARY; ++i) pack(E8_NSTRICT + i, edge[i]);
  return o;
}
constexpr bool tile_norms_ok() {
  constexpr int rows[E8_TILE_BLOCKS][16] = E8_TILE_INIT;
  constexpr signed char pts[E8_NSTRICT][8] = E8_STRICT_INIT;
  bool seen[E8_NSTRICT] = {};
  for (int b = 0; b < E8_TILE_BLOCKS; ++b)
    for (int m = 0; m < 16; ++m) {
      int n2 = 0;
      for (int r = 0; r < 8; ++r) n2 += pts[rows[b][m]][r] * pts[rows[b][m]][r];
      seen[rows[b][m]] = true;
      if (b != 3 && b != 4 && n2 != (b < 10 ? 8 : 16)) return false;
    }
  for (int i = 0; i < E8_NSTRICT; ++i)
    if (!seen[i]) return false;
  return true;
}
static_assert(E8_TILE_BLOCKS == 15 && tile_norms_ok(), "blocks of one norm but for 3 and 4, every candidate in a row");
__constant__ __align__(16) TileOps c_tile = make_tile_ops();

// Copies the product's operands (rows: tiles are searched) and the candidates to
// LDS; every thread of the workgroup, before the first search.  (Read from memory by every tile, the
// operands cost small batches three dependent loads' latency.)
template <typename SL>
__device__ __forceinline__ void init_tile(SL& S, bool rows) {
  auto copy = [](const uint32_t* from, uint32_t* to, int words) {
    const uint4* src = reinterpret_cast<const uint4*>(from);
    uint4* dst = reinterpret_cast<uint4*>(to);
    for (int i = threadIdx.x; i < words / 4; i += THREADS) dst[i] = src[i];
  };
  static_assert((CANDS + 1) % 2 == 0 && sizeof(S.tile.cand) == sizeof(c_tile.cand), "candidates in 16-byte pieces");
  if (rows) copy(&c_tile.rows[0][0], &S.tile.rows[0].x, E8_TILE_BLOCKS * TILE * 4);
  copy(&c_tile.cand[0][0], &S.tile.cand[0].x, 2 * (CANDS + 1));
  __syncthreads();
}

// f over the four lanes of a lookup (lane % 16 = lookup).
template <typename F>
__device__ __forceinline__ uint32_t over_groups(uint32_t x, F f) {
  const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = f(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return f(b[0], b[1]);
}

// Steps 1 to 3 for the frames of a tile: writes every accepted lookup's
// candidate indices to idx and returns the accepted lookups' bits.
__device__ __forceinline__ uint32_t tile_select(const Frame* fr, const TileLds<true>& tile, uint16_t (*idx)[NB], int lane) {
  // (opaque: what follows from the lane is formed again for every tile; held
  // for the whole wave it costs the row loads their registers)
  const int ln = opaque(lane), n = ln & 15, g = ln >> 4;
  const Frame& F = fr[n];
  const float r2 = F.r2;
  // the matrix's B operand: lane group g holds the g-th 8 bits of -z_r / 2
  bf16x8_t z;
  {
    const uint4 lo = reinterpret_cast<const uint4*>(F.sel)[0], hi = reinterpret_cast<const uint4*>(F.sel)[1];
    const uint32_t in[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const uint32_t m1 = g >= 1 ? 0xFFFF0000u : 0u, m2 = g >= 2 ? 0xFFFF0000u : 0u, some = g < 3 ? ~0u : 0u;
    uint32_t x[8], w[4];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float y = __uint_as_float(in[r]);
      y -= __uint_as_float(__float_as_uint(y) & m1);  // exact: the leading bits
      y -= __uint_as_float(__float_as_uint(y) & m2);
      x[r] = __float_as_uint(y);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = __builtin_amdgcn_perm(x[2 * r + 1], x[2 * r], 0x07060302u) & some;
    z = __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
  }
  auto product = [&](int b, f32x4_t c) {
    const bf16x8_t p = __builtin_bit_cast(bf16x8_t, tile.rows[16 * b + n]);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(p, z, c, 0, 0, 0);
  };
  f32x4_t mixed[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) mixed[k] = *reinterpret_cast<const f32x4_t*>(&c_tile.c[k][4 * (ln >> 4)]);
  float v[16];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const f32x4_t d = product(b, b < 3 ? f32x4_t{2.0f, 2.0f, 2.0f, 2.0f} : mixed[0]);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[4 * b + i] = d[i];
  }
  const f32x4_t va = product(4, mixed[1]);
  // the others: blocks 5-9 of norm 8, 10-14 of norm 16 (five at a time: all ten
  // would hold 60 registers)
  float rest = 1e30f;
#pragma unroll 1
  for (int b0 = 5; b0 < E8_TILE_BLOCKS; b0 += 5) {
    float least = 1e30f;
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const f32x4_t d = product(b0 + b, f32x4_t{0.0f, 0.0f, 0.0f, 0.0f});
      least = fminf(least, fminf(fminf(d[0], d[1]), fminf(d[2], d[3])));
    }
    rest = fminf(rest, least + (b0 == 5 ? 2.0f : 4.0f));
  }
  // start: least-squares fit of the threshold over uniform queries
  float T = 1.59608f - 0.214989f * r2;
  float lo = 0.0f, hi = 0.0f;
  int clo = -1, chi = -1;
  uint32_t mask = 0, up = 0, dn = 0;
  int cnt = 0, mine = 0;
#pragma unroll 1
  for (int it = 0; it < TILE_ROUNDS; ++it) {
    mask = 0;
    up = 0xFFFFFFFFu;
    dn = 0x7FFFFFFFu;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint32_t t = __float_as_uint(v[j] - T);
      mask = __builtin_amdgcn_alignbit(mask, t, 31);       // sign bits, the first candidate's highest
      up = min(up, t);                                      // smallest non-negative difference
      dn = (uint32_t)min((int)dn, (int)t);                  // negative difference of smallest magnitude
    }
    // magnitudes as bits (which order like them), infinite where the lane has none on that side
    up = min(up, KEY_INF);
    dn = min(dn ^ 0x80000000u, KEY_INF);
    mine = __popc(mask);
    cnt = (int)over_groups((uint32_t)mine, [](uint32_t a, uint32_t b) { return a + b; });
    const int miss = F.valid ? TILE_PICK - cnt : 0;
    if (__ballot(miss != 0) == 0) break;
    const bool less = miss > 0;
    // distance to the next candidate on the side that is short
    const float gap = __uint_as_float(over_groups(less ? up : dn, [](uint32_t a, uint32_t b) { return min(a, b); }));
    if (miss != 0) {
      if (less) {
        lo = T;
        clo = cnt;
      } else {
        hi = T;
        chi = cnt;
      }
      // past the next candidate, which is right when one is missing (or too many)
      const float step = less ? T + gap + TILE_STEP : T - gap - TILE_STEP;
      const bool both = clo >= 0 && chi >= 0;
      float x = both ? lo + (hi - lo) * (float)(TILE_PICK - clo) * __builtin_amdgcn_rcpf((float)(chi - clo))
                     : T + 0.0091f * (float)miss;
      x = less ? fmaxf(x, step) : fminf(x, step);
      T = abs(miss) <= 2 ? step : x;
    }
  }
  // accepted: 22 of the 64, all ten and none of the others below, none near, clear of the edge
  uint32_t below = 0;
  float near = __uint_as_float(min(up, dn));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float t = va[i] - T;
    below |= (__float_as_uint(t) >> 31) << i;
    near = fminf(near, fabsf(t));
  }
  const uint32_t want = g < 2 ? 15u : (g == 2 ? 3u : 0u);
  bool ok = cnt == TILE_PICK && below == want && near >= TILE_EPS && rest - T >= TILE_EPS &&
            4.0f * T + r2 < TILE_EDGE && F.valid != 0u;
  uint64_t m = __ballot(ok);
  m &= m >> 32;
  m &= m >> 16;
  const uint32_t accepted = (uint32_t)m & 0xFFFFu;
  // list the selected candidates behind the ten: the lane's bits follow those
  // of the lookup's lower lanes
  const auto row = __builtin_amdgcn_permlane16_swap((uint32_t)mine, (uint32_t)mine, false, false);
  const uint32_t rows2 = row[0] + row[1];
  const auto half = __builtin_amdgcn_permlane32_swap(rows2, rows2, false, false);
  uint32_t pos = TILE_ALWAYS + ((g & 1) ? row[0] : 0u) + ((g & 2) ? half[0] : 0u);
  if (!((accepted >> n) & 1u)) mask = 0;
  uint16_t* dst = idx[n] + pos;
  while (mask) {
    *dst++ = (uint16_t)(16 * g + __builtin_ctz(mask));
    mask &= mask - 1;
  }
  return accepted;
}

// Everything the kernels need of the search of the closest 32: a tile's
// frames and selection, then pairs of its lookups.  SELECT = false: the frames
// only, for saved lists; without the tile's LDS four workgroups of the merged
// scatter share a CU at m = 32 (see FusedLds).
template <int TH, int WBUF, bool SELECT = true>
struct TileSearch {
  static constexpr int NBUF = SELECT ? 2 : 1;
  using SL = SearchLds<NB, NBUF, WBUF, SELECT>;
  SL& S;
  WaveLds<NB, NBUF, WBUF>& W;
  Search<NB, NBUF, WBUF, SELECT> one;
  QuadCtx<TH> Q;
  Frame* FR;
  int wave, lane;
  uint32_t accepted;  // bits of the tile's lookups whose list starts with the ten
  uint32_t exist;     // bits of its lookups
  bool tiled;         // otherwise the general search takes every lookup

  // every thread of the workgroup constructs it (a barrier if SELECT), before any leaves
  __device__ TileSearch(const Params P, SL& s, int w, int l)
      : S(s), W(s.wave[w]), one(P, s.tab, s.wave[w], s.tile, w, l), Q(P, l), FR(s.frames[w]), wave(w), lane(l),
        accepted(0), exist(0), tiled(P.tiled != 0) {
    if constexpr (SELECT) init_tile(s, tiled);
  }

  // The lookup of this lane's quarter: position + lane / 4.
  __device__ __forceinline__ int quad() const { return Q.n; }

  // Frames of the tile whose quarters are in (nt lookups of it exist), and with
  // SELECT its candidates.
  __device__ __forceinline__ void frames(const QuadIn<TH>& in, bool have, int nt) {
    const uint2 sel = make_frames<TH>(in, have, Q, FR);
    wave_lds_sync();
    if constexpr (SELECT) {
      if (tiled) accepted = uniform(tile_select(FR, S.tile, S.tile.idx[wave], lane));
      wave_lds_sync();
    }
    finish_frames(sel, lane, FR);
    wave_lds_sync();
    if constexpr (SELECT) {
      exist = 0xFFFFu >> (TILE - nt);
      // the others: empty lists (a non-finite query) or the general search
      uint32_t left = exist & ~accepted;
#pragma unroll 1
      while (left) {
        const int t = __builtin_ctz(left);
        left &= left - 1;
        if (lane < NB) S.tile.idx[wave][t][lane] = (uint16_t)CAND_NONE;
        wave_lds_sync();
        const Sel s = read_sel(FR[t]);
        one.lane = opaque(one.lane);  // (as in tile_select)
        if (s.valid) one.run(FR[t], s, t);
      }
      wave_lds_sync();
    }
  }

  int count0, count1;  // lengths of the pair's lists

  // Lists of the lookups 2p and 2p + 1 of the tile: W.nbr[0], W.nbr[1] and the
  // weights W.wgt[wb], W.wgt[wb + 1], padded with location -1 and weight 0.
  __device__ __forceinline__ void pair(int p, int wb) {
    const int h = lane >> 5, j = lane & 31, t = 2 * p + h;
    one.build_tables(FR[2 * p], 0);
    one.build_tables(FR[2 * p + 1], 1);
    wave_lds_sync();
    const Frame& F = FR[t];
    const uint32_t off = (one.wbyte + 32u * (uint32_t)h) * 0x01010101u;
    uint32_t id = S.tile.idx[wave][t][j];
    if (j < TILE_ALWAYS && ((accepted >> t) & 1u)) id = TILE_VAR + j;
    const bool real = id != CAND_NONE && ((exist >> t) & 1u);
    const uint2 cd = S.tile.cand[real ? id : 0u];
    Nbr o;
    o.lo = cd.x + off;
    o.hi = cd.y + off;
    const uint4 s0 = reinterpret_cast<const uint4*>(F.sel)[0], s1 = reinterpret_cast<const uint4*>(F.sel)[1];
    const uint32_t sel[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    float d = 0.0f;
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = __builtin_amdgcn_perm(o.hi, o.lo, sel[i]) + 256u * i;
      const float e2 = lds_f32(one.S.qt, a);
      d = i == 0 ? e2 : d + e2;
      m += lds_u32(one.S.st, a);
    }
    const float u = 1.0f - d * 0.125f;
    const float u2 = u * u;
    o.dbits = real ? __float_as_uint(d) : KEY_INF;
    o.slot = real ? (int32_t)(m >> 1) : -1;
    W.nbr[h][j] = o;
    W.wgt[wb + h][j] = real ? (u2 * u2) * F.s : 0.0f;  // exact for plain lookups (s = 1)
    const uint64_t r = __ballot(real);
    count0 = __popc((uint32_t)r);
    count1 = __popc((uint32_t)(r >> 32));
    wave_lds_sync();
  }
};

// Input floats per lookup.
template <int TH>
__device__ __forceinline__ int in_stride(const Params& P) {
  return TH == IN_STAGED ? P.stage : (TH == IN_THETA ? 16 : 8);
}

// The input of this lane's quarter of the tile at [base, base + nl) of the
// lookups, or of the positions of the order perm (l: the quarter's lookup; an
// index outside [0, L) -- an order not written for these lookups -- gets an
// empty list, and the kernels write nothing for it).  Returns whether the
// lookup exists.
template <int TH, bool ORD>
__device__ __forceinline__ bool load_tile(const float* in, const uint32_t* __restrict__ perm, int64_t base,
                                          int nl, const Params& P, int lane, QuadIn<TH>& v, uint32_t& l) {
  const int n = lane >> 2;
  bool have = n < nl;
  const int64_t at = base + (have ? n : 0);
  l = 0;
  size_t src = (size_t)at;
  if constexpr (ORD) {
    l = perm[at];
    if ((int64_t)l >= P.L) have = false;
    src = have ? l : 0;
    if (n >= nl) l = 0xFFFFFFFFu;
  }
  v = load_quad<TH>(in, src, lane & 3, P.stage);
  return have;
}

// The tiles of a wave's lookups [base, base + nl): each tile's input is loaded
// one tile ahead, the first before the workgroup's barrier.
template <int TH, bool ORD>
struct TileInput {
  const float* in;
  const uint32_t* perm;
  int64_t base;
  int nl, lane;
  QuadIn<TH> v;
  uint32_t l, next_l;  // this lane's quarter's lookup of the current and of the next tile (ORD)
  bool have;
  __device__ TileInput(const float* i, const uint32_t* __restrict__ pm, int64_t b, int n, const Params& P,
                       int ln)
      : in(i), perm(pm), base(b), nl(n), lane(ln), l(0), next_l(0), have(false) {
    if (nl > 0) have = load_tile<TH, ORD>(in, perm, base, min(TILE, nl), P, lane, v, next_l);
  }
  // After the tile at t0 has consumed v: the next one's input.
  __device__ __forceinline__ void advance(int t0, const Params& P) {
    l = next_l;
    if (t0 + TILE < nl)
      have = load_tile<TH, ORD>(in, perm, base + t0 + TILE, min(TILE, nl - t0 - TILE), P, lane, v, next_l);
  }
  // The lookup at position t of the tile at t0, and whether anything is written for it.
  __device__ __forceinline__ int64_t lookup(int t0, int t, const Params& P, bool& ok) const {
    const int64_t at = ORD ? (int64_t)(uint32_t)__builtin_amdgcn_readlane(l, 4 * t) : base + t0 + t;
    ok = t0 + t < nl && (!ORD || at < P.L);
    return ok ? at : 0;
  }
};

// Frames of a tile for the general search (lists other than the closest 32).
__device__ __forceinline__ void tile_frames(const float* __restrict__ q, int64_t base, int nl, const Params& P, Frame* fr,
                                            const QuadCtx<IN_QUERY>& Q, int lane) {
  QuadIn<IN_QUERY> v;
  uint32_t l;
  const bool have = load_tile<IN_QUERY, false>(q, nullptr, base, nl, P, lane, v, l);
  const uint2 sel = make_frames<IN_QUERY>(v, have, Q, fr);
  wave_lds_sync();
  finish_frames(sel, lane, fr);
  wave_lds_sync();
}

}  // namespace
