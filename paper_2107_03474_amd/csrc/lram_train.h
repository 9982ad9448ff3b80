// lram_train.h -- part of liblram (included by lram.hip only).
//
// Training-side companions: access statistics and the Adam step on touched
// rows.

#pragma once

namespace {

// ---------------------------------------------------------------------------
// Access statistics (utilisation table): hist[s] += sum of the kernel weights
// of the pairs that read location s; then the fraction of locations read and
// the KL divergence of the weighted access distribution from uniform.

// A workgroup merges its lookups' pairs first: the lanes keep the (location, w)
// pairs of a tile per wave in registers, a 4,096-entry open-addressing hash in the
// search's LDS sums the weights of every distinct location, and each sum is
// added with one atomic.  Bound by the memory side's atomic requests of 64
// bytes, and by those that follow each other on one line.  Queries that share
// nothing gain nothing from it and wait for the merge (a CU's workgroups search
// and add in step), so small batches add pair by pair, and a wave takes half a
// tile until the grid holds several workgroups per CU.  us, pair by pair /
// merged with 4 / 8 / 16 lookups per wave; 8^8 rows uniform, 2^18 rows 64 clusters,
// 2^15 rows projected:
//    16,384 lookups  28 / 31 / 33 / -    40 / 41 / 42 / -    41 / 37 / 34 / -
//    32,768          50 / 58 / 55 / 62   77 / 76 / 72 / 74   79 / 71 / 60 / 54
//    65,536          94 / 103 / 104 / 108  133 / 133 / 125 / 122  150 / 134 / 109 / 93
//   131,072         185 / 196 / 188 / 199  265 / 267 / 249 / 234  294 / 255 / 212 / 172
//   262,144         361 / 379 / 378 / 379  481 / 481 / 457 / 414  588 / 507 / 418 / 330
// With the pairs in LDS (50,080 bytes, three workgroups per CU) instead of in
// registers (33,792, four): 62, 114, 203, 391 for the uniform queries and 54, 103, 172,
// 330 for the projected ones from 32,768 on.  Hot locations also receive fewer,
// larger terms, so their fp32 sums are rounded less often.
union alignas(16) HistLds {
  SearchLds<NB, 2> search;
  struct {
    int32_t tag[MERGE_H];
    float sum[MERGE_H];
  } hash;
};

// First hash entry of a location: the 16 locations of a 64-byte line of the
// histogram take 16 consecutive entries, so those a batch reads leave in one
// instruction, as one request.
__device__ __forceinline__ uint32_t hist_entry(uint32_t l) {
  return ((((l >> 4) * 0x9E3779B1u) >> (32 - (MERGE_HBITS - 4))) << 4) | (l & 15);
}

// MERGE: one tile to a wave at most, its pairs merged; otherwise pair by pair.
template <bool MERGE>
__global__ void __launch_bounds__(THREADS, 4) k_access_hist(const float* __restrict__ q, Params P,
                                                            float* __restrict__ hist) {
  __shared__ std::conditional_t<MERGE, HistLds, SearchLds<NB, 2>> S;
  WaveCtx c;
  wave_ctx(P, c);
  const int h = c.lane >> 5, j = c.lane & 31;
  TileInput<IN_QUERY, false> in(q, nullptr, c.base, c.nl, P, c.lane);
  if constexpr (!MERGE) {
    TileSearch<IN_QUERY, 2> ts(P, S, c.wave, c.lane);
    for (int t0 = 0; t0 < c.nl; t0 += TILE) {
      const int nt = min(TILE, c.nl - t0);
      ts.frames(in.v, in.have, nt);
      in.advance(t0, P);
      for (int p = 0; 2 * p < nt; ++p) {
        ts.pair(p, 0);
        const int32_t s = ts.W.nbr[h][j].slot;
        if (s >= 0) unsafeAtomicAdd(hist + s, ts.W.wgt[h][j]);
        wave_lds_sync();
      }
    }
  } else {
    constexpr int NP = TILE / 2;  // pairs of lookups per tile, one entry of each to a lane
    int32_t loc[NP];
    float w[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      loc[k] = -1;
      w[k] = 0.0f;
    }
    TileSearch<IN_QUERY, 2> ts(P, S.search, c.wave, c.lane);
    if (c.nl > 0) ts.frames(in.v, in.have, c.nl);
#pragma unroll 1
    for (int p = 0; 2 * p < c.nl; ++p) {
      ts.pair(p, 0);
      const int32_t s = ts.W.nbr[h][j].slot;
      const float wt = ts.W.wgt[h][j];
#pragma unroll
      for (int k = 0; k < NP; ++k) {  // (selected: a runtime index would put the arrays into memory)
        loc[k] = k == p ? s : loc[k];
        w[k] = k == p ? wt : w[k];
      }
      wave_lds_sync();
    }
    __syncthreads();  // the search's LDS becomes the hash
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < MERGE_HPT; ++k) {
      S.hash.tag[k * THREADS + t] = MERGE_EMPTY;
      S.hash.sum[k * THREADS + t] = 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int32_t l = loc[k];
      if (l >= 0) {
        uint32_t e = hist_entry((uint32_t)l);
        while (true) {
          const int32_t old = atomicCAS(&S.hash.tag[e], MERGE_EMPTY, l);
          if (old == MERGE_EMPTY || old == l) break;
          e = (e + 1) & (MERGE_H - 1);
        }
        unsafeAtomicAdd(&S.hash.sum[e], w[k]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < MERGE_HPT; ++k) {
      const int32_t l = S.hash.tag[k * THREADS + t];
      if (l >= 0) unsafeAtomicAdd(hist + l, S.hash.sum[k * THREADS + t]);
    }
  }
}
static_assert(WAVES * TILE * NB < MERGE_H, "a workgroup's pairs leave empty entries");

// touched[s] = 1 for every location s in a lookup's list of its closest 32
// (the rows a backward of these lookups writes): plain byte stores, every
// writer stores the same value.
__global__ void __launch_bounds__(THREADS, 4) k_mark_touched(const float* __restrict__ q, Params P,
                                                          uint8_t* __restrict__ touched) {
  __shared__ SearchLds<> S;
  WaveCtx c;
  wave_ctx(P, c);
  TileInput<IN_QUERY, false> in(q, nullptr, c.base, c.nl, P, c.lane);
  TileSearch<IN_QUERY, 2> ts(P, S, c.wave, c.lane);
  for (int t0 = 0; t0 < c.nl; t0 += TILE) {
    const int nt = min(TILE, c.nl - t0);
    ts.frames(in.v, in.have, nt);
    in.advance(t0, P);
    for (int p = 0; 2 * p < nt; ++p) {
      ts.pair(p, 0);
      const int h = c.lane >> 5, j = c.lane & 31;
      const int32_t s = ts.W.nbr[h][j].slot;
      if (s >= 0) touched[s] = 1;
      wave_lds_sync();
    }
  }
}

__global__ void k_fill_f64(double* __restrict__ p, int n, double v) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = v;
}

__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
  for (int mask = 1; mask < WAVE; mask <<= 1) x += __shfl_xor(x, mask);
  return x;
}

// acc = {workgroups done, sum h log h, sum h, #{h > 0}}, cleared; the last
// workgroup to finish turns it into out = {used fraction, KL(p || uniform) =
// log N + (sum h log h)/H - log H, H, count}.
// Bound by the fp64 logarithms once the partial sums stay out of memory: one
// atomic instruction per workgroup (three lanes, one 64-byte request) on at
// most STATS_BLOCKS workgroups.  Atomics on one address follow each other at
// about 35 ns, so a wave-by-wave accumulation from 4,096 workgroups (49,152
// atomics) took 593 us for 2^22 locations, this takes 25 us.
constexpr int STATS_THREADS = 1024;
constexpr int STATS_BLOCKS = 256;
__global__ void __launch_bounds__(STATS_THREADS) k_access_reduce(const float* __restrict__ hist, int64_t N,
                                                                 double* __restrict__ acc) {
  __shared__ double part[3][STATS_THREADS / WAVE];
  const int64_t n4 = (reinterpret_cast<uintptr_t>(hist) & 15) == 0 ? N / 4 : 0;  // 16-byte loads where aligned
  double hl = 0.0, hs = 0.0, hc = 0.0;
  auto add = [&](float v) {
    const double h = v;
    if (h > 0.0) {
      hl += h * log(h);
      hs += h;
      hc += 1.0;
    }
  };
  const int64_t first = (int64_t)blockIdx.x * STATS_THREADS + threadIdx.x, stride = (int64_t)gridDim.x * STATS_THREADS;
  for (int64_t i = first; i < n4; i += stride) {
    const float4 v = reinterpret_cast<const float4*>(hist)[i];
    add(v.x);
    add(v.y);
    add(v.z);
    add(v.w);
  }
  for (int64_t i = 4 * n4 + first; i < N; i += stride) add(hist[i]);
  hl = wave_sum_f64(hl);
  hs = wave_sum_f64(hs);
  hc = wave_sum_f64(hc);
  const int t = threadIdx.x;
  if (t % WAVE == 0) {
    part[0][t / WAVE] = hl;
    part[1][t / WAVE] = hs;
    part[2][t / WAVE] = hc;
  }
  __syncthreads();
  if (t < 3) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < STATS_THREADS / WAVE; ++w) s += part[t][w];
    unsafeAtomicAdd(acc + 1 + t, s);
    __threadfence();
  }
  __syncthreads();
  if (t == 0) {
    __threadfence();
    const double done = unsafeAtomicAdd(acc, 1.0);
    if (done == (double)(gridDim.x - 1)) {
      __threadfence();
      const double l = __hip_atomic_load(acc + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double H = __hip_atomic_load(acc + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double c = __hip_atomic_load(acc + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      acc[0] = c / (double)N;
      acc[1] = H > 0.0 ? log((double)N) + l / H - log(H) : 0.0;
    }
  }
}

// ---------------------------------------------------------------------------
// Adam step (Sec. 3.2: Adam on the memory parameters) on the rows of the table
// whose accumulated gradient row is not identically zero; the other rows keep
// value and moments.  M lanes per row (lane = column); the gradient row is
// cleared after use so the buffer is ready for the next accumulation.
struct AdamArgs {
  float lr, beta1, beta2, eps, om1, om2, bc1, bc2;  // om = 1 - beta, bc = 1 - beta^step (formed in fp64)
};

// One row's Adam update (M lanes, lane = column) when its gradient row is not
// identically zero; the gradient row is then cleared.  seg: this lane's row's
// lanes in a wave-wide ballot (every lane of the wave takes part).
template <int DT, int M>
__device__ __forceinline__ void adam_row(void* __restrict__ table, float* __restrict__ grad, float* __restrict__ m1,
                                         float* __restrict__ m2, const AdamArgs& a, int64_t r, bool in, int col,
                                         uint64_t seg) {
  const size_t o = (size_t)(in ? r : 0) * M + col;
  const float g = in ? grad[o] : 0.0f;
  const bool nonzero = (__ballot(g != 0.0f) & seg) != 0;
  if (in && nonzero) {
    const float n1 = a.beta1 * m1[o] + a.om1 * g;
    const float n2 = a.beta2 * m2[o] + a.om2 * (g * g);
    m1[o] = n1;
    m2[o] = n2;
    const float step = a.lr * (n1 / a.bc1) / (sqrtf(n2 / a.bc2) + a.eps);
    if constexpr (DT == LRAM_F32) {
      float* t = reinterpret_cast<float*>(table) + o;
      *t = *t - step;
    } else {
      __bf16* t = reinterpret_cast<__bf16*>(table) + o;
      *t = (__bf16)((float)*t - step);
    }
    grad[o] = 0.0f;
  }
}

template <int M>
constexpr uint64_t row_lanes() { return M == WAVE ? ~0ull : (1ull << (M % WAVE)) - 1ull; }

template <int DT, int M>
__global__ void __launch_bounds__(THREADS) k_sparse_adam(void* __restrict__ table, int64_t N,
                                                         float* __restrict__ grad, float* __restrict__ m1,
                                                         float* __restrict__ m2, AdamArgs a) {
  constexpr int RW = WAVE / M;  // rows per wave
  const int lane = threadIdx.x % WAVE;
  const int col = lane % M, sub = lane / M;
  const uint64_t seg = row_lanes<M>() << (M * sub);
  const int64_t waves = (int64_t)gridDim.x * WAVES;
  for (int64_t rb = ((int64_t)blockIdx.x * WAVES + threadIdx.x / WAVE) * RW; rb < N; rb += waves * RW) {
    const int64_t r = rb + sub;
    adam_row<DT, M>(table, grad, m1, m2, a, r, r < N, col, seg);
  }
}

// The same step on the rows whose flag in touched [N] is set (by
// k_mark_touched for the step's lookups): a wave reads 64 flags at once and
// updates only the flagged rows (RW at a time), so the step reads N bytes of
// flags plus the flagged rows instead of the whole N x M gradient; flags are
// cleared.  A flagged row whose gradient is identically zero keeps value and
// moments, as in k_sparse_adam.
template <int DT, int M>
__global__ void __launch_bounds__(THREADS) k_sparse_adam_touched(void* __restrict__ table, int64_t N,
                                                                 float* __restrict__ grad, float* __restrict__ m1,
                                                                 float* __restrict__ m2, uint8_t* __restrict__ touched,
                                                                 AdamArgs a) {
  constexpr int RW = WAVE / M;
  const int lane = threadIdx.x % WAVE;
  const int col = lane % M, sub = lane / M;
  const uint64_t seg = row_lanes<M>() << (M * sub);
  const int64_t waves = (int64_t)gridDim.x * WAVES;
  for (int64_t base = ((int64_t)blockIdx.x * WAVES + threadIdx.x / WAVE) * WAVE; base < N; base += waves * WAVE) {
    const bool flag = base + lane < N && touched[base + lane] != 0;
    uint64_t mask = __ballot(flag);
    if (flag) touched[base + lane] = 0;
    while (mask) {
      // the wave's next RW flagged rows, one per group of M lanes
      int pick = -1;
#pragma unroll
      for (int k = 0; k < RW; ++k) {
        const int b = mask ? (int)__builtin_ctzll(mask) : -1;
        mask &= mask - 1;
        pick = k == sub ? b : pick;
      }
      adam_row<DT, M>(table, grad, m1, m2, a, base + pick, pick >= 0, col, seg);
    }
  }
}

}  // namespace
