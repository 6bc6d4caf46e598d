// Adjoint of the count in vertex-relative tables (rel.hip), one colouring at a
// time.  With Bbar the derivative by an aggregation B = A M, both in relative
// columns:
//   Mbar(j, Q) += sum over neighbours i of w_ij Bbar(i, Q + {c_j})
//   grad(i, j) += sum over Q of M(j, Q) Bbar(i, Q + {c_j})
// over sets Q + {c_j} without i's colour.  Row j's gather of its neighbours'
// Bbar rows gives both, the second for the reverse entries (i, j) of its own
// entries (j, i).
#include <algorithm>

#include "kernels.h"
#include "launch.h"
#include "rel.h"

namespace sg2v {

// Reverse entry of every entry: a binary search in the (sorted) row of its
// neighbour.  A lane takes an entry, whose row it searches first.
__global__ void __launch_bounds__(BLOCK) k_rel_rev(RelRevArgs a) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t wave = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) / WAVE;
  const int64_t nwaves = (int64_t)gridDim.x * WAVES_PER_BLOCK;
  for (int64_t e0 = wave * WAVE; e0 < a.nnz; e0 += nwaves * WAVE) {
    const int64_t e = e0 + lane;
    if (e >= a.nnz) continue;
    // row of the entry
    int64_t lo = 0, hi = a.n;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (a.row_ptr[mid] <= e) lo = mid;
      else hi = mid;
    }
    const int64_t i = lo;
    const int32_t j = a.col_idx[e];
    lo = a.row_ptr[j];
    hi = a.row_ptr[j + 1];
    const int64_t end = hi;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (a.col_idx[mid] < i) lo = mid + 1;
      else hi = mid;
    }
    const bool ok = lo < end && a.col_idx[lo] == i;
    a.rev[e] = ok ? (uint32_t)lo : (uint32_t)e;
    if (!ok) atomicOr(a.bad, 1);
  }
}
// a repeated entry's reverse is found once: then some reverse's reverse differs
__global__ void __launch_bounds__(BLOCK) k_rel_rev_check(RelRevArgs a) {
  for (int64_t e = (int64_t)blockIdx.x * BLOCK + threadIdx.x; e < a.nnz; e += (int64_t)gridDim.x * BLOCK)
    if (a.rev[a.rev[e]] != (uint32_t)e) atomicOr(a.bad, 1);
}

// The gather of k_rel_spmm (stage in LDS, lane p owns column p of row j), with a
// dot product per entry: four entries' products are reduced together, each
// step halving the values as it halves the lanes.
template <typename T, bool WEIGHTED, int NP>
__global__ void __launch_bounds__(BLOCK) k_rel_back(RelBackArgs a) {
  constexpr int N = V16<T>::N;
  constexpr int UNR = 4, UA = 4;
  constexpr bool SC = sizeof(T) == 4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int CW = a.cw, SR = a.sr;
  uint16_t *lmap = (uint16_t *)smem;
  uint16_t *lout = lmap + a.k * CW;
  T *stg0 = (T *)(smem + ((a.k * (CW + a.wout4) * 2 + 15) & ~15));
  const int streams = a.streams, E = UNR * streams;
  T *stg = stg0 + (size_t)wv * E * SR;
  for (int q = threadIdx.x; q < a.k * CW / 2; q += BLOCK) ((unsigned *)lmap)[q] = ((const unsigned *)a.map)[q];
  for (int q = threadIdx.x; q < a.k * a.wout4 / 2; q += BLOCK) ((unsigned *)lout)[q] = ((const unsigned *)a.olist)[q];
  for (int q = lane; q < E; q += WAVE) stg[q * SR + SR - 4] = T(0);
  __syncthreads();
  const uint8_t *col = a.col;
  const T *__restrict__ X = (const T *)a.X;
  const T *__restrict__ M = (const T *)a.M;
  T *O = (T *)a.O;
  T *Pt = (T *)a.partial;
  T fs = T(1), f = T(1), fm = T(1);  // factors of the staged rows, of their sums and of M
  RelAdd add{0, 1.f, 1.f};
  double scale = a.scale;
  if constexpr (SC) {
    (WEIGHTED ? fs : f) = rel_factor(a.mxx[0]);
    fm = rel_factor(a.mxm[0]);
    const int ec = rel_frame(a.ex[0], a.mxx[0]);
    scale = ldexp(scale, ec + rel_frame(a.em[0], a.mxm[0]));
    add.e = ec;
    if (a.accumulate) add = rel_accumulate(a.e_old[0], a.mx_old[0], ec, a.mxx[0] == 0u);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.e_out[0] = add.e;
  }
  const int stream = lane / a.lp, vec = lane - stream * a.lp;
  const bool act = stream < streams;
  float cmax = 0.f;
  T acc[NP], own[NP], nown[NP];
  int pabs[NP];
  bool pok[NP];
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    pok[u] = lane + u * WAVE < a.wout;
    nown[u] = T(0);
  }
  // the passive table's next row, loaded while the current one is walked
  auto fetch_own = [&](int64_t row) {
#pragma unroll
    for (int u = 0; u < NP; ++u) nown[u] = M[row * a.ldm + min(lane + u * WAVE, a.wout - 1)];
  };
  auto open_row = [&](int r) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      acc[u] = T(0);
      own[u] = pok[u] ? nown[u] * fm : T(0);
      pabs[u] = pok[u] ? lout[r * a.wout4 + lane + u * WAVE] : 0;
    }
  };
  T *const ls = (T *)smem;
  const int stg_off = __builtin_amdgcn_readfirstlane((int)(stg - ls));
  // Entries [pos, stop) of the stage, whose first entry is t0; c8: map offset of
  // each entry's colour; dot: their products, lane = entry of the block.  Only
  // the last group of UA has bounds.
  auto add_staged = [&](int t0, int pos, int stop, int c8, float wt, T &dot) {
    auto some = [&](int i, auto full) {
      constexpr bool FULL = decltype(full)::value;
      T x[UA][NP], d[UA];
      int o[UA][NP];
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const int c = __builtin_amdgcn_readlane(c8, FULL ? i + u : min(i + u, stop - 1));
#pragma unroll
        for (int v = 0; v < NP; ++v) o[u][v] = lmap[c + pabs[v]];
      }
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const int so = stg_off + ((FULL ? i + u : min(i + u, stop - 1)) - t0) * SR;
#pragma unroll
        for (int v = 0; v < NP; ++v) x[u][v] = ls[so + o[u][v]];
      }
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        d[u] = T(0);
        float w = 1.f;
        if constexpr (WEIGHTED)
          w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wt), (i + u) & (WAVE - 1)));
        const bool ok = FULL || i + u < stop;
#pragma unroll
        for (int v = 0; v < NP; ++v) {
          d[u] += own[v] * x[u][v];
          if (ok) acc[v] += WEIGHTED ? (T)w * x[u][v] : x[u][v];
        }
      }
      // lanes with bits (5, 4) = (a, b) reduce entry a + 2 b
      const bool h5 = lane & 32, h4 = lane & 16;
      T r01 = (h5 ? d[1] : d[0]) + shfl_xor(h5 ? d[0] : d[1], 32);
      T r23 = (h5 ? d[3] : d[2]) + shfl_xor(h5 ? d[2] : d[3], 32);
      T r = (h4 ? r23 : r01) + shfl_xor(h4 ? r01 : r23, 16);
      for (int off = 8; off > 0; off >>= 1) r += shfl_xor(r, off);
      const int k4 = lane - i;  // this lane's entry among the four
      const T mine = shfl(r, ((k4 & 1) << 5) | ((k4 & 2) << 3));
      if (k4 >= 0 && k4 < UA && lane < stop) dot = mine;
    };
    int i = pos;
    for (; i + UA <= stop; i += UA) some(i, std::true_type());
    if (i < stop) some(i, std::false_type());
  };
  auto walk = [&](int64_t beg, int first, int stride, int cnt, int ro, int r0, int r1, int rcol, int64_t row0, bool seg) {
    int cur = r0;
    fetch_own(row0 + r0);
    open_row(__builtin_amdgcn_readlane(rcol, cur));
    if (cur + 1 < r1) fetch_own(row0 + cur + 1);
    auto next = [&]() {  // write row cur, open the next
      T *dst = O + (row0 + cur) * a.ldo;
#pragma unroll
      for (int v = 0; v < NP; ++v)
        if (pok[v]) {
          T y = acc[v];
          if constexpr (SC) {
            y *= f;
            if (a.accumulate) y = dst[lane + v * WAVE] * add.so + y * add.sn;
            cmax = fmaxf(cmax, y);
          } else if (a.accumulate) {
            y += dst[lane + v * WAVE];
          }
          dst[lane + v * WAVE] = y;
        }
      if (++cur == r1) return;
      open_row(__builtin_amdgcn_readlane(rcol, cur));
      if (cur + 1 < r1) fetch_own(row0 + cur + 1);
    };
    int nx_j = 0;
    uint32_t nx_r = 0;
    float nx_w = 0.f;
    auto fetch = [&](int base) {
      const int64_t e = beg + min(base + lane, cnt - 1);
      nx_j = a.col_idx[e];
      nx_r = a.rev[e];
      if constexpr (WEIGHTED) nx_w = a.w[e];
    };
    if (first < cnt) fetch(first);
    for (int base = first; base < cnt; base += stride) {
      const int nb = min(WAVE, cnt - base);
      const int my_j = nx_j;
      const uint32_t my_r = nx_r;
      const float my_w = nx_w;
      u32x4 v[UNR];
      auto issue = [&](int t0) {
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
          const int jq = shfl_i32(my_j, min(t0 + q * streams + stream, nb - 1));
          v[q] = *(const u32x4 *)(X + (int64_t)jq * a.ldx + vec * N);
        }
      };
      issue(0);
      const int my_c = col[my_j];
      const double old = a.grad[my_r];
      T dot = T(0);
      fetch(base + stride);
      for (int t0 = 0; t0 < nb; t0 += E) {
        wave_lds_fence();
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
          const int sl = q * streams + stream;
          if (act) *(u32x4 *)(stg + sl * SR + vec * N) = rel_scaled<T, WEIGHTED>(v[q], fs);
        }
        issue(t0 + E);
        wave_lds_fence();
        const int c8 = my_c * CW;
        int pos = t0;
        const int lim = min(t0 + E, nb);
        while (pos < lim) {
          if (!seg)
            while (cur < r1 - 1 && __builtin_amdgcn_readlane(ro, cur + 1) <= base + pos) next();
          const int stop = seg || cur == r1 - 1 ? lim : min(lim, __builtin_amdgcn_readlane(ro, cur + 1) - base);
          add_staged(t0, pos, stop, c8, my_w, dot);
          pos = stop;
        }
      }
      if constexpr (SC) dot *= f;
      if (lane < nb) a.grad[my_r] = old + scale * (double)dot;
    }
    if (!seg)
      while (cur < r1) next();
  };

  for (int s = blockIdx.x; s < a.n_seg; s += gridDim.x) {
    const int row = a.seg_row[s], slot = a.seg_slot[s], len = a.seg_len[s];
    walk(a.seg_beg[s], wv * WAVE, WAVE * WAVES_PER_BLOCK, len, 0, 0, 1, (int)col[row], row, true);
    __syncthreads();
    T *red = stg0;
#pragma unroll
    for (int v = 0; v < NP; ++v)
      if (pok[v]) red[wv * a.wout + lane + v * WAVE] = acc[v];
    __syncthreads();
    T *dst = slot < 0 ? O + (int64_t)row * a.ldo : Pt + (int64_t)slot * a.ldo;
    for (int p = threadIdx.x; p < a.wout; p += BLOCK) {
      T y = red[p];
      for (int w2 = 1; w2 < WAVES_PER_BLOCK; ++w2) y += red[w2 * a.wout + p];
      if constexpr (SC) y *= f;
      if (slot < 0) {
        if (a.accumulate) {
          if constexpr (SC) y = dst[p] * add.so + y * add.sn;
          else y += dst[p];
        }
        if constexpr (SC) cmax = fmaxf(cmax, y);
      }
      dst[p] = y;
    }
    __syncthreads();
    for (int q = lane; q < E; q += WAVE) stg[q * SR + SR - 4] = T(0);
    wave_lds_fence();
  }

  const int R = a.R;
  const int64_t groups = (a.n + R - 1) / R;
  for (int64_t g = (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; g < groups; g += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const int64_t row0 = g * R;
    const int nr = __builtin_amdgcn_readfirstlane((int)min<int64_t>(R, a.n - row0));
    const int64_t rp = a.row_ptr[row0 + min(lane, nr)];
    const int rcol = lane < nr ? (int)col[row0 + lane] : 0;
    const int64_t nxt = __shfl(rp, min(lane + 1, nr));
    const uint64_t lm = __ballot(lane < nr && nxt - rp >= a.tlong);
    for (int r0 = 0; r0 < nr;) {
      if (lm >> r0 & 1) {
        ++r0;
        continue;
      }
      const uint64_t rest = lm >> r0;
      const int r1 = rest ? min(nr, r0 + (int)__builtin_ctzll(rest)) : nr;
      const int64_t beg = __shfl(rp, r0);
      const int cnt = __builtin_amdgcn_readfirstlane((int)(__shfl(rp, r1) - beg));
      walk(beg, 0, WAVE, cnt, (int)(rp - beg), r0, r1, rcol, row0, false);
      r0 = r1;
    }
  }
  if constexpr (SC) rel_raise(a.mx_out, cmax);
}

// Partial rows of long rows, in slot order, to the adjoint table.
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_rel_back_combine(RelBackCombineArgs a) {
  constexpr bool SC = sizeof(T) == 4;
  const T *P = (const T *)a.partial;
  T *O = (T *)a.O;
  RelAdd add{0, 1.f, 1.f};
  if constexpr (SC)
    if (a.accumulate)
      add = rel_accumulate(a.e_old[0], a.mx_old[0], rel_frame(a.ex[0], a.mxx[0]), a.mxx[0] == 0u);
  float cmax = 0.f;
  const int64_t total = (int64_t)a.n_long * a.w;
  for (int64_t q = (int64_t)blockIdx.x * BLOCK + threadIdx.x; q < total; q += (int64_t)gridDim.x * BLOCK) {
    const int64_t h = q / a.w, p = q - h * a.w;
    const int64_t s0 = a.long_slot0[h];
    T y = P[s0 * a.ldo + p];
    for (int s = 1; s < a.long_nslot[h]; ++s) y += P[(s0 + s) * a.ldo + p];
    T *dst = O + (int64_t)a.long_row[h] * a.ldo + p;
    if (a.accumulate) {
      if constexpr (SC) y = *dst * add.so + y * add.sn;
      else y += *dst;
    }
    *dst = y;
    if constexpr (SC) cmax = fmaxf(cmax, y);
  }
  if constexpr (SC) rel_raise(a.mx_out, cmax);
}

// Derivative by the entries of the histogram: Hbar(i, c_j).
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_rel_hist_back(RelHistBackArgs a) {
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const T *H = (const T *)a.Hb;
  double scale = a.scale;
  if constexpr (sizeof(T) == 4) scale = ldexp(scale, a.e[0]);
  auto entry = [&](int64_t e, int64_t row) {
    const int r = a.col[row], c = a.col[a.col_idx[e]];
    if (c != r) a.grad[e] += scale * (double)H[row * a.ldh + (c < r ? c : c - 1)];
  };
  for (int s = blockIdx.x; s < a.n_seg; s += gridDim.x)
    for (int e = threadIdx.x; e < a.seg_len[s]; e += BLOCK) entry(a.seg_beg[s] + e, a.seg_row[s]);
  const int R = a.R;
  const int64_t groups = (a.n + R - 1) / R;
  for (int64_t g = (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; g < groups; g += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const int64_t row0 = g * R;
    const int nr = (int)min<int64_t>(R, a.n - row0);
    const int64_t rp = a.row_ptr[row0 + min(lane, nr)];
    const int64_t beg = __shfl(rp, 0), end = __shfl(rp, nr);
    const int64_t nxt = __shfl(rp, min(lane + 1, nr));
    const uint64_t lm = __ballot(lane < nr && nxt - rp >= a.tlong);
    if (lm == 0) {
      for (int64_t e = beg + lane; e - lane < end; e += WAVE) {
        int loc = 0;
        for (int r = 1; r < nr; ++r) loc += e >= __shfl(rp, r) ? 1 : 0;
        if (e < end) entry(e, row0 + loc);
      }
    } else {
      for (int r = 0; r < nr; ++r) {
        const int64_t b0 = __shfl(rp, r), b1 = __shfl(rp, r + 1);
        if (lm >> r & 1) continue;
        for (int64_t e = b0 + lane; e < b1; e += WAVE) entry(e, row0 + r);
      }
    }
  }
}

// Largest weighted degree: a wave per row, lanes over its entries.  Sums of
// absolute values order as their bits do.
__global__ void k_zero_f64(double *out) { *out = 0.0; }
__global__ void __launch_bounds__(BLOCK) k_max_wdeg(const int64_t *row_ptr, const float *w, int64_t n, double *out) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t nwaves = (int64_t)gridDim.x * WAVES_PER_BLOCK;
  double best = 0.0;
  for (int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) / WAVE; i < n; i += nwaves) {
    const int64_t b = row_ptr[i], e = row_ptr[i + 1];
    double s = 0.0;
    for (int64_t q = b + lane; q < e; q += WAVE) s += fabs((double)w[q]);
    for (int off = 1; off < WAVE; off <<= 1) s += shfl_xor(s, off);
    if (s > best) best = s;
  }
  // most waves only read: as in rel_raise
  const unsigned long long mine = __builtin_bit_cast(unsigned long long, best);
  if (lane == 0 && best > 0.0 && mine > __hip_atomic_load((unsigned long long *)out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax((unsigned long long *)out, mine);
}

void launch_max_wdeg(const int64_t *row_ptr, const float *w, int64_t n, double *out, hipStream_t s) {
  k_zero_f64<<<1, 1, 0, s>>>(out);
  k_max_wdeg<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 3) / 4, 4096)), BLOCK, 0, s>>>(row_ptr, w, n, out);
}

void launch_rel_rev(const RelRevArgs &a, hipStream_t s) {
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>((a.nnz + BLOCK - 1) / BLOCK, 16384));
  k_rel_rev<<<g, BLOCK, 0, s>>>(a);
  k_rel_rev_check<<<g, BLOCK, 0, s>>>(a);
}

template <typename T, bool WEIGHTED>
static int rel_back_t(const RelBackArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  switch ((a.wout + WAVE - 1) / WAVE) {
    case 1: rel_go(k_rel_back<T, WEIGHTED, 1>, a, grid, BLOCK, lds, s); return 0;
    case 2: rel_go(k_rel_back<T, WEIGHTED, 2>, a, grid, BLOCK, lds, s); return 0;
    default: return -1;
  }
}

int launch_rel_back(int dtype, const RelBackArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  if (dtype == DT_F32) return a.w ? rel_back_t<float, true>(a, grid, lds, s) : rel_back_t<float, false>(a, grid, lds, s);
  return a.w ? rel_back_t<double, true>(a, grid, lds, s) : rel_back_t<double, false>(a, grid, lds, s);
}

void launch_rel_back_combine(int dtype, const RelBackCombineArgs &a, hipStream_t s) {
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)a.n_long * a.w + BLOCK - 1) / BLOCK, 4096));
  if (dtype == DT_F32) k_rel_back_combine<float><<<g, BLOCK, 0, s>>>(a);
  else k_rel_back_combine<double><<<g, BLOCK, 0, s>>>(a);
}

void launch_rel_hist_back(int dtype, const RelHistBackArgs &a, dim3 grid, hipStream_t s) {
  if (dtype == DT_F32) k_rel_hist_back<float><<<grid, BLOCK, 0, s>>>(a);
  else k_rel_hist_back<double><<<grid, BLOCK, 0, s>>>(a);
}

}  // namespace sg2v
