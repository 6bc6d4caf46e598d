// Kernels of the count in vertex-relative tables for gfx950.
//
// A sub-template's table M_s(i, C) is zero unless the colour set C holds the
// colour of vertex i (the sub-template's root is i), and an aggregation
// B(i, P) is only ever multiplied by entries whose set holds that colour, so
// only sets P without it are read.  A table row therefore needs C(k-1, q)
// columns instead of C(k, q) or C(k, q+1): the q-sets of the k-1 colours other
// than the vertex's own, numbered 0..k-2 in increasing order (own colour left
// out), in colexicographic order:
//   M_s(i, C), |C| = m   ->  q = m - 1, the set C without the own colour;
//   B_p(i, P), |P| = m   ->  q = m, the set P.
// In these coordinates
//   - a split with a one-vertex active child is the identity: M_s = B_p;
//   - every other multiply-add and the root reduction use one pair table for
//     all vertices, whatever their colours, on rows in their natural order;
//   - the aggregation moves an entry of neighbour j (colour c) from set Q to
//     the set Q + {c} of the row's vertex, dropped when it holds the row's
//     colour.
// Tables are planes per colouring: element (j, i, p) at j * plane + i * ld + p.
#include <algorithm>

#include "kernels.h"
#include "launch.h"
#include "rel.h"

namespace sg2v {

// Start of a pass: exponents and largest mantissas of every table (the
// histogram's, table 0, is bounded by the largest weighted degree).
__global__ void __launch_bounds__(BLOCK) k_rel_init(int *e, unsigned *mx, int ntab, int b, unsigned hist_bits) {
  for (int q = threadIdx.x; q < ntab * b; q += BLOCK) {
    e[q] = 0;
    mx[q] = q < b ? hist_bits : 0u;
  }
}

// ---------------------------------------------------------------------------
// Neighbour-colour histogram H(i, c'), c' the relative colours of i.  A wave
// takes R consecutive rows, lanes over their entries; counts go to LDS (32-bit
// integers without weights, T with them).  JG colourings share the index loads.
// Rows of at least tlong entries are segments taken by whole blocks.
// Bound by the colour bytes' gathers (one address per lane).  LDS adds instead
// of a ballot or a butterfly per colour: 10M entries x 8 colourings 850 -> 369
// us, 4M weighted entries in FP64 363 -> 50 us.

template <typename T, bool WEIGHTED, int JG>
__global__ void __launch_bounds__(BLOCK) k_rel_hist(RelHistArgs a) {
  using C = typename std::conditional<WEIGHTED, T, unsigned>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int R = a.R, k = a.k, per = JG * R * k;
  C *accb = (C *)smem;
  C *acc = accb + (size_t)wv * per;
  T *H = (T *)a.H;
  T *Pt = (T *)a.partial;
  const int jg0 = blockIdx.y * JG;
  const int nj = min(JG, a.b - jg0);
  const uint8_t *col = a.colors + (int64_t)(a.j0 + jg0) * a.n;
  for (int q = lane; q < per; q += WAVE) acc[q] = C(0);
  wave_lds_fence();
  bool ovf = false;

  // entries [first, cnt) with the given stride of a range starting at beg
  auto walk = [&](int64_t beg, int first, int stride, int cnt, const int *ro, int nr) {
    for (int base = first; base < cnt; base += 2 * stride) {
      int j[2], loc[2], c[2][JG];
      float wt[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int e = base + q * stride + lane;
        const bool ok = e < cnt && base + q * stride < cnt;
        j[q] = ok ? a.col_idx[beg + e] : -1;
        wt[q] = 1.0f;
        if constexpr (WEIGHTED) wt[q] = ok ? a.w[beg + e] : 0.0f;
        loc[q] = 0;
        for (int r = 1; r < nr; ++r) loc[q] += e >= __builtin_amdgcn_readlane(*ro, r) ? 1 : 0;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < JG; ++u)
          c[q][u] = j[q] >= 0 && u < nj ? (int)col[(int64_t)u * a.n + j[q]] : -1;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < JG; ++u)
          if (c[q][u] >= 0) {
            C *p = acc + ((size_t)u * R + loc[q]) * k + c[q][u];
            if constexpr (WEIGHTED) rel_add<C>(p, (C)wt[q], true, ovf);
            else __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
          }
    }
  };

  // segments of long rows: the block's waves share the entries
  for (int s = blockIdx.x; s < a.n_seg; s += gridDim.x) {
    const int row = a.seg_row[s], len = a.seg_len[s], slot = a.seg_slot[s];
    const int none = 0;
    walk(a.seg_beg[s], wv * WAVE, WAVE * WAVES_PER_BLOCK, len, &none, 1);
    __syncthreads();
    for (int q = threadIdx.x; q < nj * (int)a.ldh; q += BLOCK) {
      const int u = q / (int)a.ldh, rc = q - u * (int)a.ldh;
      const int r = col[(int64_t)u * a.n + row];
      const int cc = rc < r ? rc : rc + 1;
      T v = T(0);
      if (rc < k - 1)
        for (int w2 = 0; w2 < WAVES_PER_BLOCK; ++w2) v += (T)accb[(size_t)w2 * per + (size_t)u * R * k + cc];
      T *dst = slot < 0 ? H + (jg0 + u) * a.hplane + (int64_t)row * a.ldh
                        : Pt + (jg0 + u) * a.pplane + (int64_t)slot * a.ldh;
      dst[rc] = v;
    }
    __syncthreads();
    for (int u = 0; u < JG; ++u)
      if (lane < k) acc[(size_t)u * R * k + lane] = C(0);
    wave_lds_fence();
  }

  const int64_t groups = (a.n + R - 1) / R;
  for (int64_t g = (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; g < groups; g += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const int64_t row0 = g * R;
    const int nr = (int)min<int64_t>(R, a.n - row0);
    const int64_t rp = a.row_ptr[row0 + min(lane, nr)];
    const int64_t beg = __shfl(rp, 0), end = __shfl(rp, nr);
    const int64_t nxt = __shfl(rp, min(lane + 1, nr));
    const uint64_t lm = __ballot(lane < nr && nxt - rp >= a.tlong);
    if (lm == 0) {
      const int ro = (int)(rp - beg);
      walk(beg, 0, WAVE, (int)(end - beg), &ro, nr);
    } else {
      for (int r = 0; r < nr; ++r) {
        if (lm >> r & 1) continue;
        const int64_t b0 = __shfl(rp, r), b1 = __shfl(rp, r + 1);
        // every entry of this row is at or past its own start and before the next
        const int ro = lane <= r ? 0 : INT32_MAX;
        walk(b0, 0, WAVE, (int)(b1 - b0), &ro, nr);
      }
    }
    wave_lds_fence();
    for (int q = lane; q < nj * nr * (int)a.ldh; q += WAVE) {
      const int u = q / (nr * (int)a.ldh), q2 = q - u * nr * (int)a.ldh;
      const int loc = q2 / (int)a.ldh, rc = q2 - loc * (int)a.ldh;
      if (lm >> loc & 1) continue;
      const int r = col[(int64_t)u * a.n + row0 + loc];
      const int cc = rc < r ? rc : rc + 1;
      H[(jg0 + u) * a.hplane + (row0 + loc) * a.ldh + rc] =
          rc < k - 1 ? (T)acc[((size_t)u * R + loc) * k + cc] : T(0);
    }
    wave_lds_fence();
    for (int q = lane; q < per; q += WAVE) acc[q] = C(0);
    wave_lds_fence();
  }
}

// ---------------------------------------------------------------------------
// Aggregation.  A wave takes R consecutive rows of one colouring (blockIdx.y)
// and walks their entries: streams of LP lanes read whole neighbour rows with
// 16-byte loads, UNR per lane in flight, and put them in the wave's LDS stage;
// while the next ones are in flight, lane p adds to output position p (NP per
// lane) the staged element its set takes from each row, through a map from
// (neighbour colour, absolute set) to the neighbour's column (a staged zero
// where the set lacks the colour).  Outputs of at most 32 columns are shared by
// SW = 64 / (columns, rounded up to a power of two) lane groups that take every
// SW-th entry and are summed by a butterfly at the end of the row.  Rows of at
// least tlong entries are segments taken by whole blocks, longest first, the
// four waves' sums added in wave order.
// Bound by the 128-byte lines gathered from beyond the L2: 70 columns of FP32
// (three lines) over 10M entries x 8 colourings take 4.3 ms, 7.1 TB/s of lines
// (random 256-byte rows: 8.6 TB/s from a 24 MB table, 7.2 from 128 MB, 6.0 from
// 4 GB).  Whole rows instead of column chunks read every index once per
// colouring and need no chunk's worth of row descriptors per row: 1.3M entries,
// 3 colourings, five aggregations with k = 9: 3.58 -> 1.19 ms.

template <typename T, bool WEIGHTED, int NP, bool SPLIT>
__global__ void __launch_bounds__(BLOCK) k_rel_spmm(RelSpmmArgs a) {
  constexpr int N = V16<T>::N;
  constexpr int UNR = 4, UA = 4;
  using A = Arith<T>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int jj = blockIdx.y;
  const int CW = a.cw, SR = a.sr;
  uint16_t *lmap = (uint16_t *)smem;   // [k][CW]
  uint16_t *lout = lmap + a.k * CW;    // [k][wout4]
  T *stg0 = (T *)(smem + ((a.k * (CW + a.wout4) * 2 + 15) & ~15));
  const int streams = a.streams, E = UNR * streams;
  T *stg = stg0 + (size_t)wv * E * SR;
  for (int q = threadIdx.x; q < a.k * CW / 2; q += BLOCK) ((unsigned *)lmap)[q] = ((const unsigned *)a.map)[q];
  for (int q = threadIdx.x; q < a.k * a.wout4 / 2; q += BLOCK) ((unsigned *)lout)[q] = ((const unsigned *)a.olist)[q];
  for (int q = lane; q < E; q += WAVE) stg[q * SR + SR - 4] = T(0);  // the staged zeros
  __syncthreads();
  const uint8_t *col = a.colors + (int64_t)(a.j0 + jj) * a.n;
  const T *__restrict__ M = (const T *)a.M + jj * a.mplane;
  T *__restrict__ B = (T *)a.B + jj * a.bplane;
  T *__restrict__ Pt = (T *)a.partial + jj * a.pplane;
  T fs = T(1), f = T(1);  // factors of the staged rows and of the sums
  if constexpr (sizeof(T) == 4) {
    (WEIGHTED ? fs : f) = rel_factor(a.mx_in[jj]);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.e_out[jj] = rel_frame(a.e_in[jj], a.mx_in[jj]);
  }
  const int stream = lane / a.lp, vec = lane - stream * a.lp;
  const bool act = stream < streams;
  // output position and entry group of this lane
  const int gw = SPLIT ? a.gw : WAVE;      // lanes of a group
  const int p0 = SPLIT ? lane & (gw - 1) : lane, grp = SPLIT ? lane / gw : 0;
  const int SW = SPLIT ? WAVE / gw : 1;
  float cmax = 0.f;
  bool ovf = false;
  T acc[NP];
  int pabs[NP];  // absolute sets of the current row's positions (0: past the end)
  bool pok[NP];
  int opos[NP];  // columns of those positions
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const int p = p0 + u * WAVE;
    pok[u] = p < a.wout;
    opos[u] = pok[u] && a.opos ? a.opos[p] : p;
  }

  auto open_row = [&](int r) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      acc[u] = T(0);
      pabs[u] = pok[u] ? lout[r * a.wout4 + p0 + u * WAVE] : 0;
    }
  };
  T *const ls = (T *)smem;  // the stage through the start of the LDS: one address add per element
  const int stg_off = __builtin_amdgcn_readfirstlane((int)(stg - ls));
  // Entries [pos, stop) of the stage, whose first entry is t0; c8: map offset of
  // each entry's colour, by lane.  UA * SW entries at a time, their map reads and
  // then their stage reads in flight together; only the last group has bounds
  // (with bounds in every group: weighted fp64 k = 10 1.95 ms, now 1.87).
  auto add_staged = [&](int t0, int pos, int stop, int c8, float wt) {
    auto some = [&](int i, auto full) {
      constexpr bool FULL = decltype(full)::value;
      T x[UA][NP];
      int o[UA][NP];
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const int at = SPLIT ? i + u * SW + grp : i + u, idx = FULL ? at : min(at, stop - 1);
        const int c = SPLIT ? shfl_i32(c8, idx) : __builtin_amdgcn_readlane(c8, idx);
#pragma unroll
        for (int v = 0; v < NP; ++v) o[u][v] = lmap[c + pabs[v]];
      }
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const int at = SPLIT ? i + u * SW + grp : i + u, idx = FULL ? at : min(at, stop - 1);
        const int so = stg_off + (idx - t0) * SR;
#pragma unroll
        for (int v = 0; v < NP; ++v) x[u][v] = ls[so + o[u][v]];
      }
#pragma unroll
      for (int u = 0; u < UA; ++u) {
        const int idx = SPLIT ? i + u * SW + grp : i + u;
        float w = 1.f;  // every lane is active here
        if constexpr (WEIGHTED) w = SPLIT ? shfl(wt, idx) : __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wt), idx & (WAVE - 1)));
        if (FULL || idx < stop) {
          if constexpr (WEIGHTED) {
#pragma unroll
            for (int v = 0; v < NP; ++v) acc[v] = A::fma((T)w, x[u][v], acc[v], ovf);
          } else if constexpr (is_u64<T>) {
#pragma unroll
            for (int v = 0; v < NP; ++v) {
              bool o2 = false;
              acc[v] = A::add(acc[v], x[u][v], o2);
              ovf |= o2 && pok[v];
            }
          } else {
#pragma unroll
            for (int v = 0; v < NP; ++v) acc[v] = A::add(acc[v], x[u][v], ovf);
          }
        }
      }
    };
    int i = pos;
    for (; i + UA * SW <= stop; i += UA * SW) some(i, std::true_type());
    if (i < stop) some(i, std::false_type());
  };
  auto sum_groups = [&]() {
    if constexpr (SPLIT) {
      for (int off = gw; off < WAVE; off <<= 1)
#pragma unroll
        for (int v = 0; v < NP; ++v) {
          bool o2 = false;
          acc[v] = A::add(acc[v], shfl_xor(acc[v], off), o2);
          ovf |= o2 && pok[v];
        }
    }
  };
  // Walk the entries [beg, beg + cnt) whose rows are cut at ro (lane q: offset
  // of row q); rows r0 .. r1-1 are opened and, except in a segment, written.
  // first / stride: the 64-entry blocks this wave takes.
  auto walk = [&](int64_t beg, int first, int stride, int cnt, int ro, int r0, int r1, int rcol, int64_t row0, bool seg) {
    int cur = r0;
    open_row(__builtin_amdgcn_readlane(rcol, cur));
    auto flush = [&]() {
      sum_groups();
      if (!SPLIT || grp == 0) {
        T *dst = B + (row0 + cur) * a.ldb;
#pragma unroll
        for (int v = 0; v < NP; ++v)
          if (pok[v]) {
            T x = acc[v];
            if constexpr (sizeof(T) == 4) {
              x *= f;
              cmax = fmaxf(cmax, x);
            }
            dst[opos[v]] = x;
          }
      }
    };
    // Loads are unconditional (lanes past the end repeat the last entry): a load
    // under a condition is waited for where the branches meet.
    int nx_j = 0;
    float nx_w = 0.f;
    auto fetch = [&](int base) {
      const int64_t e = beg + min(base + lane, cnt - 1);
      nx_j = a.col_idx[e];
      if constexpr (WEIGHTED) nx_w = a.w[e];
    };
    if (first < cnt) fetch(first);
    for (int base = first; base < cnt; base += stride) {
      const int nb = min(WAVE, cnt - base);
      const int my_j = nx_j;
      const float my_w = nx_w;
      u32x4 v[UNR];
      auto issue = [&](int t0) {
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
          const int jq = shfl_i32(my_j, min(t0 + q * streams + stream, nb - 1));
          v[q] = *(const u32x4 *)(M + (int64_t)jq * a.ldm + vec * N);
        }
      };
      issue(0);
      const int my_c = col[my_j];
      fetch(base + stride);
      for (int t0 = 0; t0 < nb; t0 += E) {
        wave_lds_fence();  // the previous batch has been read
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
            while (cur < r1 - 1 && __builtin_amdgcn_readlane(ro, cur + 1) <= base + pos) {
              flush();
              ++cur;
              open_row(__builtin_amdgcn_readlane(rcol, cur));
            }
          const int stop = seg || cur == r1 - 1 ? lim : min(lim, __builtin_amdgcn_readlane(ro, cur + 1) - base);
          add_staged(t0, pos, stop, c8, my_w);
          pos = stop;
        }
      }
    }
    if (!seg)
      for (;;) {
        flush();
        if (++cur == r1) break;
        open_row(__builtin_amdgcn_readlane(rcol, cur));
      }
  };

  for (int s = blockIdx.x; s < a.n_seg; s += gridDim.x) {
    const int row = a.seg_row[s], slot = a.seg_slot[s], len = a.seg_len[s];
    const int r = col[row];
    walk(a.seg_beg[s], wv * WAVE, WAVE * WAVES_PER_BLOCK, len, 0, 0, 1, r, row, true);
    sum_groups();
    __syncthreads();  // every wave is done with its stage
    T *red = stg0;    // [waves][wout]
    if (!SPLIT || grp == 0)
#pragma unroll
      for (int v = 0; v < NP; ++v)
        if (pok[v]) red[wv * a.wout + p0 + v * WAVE] = acc[v];
    __syncthreads();
    T *dst = slot < 0 ? B + (int64_t)row * a.ldb : Pt + (int64_t)slot * a.ldb;
    for (int p = threadIdx.x; p < a.wout; p += BLOCK) {
      T x = red[p];
      for (int w2 = 1; w2 < WAVES_PER_BLOCK; ++w2) x = A::add(x, red[w2 * a.wout + p], ovf);
      if constexpr (sizeof(T) == 4) {
        x *= f;
        if (slot < 0) cmax = fmaxf(cmax, x);
      }
      dst[a.opos ? a.opos[p] : p] = x;
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
    // runs of consecutive rows below tlong
    for (int r0 = 0; r0 < nr;) {
      if (lm >> r0 & 1) {
        ++r0;
        continue;
      }
      const uint64_t rest = lm >> r0;
      const int r1 = rest ? min(nr, r0 + (int)__builtin_ctzll(rest)) : nr;
      const int64_t beg = __shfl(rp, r0);
      const int cnt = __builtin_amdgcn_readfirstlane((int)(__shfl(rp, r1) - beg));
      // rows of the run are below tlong, so their offsets fit 32 bits
      walk(beg, 0, WAVE, cnt, (int)(rp - beg), r0, r1, rcol, row0, false);
      r0 = r1;
    }
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if constexpr (sizeof(T) == 4) rel_raise(a.mx_out + jj, cmax);
}

// The same aggregation for narrow outputs: a lane adds the elements it has read
// to the row's absolute sets in LDS, through the neighbour colour's map.  The
// sums are doubles for FP32 and FP64 tables (float LDS adds run at a fraction
// of the rate of 8-byte ones), 64-bit integers in U64.  R rows per wave have
// their sums in LDS at a time; a row's output positions pick its sets.

template <typename T, bool WEIGHTED>
__global__ void __launch_bounds__(BLOCK) k_rel_spmm_add(RelSpmmArgs a) {
  constexpr int N = V16<T>::N;
  constexpr int UNR = 4;
  using C = typename std::conditional<is_u64<T>, uint64_t, double>::type;
  struct alignas(2 * N) M16 { uint16_t x[N]; };
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int jj = blockIdx.y;
  const int S = a.cw + 4, R = a.R;  // the element cw takes the padding of a gathered row
  uint16_t *lmap = (uint16_t *)smem;        // [k][wmap]
  uint16_t *lout = lmap + a.k * a.wmap;     // [k][wout4]
  C *acc0 = (C *)(smem + ((a.k * (a.wmap + a.wout4) * 2 + 15) & ~15));
  C *acc = acc0 + (size_t)wv * R * S;
  for (int q = threadIdx.x; q < a.k * a.wmap / 2; q += BLOCK) ((unsigned *)lmap)[q] = ((const unsigned *)a.smap)[q];
  for (int q = threadIdx.x; q < a.k * a.wout4 / 2; q += BLOCK) ((unsigned *)lout)[q] = ((const unsigned *)a.olist)[q];
  for (int q = lane; q < R * S; q += WAVE) acc[q] = C(0);
  __syncthreads();
  const uint8_t *col = a.colors + (int64_t)(a.j0 + jj) * a.n;
  const T *__restrict__ M = (const T *)a.M + jj * a.mplane;
  T *__restrict__ B = (T *)a.B + jj * a.bplane;
  T *__restrict__ Pt = (T *)a.partial + jj * a.pplane;
  T f = T(1);
  if constexpr (sizeof(T) == 4) {
    f = rel_factor(a.mx_in[jj]);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.e_out[jj] = rel_frame(a.e_in[jj], a.mx_in[jj]);
  }
  const int streams = a.streams, E = UNR * streams;
  const int stream = lane / a.lp, vec = lane - stream * a.lp;
  const bool act = stream < streams;
  float cmax = 0.f;
  bool ovf = false;

  // entries first, first + stride, ... (64 at a time) of [beg, beg + cnt), whose
  // rows r0 .. r1-1 are cut at ro (lane q: offset of row q)
  auto walk = [&](int64_t beg, int first, int stride, int cnt, int ro, int r0, int r1) {
    int nx_j = 0;
    float nx_w = 0.f;
    auto fetch = [&](int base) {
      const int64_t e = beg + min(base + lane, cnt - 1);
      nx_j = a.col_idx[e];
      if constexpr (WEIGHTED) nx_w = a.w[e];
    };
    if (first < cnt) fetch(first);
    for (int base = first; base < cnt; base += stride) {
      const int nb = min(WAVE, cnt - base);
      const int my_j = nx_j;
      const float my_w = nx_w;
      u32x4 v[UNR];
      auto issue = [&](int q, int t0) {
        const int jq = shfl_i32(my_j, min(t0 + q * streams + stream, nb - 1));
        v[q] = *(const u32x4 *)(M + (int64_t)jq * a.ldm + vec * N);
      };
#pragma unroll
      for (int q = 0; q < UNR; ++q) issue(q, 0);
      const int mc = col[my_j];
      fetch(base + stride);
      int loc = r0;
      for (int r = r0 + 1; r < r1; ++r) loc += base + lane >= __builtin_amdgcn_readlane(ro, r) ? 1 : 0;
      // LDS offsets of the colour's map and of the row's sums
      const int inf = mc * a.wmap | (loc * S) << 16;
      for (int t0 = 0; t0 < nb; t0 += E) {
#pragma unroll
        for (int q = 0; q < UNR; ++q) {
          const int sq = t0 + q * streams + stream;
          const int iq = shfl_i32(inf, min(sq, nb - 1));
          T wq = T(1);
          if constexpr (WEIGHTED) wq = (T)shfl(my_w, min(sq, nb - 1));
          const V16<T> x = __builtin_bit_cast(V16<T>, v[q]);
          issue(q, t0 + E);
          if (act && sq < nb) {
            const M16 mp = *(const M16 *)(lmap + (iq & 0xFFFF) + vec * N);
            C *row = acc + ((unsigned)iq >> 16);
            auto add = [&](int u) {
              C y = (C)x.x[u];
              if constexpr (WEIGHTED) y *= (C)wq;
              rel_add<C>(row + mp.x[u], y, mp.x[u] != a.cw, ovf);
            };
            // The padding of one row's entries goes to one address, adds to which are
            // serial: up to three of four elements in FP32, left out (15 columns, 8 x
            // 2.1M entries, 396 -> 354 us).  In 8-byte elements it is one of two at
            // most, and the branches cost more (path of 8, U64: 1.44 -> 1.57 ms).
            if (sizeof(T) == 4 && a.padded) {
#pragma unroll
              for (int u = 0; u < N; ++u)
                if (mp.x[u] != a.cw) add(u);
            } else {
#pragma unroll
              for (int u = 0; u < N; ++u) add(u);
            }
          }
        }
      }
    }
  };

  for (int s = blockIdx.x; s < a.n_seg; s += gridDim.x) {
    const int row = a.seg_row[s], slot = a.seg_slot[s];
    const int r = col[row];
    walk(a.seg_beg[s], wv * WAVE, WAVE * WAVES_PER_BLOCK, a.seg_len[s], 0, 0, 1);
    __syncthreads();
    T *dst = slot < 0 ? B + (int64_t)row * a.ldb : Pt + (int64_t)slot * a.ldb;
    for (int p = threadIdx.x; p < a.wout; p += BLOCK) {
      const C *q = acc0 + lout[r * a.wout4 + p];
      C x = q[0];
      for (int w2 = 1; w2 < WAVES_PER_BLOCK; ++w2) x = Arith<C>::add(x, q[(size_t)w2 * R * S], ovf);
      T y;
      if constexpr (sizeof(T) == 4) {
        y = (T)(x * (C)f);  // in double: weighted sums may leave the range of a float
        if (slot < 0) cmax = fmaxf(cmax, y);
      } else {
        y = (T)x;
      }
      dst[a.opos ? a.opos[p] : p] = y;
    }
    __syncthreads();
    for (int q = lane; q < S; q += WAVE) acc[q] = C(0);
    wave_lds_fence();
  }

  const int64_t groups = (a.n + R - 1) / R;
  const int dl = WAVE / a.wout, dp = WAVE - dl * a.wout;
  const int l0 = lane / a.wout, p0 = lane - l0 * a.wout;
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
      walk(beg, 0, WAVE, cnt, (int)(rp - beg), r0, r1);
      r0 = r1;
    }
    wave_lds_fence();
    int loc = l0, p = p0;
    while (__ballot(loc < nr)) {
      const int r = shfl_i32(rcol, loc & (WAVE - 1));
      if (loc < nr && !(lm >> loc & 1)) {
        const C x = acc[loc * S + lout[r * a.wout4 + p]];
        T y;
        if constexpr (sizeof(T) == 4) {
          y = (T)(x * (C)f);
          cmax = fmaxf(cmax, y);
        } else {
          y = (T)x;
        }
        B[(row0 + loc) * a.ldb + (a.opos ? a.opos[p] : p)] = y;
      }
      p += dp;
      loc += dl;
      if (p >= a.wout) {
        p -= a.wout;
        ++loc;
      }
    }
    wave_lds_fence();
    for (int q = lane; q < R * S; q += WAVE) acc[q] = C(0);
    wave_lds_fence();
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if constexpr (sizeof(T) == 4) rel_raise(a.mx_out + jj, cmax);
}

// ---------------------------------------------------------------------------
// Wide aggregations, in chunks of the colour sets with one choice of high
// colours (blockIdx.y; the planner's rel_wide_tables).  The entries of every
// task are sorted by neighbour colour once per colouring, so that a wave adds a
// colour's runs in registers, lane by lane as they are read, and permutes the
// sum once per colour (through its LDS stage) instead of each run.  Tasks of the
// neighbour-range split are taken once per range by the blocks of one XCD.

// Entries of each task (of each range of the first x_tasks ones) by colour, in
// their order within a colour; off: where each colour starts.
template <bool WEIGHTED>
__global__ void __launch_bounds__(BLOCK) k_rel_sort(RelSortArgs a) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t wave = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) / WAVE;
  const int64_t nwaves = (int64_t)gridDim.x * WAVES_PER_BLOCK;
  const int jj = blockIdx.y, k = a.k;
  const uint8_t *col = a.colors + (int64_t)(a.j0 + jj) * a.n;
  int32_t *out = a.out + jj * a.nnz;
  float *wout = WEIGHTED ? a.wout + jj * a.nnz : nullptr;
  uint16_t *off = a.off + jj * a.n_items * 32;
  for (int64_t it = wave; it < a.n_items; it += nwaves) {
    const int64_t xs = a.x_tasks * a.xsplit;
    const int64_t t = it < xs ? it / a.xsplit : it - xs + a.x_tasks;
    int64_t beg = a.task_beg[t];
    int len = a.task_len[t];
    if (it < xs) {
      const int xr = (int)(it - t * a.xsplit);
      const uint16_t *sp = a.tsplit + t * (a.xsplit + 1);
      beg += sp[xr];
      len = sp[xr + 1] - sp[xr];
    }
    len = __builtin_amdgcn_readfirstlane(len);
    int cnt = 0;  // of colour `lane`
    for (int base = 0; base < len; base += WAVE) {
      const int c = base + lane < len ? (int)col[a.col_idx[beg + base + lane]] : 255;
      for (int cc = 0; cc < k; ++cc) {
        const int m = __popcll(__ballot(c == cc));
        if (lane == cc) cnt += m;
      }
    }
    int at = 0;  // exclusive prefix over the colours
    for (int cc = 0; cc < k; ++cc) {
      const int m = __builtin_amdgcn_readlane(cnt, cc);
      if (lane > cc) at += m;
    }
    if (lane <= k) off[it * 32 + lane] = (uint16_t)at;
    const uint64_t lt = (1ull << lane) - 1ull;
    for (int base = 0; base < len; base += WAVE) {
      const bool in = base + lane < len;
      const int j = in ? a.col_idx[beg + base + lane] : 0;
      const int c = in ? (int)col[j] : 255;
      int pos = 0;
      for (int cc = 0; cc < k; ++cc) {
        const uint64_t m = __ballot(c == cc);
        if (c == cc) pos = __builtin_amdgcn_readlane(at, cc) + __popcll(m & lt);
        if (lane == cc) at += __popcll(m);
      }
      if (in) {
        out[beg + pos] = j;
        if constexpr (WEIGHTED) wout[beg + pos] = a.w[beg + base + lane];
      }
    }
  }
}

// BEGIN k_rel_wide
// Bound by the lines in flight per CU: 82 lines per entry and table of 3003
// columns, half of them from beyond the L2 (6.3 TB/s), about 71 in flight per CU
// at 452 cycles.  Six waves per SIMD (five without the launch bound): 214 -> 199
// ms for the whole count of the 15-vertex tree on RMAT scale 20 in FP32, seven
// (spills in FP64): 205.  The absolute tables' k_spmm took 252 of 298 ms.
template <typename T, bool WEIGHTED, int NP>
__global__ void __launch_bounds__(BLOCK, 6) k_rel_wide(RelWideArgs a) {
  constexpr int N = V16<T>::N;
  constexpr int UNR = 4;
  using A = Arith<T>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int k = a.k, l = a.l;
  const int jj = blockIdx.y / a.nchunk, chunk = blockIdx.y - jj * a.nchunk;
  const int32_t *hdr = a.hdr + (int64_t)chunk * (1 + 2 * k);
  const int32_t *I = a.info + hdr[0] * 9;
  const int cw = I[0], lin_low = I[3], lin_high = I[4], lout_low = I[5], lout_high = I[6];
  const int osplit = I[7], ogap = I[8];
  uint16_t *linv = (uint16_t *)smem;
  uint16_t *lout = linv + (l + 1) * cw;
  T *stg = (T *)(smem + ((2 * (l + 1) * cw * 2 + 15) & ~15)) + (size_t)wv * a.stage;
  for (int q = threadIdx.x; q < (l + 1) * cw / 2; q += BLOCK) {
    ((unsigned *)linv)[q] = ((const unsigned *)(a.tab + I[1]))[q];
    ((unsigned *)lout)[q] = ((const unsigned *)(a.tab + I[2]))[q];
  }
  // lane c: first columns of colour c's run and of a row of colour c (-1: none)
  const int in0 = lane < k ? hdr[1 + lane] : -1, out0 = lane < k ? hdr[1 + k + lane] : -1;
  const uint32_t usable = (uint32_t)__ballot(in0 >= 0);
  __syncthreads();
  const uint8_t *col = a.colors + (int64_t)(a.j0 + jj) * a.n;
  const int32_t *scol = a.scol + jj * a.nnz;
  const float *sw = WEIGHTED ? a.sw + jj * a.nnz : nullptr;
  const uint16_t *off = a.off + jj * a.n_items * 32;
  const T *__restrict__ M = (const T *)a.M + jj * a.mplane;
  T *__restrict__ B = (T *)a.B + jj * a.bplane;
  T *__restrict__ Pt = (T *)a.partial + jj * a.pplane;
  T *__restrict__ P8 = (T *)a.partial8 + jj * a.p8plane;
  T fs = T(1), f = T(1);  // factors of the gathered rows and of the sums
  if constexpr (sizeof(T) == 4) {
    (WEIGHTED ? fs : f) = rel_factor(a.mx_in[jj]);
    if (blockIdx.x == 0 && chunk == 0 && threadIdx.x == 0) a.e_out[jj] = rel_frame(a.e_in[jj], a.mx_in[jj]);
  }
  // lanes of a run by class (low, high): vectors, lanes per run, streams
  const int nv_l = (lin_low + N - 1) / N, nv_h = (lin_high + N - 1) / N;
  const int lp_l = max(1, min(nv_l, WAVE)), lp_h = max(1, min(nv_h, WAVE));
  const int st_l = WAVE / lp_l, st_h = WAVE / lp_h;
  const int stream_l = lane / lp_l, vec_l = lane - stream_l * lp_l;
  const int stream_h = lane / lp_h, vec_h = lane - stream_h * lp_h;
  float cmax = 0.f;
  bool ovf = false;

  // one task (or one range of it): out[p] = sum over its entries
  T out[NP];
  int pabs[NP];
  auto task = [&](int64_t beg, int r, int64_t item, int nout) {
    const int rrow = r < l ? r : l;
#pragma unroll
    for (int v = 0; v < NP; ++v) {
      out[v] = T(0);
      pabs[v] = lane + v * WAVE < nout ? lout[rrow * cw + lane + v * WAVE] : 0;
    }
    const int o_c = lane <= k ? (int)off[item * 32 + lane] : 0;
    uint32_t todo = usable & ~(1u << r);
    const int o_n = shfl_i32(o_c, min(lane + 1, WAVE - 1));
    todo &= (uint32_t)__ballot(lane < k && o_c != o_n);
    if (todo == 0) return;
    // pieces of up to 64 entries of one colour; the next piece's indices are
    // loaded while this one's rows are gathered
    int c = __builtin_ctz(todo), e = __builtin_amdgcn_readlane(o_c, c), end = __builtin_amdgcn_readlane(o_c, c + 1);
    int nx_j = scol[beg + min(e + lane, end - 1)];
    float nx_w = 1.f;
    if constexpr (WEIGHTED) nx_w = sw[beg + min(e + lane, end - 1)];
    V16<T> acc;
#pragma unroll
    for (int u = 0; u < N; ++u) acc.x[u] = T(0);
    while (todo) {
      const int cc = c, nb = min(WAVE, end - e);
      const bool last = e + WAVE >= end;  // of this colour
      const int my_j = nx_j;
      const float my_w = nx_w;
      e += WAVE;
      if (last) {
        todo &= todo - 1;
        if (todo) {
          c = __builtin_ctz(todo);
          e = __builtin_amdgcn_readlane(o_c, c);
          end = __builtin_amdgcn_readlane(o_c, c + 1);
        }
      }
      if (todo) {
        nx_j = scol[beg + min(e + lane, end - 1)];
        if constexpr (WEIGHTED) nx_w = sw[beg + min(e + lane, end - 1)];
      }
      const bool low = cc < l;
      const int lp = low ? lp_l : lp_h, st = low ? st_l : st_h, nv = low ? nv_l : nv_h;
      const int stream = low ? stream_l : stream_h, vec0 = low ? vec_l : vec_h;
      const T *Mc = M + __builtin_amdgcn_readlane(in0, cc);
      const int passes = (nv + WAVE - 1) / WAVE;  // runs of more than 64 vectors (then one stream)
      for (int ps = 0; ps < passes; ++ps) {
        const int vec = min(vec0 + ps * WAVE, nv - 1);
        if (passes > 1) {
#pragma unroll
          for (int u = 0; u < N; ++u) acc.x[u] = T(0);
        }
        auto rows = [&](int t0, auto un) {
          constexpr int U = decltype(un)::value;
          u32x4 v[U];
          float wq[U];
#pragma unroll
          for (int q = 0; q < U; ++q) {
            const int sq = min(t0 + q * st + stream, nb - 1);
            const int jq = shfl_i32(my_j, sq);
            wq[q] = 1.f;
            if constexpr (WEIGHTED) wq[q] = shfl(my_w, sq);
            v[q] = *(const u32x4 *)(Mc + (int64_t)jq * a.ldm + vec * N);
          }
#pragma unroll
          for (int q = 0; q < U; ++q) {
            const bool ok = t0 + q * st + stream < nb;
            const V16<T> x = __builtin_bit_cast(V16<T>, rel_scaled<T, WEIGHTED>(v[q], fs));
#pragma unroll
            for (int u = 0; u < N; ++u) {
              const T y = ok ? x.x[u] : T(0);
              if constexpr (WEIGHTED) acc.x[u] = A::fma((T)wq[q], y, acc.x[u], ovf);
              else acc.x[u] = A::add(acc.x[u], y, ovf);
            }
          }
        };
        int t0 = 0;
        for (; nb - t0 > 2 * st; t0 += UNR * st) rows(t0, std::integral_constant<int, UNR>());
        if (nb - t0 > st) rows(t0, std::integral_constant<int, 2>());
        else if (nb > t0) rows(t0, std::integral_constant<int, 1>());
        if (!last && passes == 1) break;
        // the colour's sum (of each stream) to the stage, from there to the outputs
        wave_lds_fence();
        if (stream < st && vec0 + ps * WAVE < nv) *(V16<T> *)(stg + stream * nv * N + vec * N) = acc;
        wave_lds_fence();
        if (ps == passes - 1) {
          const int row = low ? cc : l;
#pragma unroll
          for (int v = 0; v < NP; ++v) {
            const int o = linv[row * cw + pabs[v]];
            T x = T(0);
            if (o != 0xFFFF) {
              x = stg[o];
              for (int s2 = 1; s2 < st; ++s2) x = A::add(x, stg[s2 * nv * N + o], ovf);
            }
            out[v] = A::add(out[v], x, ovf);
          }
        }
#pragma unroll
        for (int u = 0; u < N; ++u) acc.x[u] = T(0);
      }
    }
  };
  auto write = [&](T *dst, int r, int nout, bool final) {
    const int gap = r < l ? 0 : ogap;
#pragma unroll
    for (int v = 0; v < NP; ++v) {
      const int p = lane + v * WAVE;
      if (p < nout) {
        T x = out[v];
        if constexpr (sizeof(T) == 4) {
          x *= f;
          if (final) cmax = fmaxf(cmax, x);
        }
        dst[p + (p >= osplit ? gap : 0)] = x;
      }
    }
  };

  // the split tasks, range blockIdx.x % xsplit (workgroups go to the XCDs in turn)
  if (a.x_tasks > 0) {
    const int xr = blockIdx.x % a.xsplit;
    const int64_t step = (int64_t)(gridDim.x / a.xsplit) * WAVES_PER_BLOCK;
    for (int64_t t = (int64_t)(blockIdx.x / a.xsplit) * WAVES_PER_BLOCK + wv; t < a.x_tasks; t += step) {
      const int r = __builtin_amdgcn_readfirstlane((int)col[a.task_row[t]]);
      const int o0 = __builtin_amdgcn_readlane(out0, r);
      if (o0 < 0) continue;
      const int nout = r < l ? lout_low : lout_high;
      task(a.task_beg[t] + a.tsplit[t * (a.xsplit + 1) + xr], r, t * a.xsplit + xr, nout);
      write(P8 + ((int64_t)xr * a.x_tasks + t) * a.ldb + o0, r, nout, false);
    }
  }
  for (int64_t t = a.x_tasks + (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; t < a.n_tasks;
       t += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
    const int row = a.task_row[t], slot = a.task_slot[t];
    const int r = __builtin_amdgcn_readfirstlane((int)col[row]);
    const int o0 = __builtin_amdgcn_readlane(out0, r);
    if (o0 < 0) continue;
    const int nout = r < l ? lout_low : lout_high;
    task(a.task_beg[t], r, a.x_tasks * a.xsplit + t - a.x_tasks, nout);
    write((slot < 0 ? B + (int64_t)row * a.ldb : Pt + (int64_t)slot * a.ldb) + o0, r, nout, slot < 0);
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if constexpr (sizeof(T) == 4) {  // the waves of a block end at different times
    cmax = wave_max(cmax);
    if (lane == 0) rel_raise_wave(a.mx_out + jj, __float_as_uint(cmax));
  }
}

// END k_rel_wide

// The eight range partials of every split task, in range order: to its row, or to
// the slot of its segment.
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_rel_xsum(RelXsumArgs a) {
  constexpr int N = V16<T>::N;
  const int jj = blockIdx.y;
  const int64_t nvec = (a.w + N - 1) / N, total = nvec * a.n_tasks;
  const T *P = (const T *)a.partial8 + jj * a.p8plane;
  bool ovf = false;
  float cmax = 0.f;
  for (int64_t q = (int64_t)blockIdx.x * BLOCK + threadIdx.x; q < total; q += (int64_t)gridDim.x * BLOCK) {
    const int64_t t = q / nvec, v = q - t * nvec;
    V16<T> x[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = *(const V16<T> *)(P + ((int64_t)r * a.n_tasks + t) * a.ld + v * N);
    const int slot = a.task_slot[t];
    V16<T> s = x[0];
#pragma unroll
    for (int r = 1; r < 8; ++r)
#pragma unroll
      for (int u = 0; u < N; ++u) {
        bool o = false;
        s.x[u] = Arith<T>::add(s.x[u], x[r].x[u], o);
        ovf |= o && v * N + u < a.w;
      }
    T *dst = slot < 0 ? (T *)a.B + jj * a.bplane + (int64_t)a.task_row[t] * a.ld
                      : (T *)a.partial + jj * a.pplane + (int64_t)slot * a.ld;
    *(V16<T> *)(dst + v * N) = s;
    if (slot < 0)
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (v * N + u < a.w) cmax = fmaxf(cmax, (float)s.x[u]);
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if (a.mx) rel_raise(a.mx + jj, cmax);
}

// Partial rows of a long row summed in slot order.
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_rel_combine(RelCombineArgs a) {
  constexpr int N = V16<T>::N;
  const int jj = blockIdx.y;
  const int64_t nvec = (a.w + N - 1) / N, total = nvec * a.n_long;
  const T *P = (const T *)a.partial + jj * a.pplane;
  T *B = (T *)a.B + jj * a.bplane;
  bool ovf = false;
  float cmax = 0.f;
  for (int64_t q = (int64_t)blockIdx.x * BLOCK + threadIdx.x; q < total; q += (int64_t)gridDim.x * BLOCK) {
    const int64_t h = q / nvec, v = q - h * nvec;
    const int64_t s0 = a.long_slot0[h];
    const int ns = a.long_nslot[h];
    V16<T> acc = *(const V16<T> *)(P + s0 * a.ld + v * N);
    for (int s = 1; s < ns; ++s) {
      const V16<T> x = *(const V16<T> *)(P + (s0 + s) * a.ld + v * N);
#pragma unroll
      for (int u = 0; u < N; ++u) {
        bool o = false;
        acc.x[u] = Arith<T>::add(acc.x[u], x.x[u], o);
        ovf |= o && v * N + u < a.w;  // padding may hold anything
      }
    }
    *(V16<T> *)(B + (int64_t)a.long_row[h] * a.ld + v * N) = acc;
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (v * N + u < a.w) cmax = fmaxf(cmax, (float)acc.x[u]);
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if (a.mx) rel_raise(a.mx + jj, cmax);
}

// ---------------------------------------------------------------------------
// Multiply-add of a split whose active child has several vertices:
//   M_s(i, Q) = sum over the pairs (x, y) of Q of M_a(i, x) B(i, y).
// A block stages R * groups consecutive rows of both tables in LDS, transposed
// (the rows plus one 16-byte vector per column, so that lanes on different
// columns spread over the banks); a thread owns output columns and keeps R sums.
// Half the columns of the absolute tables and rows in order: 1.42 -> 0.78 ms on
// average over the splits of the nine-vertex trees (4M rows of about 60 columns
// three times, 2.9 GB: 3.7 TB/s).  Narrow outputs have a thread group for each R
// rows of the tile: binary tree of 7 vertices, 8 colourings of 65536 vertices (6 to
// 20 columns), whole count 0.99 -> 0.72 ms; all trees of 9, 124.7 -> 119.7 ms.
//
// Without X (HASX false) it counts as one: the adjoint of a root reduction.  The
// adjoint also adds to a table that holds values already (a.accumulate).

template <typename T, int R, int NT, bool HASX>
__global__ void __launch_bounds__(NT) k_rel_ema(RelEmaArgs a) {
  constexpr int N = V16<T>::N;
  constexpr bool SC = sizeof(T) == 4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int jj = blockIdx.y;
  const int RT = R * a.groups, RP = RT + N;
  T *la = (T *)smem;
  T *lb = la + (size_t)RP * (HASX ? a.wa : 0);
  const T *X = (const T *)a.X + jj * a.xplane;
  const T *Y = (const T *)a.Y + jj * a.yplane;
  T *Ms = (T *)a.M + jj * a.mplane;
  T fx = T(1), fy = T(1);
  RelAdd add{0, 1.f, 1.f};
  if constexpr (SC) {
    if constexpr (HASX) fx = rel_factor(a.mxx[jj]);
    fy = rel_factor(a.mxy[jj]);
    add.e = (HASX ? rel_frame(a.ex[jj], a.mxx[jj]) : 0) + rel_frame(a.ey[jj], a.mxy[jj]);
    if (a.accumulate) add = rel_accumulate(a.e_old[jj], a.mx_old[jj], add.e, (HASX && a.mxx[jj] == 0u) || a.mxy[jj] == 0u);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.e_out[jj] = add.e;
  }
  bool ovf = false;
  float cmax = 0.f;
  // four 16-byte loads in flight per thread
  auto stage = [&](const T *src, int64_t ld, int w, int64_t i0, int nrow, T f, T *dst) {
    const int nv = (w + N - 1) / N, total = nrow * nv;
    for (int x0 = threadIdx.x; x0 < total; x0 += 4 * NT) {
      V16<T> v[4];
      int r[4], q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int x = min(x0 + u * NT, total - 1);
        r[u] = x / nv;
        q[u] = x - r[u] * nv;
        v[u] = *(const V16<T> *)(src + (i0 + r[u]) * ld + q[u] * N);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (x0 + u * NT < total) {
#pragma unroll
          for (int e = 0; e < N; ++e)
            if (q[u] * N + e < w) dst[(q[u] * N + e) * RP + r[u]] = v[u].x[e] * f;
        }
      }
    }
  };
  // this thread's rows of a tile, its first column, and its pairs where they fit
  const int g = a.groups > 1 ? (int)threadIdx.x / a.ws : 0, rg = g * R;
  const int C0 = g < a.groups ? (int)threadIdx.x - g * a.ws : a.ws;
  const bool once = a.np <= 8 && a.ws <= NT;
  uint32_t p[8];
  auto fetch_pairs = [&](int q0, int C) {
#pragma unroll
    for (int qq = 0; qq < 8; ++qq) p[qq] = a.pairs[(int64_t)min(q0 + qq, a.np - 1) * a.ws + C];
  };
  if (once) fetch_pairs(0, min(C0, a.ws - 1));
  const int64_t ntiles = (a.n + RT - 1) / RT;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t i0 = t * RT;
    const int nrow = (int)min<int64_t>(RT, a.n - i0);
    __syncthreads();
    if constexpr (HASX) stage(X, a.ldx, a.wa, i0, nrow, fx, la);
    stage(Y, a.ldy, a.wb, i0, nrow, fy, lb);
    __syncthreads();
    for (int C = C0; C < a.ws; C += NT) {
      const int oc = a.opos ? a.opos[C] : C;
      T acc[R];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = T(0);
      for (int q0 = 0; q0 < a.np; q0 += 8) {
        if (!once) fetch_pairs(q0, C);
#pragma unroll
        for (int qq = 0; qq < 8; ++qq) {
          if (q0 + qq >= a.np) break;  // uniform
          const V16<T> *xa = (const V16<T> *)(la + (int)(p[qq] & 0xFFFFu) * RP + rg);
          const V16<T> *yb = (const V16<T> *)(lb + (int)(p[qq] >> 16) * RP + rg);
#pragma unroll
          for (int v = 0; v < R / N; ++v) {
            if constexpr (!HASX) {
              const V16<T> yv = yb[v];
#pragma unroll
              for (int e = 0; e < N; ++e) acc[v * N + e] = Arith<T>::add(acc[v * N + e], yv.x[e], ovf);
              continue;
            }
            const V16<T> xv = xa[v], yv = yb[v];
            if constexpr (is_u64<T>) {
              // rows past the end hold stale values: they may not raise the flag
#pragma unroll
              for (int e = 0; e < N; ++e) {
                bool o = false;
                acc[v * N + e] = Arith<T>::fma(xv.x[e], yv.x[e], acc[v * N + e], o);
                ovf |= o && rg + v * N + e < nrow;
              }
            } else {
#pragma unroll
              for (int e = 0; e < N; ++e) acc[v * N + e] = Arith<T>::fma(xv.x[e], yv.x[e], acc[v * N + e], ovf);
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (rg + r < nrow) {
          T *dst = Ms + (i0 + rg + r) * a.ldm + oc;
          T y = acc[r];
          if (a.accumulate) {
            if constexpr (SC) y = *dst * add.so + y * add.sn;
            else y += *dst;
          }
          *dst = y;
          if constexpr (SC) cmax = fmaxf(cmax, (float)y);
        }
      }
    }
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
  if constexpr (SC) rel_raise(a.mx_out + jj, cmax);
}

// ---------------------------------------------------------------------------
// Root reduction: sum over vertices of sum over the list of X(i, x) Y(i, y)
// (Y absent: sum of X(i, x)).  LP lanes per vertex stride over the list, U
// vertices per lane group in flight; a lane sums its share of a vertex in T
// and its vertices in double (uint64 in U64); fixed-order block reduction.  The
// list's partners are complements when k = t, so both reads are coalesced and
// nothing is staged: 0.97 -> 0.18 ms for the nine-vertex trees (4M rows, 1 GB).

template <typename T, bool HASY>
__global__ void __launch_bounds__(BLOCK) k_rel_root(RelRootArgs a) {
  using A = Arith<T>;
  using Acc = typename std::conditional<is_u64<T>, uint64_t, double>::type;
  constexpr int U = 4;
  constexpr bool SC = sizeof(T) == 4;
  __shared__ Acc red[WAVES_PER_BLOCK];
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  const int jj = blockIdx.y;
  const T *X = (const T *)a.X + jj * a.xplane;
  const T *Y = HASY ? (const T *)a.Y + jj * a.yplane : nullptr;
  T fx = T(1), fy = T(1);
  if constexpr (SC) {
    fx = rel_factor(a.mxx[jj]);
    if constexpr (HASY) fy = rel_factor(a.mxy[jj]);
  }
  bool ovf = false;
  Acc tot = Acc(0);
  const int LP = a.lp, rw = WAVE / LP;
  const int sub = lane / LP, l = lane - sub * LP;
  const int64_t step = (int64_t)rw * U;
  const int64_t nwaves = (int64_t)gridDim.x * WAVES_PER_BLOCK;
  for (int64_t i0 = ((int64_t)blockIdx.x * WAVES_PER_BLOCK + wv) * step; i0 < a.n; i0 += nwaves * step) {
    T s[U];
    const T *xr[U], *yr[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = T(0);
      const int64_t i = min(i0 + u * rw + sub, a.n - 1);
      xr[u] = X + i * a.ldx;
      yr[u] = HASY ? Y + i * a.ldy : nullptr;
    }
    for (int64_t q = l; q < a.L; q += LP) {
      const uint32_t p = a.list[q];
      T x[U], y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = xr[u][p & 0xFFFFu];
        if constexpr (HASY) y[u] = yr[u][p >> 16];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        T xv = x[u];
        if constexpr (SC) xv *= fx;
        bool o = false;
        if constexpr (HASY) {
          T yv = y[u];
          if constexpr (SC) yv *= fy;
          s[u] = A::fma(xv, yv, s[u], o);
        } else {
          s[u] = A::add(s[u], xv, o);
        }
        ovf |= o;  // rows past the end repeat the last vertex
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * rw + sub < a.n) {
        if constexpr (is_u64<Acc>) tot = A::add(tot, s[u], ovf);
        else tot += (double)s[u];
      }
    }
  }
  for (int off = 1; off < WAVE; off <<= 1) {
    if constexpr (is_u64<Acc>) tot = A::add(tot, shfl_xor(tot, off), ovf);
    else tot += shfl_xor(tot, off);
  }
  if (lane == 0) red[wv] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    Acc b = red[0];
    for (int q = 1; q < WAVES_PER_BLOCK; ++q) {
      if constexpr (is_u64<Acc>) b = A::add(b, red[q], ovf);
      else b += red[q];
    }
    ((Acc *)a.partial)[(int64_t)jj * gridDim.x + blockIdx.x] = b;
  }
  if constexpr (is_u64<T>) {
    if (ovf) atomicOr(a.ovf, 1);
  }
}

// Block partials of each colouring in a fixed order (one wave per colouring, eight
// loads in flight per lane: 2048 partials one after the other took 10 us), and in
// FP32S the exponent of the result.
template <typename Acc>
__global__ void __launch_bounds__(WAVE) k_rel_final(RelFinalArgs a) {
  const int j = blockIdx.x, lane = threadIdx.x;
  const Acc *pj = (const Acc *)a.partial + (int64_t)j * a.nblk;
  Acc s = Acc(0);
  bool o = false;
  constexpr int U = 8;
  for (int q = lane; q < a.nblk; q += U * WAVE) {
    Acc v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = pj[min(q + u * WAVE, a.nblk - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Acc x = q + u * WAVE < a.nblk ? v[u] : Acc(0);
      if constexpr (is_u64<Acc>) s = Arith<Acc>::add(s, x, o);
      else s += x;
    }
  }
  for (int off = 1; off < WAVE; off <<= 1) {
    if constexpr (is_u64<Acc>) s = Arith<Acc>::add(s, shfl_xor(s, off), o);
    else s += shfl_xor(s, off);
  }
  if (o) atomicOr(a.ovf, 1);
  if (lane == 0) {
    ((Acc *)a.out)[j] = s;
    if (a.E) a.E[j] = rel_frame(a.ex[j], a.mxx[j]) + (a.mxy ? rel_frame(a.ey[j], a.mxy[j]) : 0);
  }
}

// ===========================================================================
// launchers

void launch_rel_init(int *e, unsigned *mx, int ntab, int b, unsigned hist_bits, hipStream_t s) {
  k_rel_init<<<1, BLOCK, 0, s>>>(e, mx, ntab, b, hist_bits);
}

template <typename T>
static void rel_hist_t(const RelHistArgs &a, dim3 grid, hipStream_t s) {
  const int JG = a.b == 1 ? 1 : 4;
  const size_t lds = (size_t)WAVES_PER_BLOCK * JG * a.R * a.k * (a.w ? sizeof(T) : 4);
  if (a.b == 1) {
    if (a.w) rel_go(k_rel_hist<T, true, 1>, a, grid, BLOCK, lds, s);
    else rel_go(k_rel_hist<T, false, 1>, a, grid, BLOCK, lds, s);
  } else {
    if (a.w) rel_go(k_rel_hist<T, true, 4>, a, grid, BLOCK, lds, s);
    else rel_go(k_rel_hist<T, false, 4>, a, grid, BLOCK, lds, s);
  }
}

void launch_rel_hist(int dtype, const RelHistArgs &a, dim3 grid, hipStream_t s) {
  if (dtype == DT_F32) rel_hist_t<float>(a, grid, s);
  else if (dtype == DT_F64) rel_hist_t<double>(a, grid, s);
  else rel_hist_t<uint64_t>(a, grid, s);
}

template <typename T, bool WEIGHTED>
static int rel_spmm_t(const RelSpmmArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.add) {
    rel_go(k_rel_spmm_add<T, WEIGHTED>, a, grid, BLOCK, lds, s);
    return 0;
  }
  if (a.gw < WAVE) {
    rel_go(k_rel_spmm<T, WEIGHTED, 1, true>, a, grid, BLOCK, lds, s);
    return 0;
  }
  switch ((a.wout + WAVE - 1) / WAVE) {
    case 1: rel_go(k_rel_spmm<T, WEIGHTED, 1, false>, a, grid, BLOCK, lds, s); return 0;
    case 2: rel_go(k_rel_spmm<T, WEIGHTED, 2, false>, a, grid, BLOCK, lds, s); return 0;
    case 3: rel_go(k_rel_spmm<T, WEIGHTED, 3, false>, a, grid, BLOCK, lds, s); return 0;
    case 4: rel_go(k_rel_spmm<T, WEIGHTED, 4, false>, a, grid, BLOCK, lds, s); return 0;
    case 5: rel_go(k_rel_spmm<T, WEIGHTED, 5, false>, a, grid, BLOCK, lds, s); return 0;
    case 6: rel_go(k_rel_spmm<T, WEIGHTED, 6, false>, a, grid, BLOCK, lds, s); return 0;
    default: return -1;
  }
}

int launch_rel_spmm(int dtype, const RelSpmmArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  if (dtype == DT_F32) return a.w ? rel_spmm_t<float, true>(a, grid, lds, s) : rel_spmm_t<float, false>(a, grid, lds, s);
  if (dtype == DT_F64) return a.w ? rel_spmm_t<double, true>(a, grid, lds, s) : rel_spmm_t<double, false>(a, grid, lds, s);
  return a.w ? -1 : rel_spmm_t<uint64_t, false>(a, grid, lds, s);
}

void launch_rel_sort(const RelSortArgs &a, int b, hipStream_t s) {
  const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>((a.n_items + 3) / 4, 16384)), (unsigned)b);
  if (a.w) k_rel_sort<true><<<grid, BLOCK, 0, s>>>(a);
  else k_rel_sort<false><<<grid, BLOCK, 0, s>>>(a);
}

template <typename T, bool WEIGHTED>
static void rel_wide_t(const RelWideArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.nout_max <= 128) rel_go(k_rel_wide<T, WEIGHTED, 2>, a, grid, BLOCK, lds, s);
  else if (a.nout_max <= 256) rel_go(k_rel_wide<T, WEIGHTED, 4>, a, grid, BLOCK, lds, s);
  else rel_go(k_rel_wide<T, WEIGHTED, 6>, a, grid, BLOCK, lds, s);
}

int launch_rel_wide(int dtype, const RelWideArgs &a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.nout_max > 384) return -1;
  if (dtype == DT_F32) {
    if (a.sw) rel_wide_t<float, true>(a, grid, lds, s);
    else rel_wide_t<float, false>(a, grid, lds, s);
  } else if (dtype == DT_F64) {
    if (a.sw) rel_wide_t<double, true>(a, grid, lds, s);
    else rel_wide_t<double, false>(a, grid, lds, s);
  } else {
    rel_wide_t<uint64_t, false>(a, grid, lds, s);
  }
  return 0;
}

void launch_rel_xsum(int dtype, const RelXsumArgs &a, int b, hipStream_t s) {
  const int N = dtype == DT_F32 ? 4 : 2;
  const int64_t blocks = (a.n_tasks * ((a.w + N - 1) / N) + BLOCK - 1) / BLOCK;
  const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(blocks, 16384)), (unsigned)b);
  if (dtype == DT_F32) k_rel_xsum<float><<<grid, BLOCK, 0, s>>>(a);
  else if (dtype == DT_F64) k_rel_xsum<double><<<grid, BLOCK, 0, s>>>(a);
  else k_rel_xsum<uint64_t><<<grid, BLOCK, 0, s>>>(a);
}

void launch_rel_combine(int dtype, const RelCombineArgs &a, int b, hipStream_t s) {
  const int N = dtype == DT_F32 ? 4 : 2;
  const int64_t blocks = (a.n_long * (a.ld / N) + BLOCK - 1) / BLOCK;
  const dim3 grid((unsigned)std::min<int64_t>(blocks, 4096), (unsigned)b);
  if (dtype == DT_F32) k_rel_combine<float><<<grid, BLOCK, 0, s>>>(a);
  else if (dtype == DT_F64) k_rel_combine<double><<<grid, BLOCK, 0, s>>>(a);
  else k_rel_combine<uint64_t><<<grid, BLOCK, 0, s>>>(a);
}

template <typename T, int NT>
static int rel_ema_nt(const RelEmaArgs &a, int R, dim3 grid, size_t lds, hipStream_t s) {
  switch (R) {
    case 4: rel_go(k_rel_ema<T, 4, NT, true>, a, grid, NT, lds, s); return 0;
    case 8: rel_go(k_rel_ema<T, 8, NT, true>, a, grid, NT, lds, s); return 0;
    case 16:
      if (a.X) rel_go(k_rel_ema<T, 16, NT, true>, a, grid, NT, lds, s);
      else rel_go(k_rel_ema<T, 16, NT, false>, a, grid, NT, lds, s);
      return 0;
    default: return -1;
  }
}

template <typename T>
static int rel_ema_t(const RelEmaArgs &a, int R, int nt, dim3 grid, size_t lds, hipStream_t s) {
  if (!a.X && R != 16) return -1;
  if (nt == 512) return rel_ema_nt<T, 512>(a, R, grid, lds, s);
  if (nt == 256) return rel_ema_nt<T, 256>(a, R, grid, lds, s);
  if (nt == 128) return rel_ema_nt<T, 128>(a, R, grid, lds, s);
  return -1;
}

int launch_rel_ema(int dtype, const RelEmaArgs &a, int R, int nt, dim3 grid, size_t lds, hipStream_t s) {
  if (dtype == DT_F32) return rel_ema_t<float>(a, R, nt, grid, lds, s);
  if (dtype == DT_F64) return rel_ema_t<double>(a, R, nt, grid, lds, s);
  return rel_ema_t<uint64_t>(a, R, nt, grid, lds, s);
}

template <typename T>
static void rel_root_t(const RelRootArgs &a, dim3 grid, hipStream_t s) {
  if (a.Y) k_rel_root<T, true><<<grid, BLOCK, 0, s>>>(a);
  else k_rel_root<T, false><<<grid, BLOCK, 0, s>>>(a);
}

void launch_rel_root(int dtype, const RelRootArgs &a, dim3 grid, hipStream_t s) {
  if (dtype == DT_F32) rel_root_t<float>(a, grid, s);
  else if (dtype == DT_F64) rel_root_t<double>(a, grid, s);
  else rel_root_t<uint64_t>(a, grid, s);
}

void launch_rel_final(int dtype, const RelFinalArgs &a, int b, hipStream_t s) {
  if (dtype == DT_U64) k_rel_final<uint64_t><<<b, WAVE, 0, s>>>(a);
  else k_rel_final<double><<<b, WAVE, 0, s>>>(a);
}

}  // namespace sg2v
