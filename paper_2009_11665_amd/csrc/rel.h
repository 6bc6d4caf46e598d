// Device helpers of the vertex-relative kernels (rel.hip, relgrad.hip).
#pragma once

#include "kernels.h"

namespace sg2v {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// LDS add whose order is fixed for a given address: the adds of one wave are
// issued in program order and those of one instruction in lane order.
template <typename T>
__device__ __forceinline__ void rel_add(T *p, T v, bool valid, bool &ovf) {
  if constexpr (is_u64<T>) {
    const T old = atomicAdd((unsigned long long *)p, (unsigned long long)v);
    ovf |= valid && old + v < old;
  } else {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
}

// FP32S frame of a table of one colouring: exponent E and factor 2^(e - E)
// from its exponent and the bits of its largest mantissa (0: a zero table)
__device__ __forceinline__ int rel_frame(int e, unsigned mx) { return mx ? e + ilog2_bits(mx) + 1 : 0; }
__device__ __forceinline__ float rel_factor(unsigned mx) { return mx ? exp2_int(-(ilog2_bits(mx) + 1)) : 0.f; }

// A gathered vector in its table's frame.  Weighted FP32 sums take the factor
// before the weight: the values are then at most 1 and the sum is of the size of
// the weights, whatever the size of the values before it (sums of w x scaled
// afterwards leave the range of a float where w * max|x| does, from three edges of
// 2^-50 in a row on).  Without weights a sum is below 2^62 (degree times degree),
// and one multiplication of it costs less than one of every element.
template <typename T, bool WEIGHTED>
__device__ __forceinline__ u32x4 rel_scaled(u32x4 v, T f) {
  if constexpr (WEIGHTED && sizeof(T) == 4) {
    V16<T> x = __builtin_bit_cast(V16<T>, v);
#pragma unroll
    for (int u = 0; u < V16<T>::N; ++u) x.x[u] *= f;
    return __builtin_bit_cast(u32x4, x);
  } else {
    return v;
  }
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ float wave_max(float m) {
  for (int off = 1; off < WAVE; off <<= 1) m = fmaxf(m, shfl_xor(m, off));
  return m;
}

// Raises *mx, a table's largest mantissa, to this wave's.  The waves of a launch
// share the address, and device-wide atomics to one address run one after the other
// (about 10 ns each): a wave that would not raise it, as all but a few, only reads.
__device__ __forceinline__ void rel_raise_wave(unsigned *mx, unsigned x) {
  if (x > __hip_atomic_load(mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(mx, x);
}

// The same for a block, of which every thread calls; one thread asks.  Path of 7
// vertices, k = 9, 100,003 vertices, three colourings, with an atomic of every wave
// 1.43 ms, with a read before it 0.93, once a block 0.92; multiply-add of 20
// columns, 8 x 65536 rows, 100, 58 and 48 us.
__device__ __forceinline__ void rel_raise(unsigned *mx, float m) {
  __shared__ unsigned wave_mx[8];
  m = wave_max(m);
  if ((threadIdx.x & (WAVE - 1)) == 0) wave_mx[threadIdx.x / WAVE] = __float_as_uint(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned x = wave_mx[0];
    for (int w = 1; w < (int)(blockDim.x / WAVE); ++w) x = max(x, wave_mx[w]);
    rel_raise_wave(mx, x);
  }
}

// FP32S: a contribution of exponent ec (cz: it is zero) added to a table of
// exponent eo and largest mantissa bits mo: the exponent of the sum and the
// factors of the old values and of the contribution
struct RelAdd {
  int e;
  float so, sn;
};
__device__ __forceinline__ RelAdd rel_accumulate(int eo, unsigned mo, int ec, bool cz) {
  RelAdd r;
  if (cz) {
    r.e = eo;
    r.so = 1.f;
    r.sn = 0.f;
  } else if (mo == 0u) {
    r.e = ec;
    r.so = 0.f;
    r.sn = 1.f;
  } else {
    r.e = max(eo, ec);
    r.so = exp2_int(eo - r.e);
    r.sn = exp2_int(ec - r.e);
  }
  return r;
}

template <typename K, typename A>
inline void rel_go(K kern, const A &a, dim3 grid, int nt, size_t lds, hipStream_t s) {
  if (lds > 65536) (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  kern<<<grid, nt, lds, s>>>(a);
}

}  // namespace sg2v
