// Dense k-qubit block applied with vector FMA (the path for k <= 3, and the
// reference point for the matrix-core kernel of larger blocks).
//
// For every assignment of the n-k bits outside the block (a "group"), the 2^k
// amplitudes of the group are multiplied by the block matrix. One thread owns
// one group: it gathers the 2^k amplitudes into registers, forms each output
// row against the matrix held in LDS (every lane reads the same entry, a
// broadcast) and scatters the result. Consecutive threads own groups that
// differ in the lowest free bits, so each gather/scatter instruction of a
// wavefront touches consecutive addresses whenever bit 0 is outside the block.
#include "qs_internal.h"

namespace qs {
namespace {

constexpr int kBlock = 256;

template <typename R> struct Cx { R r, i; };

__device__ __forceinline__ uint64_t insert_zero(uint64_t x, int pos) {
  const uint64_t lo = x & ((uint64_t(1) << pos) - 1);
  return lo | ((x ^ lo) << 1);
}

struct Block6 {
  int k;
  int q[6];       // bit of row/column bit j
  int sorted[6];  // the same bits ascending
  int p0;         // bit 0 of the state is row/column bit p0 of the matrix (-1: none);
                  // q then has rows p0 and 0 exchanged, so that q[0] = 0
};

// Row or column of the matrix for index x of a block with rows p0 and 0
// exchanged.
__host__ __device__ constexpr int unswap(int x, int p0) {
  if (p0 <= 0) return x;
  const int d = (x ^ (x >> p0)) & 1;
  return x ^ (d | (d << p0));
}

// The 2^K amplitudes of a group; PAIR: bit 0 is the block's first, and
// amplitudes c and c + 1 are loaded and stored as one 16-byte vector.
template <typename R, int K, bool NT, bool PAIR>
__device__ __forceinline__ void load_group(const R* __restrict__ a, const uint64_t (&off)[1 << K],
                                           Cx<R> (&v)[1 << K]) {
  if constexpr (PAIR) {
#pragma unroll
    for (int c = 0; c < (1 << K); c += 2) {
      const float4 t = ld16<NT>(reinterpret_cast<const float4*>(a + 2 * off[c]));
      v[c] = {t.x, t.y};
      v[c + 1] = {t.z, t.w};
    }
  } else {
#pragma unroll
    for (int c = 0; c < (1 << K); ++c) ld_amp<NT>(a + 2 * off[c], &v[c].r, &v[c].i);
  }
}

template <typename R, int K, bool NT, bool PAIR>
__global__ void __launch_bounds__(kBlock) k_fused_vec(R* __restrict__ a, uint64_t groups, Block6 b,
                                                      const R* __restrict__ mat) {
  constexpr int D = 1 << K;
  __shared__ Cx<R> M[D * D];
  for (int e = threadIdx.x; e < D * D; e += kBlock) {
    const int f = PAIR ? unswap(e / D, b.p0) * D + unswap(e % D, b.p0) : e;
    M[e] = {mat[2 * f], mat[2 * f + 1]};
  }
  __syncthreads();
  for (uint64_t g = uint64_t(blockIdx.x) * kBlock + threadIdx.x; g < groups;
       g += uint64_t(gridDim.x) * kBlock) {
    uint64_t base = g;
#pragma unroll
    for (int j = 0; j < K; ++j) base = insert_zero(base, b.sorted[j]);
    uint64_t off[D];
    Cx<R> v[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      uint64_t o = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) o |= uint64_t((c >> j) & 1) << b.q[j];
      off[c] = base | o;
    }
    load_group<R, K, NT, PAIR>(a, off, v);
    R lr = 0, li = 0;  // the even row of a pair
#pragma unroll
    for (int r = 0; r < D; ++r) {
      // complex128: read the matrix row by row (left to itself the compiler
      // holds all of M in registers, 256 VGPRs at k = 3, one wave per SIMD)
      if constexpr (sizeof(R) == 8) asm volatile("" ::: "memory");
      R yr = 0, yi = 0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const Cx<R> m = M[r * D + c];
        yr = fmadd(m.r, v[c].r, fmadd(-m.i, v[c].i, yr));
        yi = fmadd(m.r, v[c].i, fmadd(m.i, v[c].r, yi));
      }
      if constexpr (PAIR) {
        if (r & 1)
          st16<NT>(reinterpret_cast<float4*>(a + 2 * off[r & ~1]), float4{lr, li, yr, yi});
        lr = yr;
        li = yi;
      } else {
        st_amp<NT>(a + 2 * off[r], yr, yi);
      }
    }
  }
}

// Blocks of one to three qubits with the matrix passed by value: the same
// arithmetic as k_fused_vec, the matrix from the kernel arguments by way of LDS
// (read from there directly, states above the last-level cache lose: 27 qubits
// 352 -> 362 us for one qubit, 365 -> 393 for two). A call on 10 to 18 qubits,
// bound by the host: 9.5-10.4 us with an upload of the matrix, 6.7-7.8 us so. (A
// body shared with k_fused_vec makes that one's code for 4 and 5 qubits complex64
// an eighth longer.)
template <typename R, int K>
struct MatArg {
  R v[2 << (2 * K)];
};

template <typename R, int K, bool NT, bool PAIR>
__global__ void __launch_bounds__(kBlock) k_fused_arg(R* __restrict__ a, uint64_t groups, Block6 b,
                                                      MatArg<R, K> mat) {
  constexpr int D = 1 << K;
  __shared__ Cx<R> M[D * D];
  if (threadIdx.x < D * D) M[threadIdx.x] = {mat.v[2 * threadIdx.x], mat.v[2 * threadIdx.x + 1]};
  __syncthreads();
  for (uint64_t g = uint64_t(blockIdx.x) * kBlock + threadIdx.x; g < groups;
       g += uint64_t(gridDim.x) * kBlock) {
    uint64_t base = g;
#pragma unroll
    for (int j = 0; j < K; ++j) base = insert_zero(base, b.sorted[j]);
    uint64_t off[D];
    Cx<R> v[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      uint64_t o = 0;
#pragma unroll
      for (int j = 0; j < K; ++j) o |= uint64_t((c >> j) & 1) << b.q[j];
      off[c] = base | o;
    }
    load_group<R, K, NT, PAIR>(a, off, v);
    R lr = 0, li = 0;  // the even row of a pair
#pragma unroll
    for (int r = 0; r < D; ++r) {
      if constexpr (sizeof(R) == 8) asm volatile("" ::: "memory");  // as above
      R yr = 0, yi = 0;
#pragma unroll
      for (int c = 0; c < D; ++c) {
        const Cx<R> m = M[r * D + c];
        yr = fmadd(m.r, v[c].r, fmadd(-m.i, v[c].i, yr));
        yi = fmadd(m.r, v[c].i, fmadd(m.i, v[c].r, yi));
      }
      if constexpr (PAIR) {
        if (r & 1)
          st16<NT>(reinterpret_cast<float4*>(a + 2 * off[r & ~1]), float4{lr, li, yr, yi});
        lr = yr;
        li = yi;
      } else {
        st_amp<NT>(a + 2 * off[r], yr, yi);
      }
    }
  }
}

// Blocks of 4 to 6 qubits on states below a matrix-core tile (at most 2^11
// amplitudes): state and matrix in the LDS of one workgroup, one thread per
// output amplitude (two at 2^11). A thread per group, as above, leaves 8 to 128
// threads with chains of 256 to 4096 products. The rows of a group are on
// consecutive lanes: an input amplitude is a broadcast, and entry (r, c) of the
// matrix at r D + (c ^ r) keeps a column's reads on different banks. Sums run
// over c in the vector kernel's order. 9 qubits complex64, k = 4, 5, 6: 7.8, 22.6,
// 94 -> 6.6, 6.2, 8.1 us, 11 qubits -, 22, 95 -> -, 8.1, 12.4; 10 qubits
// complex128 -, 18, 165 -> -, 6.8, 11.2.
constexpr int kSmallThreads = 1024;
template <typename R, int K>
__global__ void __launch_bounds__(kSmallThreads) k_fused_small(R* __restrict__ a, int n, Block6 b,
                                                               const R* __restrict__ mat) {
  constexpr int D = 1 << K;
  extern __shared__ __align__(16) unsigned char small_lds[];
  Cx<R>* M = reinterpret_cast<Cx<R>*>(small_lds);
  Cx<R>* x = M + D * D;
  const int N = 1 << n;
  for (int e = threadIdx.x; e < N; e += kSmallThreads) x[e] = reinterpret_cast<const Cx<R>*>(a)[e];
  for (int e = threadIdx.x; e < D * D; e += kSmallThreads)
    M[(e & ~(D - 1)) | ((e ^ (e >> K)) & (D - 1))] = reinterpret_cast<const Cx<R>*>(mat)[e];
  __syncthreads();
  for (int o = threadIdx.x; o < N; o += kSmallThreads) {
    const int r = o & (D - 1);
    int base = o >> K, bit[K], at = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) base = int(insert_zero(base, b.sorted[j]));
#pragma unroll
    for (int j = 0; j < K; ++j) {
      bit[j] = 1 << b.q[j];
      at |= r >> j & 1 ? bit[j] : 0;
    }
    R yr = 0, yi = 0;
#pragma unroll 8
    for (int c = 0; c < D; ++c) {
      int t = base;
#pragma unroll
      for (int j = 0; j < K; ++j) t |= c >> j & 1 ? bit[j] : 0;
      const Cx<R> m = M[(r << K) | (c ^ r)], v = x[t];
      yr = fmadd(m.r, v.r, fmadd(-m.i, v.i, yr));
      yi = fmadd(m.r, v.i, fmadd(m.i, v.r, yi));
    }
    reinterpret_cast<Cx<R>*>(a)[base | at] = {yr, yi};
  }
}

template <typename R, int K>
hipError_t launch_small_state(R* a, int n, const Block6& b, const R* mat, hipStream_t s) {
  const size_t bytes = ((size_t(1) << (2 * K)) + (size_t(1) << n)) * sizeof(Cx<R>);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_fused_small<R, K>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  hipLaunchKernelGGL((k_fused_small<R, K>), dim3(1), dim3(kSmallThreads), bytes, s, a, n, b, mat);
  return hipGetLastError();
}

unsigned fused_grid(uint64_t groups) {
  const uint64_t want = (groups + kBlock - 1) / kBlock, cap = uint64_t(1) << 20;
  return static_cast<unsigned>(want < cap ? (want > 0 ? want : 1) : cap);
}

// pair (complex64): where amplitudes are swept in pairs, rows are exchanged so
// that bit 0 comes first. That is blocks of one or three qubits with bit 0, and
// of two on bits 0 and 1: 24 qubits k = 2 52-55 -> 38 us, k = 3 on bits 0-2 92 ->
// 55, 27 qubits 431 -> 377 and 716 -> 449; k = 2 with bit 0 and a higher one
// loses above the last-level cache (27 qubits 362 -> 390 us).
Block6 make_block(const int* qubits, int k, bool pair) {
  Block6 b{};
  b.k = k;
  b.p0 = -1;
  for (int j = 0; j < k; ++j) {
    b.q[j] = b.sorted[j] = qubits[j];
    if (qubits[j] == 0) b.p0 = j;
  }
  for (int i = 1; i < k; ++i)
    for (int j = i; j > 0 && b.sorted[j - 1] > b.sorted[j]; --j) {
      const int t = b.sorted[j];
      b.sorted[j] = b.sorted[j - 1];
      b.sorted[j - 1] = t;
    }
  if (!pair || k > 3 || (k == 2 && b.sorted[1] != 1)) b.p0 = -1;
  if (b.p0 > 0) {
    b.q[b.p0] = b.q[0];
    b.q[0] = 0;
  }
  return b;
}

template <typename R, int K>
hipError_t launch_arg(R* a, int n, const Block6& b, const double* m, hipStream_t s) {
  MatArg<R, K> mat;
  constexpr int D = 1 << K;
  for (int e = 0; e < D * D; ++e) {
    const int f = unswap(e / D, b.p0) * D + unswap(e % D, b.p0);
    mat.v[2 * e] = static_cast<R>(m[2 * f]);
    mat.v[2 * e + 1] = static_cast<R>(m[2 * f + 1]);
  }
  const uint64_t groups = uint64_t(1) << (n - K);
  const bool nt = stream_sweep(n, 2 * sizeof(R), b.sorted[0]);
  auto kern = nt ? k_fused_arg<R, K, true, false> : k_fused_arg<R, K, false, false>;
  if constexpr (sizeof(R) == 4)
    if (b.p0 >= 0) kern = nt ? k_fused_arg<R, K, true, true> : k_fused_arg<R, K, false, true>;
  hipLaunchKernelGGL(kern, dim3(fused_grid(groups)), dim3(kBlock), 0, s, a, groups, b, mat);
  return hipGetLastError();
}

template <typename R, int K>
hipError_t launch_k(R* a, int n, const Block6& b, const R* mat, hipStream_t s) {
  const uint64_t groups = uint64_t(1) << (n - K);
  const bool nt = stream_sweep(n, 2 * sizeof(R), b.sorted[0]);
  auto kern = nt ? k_fused_vec<R, K, true, false> : k_fused_vec<R, K, false, false>;
  if constexpr (sizeof(R) == 4 && K <= 3)
    if (b.p0 >= 0) kern = nt ? k_fused_vec<R, K, true, true> : k_fused_vec<R, K, false, true>;
  hipLaunchKernelGGL(kern, dim3(fused_grid(groups)), dim3(kBlock), 0, s, a, groups, b, mat);
  return hipGetLastError();
}

}  // namespace

template <typename R>
hipError_t launch_apply_small(R* a, int n, const int* qubits, int k, const double* host_mat,
                              hipStream_t s) {
  const Block6 b = make_block(qubits, k, sizeof(R) == 4);
  switch (k) {
    case 1: return launch_arg<R, 1>(a, n, b, host_mat, s);
    case 2: return launch_arg<R, 2>(a, n, b, host_mat, s);
    case 3: return launch_arg<R, 3>(a, n, b, host_mat, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename R>
hipError_t launch_small_block(R* a, int n, const int* qubits, int k, const R* mat, hipStream_t s) {
  if (n > 11 || k > n) return hipErrorInvalidValue;
  const Block6 b = make_block(qubits, k, false);
  switch (k) {
    case 1: return launch_small_state<R, 1>(a, n, b, mat, s);
    case 2: return launch_small_state<R, 2>(a, n, b, mat, s);
    case 3: return launch_small_state<R, 3>(a, n, b, mat, s);
    case 4: return launch_small_state<R, 4>(a, n, b, mat, s);
    case 5: return launch_small_state<R, 5>(a, n, b, mat, s);
    case 6: return launch_small_state<R, 6>(a, n, b, mat, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename R>
hipError_t launch_apply_fused(R* a, int n, const int* qubits, int k, const R* mat,
                              hipStream_t s) {
  if (k >= 4 && n <= 11) return launch_small_block(a, n, qubits, k, mat, s);
  const Block6 b = make_block(qubits, k, sizeof(R) == 4);
  switch (k) {
    case 1: return launch_k<R, 1>(a, n, b, mat, s);
    case 2: return launch_k<R, 2>(a, n, b, mat, s);
    case 3: return launch_k<R, 3>(a, n, b, mat, s);
    case 4: return launch_k<R, 4>(a, n, b, mat, s);
    case 5: return launch_k<R, 5>(a, n, b, mat, s);
    case 6: return launch_k<R, 6>(a, n, b, mat, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_small_block<float>(float*, int, const int*, int, const float*,
                                              hipStream_t);
template hipError_t launch_small_block<double>(double*, int, const int*, int, const double*,
                                               hipStream_t);
template hipError_t launch_apply_fused<float>(float*, int, const int*, int, const float*,
                                              hipStream_t);
template hipError_t launch_apply_small<float>(float*, int, const int*, int, const double*,
                                              hipStream_t);
template hipError_t launch_apply_small<double>(double*, int, const int*, int, const double*,
                                               hipStream_t);
template hipError_t launch_apply_fused<double>(double*, int, const int*, int, const double*,
                                               hipStream_t);

}  // namespace qs
