// Tile passes of a planned circuit: one HBM read and write of the ket for all
// the gates of a pass.
//
// A tile is 2^(C+H) amplitudes: the contiguous low bits [0, C) (rows of 2^C
// amplitudes) and H = 7 row bits chosen by the planner (complex64: C = 5 by
// default, 256-byte rows and 32 KiB tiles, 4 or 6 by knob; complex128: C = 4,
// 256-byte rows, 32 KiB). The tile is staged
// in LDS and transformed round by round, each round acting on 4 tile bits.
// Three forms of rounds, of which a pass takes the one whose rounds cost less:
// two two-qubit gates in fixed places (k_tile_pair; on the FP32 matrix cores in
// complex64, with FP64 FMAs in complex128); a dense 4-qubit block on the matrix
// cores (k_tile_mfma, complex64; passes with gates of three or four qubits, and
// those whose gates stay on few qubits), each complex product as three real ones
// (Re U X_r, Im U X_i and (Re U + Im U)(X_r + X_i), 16 x 16 x 4 MFMAs: 3/4 of the
// flops of the 32 x 32 real embedding); one- and two-qubit gates one by one in
// registers (k_tile_pass: complex128 passes whose gates stay on few qubits, runs
// of one-qubit gates on factorized kets, and complex64 with tile.mfma 0).
#include "qs_internal.h"

namespace qs {
namespace {

constexpr int kW = 4;
constexpr int kV = 1 << kW;  // amplitudes per thread in a round

template <typename R> struct Cx { R r, i; };
template <typename R> struct Vec16;
template <> struct Vec16<float> { using T = float4; static constexpr int AMPS = 2; };
template <> struct Vec16<double> { using T = double2; static constexpr int AMPS = 1; };

__device__ __forceinline__ uint64_t insert_zero(uint64_t x, int pos) {
  const uint64_t lo = x & ((uint64_t(1) << pos) - 1);
  return lo | ((x ^ lo) << 1);
}
constexpr __device__ __forceinline__ int lds_pos(int x) { return x + (x >> 4); }

template <typename R>
__device__ __forceinline__ Cx<R> cmac(Cx<R> acc, Cx<R> a, Cx<R> b) {
  return {fmadd(a.r, b.r, fmadd(-a.i, b.i, acc.r)), fmadd(a.r, b.i, fmadd(a.i, b.r, acc.i))};
}

// 2x2 matrix (row-major, interleaved) on round bit J.
template <typename R, int J>
__device__ __forceinline__ void apply1(Cx<R> (&v)[kV], const R* __restrict__ m) {
  const Cx<R> m00{m[0], m[1]}, m01{m[2], m[3]}, m10{m[4], m[5]}, m11{m[6], m[7]};
#pragma unroll
  for (int x = 0; x < kV; ++x) {
    if (x & (1 << J)) continue;
    const Cx<R> a = v[x], b = v[x | (1 << J)];
    v[x] = cmac(cmac(Cx<R>{0, 0}, m00, a), m01, b);
    v[x | (1 << J)] = cmac(cmac(Cx<R>{0, 0}, m10, a), m11, b);
  }
}

// 4x4 matrix: row/column bit 0 on round bit J1, bit 1 on round bit J2.
template <typename R, int J1, int J2>
__device__ __forceinline__ void apply2(Cx<R> (&v)[kV], const R* __restrict__ m) {
  Cx<R> M[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) M[e] = {m[2 * e], m[2 * e + 1]};
#pragma unroll
  for (int x = 0; x < kV; ++x) {
    if (x & ((1 << J1) | (1 << J2))) continue;
    int idx[4];
    Cx<R> in[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      idx[c] = x | ((c & 1) << J1) | ((c >> 1) << J2);
      in[c] = v[idx[c]];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      Cx<R> y{0, 0};
#pragma unroll
      for (int c = 0; c < 4; ++c) y = cmac(y, M[4 * r + c], in[c]);
      v[idx[r]] = y;
    }
  }
}

template <typename R>
__device__ __forceinline__ void apply_gate(Cx<R> (&v)[kV], int code, const R* __restrict__ m) {
  const int kind = code & 15, j1 = (code >> 4) & 15, j2 = (code >> 8) & 15;
  if (kind == 1) {
    switch (j1) {
      case 0: apply1<R, 0>(v, m); break;
      case 1: apply1<R, 1>(v, m); break;
      case 2: apply1<R, 2>(v, m); break;
      default: apply1<R, 3>(v, m); break;
    }
    return;
  }
  switch (j1 * 4 + j2) {
    case 1: apply2<R, 0, 1>(v, m); break;
    case 2: apply2<R, 0, 2>(v, m); break;
    case 3: apply2<R, 0, 3>(v, m); break;
    case 4: apply2<R, 1, 0>(v, m); break;
    case 6: apply2<R, 1, 2>(v, m); break;
    case 7: apply2<R, 1, 3>(v, m); break;
    case 8: apply2<R, 2, 0>(v, m); break;
    case 9: apply2<R, 2, 1>(v, m); break;
    case 11: apply2<R, 2, 3>(v, m); break;
    case 12: apply2<R, 3, 0>(v, m); break;
    case 13: apply2<R, 3, 1>(v, m); break;
    default: apply2<R, 3, 2>(v, m); break;
  }
}

// The rounds of a tile staged in LDS (thread x: group x of each round).
template <typename R>
__device__ __forceinline__ void gate_rounds(Cx<R>* sm, const int4* __restrict__ rounds, int nrounds,
                                            const int2* __restrict__ gates,
                                            const R* __restrict__ mats) {
  for (int r = 0; r < nrounds; ++r) {
    const int4 rd = rounds[r];
    const int b0 = rd.x & 255, b1 = (rd.x >> 8) & 255, b2 = (rd.x >> 16) & 255,
              b3 = (rd.x >> 24) & 255;
    int x0 = threadIdx.x;
    x0 = int(insert_zero(uint64_t(x0), b0));
    x0 = int(insert_zero(uint64_t(x0), b1));
    x0 = int(insert_zero(uint64_t(x0), b2));
    x0 = int(insert_zero(uint64_t(x0), b3));
    int pos[kV];
    Cx<R> v[kV];
#pragma unroll
    for (int m = 0; m < kV; ++m) {
      pos[m] = lds_pos(x0 | ((m & 1) << b0) | (((m >> 1) & 1) << b1) | (((m >> 2) & 1) << b2) |
                       (((m >> 3) & 1) << b3));
      v[m] = sm[pos[m]];
    }
    for (int g = rd.y; g < rd.y + rd.z; ++g) {
      const int2 gg = gates[g];
      apply_gate<R>(v, gg.x, mats + gg.y);
    }
#pragma unroll
    for (int m = 0; m < kV; ++m) sm[pos[m]] = v[m];
    __syncthreads();
  }
}

template <typename R, int C, int H, bool STREAM>
__global__ void __launch_bounds__(1 << (C + H - kW))
    k_tile_pass(R* __restrict__ a, TileRows rows, const int4* __restrict__ rounds, int nrounds,
                const int2* __restrict__ gates, const R* __restrict__ mats) {
  constexpr int TB = C + H;
  constexpr int NT = 1 << (TB - kW);
  using V = typename Vec16<R>::T;
  constexpr int AP = Vec16<R>::AMPS;
  constexpr int VPR = (1 << C) / AP;       // 16-byte vectors per row
  constexpr int NV = (1 << TB) / AP / NT;  // vectors per thread
  extern __shared__ unsigned char smraw[];
  Cx<R>* sm = reinterpret_cast<Cx<R>*>(smraw);
  // tile base: the workgroup index spread over the bits outside the tile
  uint64_t base = uint64_t(blockIdx.x) << C;
#pragma unroll
  for (int j = 0; j < H; ++j) base = insert_zero(base, rows.b[j]);
  auto glob = [&](int row, int col) {
    uint64_t g = base | uint64_t(col);
#pragma unroll
    for (int j = 0; j < H; ++j) g |= uint64_t((row >> j) & 1) << rows.b[j];
    return g;
  };
  V* p = reinterpret_cast<V*>(a);
  V buf[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    buf[k] = ld16<STREAM>(p + glob(e / VPR, (e % VPR) * AP) / AP);
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const int x = ((e / VPR) << C) | (e % VPR) * AP;
    if constexpr (AP == 2) {
      sm[lds_pos(x)] = {buf[k].x, buf[k].y};
      sm[lds_pos(x + 1)] = {buf[k].z, buf[k].w};
    } else {
      sm[lds_pos(x)] = {buf[k].x, buf[k].y};
    }
  }
  __syncthreads();
  gate_rounds<R>(sm, rounds, nrounds, gates, mats);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const int x = ((e / VPR) << C) | (e % VPR) * AP;
    V o;
    const Cx<R> v0 = sm[lds_pos(x)];
    if constexpr (AP == 2) {
      const Cx<R> v1 = sm[lds_pos(x + 1)];
      o = {v0.r, v0.i, v1.r, v1.i};
    } else {
      o = {v0.r, v0.i};
    }
    st16<STREAM>(p + glob(e / VPR, (e % VPR) * AP) / AP, o);
  }
}

// ---- rounds of two two-qubit gates on the FP32 matrix cores
// Thread x owns one group of a round, its 16 amplitudes in registers; the
// round's first gate acts on bits 0 and 1 of the group, the second on bits 2
// and 3, each a 4 x 4 complex matrix on four quadruples. v_mfma_f32_4x4x1_16b
// multiplies, in each block of four lanes, a column of a 4 x 4 matrix (lane i
// of the block supplies row i) by the block's row of four inputs (lane j
// supplies its own amplitude) and leaves row r of the product in result
// register r of the lane it belongs to: one instruction adds an amplitude's
// products into its four outputs for 64 groups and nothing crosses lanes. The
// four registers of a first-gate result are inputs of four second-gate
// quadruples, so no register moves.
//
// Two-qubit gates fill a random circuit, and a dense 16 x 16 round holding two
// of them spends 48 instructions of 32 cycles (38.6 measured) on what takes 128 of
// 8 (10.4) here; the vector instructions share the FP32 matrix unit (a loop of
// both takes the sum of their times), so a round's other instructions count as
// much: the tile is kept as a plane of real and a plane of imaginary parts, which load and store
// without packing moves, and the loop runs two rounds at a time so that
// prefetched matrix rows need no copies. 8-layer circuits against the dense
// rounds: 37.7 -> 27.9 us at 12 qubits, 119 -> 99 at 20, 861 -> 709 at 24
// (states in the last-level cache; the passes alone 353), 16.8 -> 14.3 ms at
// 28 (11.7).
typedef float f32x4 __attribute__((ext_vector_type(4)));

// y = U x on four quadruples for a complex U, of which this lane holds row
// lane % 4 (u: its entries, interleaved); x(h, c) is input c of quadruple h,
// output row i of it is (yr[h][i], yi[h][i]).
template <typename In>
__device__ __forceinline__ void pair_gate(const float4 (&u)[2], In x, f32x4 (&yr)[4],
                                          f32x4 (&yi)[4]) {
  const float ur[4] = {u[0].x, u[0].z, u[1].x, u[1].z}, ui[4] = {u[0].y, u[0].w, u[1].y, u[1].w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float nim = -ui[c];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const float2 v = x(h, c);
      const f32x4 r = c ? yr[h] : f32x4{}, i = c ? yi[h] : f32x4{};
      yr[h] = __builtin_amdgcn_mfma_f32_4x4x1f32(ur[c], v.x, r, 0, 0, 0);
      yi[h] = __builtin_amdgcn_mfma_f32_4x4x1f32(ur[c], v.y, i, 0, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const float2 v = x(h, c);
      yr[h] = __builtin_amdgcn_mfma_f32_4x4x1f32(nim, v.y, yr[h], 0, 0, 0);
      yi[h] = __builtin_amdgcn_mfma_f32_4x4x1f32(ui[c], v.x, yi[h], 0, 0, 0);
    }
  }
}
__device__ __forceinline__ int insert_zero32(int x, int pos) {
  const int lo = x & ((1 << pos) - 1);
  return lo | ((x ^ lo) << 1);
}

// Dword of tile index x in a plane of the LDS tile (one dword of padding every
// 32), and the length of a plane (a multiple of 64).
constexpr __device__ __forceinline__ int plane_pos(int x) { return x + (x >> 5); }
template <int TB> constexpr int kPlane = (1 << TB) + ((1 << TB) >> 5) + 63 & ~63;

// LDS offsets of a group's 16 amplitudes in a round of a tile whose entry of
// index x is POS(x), additive over disjoint bits: thread x's group of the round
// with these bits (in the order of its gates, and ascending).
template <int (*POS)(int)>
struct GroupPos {
  int px, d[4];
  __device__ __forceinline__ GroupPos(int bits, int asc) {
    int x0 = threadIdx.x;
#pragma unroll
    for (int j = 0; j < 4; ++j) x0 = insert_zero32(x0, (asc >> (8 * j)) & 255);
    px = POS(x0);
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = POS(1 << ((bits >> (8 * j)) & 255));
  }
  __device__ __forceinline__ int operator()(int m) const {
    return px + ((m & 1) ? d[0] : 0) + ((m & 2) ? d[1] : 0) + ((m & 4) ? d[2] : 0) +
           ((m & 8) ? d[3] : 0);
  }
};

// The complex64 rounds of a tile staged in LDS (thread x: group x of each
// round). A round's entry is loaded two rounds ahead, its matrix rows one
// ahead; the first ones when the object is made, before the tile's own loads.
struct PairRounds {
  struct Round {
    int bits, asc, flags;
    float4 m1[2], m2[2];  // this lane's row of the first and second gate
  };
  const int4* __restrict__ rounds;
  int nrounds;
  const float* __restrict__ num;
  int4 next;
  Round ra;

  __device__ __forceinline__ int4 entry(int r) const {
    return rounds[r < nrounds ? r : nrounds - 1];
  }
  __device__ __forceinline__ Round load_round(int4 e) const {
    const float* row = num + 8 * (threadIdx.x & 3);
    const int second = e.z + ((e.w & 1) ? 32 : 0);  // none: the first one's row again
    auto q = [&](int off) { return *reinterpret_cast<const float4*>(row + off); };
    return Round{e.x, e.y, e.w, {q(e.z), q(e.z + 4)}, {q(second), q(second + 4)}};
  }
  __device__ __forceinline__ PairRounds(const int4* __restrict__ r, int n,
                                        const float* __restrict__ numbers)
      : rounds(r), nrounds(n), num(numbers) {
    next = entry(1);
    ra = load_round(entry(0));
  }
  __device__ __forceinline__ void step(const Round& rd, float* re, float* im) const {
    const GroupPos<plane_pos> at(rd.bits, rd.asc);
    float2 v[kV];
#pragma unroll
    for (int m = 0; m < kV; ++m) v[m] = make_float2(re[at(m)], im[at(m)]);
    f32x4 yr[4], yi[4];
    pair_gate(rd.m1, [&](int h, int c) { return v[4 * h + c]; }, yr, yi);
    if (rd.flags & 1) {
      f32x4 zr[4], zi[4];
      pair_gate(rd.m2, [&](int l, int c) { return make_float2(yr[c][l], yi[c][l]); }, zr, zi);
#pragma unroll
      for (int m = 0; m < kV; ++m) re[at(m)] = zr[m & 3][m >> 2], im[at(m)] = zi[m & 3][m >> 2];
    } else {
#pragma unroll
      for (int m = 0; m < kV; ++m) re[at(m)] = yr[m >> 2][m & 3], im[at(m)] = yi[m >> 2][m & 3];
    }
    __syncthreads();
  }
  template <typename Step>
  __device__ __forceinline__ void run(Step step) {
    for (int r = 0; r < nrounds; r += 2) {  // two by two: the rows need no copies
      const Round rb = load_round(next);
      next = entry(r + 2);
      step(ra);
      if (r + 1 == nrounds) break;
      ra = load_round(next);
      next = entry(r + 3);
      step(rb);
    }
  }
  __device__ __forceinline__ void run(float* re, float* im) {
    run([this, re, im](const Round& rd) { step(rd, re, im); });
  }
};

// LDS entry of index x of a complex128 tile: 8 lanes of 16-byte entries fill
// the banks, so the padding follows every 8 entries (every 16: 3% slower).
constexpr __host__ __device__ __forceinline__ int wide_pos(int x) { return x + (x >> 3); }

// Complex128 rounds on vector FMA (the FP64 matrix rate is the vector rate),
// the numbers read through the scalar cache. FMAs bound them; a round is two
// gates in fixed places, 4 KB of code, where k_tile_pass selects among twelve
// forms by a switch (28 KB, fetched anew by every launch for the two or three
// rounds a small state has). 8-layer circuits with its rounds and with these:
// 44.9 -> 37.2 us at 11 qubits, 204 -> 187 at 20, 1.71 -> 1.62 ms at 24. (Taking
// each gate as phases times a real matrix, 5/8 of the FMAs, gained 5% more but
// with 1.4 times the error against 64 bits.)
__device__ __forceinline__ void pair_gate_f64(Cx<double> (&v)[kV], int s, int t,
                                              const double* __restrict__ u) {
  // quadruple h: entries t h + s c
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    Cx<double> in[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) in[c] = v[t * h + s * c];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      Cx<double> y{0, 0};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        y = cmac(y, Cx<double>{u[2 * (4 * r + c)], u[2 * (4 * r + c) + 1]}, in[c]);
      v[t * h + s * r] = y;
    }
  }
}

__device__ __forceinline__ void pair_rounds_f64(Cx<double>* sm, const int4* __restrict__ rounds,
                                                int nrounds, const double* __restrict__ num) {
  int4 e = rounds[0];
  for (int r = 0; r < nrounds; ++r) {
    const int4 next = rounds[r + 1 < nrounds ? r + 1 : r];
    const double* __restrict__ u = num + e.z;
    const GroupPos<wide_pos> at(e.x, e.y);
    Cx<double> v[kV];
#pragma unroll
    for (int m = 0; m < kV; ++m) v[m] = sm[at(m)];
    pair_gate_f64(v, 1, 4, u);
    if (e.w & 1) pair_gate_f64(v, 4, 1, u + 32);
#pragma unroll
    for (int m = 0; m < kV; ++m) sm[at(m)] = v[m];
    e = next;
    __syncthreads();
  }
}

// BOUND: the state may be smaller than the tile (base 0, row bits on from C);
// indices from `amps` on are zeros and stay out of memory.
template <int C, int H, bool STREAM, bool BOUND = false>
__device__ __forceinline__ void tile_pair_body(float* __restrict__ a, uint64_t base,
                                               const TileRows& rows,
                                               const int4* __restrict__ rounds, int nrounds,
                                               const float* __restrict__ mats,
                                               uint64_t amps = 0) {
  constexpr int TB = C + H;
  constexpr int NT = 1 << (TB - kW);
  constexpr int VPR = (1 << C) / 2;        // float4 vectors per row
  constexpr int NV = (1 << TB) / 2 / NT;   // vectors per thread
  constexpr int RT = NT / VPR;             // tile rows between a thread's vectors
  constexpr int RTB = __builtin_ctz(RT);
  static_assert(RT * VPR == NT && RTB <= H, "tile shape");
  extern __shared__ unsigned char smraw[];
  float* re = reinterpret_cast<float*>(smraw);  // real parts, then imaginary ones
  float* im = re + kPlane<TB>;
  const int r0 = int(threadIdx.x) / VPR;
  uint64_t off_t = base | uint64_t((int(threadIdx.x) % VPR) * 2);
#pragma unroll
  for (int j = 0; j < RTB; ++j) off_t |= uint64_t((r0 >> j) & 1) << rows.b[j];
  auto glob_k = [&](int k) {
    uint64_t g = off_t;
#pragma unroll
    for (int j = RTB; j < H; ++j)
      if (((k * RT) >> j) & 1) g |= uint64_t(1) << rows.b[j];
    return g;
  };
  float4* p4 = reinterpret_cast<float4*>(a);
  PairRounds rr(rounds, nrounds, mats);
  {
    float4 buf[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k)
      buf[k] = !BOUND || glob_k(k) < amps ? ld16<STREAM>(p4 + glob_k(k) / 2)
                                          : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int e = threadIdx.x + k * NT;
      const int x = ((e / VPR) << C) | (e % VPR) * 2;
      re[plane_pos(x)] = buf[k].x;
      im[plane_pos(x)] = buf[k].y;
      re[plane_pos(x) + 1] = buf[k].z;
      im[plane_pos(x) + 1] = buf[k].w;
    }
  }
  __syncthreads();
  rr.run(re, im);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const int x = ((e / VPR) << C) | (e % VPR) * 2;
    const int l = plane_pos(x);
    if (!BOUND || glob_k(k) < amps)
      st16<STREAM>(p4 + glob_k(k) / 2, make_float4(re[l], im[l], re[l + 1], im[l + 1]));
  }
}

// The same pass in complex128.
template <int C, int H, bool STREAM, bool BOUND = false>
__device__ __forceinline__ void tile_pair_body(double* __restrict__ a, uint64_t base,
                                               const TileRows& rows,
                                               const int4* __restrict__ rounds, int nrounds,
                                               const double* __restrict__ num,
                                               uint64_t amps = 0) {
  constexpr int TB = C + H, NT = 1 << (TB - kW), NV = (1 << TB) / NT;
  constexpr int RT = NT >> C, RTB = __builtin_ctz(RT);  // tile rows between a thread's entries
  extern __shared__ unsigned char smraw[];
  Cx<double>* sm = reinterpret_cast<Cx<double>*>(smraw);
  const int r0 = int(threadIdx.x) >> C;
  uint64_t off_t = base | (threadIdx.x & ((1 << C) - 1));
#pragma unroll
  for (int j = 0; j < RTB; ++j) off_t |= uint64_t((r0 >> j) & 1) << rows.b[j];
  auto glob_k = [&](int k) {
    uint64_t g = off_t;
#pragma unroll
    for (int j = RTB; j < H; ++j)
      if (((k * RT) >> j) & 1) g |= uint64_t(1) << rows.b[j];
    return g;
  };
  double2* p2 = reinterpret_cast<double2*>(a);
  double2 buf[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k)
    buf[k] = !BOUND || glob_k(k) < amps ? ld16<STREAM>(p2 + glob_k(k)) : make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < NV; ++k) sm[wide_pos(threadIdx.x + k * NT)] = {buf[k].x, buf[k].y};
  __syncthreads();
  pair_rounds_f64(sm, rounds, nrounds, num);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const Cx<double> x = sm[wide_pos(threadIdx.x + k * NT)];
    if (!BOUND || glob_k(k) < amps) st16<STREAM>(p2 + glob_k(k), make_double2(x.r, x.i));
  }
}

template <typename R> constexpr int kPairWaves = sizeof(R) == 4 ? 4 : 2;  // per SIMD, by registers
// LDS bytes of a tile of pair rounds
template <typename R, int TB>
constexpr size_t pair_lds() {
  return sizeof(R) == 4 ? 2 * size_t(kPlane<TB>) * 4 : size_t(wide_pos(1 << TB)) * 16;
}

template <typename R, int C, int H, bool STREAM>
__global__ void __launch_bounds__(1 << (C + H - kW))
__attribute__((amdgpu_waves_per_eu(kPairWaves<R>)))
    k_tile_pair(R* __restrict__ a, TileRows rows, const int4* __restrict__ rounds, int nrounds,
                const R* __restrict__ num) {
  uint64_t base = uint64_t(blockIdx.x) << C;
#pragma unroll
  for (int j = 0; j < H; ++j) base = insert_zero(base, rows.b[j]);
  tile_pair_body<C, H, STREAM>(a, base, rows, rounds, nrounds, num);
}

// ---- states that fit one tile with room to spare
// A state of n <= TB qubits whole in the LDS of one workgroup, every gate of
// the circuit in one launch; indices from 2^n on are zeros that no gate moves.
// Fused blocks, one launch each, are the alternative (8 layers at 11 qubits 112
// us in 14 blocks). One workgroup leaves nothing to hide latency with, so a
// thread owns the four amplitudes of one gate's group and not the 16 of a
// round's: four times the wavefronts, each with a quarter of the chain, for one
// more barrier per round. The products and their order are those of the pair
// rounds. 8 layers with 16 amplitudes per thread and with four: complex64 at 6,
// 8, 10 and 11 qubits 13.8, 16.8, 23.8, 23.3 -> 10.9, 13.0, 17.9, 19.7 us,
// complex128 at 6, 8 and 10 21.5, 26.9, 38.2 -> 15.1, 19.8, 27.0.
struct QuadPos {  // LDS offsets of thread x's group of a gate on tile bits b0, b1
  int px, d0, d1;
  template <typename Pos>
  __device__ __forceinline__ QuadPos(int b0, int b1, Pos pos) {
    const int x0 = insert_zero32(insert_zero32(threadIdx.x, min(b0, b1)), max(b0, b1));
    px = pos(x0);
    d0 = pos(1 << b0);
    d1 = pos(1 << b1);
  }
  __device__ __forceinline__ int operator()(int m) const {
    return px + ((m & 1) ? d0 : 0) + ((m & 2) ? d1 : 0);
  }
};

__device__ __forceinline__ void quad_gate(const float4 (&u)[2], int b0, int b1, float* re,
                                          float* im) {
  const QuadPos at(b0, b1, [](int x) { return plane_pos(x); });
  const float ur[4] = {u[0].x, u[0].z, u[1].x, u[1].z}, ui[4] = {u[0].y, u[0].w, u[1].y, u[1].w};
  float2 v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = make_float2(re[at(c)], im[at(c)]);
  f32x4 yr{}, yi{};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    yr = __builtin_amdgcn_mfma_f32_4x4x1f32(ur[c], v[c].x, yr, 0, 0, 0);
    yi = __builtin_amdgcn_mfma_f32_4x4x1f32(ur[c], v[c].y, yi, 0, 0, 0);
    yr = __builtin_amdgcn_mfma_f32_4x4x1f32(-ui[c], v[c].y, yr, 0, 0, 0);
    yi = __builtin_amdgcn_mfma_f32_4x4x1f32(ui[c], v[c].x, yi, 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) re[at(c)] = yr[c], im[at(c)] = yi[c];
  __syncthreads();
}

// Bit q of a circuit's positions is bit (bits >> 4 q) & 15 of the state's index,
// and bit 0 of the latter is bit `first` of the former. (Packed: an array would
// be read bit by bit through the scalar cache.)
struct WholePerm {
  uint64_t bits;
  int first;
};
// The tile index of a state's index i.
template <int TB>
__device__ __forceinline__ int whole_pos(int i, const WholePerm& perm) {
  int x = 0;
#pragma unroll
  for (int q = 0; q < TB; ++q) x |= ((i >> int((perm.bits >> (4 * q)) & 15)) & 1) << q;
  return x;
}

template <int TB>
__global__ void __launch_bounds__(1 << (TB - 2))
    k_whole_pair(float* __restrict__ a, int n, WholePerm perm, const int4* __restrict__ rounds,
                 int nrounds, const float* __restrict__ mats) {
  constexpr int NT = 1 << (TB - 2), NV = (1 << TB) / 2 / NT;
  extern __shared__ unsigned char smraw[];
  float* re = reinterpret_cast<float*>(smraw);
  float* im = re + kPlane<TB>;
  float4* p4 = reinterpret_cast<float4*>(a);
  const int vecs = 1 << (n - 1);
  PairRounds rr(rounds, nrounds, mats);
  int at[NV][2];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const float4 b = e < vecs ? p4[e] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int x = whole_pos<TB>(2 * e, perm);
    at[k][0] = plane_pos(x);
    at[k][1] = plane_pos(x | (1 << perm.first));
    re[at[k][0]] = b.x;
    im[at[k][0]] = b.y;
    re[at[k][1]] = b.z;
    im[at[k][1]] = b.w;
  }
  __syncthreads();
  rr.run([re, im](const PairRounds::Round& rd) {
    quad_gate(rd.m1, rd.bits & 255, (rd.bits >> 8) & 255, re, im);
    if (rd.flags & 1) quad_gate(rd.m2, (rd.bits >> 16) & 255, (rd.bits >> 24) & 255, re, im);
  });
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT, l = at[k][0], m = at[k][1];
    if (e < vecs) p4[e] = make_float4(re[l], im[l], re[m], im[m]);
  }
}

__device__ __forceinline__ void quad_gate_f64(Cx<double>* sm, int b0, int b1,
                                              const double* __restrict__ u) {
  const QuadPos at(b0, b1, [](int x) { return wide_pos(x); });
  Cx<double> in[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) in[c] = sm[at(c)];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    Cx<double> y{0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c)
      y = cmac(y, Cx<double>{u[2 * (4 * r + c)], u[2 * (4 * r + c) + 1]}, in[c]);
    sm[at(r)] = y;
  }
  __syncthreads();
}

template <int TB>
__global__ void __launch_bounds__(1 << (TB - 2))
    k_whole_pair(double* __restrict__ a, int n, WholePerm perm, const int4* __restrict__ rounds,
                 int nrounds, const double* __restrict__ num) {
  constexpr int NT = 1 << (TB - 2), NV = (1 << TB) / NT;
  extern __shared__ unsigned char smraw[];
  Cx<double>* sm = reinterpret_cast<Cx<double>*>(smraw);
  double2* p2 = reinterpret_cast<double2*>(a);
  const int amps = 1 << n;
  int at[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const double2 b = e < amps ? p2[e] : make_double2(0.0, 0.0);
    at[k] = wide_pos(whole_pos<TB>(e, perm));
    sm[at[k]] = {b.x, b.y};
  }
  __syncthreads();
  int4 e = rounds[0];
  for (int r = 0; r < nrounds; ++r) {
    const int4 next = rounds[r + 1 < nrounds ? r + 1 : r];
    const double* __restrict__ u = num + e.z;
    quad_gate_f64(sm, e.x & 255, (e.x >> 8) & 255, u);
    if (e.w & 1) quad_gate_f64(sm, (e.x >> 16) & 255, (e.x >> 24) & 255, u + 32);
    e = next;
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    if (e < amps) p2[e] = make_double2(sm[at[k]].r, sm[at[k]].i);
  }
}

// Complex64 passes whose rounds are dense 4-qubit blocks on the FP32 matrix
// cores. A round multiplies the 16 amplitudes of every group (the other tile
// bits) by the round's 16 x 16 complex matrix U, as three real products on
// v_mfma_f32_16x16x4f32 (Re U X_r, Im U X_i and (Re U + Im U)(X_r + X_i)): a
// wavefront takes 16 groups at a time, lane (q, col) = (lane / 16, lane % 16)
// supplies row col of the matrices and input 4 s + q of group col in step s, and
// gets outputs 4 q + i of that group. `amats` holds each round's operands in that
// order, 12 values a lane: entry (3 s + c) 64 + lane = W_c[lane % 16][4 s + lane /
// 16] with W_0 = Re U, W_1 = Im U, W_2 = Re U + Im U.
constexpr int kOps = 12;
static_assert(kOps * 64 == kRoundOperands, "round operand layout");

// One tile of a matrix-core pass: `base` is the global index of tile entry 0
// (zeros at the low bits and the row bits), `rows` the row bits.
template <int C, int H, bool STREAM>
__device__ __forceinline__ void tile_mfma_body(float* __restrict__ a, uint64_t base,
                                               const TileRows& rows,
                                               const int4* __restrict__ rounds, int nrounds,
                                               const float* __restrict__ amats) {
  constexpr int TB = C + H;
  constexpr int NT = 1 << (TB - kW);
  constexpr int VPR = (1 << C) / 2;        // float4 vectors per row
  constexpr int NV = (1 << TB) / 2 / NT;   // vectors per thread
  constexpr int CHUNKS = (1 << (TB - kW)) / 32 / (NT / 64);  // 32-group chunks per wave
  // vector e = tid + k NT lies in tile row tid / VPR + k RT: the low row bits
  // come from the thread, the others from k (uniform across the workgroup)
  constexpr int RT = NT / VPR;
  constexpr int RTB = __builtin_ctz(RT);
  static_assert(RT * VPR == NT && RTB <= H, "tile shape");
  extern __shared__ unsigned char smraw[];
  float2* sm = reinterpret_cast<float2*>(smraw);
  const int r0 = int(threadIdx.x) / VPR;
  uint64_t off_t = base | uint64_t((int(threadIdx.x) % VPR) * 2);
#pragma unroll
  for (int j = 0; j < RTB; ++j) off_t |= uint64_t((r0 >> j) & 1) << rows.b[j];
  auto glob_k = [&](int k) {  // global index of this thread's vector k (k known at compile time)
    uint64_t g = off_t;
#pragma unroll
    for (int j = RTB; j < H; ++j)
      if (((k * RT) >> j) & 1) g |= uint64_t(1) << rows.b[j];
    return g;
  };
  float4* p4 = reinterpret_cast<float4*>(a);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, col = lane & 15;
  // this lane's part of the first round's operands, issued before the tile so
  // that its latency hides behind the tile's (the scheduling barrier keeps
  // the compiler from sinking these loads to their first use)
  float A[kOps];
#pragma unroll
  for (int k = 0; k < kOps; ++k) A[k] = amats[rounds[0].y + k * 64 + lane];
  __builtin_amdgcn_sched_barrier(0);
  {
    float4 buf[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) buf[k] = ld16<STREAM>(p4 + glob_k(k) / 2);
    // an empty use of the matrix after the tile loads are issued: it anchors
    // the matrix loads ahead of them (they complete first, in order)
#pragma unroll
    for (int k = 0; k < kOps; ++k) asm volatile("" ::"v"(A[k]));
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int e = threadIdx.x + k * NT;
      const int x = ((e / VPR) << C) | (e % VPR) * 2;
      sm[lds_pos(x)] = make_float2(buf[k].x, buf[k].y);
      sm[lds_pos(x + 1)] = make_float2(buf[k].z, buf[k].w);
    }
  }
  __syncthreads();
  for (int r = 0; r < nrounds; ++r) {
    const int4 rd = rounds[r];
    const int b0 = rd.x & 255, b1 = (rd.x >> 8) & 255, b2 = (rd.x >> 16) & 255,
              b3 = (rd.x >> 24) & 255;
    // the next round's operands are loaded while this round computes (kept
    // here by the scheduling barrier; left to itself the compiler sinks the
    // loads to the end of the round and the next round waits for them)
    float An[kOps];
    const int offn = rounds[r + 1 < nrounds ? r + 1 : r].y;
#pragma unroll
    for (int k = 0; k < kOps; ++k) An[k] = amats[offn + k * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    int dep[kV];  // LDS offset of round-local index m (the round bits and padding)
#pragma unroll
    for (int m = 0; m < kV; ++m)
      dep[m] = lds_pos(((m & 1) << b0) | (((m >> 1) & 1) << b1) | (((m >> 2) & 1) << b2) |
                       (((m >> 3) & 1) << b3));
    // lane (q, col) reads input index 4 s + q and writes output index 4 q + i;
    // lds_pos adds over disjoint bits, so these offsets are dep[4 s] + qin and
    // dep[i] + qout with per-lane qin = dep[q], qout = dep[4 q] (a
    // lane-dependent index into dep[] would compile to select chains)
    const int qin = ((q & 1) ? dep[1] : 0) + ((q & 2) ? dep[2] : 0);
    const int qout = ((q & 1) ? dep[4] : 0) + ((q & 2) ? dep[8] : 0);
#pragma unroll
    for (int ch = 0; ch < CHUNKS; ++ch) {
      int px[2];  // LDS offset of this lane's group in each 16-group block
#pragma unroll
      for (int bk = 0; bk < 2; ++bk) {
        int x0 = (wave * CHUNKS + ch) * 32 + 16 * bk + col;
        x0 = int(insert_zero(uint64_t(x0), b0));
        x0 = int(insert_zero(uint64_t(x0), b1));
        x0 = int(insert_zero(uint64_t(x0), b2));
        x0 = int(insert_zero(uint64_t(x0), b3));
        px[bk] = lds_pos(x0);
      }
      // three real 16 x 16 products per block: Re U X_r, Im U X_i,
      // (Re U + Im U)(X_r + X_i), K = 16 in 4 steps of 4
      f32x4 p1[2] = {f32x4{}, f32x4{}}, p2[2] = {f32x4{}, f32x4{}}, p3[2] = {f32x4{}, f32x4{}};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
        for (int bk = 0; bk < 2; ++bk) {
          const float2 v = sm[px[bk] + dep[4 * s4] + qin];
          p1[bk] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3 * s4], v.x, p1[bk], 0, 0, 0);
          p2[bk] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3 * s4 + 1], v.y, p2[bk], 0, 0, 0);
          p3[bk] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3 * s4 + 2], v.x + v.y, p3[bk], 0, 0,
                                                         0);
        }
      }
      // D layout: register i -> output row 4 q + i of group col;
      // Y = (p1 - p2) + i (p3 - p1 - p2)
#pragma unroll
      for (int bk = 0; bk < 2; ++bk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          sm[px[bk] + dep[i] + qout] =
              make_float2(p1[bk][i] - p2[bk][i], p3[bk][i] - (p1[bk][i] + p2[bk][i]));
    }
#pragma unroll
    for (int k = 0; k < kOps; ++k) A[k] = An[k];
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int e = threadIdx.x + k * NT;
    const int x = ((e / VPR) << C) | (e % VPR) * 2;
    const float2 v0 = sm[lds_pos(x)], v1 = sm[lds_pos(x + 1)];
    st16<STREAM>(p4 + glob_k(k) / 2, make_float4(v0.x, v0.y, v1.x, v1.y));
  }
}

template <int C, int H, bool STREAM>
__global__ void __launch_bounds__(1 << (C + H - kW))
    k_tile_mfma(float* __restrict__ a, TileRows rows, const int4* __restrict__ rounds,
                int nrounds, const float* __restrict__ amats) {
  // tile base: the workgroup index spread over the bits outside the tile
  uint64_t base = uint64_t(blockIdx.x) << C;
#pragma unroll
  for (int j = 0; j < H; ++j) base = insert_zero(base, rows.b[j]);
  tile_mfma_body<C, H, STREAM>(a, base, rows, rounds, nrounds, amats);
}

// Many kets at once: workgroup -> item by binary search over the items'
// first tiles; each item is one pass of one ket of the arena.
template <int C, int H>
__device__ __forceinline__ const TileItem& batch_item(const TileItem* __restrict__ items, int nitems,
                                                      uint64_t* base) {
  int lo = 0, hi = nitems - 1;
  const uint64_t b = blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].first_tile <= b) lo = mid;
    else hi = mid - 1;
  }
  const TileItem& it = items[lo];
  *base = (b - it.first_tile) << C;
#pragma unroll
  for (int j = 0; j < H; ++j) *base = insert_zero(*base, it.rows.b[j]);
  return it;
}

template <int C, int H>
__global__ void __launch_bounds__(1 << (C + H - kW))
    k_tile_mfma_batch(float* __restrict__ arena, const TileItem* __restrict__ items, int nitems,
                      const int4* __restrict__ rounds, const float* __restrict__ amats) {
  uint64_t base;
  const TileItem& it = batch_item<C, H>(items, nitems, &base);
  tile_mfma_body<C, H, false>(arena + 2 * it.amp_off, base, it.rows, rounds + it.r0, it.nr,
                              amats);
}

template <typename R, int C, int H>
__global__ void __launch_bounds__(1 << (C + H - kW))
__attribute__((amdgpu_waves_per_eu(kPairWaves<R>)))
    k_tile_pair_batch(R* __restrict__ arena, const TileItem* __restrict__ items, int nitems,
                      const int4* __restrict__ rounds, const R* __restrict__ num) {
  uint64_t base;
  const TileItem& it = batch_item<C, H>(items, nitems, &base);
  tile_pair_body<C, H, false, true>(arena + 2 * it.amp_off, base, it.rows, rounds + it.r0, it.nr,
                                    num, it.amps);
}

}  // namespace

namespace {
template <int C>
hipError_t launch_mfma_c(float* a, int n, const TileRows& rows, const void* rounds, int nrounds,
                         const float* amats, hipStream_t s) {
  constexpr int H = kTileRowBits, TB = C + H;
  if (n < TB || nrounds < 1) return hipErrorInvalidValue;
  for (int j = 0; j < H; ++j)
    if (rows.b[j] < C || rows.b[j] >= n || (j > 0 && rows.b[j] <= rows.b[j - 1]))
      return hipErrorInvalidValue;
  const size_t bytes = size_t((1 << TB) + ((1 << TB) >> 4)) * sizeof(float2);
  const uint64_t tiles = uint64_t(1) << (n - TB);
  auto kern = stream_sweep(n, 8, C) ? k_tile_mfma<C, H, true> : k_tile_mfma<C, H, false>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  hipLaunchKernelGGL(kern, dim3(unsigned(tiles)), dim3(1 << (TB - kW)), bytes, s, a, rows,
                     static_cast<const int4*>(rounds), nrounds, amats);
  return hipGetLastError();
}
}  // namespace


namespace {
template <typename R, int C>
hipError_t launch_pair_c(R* a, int n, const TileRows& rows, const void* rounds, int nrounds,
                         const R* num, hipStream_t s) {
  constexpr int H = kTileRowBits, TB = C + H;
  if (n < TB || nrounds < 1) return hipErrorInvalidValue;
  for (int j = 0; j < H; ++j)
    if (rows.b[j] < C || rows.b[j] >= n || (j > 0 && rows.b[j] <= rows.b[j - 1]))
      return hipErrorInvalidValue;
  const size_t bytes = pair_lds<R, TB>();
  auto kern =
      stream_sweep(n, 2 * sizeof(R), C) ? k_tile_pair<R, C, H, true> : k_tile_pair<R, C, H, false>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  hipLaunchKernelGGL(kern, dim3(unsigned(uint64_t(1) << (n - TB))), dim3(1 << (TB - kW)), bytes, s,
                     a, rows, static_cast<const int4*>(rounds), nrounds, num);
  return hipGetLastError();
}
}  // namespace

template <typename R>
hipError_t launch_tile_pair(R* a, int n, int low_bits, const TileRows& rows, const void* rounds,
                            int nrounds, const R* num, hipStream_t s) {
  if (low_bits == 4) return launch_pair_c<R, 4>(a, n, rows, rounds, nrounds, num, s);
  if constexpr (sizeof(R) == 4) {
    if (low_bits == 5) return launch_pair_c<R, 5>(a, n, rows, rounds, nrounds, num, s);
    if (low_bits == 6) return launch_pair_c<R, 6>(a, n, rows, rounds, nrounds, num, s);
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_tile_pair<float>(float*, int, int, const TileRows&, const void*, int,
                                            const float*, hipStream_t);
template hipError_t launch_tile_pair<double>(double*, int, int, const TileRows&, const void*, int,
                                             const double*, hipStream_t);

hipError_t launch_tile_mfma(float* a, int n, int low_bits, const TileRows& rows,
                            const void* rounds, int nrounds, const float* amats, hipStream_t s) {
  switch (low_bits) {
    case 4: return launch_mfma_c<4>(a, n, rows, rounds, nrounds, amats, s);
    case 5: return launch_mfma_c<5>(a, n, rows, rounds, nrounds, amats, s);
    case 6: return launch_mfma_c<6>(a, n, rows, rounds, nrounds, amats, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {
template <typename R, int TB>
hipError_t launch_whole_tb(R* a, int n, const WholePerm& perm, const void* rounds, int nrounds,
                           const R* num, hipStream_t s) {
  void (*kern)(R*, int, WholePerm, const int4*, int, const R*) = k_whole_pair<TB>;
  hipLaunchKernelGGL(kern, dim3(1), dim3(1 << (TB - 2)), (pair_lds<R, TB>()), s, a, n, perm,
                     static_cast<const int4*>(rounds), nrounds, num);
  return hipGetLastError();
}
}  // namespace

template <typename R>
hipError_t launch_whole(R* a, int n, const int* perm, const void* rounds, int nrounds, const R* num,
                        hipStream_t s) {
  if (n < 1 || n > 11 || nrounds < 1) return hipErrorInvalidValue;
  WholePerm w{};
  for (int q = 0; q < 11; ++q) {  // (bits from n on keep their place)
    const int p = q < n ? perm[q] : q;
    w.bits |= uint64_t(p) << (4 * q);
    if (p == 0) w.first = q;
  }
  if (whole_bits(n) == 10) return launch_whole_tb<R, 10>(a, n, w, rounds, nrounds, num, s);
  if constexpr (sizeof(R) == 4)
    if (whole_bits(n) == 11) return launch_whole_tb<R, 11>(a, n, w, rounds, nrounds, num, s);
  return hipErrorInvalidValue;
}
template hipError_t launch_whole<float>(float*, int, const int*, const void*, int, const float*,
                                        hipStream_t);
template hipError_t launch_whole<double>(double*, int, const int*, const void*, int, const double*,
                                         hipStream_t);

// complex64 (dtype 1): rows of 2^g_tile_low_c64 amplitudes (4: 128 bytes, 5:
// 256 bytes, 6: 512 bytes); complex128: 16 (256 bytes). Rows of 32 complex64
// amplitudes measured fastest for 10-layer random circuits (a 32 KiB tile
// leaves room for four workgroups per CU, against two 64 KiB ones); for
// complex128, rows of 16 (32 KiB tiles) took 4% less time per circuit than
// rows of 32 (64 KiB), one more pass at 7% less time each.
int g_tile_low_c64 = 5;
int tile_low_bits(int dtype) { return dtype == 1 ? g_tile_low_c64 : 4; }

namespace {
template <typename R, int C>
hipError_t launch_pass_c(R* a, int n, const TileRows& rows, const void* rounds, int nrounds,
                         const void* gates, const R* mats, hipStream_t s) {
  constexpr int H = kTileRowBits;
  constexpr int TB = C + H;
  if (n < TB) return hipErrorInvalidValue;
  for (int j = 0; j < H; ++j)
    if (rows.b[j] < C || rows.b[j] >= n || (j > 0 && rows.b[j] <= rows.b[j - 1]))
      return hipErrorInvalidValue;
  const size_t bytes = size_t((1 << TB) + ((1 << TB) >> 4)) * 2 * sizeof(R);
  auto kern = stream_sweep(n, 2 * sizeof(R), C) ? k_tile_pass<R, C, H, true>
                                                : k_tile_pass<R, C, H, false>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  const unsigned grid = unsigned(uint64_t(1) << (n - TB));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(1 << (TB - kW)), bytes, s, a, rows,
                     static_cast<const int4*>(rounds), nrounds, static_cast<const int2*>(gates),
                     mats);
  return hipGetLastError();
}
}  // namespace

template <typename R>
hipError_t launch_tile_pass(R* a, int n, int low_bits, const TileRows& rows, const void* rounds,
                            int nrounds, const void* gates, const R* mats, hipStream_t s) {
  if (low_bits == 4) return launch_pass_c<R, 4>(a, n, rows, rounds, nrounds, gates, mats, s);
  if (low_bits == 5) return launch_pass_c<R, 5>(a, n, rows, rounds, nrounds, gates, mats, s);
  if constexpr (sizeof(R) == 4)
    if (low_bits == 6) return launch_pass_c<R, 6>(a, n, rows, rounds, nrounds, gates, mats, s);
  return hipErrorInvalidValue;
}

hipError_t launch_tile_mfma_batch(float* arena, const TileItem* items, int nitems, uint64_t tiles,
                                  const void* rounds, const float* amats, hipStream_t s) {
  constexpr int C = kBatchTileLow, H = kTileRowBits, TB = C + H;
  if (nitems < 1 || tiles < 1 || tiles > 0x7fffffffu) return hipErrorInvalidValue;
  const size_t bytes = size_t((1 << TB) + ((1 << TB) >> 4)) * sizeof(float2);
  auto kern = k_tile_mfma_batch<C, H>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  hipLaunchKernelGGL(kern, dim3(unsigned(tiles)), dim3(1 << (TB - kW)), bytes, s, arena, items,
                     nitems, static_cast<const int4*>(rounds), amats);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_tile_pair_batch(R* arena, const TileItem* items, int nitems, uint64_t tiles,
                                  const void* rounds, const R* num, hipStream_t s) {
  constexpr int C = sizeof(R) == 4 ? kBatchTileLow : kBatchTileLowWide, H = kTileRowBits,
                TB = C + H;
  if (nitems < 1 || tiles < 1 || tiles > 0x7fffffffu) return hipErrorInvalidValue;
  const size_t bytes = pair_lds<R, TB>();
  auto kern = k_tile_pair_batch<R, C, H>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  hipLaunchKernelGGL(kern, dim3(unsigned(tiles)), dim3(1 << (TB - kW)), bytes, s, arena, items,
                     nitems, static_cast<const int4*>(rounds), num);
  return hipGetLastError();
}
template hipError_t launch_tile_pair_batch<float>(float*, const TileItem*, int, uint64_t,
                                                  const void*, const float*, hipStream_t);
template hipError_t launch_tile_pair_batch<double>(double*, const TileItem*, int, uint64_t,
                                                   const void*, const double*, hipStream_t);

template hipError_t launch_tile_pass<float>(float*, int, int, const TileRows&, const void*, int,
                                            const void*, const float*, hipStream_t);
template hipError_t launch_tile_pass<double>(double*, int, int, const TileRows&, const void*, int,
                                             const void*, const double*, hipStream_t);

}  // namespace qs
