// Passes over image planes held in LDS: rows and columns of a 2-D transform meet in an
// LDS plane, so that a workgroup can run several transforms of one plane without a trip
// through memory.  Used by the stack's tail, the small 2-D transforms (tail.hip) and the
// one-launch small layers (small.hip).
#pragma once

#include "device.h"
#include "fft.h"
#include "internal.h"
#include "lds_limit.h"

#include <hip/hip_runtime.h>

namespace fdc {
namespace plane {

// Every transform here uses the column plans: E = 8 elements per thread.
template <int N>
using Plan = ColCfg<N>;

// LDS planes: `rows` rows of ld complex values, padded after every 8 rows (plane_at in
// fft.h), ld > L (the spare columns give idle lanes somewhere harmless to exchange through).
// ld depends on the plan of the plane's columns, so that neither its in-place exchanges nor
// the row passes conflict: an LDS cycle serves 16 lanes' writes over 32 banks or 32 lanes'
// reads over 64; the 8 columns a wave has side by side at 64 points want rows 16 banks apart
// modulo 32 (ld = 8 modulo 16), the 4 at 128 points 8 (ld = 4 modulo 8), also the 4 lanes of a
// 32-point row.  (With ld odd the conflicts took a third of the tail kernels' LDS cycles.)
template <int COLN>
__host__ __device__ constexpr int plane_ld(int L) {
  int ld = L + 1;
  while (COLN == 64 ? ld % 16 != 8 : ld % 8 != 4) ++ld;
  return ld;
}
__host__ __device__ constexpr int plane_size(int rows, int ld) { return rows * ld + rows / 8 * plane_pad(ld); }

template <int N, int M>
__device__ __forceinline__ int kept(int mrow) {
  return mrow < M / 2 ? mrow : mrow + (N - M);
}

__device__ __forceinline__ float weight(int l, int n, float alpha, float beta) {
  return (l == 0 || 2 * l == n) ? alpha : alpha * beta;
}

// Bin (plane, row, l) of a spectrum (SpecLayout) in HBM.
__device__ __forceinline__ float2 *spec_at(const SpecLayout &s, long long plane, int row, int l, int L) {
  return l < L - 1 ? s.main + plane * s.ps + (long long)row * s.rs + bin_off(s, l)
                   : s.side + plane * s.sps + (long long)row * s.srs;
}

// Lane roles.  Row passes: t fastest (a wave reads whole rows).  Column passes:
// the W = 64 / TPS columns of a wave fastest (a wave's global accesses are runs of
// W consecutive bins of a row).
template <int N>
struct RowLanes {
  static constexpr int TPS = Plan<N>::TPS, W = 64 / TPS;
  int t, s, first;
  __device__ RowLanes() : RowLanes(threadIdx.x) {}
  __device__ explicit RowLanes(int tid) {
    const int lane = tid & 63;
    t = lane % TPS;
    s = lane / TPS;
    first = (tid >> 6) * W;
  }
};
template <int N>
struct ColLanes {
  static constexpr int TPS = Plan<N>::TPS, W = 64 / TPS;
  int t, s, first;
  __device__ ColLanes() : ColLanes(threadIdx.x) {}
  __device__ explicit ColLanes(int tid) {
    const int lane = tid & 63;
    s = lane % W;
    t = lane / W;
    first = (tid >> 6) * W;
  }
};

// ----------------------------------------------------------------------------
// row passes (pairs of real rows packed as one complex sequence z = a + i b)
// ----------------------------------------------------------------------------
// Packed inverse input of two rows: v[m] = A_k + i B_k at k = t + TPS m, the Hermitian
// extensions of the rows' first LIN bins, bin(row 0 or 1, k), weighted by c-weights (a1 at
// l = 0 and N/2, a1 b1 elsewhere), with real-part semantics at l = 0 and N/2: the imaginary
// parts there are left out, not multiplied by zero, whatever they hold.  Which elements are
// bins, conjugated bins or zero is known at compile time but for lane t = 0 at the ends.
template <int N, int LIN, class Bin>
__device__ __forceinline__ void c2r_in(float2 (&v)[Plan<N>::E], Bin bin, int t, float a1, float b1) {
  constexpr int TPS = Plan<N>::TPS, E = Plan<N>::E, Q = (LIN - 1) / TPS;  // Q whole groups of TPS bins
  static_assert(Q * TPS == LIN - 1 && 2 * Q <= E, "bins in whole groups of the row plan");
  const float w = a1 * b1;
  const bool t0 = t == 0;
  const float edge_w = t0 ? a1 : w;  // weight of the edge bins, lane t = 0
  static_for<0, E>([&](auto mc) {
    constexpr int m = decltype(mc)::value;
    constexpr bool edge = m == 0 || 2 * m == E;
    const float wr = edge ? edge_w : w;
    if constexpr (m < Q) {  // bin t + TPS m
      const float2 a = bin(0, t + TPS * m), b = bin(1, t + TPS * m);
      const float ai = edge && t0 ? 0.f : a.y, bi = edge && t0 ? 0.f : b.y;
      v[m] = make_float2(fmaf(-w, bi, wr * a.x), fmaf(wr, b.x, w * ai));
    } else if constexpr (m >= E - Q) {  // bin N - t - TPS m, conjugated (N/2 itself: m = E/2, t = 0)
      const float2 a = bin(0, N - TPS * m - t), b = bin(1, N - TPS * m - t);
      const float ai = edge && t0 ? 0.f : a.y, bi = edge && t0 ? 0.f : b.y;
      v[m] = make_float2(fmaf(w, bi, wr * a.x), fmaf(wr, b.x, -(w * ai)));
    } else if constexpr (m == Q) {  // lane t = 0: bin LIN - 1 < N/2
      const float2 a = bin(0, LIN - 1), b = bin(1, LIN - 1);
      v[m] = t0 ? make_float2(w * (a.x - b.y), w * (a.y + b.x)) : make_float2(0.f, 0.f);
    } else {
      v[m] = make_float2(0.f, 0.f);
    }
  });
}

// Forward transform output of a packed pair (held in registers, comb order) -> the two rows'
// weighted bins k < LOUT (a2 at l = 0 and N/2, a2 b2 elsewhere): emit(row 0 or 1, k, value).
// scr: this sequence's slot (row_slot<N>() values).
template <int N, int LOUT, class Emit>
__device__ __forceinline__ void r2c_out(const float2 (&v)[Plan<N>::E], float2 *scr, int t, float a2, float b2,
                                        Emit emit) {
  constexpr int TPS = Plan<N>::TPS, E = Plan<N>::E, Q = (LOUT - 1) / TPS;
  static_assert(Q * TPS == LOUT - 1, "bins in whole groups of the row plan");
  lds_barrier<true>();
#pragma unroll
  for (int m = 0; m < E; ++m) scr[seq_at<kLdsSeq, N>(0, t + TPS * m, 1)] = v[m];
  lds_barrier<true>();
  const float w = 0.5f * a2 * b2, w0 = 0.5f * a2;
  auto pair = [&](int k, int n, float wgt) {
    const float2 zk = scr[seq_at<kLdsSeq, N>(0, k, 1)], zn = scr[seq_at<kLdsSeq, N>(0, n, 1)];
    emit(0, k, make_float2((zk.x + zn.x) * wgt, (zk.y - zn.y) * wgt));
    emit(1, k, make_float2((zk.y + zn.y) * wgt, (zn.x - zk.x) * wgt));
  };
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int k = t + TPS * i;
    pair(k, i == 0 && t == 0 ? 0 : N - k, i == 0 && t == 0 ? w0 : w);
  }
  if (t == 0) pair(LOUT - 1, N - LOUT + 1, 2 * (LOUT - 1) == N ? w0 : w);
}

// ----------------------------------------------------------------------------
// column passes (in place in an LDS plane)
// ----------------------------------------------------------------------------
// For every item (plane q < nq, column l < L): load(v, q, l, t, act) fills the
// column, the N-point transform (direction DIR) runs through column l of plane(q),
// store(v, q, l, t, act) takes the result.  Idle lanes (act = false) work on the
// spare column L of plane 0 and must not store.
// COLN: the plan the planes' ld was chosen for.
template <int N, int DIR, int NT, int COLN = N, class Load, class PlaneOf, class Store>
__device__ __forceinline__ void col_pass(int nq, int L, const float2 *tw, int tws, Load load, PlaneOf plane,
                                         Store store) {
  using C = Plan<N>;
  constexpr int SEQ = NT / C::TPS;
  const ColLanes<N> ln;
  const int items = nq * L;
  for (int r0 = 0; r0 + ln.first < items; r0 += SEQ) {
    const int it = r0 + ln.first + ln.s;
    const bool act = it < items;
    const int q = act ? it / L : 0, l = act ? it - (it / L) * L : L;
    float2 v[C::E];
    load(v, q, l, ln.t, act);
    fft_seq<N, DIR, true, true, kLdsPlane, C>(v, ln.t, plane(q), l, plane_ld<COLN>(L), tw, tws);
    store(v, q, l, ln.t, act);
  }
}

// Scratch of a row pass of `items` pairs of N-point rows with NT threads: one slot per
// sequence in flight, whole waves of them up to NT / TPS.
template <int N, int NT>
__host__ __device__ constexpr int row_scratch(int items) {
  constexpr int TPS = Plan<N>::TPS, W = 64 / TPS, SEQ = NT / TPS;
  const int used = (items + W - 1) / W * W;
  return (used < SEQ ? used : SEQ) * row_slot<N>();
}

}  // namespace plane

}  // namespace fdc
