// Small CIC + FDP layers (section 2.4.1, Eq. 5, FDP of section 2.4.2) in one launch each
// way: one workgroup takes an input plane through every transform of the layer in LDS.
//
//   k_small_fwd: x plane (b, c) -> row transforms -> column DFT, the bins FDP keeps (the
//                saved spectrum) -> per output channel the CIC product, the inverse column
//                DFT and the inverse rows -> y
//   k_small_bwd: upstream-gradient planes of channel c -> rows, column DFTs -> dK products
//                (summed over the workgroup's images) and dXh summed over the channel's
//                outputs -> FDP adjoint, inverse columns and rows -> gx
//
// What bounds them: HBM traffic when there are many planes (x, the saved spectrum and y are
// each moved once, against three passes with two spectra written and read between them),
// launches and the latency of one workgroup's chain of stages when there are few.
#include "plane.h"

#include <algorithm>
#include <string>

namespace fdc {

extern __shared__ float2 s_lds[];

using namespace plane;

// Element offset of logical pixel (r, w) of an image seen through v, -1 when it is not stored.
__device__ __forceinline__ int view_at(const ImgView &v, int ncols, int r, int w) {
  if (v.mode == 0) return r * v.cols_stored + w;
  int rr = r - v.shift, ww = w - v.shift;
  if (v.mode == 1) return (rr < 0 || ww < 0) ? -1 : rr * v.cols_stored + ww;
  rr += rr < 0 ? v.rows : 0;
  ww += ww < 0 ? ncols : 0;
  return rr * v.cols_stored + ww;
}

// threadIdx.x as a value the compiler cannot trace: the lane indices derived from it are
// formed again in every turn of a loop instead of being hoisted, a few instructions against
// the 60 to 120 registers that the hoisted addresses of all stages took (190-256 VGPRs, one
// or two waves per SIMD).
__device__ __forceinline__ int loop_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int cmin(int a, int b) { return a < b ? a : b; }
// Waves that take `items` sequences of an n-point plan in one round.
template <int n>
constexpr int plan_waves(int items) {
  return (items * Plan<n>::TPS + 63) / 64;
}

// Geometry (complex values) of the forward: TA [N][ld] (row spectrum, then its kept rows XA
// [M][ld] in place), U [M][ld]; the row passes' scratch aliases what is not in use.
template <int N, int M>
struct SmallFwd {
  static constexpr int L = M / 2 + 1, ldT = plane_ld<N>(L), ldU = plane_ld<M>(L);
  static constexpr int sT = plane_size(N, ldT), sX = plane_size(M, ldT), sU = plane_size(M, ldU);
  // every column in one round, the rows in at most two (128 points) or one
  static constexpr int WAVES = cmax(cmax(plan_waves<N>(L), plan_waves<M>(L)), cmin(plan_waves<N>(N / 2), 8));
  static constexpr int NT = 64 * WAVES;
  static constexpr int TW = twiddle_lds_elems<N>(), sN = row_scratch<N, NT>(N / 2), sM = row_scratch<M, NT>(M / 2);
  static constexpr int TA = TW, DSCR = M == N ? TA : TA + sX;  // XA stays in registers when M == N
  static constexpr int U = cmax(TA + sT, DSCR + sM), END = U + cmax(sU, sN);
};

// One workgroup per input plane (b, c) and group of JL of its J output channels (group 0
// stores the saved spectrum; each group repeats the plane's own transforms).  Workgroup w
// after the XCD remap: b fastest, then the group, then c (the images read the same kernels).
template <int N, int M>
__global__ __launch_bounds__((SmallFwd<N, M>::NT), 4) void k_small_fwd(const float *__restrict__ x,
                                                                   const float2 *__restrict__ K, SpecLayout saved,
                                                                   float *__restrict__ y, ImgView view,
                                                                   long long out_plane, int B, int C, int J, int JL) {
  using G = SmallFwd<N, M>;
  using PN = Plan<N>;
  using PM = Plan<M>;
  constexpr int L = G::L, ldT = G::ldT, ldU = G::ldU, NT = G::NT, NF = N / 2 + 1;
  float2 *tw = s_lds, *TA = s_lds + G::TA, *U = s_lds + G::U;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int b = w % B, cg = w / B, JG = J / JL;
  const int c = cg / JG, jg = cg - c * JG;
  const long long xplane = (long long)b * C + c;
  const int o0 = c * J + jg * JL;

  // this thread's column in the per-channel stage, and its first kernel column
  const ColLanes<M> cm;
  const int l = cm.first + cm.s;
  const bool cact = l < L;
  const int lc = cact ? l : 0;
  float2 kn[PM::E];
  auto load_k = [&](int o) __attribute__((always_inline)) {
    const float2 *kc = K + (long long)o * N * NF + lc;
#pragma unroll
    for (int m = 0; m < PM::E; ++m) kn[m] = kc[kept<N, M>(cm.t + PM::TPS * m) * NF];
  };

  stage_twiddles<N>(tw, threadIdx.x, NT);
  {  // rows of x -> TA [N][L]
    constexpr int SEQ = NT / PN::TPS, H = N / 2;
    const RowLanes<N> ln;
    for (int r0 = 0; r0 + ln.first < H; r0 += SEQ) {
      const int p = r0 + ln.first + ln.s;
      const bool act = p < H;
      const int r = act ? p : 0;
      const float *xr = x + xplane * N * N + r * N;
      float2 v[PN::E];
#pragma unroll
      for (int m = 0; m < PN::E; ++m) v[m] = make_float2(xr[ln.t + PN::TPS * m], xr[N / 2 * N + ln.t + PN::TPS * m]);
      fft_seq<N, -1, true, true, kLdsSeq, PN>(v, ln.t, U, (ln.first + ln.s) * row_slot<N>(), 1, tw, 1);
      float2 *ta = TA + plane_at(r, ldT);
      r2c_out<N, L>(v, U + (ln.first + ln.s) * row_slot<N>(), ln.t, 1.f, 1.f, [&](int rr, int k, float2 val) {
        if (act) ta[rr * plane_at(N / 2, ldT) + k] = val;
      });
    }
  }
  if (cm.first < L) load_k(o0);
  __syncthreads();
  float2 xv[PM::E];  // M == N: this thread's pooled-spectrum values
  {  // columns of TA, the kept rows -> XA (in place; registers when M == N) and saved
    const ColLanes<N> ln;
    const int ln_l = ln.first + ln.s;
    if (ln.first < L) {
      const int ll = ln_l < L ? ln_l : L;
      float2 v[PN::E];
#pragma unroll
      for (int m = 0; m < PN::E; ++m) v[m] = TA[plane_at(ln.t + PN::TPS * m, ldT) + ll];
      fft_seq<N, -1, true, true, kLdsPlane, PN>(v, ln.t, TA, ll, ldT, tw, 1);
      lds_barrier<true>();
      if constexpr (M == N) {
#pragma unroll
        for (int m = 0; m < PM::E; ++m) xv[m] = v[m];
      }
#pragma unroll
      for (int m = 0; m < PN::E; ++m) {
        const int k = ln.t + PN::TPS * m;
        if (M == N || k < M / 2 || k >= N - M / 2) {
          const int mrow = k < M / 2 ? k : k - (N - M);
          if (M != N) TA[plane_at(mrow, ldT) + ll] = v[m];
          if (saved.main != nullptr && jg == 0 && ln_l < L) *spec_at(saved, xplane, mrow, ln_l, L) = v[m];
        }
      }
    }
  }
  __syncthreads();
  const float inv = 1.f / ((float)M * (float)M);
  for (int jj = 0; jj < JL; ++jj) {
    // CIC product (Eq. 5) and inverse column DFT (M) -> U
    if (cm.first < L) {
      const int ll = cact ? l : L;
      float2 z[PM::E];
#pragma unroll
      for (int m = 0; m < PM::E; ++m)
        z[m] = cmul(M == N ? xv[m] : TA[plane_at(cm.t + PM::TPS * m, ldT) + ll], kn[m]);
      if (jj + 1 < JL) load_k(o0 + jj + 1);  // the next kernel column loads during this channel's transforms
      fft_seq<M, +1, true, true, kLdsPlane, PM>(z, cm.t, U, ll, ldU, tw, N / M);
      lds_barrier<true>();
#pragma unroll
      for (int m = 0; m < PM::E; ++m) U[plane_at(cm.t + PM::TPS * m, ldU) + ll] = z[m];
    }
    __syncthreads();
    {  // inverse rows of U (1 / M^2) -> y
      float2 *scr = s_lds + G::DSCR;
      constexpr int SEQ = NT / PM::TPS, H = M / 2;
      const RowLanes<M> ln;
      float *yp = y + ((long long)b * C * J + o0 + jj) * out_plane;
      for (int r0 = 0; r0 + ln.first < H; r0 += SEQ) {
        const int p = r0 + ln.first + ln.s;
        const bool act = p < H;
        const int r = act ? p : 0;
        const float2 *u = U + plane_at(r, ldU);
        float2 v[PM::E];
        c2r_in<M, L>(v, [&](int rr, int k) { return u[rr * plane_at(M / 2, ldU) + k]; }, ln.t, inv, 1.f);
        fft_seq<M, +1, true, true, kLdsSeq, PM>(v, ln.t, scr, (ln.first + ln.s) * row_slot<M>(), 1, tw, N / M);
#pragma unroll
        for (int m = 0; m < PM::E; ++m) {
          const int oa = view_at(view, M, r, ln.t + PM::TPS * m), ob = view_at(view, M, r + M / 2, ln.t + PM::TPS * m);
          if (act && oa >= 0) yp[oa] = v[m].x;
          if (act && ob >= 0) yp[ob] = v[m].y;
        }
      }
    }
    __syncthreads();
  }
}

// Geometry of the backward, JP output channels at a time: G [JP][M][ld], V [N][ld] (M == N,
// JP == 1: V is G), row scratch.
template <int N, int M, int JP>
struct SmallBwd {
  static constexpr int L = M / 2 + 1, ldG = plane_ld<M>(L), ldV = plane_ld<N>(L);
  static constexpr int sG = plane_size(M, ldG), sV = plane_size(N, ldV);
  static constexpr int WAVES =
      cmax(cmax(plan_waves<N>(L), plan_waves<M>(JP * L)),
           cmin(cmax(plan_waves<N>(N / 2), plan_waves<M>(JP * M / 2)), 8));
  static constexpr int NT = 64 * WAVES;
  static constexpr bool ONE = M == N && JP == 1;
  static constexpr int TW = twiddle_lds_elems<N>(), sN = row_scratch<N, NT>(N / 2),
                       sM = row_scratch<M, NT>(JP * M / 2);
  static constexpr int GP = TW;
  // ONE: [tw][G][scratch]; else [tw][G, N-row scratch][V, M-row scratch]
  static constexpr int VP = ONE ? GP : GP + cmax(JP * sG, sN);
  static constexpr int SM = ONE ? GP + sG : VP, SN = ONE ? SM : GP;
  static constexpr int END = ONE ? SM + cmax(sN, sM) : VP + cmax(sV, sM);
};

// One workgroup per input channel c and range of images (R ranges; workgroup w after the
// XCD remap: the range fastest).  For each image, JP output channels at a time: rows and
// column DFTs of the upstream gradient, the dK product with the saved spectrum, and
// dXh += G conj(K); then the FDP adjoint and the inverse transforms -> gx (NULL: skipped).
//   NJ = 1 (J = JP): dK summed over the range's images in registers, in order (two rounds of
//   channels, 32 more registers, spilled and ran 1.6 times longer);
//   NJ = 0: any J, one image per range (R = B), the products written as they are formed.
// (Registers: four waves a SIMD, three with dK's sums, which spilled 30 to 60 values at four.)
// dst (NULL: dK skipped): parts = 1: part [R][S][M][L]; parts = 0 (R == 1): gK [S][N][N/2+1]
// with zeros at the bins FDP drops.
template <int N, int M, int JP, int NJ>
__global__ __launch_bounds__((SmallBwd<N, M, JP>::NT), NJ == 1 ? 3 : 4) void k_small_bwd(
    const float *__restrict__ gy, ImgView view, long long out_plane, SpecLayout saved, const float2 *__restrict__ K,
    float *__restrict__ gx, float2 *__restrict__ dst, int B, int C, int J, int R, int parts) {
  using G = SmallBwd<N, M, JP>;
  using PN = Plan<N>;
  using PM = Plan<M>;
  constexpr int L = G::L, ldG = G::ldG, ldV = G::ldV, sG = G::sG, NT = G::NT, NF = N / 2 + 1;
  static_assert(NJ == 0 || NJ == 1, "dK of one round of channels in registers, or none");
  float2 *tw = s_lds, *GP = s_lds + G::GP, *VP = s_lds + G::VP;
  const int w = xcd_remap(blockIdx.x, gridDim.x);
  const int c = w / R, range = w - c * R;
  const int b_lo = (int)((long long)range * B / R), b_hi = (int)((long long)(range + 1) * B / R);
  const int S = C * J, nch = (J + JP - 1) / JP;
  const float inv = 1.f / ((float)M * (float)M);

  constexpr int SEQM = NT / PM::TPS, HM = JP * (M / 2);
  constexpr bool PRE = HM <= SEQM;  // one round: its row loads are issued a stage ahead
  float2 pre[PM::E];
  // row pair p of the JP planes from output channel j0 of image b
  auto load_rows = [&](float2(&v)[PM::E], int t, int p, int b, int j0) __attribute__((always_inline)) {
    const bool act = p < HM;
    const int qq = act ? p / (M / 2) : 0, r = act ? p % (M / 2) : 0;
    const int j = min(j0 + qq, J - 1);
    const float *gp = gy + ((long long)b * S + c * J + j) * out_plane;
#pragma unroll
    for (int m = 0; m < PM::E; ++m) {
      const int ia = view_at(view, M, r, t + PM::TPS * m), ib = view_at(view, M, r + M / 2, t + PM::TPS * m);
      const float a = gp[ia < 0 ? 0 : ia], bb = gp[ib < 0 ? 0 : ib];  // unconditional, zeroed when cropped away
      v[m] = make_float2(ia >= 0 ? a : 0.f, ib >= 0 ? bb : 0.f);
    }
  };
  // a thread's column in the column stages: bin l (bin L, the spare one, for idle lanes) of
  // plane q of the JP
  struct Col {
    int t, q, l, lc;
    bool act, wave;
    __device__ explicit Col(int tid) {
      const ColLanes<M> cm(tid);
      const int it = cm.first + cm.s;
      t = cm.t;
      act = it < JP * L, wave = cm.first < JP * L;
      q = act ? it / L : 0, l = act ? it - q * L : L, lc = act ? l : 0;
    }
  };

  float2 dk[PM::E];
#pragma unroll
  for (int m = 0; m < PM::E; ++m) dk[m] = make_float2(0.f, 0.f);
  // dK of output channel o at this thread's column
  auto store_dk = [&](int o, const Col &cl, const float2(&d)[PM::E]) __attribute__((always_inline)) {
    if (parts) {
      float2 *p = dst + ((long long)range * S + o) * M * L + cl.lc;
#pragma unroll
      for (int m = 0; m < PM::E; ++m) p[(cl.t + PM::TPS * m) * L] = d[m];
    } else {
      float2 *p = dst + (long long)o * N * NF + cl.lc;
#pragma unroll
      for (int m = 0; m < PM::E; ++m) p[kept<N, M>(cl.t + PM::TPS * m) * NF] = d[m];
    }
  };

  if constexpr (PRE) {
    const RowLanes<M> rm;
    load_rows(pre, rm.t, rm.first + rm.s, b_lo, 0);
  }
  stage_twiddles<N>(tw, threadIdx.x, NT);
  for (int b = b_lo; b < b_hi; ++b) {
    float2 xv[PM::E], acc[PM::E];
    {
      const Col cl(loop_tid());
#pragma unroll
      for (int m = 0; m < PM::E; ++m) {
        acc[m] = xv[m] = make_float2(0.f, 0.f);
        if (dst != nullptr) xv[m] = *spec_at(saved, (long long)b * C + c, cl.t + PM::TPS * m, cl.lc, L);
      }
    }
    for (int ch = 0; ch < nch; ++ch) {
      const int j0 = ch * JP, tid = loop_tid();
      const RowLanes<M> rm(tid);
      // rows of the upstream gradients (c_l / M^2) -> G [JP][M][L]
      for (int r0 = 0; r0 + rm.first < HM; r0 += SEQM) {
        const int p = r0 + rm.first + rm.s;
        const bool act = p < HM;
        const int qq = act ? p / (M / 2) : 0, r = act ? p % (M / 2) : 0;
        float2 v[PM::E];
        if constexpr (PRE) {
#pragma unroll
          for (int m = 0; m < PM::E; ++m) v[m] = pre[m];
        } else {
          load_rows(v, rm.t, p, b, j0);
        }
        float2 *scr = s_lds + G::SM;
        fft_seq<M, -1, true, true, kLdsSeq, PM>(v, rm.t, scr, (rm.first + rm.s) * row_slot<M>(), 1, tw, N / M);
        float2 *g = GP + qq * sG + plane_at(r, ldG);
        r2c_out<M, L>(v, scr + (rm.first + rm.s) * row_slot<M>(), rm.t, inv, 2.f, [&](int rr, int k, float2 val) {
          if (act) g[rr * plane_at(M / 2, ldG) + k] = val;
        });
      }
      if constexpr (PRE) {  // the next channels' (or image's) rows load during the column stage
        const bool more = j0 + JP < J;
        if (more || b + 1 < b_hi) load_rows(pre, rm.t, rm.first + rm.s, more ? b : b + 1, more ? j0 + JP : 0);
      }
      const Col cl(tid);
      const int j = j0 + cl.q;
      const bool jact = cl.act && j < J;
      float2 kv[PM::E];
      if (cl.wave && gx != nullptr) {
        const float2 *kc = K + (long long)(c * J + min(j, J - 1)) * N * NF + cl.lc;
#pragma unroll
        for (int m = 0; m < PM::E; ++m) kv[m] = kc[kept<N, M>(cl.t + PM::TPS * m) * NF];
      }
      __syncthreads();
      if (cl.wave) {
        float2 v[PM::E], *gp = GP + cl.q * sG;
#pragma unroll
        for (int m = 0; m < PM::E; ++m) v[m] = gp[plane_at(cl.t + PM::TPS * m, ldG) + cl.l];
        fft_seq<M, -1, true, true, kLdsPlane, PM>(v, cl.t, gp, cl.l, ldG, tw, N / M);
        if (dst != nullptr) {
          if constexpr (NJ > 0) {
#pragma unroll
            for (int m = 0; m < PM::E; ++m) dk[m] = cfmac(dk[m], v[m], xv[m]);
          } else {
#pragma unroll
            for (int m = 0; m < PM::E; ++m) dk[m] = cmulc(v[m], xv[m]);
            if (jact) store_dk(c * J + j, cl, dk);
          }
        }
        if (gx != nullptr && jact) {
#pragma unroll
          for (int m = 0; m < PM::E; ++m) acc[m] = cfmac(acc[m], v[m], kv[m]);
        }
      }
      if (ch + 1 < nch || b + 1 < b_hi || !G::ONE) __syncthreads();  // G is written again
    }
    if (gx == nullptr) continue;
    // dXh of this image -> FDP adjoint, inverse columns (N) -> V
    const int tid = loop_tid();
    const Col cl(tid);
    if constexpr (G::ONE) {
      if (cl.wave) {  // the same column, in place: ordering within the wave is enough
        fft_seq<N, +1, true, true, kLdsPlane, PN>(acc, cl.t, GP, cl.l, ldG, tw, 1);
        lds_barrier<true>();
#pragma unroll
        for (int m = 0; m < PM::E; ++m) GP[plane_at(cl.t + PN::TPS * m, ldG) + cl.l] = acc[m];
      }
    } else {
      if (cl.act) {
#pragma unroll
        for (int m = 0; m < PM::E; ++m) GP[cl.q * sG + plane_at(cl.t + PM::TPS * m, ldG) + cl.l] = acc[m];
      }
      __syncthreads();
      const ColLanes<N> cn(tid);
      if (cn.first < L) {
        const int ll = cn.first + cn.s < L ? cn.first + cn.s : L;
        float2 v[PN::E];
#pragma unroll
        for (int m = 0; m < PN::E; ++m) {
          const int k = cn.t + PN::TPS * m;
          float2 s = make_float2(0.f, 0.f);
          if (M == N || k < M / 2 || k >= N - M / 2) {
            const int mrow = k < M / 2 ? k : k - (N - M);
#pragma unroll
            for (int i = 0; i < JP; ++i) s = cadd(s, GP[i * sG + plane_at(mrow, ldG) + ll]);
          }
          v[m] = s;
        }
        fft_seq<N, +1, true, true, kLdsPlane, PN>(v, cn.t, VP, ll, ldV, tw, 1);
        lds_barrier<true>();
#pragma unroll
        for (int m = 0; m < PN::E; ++m) VP[plane_at(cn.t + PN::TPS * m, ldV) + ll] = v[m];
      }
    }
    __syncthreads();
    {  // rfft2-adjoint rows of V (weights 1, 1/2) -> gx
      float2 *scr = s_lds + G::SN;
      constexpr int SEQ = NT / PN::TPS, H = N / 2;
      const RowLanes<N> ln(loop_tid());
      float *gp = gx + ((long long)b * C + c) * N * N;
      for (int r0 = 0; r0 + ln.first < H; r0 += SEQ) {
        const int p = r0 + ln.first + ln.s;
        const bool act = p < H;
        const int r = act ? p : 0;
        const float2 *u = VP + plane_at(r, ldV);
        float2 v[PN::E];
        c2r_in<N, L>(v, [&](int rr, int k) { return u[rr * plane_at(N / 2, ldV) + k]; }, ln.t, 1.f, 0.5f);
        fft_seq<N, +1, true, true, kLdsSeq, PN>(v, ln.t, scr, (ln.first + ln.s) * row_slot<N>(), 1, tw, 1);
        if (act) {
#pragma unroll
          for (int m = 0; m < PN::E; ++m)
            gp[r * N + ln.t + PN::TPS * m] = v[m].x, gp[(r + N / 2) * N + ln.t + PN::TPS * m] = v[m].y;
        }
      }
    }
    if (b + 1 < b_hi) __syncthreads();
  }
  if (dst == nullptr) return;
  if constexpr (NJ > 0) {
    const Col cl(loop_tid());
    if (cl.act) store_dk(c * J + cl.q, cl, dk);
  }
  if (!parts && M < N) {  // zeros at the dropped bins of this channel's gK planes
    for (int r = threadIdx.x / 64; r < J * N; r += NT / 64) {
      const int o = c * J + r / N, k = r % N;
      const bool keep = k < M / 2 || k >= N - M / 2;
      float2 *p = dst + ((long long)o * N + k) * NF;
      for (int i = (keep ? L : 0) + (threadIdx.x & 63); i < NF; i += 64) p[i] = make_float2(0.f, 0.f);
    }
  }
}

// ----------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------
template <int V>
using Int = std::integral_constant<int, V>;

template <class F>
static bool dispatch_small(int n, int m, F &&f) {
#define FDC_SMALL(N_, M_)       \
  if (n == N_ && m == M_) {     \
    f(Int<N_>{}, Int<M_>{});    \
    return true;                \
  }
  FDC_SMALL(32, 32) FDC_SMALL(32, 16) FDC_SMALL(32, 8) FDC_SMALL(64, 64) FDC_SMALL(64, 32) FDC_SMALL(64, 16)
  FDC_SMALL(128, 64) FDC_SMALL(128, 32)
#undef FDC_SMALL
  return false;
}

bool small_layer_supported(int n, int m) {
  // (128 -> 128 has 65 columns of 16 lanes, more than the 1024 threads of a workgroup)
  return dispatch_small(n, m, [](auto, auto) {});
}

constexpr int kSmallCus = 256;
constexpr int kSmallJps = 3;  // backward forms: 1, 2 or 4 output channels at a time

// Workgroups of a form resident at a time: by waves (the kernels' launch bounds) and LDS.  The
// backward to 64 points counts one a CU: a second one there gains nothing (16 images of 36
// channels, 64 -> 64: 8 ranges 0.82 of the separate launches, 16 ranges 0.72).
static int small_slots(int simd_waves, int waves, size_t lds) {
  return kSmallCus * std::max(1, std::min(4 * simd_waves / waves, (int)(160 * 1024 / lds)));
}
struct SmallForms {  // waves of a workgroup and workgroups resident
  int fwd_slots, bwd_waves[kSmallJps], bwd_slots[kSmallJps];
};
static SmallForms small_forms(int n, int m) {
  SmallForms f{};
  dispatch_small(n, m, [&](auto nc, auto mc) {
    constexpr int N = decltype(nc)::value, M = decltype(mc)::value;
    f.fwd_slots = small_slots(4, SmallFwd<N, M>::WAVES, SmallFwd<N, M>::END * sizeof(float2));
    auto bwd = [&](auto jpc, int i) {
      using G = SmallBwd<N, M, decltype(jpc)::value>;
      f.bwd_waves[i] = G::WAVES;
      f.bwd_slots[i] = M == 64 ? kSmallCus : small_slots(3, G::WAVES, G::END * sizeof(float2));
    };
    bwd(Int<1>{}, 0);
    if constexpr (M <= 32) bwd(Int<2>{}, 1), bwd(Int<4>{}, 2);
  });
  return f;
}

// Output channels a workgroup of the forward takes: each workgroup transforms its input plane
// again, so few channels a workgroup pay only while the launch is short of workgroups.
//   128 points (one or two workgroups a CU): the least (2 + JL) (rounds + w / 512) for w
//     workgroups in `rounds` rounds of the resident ones, a plane's own transforms counted as 2
//     channels: within 1 % of the best JL on average over 2 to 12 channels and 1 to 4096 planes,
//     22 % at worst.  (The rule below took up to 2.2 times the best: 448 planes of 5 channels,
//     128 -> 64: 47 us on separate launches, 78 with JL = 1, 38 with JL = 5.)
//   smaller planes: the most with at least 512 workgroups (1024 for 32 points and 8 channels or
//     more: 512 planes of 8, 32 -> 8: 12.3 us with JL = 8, 9.1 with 4, 11.8 on separate
//     launches); half of J where all of J would start a nearly empty second round (1040 planes of
//     12, 64 -> 16: 41.8 us with JL = 12, 36.6 with 6, 37.9 on separate launches).
static int small_jl(int n, int m, long long planes, int J) {
  const int slots = small_forms(n, m).fwd_slots;
  int JL = J;
  if (n == 128) {
    double least = 0.;
    auto consider = [&](int jl) {
      const long long w = planes * (J / jl);
      const double cost = (2. + jl) * ((double)((w + slots - 1) / slots) + w / 512.);
      if (jl == J || cost < least) least = cost, JL = jl;
    };
    for (int d = 1; (long long)d * d <= J; ++d)
      if (J % d == 0) consider(J / d), consider(d);
    return JL;
  }
  const long long target = n == 32 && J >= 8 ? 1024 : 512;
  for (int d = 2; d <= J && planes * (J / JL) < target; ++d)
    if (J % d == 0) JL = J / d;
  if (JL == J && J % 2 == 0 && J >= 8 && n == 64 && m < n && planes > slots && 4 * planes <= 5 * slots) JL = J / 2;
  return JL;
}

// Where the one-launch forward is the faster one: everywhere (16 planes 11 -> 6 us, 3000 planes
// of 64 -> 32 63 -> 44; 64 -> 16 with 8 channels 1.04 to 1.07 at 528 and 1040 planes) but for
// 128 -> 64 and 128 -> 32 with a last round of workgroups that is nearly empty, against separate
// launches that share the pooled columns between an even number of channels (one launch over
// separate ones, 16 images a call):
//   128 -> 64, 256 workgroups a round: 320 planes J = 4, 6, 8, 12: 1.02 to 1.08; 576 planes J = 2,
//     4, 6, 8: 1.02 to 1.08, but J = 3, 5, 12: 0.95, 0.96, 0.83; 1040 planes J = 1, 2: 1.04, 1.10,
//     J = 3 to 8: 0.99 to 0.73; full rounds 0.6 to 0.9
//   128 -> 32, 512 a round: 576 to 704 planes J = 8, 12: 1.00 to 1.06; 1040: 1.02, 1.09; J <= 6: 0.7 to 0.95
bool small_fwd_supported(int n, int m, int B, int C, int S) {
  if (!small_layer_supported(n, m)) return false;
  if (n != 128) return true;
  const int J = S / C;
  const long long planes = (long long)B * C;
  if (m == 64) {
    const double full = planes / (256. * ((planes + 255) / 256));  // share of the rounds at JL = J
    if (planes > 1024) return J > 2 || full >= 0.9;
    return J % 2 != 0 || full >= 0.8 || planes <= 256 || (planes > 512 && J > 8);
  }
  return J < 8 || planes <= 512 || planes > 1536 || planes / (512. * ((planes + 511) / 512)) >= 0.72;
}

// How the backward of a layer runs: JP output channels at a time, NJ = 1 where that is all of
// them (0: one image per workgroup), R image ranges, dK through partial sums or straight to gK.
struct SmallPlan {
  int JP, NJ, R, parts;
};
static SmallPlan small_plan(int n, int m, int B, int C, int J) {
  const SmallForms f = small_forms(n, m);
  const long long planes = (long long)B * C;
  SmallPlan p{1, 0, B, 1};
  // Channels side by side in LDS, 4 or 2: one at a time they are a chain of J turns, and each
  // turn reads the plane's stages again (64 -> 16, 1040 planes of 8: 33 us, 57 with one, 38 on
  // separate launches; 32 -> 8, 512 planes of 12: 17, 37, 22).  Two at 32 points with enough
  // planes, where four leave two workgroups a CU (64 -> 32, 576 planes of 4: 24 us, 30 with four).
  if (m <= 32 && J % 2 == 0) {
    p.JP = J % 4 == 0 ? 4 : 2;
    if (p.JP == 4 && m == 32 && n <= 64 && planes >= (J == 4 ? 320 : 576)) p.JP = 2;
  }
  const int form = p.JP / 2;  // 1, 2, 4 -> 0, 1, 2
  p.NJ = J == p.JP ? 1 : 0;
  if (p.NJ > 0 && B > 1) {
    // Images a range, all or a power of two: the least of rounds x images + what adding the ranges
    // costs, in units of one image's stages (within 0.4 % of the best power of two on average,
    // 29 % at worst; a fixed 1024 workgroups: 4 %, 90 %: 128 -> 32, 2 x 160 planes of 4: 47 us with 2
    // ranges, 28 with 1).
    const int slots = f.bwd_slots[form];
    double least = (double)((C + slots - 1) / slots) * B;
    p.R = 1;
    for (long long images = 1; images < B; images *= 2) {
      const long long R = (B + images - 1) / images, w = C * R;
      const double cost = (double)((w + slots - 1) / slots) * images + 0.75 + 0.4 * w / slots;
      if (cost < least) least = cost, p.R = (int)R;
    }
  }
  // One range writes gK itself unless too few threads would write its zeros (32 -> 8, one plane of
  // 8 channels: 29 us, 11 through partial sums and the launch that adds them)
  if (p.R == 1) {
    const int waves = f.bwd_waves[form];
    const long long zeros = (long long)J * ((long long)n * (n / 2 + 1) - (long long)m * (m / 2 + 1));
    p.parts = n > m && zeros > (waves >= 4 ? 16 : 8) * 64 * waves && (long long)C * waves * waves < 1024;
  }
  return p;
}

// Where the one-launch backward is the faster one (graph replays of both; one launch over
// separate ones, 1 to 16 images, 1 to 4096 planes):
//   to 32 points and below, J = 1, 2, 4 and even J: 0.3 to 1.0, but 128 -> 32 below
//   J = 3: 0.3 to 0.95, but 64 -> 16 past 1024 planes 1.05 at 2 images, 1.16 at 4096 planes
//   odd J from 5 go one at a time; J = 5: 32 -> 32, 64 -> 32, 32 -> 16 up to 1.7 below 320 planes, 0.4 to
//     0.95 from there (64 -> 32 1.08 to 1.12 past 1024); 32 -> 8, 64 -> 16 1.03 to 1.24
//   128 -> 32: at 2 images 64 to 704 channels of J = 3, 6, 8, 12 1.03 to 1.19 (two ranges of
//     partial sums against sums written once); at 16 J = 3 1.06 from 2048 planes, J = 12, 16 1.05 to 1.09
//     at 576 to 704; J = 5 1.03 to 1.26 but for 16 images and 64 to 512 planes, 0.77 to 0.97
//   64 -> 64: J = 1, 2 0.3 to 1.0 (J = 2, 16 images of 3072 planes 1.05, but 4096 cropped ones,
//     forward and backward, 306 us against 314); J = 3 0.3 to 1.03 up to 511 planes; J = 4 0.55 to
//     0.97 from 32 to 511 planes, up to 1.17 elsewhere; J >= 5 up to 1.5
//   128 -> 64: J = 1 0.4 to 0.9; J = 2 0.43 to 1.0 where the rounds of 256 workgroups are full, 1.03
//     at 320 planes, 1.05 to 1.24 from 576; J >= 3 up to 2.1
bool small_bwd_supported(int n, int m, int B, int C, int S) {
  if (!small_layer_supported(n, m)) return false;
  const int J = S / C;
  const long long planes = (long long)B * C;
  const bool odd = J % 2 != 0 && J > 3;
  if (m == 64) {
    if (J == 1) return true;
    if (n == 128) return J == 2 && (planes <= 256 || (planes >= 416 && planes < 512));
    return J == 2 || (planes < 512 && (J == 3 || (J == 4 && (planes >= 32 || B == 1))));
  }
  if (n == 128) {
    if (odd) return planes >= 64 && (B == 1 || (B >= 8 && planes <= 512));
    if (B == 1 || J == 1 || J == 2 || J == 4) return true;
    if (B < 8) return C < 64 || C > 704;
    return !(J == 3 && planes >= 1536) && !(J >= 12 && planes > 512 && planes <= 704);
  }
  if (odd) return planes >= 320 && ((m == 32 && (n == 32 || planes < 1024)) || (m == 16 && n == 32));
  if (n == 64 && m == 16 && J == 3 && planes > 1024) return B >= 8 && planes < 3072;
  return true;
}

hipError_t launch_small_fwd(int n, int m, const float *x, const float2 *K, SpecLayout saved, float *y, ImgView view,
                            long long out_plane, int B, int C, int S, hipStream_t s) {
  hipError_t err = hipErrorInvalidValue;
  const int J = S / C, JL = small_jl(n, m, (long long)B * C, J);
  const long long grid = (long long)B * C * (J / JL);
  if (grid >= (1LL << 31)) return err;
  dispatch_small(n, m, [&](auto nc, auto mc) {
    constexpr int N = decltype(nc)::value, M = decltype(mc)::value;
    using G = SmallFwd<N, M>;
    constexpr size_t lds = (size_t)G::END * sizeof(float2);
    static_assert(lds <= 160 * 1024, "small layer forward: LDS");
    static const std::string nm = "small_fwd_" + std::to_string(N) + "_" + std::to_string(M);
    err = allow_lds<k_small_fwd<N, M>>(lds);
    if (err != hipSuccess) return;
    err = timed_launch(nm.c_str(), k_small_fwd<N, M>, dim3((unsigned)grid), dim3(G::NT), lds, s, x, K, saved, y, view,
                       out_plane, B, C, J, JL);
  });
  return err;
}

int small_bwd_ranges(int n, int m, int B, int C, int S) { return small_plan(n, m, B, C, S / C).R; }
bool small_bwd_parts(int n, int m, int B, int C, int S) { return small_plan(n, m, B, C, S / C).parts != 0; }

hipError_t launch_small_bwd(int n, int m, const float *gy, ImgView view, long long out_plane, SpecLayout saved,
                            const float2 *K, float *gx, float2 *gK, float2 *part, int B, int C, int S,
                            hipStream_t s) {
  hipError_t err = hipErrorInvalidValue;
  const int J = S / C;
  const SmallPlan p = small_plan(n, m, B, C, J);
  const long long grid = (long long)C * p.R;
  if (grid >= (1LL << 31)) return err;
  float2 *dst = gK == nullptr ? nullptr : (p.parts ? part : gK);
  dispatch_small(n, m, [&](auto nc, auto mc) {
    constexpr int N = decltype(nc)::value, M = decltype(mc)::value;
    static const std::string nm = "small_bwd_" + std::to_string(N) + "_" + std::to_string(M);
    auto go = [&](auto jpc, auto njc) {
      constexpr int JP = decltype(jpc)::value, NJ = decltype(njc)::value;
      using G = SmallBwd<N, M, JP>;
      constexpr size_t lds = (size_t)G::END * sizeof(float2);
      static_assert(lds <= 160 * 1024, "small layer backward: LDS");
      err = allow_lds<k_small_bwd<N, M, JP, NJ>>(lds);
      if (err != hipSuccess) return;
      err = timed_launch(nm.c_str(), k_small_bwd<N, M, JP, NJ>, dim3((unsigned)grid), dim3(G::NT), lds, s, gy, view,
                         out_plane, saved, K, gx, dst, B, C, J, p.R, p.parts);
    };
    if constexpr (M <= 32) {
      if (p.JP == 4) {
        if (p.NJ == 1) go(Int<4>{}, Int<1>{});
        else go(Int<4>{}, Int<0>{});
        return;
      }
      if (p.JP == 2) {
        if (p.NJ == 1) go(Int<2>{}, Int<1>{});
        else go(Int<2>{}, Int<0>{});
        return;
      }
    }
    if (p.NJ == 1) go(Int<1>{}, Int<1>{});
    else go(Int<1>{}, Int<0>{});
  });
  if (err != hipSuccess || gK == nullptr || !p.parts) return err;
  return launch_gk_reduce2(part, gK, S, m, n, nullptr, nullptr, 0, 0, 0, p.R, s);
}

}  // namespace fdc
