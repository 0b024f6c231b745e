// Full FDC (Algorithm 2 with the per-bin sum over input channels of Eq. 2) on the
// fp32 matrix cores of gfx950, and its backward.
//
// At every frequency bin (k, l) of the P x (P/2+1) half spectrum the layer is a
// small complex matrix product over the batch:
//   forward  Y[b][s] = sum_c X[b][c] K[s][c]            (M = b, N = s, K-dim = c)
//   dL/dX    gX[b][c] = sum_s G[b][s] conj(K[s][c])      (M = b, N = c, K-dim = s)
//   dL/dK    gK[s][c] = sum_b G[b][s] conj(X[b][c])      (M = s, N = c, K-dim = b)
// with K[s][c](k, l) = sum_{a,b < n} w[s][c][a][b] W^(k a) W^(l b), W = e^{-2 pi i / P}:
// the n x n spatial kernel padded at the top-left corner to P x P and transformed
// (section 2.4.1.2).  K is never stored: each lane forms the element it feeds to the
// matrix core from the n*n weights and the bin's phases, so the contraction reads
// only X (or G) and the weights.  dL/dw is the adjoint of that map restricted to the
// n x n support, dL/dw[s][c][a][b] = Re sum_bins gK[s][c] conj(W^(k a) W^(l b)),
// accumulated per bin chunk and reduced in a fixed order.
//
// Spectra use the split layout of a P x (P/2+1) half spectrum: a main block of
// P x P/2 planes (columns 0..P/2-1) followed by a side block of P-element planes (the
// Nyquist column l = P/2), so that runs of 4 bins are 32-byte aligned.  In the main
// block row k of every plane lies side by side (full_spec_layout), so the planes a
// run's contraction reads are a few MB apart rather than a plane apart.
//
// Lane layout of v_mfma_f32_16x16x4f32 (A 16x4, B 4x16, D 16x16): lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and D[4 (l / 16) + j][l % 16] in register j.
#include "device.h"
#include "internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>

namespace fdc {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <class F>
__device__ __forceinline__ void static_for4(F &&f) {
  f(std::integral_constant<int, 0>{});
  f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{});
  f(std::integral_constant<int, 3>{});
}

// Taps of an n x n kernel, padded to a multiple of 4 for whole 16-byte loads.
template <int NK>
__host__ __device__ constexpr int tap_pad() {
  return (NK * NK + 3) & ~3;
}

// ---------------------------------------------------------------------------
// Forward (gx = false) and dL/dX (gx = true) contraction on split-layout spectra.
//   in  [B][KD] spectra: X (KD = Cin) or G (KD = Cout)
//   wt  weights rearranged as [KDp][NDp][TP], zero-padded (forward: [c][s][tap];
//       dL/dX: [s][c][tap]); KDp = KD rounded up to 4, NDp = ND rounded up to 64
//   out [B][ND] spectra: Y (ND = Cout) or gX (ND = Cin)
//
// Matrix-core tiles.  Rows m of a 16 x 16 x 4 tile are 8 images in real and imaginary
// part, m = 2 b + part, columns 16 outputs, depth 4 channels:
//   D += A1 Kr + A2 Ki,  A1 = (Xr; Xi),  A2 = (-Xi; Xr)   (conj K: A2 = (Xi; -Xr)),
// so a tile holds 8 images (with a row per image, 4 images filled 4 of 16 rows and took
// the time of 16), and a lane's four D registers are two images' complex values.
//
// Bins.  The weights are real, so rows k and -k of the kernel spectrum share
// C_b = sum_a w_ab W^(k a) (conjugated for -k):
//   K(+-k, l) = p -+ q + i (t +- r),  with v_b = W^(l b):
//   p = sum Re v Re C, q = sum Im v Im C, r = sum Re v Im C, t = sum Im v Re C,
// 12 operations for two bins at 3 x 3 taps (22 when each bin is formed from C alone).  A
// workgroup (4 waves) owns the row pair (k, -k) and 4 LB columns, LB a wave; each 4-channel
// step its threads form the C_b of 4 channels x 16 NTL outputs once, in LDS, for all waves.
// The Nyquist column (side block, l = P/2) takes the same form with the roles of rows and
// columns exchanged: C_a = R_a = sum_b (-1)^b w_ab is real, v_a = W^(k a), K(-k) = conj K(k).
//
// What bounds it: matrix and vector issue together.  On gfx950 fp32 MFMA and vector
// instructions of one SIMD do not overlap, not even from different waves (a probe of both:
// 6.3 ms together, 4.6 and 2.3 ms alone), so a step of 64 MFMAs (2048 cycles) and 160 vector
// instructions (640 cycles) takes at least their sum; measured 3200-3500 cycles, i.e. 80 %.
// Before (a row per image, bins singly): 16 images of 224^2, 64 -> 64 channels 225 -> 203 us;
// 4 images of 512^2, 128 -> 128 channels 3.0 -> 1.68 ms; 3 images of 128^2, 48 -> 80 channels,
// 5 x 5 taps 164 -> 64 us.  BT 8-image tiles share each K: BT = 1 with LB = 4 columns up to 8 images,
// BT = 2 with LB = 2 beyond (the same 32 NTL accumulator registers: two waves a SIMD).
// Every load is unconditional: images and channels past the end are clamped to the last
// valid ones (their weights are zero, their outputs are not stored).
// ---------------------------------------------------------------------------
constexpr int kCtOut = 64;  // output padding of the rearranged weights, and the widest tile group

// LDS of one step's C: [NK][4 channels][64 outputs and 16 of padding] (the padding puts the
// channels of a wave's read on different banks), two steps' buffers.
constexpr int kCtRow = kCtOut + 16;
template <int NK>
constexpr int ct_lds_elems() {
  return 2 * NK * 4 * kCtRow;
}

// The workgroup's C_b of 4 channels x 16 NTL outputs (from n0): each thread loads the weights
// of one (channel, output) and forms its C_b (SIDE: R_a) into one of the two step buffers.
template <int NK, int NTL, bool SIDE>
struct KernelRows {
  static constexpr int TP = tap_pad<NK>();
  const float *w0;
  long long kstride;
  float2 *dst;
  float2 u[NK];  // W^(k a)
  float4 wn[TP / 4];
  bool mine;
  __device__ __forceinline__ KernelRows(const float *wt, const float2 *tw, float2 *cbuf, int NDp, int n0, int P,
                                        int k) {
    const int ck = threadIdx.x / (16 * NTL), cn = threadIdx.x % (16 * NTL);
    mine = ck < 4;
    w0 = wt + ((long long)(mine ? ck : 0) * NDp + n0 + cn) * TP;
    kstride = (long long)NDp * TP;
    dst = cbuf + (mine ? ck : 0) * kCtRow + cn;
#pragma unroll
    for (int a = 1; a < NK; ++a) u[a] = SIDE ? make_float2(0.f, 0.f) : tw[(k * a) % P];
  }
  __device__ __forceinline__ void load(int k0) {
    const float4 *w4 = reinterpret_cast<const float4 *>(w0 + k0 * kstride);
#pragma unroll
    for (int i = 0; i < TP / 4; ++i) wn[i] = w4[i];
  }
  __device__ __forceinline__ void form(int buf) const {
    float w[TP];
#pragma unroll
    for (int i = 0; i < TP / 4; ++i)
      w[4 * i] = wn[i].x, w[4 * i + 1] = wn[i].y, w[4 * i + 2] = wn[i].z, w[4 * i + 3] = wn[i].w;
    if (!mine) return;
    float2 *d = dst + buf * NK * 4 * kCtRow;
    if constexpr (!SIDE) {
#pragma unroll
      for (int b = 0; b < NK; ++b) {  // C_b = w_0b + sum_{a>=1} w_ab u_a
        float cx = w[b], cy = 0.f;
#pragma unroll
        for (int a = 1; a < NK; ++a) {
          cx = fmaf(w[a * NK + b], u[a].x, cx);
          cy = fmaf(w[a * NK + b], u[a].y, cy);
        }
        d[b * 4 * kCtRow] = make_float2(cx, cy);
      }
    } else {
#pragma unroll
      for (int a = 0; a < NK; ++a) {  // R_a = sum_b (-1)^b w_ab
        float r = w[a * NK];
#pragma unroll
        for (int b = 1; b < NK; ++b) r += (b & 1) ? -w[a * NK + b] : w[a * NK + b];
        d[a * 4 * kCtRow] = make_float2(r, 0.f);
      }
    }
  }
};

// Kernel spectrum at rows +-k (SIDE: rows +-r) of one column (row) from its C (R) and phases
// v_b = zc + i zs: kr, ki[0] for +, [1] for -.
template <int NK, bool SIDE>
__device__ __forceinline__ void kernel_pair(const float2 (&c)[NK], const float (&zc)[NK], const float (&zs)[NK],
                                            float (&kr)[2], float (&ki)[2]) {
  float p = c[0].x, t = 0.f;
#pragma unroll
  for (int b = 1; b < NK; ++b) {
    p = fmaf(zc[b], c[b].x, p);
    t = b == 1 ? zs[b] * c[b].x : fmaf(zs[b], c[b].x, t);
  }
  if constexpr (!SIDE) {
    float r = c[0].y, q = 0.f;
#pragma unroll
    for (int b = 1; b < NK; ++b) {
      r = fmaf(zc[b], c[b].y, r);
      q = b == 1 ? zs[b] * c[b].y : fmaf(zs[b], c[b].y, q);
    }
    kr[0] = p - q, kr[1] = p + q;
    ki[0] = t + r, ki[1] = t - r;
  } else {
    kr[0] = kr[1] = p;
    ki[0] = t, ki[1] = -t;
  }
}

// One workgroup's bins: main, row pair (k, P - k) and columns l0..l0 + LB - 1 of this wave;
// SIDE, rows l0..l0 + LB - 1 <= P/2 and their negatives of the Nyquist column.
template <int NK, int BT, int NTL, bool SIDE>
__device__ __forceinline__ void contract_bins(const SpecLayout &in, const float *__restrict__ wt,
                                              const float2 *__restrict__ tw, const SpecLayout &out, float2 *cbuf,
                                              int B, int KD, int KDp, int ND, int NDp, int P, bool gx, int k, int l0,
                                              int b0, int n0) {
  constexpr int LB = BT == 1 ? 4 : 2;
  const int H = P / 2;
  const int lane = threadIdx.x & 63, mrow = lane & 15, kk = lane >> 4;
  const bool valid = SIDE ? l0 <= H : l0 < H;  // this wave's bins (idle waves run along, storing nothing)
  if (!valid) l0 = 0;

  // v_b at this wave's columns (SIDE: rows)
  float zc[LB][NK], zs[LB][NK];
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const int l = SIDE ? min(l0 + q, H) : l0 + q;
#pragma unroll
    for (int b = 1; b < NK; ++b) {
      const float2 z = tw[(l * b) % P];
      zc[q][b] = z.x, zs[q][b] = z.y;
    }
  }
  KernelRows<NK, NTL, SIDE> rows(wt, tw, cbuf, NDp, n0, P, k);

  // the inputs of this lane: image b0 + 8 i + mrow / 2 of tile i, channel k0 + kk, both rows
  const float2 *xr[BT];
#pragma unroll
  for (int i = 0; i < BT; ++i) {
    const long long plane = (long long)min(b0 + 8 * i + (mrow >> 1), B - 1) * KD;
    xr[i] = SIDE ? in.side + plane * in.sps : in.main + plane * in.ps + l0;
  }
  const long long chs = SIDE ? in.sps : in.ps;
  const long long row0 = SIDE ? 0 : k * in.rs, row1 = SIDE ? 0 : (k == 0 ? 0 : P - k) * in.rs;
  float2 xn[BT][2][LB];
  auto load_x = [&](int k0) {
    const long long co = (long long)min(k0 + kk, KD - 1) * chs;
#pragma unroll
    for (int i = 0; i < BT; ++i) {
      if constexpr (!SIDE) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const float4 *a4 = reinterpret_cast<const float4 *>(xr[i] + co + (s ? row1 : row0));
#pragma unroll
          for (int q = 0; q < LB; q += 2) {
            const float4 a = a4[q / 2];
            xn[i][s][q] = make_float2(a.x, a.y), xn[i][s][q + 1] = make_float2(a.z, a.w);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < LB; ++q) {
          const int r = min(l0 + q, H);
          xn[i][0][q] = xr[i][co + r];
          xn[i][1][q] = xr[i][co + (r == 0 ? 0 : P - r)];
        }
      }
    }
  };

  v4f acc[BT][2][LB][NTL];
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < LB; ++q)
#pragma unroll
        for (int t = 0; t < NTL; ++t) acc[i][s][q][t] = v4f{0.f, 0.f, 0.f, 0.f};

  const bool im = mrow & 1;
  const unsigned flip = (im == gx) ? 0x80000000u : 0u;  // sign of A2: -Xi on real rows, conj K the other way round
  rows.load(0);
  load_x(0);
  rows.form(0);
  rows.load(min(4, KDp - 4));
  __syncthreads();
  for (int k0 = 0; k0 < KDp; k0 += 4) {
    const int buf = (k0 >> 2) & 1;
    float a1[BT][2][LB], a2[BT][2][LB];
#pragma unroll
    for (int i = 0; i < BT; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < LB; ++q) {
          const float2 v = xn[i][s][q];
          a1[i][s][q] = im ? v.y : v.x;
          a2[i][s][q] = __uint_as_float(__float_as_uint(im ? v.x : v.y) ^ flip);
          // formed here, so that the next loads can take the registers of xn: otherwise they
          // are sunk past those loads, which then go to other registers and are copied back
          // within this step, behind a wait for the loads just issued
          asm volatile("" : "+v"(a1[i][s][q]), "+v"(a2[i][s][q]));
        }
    __builtin_amdgcn_sched_barrier(0);
    // the next step's C (its weights arrived during the last step), inputs and weights; past
    // the last step the last one's again, unused
    load_x(min(k0 + 4, KDp - 4));
    rows.form(buf ^ 1);
    rows.load(min(k0 + 8, KDp - 4));
    const float2 *cb = cbuf + buf * NK * 4 * kCtRow + kk * kCtRow + mrow;
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      float2 c[NK];
#pragma unroll
      for (int b = 0; b < NK; ++b) c[b] = cb[b * 4 * kCtRow + 16 * t];
      float kr[2][LB], ki[2][LB];
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        float r2[2], i2[2];
        kernel_pair<NK, SIDE>(c, zc[q], zs[q], r2, i2);
        kr[0][q] = r2[0], kr[1][q] = r2[1], ki[0][q] = i2[0], ki[1][q] = i2[1];
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < LB; ++q)
#pragma unroll
          for (int i = 0; i < BT; ++i) acc[i][s][q][t] = mfma4(a1[i][s][q], kr[s][q], acc[i][s][q][t]);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < LB; ++q)
#pragma unroll
          for (int i = 0; i < BT; ++i) acc[i][s][q][t] = mfma4(a2[i][s][q], ki[s][q], acc[i][s][q][t]);
    }
    __syncthreads();
  }
  if (!valid) return;
  // D rows 4 (lane / 16) + j: images 2 (lane / 16) (registers 0, 1) and the next (2, 3)
#pragma unroll
  for (int i = 0; i < BT; ++i)
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const int n = n0 + 16 * t + mrow;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int b = b0 + 8 * i + 2 * kk + j;
        if (b >= B || n >= ND) continue;
        const long long plane = (long long)b * ND + n;
        if constexpr (!SIDE) {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            if (s == 1 && (k == 0 || k == H)) continue;  // the pair is one row
            float4 *o = reinterpret_cast<float4 *>(out.main + plane * out.ps + (s ? P - k : k) * out.rs + l0);
#pragma unroll
            for (int q = 0; q < LB; q += 2)
              o[q / 2] = make_float4(acc[i][s][q][t][2 * j], acc[i][s][q][t][2 * j + 1], acc[i][s][q + 1][t][2 * j],
                                     acc[i][s][q + 1][t][2 * j + 1]);
          }
        } else {
          float2 *o = out.side + plane * out.sps;
#pragma unroll
          for (int q = 0; q < LB; ++q) {
            const int r = l0 + q;
            if (r > H) continue;
            o[r] = make_float2(acc[i][0][q][t][2 * j], acc[i][0][q][t][2 * j + 1]);
            if (r != 0 && r != H)
              o[P - r] = make_float2(acc[i][1][q][t][2 * j], acc[i][1][q][t][2 * j + 1]);
          }
        }
      }
    }
}

// The same for at most 4 images, on v_mfma_f32_4x4x1f32 (16 blocks of 4 x 4 x 1, 8 cycles, the
// rate of the larger tiles): rows are the 4 images, a block's columns 4 outputs, so a wave
// takes 64 outputs (lane n) and no row is idle: 32 cycles for 64 kernel bins where a half-empty
// 16 x 16 tile takes 64.  The A operand comes from one block, broadcast to all 16 (CBSZ = 4,
// ABID): block b of a lane's load holds channel b / 4, row +-k (b / 2 % 2) and columns
// 2 (b % 2), 2 (b % 2) + 1 of the wave's four, one 16-byte load a 4-channel step.
// A 4-channel step is 128 MFMAs (1024 cycles) and 192 vector instructions for K (768).
template <int NK, bool SIDE>
__device__ __forceinline__ void contract4_bins(const SpecLayout &in, const float *__restrict__ wt,
                                               const float2 *__restrict__ tw, const SpecLayout &out, float2 *cbuf,
                                               int B, int KD, int KDp, int ND, int NDp, int P, bool gx, int k, int l0,
                                               int b0, int n0) {
  constexpr int LB = 4;
  const int H = P / 2;
  const int lane = threadIdx.x & 63, blk = lane >> 2;
  const bool valid = SIDE ? l0 <= H : l0 < H;
  if (!valid) l0 = 0;

  float zc[LB][NK], zs[LB][NK];
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const int l = SIDE ? min(l0 + q, H) : l0 + q;
#pragma unroll
    for (int b = 1; b < NK; ++b) {
      const float2 z = tw[(l * b) % P];
      zc[q][b] = z.x, zs[q][b] = z.y;
    }
  }
  KernelRows<NK, 4, SIDE> rows(wt, tw, cbuf, NDp, n0, P, k);

  // this lane's inputs: image b0 + lane % 4, channel k0 + blk / 4, row +-k, two columns
  const int ch = blk >> 2, xs = (blk >> 1) & 1, xh = 2 * (blk & 1);
  const long long plane = (long long)min(b0 + (lane & 3), B - 1) * KD;
  const float2 *xp;
  int off1 = 0;  // SIDE: the second bin relative to the first
  if constexpr (!SIDE) {
    xp = in.main + plane * in.ps + (long long)(xs ? (k == 0 ? 0 : P - k) : k) * in.rs + l0 + xh;
  } else {
    const int r0 = min(l0 + xh, H), r1 = min(l0 + xh + 1, H);
    const int e0 = xs ? (r0 == 0 ? 0 : P - r0) : r0, e1 = xs ? (r1 == 0 ? 0 : P - r1) : r1;
    xp = in.side + plane * in.sps + e0;
    off1 = e1 - e0;
  }
  const long long chs = SIDE ? in.sps : in.ps;
  float4 xn;
  auto load_x = [&](int k0) {
    const float2 *q = xp + min(k0 + ch, KD - 1) * chs;
    if constexpr (!SIDE) {
      xn = *reinterpret_cast<const float4 *>(q);
    } else {
      const float2 u = q[0], v = q[off1];
      xn = make_float4(u.x, u.y, v.x, v.y);
    }
  };

  v4f ar[2][LB], ai[2][LB];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < LB; ++q) ar[s][q] = ai[s][q] = v4f{0.f, 0.f, 0.f, 0.f};

  rows.load(0);
  load_x(0);
  rows.form(0);
  rows.load(min(4, KDp - 4));
  __syncthreads();
  for (int k0 = 0; k0 < KDp; k0 += 4) {
    const int buf = (k0 >> 2) & 1;
    // re += Xr Kr + pr Ki, im += Xi Kr + pi Ki:  (pr, pi) = (-Xi, Xr), conj K: (Xi, -Xr)
    float xr[2], xi[2], pr[2], pi[2];
    xr[0] = xn.x, xi[0] = xn.y, xr[1] = xn.z, xi[1] = xn.w;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      pr[e] = gx ? xi[e] : -xi[e], pi[e] = gx ? -xr[e] : xr[e];
      // (formed before the next loads, see contract_bins)
      asm volatile("" : "+v"(xr[e]), "+v"(xi[e]), "+v"(pr[e]), "+v"(pi[e]));
    }
    __builtin_amdgcn_sched_barrier(0);
    load_x(min(k0 + 4, KDp - 4));
    rows.form(buf ^ 1);
    rows.load(min(k0 + 8, KDp - 4));
    const float2 *cb = cbuf + buf * NK * 4 * kCtRow + lane;
    static_for4([&](auto xc) {
      constexpr int x = decltype(xc)::value;
      float2 c[NK];
#pragma unroll
      for (int b = 0; b < NK; ++b) c[b] = cb[(b * 4 + x) * kCtRow];
      float kr[2][LB], ki[2][LB];
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        float r2[2], i2[2];
        kernel_pair<NK, SIDE>(c, zc[q], zs[q], r2, i2);
        kr[0][q] = r2[0], kr[1][q] = r2[1], ki[0][q] = i2[0], ki[1][q] = i2[1];
      }
      auto mul = [&](auto sc, auto hc) {
        constexpr int s = decltype(sc)::value, h = decltype(hc)::value, id = 4 * x + 2 * s + h;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int q = 2 * h + e;
          ar[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xr[e], kr[s][q], ar[s][q], 4, id, 0);
          ai[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xi[e], kr[s][q], ai[s][q], 4, id, 0);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int q = 2 * h + e;
          ar[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(pr[e], ki[s][q], ar[s][q], 4, id, 0);
          ai[s][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(pi[e], ki[s][q], ai[s][q], 4, id, 0);
        }
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      mul(I0{}, I0{});
      mul(I0{}, I1{});
      mul(I1{}, I0{});
      mul(I1{}, I1{});
    });
    __syncthreads();
  }
  const int n = n0 + lane;
  if (!valid || n >= ND) return;
  // D register r: image b0 + r of output n
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (b0 + r >= B) continue;
    const long long pl = (long long)(b0 + r) * ND + n;
    if constexpr (!SIDE) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (s == 1 && (k == 0 || k == H)) continue;  // the pair is one row
        float4 *o = reinterpret_cast<float4 *>(out.main + pl * out.ps + (s ? P - k : k) * out.rs + l0);
        o[0] = make_float4(ar[s][0][r], ai[s][0][r], ar[s][1][r], ai[s][1][r]);
        o[1] = make_float4(ar[s][2][r], ai[s][2][r], ar[s][3][r], ai[s][3][r]);
      }
    } else {
      float2 *o = out.side + pl * out.sps;
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        const int row = l0 + q;
        if (row > H) continue;
        o[row] = make_float2(ar[0][q][r], ai[0][q][r]);
        if (row != 0 && row != H) o[P - row] = make_float2(ar[1][q][r], ai[1][q][r]);
      }
    }
  }
}

// Workgroups per (output group, image tile): row pairs k = 0..P/2 times groups of 4 LB
// columns, then the Nyquist column's groups of 4 LB rows 0..P/2.
template <int BT>
__host__ __device__ constexpr int ct_cols() {
  return 4 * (BT == 1 ? 4 : 2);
}
static inline int ct_groups(int P, int cols) {
  const int H = P / 2;
  return (H + 1) * ((H + cols - 1) / cols) + (H + cols) / cols;
}

template <int NK, int BT, int NTL>
__global__ __launch_bounds__(256, 2) void k_full_contract(SpecLayout in, const float *__restrict__ wt,
                                                          const float2 *__restrict__ tw, SpecLayout out, int B, int KD,
                                                          int KDp, int ND, int NDp, int P, int gx, int ngroups,
                                                          int nsb, int b_first) {
  __shared__ float2 cbuf[ct_lds_elems<NK>()];
  constexpr int COLS = ct_cols<BT>();
  const int H = P / 2, ncg = (H + COLS - 1) / COLS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int sb = blk % nsb, rest = blk / nsb;
  const int g = rest % ngroups, b0 = b_first + (rest / ngroups) * 8 * BT, n0 = sb * 16 * NTL;
  if (g < (H + 1) * ncg) {
    const int k = g / ncg;
    contract_bins<NK, BT, NTL, false>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, k,
                                      (g - k * ncg) * COLS + wave * (COLS / 4), b0, n0);
  } else {
    contract_bins<NK, BT, NTL, true>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, 0,
                                     (g - (H + 1) * ncg) * COLS + wave * (COLS / 4), b0, n0);
  }
}

// 4 images, 64 outputs a workgroup (grid as k_full_contract with BT = 1, one image tile).
template <int NK>
__global__ __launch_bounds__(256, 3) void k_full_contract4(SpecLayout in, const float *__restrict__ wt,
                                                           const float2 *__restrict__ tw, SpecLayout out, int B,
                                                           int KD, int KDp, int ND, int NDp, int P, int gx, int nsb,
                                                           int b0) {
  __shared__ float2 cbuf[ct_lds_elems<NK>()];
  constexpr int COLS = ct_cols<1>();
  const int H = P / 2, ncg = (H + COLS - 1) / COLS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int g = blk / nsb, n0 = (blk - g * nsb) * kCtOut;
  if (g < (H + 1) * ncg) {
    const int k = g / ncg;
    contract4_bins<NK, false>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, k,
                              (g - k * ncg) * COLS + wave * 4, b0, n0);
  } else {
    contract4_bins<NK, true>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, 0,
                             (g - (H + 1) * ncg) * COLS + wave * 4, b0, n0);
  }
}

// ---------------------------------------------------------------------------
// dL/dw partial sums over one chunk of runs (runs as in the contraction).
//   G [B][S], X [B][C] split-layout spectra; part [chunk][S][C][NK*NK] float
// Per bin gK[s][c] = sum_b G[b][s] conj(X[b][c]) on the matrix cores (M = s, N = c,
// K-dim = b, 4 batch rows per step), then
//   dL/dw[s][c][a][b] = Re sum_bins gK conj(W^(k a) W^(l b)),
// done per run: a row run sums E_b = sum_q gK_q conj(W^(l_q b)) and adds
// Re(E_b conj(W^(k a))); a Nyquist run sums F_a = sum_q gK_q conj(W^(k_q a)) and adds
// (-1)^b Re(F_a).  A workgroup (4 waves) owns a 32 x 32 (s, c) block, each wave a
// 16 x 16 tile, and walks its chunk one run (4 bins) at a time, 4 batch rows per step.
// A step's G and X rows are loaded once per workgroup and staged in LDS, and the
// loads of step t + 2 are in flight while step t computes.  Loads are unconditional:
// batch rows past the end are clamped and staged as zeros, channels and runs past the
// end are clamped and their results dropped.
// ---------------------------------------------------------------------------
// Twiddles W^i for i < n P in LDS: every phase index the projection forms (k a,
// (l + q) b with k < P, l + q < P/2, a, b < n) is then a plain table index.
template <int NK>
__host__ __device__ constexpr int gw_tw_elems(int P) {
  return (NK * P + 31) & ~31;
}

// Adds one run's gK (4 bins: dr/di[q], lane rows j) projected onto the taps to gw.
// Row run (k, l0..l0+3); Nyquist run (k0..k0+3, P/2) when SIDE.  The phases of tap
// row / column 0 are exactly 1, so their products are plain sums.
template <int NK, bool SIDE>
__device__ __forceinline__ void gw_project_run(float (&gw)[4][NK * NK], const v4f (&dr)[4], const v4f (&di)[4], int k,
                                               int l0, const float2 *tw) {
  if constexpr (!SIDE) {
    float2 u[NK], v[4][NK];
#pragma unroll
    for (int a = 1; a < NK; ++a) u[a] = tw[k * a];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int b = 1; b < NK; ++b) v[q][b] = tw[(l0 + q) * b];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int b = 0; b < NK; ++b) {
        float ex, ey;  // E_b = sum_q D_q conj(v_qb)
        if (b == 0) {
          ex = (dr[0][j] + dr[1][j]) + (dr[2][j] + dr[3][j]);
          ey = (di[0][j] + di[1][j]) + (di[2][j] + di[3][j]);
        } else {
          ex = ey = 0.f;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            ex = fmaf(dr[q][j], v[q][b].x, ex);
            ex = fmaf(di[q][j], v[q][b].y, ex);
            ey = fmaf(di[q][j], v[q][b].x, ey);
            ey = fmaf(-dr[q][j], v[q][b].y, ey);
          }
        }
        gw[j][b] += ex;
#pragma unroll
        for (int a = 1; a < NK; ++a) gw[j][a * NK + b] = fmaf(ey, u[a].y, fmaf(ex, u[a].x, gw[j][a * NK + b]));
      }
  } else {
    float2 u[4][NK];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int a = 1; a < NK; ++a) u[q][a] = tw[(k + q) * a];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int a = 0; a < NK; ++a) {
        float f;  // Re F_a = Re sum_q D_q conj(u_qa)
        if (a == 0) {
          f = (dr[0][j] + dr[1][j]) + (dr[2][j] + dr[3][j]);
        } else {
          f = 0.f;
#pragma unroll
          for (int q = 0; q < 4; ++q) f = fmaf(di[q][j], u[q][a].y, fmaf(dr[q][j], u[q][a].x, f));
        }
#pragma unroll
        for (int b = 0; b < NK; ++b) gw[j][a * NK + b] += (b & 1) ? -f : f;
      }
  }
}

// Position of a run of 4 bins, advanced one run at a time (no divisions on the way).
struct GwRun {
  int g, k, l0;  // run index; row k and first column l0 (row runs) or first row k (Nyquist runs)
  __device__ void start(int g0, int nmain, int H) {
    g = g0;
    if (g < nmain) {
      k = (4 * g) / H, l0 = 4 * g - k * H;
    } else {
      k = 4 * (g - nmain), l0 = 0;
    }
  }
  __device__ void next(int nmain, int H) {
    ++g;
    if (g == nmain) {
      k = 0, l0 = 0;
    } else if (g > nmain) {
      k += 4;
    } else if ((l0 += 4) == H) {
      l0 = 0, ++k;
    }
  }
};

// LDS staging of one step (4 batch rows, one run of 4 bins) for a 32 x 32 (s, c)
// block: G rows [4][32][5] and X rows [4][32][5] complex, each (b, s) row holding the
// run's 4 bins and one of padding.  Every element is loaded from memory once per
// workgroup (the four waves read each operand row twice: waves 0/1 share s rows, 0/2
// share c rows).
constexpr int kGwStageRow = 5;
// X rows start 8 elements (16 banks of 4 bytes) after the G rows: the staging writes of
// a 16-lane group (8 rows of G and the same 8 rows of X) then fall on distinct banks
// (with the two blocks a multiple of 32 banks apart every write was a 2-way conflict)
constexpr int kGwStageUnit = 4 * 32 * kGwStageRow + 8;
constexpr int kGwStageElems = 2 * kGwStageUnit;

// EVEN: the batch takes an even number of 4-row steps (B rounded up to 4 is a multiple
// of 8), which allows the run-by-run loop.
template <int NK, bool EVEN>
__global__ __launch_bounds__(256, 2) void k_full_gw(SpecLayout G, SpecLayout X, const float2 *__restrict__ twg,
                                                 float *__restrict__ part, int B, int S, int C, int P,
                                                 int runs_per_chunk) {
  constexpr int T = NK * NK, SR = kGwStageRow, SE = kGwStageElems;
  extern __shared__ float smem[];
  float2 *tw = reinterpret_cast<float2 *>(smem);
  float2 *stage = tw + gw_tw_elems<NK>(P);  // two buffers of SE
  for (int i = threadIdx.x; i < NK * P; i += 256) tw[i] = twg[i % P];
  __syncthreads();

  const int H = P / 2, nmain = P * H / 4, nrun = nmain + P / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mrow = lane & 15, kq = lane >> 4;
  const int sblocks = (S + 31) / 32, cblocks = (C + 31) / 32;
  const int blk = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = blk % (sblocks * cblocks), chunk = blk / (sblocks * cblocks);
  const int sbase = (tile / cblocks) * 32, cbase = (tile % cblocks) * 32;
  const int s0 = sbase + (wave >> 1) * 16, c0 = cbase + (wave & 1) * 16;
  const int r_begin = chunk * runs_per_chunk, r_end = min(nrun, r_begin + runs_per_chunk);

  // Cooperative loads: wave lb takes batch row b0 + lb of the step; lane (lr, unit)
  // loads the run's 4 bins of G row sbase + lr (unit 0) or X row cbase + lr (unit 1).
  // Per-lane bases and batch strides of both blocks, so that a step's address is one
  // multiply-add.
  const int lb = wave, unit = lane & 1, lr = lane >> 1;
  const SpecLayout &L = unit ? X : G;
  const long long row = unit ? min(cbase + lr, C - 1) : min(sbase + lr, S - 1);
  const long long nch = unit ? C : S;
  const float2 *mbase = L.main + row * L.ps, *sbase_p = L.side + row * L.sps;
  const long long mbst = nch * L.ps, sbst = nch * L.sps, mrs = L.rs;

  float gw[4][T];  // rows s0 + 4 (lane / 16) + j, column c0 + lane % 16
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < T; ++t) gw[j][t] = 0.f;

  // Two register sets hold the loads of the next two steps, so that the loads of step
  // t + 2 are in flight while step t computes.  Past the chunk's last step the run is
  // clamped and the load is not used: an unconditional load keeps the wait counts
  // exact, so step t waits for its own loads only.
  GwRun lrun;
  lrun.start(r_begin, nmain, H);
  int lb0 = 0;  // load cursor: run lrun, batch rows lb0..lb0+3
  auto load_next = [&](float4(&r)[2]) {
    const long long bc = min(lb0 + lb, B - 1);
    const bool side = lrun.g >= nmain;
    const int gk = min(lrun.k, side ? P - 4 : P - 1);  // in range past the last run
    const float2 *a = side ? sbase_p + bc * sbst + gk : mbase + bc * mbst + gk * mrs + lrun.l0;
    const float4 *a4 = reinterpret_cast<const float4 *>(a);
    r[0] = a4[0], r[1] = a4[1];
    lb0 += 4;
    if (lb0 >= B) lb0 = 0, lrun.next(nmain, H);
  };
  float4 ra[2], rb[2];
  load_next(ra);
  load_next(rb);
  // Up to 3 x 3 taps and with the run-by-run loop, Gauss's form of the complex
  // product: t1 = sum Gr Xr, t2 = sum Gi Xi and t3 = sum (Gr + Gi)(Xr - Xi) over the
  // batch, three matrix products per bin instead of four; the run's D = G conj(X) is
  // then re = t1 + t2, im = t3 - t1 + t2.  (Elsewhere the third accumulator would
  // cost occupancy or spill, and four products are kept.)
  constexpr bool kGauss = EVEN && NK <= 3;
  v4f t1[4], t2[4], t3[4], dr[4], di[4];
  GwRun crun;
  crun.start(r_begin, nmain, H);
  int b0 = 0;  // compute cursor
  // Stage the registers r (loaded two steps ago) into LDS buffer buf, then this step's
  // products (4 batch rows of the run crun).
  auto stage_and_multiply = [&](float4(&r)[2], int buf) __attribute__((always_inline)) {
    // (the barrier below also ends every wave's reads of this buffer two steps ago)
    {
      float2 *d = stage + buf * SE + unit * kGwStageUnit + (lb * 32 + lr) * SR;
      if (b0 + lb < B) {
        d[0] = make_float2(r[0].x, r[0].y), d[1] = make_float2(r[0].z, r[0].w);
        d[2] = make_float2(r[1].x, r[1].y), d[3] = make_float2(r[1].z, r[1].w);
      } else {  // batch rows past the end add nothing
        d[0] = d[1] = d[2] = d[3] = make_float2(0.f, 0.f);
      }
    }
    __syncthreads();
    load_next(r);
    const float2 *ag = stage + buf * SE + (kq * 32 + (s0 - sbase) + mrow) * SR;
    const float2 *ax = stage + buf * SE + kGwStageUnit + (kq * 32 + (c0 - cbase) + mrow) * SR;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float2 g2 = ag[q], x2 = ax[q];
      if constexpr (kGauss) {
        t1[q] = mfma4(g2.x, x2.x, t1[q]);
        t2[q] = mfma4(g2.y, x2.y, t2[q]);
        t3[q] = mfma4(g2.x + g2.y, x2.x - x2.y, t3[q]);
      } else {  // D = G conj(X):  re = Gr Xr + Gi Xi,  im = Gi Xr - Gr Xi
        dr[q] = mfma4(g2.x, x2.x, dr[q]);
        dr[q] = mfma4(g2.y, x2.y, dr[q]);
        di[q] = mfma4(g2.y, x2.x, di[q]);
        di[q] = mfma4(-g2.x, x2.y, di[q]);
      }
    }
    b0 += 4;
  };
  auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (kGauss)
        t1[q] = t2[q] = t3[q] = v4f{0.f, 0.f, 0.f, 0.f};
      else
        dr[q] = di[q] = v4f{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto finish_run = [&]() __attribute__((always_inline)) {  // project the run onto the taps
    if constexpr (kGauss) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        dr[q] = t1[q] + t2[q];
        di[q] = (t3[q] - t1[q]) + t2[q];
      }
    }
    if (crun.g >= nmain)
      gw_project_run<NK, true>(gw, dr, di, crun.k, crun.l0, tw);
    else
      gw_project_run<NK, false>(gw, dr, di, crun.k, crun.l0, tw);
    b0 = 0;
    crun.next(nmain, H);
  };
  const int spr = (B + 3) / 4;  // steps per run
  if constexpr (EVEN) {
    // An even step count per run (the launcher checks): a run is whole pairs of steps,
    // so the register sets alternate inside it, and the sums are cleared before and
    // projected after it, with no branch on them inside the step loop.
    for (int g = r_begin; g < r_end; ++g) {
      clear_sums();
      for (int t = 0; t < spr; t += 2) {  // one path round the loop keeps the wait counts exact
        stage_and_multiply(ra, 0);
        stage_and_multiply(rb, 1);
      }
      finish_run();
    }
  } else {
    auto step = [&](float4(&r)[2], int buf) __attribute__((always_inline)) {
      if (b0 == 0) clear_sums();
      stage_and_multiply(r, buf);
      if (b0 >= B) finish_run();
    };
    const int nsteps = max(0, r_end - r_begin) * spr;
    int t = 0;
    for (; t + 1 < nsteps; t += 2) {  // one path round the loop keeps the wait counts exact
      step(ra, 0);
      step(rb, 1);
    }
    if (t < nsteps) step(ra, 0);
  }
  // this chunk's partial sums
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int os = s0 + 4 * kq + j, oc = c0 + mrow;
    if (os >= S || oc >= C) continue;
    float *p = part + (((long long)chunk * S + os) * C + oc) * T;
#pragma unroll
    for (int t = 0; t < T; ++t) p[t] = gw[j][t];
  }
}

// dL/dw = sum over chunks in a fixed order: a workgroup owns 64 outputs; its four
// waves sum the chunks congruent to 0, 1, 2, 3 mod 4 (four accumulators each, chunk
// c into accumulator (c / 4) mod 4), and the 16 partial sums are added in order.
__global__ __launch_bounds__(256) void k_full_gw_reduce(const float *__restrict__ part, float *__restrict__ gw,
                                                        long long n, int chunks) {
  __shared__ float red[4][64];
  const int o = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long i = (long long)blockIdx.x * 64 + o;
  const long long ii = i < n ? i : n - 1;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  int c = w;
  for (; c + 12 < chunks; c += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += part[(long long)(c + 4 * u) * n + ii];
  }
  for (int u = 0; c < chunks; c += 4, ++u) acc[u] += part[(long long)c * n + ii];
  red[w][o] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (w == 0 && i < n) gw[i] = (red[0][o] + red[1][o]) + (red[2][o] + red[3][o]);
}

// Weights rearranged for the contraction, zero-padded: wt[kd][nd][tap] of
// [KDp][NDp][TP] with w[s][c][tap] at (kd, nd) = (c, s) forward, (s, c) for dL/dX.
__global__ void k_full_weights(const float *__restrict__ w, float *__restrict__ wt, int S, int C, int T, int TP,
                               int gx, int KDp, int NDp) {
  const int KD = gx ? S : C, ND = gx ? C : S;
  const long long n = (long long)KDp * NDp * TP;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const int tap = (int)(i % TP);
    const long long r = i / TP;
    const int nd = (int)(r % NDp), kd = (int)(r / NDp);
    float v = 0.f;
    if (kd < KD && nd < ND && tap < T) {
      const int s_ = gx ? kd : nd, c_ = gx ? nd : kd;
      v = w[((long long)s_ * C + c_) * T + tap];
    }
    wt[i] = v;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <class F>
static bool dispatch_nk(int nk, F &&f) {
  switch (nk) {
    case 1: f(std::integral_constant<int, 1>{}); return true;
    case 2: f(std::integral_constant<int, 2>{}); return true;
    case 3: f(std::integral_constant<int, 3>{}); return true;
    case 4: f(std::integral_constant<int, 4>{}); return true;
    case 5: f(std::integral_constant<int, 5>{}); return true;
    default: return false;
  }
}

bool full_kernel_size_supported(int nk) { return nk >= 1 && nk <= 5; }

bool full_launch_fits(int B, int Cin, int Cout, int P, int nk) {
  if (P % 8 != 0 || B < 1 || B > 65535 * 16) return false;
  const long long nrun = (long long)P * (P / 2) / 4 + P / 4;
  const long long nwg_run = (nrun + 3) / 4, nbt = (B + 15) / 16;
  const long long lim = 1LL << 31;
  // the two contractions
  if (nwg_run * ((Cout + kCtOut - 1) / kCtOut) * nbt >= lim) return false;
  if (nwg_run * ((Cin + kCtOut - 1) / kCtOut) * nbt >= lim) return false;
  // dL/dw: tiles of 32 x 32 (s, c) times bin chunks, and the fixed-order reduction
  const long long tiles = (long long)((Cout + 31) / 32) * ((Cin + 31) / 32);
  if (tiles * full_gw_chunks(B, Cout, Cin, P, nk) >= lim) return false;
  if (((long long)Cout * Cin * nk * nk + 63) / 64 >= lim) return false;
  return true;
}

static int round_up(int v, int m) { return (v + m - 1) / m * m; }
static int tap_pad_rt(int nk) { return (nk * nk + 3) & ~3; }

size_t full_weight_floats(int KD, int ND, int nk) {
  return (size_t)round_up(KD, 4) * round_up(ND, kCtOut) * tap_pad_rt(nk);
}

hipError_t launch_full_weights(const float *w, float *wt, bool gx, int S, int C, int nk, hipStream_t s) {
  const int KDp = round_up(gx ? S : C, 4), NDp = round_up(gx ? C : S, kCtOut), TP = tap_pad_rt(nk);
  const long long n = (long long)KDp * NDp * TP;
  long long g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  return timed_launch("full_weights", k_full_weights, dim3((unsigned)g), dim3(256), 0, s, w, wt, S, C, nk * nk, TP,
                      gx ? 1 : 0, KDp, NDp);
}

hipError_t launch_full_contract(bool gx, int nk, SpecLayout in, const float *wt, const float2 *tw, SpecLayout out,
                                int B, int KD, int ND, int P, hipStream_t s) {
  if (P % 8 != 0) return hipErrorInvalidValue;
  const int KDp = round_up(KD, 4), NDp = round_up(ND, kCtOut);
  // output groups of NTL 16-output tiles: as few groups as 64 outputs give, each as narrow
  // as they allow (80 outputs: two groups of 48 instead of two of 64)
  const int tiles = (ND + 15) / 16, nsb = (tiles + 3) / 4;
  const char *nm = gx ? "full_contract_gx" : "full_contract_fwd";
  hipError_t err = hipErrorInvalidValue;
  // 16-image tiles, and 8-image tiles for the last 8 or fewer images
  const int n16 = (B + 7) / 8 / 2, rest = B - 16 * n16;
  dispatch_nk(nk, [&](auto nc) {
    constexpr int NK = decltype(nc)::value;
    auto go = [&](auto btc, auto ntc, int b_first, long long nbt) {
      constexpr int BT = decltype(btc)::value, NTL = decltype(ntc)::value;
      const int ng = ct_groups(P, ct_cols<BT>());
      const long long per = (long long)ng * nsb, most = ((1LL << 31) - 1) / per;  // image tiles a launch can take
      if (most < 1) {
        err = hipErrorInvalidValue;
        return;
      }
      for (long long i = 0; i < nbt; i += most) {
        const long long n = std::min(most, nbt - i);
        err = timed_launch(nm, k_full_contract<NK, BT, NTL>, dim3((unsigned)(per * n)), dim3(256), 0, s, in, wt, tw,
                           out, B, KD, KDp, ND, NDp, P, gx ? 1 : 0, ng, nsb, (int)(b_first + i * 8 * BT));
        if (err != hipSuccess) return;
      }
    };
    auto with_ntl = [&](auto ntc) {
      if (n16 > 0) go(std::integral_constant<int, 2>{}, ntc, 0, n16);
      if (n16 > 0 && err != hipSuccess) return;
      if (rest > 0) go(std::integral_constant<int, 1>{}, ntc, 16 * n16, 1);
    };
    // the last 1 to 4 images: 64 outputs a workgroup without idle rows, about 62 cycles for 64
    // kernel bins (3 x 3) where 8-image tiles take about 98, unless 16-output tiles waste less:
    // up to 32 of 64 outputs at 3 x 3 taps, up to 48 at 5 x 5, where K takes more of both (48
    // outputs of 128^2, 3 images: 68 us here, 65 on 8-image tiles; 128 -> 128 channels of
    // 512^2, 4 images, 3 x 3: 1.12 ms here, 1.68 there)
    if constexpr (NK == 3 || NK == 5) {
      if (rest > 0 && rest <= 4 && (NK == 3 ? 2 * tiles >= 5 * nsb : 5 * tiles >= 16 * nsb)) {
        if (n16 > 0) {
          err = launch_full_contract(gx, nk, in, wt, tw, out, 16 * n16, KD, ND, P, s);
          if (err != hipSuccess) return;
        }
        const long long grid = (long long)ct_groups(P, ct_cols<1>()) * nsb;
        if (grid >= (1LL << 31)) {
          err = hipErrorInvalidValue;
          return;
        }
        err = timed_launch(nm, k_full_contract4<NK>, dim3((unsigned)grid), dim3(256), 0, s, in, wt, tw, out, B, KD,
                           KDp, ND, NDp, P, gx ? 1 : 0, nsb, 16 * n16);
        return;
      }
    }
    if constexpr (NK == 3 || NK == 5) {
      switch ((tiles + nsb - 1) / nsb) {
        case 1: with_ntl(std::integral_constant<int, 1>{}); return;
        case 2: with_ntl(std::integral_constant<int, 2>{}); return;
        case 3: with_ntl(std::integral_constant<int, 3>{}); return;
        default: break;
      }
    }
    with_ntl(std::integral_constant<int, 4>{});
  });
  return err;
}

// Bin chunks of the dL/dw pass: about 8192 workgroups, so that the workgroups running
// at one time on an XCD are the tiles of one or two short chunks and share the spectra
// they read through L2, and at most 97 runs (388 bins) per chunk; at most 512 chunks of
// partial sums.  At 512 pixels and 256 channels (64 tiles) the pass took 13.3-13.8 ms
// with 97 or 129 runs per chunk, 15.1 ms with 65, 17-22 ms with 128 (two whole rows:
// every chunk starts at the same column), 22-24 ms with 161 or 193, and 15-19 ms, uneven
// from run to run and with 2.3 times the HBM reads, with the 257 that 8192 workgroups
// alone give.
constexpr int kGwMaxRunsPerChunk = 97;
int full_gw_chunks(int B, int S, int C, int P, int nk) {
  (void)B, (void)nk;
  const int nrun = P * (P / 2) / 4 + P / 4;
  const int tiles = ((S + 31) / 32) * ((C + 31) / 32);
  int chunks = std::max((8192 + tiles - 1) / tiles, (nrun + kGwMaxRunsPerChunk - 1) / kGwMaxRunsPerChunk);
  if (chunks > 512) chunks = 512;
  if (chunks > nrun) chunks = nrun;
  if (chunks < 1) chunks = 1;
  return chunks;
}

hipError_t launch_full_gw(int nk, SpecLayout G, SpecLayout X, const float2 *tw, float *part, float *gw, int B, int S,
                          int C, int P, hipStream_t s) {
  if (P % 8 != 0) return hipErrorInvalidValue;
  const int nrun = P * (P / 2) / 4 + P / 4;
  const int chunks = full_gw_chunks(B, S, C, P, nk);
  const int runs_per_chunk = (nrun + chunks - 1) / chunks;
  const int tiles = ((S + 31) / 32) * ((C + 31) / 32);
  hipError_t err = hipErrorInvalidValue;
  dispatch_nk(nk, [&](auto nc) {
    constexpr int NK = decltype(nc)::value;
    const size_t lds = ((size_t)gw_tw_elems<NK>(P) + 2 * kGwStageElems) * sizeof(float2);
    if (lds > 65536) return;  // (P <= 1024, n <= 5 stays within 60 KB)
    if (((B + 3) / 4) % 2 == 0)
      err = timed_launch("full_gw", k_full_gw<NK, true>, dim3((unsigned)(tiles * chunks)), dim3(256), lds, s, G, X, tw,
                         part, B, S, C, P, runs_per_chunk);
    else
      err = timed_launch("full_gw", k_full_gw<NK, false>, dim3((unsigned)(tiles * chunks)), dim3(256), lds, s, G, X,
                         tw, part, B, S, C, P, runs_per_chunk);
  });
  if (err != hipSuccess) return err;
  const long long n = (long long)S * C * nk * nk;
  const long long g = (n + 63) / 64;
  if (g >= (1LL << 31)) return hipErrorInvalidValue;
  return timed_launch("full_gw_reduce", k_full_gw_reduce, dim3((unsigned)g), dim3(256), 0, s, part, gw, n, chunks);
}

}  // namespace fdc
