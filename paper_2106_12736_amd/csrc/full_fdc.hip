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
#include "launch_limit.h"
#include "lds_limit.h"

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
// instructions of one SIMD overlap by under 10 %, also from different waves (a probe of both:
// 6.3 ms together, 4.6 and 2.3 ms alone), so a step of 64 MFMAs (2048 cycles) and 160 vector
// instructions (640 cycles) takes about their sum.  Matrix plus vector issue is 85 % of the cycles for
// 16 images of 512^2, 256 -> 256 channels, and 57 % for 224^2, 64 -> 64, whose 1597 workgroups are 3.1
// rounds of the resident ones with 16 steps each.
// Before (a row per image, bins singly): 16 images of 224^2, 64 -> 64 channels 223 -> 202 us;
// 4 images of 512^2, 128 -> 128 channels 2.94 -> 1.13 ms; 3 images of 128^2, 48 -> 80 channels,
// 5 x 5 taps 159 -> 58 us.  BT 8-image tiles share each K: BT = 1 with LB = 4 columns up to 8 images,
// BT = 2 with LB = 2 beyond (the same 32 NTL accumulator registers: two waves a SIMD); BT = 1 with LB = 2
// where the launch has too few workgroups for that to matter.
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
template <int NK, int BT, int LB, int NTL, bool SIDE>
__device__ __forceinline__ void contract_bins(const SpecLayout &in, const float *__restrict__ wt,
                                              const float2 *__restrict__ tw, const SpecLayout &out, float2 *cbuf,
                                              int B, int KD, int KDp, int ND, int NDp, int P, bool gx, int k, int l0,
                                              int b0, int n0) {
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
static inline int ct_groups(int P, int lb) {
  const int H = P / 2, cols = 4 * lb;
  return (H + 1) * ((H + cols - 1) / cols) + (H + cols) / cols;
}

// Group g of them on one image tile and output group.
template <int NK, int BT, int LB, int NTL>
__device__ __forceinline__ void contract_group(const SpecLayout &in, const float *__restrict__ wt,
                                               const float2 *__restrict__ tw, const SpecLayout &out, float2 *cbuf,
                                               int B, int KD, int KDp, int ND, int NDp, int P, bool gx, int g, int b0,
                                               int n0) {
  constexpr int COLS = 4 * LB;
  const int H = P / 2, ncg = (H + COLS - 1) / COLS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g < (H + 1) * ncg) {
    const int k = g / ncg;
    contract_bins<NK, BT, LB, NTL, false>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx, k,
                                          (g - k * ncg) * COLS + wave * LB, b0, n0);
  } else {
    contract_bins<NK, BT, LB, NTL, true>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx, 0,
                                         (g - (H + 1) * ncg) * COLS + wave * LB, b0, n0);
  }
}

// Image tiles of 8 BT images from b_first on; workgroups from `first` on.
template <int NK, int BT, int LB, int NTL>
__global__ __launch_bounds__(256, 2) void k_full_contract(SpecLayout in, const float *__restrict__ wt,
                                                          const float2 *__restrict__ tw, SpecLayout out, int B, int KD,
                                                          int KDp, int ND, int NDp, int P, int gx, int ngroups,
                                                          int nsb, int b_first, unsigned first) {
  __shared__ float2 cbuf[ct_lds_elems<NK>()];
  const unsigned blk = first + xcd_remap(blockIdx.x, gridDim.x), rest = blk / nsb;
  const int sb = blk % nsb;
  contract_group<NK, BT, LB, NTL>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, rest % ngroups,
                                  b_first + (int)(rest / ngroups) * 8 * BT, sb * 16 * NTL);
}

// n16 tiles of 16 images and one of 8 for the rest: in a launch of their own the rest's
// workgroups would wait for a last round of the others.
template <int NK, int NTL>
__global__ __launch_bounds__(256, 2) void k_full_contract_rest(SpecLayout in, const float *__restrict__ wt,
                                                               const float2 *__restrict__ tw, SpecLayout out, int B,
                                                               int KD, int KDp, int ND, int NDp, int P, int gx,
                                                               int ng16, int n16, int nsb, unsigned first) {
  __shared__ float2 cbuf[ct_lds_elems<NK>()];
  const unsigned blk = first + xcd_remap(blockIdx.x, gridDim.x), rest = blk / nsb;
  const int sb = blk % nsb;
  if (rest < (unsigned)(ng16 * n16))
    contract_group<NK, 2, 2, NTL>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, rest % ng16,
                                  (rest / ng16) * 16, sb * 16 * NTL);
  else
    contract_group<NK, 1, 4, NTL>(in, wt, tw, out, cbuf, B, KD, KDp, ND, NDp, P, gx != 0, rest - ng16 * n16, 16 * n16,
                                  sb * 16 * NTL);
}

// 4 images, 64 outputs a workgroup (grid as k_full_contract with BT = 1, one image tile).
template <int NK>
__global__ __launch_bounds__(256, 3) void k_full_contract4(SpecLayout in, const float *__restrict__ wt,
                                                           const float2 *__restrict__ tw, SpecLayout out, int B,
                                                           int KD, int KDp, int ND, int NDp, int P, int gx, int nsb,
                                                           int b0, unsigned first) {
  __shared__ float2 cbuf[ct_lds_elems<NK>()];
  constexpr int COLS = 16;
  const int H = P / 2, ncg = (H + COLS - 1) / COLS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned blk = first + xcd_remap(blockIdx.x, gridDim.x);
  const int g = blk / nsb, n0 = (int)(blk - g * nsb) * kCtOut;
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
// dL/dw partial sums.  G [B][S], X [B][C] split-layout spectra.
// Per bin D[s][c] = sum_b G[b][s] conj(X[b][c]) on the matrix cores (M = s, N = c, depth =
// images, 4 a step), then the adjoint of the kernel spectrum,
//   dL/dw[s][c][a][b] = Re sum_bins D conj(u_a(k) v_b(l)),  u_a = W^(k a), v_b = W^(l b).
// Over a row pair (k, -k), with u_a(-k) = conj u_a(k), P = D(k) + D(-k), Q = D(k) - D(-k):
//   sum = Re u_a EP_b + Im u_a EQ_b,  EP_b = sum_l Re(P conj v_b), EQ_b = sum_l Im(Q conj v_b),
// so that a bin costs 1 + 2 NK vector instructions, 7 at 3 x 3 taps (13 with the n^2 sums), and 3
// more where D comes from Gauss's products.  These, three matrix products for four, take every
// batch of more than 4 images up to 3 x 3 taps, also an odd number of 4-image steps: 8 images a
// stage, absent ones zero.  The a-sum is left to the reduction, once per row pair: a workgroup
// keeps 2 NK sums a (s, c) instead of NK^2.  The Nyquist column l = P/2 runs as one more "row" over k < P/2 with
// rows k and k + P/2 as its pair: u_a(k + P/2) = (-1)^a u_a(k),
//   dL/dw += (-1)^b EP_a,  EP_a = sum_k Re((D(k) + (-1)^a D(k + P/2)) conj u_a).
//
// A workgroup of 16 waves owns a 32 x 32 (s, c) block of one row pair (or part of its
// columns): each wave a 16 x 16 tile and a quarter of the columns in flight.  A stage is LB
// columns of both rows for IMG images: 32 G and 32 X planes, LB * 8 bytes each, loaded by LB/2
// neighbouring lanes and staged in LDS; the loads of stage t + 2 are in flight and stage t + 1
// is written while stage t is multiplied.  IMG = 8, LB = 8 (64-byte pieces); up to 4 images
// IMG = 4, LB = 16 (whole 128-byte lines).  What bounds it: matrix plus vector issue (they hardly
// overlap; 79 % of the cycles for 16 images of 512^2, 256 x 256 channels, 61 % for 224^2, 64 x 64), and
// reading the spectra from L2, S/32 + C/32 times: with 32-byte pieces (one
// run of 4 columns) every piece was a request of its own, 21 TB/s of lines at 256 channels.
// Measured, pass and reduction, before and after, 3 x 3 taps: 16 images (Gauss's products) of
// 224^2, 64 x 64 channels 300 -> 180 us, 256 x 256 2.64 -> 2.35 ms; 4 images (four products) of 512^2,
// 128 x 128 1.53 -> 1.12 ms; 3 images of 128^2, 80 x 48, 5 x 5 taps 219 -> 66 us (the NK^2 sums had
// spilled).
// ---------------------------------------------------------------------------
template <int IMG>
struct GwStage {
  static constexpr int LB = IMG == 8 ? 8 : 16;       // columns a stage
  static constexpr int RS = 2 * LB + 2;              // complex values a plane: both rows, and 2 that spread the banks
  static constexpr int IMAGE = 64 * RS, BUF = IMG * IMAGE;
};
constexpr int kGwThreads = 1024;
// floats of a partial sum: EP_b and EQ_b (for 1 x 1 kernels EP_0 alone)
constexpr int gw_record(int nk) { return nk == 1 ? 1 : 2 * nk; }

template <int NK, int IMG, bool GAUSS, bool SIDE>
__device__ __forceinline__ void gw_rows(const SpecLayout &G, const SpecLayout &X, const float2 *__restrict__ tw,
                                        float *__restrict__ part, float2 *stage, int B, int S, int C, int P, int k,
                                        int l_lo, int l_hi, int sbase, int cbase, int chunk) {
  using St = GwStage<IMG>;
  constexpr int LB = St::LB, RS = St::RS, LP = LB / 2, R = gw_record(NK);
  constexpr int SUB = LB / 8;  // 2-column batches a wave takes of a stage
  const int H = P / 2, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mrow = lane & 15, kq = lane >> 4;
  const int sq = (wave >> 1) & 1, cq = wave & 1, bg = wave >> 2;

  // this thread's pieces: plane row r of G and of X, image i of the stage, columns 2 j, 2 j + 1
  // of rows k and -k (SIDE: rows l and l + P/2 of the Nyquist column)
  const int j = tid % LP, r = (tid / LP) & 31, i = tid / (LP * 32);
  const bool paired = SIDE || (k != 0 && k != H);
  const long long gp = min(sbase + r, S - 1), xp = min(cbase + r, C - 1);
  const float2 *gb, *xb;
  long long gimg, ximg, row1;  // plane strides of an image; second row relative to the first
  if constexpr (SIDE) {
    gb = G.side + gp * G.sps, xb = X.side + xp * X.sps;
    gimg = (long long)S * G.sps, ximg = (long long)C * X.sps, row1 = H;
  } else {
    gb = G.main + gp * G.ps + k * G.rs, xb = X.main + xp * X.ps + k * X.rs;
    gimg = (long long)S * G.ps, ximg = (long long)C * X.ps, row1 = 0;
  }
  const long long grow = SIDE ? row1 : (paired ? (long long)(P - 2 * k) * G.rs : 0);
  const long long xrow = SIDE ? row1 : (paired ? (long long)(P - 2 * k) * X.rs : 0);
  const int halves = (B + IMG - 1) / IMG;
  float4 pre[4];
  int ll = l_lo, lh = 0;          // load cursor: column, image group
  int held_l = l_lo, held_h = 0;  // the stage that pre holds
  auto load = [&]() {
    held_l = ll, held_h = lh;
    const int l = ll + 2 * j, b = lh * IMG + i;
    const long long lo = min(l, H - 2), bo = min(b, B - 1);
    const float2 *g = gb + bo * gimg + lo, *x = xb + bo * ximg + lo;
    pre[0] = *reinterpret_cast<const float4 *>(g);
    pre[1] = *reinterpret_cast<const float4 *>(g + grow);
    pre[2] = *reinterpret_cast<const float4 *>(x);
    pre[3] = *reinterpret_cast<const float4 *>(x + xrow);
  };
  auto put = [&](int buf) {
    float2 *d = stage + buf * St::BUF + (i * 64 + r) * RS + 2 * j;
    float4 v[4] = {pre[0], pre[1], pre[2], pre[3]};
    if (held_l + LB > l_hi || (held_h + 1) * IMG > B || !paired) {  // a stage with absent columns, images or row -k
      const bool on = held_l + 2 * j < l_hi && held_h * IMG + i < B;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool c = (e & 1) ? on && paired : on;
        v[e] = make_float4(c ? v[e].x : 0.f, c ? v[e].y : 0.f, c ? v[e].z : 0.f, c ? v[e].w : 0.f);
      }
    }
    *reinterpret_cast<float4 *>(d) = v[0];
    *reinterpret_cast<float4 *>(d + LB) = v[1];
    *reinterpret_cast<float4 *>(d + 32 * RS) = v[2];
    *reinterpret_cast<float4 *>(d + 32 * RS + LB) = v[3];
  };
  auto advance = [&]() {  // past the last stage the cursor stays on valid addresses (load clamps the column)
    if (++lh == halves) lh = 0, ll += LB;
  };

  float ep[NK][4], eq[NK][4];
#pragma unroll
  for (int b = 0; b < NK; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) ep[b][e] = eq[b][e] = 0.f;

  v4f t1[2][2], t2[2][2], t3[2][2];  // [row][column]; D = (t1, t2) without GAUSS
  // products of the stage's images with this wave's columns 2 u, 2 u + 1; FIRST: the sums start here
  auto multiply = [&](auto first, const float2 *st, int images) __attribute__((always_inline)) {
#pragma unroll
    for (int step = 0; step < IMG / 4; ++step) {
      if (step > 0 && 4 * step >= images) break;  // no such images
      const float2 *ga = st + ((4 * step + kq) * 64 + sq * 16 + mrow) * RS;
      const float2 *xa = st + ((4 * step + kq) * 64 + 32 + cq * 16 + mrow) * RS;
      const bool start = decltype(first)::value && step == 0;
      const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float4 g4 = *reinterpret_cast<const float4 *>(ga + e * LB);
        const float4 x4 = *reinterpret_cast<const float4 *>(xa + e * LB);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const float gr = q ? g4.z : g4.x, gi = q ? g4.w : g4.y, xr = q ? x4.z : x4.x, xi = q ? x4.w : x4.y;
          if constexpr (GAUSS) {
            // Gauss's form: t1 = sum Gr Xr, t2 = sum Gi Xi, t3 = sum (Gr + Gi)(Xr - Xi)
            t1[e][q] = mfma4(gr, xr, start ? zero : t1[e][q]);
            t2[e][q] = mfma4(gi, xi, start ? zero : t2[e][q]);
            t3[e][q] = mfma4(gr + gi, xr - xi, start ? zero : t3[e][q]);
          } else {  // re = Gr Xr + Gi Xi, im = Gi Xr - Gr Xi
            t1[e][q] = mfma4(gr, xr, start ? zero : t1[e][q]);
            t2[e][q] = mfma4(gi, xr, start ? zero : t2[e][q]);
            t1[e][q] = mfma4(gi, xi, t1[e][q]);
            t2[e][q] = mfma4(-gr, xi, t2[e][q]);
          }
        }
      }
    }
  };
  // the finished D of columns l, l + 1 (wave-uniform; zeros were staged past l_hi)
  auto project = [&](int l) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float zc[NK], zs[NK];
      const int lq = min(l + q, H - 1);
      int at = 0;  // l b mod P
#pragma unroll
      for (int b = 1; b < NK; ++b) {
        at += lq;
        at -= at >= P ? P : 0;
        const float2 z = tw[at];
        zc[b] = z.x, zs[b] = z.y;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float re[2], im[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float a1 = t1[h][q][e], a2 = t2[h][q][e];
          if constexpr (GAUSS) {
            re[h] = a1 + a2, im[h] = (t3[h][q][e] - a1) + a2;
          } else {
            re[h] = a1, im[h] = a2;
          }
        }
        const float pr = re[0] + re[1], pi = im[0] + im[1], qr = re[0] - re[1], qi = im[0] - im[1];
        if constexpr (SIDE) {  // EP_a alone, the pair's sum or difference by the parity of a
          ep[0][e] += pr;
#pragma unroll
          for (int b = 1; b < NK; ++b) {
            ep[b][e] = fmaf((b & 1) ? qr : pr, zc[b], ep[b][e]);
            ep[b][e] = fmaf((b & 1) ? qi : pi, zs[b], ep[b][e]);
          }
        } else {
          ep[0][e] += pr;
          if (NK > 1) eq[0][e] += qi;
#pragma unroll
          for (int b = 1; b < NK; ++b) {
            ep[b][e] = fmaf(pi, zs[b], fmaf(pr, zc[b], ep[b][e]));
            eq[b][e] = fmaf(-qr, zs[b], fmaf(qi, zc[b], eq[b][e]));
          }
        }
      }
    }
  };

  load();
  put(0);
  advance();
  load();
  __syncthreads();
  int buf = 0;
  for (int cl = l_lo; cl < l_hi; cl += LB)
    for (int ch = 0; ch < halves; ++ch) {
      // the next stage into the other buffer (read last a stage ago), the loads of the one after
      advance();
      put(buf ^ 1);
      load();
      const float2 *st = stage + buf * St::BUF + bg * (LB / 4);
      if constexpr (IMG == 4) {  // all images are in the stage; the wave's columns go two at a time
        for (int u = 0; u < SUB; ++u) {
          multiply(std::true_type{}, st + 2 * u, B);
          project(cl + bg * (LB / 4) + 2 * u);
        }
      } else {
        if (ch == 0)
          multiply(std::true_type{}, st, B);
        else
          multiply(std::false_type{}, st, B - ch * IMG);
        if (ch + 1 == halves) project(cl + bg * (LB / 4));
      }
      buf ^= 1;
      __syncthreads();
    }

  // the four column quarters' sums, added in order by the waves of quarter 0
  float *red = reinterpret_cast<float *>(stage);
  const int slot = (wave & 3) * 64 + lane;
  if (bg > 0) {
    float *d = red + (bg - 1) * 256 * 8 * NK + slot;
#pragma unroll
    for (int b = 0; b < NK; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) d[(b * 8 + e) * 256] = ep[b][e], d[(b * 8 + 4 + e) * 256] = eq[b][e];
  }
  __syncthreads();
  if (bg > 0) return;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    const float *d = red + g * 256 * 8 * NK + slot;
#pragma unroll
    for (int b = 0; b < NK; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) ep[b][e] += d[(b * 8 + e) * 256], eq[b][e] += d[(b * 8 + 4 + e) * 256];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int os = sbase + sq * 16 + 4 * kq + e, oc = cbase + cq * 16 + mrow;
    if (os >= S || oc >= C) continue;
    float *p = part + (((long long)chunk * S + os) * C + oc) * R;
#pragma unroll
    for (int b = 0; b < NK; ++b) {
      p[b] = ep[b][e];
      if (NK > 1) p[NK + b] = eq[b][e];
    }
  }
}

// Chunks: row pairs k = 0..P/2, then the Nyquist column, each in `ls` column ranges; workgroups
// from `first` on.
template <int NK, int IMG, bool GAUSS>
__global__ __launch_bounds__(kGwThreads) void k_full_gw(SpecLayout G, SpecLayout X, const float2 *__restrict__ tw,
                                                        float *__restrict__ part, int B, int S, int C, int P,
                                                        int ls, unsigned first) {
  extern __shared__ float2 gw_lds[];
  const int H = P / 2;
  const int cblocks = (C + 31) / 32, tiles = ((S + 31) / 32) * cblocks;
  const int blk = (int)first + xcd_remap(blockIdx.x, gridDim.x);
  const int chunk = blk / tiles, tile = blk - chunk * tiles;
  const int k = chunk / ls, range = chunk - k * ls;
  // whole stages a range
  const int nl = (H + GwStage<IMG>::LB - 1) / GwStage<IMG>::LB;
  const int l_lo = range * nl / ls * GwStage<IMG>::LB, l_hi = min(H, (range + 1) * nl / ls * GwStage<IMG>::LB);
  const int sbase = (tile / cblocks) * 32, cbase = (tile % cblocks) * 32;
  if (k <= H)
    gw_rows<NK, IMG, GAUSS, false>(G, X, tw, part, gw_lds, B, S, C, P, k, l_lo, l_hi, sbase, cbase, chunk);
  else
    gw_rows<NK, IMG, GAUSS, true>(G, X, tw, part, gw_lds, B, S, C, P, 0, l_lo, l_hi, sbase, cbase, chunk);
}

// dL/dw from the partial sums: a workgroup owns PP (s, c) pairs; its 256 / PP thread groups
// take the chunks in turn, apply the row phases, and their sums are added in order.  PP = 8
// where 32 would leave few workgroups (64 -> 64 channels: 128 workgroups, 40 us).  The sums
// are kept in 64 bits: up to 514 chunks added one after the other in 32 made the error of dL/dw
// 3 to 9 % larger than sums by 16 accumulators had it (128^2, 9 images, 3 x 3 taps: 2.52e-7,
// 2.70e-7, now 2.30e-7 of which 1.95e-7 are the transforms').  It costs 2 to 4 us: 16 images of
// 224^2, 64 x 64 channels 14.3 -> 16.1 us, 4 of 128^2, 128 x 128, 5 x 5 taps 14.0 -> 18.4 us.
template <int NK, int PP>
__global__ __launch_bounds__(256) void k_full_gw_reduce(const float *__restrict__ part, const float2 *__restrict__ tw,
                                                        float *__restrict__ gw, long long pairs, int P, int ls,
                                                        unsigned first) {
  constexpr int T = NK * NK, R = gw_record(NK);
  constexpr int GR = 256 / PP;
  __shared__ double red[GR][PP][T + 1];
  const int H = P / 2, o = threadIdx.x % PP, w = threadIdx.x / PP, chunks = (H + 2) * ls;
  const long long base = ((long long)first + blockIdx.x) * PP, i = base + o, ii = i < pairs ? i : pairs - 1;
  double acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = 0.;
#pragma unroll 4
  for (int c = w; c < chunks; c += GR) {
    const float *p = part + ((long long)c * pairs + ii) * R;
    float v[R];
#pragma unroll
    for (int e = 0; e < R; ++e) v[e] = p[e];
    const int k = c / ls;
    if (k <= H) {
#pragma unroll
      for (int a = 0; a < NK; ++a) {
        const float2 u = a ? tw[(k * a) % P] : make_float2(1.f, 0.f);
#pragma unroll
        for (int b = 0; b < NK; ++b) {
          acc[a * NK + b] = fma((double)u.x, (double)v[b], acc[a * NK + b]);
          if (a) acc[a * NK + b] = fma((double)u.y, (double)v[R > 1 ? NK + b : 0], acc[a * NK + b]);
        }
      }
    } else {
#pragma unroll
      for (int a = 0; a < NK; ++a)
#pragma unroll
        for (int b = 0; b < NK; ++b) acc[a * NK + b] += (b & 1) ? -v[a] : v[a];
    }
  }
#pragma unroll
  for (int t = 0; t < T; ++t) red[w][o][t] = acc[t];
  __syncthreads();
  for (int e = threadIdx.x; e < PP * T; e += 256) {
    const int oo = e / T, t = e - oo * T;
    if (base + oo >= pairs) break;
    double s = red[0][oo][t];
#pragma unroll
    for (int q = 1; q < GR; ++q) s += red[q][oo][t];
    gw[(base + oo) * T + t] = (float)s;
  }
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

// Column ranges each row pair is cut into: one workgroup is resident a compute unit (its LDS), so
// the least of rounds x (stages + what a workgroup takes besides, 3 to 4 stages).  Against cutting
// for 1024 workgroups, pass and reduction: 16 images of 224^2, 64 x 64 channels, 3 x 3 taps 207 -> 178 us;
// 5 images of 128^2, 5 x 64 channels 50 -> 39; 2 images of 224^2, 33 x 16 64 -> 47.
static int gw_ranges(int B, int S, int C, int P) {
  const int lb = B <= 4 ? GwStage<4>::LB : GwStage<8>::LB, H = P / 2, nl = (H + lb - 1) / lb;
  const int halves = B <= 4 ? 1 : (B + 7) / 8;
  const long long wgs = (long long)((S + 31) / 32) * ((C + 31) / 32) * (H + 2);
  int ranges = 1;
  double least = 0.;
  for (int ls = 1; ls <= nl; ++ls) {
    const double rounds = (double)((wgs * ls + 255) / 256);
    const double cost = rounds * ((nl + ls - 1) / ls * (double)halves + 2.5 + 0.5 * halves);
    if (ls == 1 || cost < least) least = cost, ranges = ls;
  }
  return ranges;
}

// Floats of the dL/dw pass's partial sums.
size_t full_gw_part_floats(int B, int S, int C, int P, int nk) {
  return (size_t)(P / 2 + 2) * gw_ranges(B, S, C, P) * S * C * gw_record(nk);
}

// Sizes a plan accepts: below 2^31 contraction tiles (4 runs of 4 bins, 64 outputs, 16 images), dL/dw
// workgroups and workgroups of its reduction.  Launches of any size in these limits run (in_launches).
bool full_launch_fits(int B, int Cin, int Cout, int P, int nk) {
  if (P % 8 != 0 || B < 1 || B > 65535 * 16) return false;
  const long long nrun = (long long)P * (P / 2) / 4 + P / 4;
  const long long nrun4 = (nrun + 3) / 4, nbt = (B + 15) / 16;
  const long long lim = 1LL << 31;
  if (nrun4 * ((Cout + kCtOut - 1) / kCtOut) * nbt >= lim) return false;
  if (nrun4 * ((Cin + kCtOut - 1) / kCtOut) * nbt >= lim) return false;
  // dL/dw: tiles of 32 x 32 (s, c) times bin chunks, and the fixed-order reduction
  const long long tiles = (long long)((Cout + 31) / 32) * ((Cin + 31) / 32);
  if (tiles * (P / 2 + 2) * gw_ranges(B, Cout, Cin, P) >= lim) return false;
  if (((long long)Cout * Cin * nk * nk + 31) / 32 >= lim) return false;
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
  // 16-image tiles, and an 8-image tile for the last 8 or fewer images
  const int n16 = (B + 7) / 8 / 2, rest = B - 16 * n16;
  const int ng16 = ct_groups(P, 2), ng8 = ct_groups(P, 4);
  dispatch_nk(nk, [&](auto nc) {
    constexpr int NK = decltype(nc)::value;
    // ng x sbs workgroups for each of `units` image tiles from b_first on
    auto go = [&](auto kern, int ng, int sbs, int b_first, long long units) {
      err = in_launches((long long)ng * sbs * units, 256, hipSuccess, [&](unsigned n, unsigned first) {
        return timed_launch(nm, kern, dim3(n), dim3(256), 0, s, in, wt, tw, out, B, KD, KDp, ND, NDp, P, gx ? 1 : 0,
                            ng, sbs, b_first, first);
      });
    };
    // A launch of few workgroups, or of one or two steps, takes 8 images, 2 columns a wave and 32 or
    // 16 outputs a workgroup: its time is a chain of steps, and these are the shortest.  3 x 3 taps:
    // 64 -> 64 channels, 8 images of 32^2 16 us, 37 in the forms below, 20 images of 64^2 37 us, 66; 3 -> 64
    // channels, 8 images of 224^2 38 us, 46 (but of 512^2, 5 x 5 taps, 4 images 117, 98).  Up to 512
    // workgroups where half of a pair of tiles is idle (64^2, 9 images, 32 -> 48 channels, 548 workgroups:
    // 19 us here, 17 below).
    const int sbs = (tiles + 1) / 2;
    const long long small = (long long)ng16 * sbs * ((B + 7) / 8);
    const bool even = tiles % 2 == 0;
    if (small <= (even ? 1024 : 512) || (KDp <= 8 && even && P < 512 && small < (1LL << 31))) {
      if (tiles == 1)
        go(k_full_contract<NK, 1, 2, 1>, ng16, 1, 0, (B + 7) / 8);
      else
        go(k_full_contract<NK, 1, 2, 2>, ng16, sbs, 0, (B + 7) / 8);
      return;
    }
    auto with_ntl = [&](auto ntc) {
      constexpr int NTL = decltype(ntc)::value;
      if (n16 > 0 && rest > 0)
        err = in_launches(((long long)ng16 * n16 + ng8) * nsb, 256, hipSuccess, [&](unsigned n, unsigned first) {
          return timed_launch(nm, k_full_contract_rest<NK, NTL>, dim3(n), dim3(256), 0, s, in, wt, tw, out, B, KD, KDp,
                              ND, NDp, P, gx ? 1 : 0, ng16, n16, nsb, first);
        });
      else if (n16 > 0)
        go(k_full_contract<NK, 2, 2, NTL>, ng16, nsb, 0, n16);
      else
        go(k_full_contract<NK, 1, 4, NTL>, ng8, nsb, 0, 1);
    };
    // the last 1 to 4 images: 64 outputs a workgroup without idle rows, about 62 cycles for 64
    // kernel bins (3 x 3) where 8-image tiles take about 98, unless 16-output tiles waste less:
    // up to 32 of 64 outputs up to 3 x 3 taps, up to 48 beyond, where K takes more of both (48
    // outputs of 128^2, 3 images, 5 x 5: 68 us here, 65 on 8-image tiles; 128 -> 128 channels of
    // 512^2, 4 images, 3 x 3: 1.12 ms here, 1.68 there; 256 -> 256 channels of 224^2, 4 images: 1 x 1 500 us
    // here, 890 there, 2 x 2 745, 1110, 4 x 4 1023, 1340)
    if (rest > 0 && rest <= 4 && (NK <= 3 ? 2 * tiles >= 5 * nsb : 5 * tiles >= 16 * nsb)) {
      if (n16 > 0) {
        err = launch_full_contract(gx, nk, in, wt, tw, out, 16 * n16, KD, ND, P, s);
        if (err != hipSuccess) return;
      }
      err = in_launches((long long)ng8 * nsb, 256, hipSuccess, [&](unsigned n, unsigned first) {
        return timed_launch(nm, k_full_contract4<NK>, dim3(n), dim3(256), 0, s, in, wt, tw, out, B, KD, KDp, ND, NDp,
                            P, gx ? 1 : 0, nsb, 16 * n16, first);
      });
      return;
    }
    switch ((tiles + nsb - 1) / nsb) {
      case 1: with_ntl(std::integral_constant<int, 1>{}); return;
      case 2: with_ntl(std::integral_constant<int, 2>{}); return;
      case 3: with_ntl(std::integral_constant<int, 3>{}); return;
      default: with_ntl(std::integral_constant<int, 4>{});
    }
  });
  return err;
}

hipError_t launch_full_gw(int nk, SpecLayout G, SpecLayout X, const float2 *tw, float *part, float *gw, int B, int S,
                          int C, int P, hipStream_t s) {
  if (P % 8 != 0) return hipErrorInvalidValue;
  const int ls = gw_ranges(B, S, C, P);
  const long long tiles = (long long)((S + 31) / 32) * ((C + 31) / 32), grid = tiles * (P / 2 + 2) * ls;
  const long long pairs = (long long)S * C;
  const int pp = pairs < 32 * 1024 ? 8 : 32;
  const long long rgrid = (pairs + pp - 1) / pp;
  if (grid >= (1LL << 31) || rgrid >= (1LL << 31)) return hipErrorInvalidValue;
  hipError_t err = hipErrorInvalidValue;
  dispatch_nk(nk, [&](auto nc) {
    constexpr int NK = decltype(nc)::value;
    auto go = [&](auto ic) {
      constexpr int IMG = decltype(ic)::value;
      // Gauss's three products pay in stages of two 4-image steps; with more taps the third
      // accumulator would spill.  Their error (9, 10, 12 or 18 images, 1 x 1 to 3 x 3 taps) is 0.86 to
      // 0.97 of four products' with the row pairs added in 32 bits
      constexpr bool kGauss = IMG == 8 && NK <= 3;
      constexpr size_t lds = (size_t)2 * GwStage<IMG>::BUF * sizeof(float2);
      static_assert(lds <= 160 * 1024 && lds >= (size_t)3 * 256 * 8 * NK * sizeof(float), "dL/dw: LDS");
      err = allow_lds<k_full_gw<NK, IMG, kGauss>>(lds);
      if (err != hipSuccess) return;
      err = in_launches(grid, kGwThreads, hipSuccess, [&](unsigned n, unsigned first) {
        return timed_launch("full_gw", k_full_gw<NK, IMG, kGauss>, dim3(n), dim3(kGwThreads), lds, s, G, X, tw, part,
                            B, S, C, P, ls, first);
      });
    };
    if (B <= 4)
      go(std::integral_constant<int, 4>{});
    else
      go(std::integral_constant<int, 8>{});
    if (err != hipSuccess) return;
    err = in_launches(rgrid, 256, hipSuccess, [&](unsigned n, unsigned first) {
      return timed_launch("full_gw_reduce", pp == 8 ? k_full_gw_reduce<NK, 8> : k_full_gw_reduce<NK, 32>, dim3(n),
                          dim3(256), 0, s, part, tw, gw, pairs, P, ls, first);
    });
  });
  return err;
}

}  // namespace fdc
