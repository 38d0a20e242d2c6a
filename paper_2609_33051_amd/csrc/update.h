// Flush step of SketchSSM (Algorithm 1, t = W; Sec. 4.1, per-window sketch)
// and the initial sketch: one read and one write of the full state.
//
// With the window's tokens in ring slots 0..n (slot n: the current token),
// cumulative log decays g_s and c_s = exp(g_n - g_s):
//   L[s]   = exp(g_n - g_s) . k_s                  (left factors l_s(W), Appendix C.1)
//   pi_s   = beta_s (e^{g_s} . k_s - sum_{j<s} b_{s,j} pi_j)           (eq. wy)
//          = sum_{j<=s} (T^{-1})_{s,j} beta_j e^{g_j} . k_j,  T = I + Diag(beta) B
//            (rows s < n of T^{-1} come from the ring; row n's couplings
//            b_{n,j} are formed here)
//   w_s    = u_s - X_0 pi_s                         (true write vectors; Mamba-2: beta_s v_s)
//   X_W    = X_0 Diag(e^{g_n}) + sum_s w_s L[s]^T   (eq. update in rank-(n+1) form)
//   o_W    = X_W q_W,   U = X_W Omega
// where X = S^T is the stored [V][K] state.  For a scalar decay c_s is one
// number per slot and moves to the value side (w_s L[s]^T = (c_s w_s) k_s^T),
// so the raw keys are the matrix-core operand.  The two contractions over the
// state (X_0 Pi^T, K-deep; the rank-(n+1) update, slot-deep) and the sketch
// projection X_W Omega run on fp32 matrix cores (v_mfma_f32_16x16x4f32).
//
// Mapping: one workgroup (4 waves) per (request, head) item.  The window's
// slots are staged into LDS with wide loads (row layout: four slots per load
// instruction, wave w taking slot groups w, w + 4, ...), the keys transposed so
// that a matrix-core operand over slots (or, for -Pi and Omega^T, over
// channels) is one 16-byte LDS read.  Each wave owns
// 16-column value tiles of X^T (K rows x 16 values), held in MFMA
// accumulator layout: lane l holds X[v0 + l%16][16 kt + 4 (l/16) + i],
// i = 0..3.  The state is stored in exactly this order (tile-major: tile
// (v0/16, kt) is 1 KB contiguous with lane l's four values at 4 l), so each
// load and store instruction moves 1 KB contiguous; both are non-temporal,
// as the state is touched once per flush.  Because the
// contraction index of the K-deep products may be visited in any order, the
// same registers serve as the B operand of X_0 Pi^T and X_W Omega (step i of
// k-tile kt contracts over k = 16 kt + 4 g + i for lane group g) and as the
// accumulator of the rank update, so the state never leaves registers
// between its load and its store.
#pragma once

#include <float.h>

#include "args.h"
#include "device.h"

namespace skssm {

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ floatx4 lds4(const float* p) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  return floatx4{t.x, t.y, t.z, t.w};
}

// Omega^T in LDS, [sketch column j][K]: the four-channel groups of a row are
// exchanged by its index, so that the same channels of eight columns lie in
// different banks without padding.
template <int K> __device__ __forceinline__ int om_at(int j, int k) { return j * K + (k ^ ((j & 7) << 2)); }

// Element e of a head's Omega in global memory: uniform base and 32-bit byte
// offset.  With 64-bit lane addresses, and the next tile's loads held back by
// the branch of a rank check, the full-rank initial sketch took a third longer
// (GDN K = 128, V = 64, 1 GiB of state, fp32 sketch: 1,143 -> 775 us).
__device__ __forceinline__ float om_ld(const float* om, uint32_t e) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(om) + 4 * e);
}

// Sixteen 4 x 4 x 1 products at once, block b on lanes 4 b .. 4 b + 3:
// c[i] of lane j += (a of lane i) (b of lane j), i and j within the quad.
__device__ __forceinline__ floatx4 mfma4x4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

template <typename IO> __device__ __forceinline__ float load1(const IO* p);
template <> __device__ __forceinline__ float load1<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load1<bf16_t>(const bf16_t* p) { return bf16_lo((uint32_t)*p); }

// The state-dependent coefficient map (Sec. 4.1, eq. m-coeff with the ridge
// term and the low-rank-plus-diagonal metric of the appendix on the P = 4
// pivot approximation), from the partial sums the tiles left behind:
//   mu   = |S|_F^2 / K (1 for a zero state)
//   U_p  = the first P sketch columns,  U_p^T U_p = R^T R (Cholesky; a column
//          dependent on the earlier ones is dropped: its row of R^{-1} is 0)
//   L_G  = U^T U_p R^{-1} / sqrt(mu)             (G x P; Q = U_p R^{-1})
//   M    = R^{-T} U_p^T S^T / sqrt(mu)           (P x K, i.e. Q^T S^T / sqrt(mu))
//   d    = max(diag(U^T U) / mu - |L_G rows|^2, 0),  D = d + lambda
//   T    = I + L_G^T D^{-1} L_G                  (Woodbury: only T is inverted)
//   F1   = D^{-1} L_G T^{-1}  (= A^{-1} L_G),  F2 = A^{-1} Diag(d),
//   A^{-1} = D^{-1} - D^{-1} L_G T^{-1} L_G^T D^{-1}
// so the map is C = F1 M + F2 Omega^T (G x K).  With w = d / (d + lambda),
// F2 = Diag(w) - F1 L_G^T Diag(w), hence
//   C = F1 M' + Diag(w) Omega^T,   M' = M - L_G^T Diag(w) Omega^T   (P x K):
// thread k forms column k of M' beside that of M, and the flush forms
// C^T = M'^T F1^T on the matrix cores (one 16x16x4 step per block) plus
// w_j Omega[k][j] per element, then stores the dense map per item in the
// sketch's dtype (bf16 with the paper's storage, rounded to nearest even) in
// 16-byte channel panels cmap[B][H][K/CPW][G][CPW].  Rows past the head's
// rank are not stored.  Every thread of the workgroup calls this.
template <int K, int R, int P, int MT, int RT, int LSZ, int USZ, typename SK>
__device__ __forceinline__ void coef_map_tail(const UpdateArgs& a, size_t item, int wave, int lane, int tid, int rh,
                                              const floatx4 (&nacc)[MT], const floatx4 (&gram)[RT],
                                              const float (&dsq)[RT], float msq,
                                              float* Ls, float* Us, float* cmS, const float* OmL) {
  static_assert(MT % 4 == 0, "the four waves split the k tiles evenly");
  constexpr int FBP = P + 1;                           // row pitch of F1 (odd: lanes of a read spread over banks)
  // in Ls: the waves' N rows (4 K P words), then in their place M'^T and F1, and
  // past them L_G and w
  static_assert(LSZ >= 4 * K * P + 5 * R && 4 * K * P >= P * K + 16 * RT * FBP && USZ >= 4 * R * 5,
                "staging buffers too small for the map's partial sums");
  const int lr = lane & 15, lg = lane >> 4;
  // the squared sketch columns summed over the four lane rows (the Gram
  // products already summed over this wave's values)
  float dq[RT];
#pragma unroll
  for (int jt = 0; jt < RT; ++jt) dq[jt] = cross_row_sum(dsq[jt]);
  msq = wave_sum(msq);
  lds_barrier();  // every wave is done with the window staging (Ls, Us), reused below
  float* cmN = Ls;  // [wave][K][P]
  float* cmG = Us;  // [wave][R][5]
  float* sL = Ls + 4 * K * P;  // [R][P] -w L_G, then [R] w = D^{-1} d
  if (lg == 0) {
#pragma unroll
    for (int kt = 0; kt < MT; ++kt)
      *reinterpret_cast<float4*>(&cmN[(wave * K + 16 * kt + lr) * P]) = make_float4(nacc[kt][0], nacc[kt][1], nacc[kt][2], nacc[kt][3]);
  }
  // row j of cmG: U_j . U_a for the pivots a < P, then |U_j|^2
#pragma unroll
  for (int jt = 0; jt < RT; ++jt) {
    if (lr < P) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 16 * jt + 4 * lg + i;
        if (j < R) cmG[(wave * R + j) * 5 + lr] = gram[jt][i];
      }
    }
    if (lg == 0 && 16 * jt + lr < R) cmG[(wave * R + 16 * jt + lr) * 5 + 4] = dq[jt];
  }
  if (lane == 0) cmS[wave] = msq;
  lds_barrier();

  float F1[P] = {};  // wave 0, lane g < R: row g of F1
  if (wave == 0) {
    const float fro = cmS[0] + cmS[1] + cmS[2] + cmS[3];
    const float mu = fro > 0.f ? fro / K : 1.f;
    // the algebra is one serial chain on one wave while the other waves wait:
    // hardware reciprocal, square root and reciprocal square root (1 ulp) keep it short
    const float rs = __builtin_amdgcn_rsqf(mu);
    // pivot Gram, Cholesky with dropping, R^{-1} (all lanes, uniform)
    float Gp[P][P], Rm[P][P], Ri[P][P];
#pragma unroll
    for (int x = 0; x < P; ++x)
#pragma unroll
      for (int y = 0; y < P; ++y) {
        Gp[x][y] = cmG[(0 * R + x) * 5 + y] + cmG[(1 * R + x) * 5 + y] + cmG[(2 * R + x) * 5 + y] + cmG[(3 * R + x) * 5 + y];
        Rm[x][y] = 0.f;
        Ri[x][y] = 0.f;
      }
#pragma unroll
    for (int x = 0; x < P; ++x) {
      float sd = Gp[x][x];
#pragma unroll
      for (int b = 0; b < x; ++b) sd -= Rm[b][x] * Rm[b][x];
      if (Gp[x][x] > 0.f && sd > 1e-6f * Gp[x][x]) {
        const float rxx = __builtin_amdgcn_sqrtf(sd), irx = __builtin_amdgcn_rcpf(rxx);
        Rm[x][x] = rxx;
#pragma unroll
        for (int y = x + 1; y < P; ++y) {
          float e = Gp[x][y];
#pragma unroll
          for (int b = 0; b < x; ++b) e -= Rm[b][x] * Rm[b][y];
          Rm[x][y] = e * irx;
        }
      }
    }
#pragma unroll
    for (int x = 0; x < P; ++x)
      if (Rm[x][x] > 0.f) Ri[x][x] = __builtin_amdgcn_rcpf(Rm[x][x]);
#pragma unroll
    for (int x = 0; x < P; ++x) {
#pragma unroll
      for (int y = x + 1; y < P; ++y) {
        if (Rm[y][y] > 0.f) {
          float e = 0.f;
#pragma unroll
          for (int b = x; b < y; ++b) e += Ri[x][b] * Rm[b][y];
          Ri[x][y] = -e * Ri[y][y];
        }
      }
    }
    // lane g < R: row g of L_G, d, D^{-1}
    const int g = lane;
    float LG[P] = {}, dg = 0.f, dinv = 0.f;
    if (g < R) {
      float Bg[P], diag = 0.f;
#pragma unroll
      for (int b = 0; b < P; ++b)
        Bg[b] = cmG[(0 * R + g) * 5 + b] + cmG[(1 * R + g) * 5 + b] + cmG[(2 * R + g) * 5 + b] + cmG[(3 * R + g) * 5 + b];
      diag = cmG[(0 * R + g) * 5 + 4] + cmG[(1 * R + g) * 5 + 4] + cmG[(2 * R + g) * 5 + 4] + cmG[(3 * R + g) * 5 + 4];
      float l2 = 0.f;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        float e = 0.f;
#pragma unroll
        for (int b = 0; b < P; ++b) e += Bg[b] * Ri[b][c];
        LG[c] = e * rs;
        l2 += LG[c] * LG[c];
      }
      dg = fmaxf(diag / mu - l2, 0.f);
      dinv = __builtin_amdgcn_rcpf(dg + a.ridge);  // ridge > 0 (the ABI rejects others)
    }
    // T = I + L_G^T D^{-1} L_G (sum over the lanes g), then its inverse
    float Tm[P][P];
#pragma unroll
    for (int x = 0; x < P; ++x)
#pragma unroll
      for (int y = x; y < P; ++y) {
        const float e = wave_sum(LG[x] * dinv * LG[y]);
        Tm[x][y] = e + (x == y ? 1.f : 0.f);
        Tm[y][x] = Tm[x][y];
      }
    float Ti[P][P];
#pragma unroll
    for (int x = 0; x < P; ++x)
#pragma unroll
      for (int y = 0; y < P; ++y) Ti[x][y] = (x == y) ? 1.f : 0.f;
#pragma unroll
    for (int c = 0; c < P; ++c) {  // Gauss-Jordan on the SPD T (pivots >= 1)
      const float inv = __builtin_amdgcn_rcpf(Tm[c][c]);
#pragma unroll
      for (int y = 0; y < P; ++y) {
        Tm[c][y] *= inv;
        Ti[c][y] *= inv;
      }
#pragma unroll
      for (int x = 0; x < P; ++x) {
        if (x == c) continue;
        const float f = Tm[x][c];
#pragma unroll
        for (int y = 0; y < P; ++y) {
          Tm[x][y] -= f * Tm[c][y];
          Ti[x][y] -= f * Ti[c][y];
        }
      }
    }
    // F1 row g; w = D^{-1} d and -w L_G of every g for the correction M' = M - L_G^T Diag(w) Omega^T
#pragma unroll
    for (int c = 0; c < P; ++c) {
      float e = 0.f;
#pragma unroll
      for (int b = 0; b < P; ++b) e += LG[b] * Ti[b][c];
      F1[c] = dinv * e;
    }
    if (g < R) {
#pragma unroll
      for (int c = 0; c < P; ++c) sL[g * P + c] = -dinv * dg * LG[c];
      sL[R * P + g] = dinv * dg;
    }
    if (lane == 0) {
#pragma unroll
      for (int x = 0; x < P; ++x)
#pragma unroll
        for (int y = 0; y < P; ++y) cmS[8 + x * P + y] = Ri[x][y] * rs;
    }
  }
  lds_barrier();
  // M' = R^{-T} N^T / sqrt(mu) - L_G^T Diag(w) Omega^T: thread k sums the four
  // waves' N rows for column k of M; the correction sum_h (-w_h L_G[h][x])
  // Omega[k][h] is one 4 x 4 x 1 product per h, a wave's 64 channels at a time
  // (on the vector units it took five instructions per h)
  float Mk[P] = {};
  if (wave < K / 64) {
    const int k = tid;
    float Nk[P];
#pragma unroll
    for (int b = 0; b < P; ++b)
      Nk[b] = cmN[(0 * K + k) * P + b] + cmN[(1 * K + k) * P + b] + cmN[(2 * K + k) * P + b] + cmN[(3 * K + k) * P + b];
    floatx4 d[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int h = 0; h < R; ++h) d[h & 1] = mfma4x4(sL[P * h + (lane & 3)], OmL[om_at<K>(h, k)], d[h & 1]);
#pragma unroll
    for (int x = 0; x < P; ++x) {
      Mk[x] = d[0][x] + d[1][x];
#pragma unroll
      for (int b = 0; b < P; ++b) Mk[x] += cmS[8 + b * P + x] * Nk[b];
    }
  }
  lds_barrier();  // the waves' N rows are consumed: M'^T and F1 take their place
  float* Mb = Ls;                              // [K][P]   M'^T
  float* Fb = Ls + P * K;                      // [16 RT][FBP]  row j = F1 row j, zero past R
  if (tid < K) *reinterpret_cast<float4*>(&Mb[tid * P]) = make_float4(Mk[0], Mk[1], Mk[2], Mk[3]);
  if (wave == 0 && lane < 16 * RT) {
    float* fr = Fb + lane * FBP;
#pragma unroll
    for (int c = 0; c < P; ++c) fr[c] = lane < R ? F1[c] : 0.f;
  }
  lds_barrier();
  // C^T = M'^T F1^T + (Diag(w) Omega^T)^T: wave w takes k tiles w, w + 4, ...;
  // lane (lr, lg) ends with C[16 jt + lr][16 kt + 4 lg + i], i = 0..3
  constexpr int CPW = 16 / (int)sizeof(SK);
  SK* cm = static_cast<SK*>(a.cmap) + item * (size_t)(R * K);
#pragma unroll
  for (int kq = 0; kq < MT / 4; ++kq) {
    const int kt = wave + 4 * kq;
#pragma unroll
    for (int jt = 0; jt < RT; ++jt) {
      const int j = 16 * jt + lr, k0 = 16 * kt + 4 * lg;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = mfma4(Mb[(16 * kt + lr) * P + lg], Fb[(16 * jt + lr) * FBP + lg], acc);
      const float wj = j < R ? sL[R * P + j] : 0.f;
      const float4 o4 = *reinterpret_cast<const float4*>(&OmL[om_at<K>(j, k0)]);
      acc[0] += wj * o4.x;
      acc[1] += wj * o4.y;
      acc[2] += wj * o4.z;
      acc[3] += wj * o4.w;
      if (j < rh) st_elem4<SK>(cm + ((size_t)(k0 / CPW) * R + j) * CPW + k0 % CPW, acc[0], acc[1], acc[2], acc[3]);
    }
  }
}

// The state-dependent map with the exact state metric (eq. pivot-ridge with
// the dense H; Table 2's "Exact"): with Omega orthonormal and R^T R = I,
// J^T H J = U^T U / mu and J^T H R = U^T S^T / mu, so
//   C = (U^T U / mu + lambda I)^{-1} N / mu,   N = U^T X = U^T S^T (G x K).
// The sketch pass leaves per-wave partial products of N^T = U^T X and the
// Gram U^T U (matrix cores, contraction over the wave's value tiles) and of
// |S|_F^2.  They are summed over the waves in LDS in a fixed order (wave 0
// stores, waves 1..3 add in turn), the Gram system is factored by Cholesky
// on one wave (lane = row), every channel's column of the map is solved by
// forward and back substitution (thread k), and the dense map is stored like
// the pivot map's (16-byte channel panels).  G <= 16.  Every thread calls this.
template <int K, int R, typename SK>
__device__ __forceinline__ void coef_map_exact_tail(const UpdateArgs& a, size_t item, int wave, int lane, int tid,
                                                    int rh, const floatx4 (&nacc)[K / 16], const floatx4& gacc,
                                                    float msq, float* Ls, float* Us, float* cmS) {
  constexpr int MT = K / 16, NP = K + 4, GP = R + 1;
  static_assert(R <= 16, "the exact map is compiled for ranks up to 16");
  const int lr = lane & 15, lg = lane >> 4;
  float* Ns = Ls;            // [R][NP]   N, then the map
  float* Gs = Us;            // [R][GP]   U^T U
  float* Lm = Us + R * GP;   // [R][GP]   its Cholesky factor; then 1 / diagonal at Lm[j * GP + j]
  msq = wave_sum(msq);
  // rows j = 4 lg + i of N^T and of the Gram live in lane group lg
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    lds_barrier();  // w = 0: every wave is done with the pass's scratch in Ls
    if (wave == w) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 4 * lg + i;
        if (j < R) {
#pragma unroll
          for (int kt = 0; kt < MT; ++kt) {
            float* p = &Ns[j * NP + 16 * kt + lr];
            *p = (w == 0 ? 0.f : *p) + nacc[kt][i];
          }
          if (lr < R) {
            float* p = &Gs[j * GP + lr];
            *p = (w == 0 ? 0.f : *p) + gacc[i];
          }
        }
      }
      if (lane == 0) cmS[w] = msq;
    }
  }
  lds_barrier();
  const float fro = cmS[0] + cmS[1] + cmS[2] + cmS[3];
  const float mu = fro > 0.f ? fro / K : 1.f;
  const float imu = 1.f / mu;
  if (wave == 0) {
    // Cholesky of A = U^T U / mu + lambda I: lane j holds row j
    float ar[R];
#pragma unroll
    for (int g = 0; g < R; ++g) ar[g] = (lane < R ? Gs[lane * GP + g] * imu : 0.f) + (lane == g ? a.ridge : 0.f);
    float lrow[R];
#pragma unroll
    for (int c = 0; c < R; ++c) {
      const float piv = lane_bcast(ar[c], c);          // A_cc after the updates of columns < c (> 0: SPD)
      const float ip = __builtin_amdgcn_rsqf(piv);
      const float l = ar[c] * ip;                      // L_jc for j >= c
      lrow[c] = lane >= c ? l : 0.f;
#pragma unroll
      for (int g = c + 1; g < R; ++g) ar[g] -= l * lane_bcast(l, g);
    }
    if (lane < R) {
#pragma unroll
      for (int c = 0; c < R; ++c) Lm[lane * GP + c] = c == lane ? 1.f / lrow[c] : lrow[c];
    }
  }
  lds_barrier();
  // column k of the map: L y = N_k / mu, L^T c = y.  Each row's reads of L
  // stay within its own step (scheduling barrier): hoisting the whole
  // triangle's reads ahead held 136 values live at rank 16 and took the
  // kernel from 80 to 162 registers.
  if (tid < K) {
    const int k = tid;
    float y[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      float e = Ns[j * NP + k] * imu;
#pragma unroll
      for (int c = 0; c < j; ++c) e -= Lm[j * GP + c] * y[c];
      y[j] = e * Lm[j * GP + j];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = R - 1; j >= 0; --j) {
      float e = y[j];
#pragma unroll
      for (int c = j + 1; c < R; ++c) e -= Lm[c * GP + j] * y[c];
      y[j] = e * Lm[j * GP + j];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) Ns[j * NP + k] = y[j];
  }
  lds_barrier();
  // the dense map in 16-byte channel panels: thread (kp, j), j fastest
  constexpr int CPW = 16 / (int)sizeof(SK);
  SK* cm = static_cast<SK*>(a.cmap) + item * (size_t)(R * K);
#pragma unroll
  for (int t = tid; t < R * K / CPW; t += 256) {
    const int j = t % R, kp = t / R;
    if (j < rh) {
      const float* src = &Ns[j * NP + kp * CPW];
#pragma unroll
      for (int e = 0; e < CPW; e += 4) st_elem4<SK>(cm + (size_t)t * CPW + e, src[e], src[e + 1], src[e + 2], src[e + 3]);
    }
  }
}

// LDS layout of a [K][S] array of per-channel slot vectors (keys or left
// factors, transposed): channel ch starts at slot_row<S>(ch), its S slots
// contiguous, so an operand over slots is one 16-byte read.  Rows are S + 4
// words apart (the operand reads of 16 consecutive channels hit all banks) and
// every eighth row is shifted by 4 more (as do the staging writes, whose lanes
// are 8 channels apart).
template <int S> __device__ __forceinline__ int slot_row(int ch) { return ch * (S + 4) + (ch >> 3) * 4; }

// The rank update of a wave's 16-value tiles of X = S^T from the factors of a
// window (or a chunk of one) in LDS, eq. wy: lane (lr, lg) holds
// X[v][16 kt + 4 lg + i] of tile t in x[t][kt][i], v = 16 (wave + 4 t) + lr, and
//   X^T <- Diag(e^{g_n}) X^T + (keys or L)^T W^T,
// with w_s = c_s (u_s - (Pi X^T)[s]) (GDN), u_s - (Pi X^T)[s] (KDA, whose decays
// are in L and ds) or c_s beta_s v_s (Mamba-2), slot s = 16 st + 4 lg + i.  For
// the erase families u = T^{-1} (beta . v) is formed here too: tu holds this
// lane's entries of T^{-1} Diag(beta) (row lr, columns 4 lg ..), Vs the raw
// values, and nPi is -Pi.  Every operand read serves all of the wave's tiles.
template <int KIND, int MT, int ST, int VTW, int LP, int UP, int NC>
__device__ __forceinline__ void rank_update(floatx4 (&x)[VTW][MT], int wave, int lr, int lg, float egn, const float* LT,
                                            const float* nPi, const float* Vs, const floatx4& tu, const float* bsl,
                                            const float* csc, const float* ds) {
  constexpr bool ERASE = KIND != MAMBA2;
  constexpr bool CHAN = KIND == KDA;
  floatx4 wv[VTW][ST];
  if constexpr (ERASE) {
    static_assert(ST == 1, "an erase family's chunk has 16 slots");
    // -(Pi X^T)[s] in NC accumulation chains per tile, u apart from them: u is
    // the larger term, and sums started from it round to its size (state error
    // against 64 bits 2.2e-7, with this order 1.0e-7)
    floatx4 pc[VTW][NC];
#pragma unroll
    for (int t = 0; t < VTW; ++t)
#pragma unroll
      for (int c = 0; c < NC; ++c) pc[t][c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < MT; ++kt) {
      const floatx4 a = lds4(&nPi[lr * LP + 16 * kt + 4 * lg]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < VTW; ++t) pc[t][i % NC] = mfma4(a[i], x[t][kt][i], pc[t][i % NC]);
    }
#pragma unroll
    for (int t = 0; t < VTW; ++t) {
      wv[t][0] = pc[t][0] + pc[t][1];
      if constexpr (NC == 4) wv[t][0] += pc[t][2] + pc[t][3];
    }
#pragma unroll
    for (int t = 0; t < VTW; ++t) {
      // an infinite value enters the product as the largest finite one, whose
      // products with the structural zeros of T^{-1} (earlier slots, slots past
      // n) are zeros and not NaNs, and its own slot's u as it is
      floatx4 u;
      float vf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s = 4 * lg + i;
        const float v = Vs[s * UP + 16 * (wave + 4 * t) + lr];
        vf[i] = __builtin_amdgcn_fmed3f(v, -FLT_MAX, FLT_MAX);
        u[i] = v - vf[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) u = mfma4(tu[i], vf[i], u);
      wv[t][0] += u;
      if constexpr (!CHAN) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wv[t][0][i] *= csc[4 * lg + i];
      }
    }
  } else {
#pragma unroll
    for (int st = 0; st < ST; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s = 16 * st + 4 * lg + i;
        const float f = bsl[s] * csc[s];
#pragma unroll
        for (int t = 0; t < VTW; ++t) wv[t][st][i] = Vs[s * UP + 16 * (wave + 4 * t) + lr] * f;
      }
  }
#pragma unroll
  for (int kt = 0; kt < MT; ++kt) {
    floatx4 d = {egn, egn, egn, egn};
    if constexpr (CHAN) d = lds4(&ds[16 * kt + 4 * lg]);
#pragma unroll
    for (int t = 0; t < VTW; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[t][kt][i] *= d[i];
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      const floatx4 a = lds4(&LT[slot_row<16 * ST>(16 * kt + lr) + 16 * st + 4 * lg]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int t = 0; t < VTW; ++t) x[t][kt] = mfma4(a[i], wv[t][st][i], x[t][kt]);
    }
  }
}

// What bounds it: the in-place stream of the state (8 K V bytes an item).  A GDN
// item (K = V = 128, W = 16) alone on a CU takes 8.7 us from launch to end, 2.6
// of them fp32 matrix-core time; with the channel work on the vector units it
// took 12.9.  That move and the later state read (STATE_LATE, below) together
// took B = 512 flushes (2.5 GB) from 452 to 427 us (GDN) and from 476 to 445
// (KDA); the move alone the two-chunk W = 32 flush at B = 256 from 335 to 266 and
// those with a P = 4 map from 517 to 472 (GDN) and 591 to 509 (KDA).
//
// Three workgroups per CU, or four for the state-dependent maps (P = 4 and
// exact) at window 16 and rank <= 16: their flush spends part of each
// workgroup's life off the memory bus (the map's products and algebra), so
// occupancy pays there (within the bound's 128 registers only KDA's exact map at
// rank 8 with a bf16 sketch spills, 8 bytes).  Mamba-2's at V = 64 need no bound:
// 70 to 80 registers, six workgroups.
template <int KIND, int K, int V, int R, int WMAX, typename IO, typename SK, int P>
__global__ __launch_bounds__(256, (P != 0 && WMAX == 16 && R <= 16) ? 4 : 3) void update_kernel(const UpdateArgs a) {
  constexpr bool ERASE = KIND != MAMBA2;
  constexpr bool CHAN = KIND == KDA;
  constexpr int MT = K / 16;          // k tiles
  constexpr int VT = V / 16;          // value tiles
  constexpr int VTW = (VT + 3) / 4;   // value tiles per wave
  // The erase families flush a window of up to 32 slots as chunks of 16 on
  // the register-resident state: T is unit lower triangular, so the rows of
  // T^{-1} that couple a chunk's slots among themselves are the inverse of
  // that chunk's own T, and a chunk started from the state the previous one
  // left is a window of its own (decays taken from the chunk's first slot).
  // The staging and registers are then those of a 16-slot window.
  constexpr int SP = ERASE ? 16 : WMAX;  // staged slot rows (16 or 32)
  constexpr int CH = WMAX / SP;          // chunks per flush
  constexpr int ST = SP / 16;         // slot tiles
  constexpr int NG = SP / 4;          // slot groups of four
  constexpr int RT = (R + 15) / 16;   // sketch tiles
  // accumulation chains per tile of X_0 Pi^T and of the sketch: more chains
  // shorten the dependent sums (and round less), two tiles' worth of four spill
  // where the map's bound leaves 128 registers (KDA, P = 4: 132 bytes per lane)
  // and where a window of two chunks holds the state through the second's
  // staging (KDA, W = 32, rank 32, bf16 sketch, B = 256: 422 us, with two chains
  // 397 and no spill)
  constexpr bool DEEP = (P == 0 && CH == 1) || VTW == 1;
  constexpr int NCW = DEEP ? 4 : 2;
  constexpr int NCU = DEEP ? 2 : 1;
  constexpr int KPL = K / 16;         // key channels per lane (row layout)
  constexpr int VR = V / 16;          // value channels per lane (row layout)
  constexpr int LP = K + 4;           // LDS pitches chosen so that the 4 lane
  constexpr int UP = V + 4;           // groups of an operand read land in different banks
  constexpr int LSZ = K * (SP + 4) + K / 2;  // words of a slot_row array

  __shared__ __align__(16) float Ls[LSZ];                     // keys k_s (KDA: then L[s]), transposed (slot_row)
  // -Pi, [s][k]; for KDA first e^{g_s} . k_s, transposed (slot_row)
  __shared__ __align__(16) float Pi[!ERASE ? 4 : CHAN && LSZ > SP * LP ? LSZ : SP * LP];
  __shared__ __align__(16) float Us[SP * UP];                 // raw v_s, [s][v]
  __shared__ __align__(16) float Bs[ERASE ? SP * SP : 4];     // (T^{-1})_{s,j}, j < s < n
  __shared__ float dl[ERASE ? SP : 4];                        // <k_s, k_n> (KDA: <L[s], k_n> = b_{n,s})
  __shared__ __align__(16) float qs[K];
  __shared__ __align__(16) float ds[CHAN ? K : 4];            // e^{g_n} per channel (KDA)
  __shared__ __align__(16) float csc[SP];                     // c_s = e^{g_n - g_s} (scalar decay), 0 past slot n
  __shared__ __align__(16) float bsl[SP], bel[SP];            // beta_s, beta_s e^{g_s} (0 past slot n)
  __shared__ float egl[4];                                    // e^{g_n} (scalar decay)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;   // MFMA lane coordinates
  const int row = lg, col = lr;               // row-layout coordinates (same lanes)
  const int H = a.H, W = a.W, nw = a.n;  // nw: the window's current slot
  const size_t item = blockIdx.x;  // b * H + h (B*H < 2^23)
  const int h = (int)(blockIdx.x % (uint32_t)H);
  const bool flush = a.nt > 0;
  // slot s of an item: raw ring fields at (item * W + s) * width, derived
  // fields at (s * B*H + dp) * width, dp = h * B + b
  const size_t NI = (size_t)a.B * H, dp = (size_t)h * a.B + blockIdx.x / (uint32_t)H;

  // Omega^T of this head goes to LDS (om_at; columns padded with zeros to whole
  // 16-column tiles) when it is small; the full-rank case reads it from global
  // memory.
  constexpr bool OM_LDS = R > 0 && R <= 32;
  constexpr int OQ = OM_LDS ? (K * R / 4 + 255) / 256 : 1;  // float4 of Omega per thread
  __shared__ __align__(16) float OmL[OM_LDS ? 16 * RT * K : 4];
  // this head's rank (per-head rank table): the sketch uses Omega's first rh
  // columns (the rest are zeroed in LDS, so U's columns past rh come out 0 and
  // the state-dependent map's rows past rh too); rh = 0: a dense-fallback head
  const int rh = a.ragged ? arg_byte(a.hrank, h) : R;
  const bool want_U = R > 0 && a.U != nullptr && rh > 0;

  // state-dependent coefficient map (P = 4 pivots, or the exact metric, P < 0):
  // per-wave scratch for the block transposes of X and of the sketch columns,
  // and the small factors shared by the workgroup
  constexpr bool EXACT = P < 0;
  static_assert(P == 0 || (P == 4 && R >= 8 && R <= 32) || (EXACT && R >= 8 && R <= 16),
                "state-dependent maps: P = 4 with rank 8..32, or the exact metric with rank 8..16");
  constexpr int XP = 20;                                        // row pitch of a transposed 16 x 16 block
  // That scratch lives in the key staging Ls: every tile is updated first and
  // sketched after a barrier, once Ls is dead.  This keeps the kernel's LDS that
  // of the offline-map flush (four workgroups per CU at K = V = 128).  Each tile's
  // sketch columns go through the same per-wave block as X's (one after the
  // other).
  static_assert(P == 0 || LSZ >= 4 * 16 * XP, "the transposed blocks must fit the key staging");
  float* const cmX = Ls;                                   // [wave][16 values][16 keys]
  float* const cmU = cmX;                                  // [wave][16 values][16 sketch columns], before X's blocks
  __shared__ __align__(16) float cmS[P == 0 ? 4 : 24];     // mu parts, R^{-1}/sqrt(mu)
  static_assert(!EXACT || (LSZ >= R * (K + 4) && SP * UP >= 2 * R * (R + 1)),
                "the exact map's sums must fit the window staging");
  floatx4 nacc[P != 0 ? MT : 1];   // N^T (rows 4 lg + i: pivots a < 4, or every sketch column), this wave's values
  floatx4 gram[P > 0 ? RT : 1];    // sketch Gram U^T U_p: lane (lr, lg), i: row 16 jt + 4 lg + i, column lr < P; this wave's values
  float dsq[P > 0 ? RT : 1];       // squared sketch column 16 jt + lr over this lane row's values
  [[maybe_unused]] floatx4 gacc = {0.f, 0.f, 0.f, 0.f};  // exact: U^T U (rows 4 lg + i, column lr), this wave's values
  float msq = 0.f;                 // this lane's share of |S|_F^2
  if constexpr (P != 0) {
#pragma unroll
    for (int kt = 0; kt < MT; ++kt) nacc[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  if constexpr (P > 0) {
#pragma unroll
    for (int jt = 0; jt < RT; ++jt) {
      gram[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
      dsq[jt] = 0.f;
    }
  }

  // ---- every small load first (window, query, rows of T^{-1}, Omega), then the
  // state: the staged values reach LDS while the state read is still in flight
  // (STATE_LATE: before it is issued)
  float egn = 1.f;  // the chunk's e^{g_n} (scalar decay)
  floatx4 tu = {0.f, 0.f, 0.f, 0.f};  // this lane's entries of T^{-1} Diag(beta): row lr, columns 4 lg .. (erase families)
  Raw<IO, 1> qr;  // this thread's query channel, raw (converted at the staging, so no wait here)
  constexpr int BQ = ERASE ? (SP * SP + 255) / 256 : 1;
  Vec<4> omv[OQ];
  floatx4 xs[VTW][MT];
  // ---- the single read of the state.  The offline-map flushes of the erase
  // families issue it once the window is staged (its latency then overlaps the
  // channel work): at B = 512, K = V = 128 the in-place stream runs faster the
  // shorter a workgroup's 64 KB are in flight (three workgroups per CU, issued
  // with the staging's loads: GDN 452 us, KDA 470; after the staging: 427, 443;
  // after the channel work: 436, 462).  The others issue it with the staging's
  // loads, unconditionally, so that waiting for the staged values never waits
  // for it: Mamba-2's 32 KB (397 us either way), windows of two chunks (284
  // against 295), the flushes that build a map, which are not bound by the
  // stream (GDN 492 against 507), and the full rank's, bound by Omega's reads.
  constexpr bool STATE_LATE = ERASE && CH == 1 && P == 0 && R <= 32;
  static_assert(VT % 4 == 0, "every wave owns the same number of value tiles");
  // A token of its own arrays (sketchssm_step): one load from a base chosen per
  // lane needs 64-bit lane addresses, whether or not the call was given a token
  // (64 MiB of state, Mamba-2 K = 128, V = 64, r = 16: 27.4 us against 26.8 with
  // the token loaded apart, r = 8 27.3 against 26.1).  Where the loads take more
  // registers the branch costs more: fp32 inputs (K = V = 128, W = 32, 1 GiB 447
  // against 489), V = 128 (64 MiB, rank 0: 24.0 against 25.5) and the erase
  // families' two chunks (GDN 39.4 against 41.1, KDA 42.9 against 44.3; one chunk
  // the same).
  constexpr bool APART = !ERASE && sizeof(IO) == 2 && V == 64;
  auto load_state = [&]() {
#pragma unroll
    for (int t = 0; t < VTW; ++t) {
      // tile (vt, kt) of the state is 1 KB contiguous, lane l's float4 at 4 l
      const float* src = a.S + item * V * K + (size_t)((wave + 4 * t) * MT) * 256 + 4 * lane;
#pragma unroll
      for (int kt = 0; kt < MT; ++kt) {
        const float4 x = ld_nt(reinterpret_cast<const float4*>(src + 256 * kt));
        xs[t][kt] = floatx4{x.x, x.y, x.z, x.w};
      }
    }
  };
  auto load_omega = [&]() {
#pragma unroll
    for (int c = 0; c < OQ; ++c) {
      const int i = tid + 256 * c;
#pragma unroll
      for (int e = 0; e < 4; ++e) omv[c].e[e] = 0.f;
      if (i < K * R / 4 && 4 * (i % (R / 4)) < rh) omv[c].load(a.omega + (size_t)h * K * R + 4 * i);
    }
  };
  auto stage_omega = [&]() {
#pragma unroll
    for (int c = 0; c < OQ; ++c) {
      const int i = tid + 256 * c;
      if (i < K * R / 4) {
        Vec<4> w = omv[c];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * (i % (R / 4)) + e >= rh) w.e[e] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) OmL[om_at<K>(4 * (i % (R / 4)) + e, i / (R / 4))] = w.e[e];
      }
    }
    if constexpr (R < 16 * RT) {  // zero columns R..16 RT-1
      for (int i = tid; i < (16 * RT - R) * K / 4; i += 256)
        *reinterpret_cast<float4*>(&OmL[R * K + 4 * i]) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  if (STATE_LATE && !flush) {
    // the initial sketch has nothing to hide the state's latency behind but
    // Omega's: its loads on a path of their own, where no wait covers both
    if constexpr (OM_LDS) load_omega();
    load_state();
    compiler_fence();
    if constexpr (OM_LDS) stage_omega();
  }
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    const int sb = 16 * ch;                                 // the chunk's first slot in the ring
    // the chunk's current slot (counted from sb), and whether the chunk holds
    // the window's current slot (then it is the last one)
    const int n = CH == 1 ? nw : !flush ? 0 : (nw - sb < SP ? nw - sb : SP - 1);
    const bool last = CH == 1 || !flush || nw < sb + SP;
    // slot n of this chunk comes from the token's own arrays (and is appended
    // to the ring below) when the call was given them
    const bool own = last && a.tk != nullptr;
    float bl = 0.f, ll = 0.f;             // wave 0, lane s: beta_s and (scalar decay) log alpha_s
    float bt = 0.f, lt = 0.f;             // the token's own (uniform)
    float gk[CHAN ? SP : 1];              // KDA: g_s of channel tid % K
    Raw<IO, KPL> kr[NG / 4];              // ring keys, row layout (slot 4 (wave + 4 gq) + row)
    Raw<IO, VR> vr[NG / 4];               // raw values
    [[maybe_unused]] Raw<IO, KPL> knr;    // GDN: the key of slot n (same in every row)
    float bv[BQ];
    if (flush) {
      // per-slot scalars: lane s of wave 0 loads slot s; every slot load is
      // issued before any is used (slots past n re-read slot n, in bounds, and
      // are masked afterwards), so no load waits on a branch.  APART: ring and
      // token are loaded by loads of their own, each from a uniform base
      if (tid < SP) {
        const bool tok = !APART && own && tid >= n;
        const size_t si = tok ? item : item * W + sb + (tid < n ? tid : n);
        bl = (tok ? a.tbeta : a.rbeta)[si];
        if constexpr (!CHAN) ll = (tok ? a.tla : a.rla)[si];
      }
      if (APART && own) {
        bt = a.tbeta[item];
        if constexpr (!CHAN) lt = a.tla[item];
      }
      if constexpr (CHAN) {
        const float* lcur = own ? a.tla + item * K : a.rla + (item * W + sb + n) * K;
#pragma unroll
        for (int s = 0; s < SP; ++s) gk[s] = (s < n ? a.rla + (item * W + sb + s) * K : lcur)[tid % K];
      }
#pragma unroll
      for (int gq = 0; gq < NG / 4; ++gq) {
        const int s = 4 * (wave + 4 * gq) + row;
        const size_t si = item * W + sb + s;
        if (s <= n) {
          const bool tok = !APART && own && s == n;
          kr[gq].load((tok ? static_cast<const IO*>(a.tk) + item * K : static_cast<const IO*>(a.rk) + si * K) + col * KPL);
          vr[gq].load((tok ? static_cast<const IO*>(a.tv) + item * V : static_cast<const IO*>(a.rv) + si * V) + col * VR);
        }
        if (APART && own && s == n) {
          kr[gq].load(static_cast<const IO*>(a.tk) + item * K + col * KPL);
          vr[gq].load(static_cast<const IO*>(a.tv) + item * V + col * VR);
        }
      }
      if constexpr (ERASE && !CHAN)
        knr.load((own ? static_cast<const IO*>(a.tk) + item * K : static_cast<const IO*>(a.rk) + (item * W + sb + n) * K) +
                 col * KPL);
      if (ch == 0) qr.load(static_cast<const IO*>(a.q) + item * K + (tid < K ? tid : K - 1));
      if constexpr (ERASE) {
#pragma unroll
        for (int c = 0; c < BQ; ++c) {
          const int idx = tid + 256 * c;
          const int s = idx / SP, j = idx % SP;
          bv[c] = (idx < SP * SP && s < n && j < s) ? a.rt[((size_t)(sb + s) * NI + dp) * W + sb + j] : 0.f;
        }
      }
    }
    if constexpr (OM_LDS) {
      if (ch == 0 && want_U && (flush || !STATE_LATE)) load_omega();
    }

    if (!STATE_LATE && ch == 0) load_state();
    compiler_fence();

    // ---- staged values into LDS
    if constexpr (OM_LDS) {
      if (ch == 0 && want_U && (flush || !STATE_LATE)) stage_omega();
    }
    if (flush) {
#pragma unroll
      for (int gq = 0; gq < NG / 4; ++gq) {
        const int s = 4 * (wave + 4 * gq) + row;
        float ksv[KPL], vsv[VR];
#pragma unroll
        for (int m = 0; m < KPL; ++m) ksv[m] = 0.f;
#pragma unroll
        for (int m = 0; m < VR; ++m) vsv[m] = 0.f;
        if (s <= n) {
#pragma unroll
          for (int m = 0; m < KPL; ++m) ksv[m] = kr[gq].get(m);
          // raw values (Mamba-2 scales them by beta_s c_s where they are used)
#pragma unroll
          for (int m = 0; m < VR; ++m) vsv[m] = vr[gq].get(m);
        }
#pragma unroll
        for (int m = 0; m < KPL; ++m) Ls[slot_row<SP>(col * KPL + m) + s] = ksv[m];
        if constexpr (ERASE && !CHAN) {  // <k_s, k_n>, s < n, while the keys are in registers
          float d = 0.f;
#pragma unroll
          for (int m = 0; m < KPL; ++m) d += ksv[m] * knr.get(m);
          d = row_sum16(d);
          if (col == 0) dl[s] = d;
        }
#pragma unroll
        for (int m = 0; m < VR; m += 4)
          *reinterpret_cast<float4*>(&Us[s * UP + col * VR + m]) = make_float4(vsv[m], vsv[m + 1], vsv[m + 2], vsv[m + 3]);
      }
      if (own) {  // append the token to the ring
        const size_t cur = item * W + nw;
#pragma unroll
        for (int gq = 0; gq < NG / 4; ++gq) {
          if (4 * (wave + 4 * gq) + row == n) {
            kr[gq].store(const_cast<IO*>(static_cast<const IO*>(a.rk)) + cur * K + col * KPL);
            vr[gq].store(const_cast<IO*>(static_cast<const IO*>(a.rv)) + cur * V + col * VR);
          }
        }
        if (tid == n) {
          const_cast<float*>(a.rbeta)[cur] = APART ? bt : bl;
          if constexpr (!CHAN) const_cast<float*>(a.rla)[cur] = APART ? lt : ll;
        }
        if constexpr (CHAN) {
          if (tid < K) const_cast<float*>(a.rla)[cur * K + tid] = gk[SP - 1];  // every slot from n on holds log alpha_n
        }
      }
      if (ch == 0 && tid < K) qs[tid] = qr.get(0);
      if (tid < 64) {
        // wave 0: beta_s, g_s = sum_{j<=s} log alpha_j (inclusive scan over the
        // lanes) and c_s = e^{g_n - g_s}, slots past n zero
        const int sl = tid;
        const bool live = sl <= n && sl < SP;
        if (APART && own && sl == n) {
          bl = bt;
          ll = lt;
        }
        float g = (!CHAN && live) ? ll : 0.f;
#pragma unroll
        for (int d = 1; d < SP; d <<= 1) {
          const float u = __shfl_up(g, d);
          if (sl >= d) g += u;
        }
        const float gnn = __shfl(g, n);
        if (sl < SP) {
          bsl[sl] = live ? bl : 0.f;
          if constexpr (!CHAN) {
            // (c_n = 1 also where alpha_n = 0, whose log decay is -inf)
            csc[sl] = sl == n ? 1.f : live ? fast_exp(gnn - g) : 0.f;
            bel[sl] = live ? bl * fast_exp(g) : 0.f;
          }
        }
        if constexpr (!CHAN) {
          if (sl == 0) egl[0] = fast_exp(gnn);
        }
      }
      if constexpr (ERASE) {
#pragma unroll
        for (int c = 0; c < BQ; ++c) {
          const int idx = tid + 256 * c;
          if (idx < SP * SP) Bs[idx] = bv[c];
        }
      }
    }
    lds_barrier();
    if (STATE_LATE && flush) {
      load_state();
      compiler_fence();
    }
    if (flush) {
      if constexpr (!CHAN) egn = egl[0];
      if constexpr (ERASE) {
        // ---- the channel work: Pi = T^{-1} (beta . e^g . k) and the A operand
        // of u = T^{-1} (beta . v), for all slots at once on the matrix cores.
        // Rows of T^{-1} past slot n and keys past it are zero in LDS, so no
        // slot needs a branch (one per slot, as n is a run-time value, had each
        // LDS read wait for the one before: 4.1 of the 12.9 us a GDN item takes
        // alone on a CU, against about 0.5 us now).
        constexpr int KQT = (MT + 3) / 4;  // channel tiles per wave
        [[maybe_unused]] floatx4 xb[KQT];  // KDA: e^{g_j} . k_j, j = 4 lg .., of channel 16 kt + lr
        if constexpr (CHAN) {
          // thread: channel k, the slots of one of 256 / K groups (wave-uniform)
          constexpr int NGRP = 256 / K, SPG = SP / NGRP;
          const int k = tid % K;
          float acc = 0.f;  // g_s: running sum of the chunk's log alphas
#pragma unroll
          for (int s = 0; s < SP; ++s) {
            acc += s <= n ? gk[s] : 0.f;
            gk[s] = acc;
          }
          if (tid < K) ds[k] = fast_exp(acc);
#pragma unroll
          for (int g = 0; g < NGRP; ++g) {
            if (wave / (4 / NGRP) != g) continue;
#pragma unroll
            for (int s = SPG * g; s < SPG * (g + 1); s += 4) {
              float* lp = &Ls[slot_row<SP>(k) + s];
              const floatx4 kk = lds4(lp);
              floatx4 l, x;
#pragma unroll
              for (int i = 0; i < 4; ++i) {  // (keys past slot n are zero)
                l[i] = s + i < n ? kk[i] * fast_exp(acc - gk[s + i]) : kk[i];
                x[i] = kk[i] * fast_exp(gk[s + i]);
              }
              *reinterpret_cast<float4*>(lp) = make_float4(l[0], l[1], l[2], l[3]);
              *reinterpret_cast<float4*>(&Pi[slot_row<SP>(k) + s]) = make_float4(x[0], x[1], x[2], x[3]);
            }
          }
          lds_barrier();
          // b_{n,s} = <L[s], k_n> (L[n] = k_n): one slot per 16 lanes
          float d = 0.f;
#pragma unroll
          for (int m = 0; m < K / 16; ++m) {
            const float* lp = &Ls[slot_row<SP>(col + 16 * m)];
            d += lp[4 * wave + row] * lp[n];
          }
          d = row_sum16(d);
          if (col == 0) dl[4 * wave + row] = d;
#pragma unroll
          for (int q = 0; q < KQT; ++q)
            if (wave + 4 * q < MT) xb[q] = lds4(&Pi[slot_row<SP>(16 * (wave + 4 * q) + lr) + 4 * lg]);
          lds_barrier();  // Pi takes the place of e^g . k
        }
        // row lr of T^{-1}, columns 4 lg ..: the stored rows, and row n =
        // -beta_n b_{n,.} T^{-1} (row n of T T^{-1} = I)
        floatx4 tr = lds4(&Bs[lr * SP + 4 * lg]);
        const float bl_n = lr < n ? dl[lr] * (CHAN ? 1.f : csc[lr]) : 0.f;
        const float bn = bsl[n];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 4 * lg + i;
          if (j == lr && lr <= n) tr[i] = 1.f;
          const float p = row_sum16(bl_n * tr[i]);  // sum_s b_{n,s} (T^{-1})_{s,j}
          if (lr == n && j < n) tr[i] = -bn * p;
        }
        const floatx4 be = lds4(&(CHAN ? bsl : bel)[4 * lg]), bb = lds4(&bsl[4 * lg]);
        floatx4 tp;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          tp[i] = -tr[i] * be[i];
          tu[i] = tr[i] * bb[i];
        }
#pragma unroll
        for (int q = 0; q < KQT; ++q) {
          const int kt = wave + 4 * q;
          if (kt < MT) {
            floatx4 x;
            if constexpr (CHAN) x = xb[q];
            else x = lds4(&Ls[slot_row<SP>(16 * kt + lr) + 4 * lg]);
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = mfma4(tp[i], x[i], acc);
#pragma unroll
            for (int i = 0; i < 4; ++i) Pi[(4 * lg + i) * LP + 16 * kt + lr] = acc[i];
          }
        }
        lds_barrier();
      }
    }
    if (last) break;
    // an earlier chunk: its update, before the next chunk's staging reuses the LDS
    rank_update<KIND, MT, ST, VTW, LP, UP, NCW>(xs, wave, lr, lg, egn, Ls, Pi, Us, tu, bsl, csc, ds);
    lds_barrier();
  }

  // ---- matrix-core phase, one 16-column value tile at a time (with a
  // state-dependent map: pass 0 updates and stores every tile, pass 1
  // sketches them)
  constexpr int PASSES = P != 0 ? 2 : 1;
  float msc = 1.f;  // pass 1: the power of two the map's partial sums scale the state by
  float xmax = 0.f;  // pass 0: this lane's largest state magnitude (state-dependent map)
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
  if constexpr (P != 0) {
  if (ps == 1) {
    // The map is invariant to the state's scale.  Its partial sums (|S|^2,
    // the Gram of the sketch, N) are quadratic in the state, so they are
    // formed from the state scaled by 2^-e, e the exponent of the item's
    // largest magnitude (exact; the scaled largest magnitude is in [0.5, 1)):
    // a state that has decayed far (below ~1e-19) would otherwise square
    // into fp32's denormal range and break the map's algebra.
    const float m0 = wave_max(xmax);
    if (lane == 0) cmS[4 + wave] = m0;
    lds_barrier();  // also: every wave is done with Ls before the map's scratch reuses it
    const float m = fmaxf(fmaxf(cmS[4], cmS[5]), fmaxf(cmS[6], cmS[7]));
    int e = 0;
    (void)frexpf(m, &e);
    msc = m > 0.f ? ldexpf(1.f, -e) : 1.f;
  }
  }
  if (ps == 0) {
    if (flush) {
      rank_update<KIND, MT, ST, VTW, LP, UP, NCW>(xs, wave, lr, lg, egn, Ls, Pi, Us, tu, bsl, csc, ds);
#pragma unroll
      for (int t = 0; t < VTW; ++t) {
        const int vt = wave + 4 * t, v = 16 * vt + lr;
        // exact output o_W[v] = sum_k X_W[v][k] q_W[k]
        if (a.o) {
          float p = 0.f;
#pragma unroll
          for (int kt = 0; kt < MT; ++kt) {
            const floatx4 q4 = lds4(&qs[16 * kt + 4 * lg]);
#pragma unroll
            for (int i = 0; i < 4; ++i) p += xs[t][kt][i] * q4[i];
          }
          p = cross_row_sum(p);
          if (lg == 0) a.o[item * V + v] = p;
        }
        // the state is final: store it before the sketch and map products
        float* dst = a.S + item * V * K + (size_t)(vt * MT) * 256 + 4 * lane;
#pragma unroll
        for (int kt = 0; kt < MT; ++kt)
          st_nt(reinterpret_cast<float4*>(dst + 256 * kt), make_float4(xs[t][kt][0], xs[t][kt][1], xs[t][kt][2], xs[t][kt][3]));
      }
    }
    if constexpr (P != 0) {  // the tiles are final (updated, or as loaded for the initial sketch)
#pragma unroll
      for (int t = 0; t < VTW; ++t)
#pragma unroll
        for (int kt = 0; kt < MT; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) xmax = fmaxf(xmax, fabsf(xs[t][kt][i]));
    }
  }
  // sketch U^T = Omega^T X^T  (rows j = 16 jt + 4 lg + i of the C layout)
  if constexpr (R > 0) {
    if (want_U && ps == PASSES - 1) {
      const float* om = a.omega + (size_t)h * K * R;
      float aop[VTW][4];                              // U_p^T (exact: U^T) as the A operand of N^T = U_p^T X
#pragma unroll
      for (int jt = 0; jt < RT; ++jt) {
        const int jj = 16 * jt + lr;
        floatx4 uc[VTW][NCU];
#pragma unroll
        for (int t = 0; t < VTW; ++t)
#pragma unroll
          for (int e = 0; e < NCU; ++e) uc[t][e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < MT; ++kt) {
          floatx4 w;
          if constexpr (OM_LDS) {
            w = lds4(&OmL[om_at<K>(jj, 16 * kt + 4 * lg)]);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = om_ld(om, (uint32_t)((16 * kt + 4 * lg + i) * R + jj));
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < VTW; ++t) uc[t][i % NCU] = mfma4(w[i], xs[t][kt][i], uc[t][i % NCU]);
        }
#pragma unroll
        for (int t = 0; t < VTW; ++t) {
          const int v = 16 * (wave + 4 * t) + lr;
          floatx4 acc = uc[t][0];
          if constexpr (NCU == 2) acc += uc[t][1];
          if constexpr (P != 0) {
            // every sketch column of the tile's 16 values goes through LDS, so
            // that U^T becomes an operand with the value index as the
            // contraction index: ut[st] = U[v = 4 st + lg][16 jt + lr], scaled
            float* cu = cmU + wave * 16 * XP;
            wave_lds_sync();
            *reinterpret_cast<float4*>(&cu[lr * XP + 4 * lg]) =
                make_float4(acc[0] * msc, acc[1] * msc, acc[2] * msc, acc[3] * msc);
            wave_lds_sync();
            float ut[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) ut[st] = cu[(4 * st + lg) * XP + lr];
            if constexpr (EXACT) {
              // the whole Gram U^T U (R <= 16: one block)
#pragma unroll
              for (int st = 0; st < 4; ++st) {
                aop[t][st] = ut[st];
                gacc = mfma4(ut[st], ut[st], gacc);
              }
            } else {
              // the Gram against the first P columns (tile 0's, kept from
              // jt = 0) on the matrix cores, and the squared columns
              if (jt == 0) {
#pragma unroll
                for (int st = 0; st < 4; ++st) aop[t][st] = lr < P ? ut[st] : 0.f;
              }
#pragma unroll
              for (int st = 0; st < 4; ++st) {
                gram[jt] = mfma4(ut[st], aop[t][st], gram[jt]);
                dsq[jt] += ut[st] * ut[st];
              }
            }
          }
          // columns 16 jt + 4 lg .. +3 of value v; panels of 16 bytes per value:
          // fp32 U[B][H][R/4][V][4], bf16 U[B][H][R/8][V][8]
          constexpr int PWU = 16 / (int)sizeof(SK);
          // panels past this head's rank are not stored; the tail of its last panel
          // holds zeros (the full rank has no table: without the branch the next
          // tile's Omega is read ahead of these stores)
          if (!OM_LDS || (16 * jt + 4 * lg < R && ((16 * jt + 4 * lg) / PWU) * PWU < rh)) {
            SK* Ui = static_cast<SK*>(a.U) + item * (size_t)V * R;
            if constexpr (sizeof(SK) == 4) {
              reinterpret_cast<float4*>(Ui)[(4 * jt + lg) * V + v] = make_float4(acc[0], acc[1], acc[2], acc[3]);
            } else {
              reinterpret_cast<uint2*>(Ui)[((2 * jt + (lg >> 1)) * V + v) * 2 + (lg & 1)] =
                  make_uint2(bf16_pack2(acc[0], acc[1]), bf16_pack2(acc[2], acc[3]));
            }
          }
        }
      }
      if constexpr (P != 0) {
#pragma unroll
        for (int t = 0; t < VTW; ++t) {
          // N^T = U_p^T X (exact map: U^T X) over this tile's 16 values on the matrix cores: each 16 x 16
          // block of X goes through LDS so that the value index becomes the
          // contraction index (lane group), then four 16x16x4 steps
          float* cx = cmX + wave * 16 * XP;
#pragma unroll
          for (int kt = 0; kt < MT; ++kt) {
            wave_lds_sync();
            const float4 xsc = make_float4(xs[t][kt][0] * msc, xs[t][kt][1] * msc, xs[t][kt][2] * msc,
                                           xs[t][kt][3] * msc);
            *reinterpret_cast<float4*>(&cx[lr * XP + 4 * lg]) = xsc;
            wave_lds_sync();
#pragma unroll
            for (int st = 0; st < 4; ++st) nacc[kt] = mfma4(aop[t][st], cx[(4 * st + lg) * XP + lr], nacc[kt]);
            // summed here and now: left to the compiler, the whole chain sinks below
            // the last block and holds every scaled value till then (81 to 83
            // registers for Mamba-2's exact map at V = 64, 168 for its P = 4 map at
            // K = V = 128, r = 32)
            msq += xsc.x * xsc.x;
            msq += xsc.y * xsc.y;
            msq += xsc.z * xsc.z;
            msq += xsc.w * xsc.w;
            asm volatile("" : "+v"(msq));
          }
        }
      }
    }
  }
  }

  if constexpr (P > 0) {
    if (want_U)
      coef_map_tail<K, R, P, MT, RT, LSZ, SP * UP, SK>(a, item, wave, lane, tid, rh, nacc, gram, dsq, msq, Ls, Us, cmS, OmL);
  }
  if constexpr (EXACT) {
    if (want_U) coef_map_exact_tail<K, R, SK>(a, item, wave, lane, tid, rh, nacc, gacc, msq, Ls, Us, cmS);
  }
}


// One token and no sketch: the whole-state recurrence (Sec. 3.2, eq.
// transition-update: decay, then erase, then write) applied to S read once
// and written once, and o = S^T q from the updated state (eq. read).  This is
// the update with a single buffered token at rank 0, i.e. the window-1
// decoding a conventional recurrent layer does.  The window's machinery
// (staged slots, rows of T^{-1}, rank-W products on the matrix cores) reduces
// to one rank-1 update per state element, so the state streams through
// registers: in the tile-major layout lane (lr, lg) of a wave holds
// X[16 vt + lr][16 kt + 4 lg + i] (X = S^T), and the two contractions over
// keys (X k for the erase, X q for the output) are per-lane partial sums and
// one cross-row sum.  In X's terms the update is
//   X <- X Diag(alpha) + beta (v - X Diag(alpha) k) k^T     (GDN, KDA)
//   X <- alpha X + beta v k^T                               (Mamba-2).
//
// What bounds it: the in-place stream, whose rate depends on how many bytes a
// CU has in flight between their load and their store.  A probe that rewrites
// 1 GiB in place reached 6.8 TB/s with about 32 KB in flight per CU (8 MB over
// the chip), 5.3 to 5.5 with two or more 64 KB items per CU, and 6.2 with twice
// the bytes in the same 8 KB pieces.  So a workgroup is one wave with one
// 16-value tile (8 KB at K = 128), the launch holds about 40 KB of them per CU
// (token_bytes_per_cu), and no wave waits for another.  At 1 GiB of state, against
// one workgroup of four waves per item (its best cap): GDN K = V = 128 406 ->
// 322 us, KDA 403 -> 322, Mamba-2 K = 128, V = 64 350 -> 332, GDN K = 128, V = 64
// 342 -> 331, K = V = 64 336 -> 329 (GDN).  Two or four tiles a wave: 330, 349.
// The tiles of an item go to workgroups of the same XCD (round robin over
// eight items), so that its k, q and decays are fetched once: 337 -> 322 us.
template <int KIND, int K, int V, typename IO>
__global__ __launch_bounds__(64) void token_kernel(const UpdateArgs a) {
  constexpr bool ERASE = KIND != MAMBA2;
  constexpr bool CHAN = KIND == KDA;
  constexpr int MT = K / 16, VT = V / 16;
  constexpr int C = K / 64;                          // key channels per lane
  __shared__ __align__(16) float ks[K];              // k
  __shared__ __align__(16) float qs[K];              // q
  __shared__ __align__(16) float as[CHAN ? K : 4];   // per-channel decay alpha (KDA)
  const int lane = threadIdx.x, lr = lane & 15, lg = lane >> 4;
  // workgroup -> (item, tile): groups of eight items, one per XCD; the last
  // items, where fewer than eight are left, in plain order
  const uint32_t NI = gridDim.x / VT, wg = blockIdx.x, full = NI / 8 * 8;
  uint32_t it, vt;
  if (wg < full * VT) {
    const uint32_t j = wg >> 3;
    it = j / VT * 8 + (wg & 7);
    vt = j % VT;
  } else {
    it = wg / VT;
    vt = wg % VT;
  }
  const size_t item = it;                            // b * H + h
  // the token's raw inputs: its ring slot, or its own arrays (then appended)
  const bool own = a.tk != nullptr;
  const size_t slot = item * (size_t)a.W + a.n, cur = own ? item : slot;

  // ---- the token's small loads, then the tile's single read
  Raw<IO, C> kr, qr;
  kr.load(static_cast<const IO*>(own ? a.tk : a.rk) + cur * K + lane * C);
  qr.load(static_cast<const IO*>(a.q) + item * K + lane * C);
  const float* la = own ? a.tla : a.rla;
  Raw<float, CHAN ? C : 1> lr_raw;
  lr_raw.load(CHAN ? la + cur * K + lane * C : la + cur);
  const float beta = (own ? a.tbeta : a.rbeta)[cur];
  const float vv = load1<IO>(static_cast<const IO*>(own ? a.tv : a.rv) + cur * V + 16 * vt + lr);
  float* S = a.S + item * V * K + (size_t)(vt * MT) * 256 + 4 * lane;
  floatx4 xs[MT];
#pragma unroll
  for (int kt = 0; kt < MT; ++kt) {
    const float4 x = ld_nt(reinterpret_cast<const float4*>(S + 256 * kt));
    xs[kt] = floatx4{x.x, x.y, x.z, x.w};
  }
  compiler_fence();
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ks[lane * C + c] = kr.get(c);
    qs[lane * C + c] = qr.get(c);
    if constexpr (CHAN) as[lane * C + c] = fast_exp(lr_raw.get(c));
  }
  if (own) {  // append the token to the ring: v by every tile, the rest by the item's first
    if (lg == 0) st_elem<IO>(const_cast<IO*>(static_cast<const IO*>(a.rv)) + slot * V + 16 * vt + lr, vv);
    if (vt == 0) {
      kr.store(const_cast<IO*>(static_cast<const IO*>(a.rk)) + slot * K + lane * C);
      if constexpr (CHAN) lr_raw.store(const_cast<float*>(a.rla) + slot * K + lane * C);
      if (lane == 0) {
        const_cast<float*>(a.rbeta)[slot] = beta;
        if constexpr (!CHAN) const_cast<float*>(a.rla)[slot] = lr_raw.get(0);
      }
    }
  }
  wave_lds_sync();
  const float alpha = CHAN ? 1.f : fast_exp(lr_raw.get(0));

  // w = beta (v - X Diag(alpha) k), or beta v without the erase
  float w = beta * vv;
  if constexpr (ERASE) {
    float y = 0.f;
#pragma unroll
    for (int kt = 0; kt < MT; ++kt) {
      const floatx4 k4 = lds4(&ks[16 * kt + 4 * lg]);
      floatx4 d4 = {alpha, alpha, alpha, alpha};
      if constexpr (CHAN) d4 = lds4(&as[16 * kt + 4 * lg]);
      y += xs[kt][0] * (d4[0] * k4[0]) + xs[kt][1] * (d4[1] * k4[1]) + xs[kt][2] * (d4[2] * k4[2]) +
           xs[kt][3] * (d4[3] * k4[3]);
    }
    w = beta * (vv - cross_row_sum(y));
  }
  // X <- X Diag(alpha) + w k^T, then o = X q
  float p = 0.f;
#pragma unroll
  for (int kt = 0; kt < MT; ++kt) {
    const floatx4 k4 = lds4(&ks[16 * kt + 4 * lg]), q4 = lds4(&qs[16 * kt + 4 * lg]);
    floatx4 d4 = {alpha, alpha, alpha, alpha};
    if constexpr (CHAN) d4 = lds4(&as[16 * kt + 4 * lg]);
    floatx4 x = xs[kt];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = x[i] * d4[i] + w * k4[i];
    p += x[0] * q4[0] + x[1] * q4[1] + x[2] * q4[2] + x[3] * q4[3];
    st_nt(reinterpret_cast<float4*>(S + 256 * kt), make_float4(x[0], x[1], x[2], x[3]));
  }
  p = cross_row_sum(p);
  if (a.o && lg == 0) a.o[item * V + 16 * vt + lr] = p;
}

}  // namespace skssm
