// Elimination of the velocity and bias unknowns ("V": 9 per keyframe, the last
// 9 of its 15) ahead of the reduced pose system, one segment of consecutive
// keyframes per workgroup.  Only the inertial factors touch them, so with the
// poses and the V of the neighbouring separators as columns their rows of the
// normal equations read
//   [ M  C ] [v]   [c]         M: block tridiagonal (9 x 9 blocks),
//   [ C' S ] [x] = [s]         C: at most three keyframes per block row.
// With M = L L^T and Y = L^-1 [C c] the reduced system loses Y^T Y, and the
// back-substitution is L^T v = y_c - Y x.  M is factored from both ends
// towards the keyframe m in the middle (half as many dependent steps):
//   L_i L_i^T = M_ii - B_i B_i^T,  B_i = M_i,i-1 L_i-1^-T   (i < m, mirrored for i > m),
// with both neighbours' terms at m.
//
// Three stages, each inside a launch of the step that takes longer than it:
//   cond_segment  beside the vision assembly, by the workgroup that finishes
//                 the segment's last inertial factor: the two chains on one
//                 wave each (a 9 x 9 factor in registers on every lane), then
//                 Y on FP64 MFMA;
//   cond_gram     beside the per-source blocks: the lower 16 x 16 tiles of
//                 Y^T Y on FP64 MFMA, one wave each;
//   cond_backsub  beside the depth back-substitution.
#pragma once
#include "vi_internal.h"
#include "vi_math.h"

namespace vi {
namespace {

__device__ __forceinline__ bool coord_active(const OptsDev& o, int a, int ra, int N) {
  if (ra < 6) return a >= o.n_fixed;
  if (!o.use_imu) return false;
  if (ra >= 9 && o.bias_fixed) return false;
  if (ra >= 9 && o.bias_global) return a == N - 1;   // the shared bias sits in the last keyframe's slot
  return true;
}

// inertial part of the entry ((a, ra), (b, cb)) of B: the blocks of the
// factors (a - 1, a) and (a, a + 1) of the window (Hw: [F][30][30]).  AG: in
// the launch that forms them.
template <bool AG = false>
__device__ __forceinline__ double imu_hess(const double* Hw, int N, int a, int ra, int b, int cb) {
  double v = 0.0;
  if (a == b) {
    if (a > 0) v += agent_load<AG>(Hw + (size_t)(a - 1) * 900 + (15 + ra) * 30 + 15 + cb);
    if (a < N - 1) v += agent_load<AG>(Hw + (size_t)a * 900 + ra * 30 + cb);
  } else if (b == a + 1) {
    v += agent_load<AG>(Hw + (size_t)a * 900 + ra * 30 + 15 + cb);
  } else if (a == b + 1) {
    v += agent_load<AG>(Hw + (size_t)b * 900 + (15 + ra) * 30 + cb);
  }
  return v;
}

// inertial part of w_xi at (b, cb) (gw: [F][30])
template <bool AG = false>
__device__ __forceinline__ double imu_grad(const double* gw, int N, int b, int cb) {
  double v = 0.0;
  if (b > 0) v += agent_load<AG>(gw + (size_t)(b - 1) * 30 + 15 + cb);
  if (b < N - 1) v += agent_load<AG>(gw + (size_t)b * 30 + cb);
  return v;
}

// The same entries with one bias for the window (Table 6 (f)): the bias
// coordinates of every keyframe are the one unknown in the last keyframe's
// slot, so the folded system G^T B G sums an entry over the keyframes whose
// bias it touches (those of the inertial factors next to the other index)
__device__ __forceinline__ double imu_hess_folded(const double* Hw, int N, int a, int ra, int b, int cb, bool global) {
  const bool ga = global && ra >= 9, gb = global && cb >= 9;
  if (!ga && !gb) return imu_hess(Hw, N, a, ra, b, cb);
  double v = 0.0;
  if (ga && gb) {
    for (int f = 0; f < N - 1; ++f) {
      const double* H = Hw + (size_t)f * 900;
      v += H[ra * 30 + cb] + H[ra * 30 + 15 + cb] + H[(15 + ra) * 30 + cb] + H[(15 + ra) * 30 + 15 + cb];
    }
  } else if (gb) {
    for (int b2 = max(a - 1, 0); b2 <= min(a + 1, N - 1); ++b2) v += imu_hess(Hw, N, a, ra, b2, cb);
  } else {
    for (int a2 = max(b - 1, 0); a2 <= min(b + 1, N - 1); ++a2) v += imu_hess(Hw, N, a2, ra, b, cb);
  }
  return v;
}

__device__ __forceinline__ double imu_grad_folded(const double* gw, int N, int b, int cb, bool global) {
  if (!(global && cb >= 9)) return imu_grad(gw, N, b, cb);
  double v = 0.0;
  for (int b2 = 0; b2 < N; ++b2) v += imu_grad(gw, N, b2, cb);
  return v;
}

// column of unknown (kf, c) in segment S, -1: not one of its columns
__device__ __forceinline__ int seg_col(const SegDev& S, int kf, int c, bool bias_global) {
  if (bias_global && c >= 9) return S.gb < 0 ? -1 : S.gb + c - 9;
  if (c < 6) return (kf >= S.k0 && kf <= S.k1) ? 6 * (kf - S.k0) + c : -1;
  if (S.vl >= 0 && kf == S.a - 1) return S.vl + c - 6;
  if (S.vr >= 0 && kf == S.b + 1) return S.vr + c - 6;
  return -1;
}

// what the segments' elimination takes from the entry ((a, ra), (b, cb)) of
// the window's reduced system: the sum of their Gram entries there
__device__ __forceinline__ double seg_entry(const DevPlan& D, const WinDev& W, const double* cond, int a, int ra, int b,
                                            int cb, bool bias_global) {
  const bool ga = bias_global && ra >= 9, gb = bias_global && cb >= 9;
  const int* ks = D.kf_seg + 2 * (size_t)(W.kf_base + (ga ? b : a));
  const bool all = ga && gb;                 // the shared bias is a column of every segment
  const int cnt = all ? W.nseg : 2;
  double v = 0.0;
  for (int q = 0; q < cnt; ++q) {
    const int id = all ? W.seg_base + q : ks[q];
    if (id < 0) break;
    const SegDev& S = D.segs[id];
    const int ca = seg_col(S, a, ra, bias_global), cc = seg_col(S, b, cb, bias_global);
    if (ca >= 0 && cc >= 0) v += cond[S.g_off + (long long)max(ca, cc) * S.ld + min(ca, cc)];
  }
  return v;
}

// the same for the right-hand side at (b, cb)
__device__ __forceinline__ double seg_rhs(const DevPlan& D, const WinDev& W, const double* cond, int b, int cb,
                                          bool bias_global) {
  const bool all = bias_global && cb >= 9;
  const int* ks = D.kf_seg + 2 * (size_t)(W.kf_base + b);
  const int cnt = all ? W.nseg : 2;
  double v = 0.0;
  for (int q = 0; q < cnt; ++q) {
    const int id = all ? W.seg_base + q : ks[q];
    if (id < 0) break;
    const SegDev& S = D.segs[id];
    const int cc = seg_col(S, b, cb, bias_global);
    if (cc >= 0) v += cond[S.g_off + (long long)S.nc * S.ld + cc];
  }
  return v;
}

constexpr int kCondCols = 256;                         // columns (with the right-hand side) of a segment
constexpr int kCondEv = 7;                             // columns that may touch every keyframe: right-hand side, global bias
constexpr int kCondHx = 18 * 12;                       // per factor: V rows of both keyframes x their poses

// LDS of cond_segment for segments of up to len keyframes, in doubles: inverse
// factors, couplings (one more: the right one of the middle), chain scratch,
// the dense columns, the separators' V columns, the factors' V x pose blocks
// (49 KB for kCondSpan + 1 keyframes, the longest segment)
__host__ __device__ constexpr size_t cond_lds_doubles(int len) {
  return (size_t)96 + 81 * (2 * len + 1) + (size_t)kCondNV * kCondEv * len + 162 + (size_t)kCondHx * (len + 1);
}

// entry e (row-major 9 x 9) of the coupling M_i,j (j = i -+ 1); zero where an
// unknown is not solved
__device__ __forceinline__ double cond_off(const OptsDev& o, const double* Hw, int N, int i, int j, int e) {
  const int r = e / 9, c = e % 9;
  if (!coord_active(o, i, 6 + r, N) || !coord_active(o, j, 6 + c, N)) return 0.0;
  return imu_hess<true>(Hw, N, i, 6 + r, j, 6 + c);
}

// The columns that tile t (16 of them) of a segment reaches: a pose column p is
// zero in the left half before keyframe p - 1 and in the right half after
// p + 1; a tile with any other column counts as reaching all keyframes.
__device__ __forceinline__ int seg_tile_from(const SegDev& S, int t) {
  return 16 * t + 15 >= 6 * (S.k1 - S.k0 + 1) ? S.a : max(S.a, S.k0 + 16 * t / 6 - 1);
}
__device__ __forceinline__ int seg_tile_to(const SegDev& S, int t) {
  return 16 * t + 15 >= 6 * (S.k1 - S.k0 + 1) ? S.b : min(S.b, S.k0 + (16 * t + 15) / 6 + 1);
}

// One segment, one workgroup of 512 threads.  Bound by the dependent steps of
// the two chains, about 1 us each: a 9 x 9 factor is 9 pivots of some 100
// clocks, and each lane carries a row of its own through it, lanes 0-8 the
// next coupling block (their row of B = K L^-T), lanes 16-24 the identity
// (their column of L^-1), so that no solve follows the factor.  Y is formed on
// FP64 MFMA, 16 columns per wave at a time: a product's result has the layout
// of the next one's operand, so a column tile stays in registers through the
// whole chain.  (First version, with the inverse and the couplings formed
// after the factor and Y one thread per column: 100 us for 24 keyframes.)
__device__ __forceinline__ void cond_segment(const OptsDev& o, const SegDev& S, const WinDev& W,
                                             const double* __restrict__ Hf, const double* __restrict__ gf,
                                             double* __restrict__ cond, double* sm, DevStatus* st) {
  typedef double d4 __attribute__((ext_vector_type(4)));
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = W.N, a = S.a, b = S.b, len = b - a + 1, mid = (a + b) / 2, nc = S.nc, ld = S.ld;
  const double* Hw = Hf + (size_t)W.f_base * 900;
  const double* gw = gf + (size_t)W.f_base * 30;
  double* scr = sm;                                    // [2][48]        a packed 9 x 9 block per chain (16-byte aligned)
  double* Lw = scr + 96;                               // [len][81]      L_i^-1
  double* Bw = Lw + 81 * len;                          // [len + 1][81]  B_i; [len]: the right one of the middle
  double* ev = Bw + 81 * (len + 1);                    // [len][9][7]
  double* sv = ev + kCondNV * kCondEv * len;           // [2][9][9]      V of a against a - 1, of b against b + 1
  double* Hx = sv + 162;                               // [k1 - k0][18][12], factor k0 + f: (V_f, V_f+1) x (pose_f, pose_f+1)
  int wrong = 0;                                       // what this thread finds (DevStatus::elim)
  auto check = [&](bool ok, int kind, int kf, int v) {   // unknown v of keyframe kf's V
    if (!ok) wrong = max(wrong, kind + kElimPivot - 1 - (15 * kf + 6 + v));
  };
  // unknowns 0..nv-1 of every keyframe of the segment are solved (the biases
  // may be held, or be the shared one of the last keyframe, never in a segment);
  // the rows and columns of the others are those of the identity
  const int nv = (o.bias_fixed || o.bias_global) ? 3 : kCondNV;
  int er = 0;                                          // entry (er, ec) of a packed 9 x 9 block
  while ((er + 1) * (er + 2) / 2 <= lane) ++er;
  const int ec = lane - er * (er + 1) / 2;
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
    // the two chains (waves 0 and 1), then the middle keyframe (wave 0)
    const int dir = wave == 0 ? 1 : -1, first = part ? mid : (wave == 0 ? a : b), end = part ? mid + 1 : mid;
    double* sc = scr + 48 * (wave & 1);
    if (wave < 2 - part && first != end) {
      // the next keyframe's diagonal block (one entry per lane) and the next
      // coupling's rows are loaded a step ahead, unconditionally (masked when
      // they are used, so that nothing waits for them here)
      double dn[2], kn[9];
      const int dr = min(er, 8), dc = min(ec, 8);
      auto fetch = [&](int i) {
        dn[0] = agent_load<true>(Hw + (size_t)max(i - 1, 0) * 900 + (21 + dr) * 30 + 21 + dc);
        dn[1] = agent_load<true>(Hw + (size_t)min(i, N - 2) * 900 + (6 + dr) * 30 + 6 + dc);
        const double* kp = dir > 0 ? Hw + (size_t)min(i, N - 2) * 900 + (21 + min(lane, 8)) * 30 + 6
                                   : Hw + (size_t)max(i - 1, 0) * 900 + (6 + min(lane, 8)) * 30 + 21;
#pragma unroll
        for (int q = 0; q < 9; ++q) kn[q] = agent_load<true>(kp + q);
      };
      fetch(first);
#pragma unroll 1
      for (int i = first; i != end; i += dir) {
        double m = (i > 0 ? dn[0] : 0.0) + (i < N - 1 ? dn[1] : 0.0), v[9];
        if (er == ec) m += o.lambda * m;
        if (er >= nv) m = er == ec ? 1.0 : 0.0;
        bool finite = lane >= 45 || isfinite(m);
        // lanes 0-8: their row of the next coupling; lanes 16-24: of the identity
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          v[q] = (lane < nv && q < nv && !part) ? kn[q] : (lane == 16 + q ? 1.0 : 0.0);
          finite = finite && isfinite(v[q]);
        }
        check(finite, kElimNonfinite, i, dr);
        if (i + dir != end) fetch(i + dir);
        // minus the neighbours' terms: the one before in the chain, both at the middle
#pragma unroll 1
        for (int nb = 0; nb < 1 + part; ++nb) {
          if (part ? (nb == 0 ? mid == a : mid == b) : i == first) continue;
          const double* B = Bw + 81 * (nb ? len : i - a);
#pragma unroll
          for (int q = 0; q < 9; ++q) m -= B[9 * dr + q] * B[9 * dc + q];
        }
        if (lane < 45) sc[lane] = m;
        wave_lds_sync();
        double L[46];
#pragma unroll
        for (int q = 0; q < 23; ++q) {
          const d2 x = ((const d2*)sc)[q];
          L[2 * q] = x[0];
          L[2 * q + 1] = x[1];
        }
        const int bad = factor9_solve(L, v);
        check(bad < 0, kElimPivot, i, bad);
        // B of the next keyframe (the middle keeps its right one apart)
        if (lane < 9 && !part) {
          double* B = Bw + 81 * (i + dir == mid && dir < 0 ? len : i + dir - a) + 9 * lane;
#pragma unroll
          for (int q = 0; q < 9; ++q) B[q] = v[q];
        }
        if (lane >= 16 && lane < 25) {
#pragma unroll
          for (int q = 0; q < 9; ++q) Lw[81 * (i - a) + 9 * q + lane - 16] = v[q];
        }
        wave_lds_sync();
      }
    }
    // meanwhile the other waves bring in what the columns start from
    if (part == 0 && wave >= 2) {
      const int t = tid - 128;
      if (t < 162) {
        const int e = t % 81, i = t < 81 ? a : b, j = t < 81 ? a - 1 : b + 1;
        const double v = (j >= 0 && j < N) ? cond_off(o, Hw, N, i, j, e) : 0.0;
        check(isfinite(v), kElimNonfinite, i, e / 9);
        sv[t] = v;
      }
#pragma unroll 1
      for (int e = t; e < kCondNV * len; e += 384) {
        const int i = a + e / kCondNV, r = e % kCondNV;
        const double v = r < nv ? imu_grad<true>(gw, N, i, 6 + r) : 0.0;
        check(isfinite(v), kElimNonfinite, i, r);
        ev[kCondEv * e] = v;
        if (S.gb >= 0) {
          // the shared bias: the entries against the biases of i - 1, i, i + 1
#pragma unroll 1
          for (int q = 0; q < 6; ++q) {
            double u = 0.0;
            if (r < nv)
              for (int b2 = max(i - 1, 0); b2 <= min(i + 1, N - 1); ++b2) u += imu_hess<true>(Hw, N, i, 6 + r, b2, 9 + q);
            check(isfinite(u), kElimNonfinite, i, r);
            ev[kCondEv * e + 1 + q] = u;
          }
        }
      }
#pragma unroll 4
      for (int e = t; e < kCondHx * (S.k1 - S.k0); e += 384) {
        const int f = S.k0 + e / kCondHx, r = e % kCondHx / 12, c = e % 12;
        const int i = f + r / 9;
        const double h = agent_load<true>(Hw + (size_t)f * 900 + (15 * (r / 9) + 6 + r % 9) * 30 + 15 * (c / 6) + c % 6);
        const double v = (i >= a && i <= b && r % 9 < nv && f + c / 6 >= o.n_fixed) ? h : 0.0;
        check(isfinite(v), kElimNonfinite, i, r % 9);
        Hx[e] = v;
      }
    }
    __syncthreads();
  }
  if (wrong && st) atomicMax(&st->elim, wrong);
  // Y by tiles of 16 columns: along each side T = C_i - B_i Y_prev,
  // Y_i = L_i^-1 T, then the middle with both sides' terms
  double* Y = cond + S.y_off;
  const int m16 = lane & 15, k4 = lane >> 4;
  const int np = 6 * (S.k1 - S.k0 + 1);
  // operand A[m16][4 s + k4] of a 9 x 9 block
  auto load_a = [&](const double* M, double (&x)[3]) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int k = 4 * s + k4;
      const double v = M[min(9 * m16 + k, 80)];
      x[s] = (m16 < 9 && k < 9) ? v : 0.0;
    }
  };
  // part 0: the sides of every tile, part 1: the middle row of every tile (from
  // the rows beside it, read back from Y)
  const int nt = ld / 16;
  const d4 zero = {0.0, 0.0, 0.0, 0.0};
  auto mul = [&](d4 c, const double (&x)[3], const d4& y, double sign) {
#pragma unroll
    for (int s = 0; s < 3; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(sign * x[s], y[s], c, 0, 0, 0);
    return c;
  };
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
#pragma unroll 1
    for (int u = wave; u < (part ? nt : 2 * nt); u += 8) {
      const int side = part ? 0 : u & 1, J = part ? u : u >> 1, dir = side ? -1 : 1;
      const int col = 16 * J + m16;
      // what this lane's column is: a pose unknown (p, cc), a dense column (evq),
      // a V of a separator (svq: its entries against the end of the segment beside it)
      int p = -100, cc = 0, evq = -1, svq = -1, svi = -1;
      if (col < np) {
        p = S.k0 + col / 6;
        cc = col % 6;
      } else if (col == nc) {
        evq = 0;
      } else if (S.gb >= 0 && col >= S.gb && col < S.gb + 6) {
        evq = 1 + col - S.gb;
      } else if (S.vr >= 0 && col >= S.vr && col < S.vr + 9) {
        svq = 81 + col - S.vr;
        svi = b;
      } else if (S.vl >= 0 && col >= S.vl && col < S.vl + 9) {
        svq = col - S.vl;
        svi = a;
      }
      auto load_c = [&](int i) {
        d4 c = zero;
        const bool touch = evq >= 0 || svi == i || (i >= p - 1 && i <= p + 1);
        if (__ballot(touch) == 0) return c;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          const int q = min(k4 + 4 * r, 8);
          double v = 0.0;
          if (touch && k4 + 4 * r < 9) {
            if (evq >= 0) {
              v = ev[((i - a) * kCondNV + q) * kCondEv + evq];
            } else if (svq >= 0) {
              v = sv[9 * q + svq];
            } else {
              // factors i - 1 (as its later keyframe) and i (as its earlier one)
              const double* h1 = Hx + kCondHx * (i - 1 - S.k0) + (9 + q) * 12 + cc;
              const double* h0 = Hx + kCondHx * (i - S.k0) + q * 12 + cc;
              if (p < i) v = h1[0];
              else if (p > i) v = h0[6];
              else v = (i > S.k0 ? h1[6] : 0.0) + (i < S.k1 ? h0[0] : 0.0);
            }
          }
          c[r] = v;
        }
        return c;
      };
      auto store = [&](int i, const d4& y) {
#pragma unroll
        for (int r = 0; r < 3; ++r)
          if (k4 + 4 * r < 9) Y[(size_t)(kCondNV * (i - a) + k4 + 4 * r) * ld + col] = y[r];
      };
      double xb[3], xl[3];
      if (part == 0) {
        int i = side ? max(seg_tile_to(S, J), mid) : min(seg_tile_from(S, J), mid);
        d4 y = zero, c = zero;
        if (i != mid) {
          c = load_c(i);
          load_a(Lw + 81 * (i - a), xl);
        }
        bool coupled = false;
#pragma unroll 1
        while (i != mid) {
          d4 t = c;
          if (coupled) t = mul(t, xb, y, -1.0);
          y = mul(zero, xl, t, 1.0);
          const int n = i + dir;
          if (n != mid) {
            // the next row's operands
            c = load_c(n);
            load_a(Bw + 81 * (n - a), xb);
            load_a(Lw + 81 * (n - a), xl);
          }
          store(i, y);
          coupled = true;
          i = n;
        }
      } else {
        d4 t = load_c(mid);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          if (s ? seg_tile_to(S, J) <= mid : seg_tile_from(S, J) >= mid) continue;   // zero there
          d4 y = zero;
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            const double v = Y[(size_t)(kCondNV * ((s ? mid + 1 : mid - 1) - a) + min(k4 + 4 * r, 8)) * ld + col];
            y[r] = k4 + 4 * r < 9 ? v : 0.0;
          }
          load_a(Bw + 81 * (s ? len : mid - a), xb);
          t = mul(t, xb, y, -1.0);
        }
        load_a(Lw + 81 * (mid - a), xl);
        store(mid, mul(zero, xl, t, 1.0));
      }
    }
    __syncthreads();
  }
  // for the back-substitution: L_i^-1, and G_i = B_n L_i^-1 of the neighbour n
  // nearer the middle (v_i = L_i^-T z_i - G_i^T v_n; none for the middle)
  double* F = cond + S.l_off;
#pragma unroll 1
  for (int e = tid; e < 81 * len; e += 512) {
    const int l = e / 81, r = e % 81 / 9, c = e % 9, i = a + l;
    F[e] = Lw[e];
    const double* B = Bw + 81 * (i < mid ? l + 1 : (i - 1 == mid ? len : l - 1));
    double v = 0.0;
    if (i != mid) {
#pragma unroll
      for (int q = 0; q < 9; ++q) v += B[9 * r + q] * Lw[81 * l + 9 * q + c];
    }
    F[81 * len + e] = v;
  }
}

// Tile t of the Gram Y^T Y of a segment, one wave.  (MFMA 16x16x4: lane l
// supplies A[l % 16][l / 16] = Y[l / 16][16 I + l % 16], B alike, and receives
// rows l / 16 + 4 r, column l % 16.)
__device__ __forceinline__ void cond_gram(const SegDev& S, double* __restrict__ cond, int t) {
  typedef double d4 __attribute__((ext_vector_type(4)));
  const int T = S.ld / 16, lane = threadIdx.x & 63, m16 = lane & 15, k4 = lane >> 4;
  if (t >= T * (T + 1) / 2) return;
  int I = 0;
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  const int J = t - I * (I + 1) / 2;
  // only the rows that both column tiles reach are summed
  const int mid = (S.a + S.b) / 2;
  const int beg = kCondNV * (min(max(seg_tile_from(S, I), seg_tile_from(S, J)), mid) - S.a);
  const int rows = kCondNV * (max(min(seg_tile_to(S, I), seg_tile_to(S, J)), mid) + 1 - S.a);
  const double* Y = cond + S.y_off;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int q0 = beg; q0 < rows; q0 += 32) {
    double va[8], vb[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int q = q0 + 4 * s + k4;
      const size_t off = (size_t)min(q, rows - 1) * S.ld + m16;
      va[s] = q < rows ? Y[off + 16 * I] : 0.0;
      vb[s] = Y[off + 16 * J];
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[s], vb[s], acc, 0, 0, 0);
  }
  double* G = cond + S.g_off;
#pragma unroll
  for (int r = 0; r < 4; ++r) G[(size_t)(16 * I + k4 + 4 * r) * S.ld + 16 * J + m16] = acc[r];
}

// V increments of a segment's keyframes from the solution xw of the reduced
// system, and their retraction; one 256-thread workgroup.  sm: 18 len + 256
// doubles of LDS.  z = y_c - Y x and w = L^-T z over all rows at once, then the
// two chains outwards from the middle, v_i = w_i - G_i^T v_n, one 9 x 9 product
// per step.
__device__ __forceinline__ void cond_backsub(const OptsDev& o, const DevPlan& D, const SegDev& S, const WinDev& W,
                                             const double* __restrict__ cond, const double* __restrict__ xw, double* sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int a = S.a, b = S.b, len = b - a + 1, mid = (a + b) / 2, nc = S.nc, ld = S.ld;
  double* z = sm;                           // [9 len]
  double* v = z + kCondNV * len;            // [9 len]  w, then the increments
  double* xs = v + kCondNV * len;           // [256]
  const int* off = D.kf_off + W.kf_base;
  if (tid < nc) {
    int r;
    if (tid < 6 * (S.k1 - S.k0 + 1)) r = off[S.k0 + tid / 6] + tid % 6;
    else if (S.gb >= 0 && tid >= S.gb && tid < S.gb + 6) r = off[W.N - 1] + 9 + tid - S.gb;
    else if (S.vr >= 0 && tid >= S.vr && tid < S.vr + 9) r = off[b + 1] + 6 + tid - S.vr;
    else r = off[a - 1] + 6 + tid - S.vl;
    xs[tid] = xw[r];
  }
  __syncthreads();
  // 16 rows a wave at a time, lanes over the columns of the tiles that reach
  // the row's keyframe
  const double* Y = cond + S.y_off;
  const int rows = kCondNV * len;
  for (int r0 = 16 * wave; r0 < rows; r0 += 64) {
    double s[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.0;
#pragma unroll 1
    for (int q = lane; q < ld; q += 64) {
      const double xv = q < nc ? xs[q] : (q == nc ? -1.0 : 0.0);
      // rows that the column's tile does not reach read the middle's instead
      const int half = kCondNV * (mid - a), rf = min(kCondNV * (seg_tile_from(S, q >> 4) - a), half),
                rt = max(kCondNV * (seg_tile_to(S, q >> 4) + 1 - a), half + kCondNV);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = min(r0 + r, rows - 1);
        const bool in = row >= rf && row < rt;
        const double y = Y[(in ? row : half) * ld + q];
        s[r] += in ? y * xv : 0.0;
      }
    }
    const double sum = reduce16(s, lane);            // row r0 + lane / 4
    if ((lane & 3) == 0 && r0 + (lane >> 2) < rows) z[r0 + (lane >> 2)] = -sum;
  }
  __syncthreads();
  const double* F = cond + S.l_off;
  for (int e = tid; e < rows; e += 256) {
    const double* L = F + 81 * (e / 9) + e % 9;
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 9; ++r) s += L[9 * r] * z[e / 9 * 9 + r];
    v[e] = s;
  }
  __syncthreads();
  if (wave < 2) {
    const int dir = wave == 0 ? -1 : 1, cnt = wave == 0 ? mid - a : b - mid;
    const int c = lane < 9 ? lane : 0;
    const double* G = F + 81 * len + c;
    double g0[9], g1[9];                     // G of this step and of the next, two loads ahead
    auto fetch = [&](double (&g)[9], int s) {
      const double* Gi = G + 81 * (mid - a + dir * min(s, cnt));
#pragma unroll
      for (int r = 0; r < 9; ++r) g[r] = Gi[9 * r];
    };
    auto step = [&](const double (&g)[9], int s) {
      const int i = mid - a + dir * s;
      double w = v[9 * i + c];
#pragma unroll
      for (int r = 0; r < 9; ++r) w -= g[r] * v[9 * (i - dir) + r];
      if (lane < 9) v[9 * i + c] = w;
      wave_lds_sync();
    };
    fetch(g0, 1);
    fetch(g1, 2);
#pragma unroll 1
    for (int s = 1; s <= cnt; s += 2) {
      step(g0, s);
      fetch(g0, s + 2);
      if (s + 1 <= cnt) step(g1, s + 1);
      fetch(g1, s + 3);
    }
  }
  __syncthreads();
  for (int e = tid; e < rows; e += 256) {
    const int t = a + e / 9, r = e % 9;
    if (r < 3)
      W.vel[(size_t)t * 3 + r] += v[e];
    else if (!o.bias_global)
      W.bias[(size_t)t * 6 + r - 3] += v[e];
    if (W.rep_dxi && (r < 3 || !o.bias_global)) W.rep_dxi[(size_t)t * 15 + 6 + r] = v[e];
  }
}

}  // namespace
}  // namespace vi
