// Line kernels for levels with few columns: a workgroup per CB columns.
// (One translation unit, line_block.hip, includes this file.)
//
// A level of some thousand columns cannot fill the GPU with two lanes per
// column, and what its kernels then cost is the time of one wavefront, the
// issue of every row's loads and arithmetic in turn.  Here eight wavefronts
// share CB columns.  Seven form the right-hand sides of all rows at once, a few
// rows each; meanwhile the eighth eliminates the matrix, whose pivots do not
// depend on the right-hand side, and keeps their reciprocals (in registers, in
// LDS where block_lds says so).  What is left in sequence is one multiply-add
// and one product a row inwards and one multiply-add a row back, on right-hand
// sides that wait in LDS; then the other wavefronts store.
//
// CB is 8, 16 or 32: the fewest columns with which the workgroups still find a
// compute unit each (256 of them).  Fewer columns spread the right-hand sides
// over more units; a second round of workgroups costs more than that gains.
// FP64, 128 layers, us, 8 / 16 / 32 columns: Smooth with the prolongation on
// 32^2 10.1 / 11.1 / 14.5, 64^2 19.2 / 11.8 / 15.1, 128^2 74 / 41 / 30 (the
// 32-column kernels of kernels.hip with the prolongation apart: 16 + 8, 24 + 6
// and 24 + 12).
//
// The elimination runs from both ends of a column (one lane
// upwards, one downwards), on columns padded to 2 * HALF rows with identity
// rows, and every operation and its order are those of the padded 32-column
// kernels of a larger level: the same values bit for bit.  Two differ by
// rounding: the FP64 smoothers at heights other than 32, 64 and 128, which on a
// larger level meet in the middle of the real rows, and the CG step, which
// stores r - alpha q itself, where the larger kernel rebuilds it from the
// elimination.
#pragma once

#include "device_common.h"

namespace gmg {

namespace {

constexpr int kBlockWaves = 8;  // 0: the elimination, the others: the right-hand sides
constexpr int kBlockThreads = 64 * kBlockWaves;

// vertical profiles of a row
template <typename T>
using BlockProf = T __attribute__((ext_vector_type(4)));

// Whether the reciprocal pivots and d' wait in LDS instead of registers, so that
// two workgroups fit a compute unit where there are more than 256 of them: the
// forms whose right-hand sides leave the room (FP64 64 layers 128^2: line solve
// 9.3 -> 7.5 us, Smooth 12.0 -> 10.1; FP32 128 layers 128^2: 13.1 -> 11.0, 14.6
// -> 12.9, with the prolongation 19.2 -> 17.3; the others spill and lose).
template <typename T, int MODE, int HALF, int CB>
constexpr bool block_lds() {
  constexpr bool plain = MODE == (int)BlockOp::SOLVE || MODE == (int)BlockOp::SMOOTH ||
                         MODE == (int)BlockOp::SMOOTH_NORM;
  if (CB != 32) return false;
  if (sizeof(T) == 4) return HALF == 64 && MODE != (int)BlockOp::RESTRICT_SOLVE;
  return (HALF == 32 && plain) || (HALF == 64 && MODE == (int)BlockOp::SOLVE);
}

// CB: columns of the workgroup (8, 16 or 32).
template <typename T, int MODE, int HALF, int CB>
__device__ __forceinline__ void block_body(const Lvl<T>& L, const BlockArgs<T>& a, int ncols,
                                           int b) {
  constexpr bool kNorm = MODE == (int)BlockOp::SMOOTH_NORM;
  constexpr bool kPro = MODE == (int)BlockOp::PROLONG_SMOOTH;
  constexpr bool kSmooth = MODE == (int)BlockOp::SMOOTH || kNorm || kPro;
  constexpr bool kRes = MODE == (int)BlockOp::RESTRICT_SOLVE;
  constexpr bool kCg = MODE == (int)BlockOp::CG;
  constexpr bool kLds = block_lds<T, MODE, HALF, CB>();
  constexpr int NR = 2 * HALF;                            // padded rows of a column
  constexpr int LG = 64 / CB;                             // row groups of a wavefront
  constexpr int NG = LG * (kBlockWaves - 1);              // ... of the workgroup
  constexpr int R = (NR + NG - 1) / NG;                   // rows of a group (one lane each)
  // rows whose loads are issued together (as many as the registers of two
  // wavefronts per SIMD hold)
  constexpr int CHW = (sizeof(T) == 8 ? 4 : 5);
  constexpr int CH = R < CHW ? R : CHW;
  constexpr int U = 4;                                    // rows of a chunk of the elimination
  using V2 = typename Vec2<T>::type;

  // profiles in each half's elimination order: coupling to the previous row,
  // to the next row, diagonal, dz (identity rows beyond nz; one entry of
  // padding, so that the two halves' reads hit different banks)
  __shared__ BlockProf<T> s_t[2][HALF + 1];
  __shared__ BlockProf<T> s_q[kRes ? NR : 1];             // the fine level's sub, sup, dg, dz
  __shared__ T s_r[NR][CB];                       // right-hand sides, d', x
  __shared__ T s_i[kLds ? NR : 1][kLds ? CB : 1];  // reciprocal pivots (kLds)

  const int nz = L.nz, nx = L.nx, ny = L.ny;
  for (int q = threadIdx.x; q < NR; q += kBlockThreads) {
    const int h = q >= HALF ? 1 : 0, k = q;
    const bool real = k < nz;
    const T sub = real ? L.sub[k] : T(0), sup = real ? L.sup[k] : T(0);
    s_t[h][h ? NR - 1 - k : k] = BlockProf<T>{h ? sup : sub, h ? sub : sup,
                                              real ? L.dg[k] : T(1), real ? L.dz[k] : T(0)};
    if constexpr (kRes) {
      const int kc = min(k, nz - 1);
      s_q[k] = BlockProf<T>{a.X.sub[kc], a.X.sup[kc], a.X.dg[kc], a.X.dz[kc]};
    }
  }

  const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
  const int col = lane & (CB - 1), grp = lane / CB;
  const int hs = grp & 1;  // wavefront 0: the lane's half (lanes past 2 CB repeat them)
  const int cid = b * CB + col;
  const bool active = cid < ncols;
  const int cc = min(cid, ncols - 1);
  const int j = cc / nx, i = cc - j * nx;
  const int ie = i + 1 == nx ? 0 : i + 1, iw = i == 0 ? nx - 1 : i - 1;
  const int jn = j + 1 == ny ? 0 : j + 1, js = j == 0 ? ny - 1 : j - 1;
  const T ce = L.cx[j * nx + i], cw = L.cx[j * nx + iw];
  const T cn = L.cy[j * nx + i], cs = L.cy[js * nx + i];
  const T S = ce + cw + cn + cs + L.wall[j * nx + i];
  // fields are addressed by their base and a 32-bit byte offset (a level that
  // these kernels serve, and the next finer one, is far below 4 GB)
  constexpr uint32_t ES = sizeof(T);
  const uint32_t kb = (uint32_t)L.ldx * ES, jst = (uint32_t)nz * kb;
  const uint32_t base = (uint32_t)j * jst + (uint32_t)i * ES;
  const char* const pa = reinterpret_cast<const char*>(a.a);
  const char* const pf = reinterpret_cast<const char*>(a.f);
  char* const po = reinterpret_cast<char*>(a.o);
  char* const po1 = reinterpret_cast<char*>(a.o1);

  double acc[2] = {0.0, 0.0};
  T keep[kCg ? R : 1];  // CG: the right-hand sides, for <r, z>
  const int k0 = (LG * (w - 1) + grp) * R;  // the lane's rows
  T inv[kLds ? 1 : HALF];                 // wavefront 0: reciprocal pivots
  T* const io = &s_i[kLds && hs ? NR - 1 : 0][kLds ? col : 0];
  const int step = hs ? -CB : CB;

  if (w > 0) {
    const T alpha = kCg && !a.init ? (T)a.st->alpha : T(0);
    const T wmu = (T(1) - a.rho) / a.rho;
    auto clamp = [&](int k) { return (uint32_t)min(max(k, 0), nz - 1); };
    if constexpr (kSmooth) {
      const uint32_t be = (uint32_t)j * jst + (uint32_t)ie * ES;
      const uint32_t bw = (uint32_t)j * jst + (uint32_t)iw * ES;
      const uint32_t bn = (uint32_t)jn * jst + (uint32_t)i * ES;
      const uint32_t bs = (uint32_t)js * jst + (uint32_t)i * ES;
      // prolongation: coarse columns of the parent (0), the second one of the
      // own correction (2) and the one on the other side (3), in x and y, with
      // the mirror signs of those behind a wall
      const char* const pc = reinterpret_cast<const char*>(a.uc);
      uint32_t p00 = 0, p20 = 0, p30 = 0, p02 = 0, p22 = 0, p32 = 0, p03 = 0, p23 = 0, ckb = 0;
      T sx2 = T(1), sx3 = T(1), sy2 = T(1), sy3 = T(1);
      const bool oi = i & 1, oj = j & 1;
      if constexpr (kPro) {
        const Lvl<T>& C = a.X;
        auto fold = [&](int v, int m, int self, T& sg) {
          if (v >= 0 && v < m) return v;
          if (!C.bch) return v < 0 ? m - 1 : 0;
          sg = T(-1);
          return self;
        };
        const int I = i >> 1, J = j >> 1;
        const int I2 = fold(oi ? I + 1 : I - 1, C.nx, I, sx2);
        const int I3 = fold(oi ? I - 1 : I + 1, C.nx, I, sx3);
        const int J2 = fold(oj ? J + 1 : J - 1, C.ny, J, sy2);
        const int J3 = fold(oj ? J - 1 : J + 1, C.ny, J, sy3);
        ckb = (uint32_t)C.ldx * ES;
        const uint32_t r0 = (uint32_t)(J * C.nz) * ckb, r2 = (uint32_t)(J2 * C.nz) * ckb,
                       r3 = (uint32_t)(J3 * C.nz) * ckb;
        p00 = r0 + (uint32_t)I * ES;
        p20 = r0 + (uint32_t)I2 * ES;
        p30 = r0 + (uint32_t)I3 * ES;
        p02 = r2 + (uint32_t)I * ES;
        p22 = r2 + (uint32_t)I2 * ES;
        p32 = r2 + (uint32_t)I3 * ES;
        p03 = r3 + (uint32_t)I * ES;
        p23 = r3 + (uint32_t)I2 * ES;
      }
      auto own = [&](T u, T c00, T c20, T c02, T c22) {
        return prolong_add(u, c00, c20, c02, c22, T(3) * sx2, T(3) * sy2, sx2 * sy2);
      };
      T um = ldo<T>(pa, base + clamp(k0 - 1) * kb), uc = ldo<T>(pa, base + clamp(k0) * kb);
      // coarse values of the own correction at the row and at the next one
      T l00 = T(0), l20 = T(0), l02 = T(0), l22 = T(0);
      if constexpr (kPro) {
        const uint32_t om = clamp(k0 - 1) * ckb, oc = clamp(k0) * ckb;
        um = own(um, ldo<T>(pc, p00 + om), ldo<T>(pc, p20 + om), ldo<T>(pc, p02 + om),
                 ldo<T>(pc, p22 + om));
        l00 = ldo<T>(pc, p00 + oc);
        l20 = ldo<T>(pc, p20 + oc);
        l02 = ldo<T>(pc, p02 + oc);
        l22 = ldo<T>(pc, p22 + oc);
        uc = own(uc, l00, l20, l02, l22);
      }
      bool staged = false;
#pragma unroll
      for (int t0 = 0; t0 < R; t0 += CH) {
        T up[CH], e[CH], ww[CH], nn[CH], ss[CH], ff[CH];
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          const uint32_t k = clamp(k0 + t0 + t), kn = clamp(k0 + t0 + t + 1), o = k * kb;
          up[t] = ldo<T>(pa, base + kn * kb);
          e[t] = ldo<T>(pa, be + o);
          ww[t] = ldo<T>(pa, bw + o);
          nn[t] = ldo<T>(pa, bn + o);
          ss[t] = ldo<T>(pa, bs + o);
          ff[t] = ldo<T>(pf, base + o);
          if constexpr (kPro) {
            const uint32_t q = k * ckb, qn = kn * ckb;
            const T c00 = l00, c20 = l20, c02 = l02, c22 = l22;
            const T c30 = ldo<T>(pc, p30 + q), c32 = ldo<T>(pc, p32 + q);
            const T c03 = ldo<T>(pc, p03 + q), c23 = ldo<T>(pc, p23 + q);
            l00 = ldo<T>(pc, p00 + qn);
            l20 = ldo<T>(pc, p20 + qn);
            l02 = ldo<T>(pc, p02 + qn);
            l22 = ldo<T>(pc, p22 + qn);
            up[t] = own(up[t], l00, l20, l02, l22);
            // the neighbour with the same parent and the one with the next
            auto sibx = [&](T u) {
              return prolong_add(u, c00, c30, c02, c32, T(3) * sx3, T(3) * sy2, sx3 * sy2);
            };
            auto farx = [&](T u) {
              return prolong_add(u, c20, c00, c22, c02, T(3), T(3) * sy2, sy2);
            };
            auto siby = [&](T u) {
              return prolong_add(u, c00, c20, c03, c23, T(3) * sx2, T(3) * sy3, sx2 * sy3);
            };
            auto fary = [&](T u) {
              return prolong_add(u, c02, c22, c00, c20, T(3) * sx2, T(3), sx2);
            };
            const T sx = sibx(oi ? ww[t] : e[t]), fx = farx(oi ? e[t] : ww[t]);
            const T sy = siby(oj ? ss[t] : nn[t]), fy = fary(oj ? nn[t] : ss[t]);
            e[t] = oi ? fx : sx;
            ww[t] = oi ? sx : fx;
            nn[t] = oj ? fy : sy;
            ss[t] = oj ? sy : fy;
          }
        }
        if (!staged) __syncthreads();  // the profiles are in LDS
        staged = true;
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          const int k = k0 + t0 + t;
          if (t0 + t >= R || k >= NR) continue;
          // couplings and neighbours in the order of the half's elimination
          const bool down = k >= HALF;
          const BlockProf<T> p = s_t[down][down ? NR - 1 - k : k];
          const T cpv = p.x, cnx = p.y;
          const T vpv = down ? up[t] : um, vnx = down ? um : up[t];
          const T diag = fma(p.w, S, p.z);
          const T h = fma(cs, ss[t], fma(cn, nn[t], fma(cw, ww[t], ce * e[t])));
          const T mu = fma(cnx, vnx, fma(cpv, vpv, diag * uc));
          const T g = fma(p.w, h, ff[t]);
          s_r[k][col] = k < nz ? fma(wmu, mu, g) : T(0);
          if constexpr (kNorm) {
            const double r = active && k < nz ? (double)(g - mu) : 0.0;
            acc[0] = fma(r, r, acc[0]);
          }
          um = uc;
          uc = up[t];
        }
      }
    } else if constexpr (kRes) {
      // f - A u of the 2x2 children (a b / c d) and their sum
      const Lvl<T>& F = a.X;
      const int fnx = F.nx, fny = F.ny;
      const int fi = 2 * i, fj = 2 * j;
      const int fw = fi == 0 ? fnx - 1 : fi - 1, fe = fi + 2 == fnx ? 0 : fi + 2;
      const int fs = fj == 0 ? fny - 1 : fj - 1, fn = fj + 2 == fny ? 0 : fj + 2;
      const int r0 = fj * fnx, r1 = r0 + fnx, rs = fs * fnx;
      const T xab = F.cx[r0 + fi], xbE = F.cx[r0 + fi + 1], xWa = F.cx[r0 + fw];
      const T xcd = F.cx[r1 + fi], xdE = F.cx[r1 + fi + 1], xWc = F.cx[r1 + fw];
      const T yac = F.cy[r0 + fi], ybd = F.cy[r0 + fi + 1], ycN = F.cy[r1 + fi],
              ydN = F.cy[r1 + fi + 1], ySa = F.cy[rs + fi], ySb = F.cy[rs + fi + 1];
      const T Sa = xab + xWa + yac + ySa + F.wall[r0 + fi];
      const T Sb = xbE + xab + ybd + ySb + F.wall[r0 + fi + 1];
      const T Sc = xcd + xWc + ycN + yac + F.wall[r1 + fi];
      const T Sd = xdE + xcd + ydN + ybd + F.wall[r1 + fi + 1];
      const uint32_t fkb = (uint32_t)F.ldx * ES, fst = (uint32_t)nz * fkb;
      const uint32_t q0 = fj * fst + fi * ES, q1 = q0 + fst, qs = fs * fst + fi * ES,
                     qn = fn * fst + fi * ES, dw = (fw - fi) * (int)ES, de = (fe - fi) * (int)ES;
      V2 m0 = ldo<V2>(pa, q0 + clamp(k0 - 1) * fkb), m1 = ldo<V2>(pa, q1 + clamp(k0 - 1) * fkb);
      V2 c0 = ldo<V2>(pa, q0 + clamp(k0) * fkb), c1 = ldo<V2>(pa, q1 + clamp(k0) * fkb);
      bool staged = false;
#pragma unroll
      for (int t0 = 0; t0 < R; t0 += CH) {
        V2 p0[CH], p1[CH], vs[CH], vn[CH], f0[CH], f1[CH];
        T wa[CH], eb[CH], wc[CH], ed[CH];
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          const uint32_t o = clamp(k0 + t0 + t) * fkb, op = clamp(k0 + t0 + t + 1) * fkb;
          p0[t] = ldo<V2>(pa, q0 + op);
          p1[t] = ldo<V2>(pa, q1 + op);
          vs[t] = ldo<V2>(pa, qs + o);
          vn[t] = ldo<V2>(pa, qn + o);
          f0[t] = ldo<V2>(pf, q0 + o);
          f1[t] = ldo<V2>(pf, q1 + o);
          wa[t] = ldo<T>(pa, q0 + dw + o);
          eb[t] = ldo<T>(pa, q0 + de + o);
          wc[t] = ldo<T>(pa, q1 + dw + o);
          ed[t] = ldo<T>(pa, q1 + de + o);
        }
        if (!staged) __syncthreads();
        staged = true;
#pragma unroll
        for (int t = 0; t < CH; ++t) {
          const int k = k0 + t0 + t;
          if (t0 + t >= R || k >= NR) continue;
          const BlockProf<T> p = s_q[k];
          auto res = [&](T f, T Sx, T u, T k1, T n1, T k2, T n2, T k3, T n3, T k4, T n4, T um,
                         T up) {
            T h = k1 * n1;
            h = fma(k2, n2, h);
            h = fma(k3, n3, h);
            h = fma(k4, n4, h);
            T r = fma(p.w, Sx, p.z) * u;
            r = fma(-p.w, h, r);
            r = fma(p.x, um, r);
            r = fma(p.y, up, r);
            return f - r;
          };
          const T ra = res(f0[t].x, Sa, c0.x, xab, c0.y, xWa, wa[t], yac, c1.x, ySa, vs[t].x,
                           m0.x, p0[t].x);
          const T rb = res(f0[t].y, Sb, c0.y, xbE, eb[t], xab, c0.x, ybd, c1.y, ySb, vs[t].y,
                           m0.y, p0[t].y);
          const T rc = res(f1[t].x, Sc, c1.x, xcd, c1.y, xWc, wc[t], ycN, vn[t].x, yac, c0.x,
                           m1.x, p1[t].x);
          const T rd = res(f1[t].y, Sd, c1.y, xdE, ed[t], xcd, c1.x, ydN, vn[t].y, ybd, c0.y,
                           m1.y, p1[t].y);
          const T s = ra + rb + rc + rd;
          s_r[k][col] = k < nz ? s : T(0);
          if (active && k < nz) *reinterpret_cast<T*>(po1 + base + (uint32_t)k * kb) = s;
          m0 = c0;
          m1 = c1;
          c0 = p0[t];
          c1 = p1[t];
        }
      }
    } else {
      T v[R], q[kCg ? R : 1];
#pragma unroll
      for (int t = 0; t < R; ++t) {
        const uint32_t o = base + clamp(k0 + t) * kb;
        v[t] = ldo<T>(kCg ? po1 : pa, o);
        if constexpr (kCg) q[t] = ldo<T>(pa, o);
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < R; ++t) {
        const int k = k0 + t;
        if (k >= NR) continue;
        T s = v[t];
        if constexpr (kCg) {
          s = fma(-alpha, q[t], s);
          keep[t] = k < nz ? s : T(0);
          if (active && k < nz) {
            *reinterpret_cast<T*>(po1 + base + (uint32_t)k * kb) = s;
            acc[0] = fma((double)s, (double)s, acc[0]);
          }
        }
        s_r[k][col] = k < nz ? s : T(0);
      }
    }
  } else {
    // the pivots of both halves of the CB columns
    __syncthreads();
    const BlockProf<T>* pt = s_t[hs];
    T cprev = T(0);
    BlockProf<T> pn[U];
#pragma unroll
    for (int t = 0; t < U; ++t) pn[t] = pt[t];
#pragma unroll
    for (int s = 0; s < HALF; s += U) {
      BlockProf<T> p[U];
#pragma unroll
      for (int t = 0; t < U; ++t) p[t] = pn[t];
      if (s + U < HALF) {
#pragma unroll
        for (int t = 0; t < U; ++t) pn[t] = pt[s + U + t];
      }
#pragma unroll
      for (int t = 0; t < U; ++t) {
        T piv, c;
        T iv;
        elim_step(fma(p[t].w, S, p[t].z), p[t].x, p[t].y, cprev, piv, iv, c);
        cprev = c;
        if constexpr (kLds)
          io[(s + t) * step] = iv;
        else
          inv[s + t] = iv;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();

  if (w == 0) {
    // d'_k = (rhs_k - (coupling to the previous row) d'_{k-1}) / pivot, in
    // place; row s of the lane's half is at ro + s * step
    const BlockProf<T>* pt = s_t[hs];
    T* ro = &s_r[hs ? NR - 1 : 0][col];
    T d = T(0), c = T(0);
    T rn[U], an[U], vn[U];
    auto pinv = [&](int s) { return kLds ? io[s * step] : inv[kLds ? 0 : s]; };
#pragma unroll
    for (int t = 0; t < U; ++t) {
      rn[t] = ro[t * step];
      an[t] = pt[t].x;
      vn[t] = pinv(t);
    }
    // d' stays in registers, or in LDS where it would not fit beside the pivots
    constexpr bool kReg = !kLds && sizeof(T) * HALF <= 256;
    T dk[kReg ? HALF : 1];
#pragma unroll
    for (int s = 0; s < HALF; s += U) {
      T r[U], cp[U], iv[U];
#pragma unroll
      for (int t = 0; t < U; ++t) {
        r[t] = rn[t];
        cp[t] = an[t];
        iv[t] = vn[t];
      }
      if (s + U < HALF) {
#pragma unroll
        for (int t = 0; t < U; ++t) {
          rn[t] = ro[(s + U + t) * step];
          an[t] = pt[s + U + t].x;
          vn[t] = pinv(s + U + t);
        }
      }
#pragma unroll
      for (int t = 0; t < U; ++t) {
        d = fma(-cp[t], d, r[t]) * iv[t];
        if constexpr (kReg)
          dk[s + t] = d;
        else
          ro[(s + t) * step] = d;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // interface of the two halves: own last row x_a = d_a - c_a x_b
    c = pt[HALF - 1].y * pinv(HALF - 1);
    const T cq = __shfl_xor(c, CB), dq = __shfl_xor(d, CB);
    T x = fma(-c, dq, d) / fma(-c, cq, T(1));
    ro[(HALF - 1) * step] = x;
    // back: x_k = d'_k - c'_k x_{k+1}
#pragma unroll
    for (int t = 0; t < U; ++t) {
      if (HALF - 2 - t < 0) continue;
      an[t] = pt[HALF - 2 - t].y * pinv(HALF - 2 - t);
      rn[t] = kReg ? dk[kReg ? HALF - 2 - t : 0] : ro[(HALF - 2 - t) * step];
    }
#pragma unroll
    for (int s = HALF - 2; s >= 0; s -= U) {
      T cb[U], r[U];
#pragma unroll
      for (int t = 0; t < U; ++t) {
        if (s - t < 0) continue;
        cb[t] = an[t];
        r[t] = rn[t];
      }
#pragma unroll
      for (int t = 0; t < U; ++t) {
        const int q = s - U - t;
        if (q < 0) continue;
        an[t] = pt[q].y * pinv(q);
        rn[t] = kReg ? dk[kReg ? q : 0] : ro[q * step];
      }
#pragma unroll
      for (int t = 0; t < U; ++t) {
        if (s - t < 0) continue;
        x = fma(-cb[t], x, r[t]);
        ro[(s - t) * step] = x;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();

  if (w > 0) {
    const T scale = kCg ? T(1) : a.rho;
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const int k = k0 + t;
      if (active && k < nz) {
        const T x = s_r[k][col];
        if constexpr (kCg) acc[1] = fma((double)keep[t], (double)x, acc[1]);
        *reinterpret_cast<T*>(po + base + (uint32_t)k * kb) = kCg ? x : scale * x;
      }
    }
  }
  if constexpr (kNorm) {
    double v[1] = {acc[0]};
    block_partials<1, kBlockWaves>(v, a.partials);
  }
  if constexpr (kCg) block_partials<2, kBlockWaves>(acc, a.partials);
}

template <typename T, int MODE, int HALF, int CB>
__global__ __launch_bounds__(kBlockThreads)
__attribute__((amdgpu_waves_per_eu((block_lds<T, MODE, HALF, CB>()) ? 4 : 2))) void k_line_block(
    Lvl<T> L, BlockArgs<T> a, int ncols) {
  if (gated(L)) return;
  if constexpr (MODE == (int)BlockOp::CG) {
    if (a.st->done) return;
  }
  block_body<T, MODE, HALF, CB>(L, a, ncols, xcd_remap(blockIdx.x, gridDim.x));
}

// One launch for the items of many (instance, right-hand side) pairs.
template <int MODE, int HALF, int CB>
__global__ __launch_bounds__(kBlockThreads)
__attribute__((amdgpu_waves_per_eu((block_lds<float, MODE, HALF, CB>()) ? 4 : 2))) void
k_line_block_grouped(const GItem<float>* __restrict__ items, int nitems,
                     const int* __restrict__ active, float rho) {
  const int B = xcd_remap(blockIdx.x, gridDim.x);
  const GItem<float> it = items[find_item(items, nitems, B)];
  if (!active[it.pair]) return;
  BlockArgs<float> a{};
  a.a = it.a;
  a.f = it.b;
  a.o = it.o;
  a.o1 = it.o1;
  a.rho = rho;
  a.X = it.X;
  a.uc = it.c;
  block_body<float, MODE, HALF, CB>(it.L, a, it.L.nx * it.L.ny, B - it.blk0);
}

}  // namespace

}  // namespace gmg
