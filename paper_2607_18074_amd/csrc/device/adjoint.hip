// Adjoint edge stage in moment form, for plans with K = 16 radial features and input multiplicities in
// multiples of 16.  With the adjoint moments of receiver i (the coupling applied to its adjoint state,
// once per receiver instead of once per edge)
//   Rb[(m_y, q), (m_i, u)] = sum over paths and m_o of c[m_i, m_y, m_o] Sbar[pi, m_o, q, u]
// every edge term of Section 4.3 is one of two matrix products over the receiver's edges:
//   xbar_e[m_i, u]  = sum over (m_y, q) of (phi_q Y_my)(e) Rb     (contribution to the sender's row)
//   T_e[m_y, q]     = sum over (m_i, u) of x_j(e)[u, m_i] Rb,
//   phibar_e[q] = sum_my Y_my T_e[m_y, q],   Ybar_e[m_y] = sum_q phi_q T_e[m_y, q].
// The double backward's directional terms (Section 4.4) replace phi Y by its tangent in the first
// product and contract the same T with Ydot, phidot and (Hessian term) phi.
//
// A block takes one receiver and 64 of its edges: four tiles of 16 edges, two waves a tile, one for
// each half of a step's columns.  A step is two m_y against a group of up to six slots (input irrep, m_i;
// seven for an irrep of l = 3) on one 16-channel tile: a wave forms one slot's Rb from the adjoint state (lane = (u, four q)),
// split into three bf16 planes in LDS (two buffers, one barrier a step), and both products read that
// copy, the second one transposed.  The adjoint state of the next step and the sender rows of the next
// channel tile are loaded ahead of a step's products.  The planes of phi Y are formed once per 64 edges.
// Products are taken transposed (columns = edges), so a lane ends with the results of one edge.
//
// The adjoint state is stored [path, u][q] for these plans: a wave's load of one entry is 1 KB contiguous
// (four dwords C apart in the [path][q][u] order; 9.3 -> 8.1 ms in the first case below).  What bounds it
// is a step's chain (load, form and split, barrier, LDS reads, six dependent products), about 1 us with
// two waves a SIMD; without the products a receiver of four edges still takes four fifths of the time.
// Edge time of one backward, per-edge kernel before and this one now:
//   64x0e+64x1o+64x1e+64x2e lmax 3, 20,000 receivers, 1,000,000 edges     13.3 -> 7.8 ms
//   128x0e+128x1o+128x2e+64x3o lmax 3, 480,000 edges                      14.3 -> 11.1 ms
//   its radius-only double backward, first plan                           12.3 -> 8.3 ms

#define SBA_BLK 640                         // bytes of one (m_y, slot): [q octet][u][8 q], octets 320 apart
#define SBA_NC ((NSH + 1) / 2)              // steps per channel tile: two m_y each
#define SBA_THREADS 512

// v += a x b from zero, small products first, for two independent pairs
SB_DEV void sba_six2(sbm_f4& c0, sbm_f4& c1, const sbm_p3& a0, const sbm_p3& b0, const sbm_p3& a1, const sbm_p3& b1) {
  constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int n = 0; n < 6; ++n) {
    c0 = sbm_mfma(a0.p[pa[n]], b0.p[pb[n]], c0);
    c1 = sbm_mfma(a1.p[pa[n]], b1.p[pb[n]], c1);
  }
}

// four radial entries of one (m_y, slot) block to the three planes
SB_DEV void sba_put4(char* d, int plane, const sbm_f4 v) {
  const sbm_w2 h0 = sbm_pk(v[0], v[1]), h1 = sbm_pk(v[2], v[3]);
  const float r0 = v[0] - h0.a, r1 = v[1] - h0.b, r2 = v[2] - h1.a, r3 = v[3] - h1.b;
  const sbm_w2 m0 = sbm_pk(r0, r1), m1 = sbm_pk(r2, r3);
  const sbm_w2 l0 = sbm_pk(r0 - m0.a, r1 - m0.b), l1 = sbm_pk(r2 - m1.a, r3 - m1.b);
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  *(u2*)d = (u2){h0.w, h1.w};
  *(u2*)(d + plane) = (u2){m0.w, m1.w};
  *(u2*)(d + 2 * plane) = (u2){l0.w, l1.w};
}

// a wave-uniform pointer kept in scalar registers: loads then take it with a 32-bit lane offset, and no
// 64-bit lane address of a later step is formed early and kept (257 spilled registers without it)
#ifndef SBA_SCALAR
#define SBA_SCALAR(p) asm volatile("" : "+s"(p))
#endif

// four radial entries of one channel of an adjoint-state row (stored [path, u][q] on this route: 1 KB
// contiguous a wave); off: the lane's bytes past the base
SB_DEV sbm_f4 sba_ld4(const float* __restrict__ base, unsigned off) {
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) sbm_f4 gf4;
  gchar* b = (gchar*)base;
  SBA_SCALAR(b);
  return *(gf4*)(b + off);
}

// One step's products for a wave (column half hf): xbar of its slots, T of its m_y (NMY: m_y of the step).
// Chains of six run in twos; the odd ones of xbar and T go together (apart, their latencies added up:
// 8.1 -> 7.8 ms in the first case above).
template <int SL, int NMY>
SB_DEV void sba_step(const char* buf, int j, int g, int hf, bool has_x, const sbm_b8* phi_planes,
                     const sbm_p3 (&xp)[(SL + 1) / 2], sbm_f4 (&xacc)[(SL + 1) / 2], sbm_f4& T) {
  constexpr int PL = 2 * SL * SBA_BLK, SH = (SL + 1) / 2;
  // a step of one m_y: its phi Y is zero in the other's places, which read the first one's values
  const char* bx = buf + min(g >> 1, NMY - 1) * (SL * SBA_BLK) + (g & 1) * 320 + j * 16;
  auto xop = [&](int s) {
    const char* bs = bx + min(hf * SH + s, SL - 1) * SBA_BLK;
    sbm_p3 B;
#pragma unroll
    for (int p = 0; p < 3; ++p) B.p[p] = *(const sbm_b8*)(bs + p * PL);
    return B;
  };
  const int row = j >> 2, c = j & 3;
  const char* bt = buf + min(hf, NMY - 1) * (SL * SBA_BLK) + (c >> 1) * 320 + (8 * (g & 1) + row) * 16 + (c & 1) * 8;
  auto top = [&](int s) {
    const char* bs = bt + min(2 * s + (g >> 1), SL - 1) * SBA_BLK;
    sbm_p3 B;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const sbm_b4 lo = sbm_tr4(bs + p * PL), hi = sbm_tr4(bs + p * PL + 64);
      B.p[p] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    return B;
  };
  sbm_p3 pa;
#pragma unroll
  for (int p = 0; p < 3; ++p) pa.p[p] = phi_planes[p * 64];
  if (has_x) {
#pragma unroll
    for (int s = 0; s + 1 < SH; s += 2) {
      const sbm_p3 B0 = xop(s), B1 = xop(s + 1);
      sbm_f4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
      sba_six2(v0, v1, B0, pa, B1, pa);
      xacc[s] += v0;
      xacc[s + 1] += v1;
    }
  }
  const bool has_t = hf < NMY;
  sbm_f4 t = {0.f, 0.f, 0.f, 0.f};
  if (has_t) {
#pragma unroll
    for (int s = 0; s + 1 < SH; s += 2) {
      const sbm_p3 B0 = top(s), B1 = top(s + 1);
      sbm_f4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
      sba_six2(v0, v1, B0, xp[s], B1, xp[s + 1]);
      t += v0 + v1;
    }
  }
  if (SH % 2) {   // both, whether or not each is wanted
    const sbm_p3 B0 = xop(SH - 1), B1 = top(SH - 1);
    sbm_f4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = {0.f, 0.f, 0.f, 0.f};
    sba_six2(v0, v1, B0, pa, B1, xp[SH - 1]);
    xacc[SH - 1] += v0;
    t += v1;
  }
  if (has_t) T += t;
}

// Edge outputs of a wave's m_y (2 c + hf): lane (edge j, g) holds T[c][r] of q = 4 g + r.  The other
// half's sums come through sX (eight floats a lane).  Called by every wave of the block.
template <bool DB>
SB_DEV void sba_finish(const sbm_f4 (&T)[SBA_NC], const float* sYw, float* sX, int lane, int hf, bool act, sb_i64 e,
                       bool valid, float ux, float uy, float uz, float rinv, float dx, float dy, float dz,
                       const float* __restrict__ phi, const float* __restrict__ phidot, int flags,
                       float* __restrict__ gphi, float* __restrict__ gevec, int accum) {
  const int j = lane & 15, g = lane >> 4;
  sbm_f4 gp = {0.f, 0.f, 0.f, 0.f};
  float gg[3] = {0.f, 0.f, 0.f};
  if (act) {
    const sbm_f4 ph = *(const sbm_f4*)(phi + e * K + 4 * g);
    sbm_f4 phd = {0.f, 0.f, 0.f, 0.f};
    if (DB && (flags & 1)) phd = *(const sbm_f4*)(phidot + e * K + 4 * g);
    float yb[NSH], hb[NSH];
#pragma unroll
    for (int m = 0; m < NSH; ++m) yb[m] = hb[m] = 0.f;
#pragma unroll
    for (int c = 0; c < SBA_NC; ++c) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (2 * c + h < NSH && h == hf) {
          const int my = 2 * c + h < NSH ? 2 * c + h : 0;
          const float y = sYw[my * 16 + j];   // Y, DB: Ydot
          gp += T[c] * y;
          if (gevec) {
            const sbm_f4 w = DB ? phd : ph;
            float a = T[c][0] * w[0] + T[c][1] * w[1] + T[c][2] * w[2] + T[c][3] * w[3];
            a += __shfl_xor(a, 16);
            a += __shfl_xor(a, 32);
            yb[my] = a;
            if (DB) {
              float b = T[c][0] * ph[0] + T[c][1] * ph[1] + T[c][2] * ph[2] + T[c][3] * ph[3];
              b += __shfl_xor(b, 16);
              b += __shfl_xor(b, 32);
              hb[my] = b;
            }
          }
        }
      }
    }
    if (gevec) {
      sb_sh_vjp(ux, uy, uz, rinv, yb, gg);
      if (DB && (flags & 4)) {
        float hh[3];
        sb_sh_hvp(ux, uy, uz, rinv, hb, dx, dy, dz, hh);
        gg[0] += hh[0]; gg[1] += hh[1]; gg[2] += hh[2];
      }
    }
    if (DB && !(flags & 4)) gp = (sbm_f4){0.f, 0.f, 0.f, 0.f};
    if (hf) {
      *(sbm_f4*)(sX + 8 * lane) = gp;
      sX[8 * lane + 4] = gg[0]; sX[8 * lane + 5] = gg[1]; sX[8 * lane + 6] = gg[2];
    }
  }
  __syncthreads();
  if (act && !hf && valid) {
    if (gphi) {
      sbm_f4* o = (sbm_f4*)(gphi + e * K + 4 * g);
      gp += *(const sbm_f4*)(sX + 8 * lane);
      *o = accum ? *o + gp : gp;
    }
    if (gevec && g == 0) {
      float* o = gevec + 3 * e;
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const float v = gg[m] + sX[8 * lane + 4 + m];
        o[m] = accum ? o[m] + v : v;
      }
    }
  }
  __syncthreads();
}
