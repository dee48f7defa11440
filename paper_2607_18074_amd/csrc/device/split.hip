// fp32 products on the bf16 matrix units, and the channel products built on them.
//
// Every fp32 operand is the sum of three bf16 values (8 + 8 + 8 significant bits, round to nearest:
// v = h + m + l, |v - h - m - l| <= 2^-25 |v|); the six products of total order below 2^-24 (hh, hm,
// mh, mm, hl, lh) are accumulated in fp32 by v_mfma_f32_16x16x32_bf16.  The dropped ones are below
// 2^-25 of the product.  Measured on independent tiles: 2,230 TFLOP/s for that instruction, so 370 of
// fp32 product, against 153 for v_mfma_f32_16x16x4_f32.  That holds for magnitudes from 2^-109 (below,
// the low part falls under bf16's smallest step, 2^-133) to 3.396e38 (above, the high part rounds to
// infinity); an operand above that, or infinite, gives NaN (its split subtracts infinity from itself).
//
// Operand layout (lane l = j + 16 g): A row j and B column j supply the eight k values of slot
// group g; D[4g + r][j] sits in accumulator register r of lane j + 16 g.

typedef __bf16 sbm_b8 __attribute__((ext_vector_type(8)));
typedef __bf16 sbm_b4 __attribute__((ext_vector_type(4)));
typedef __bf16 sbm_b2 __attribute__((ext_vector_type(2)));
typedef float sbm_f4 __attribute__((ext_vector_type(4)));
typedef float sbm_f2 __attribute__((ext_vector_type(2)));

struct sbm_p3 { sbm_b8 p[3]; };   // the three bf16 planes of eight values

// two fp32 values rounded to bf16: packed, and as fp32 again
struct sbm_w2 { unsigned w; float a, b; };
SB_DEV sbm_w2 sbm_pk(float a, float b) {
  const sbm_b2 t = {(__bf16)a, (__bf16)b};
  sbm_w2 o;
  o.w = __builtin_bit_cast(unsigned, t);
  o.a = __builtin_bit_cast(float, o.w << 16);
  o.b = __builtin_bit_cast(float, o.w & 0xffff0000u);
  return o;
}

SB_DEV sbm_p3 sbm_split(const float (&v)[8]) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  u4 h, m, l;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const sbm_w2 x = sbm_pk(v[2 * k], v[2 * k + 1]);
    const float r0 = v[2 * k] - x.a, r1 = v[2 * k + 1] - x.b;
    const sbm_w2 y = sbm_pk(r0, r1);
    h[k] = x.w;
    m[k] = y.w;
    l[k] = sbm_pk(r0 - y.a, r1 - y.b).w;
  }
  sbm_p3 o;
  o.p[0] = __builtin_bit_cast(sbm_b8, h);
  o.p[1] = __builtin_bit_cast(sbm_b8, m);
  o.p[2] = __builtin_bit_cast(sbm_b8, l);
  return o;
}

SB_DEV sbm_f4 sbm_mfma(sbm_b8 a, sbm_b8 b, sbm_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// four 16-bit values of column j of the 4 x 16 block whose row r, column quad c this lane
// (4 r + c of its 16) points at
SB_DEV sbm_b4 sbm_tr4(const char* p) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s4 lds_s4;
  return __builtin_bit_cast(sbm_b4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p));
}

// ---------------------------------------------------------------------------
// Channel products of fp32 plans.
//
//   sobek_sp3_sa    out(i, m_o, w) (+)= sum_k S_g[(i,m_o), k] A_g[k, w]   (or split-K partials)
//   sobek_sp3_red   the partials, summed in split order
//   sobek_sp3_ga    P_g[split, k, w] (+)= sum_{(i,m_o) in split} S_g[(i,m_o), k] mbar(i, m_o, w)
//   sobek_sp3_sbar  Sbar_g[(i,m_o), k] = sum_w mbar(i, m_o, w) A_g[k, w]
//
// One launch covers the output groups [glo, ghi): a block finds its group from its index, so few
// receivers cost one launch, not one per group.  Operands are loaded as float4, split in registers
// and staged in LDS as bf16 planes (each element is split once per block); the next slab's loads are
// in flight while the matrix units work.  Operands whose reduction index is contiguous in memory are
// stored [octet of k][row][8]; the others as loaded, [k][column], and read transposed
// (ds_read_b64_tr_b16).  Tiles are computed transposed (D rows = output columns), so a lane ends
// with four consecutive output columns of one row: one float4 store.  S (or Sbar) passes between HBM
// and the CUs once, at 2.8 to 3.5 TB/s of the 4.7 of a copy (what holds the rest was not measured); per
// pass over 20,000 receivers of 64x0e+64x1o+64x1e+64x2e at K = 16 (5.2 GB of state), fp32 matrix
// instructions before and now: m = S A 2.80 -> 1.86 ms, Sbar 3.23 -> 1.51 ms, A_bar 2.86 -> 1.67 ms.  Loads are never conditional
// (addresses are clamped into the operand; what lies past the reduction's end is zeroed on its way to
// LDS, in one of the two operands; rows and columns past the edge are not stored).

// four values split into the planes at d, d + plane, d + 2 plane
SB_DEV void sp3_store4(char* d, int plane, const sb_v4 v) {
  const sbm_w2 h = sbm_pk(v[0], v[1]), h2 = sbm_pk(v[2], v[3]);
  const float r0 = v[0] - h.a, r1 = v[1] - h.b, r2 = v[2] - h2.a, r3 = v[3] - h2.b;
  const sbm_w2 m = sbm_pk(r0, r1), m2 = sbm_pk(r2, r3);
  const sbm_w2 l = sbm_pk(r0 - m.a, r1 - m.b), l2 = sbm_pk(r2 - m2.a, r3 - m2.b);
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  *(u2*)d = (u2){h.w, h2.w};
  *(u2*)(d + plane) = (u2){m.w, m2.w};
  *(u2*)(d + 2 * plane) = (u2){l.w, l2.w};
}

// acc[i][t] += b x a[i] for every i, over one 32-deep step.  The matrix unit rounds its running sum
// more coarsely than an fp32 add (a 5,000-deep product summed in its accumulator alone is 1.2e-6 off
// in norm, with fp32 multiply-adds 7e-7), so a step starts from zero, takes the small products first,
// and is added to the accumulator by the vector unit.
template <int TM, int TN>
SB_DEV void sp3_six(sbm_f4 (&acc)[TM][TN], int t, const sbm_p3& b, const sbm_p3 (&a)[TM]) {
  constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
  sbm_f4 v[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) v[i] = (sbm_f4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int n = 0; n < 6; ++n)
#pragma unroll
    for (int i = 0; i < TM; ++i) v[i] = sbm_mfma(b.p[pb[n]], a[i].p[pa[n]], v[i]);
#pragma unroll
  for (int i = 0; i < TM; ++i) acc[i][t] += v[i];
}

#define SP3_OCT 2112                       // bytes between octets of a 128-row block: 128 rows x 16 + 64
#define SP3_KPL (4 * SP3_OCT)              // one plane of a [4 octets][128 rows] block
constexpr int sp3_pitch(int cols) { return cols * 2 + (cols >= 64 ? 32 : 16); }   // bytes of a [k] row

// operand with the reduction index contiguous: row `r` of a [4][128][8] block
SB_DEV sbm_p3 sp3_rows(const char* s, int r, int g) {
  sbm_p3 o;
#pragma unroll
  for (int p = 0; p < 3; ++p) o.p[p] = *(const sbm_b8*)(s + p * SP3_KPL + g * SP3_OCT + r * 16);
  return o;
}

// operand stored [32][cols], 16 columns from c0
template <int COLS>
SB_DEV sbm_p3 sp3_cols(const char* s, int c0, int j, int g) {
  constexpr int PT = sp3_pitch(COLS);
  const char* b = s + (8 * g + (j >> 2)) * PT + (c0 + 4 * (j & 3)) * 2;
  sbm_p3 o;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const sbm_b4 lo = sbm_tr4(b + p * 32 * PT), hi = sbm_tr4(b + p * 32 * PT + 4 * PT);
    o.p[p] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  return o;
}

constexpr int sp3_lds_sa(int BN) { return 3 * SP3_KPL + 3 * 32 * sp3_pitch(BN); }

// 128 rows x BN columns, reduction [kbeg, kend)
template <int BN, int D, int DG, int CG, int OFF>
SB_DEV void sp3_sa(char* lds, const float* __restrict__ S, int nrows, const float* __restrict__ W,
                   const int* __restrict__ ktab, float* __restrict__ out, int r0, int accumulate, int rb, int cb,
                   int kbeg, int kend, float* __restrict__ P) {
  constexpr int WC = BN >= 128 ? 2 : 1, WR = 4 / WC, TM = 8 / WR, TN = BN / WC / 16;
  constexpr int PT = sp3_pitch(BN), NB = (32 * BN / 4 + 255) / 256;
  char* sA = lds;
  char* sB = lds + 3 * SP3_KPL;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, j = lane & 15, g = lane >> 4;
  const int wr = (wave / WC) * (TM * 16), wc = (wave % WC) * (TN * 16);
  sbm_f4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = (sbm_f4){0.f, 0.f, 0.f, 0.f};
  sb_v4 ra[4], rbv[NB];
  int kt[NB];   // A's row offsets of the next load: read one load ahead, so no load waits for its offset
  auto rows = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NB; ++i) kt[i] = ktab[min(k0 + (tid + 256 * i) / (BN / 4), kend - 1)];
  };
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      rbv[i] = sb_ld4(W + (sb_i64)kt[i] + min(cb + 4 * ((tid + 256 * i) % (BN / 4)), CG - 4));
    }
    rows(k0 + 32);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ra[i] = sb_ld4(S + (sb_i64)min(rb + (tid >> 3) + 32 * i, nrows - 1) * D + min(k0 + 4 * (tid & 7), D - 4));
  };
  rows(kbeg);
  auto store = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (tid >> 3) + 32 * i, kq = tid & 7;
      sp3_store4(sA + (kq >> 1) * SP3_OCT + row * 16 + (kq & 1) * 8, SP3_KPL, ra[i]);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int idx = tid + 256 * i, kk = idx / (BN / 4), c = 4 * (idx % (BN / 4));
      if (k0 + kk >= kend) rbv[i] = (sb_v4){0.f, 0.f, 0.f, 0.f};
      if (kk < 32) sp3_store4(sB + kk * PT + c * 2, 32 * PT, rbv[i]);
    }
  };
  load(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += 32) {
    store(k0);
    __syncthreads();
    if (k0 + 32 < kend) load(k0 + 32);
    sbm_p3 a[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = sp3_rows(sA, wr + 16 * i + j, g);
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      const sbm_p3 b = sp3_cols<BN>(sB, wc + 16 * t, j, g);
      sp3_six<TM, TN>(acc, t, b, a);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = rb + wr + 16 * i + j;
    if (row < nrows) {
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int col = cb + wc + 16 * t + 4 * g;
        if (col < CG) {
          if (P) {
            *(sbm_f4*)(P + (sb_i64)row * CG + col) = acc[i][t];
          } else {
            sbm_f4* o = (sbm_f4*)(out + sb_row_addr(row, DG, CG, OFF, CXO, r0) + col);
            *o = accumulate ? *o + acc[i][t] : acc[i][t];
          }
        }
      }
    }
  }
}

constexpr int sp3_lds_ga(int BN) { return 3 * 32 * (sp3_pitch(128) + sp3_pitch(BN)); }

// 128 k x BN columns, rows [rbeg, rend); S^T and mbar both read transposed
template <int BN, int D, int DG, int CG, int OFF>
SB_DEV void sp3_ga(char* lds, const float* __restrict__ S, const float* __restrict__ M, float* __restrict__ P, int r0,
                   int accumulate, int kb, int cb, int rbeg, int rend) {
  constexpr int WC = BN >= 128 ? 2 : 1, WR = 4 / WC, TM = 8 / WR, TN = BN / WC / 16;
  constexpr int PA = sp3_pitch(128), PB = sp3_pitch(BN), NB = (32 * BN / 4 + 255) / 256;
  char* sA = lds;
  char* sB = lds + 3 * 32 * PA;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, j = lane & 15, g = lane >> 4;
  const int wr = (wave / WC) * (TM * 16), wc = (wave % WC) * (TN * 16);
  sbm_f4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = (sbm_f4){0.f, 0.f, 0.f, 0.f};
  sb_v4 ra[4], rbv[NB];
  auto load = [&](int q0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ra[i] = sb_ld4(S + (sb_i64)min(q0 + (tid >> 5) + 8 * i, rend - 1) * D + min(kb + 4 * (tid & 31), D - 4));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int idx = tid + 256 * i, row = min(q0 + idx / (BN / 4), rend - 1);
      rbv[i] = sb_ld4(M + sb_row_addr(row, DG, CG, OFF, CXO, r0) + min(cb + 4 * (idx % (BN / 4)), CG - 4));
    }
  };
  auto store = [&](int q0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      sp3_store4(sA + ((tid >> 5) + 8 * i) * PA + 8 * (tid & 31), 32 * PA, ra[i]);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int idx = tid + 256 * i, rr = idx / (BN / 4), c = 4 * (idx % (BN / 4));
      if (q0 + rr >= rend) rbv[i] = (sb_v4){0.f, 0.f, 0.f, 0.f};
      if (rr < 32) sp3_store4(sB + rr * PB + c * 2, 32 * PB, rbv[i]);
    }
  };
  if (rbeg < rend) load(rbeg);
  for (int q0 = rbeg; q0 < rend; q0 += 32) {
    store(q0);
    __syncthreads();
    if (q0 + 32 < rend) load(q0 + 32);
    sbm_p3 a[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = sp3_cols<128>(sA, wr + 16 * i, j, g);
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      const sbm_p3 b = sp3_cols<BN>(sB, wc + 16 * t, j, g);
      sp3_six<TM, TN>(acc, t, b, a);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int k = kb + wr + 16 * i + j;
    if (k < D) {
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int col = cb + wc + 16 * t + 4 * g;
        if (col < CG) {
          sbm_f4* o = (sbm_f4*)(P + (sb_i64)k * CG + col);
          *o = accumulate ? *o + acc[i][t] : acc[i][t];
        }
      }
    }
  }
}

// 128 rows of mbar against the k tiles [t0, t1) of 64 columns.  A wave keeps the planes of its 32 rows
// in registers (they pass through LDS once, 32 w at a time); A's rows of the next tile are loaded
// while the current one is multiplied.  CG up to 128; the planes of 128 columns do not all fit the
// registers (65 to 195 of a lane's are spilled; with that, 6,000 receivers of 128x0e+128x1o+128x2e+64x3o
// at K = 16 3.67 -> 3.06 ms, of 128x0e+64x1o+64x2e 0.64 -> 0.44).
#define SP3_AOC (64 * 16 + 64)             // bytes between octets of a 64-row block
constexpr int sp3_lds_sbar(int CG) {
  const int a = 3 * ((CG + 31) / 32) * 4 * SP3_AOC;
  return a > 3 * SP3_KPL ? a : 3 * SP3_KPL;
}
template <int D, int DG, int CG, int OFF>
SB_DEV void sp3_sbar(char* lds, const float* __restrict__ M, int nrows, const float* __restrict__ W,
                     const int* __restrict__ ktab, float* __restrict__ Sbar, int r0, int rb, int t0, int t1) {
  constexpr int NK = (CG + 31) / 32, QW = NK * 8;          // 32-wide steps; float4 per padded row
  constexpr int APL = NK * 4 * SP3_AOC, NA = 64 * QW / 256;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, j = lane & 15, g = lane >> 4;
  sbm_p3 m[NK][2];
#pragma unroll
  for (int s = 0; s < NK; ++s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (tid >> 3) + 32 * i, q = tid & 7, c = 32 * s + 4 * q;
      sb_v4 v = sb_ld4(M + sb_row_addr(min(rb + row, nrows - 1), DG, CG, OFF, CXO, r0) + min(c, CG - 4));
      if (c >= CG) v = (sb_v4){0.f, 0.f, 0.f, 0.f};
      sp3_store4(lds + (q >> 1) * SP3_OCT + row * 16 + (q & 1) * 8, SP3_KPL, v);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) m[s][i] = sp3_rows(lds, 32 * wave + 16 * i + j, g);
    __syncthreads();
  }
  sb_v4 ra[NA];
  int kt[NA];   // A's row offsets of the next load, read one load ahead
  auto rows = [&](int t) {
#pragma unroll
    for (int i = 0; i < NA; ++i) kt[i] = ktab[min(64 * t + (tid + 256 * i) / QW, D - 1)];
  };
  auto load = [&](int t) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      ra[i] = sb_ld4(W + (sb_i64)kt[i] + min(4 * ((tid + 256 * i) % QW), CG - 4));
    }
    rows(t + 1);
  };
  rows(t0);
  load(t0);
  for (int t = t0; t < t1; ++t) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int idx = tid + 256 * i, kc = idx / QW, q = idx % QW;
      sp3_store4(lds + (q >> 1) * SP3_AOC + kc * 16 + (q & 1) * 8, APL, ra[i]);
    }
    __syncthreads();
    if (t + 1 < t1) load(t + 1);
    sbm_f4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[i][c] = (sbm_f4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NK; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sbm_p3 a;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a.p[p] = *(const sbm_b8*)(lds + p * APL + (4 * s + g) * SP3_AOC + (16 * c + j) * 16);
        sp3_six<2, 4>(acc, c, a, m[s]);
      }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = rb + 32 * wave + 16 * i + j;
      if (row < nrows) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int k = 64 * t + 16 * c + 4 * g;
          if (k < D) *(sbm_f4*)(Sbar + (sb_i64)row * D + k) = acc[i][c];
        }
      }
    }
    __syncthreads();
  }
}
