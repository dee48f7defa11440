// Generator of the split channel products' entry points (device/split.hip), one launch for all output
// groups, with every group's sizes as constants.
#include <algorithm>
#include <sstream>

#include "split.h"

namespace sobek {

namespace {
const char* kSplit =
#include "split_embed.inc"
    ;
}  // namespace

bool split_plan(const Plan& p) { return p.mode == 0 && p.dtype == 0 && p.vec4 && !p.paths.empty(); }

int split_bn(int C) { return C <= 16 ? 16 : C <= 32 ? 32 : C <= 64 ? 64 : 128; }

namespace {

// The channel products' entry points: blocks of the output groups [glo, ghi) in group order, each
// group's own tile counts; S holds group blocks s_ncap receivers apart (0: one group at S).
void emit_split(std::ostringstream& o, const Plan& p) {
  const int G = (int)p.groups.size();
  auto lds = [&](const char* f, bool bn) {
    std::ostringstream e;
    for (int i = 0; i + 1 < G; ++i) e << "sp3_max(";
    for (int i = 0; i < G; ++i) {
      const int C = p.groups[i].C;
      if (i) e << ", ";
      e << f << "(" << (bn ? split_bn(C) : std::min(C, 128)) << ")" << (i ? ")" : "");
    }
    return e.str();
  };
  o << "constexpr int sp3_max(int a, int b) { return a > b ? a : b; }\n";
  const char* head = "extern \"C\" __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void ";
  // out rows of receivers [r0, r0 + n)
  o << head << "sobek_sp3_sa(const float* __restrict__ S, sb_i64 s_ncap, int r0, int n, const float* __restrict__ W,"
       " const int* __restrict__ ktab, float* __restrict__ out, int accumulate, float* __restrict__ P, int ns, int glo,"
       " int ghi) {\n  __shared__ __attribute__((aligned(128))) char lds[" << lds("sp3_lds_sa", true) << "];\n"
       "  int b = blockIdx.x;\n  sb_i64 po = 0;\n";
  for (int i = 0; i < G; ++i) {
    const Group& g = p.groups[i];
    const int bn = split_bn(g.C), ct = (g.C + bn - 1) / bn;
    o << "  if (" << i << " >= glo && " << i << " < ghi) {\n    constexpr int D = " << g.D << ", DG = " << g.d << ", CG = " << g.C
      << ";\n    const int kper = max(128, ((D + ns - 1) / ns + 31) / 32 * 32), nz = (D + kper - 1) / kper, rt = (n * DG + 127) / 128;\n"
      << "    if (b < rt * nz * " << ct << ") {\n"
      << "      const int z = b / (rt * " << ct << "), t = b % (rt * " << ct << ");\n"
      << "      sp3_sa<" << bn << ", D, DG, CG, " << g.off << ">(lds, S + s_ncap * " << g.s_off << "LL, n * DG, W, ktab + "
      << g.ktab_off << ", out, r0, accumulate, t / " << ct << " * 128, t % " << ct << " * " << bn
      << ", z * kper, min(D, (z + 1) * kper), P ? P + po + (sb_i64)z * n * (DG * CG) : nullptr);\n      return;\n    }\n"
      << "    b -= rt * nz * " << ct << ";\n    po += (sb_i64)nz * n * (DG * CG);\n  }\n";
  }
  o << "}\n";
  o << "extern \"C\" __global__ __launch_bounds__(256) void sobek_sp3_red(const float* __restrict__ P, int r0, int n,"
       " float* __restrict__ out, int accumulate, int ns, int glo, int ghi) {\n"
       "  sb_i64 t = (sb_i64)blockIdx.x * 256 + threadIdx.x, po = 0;\n";
  for (int i = 0; i < G; ++i) {
    const Group& g = p.groups[i];
    o << "  if (" << i << " >= glo && " << i << " < ghi) {\n    constexpr int D = " << g.D << ", DG = " << g.d << ", CG = " << g.C
      << ";\n    const int kper = max(128, ((D + ns - 1) / ns + 31) / 32 * 32), nz = (D + kper - 1) / kper;\n"
      << "    const sb_i64 nq = (sb_i64)n * (DG * CG / 4);\n    if (t < nq) {\n"
      << "      const int row = (int)(t / (CG / 4)), c = 4 * (int)(t % (CG / 4));\n"
      << "      const float* src = P + po + 4 * t;\n      sb_v4 v = sb_ld4(src);\n"
      << "      for (int z = 1; z < nz; ++z) v += sb_ld4(src + z * 4 * nq);\n"
      << "      sb_v4* o = (sb_v4*)(out + sb_row_addr(row, DG, CG, " << g.off << ", CXO, r0) + c);\n"
      << "      *o = accumulate ? *o + v : v;\n      return;\n    }\n    t -= nq;\n    po += nz * 4 * nq;\n  }\n";
  }
  o << "}\n";
  // weight-gradient partials: the split count of a group follows the pass's receiver capacity
  auto ga_group = [&](int i) {
    const Group& g = p.groups[i];
    std::ostringstream e;
    e << "  if (" << i << " >= glo && " << i << " < ghi) {\n    constexpr int D = " << g.D << ", DG = " << g.d << ", CG = " << g.C
      << ";\n    const int ns = (int)min((sb_i64)" << ga_max_splits(p, g) << ", max((sb_i64)1, cap * DG / 64));\n";
    return e.str();
  };
  o << head << "sobek_sp3_ga(const float* __restrict__ S, sb_i64 s_ncap, int r0, int n, const float* __restrict__ M,"
       " float* __restrict__ P, sb_i64 cap, int accumulate, int glo, int ghi) {\n"
       "  __shared__ __attribute__((aligned(128))) char lds[" << lds("sp3_lds_ga", true) << "];\n  int b = blockIdx.x;\n";
  for (int i = 0; i < G; ++i) {
    const Group& g = p.groups[i];
    const int bn = split_bn(g.C), ct = (g.C + bn - 1) / bn, kt = (int)((g.D + 127) / 128) * ct;
    o << ga_group(i) << "    if (b < " << kt << " * ns) {\n      const int z = b / " << kt << ", t = b % " << kt << ";\n"
      << "      const int rps = ((n * DG + ns - 1) / ns + 31) / 32 * 32;\n"
      << "      sp3_ga<" << bn << ", D, DG, CG, " << g.off << ">(lds, S + s_ncap * " << g.s_off
      << "LL, M, P + (sb_i64)z * (D * CG), r0, accumulate, t / " << ct << " * 128, t % " << ct << " * " << bn
      << ", z * rps, min(n * DG, (z + 1) * rps));\n      return;\n    }\n    b -= " << kt << " * ns;\n"
      << "  }\n  P += (sb_i64)min((sb_i64)" << ga_max_splits(p, g) << ", max((sb_i64)1, cap * " << g.d << " / 64)) * "
      << (int64_t)g.D * g.C << "LL;\n";
  }
  o << "}\n";
  // Up to 64 splits of few elements: what bounds it is the latency of a thread's loads, 32 of them in flight
  // (one at a time 33 us for 20x0e+12x1o to 36x0e+72x1o, 19 for 12x0e to 16x0e; 12 and 8 now)
  o << "extern \"C\" __global__ __launch_bounds__(256) void sobek_sp3_gared(const float* __restrict__ P, sb_i64 cap,"
       " const int* __restrict__ ktab, float* __restrict__ gW, int glo, int ghi) {\n"
       "  sb_i64 t = (sb_i64)blockIdx.x * 256 + threadIdx.x;\n";
  for (int i = 0; i < G; ++i) {
    const Group& g = p.groups[i];
    o << ga_group(i) << "    if (t < D * CG / 4) {\n      const int k = (int)t / (CG / 4), c = 4 * ((int)t % (CG / 4));\n"
      << "      const float* src = P + 4 * t;\n      sb_v4 v = sb_ld4(src);\n"
      << "      for (int z = 1; z < ns; z += 32) {\n        sb_v4 u[32];\n#pragma unroll\n"
      << "        for (int k = 0; k < 32; ++k) u[k] = sb_ld4(src + (sb_i64)min(z + k, ns - 1) * (D * CG));\n#pragma unroll\n"
      << "        for (int k = 0; k < 32; ++k)\n          if (z + k < ns) v += u[k];\n      }\n"
      << "      *(sb_v4*)(gW + (sb_i64)ktab[" << g.ktab_off << " + k] + c) = v;\n      return;\n    }\n    t -= D * CG / 4;\n"
      << "  }\n  P += (sb_i64)min((sb_i64)" << ga_max_splits(p, g) << ", max((sb_i64)1, cap * " << g.d << " / 64)) * "
      << (int64_t)g.D * g.C << "LL;\n";
  }
  o << "}\n";
  // adjoint state of the groups up to 128 wide; tpb: 64-column tiles per block
  o << head << "sobek_sp3_sbar(const float* __restrict__ M, int r0, int n, const float* __restrict__ W,"
       " const int* __restrict__ ktab, float* __restrict__ Sbar, sb_i64 s_ncap, int tpb) {\n"
       "  __shared__ __attribute__((aligned(128))) char lds[" << lds("sp3_lds_sbar", false) << "];\n  int b = blockIdx.x;\n";
  for (int i = 0; i < G; ++i) {
    const Group& g = p.groups[i];
    if (g.C > 128) continue;
    o << "  {\n    constexpr int D = " << g.D << ", DG = " << g.d << ", CG = " << g.C
      << ";\n    const int rt = (n * DG + 127) / 128, nt = (D + 63) / 64, nc = (nt + tpb - 1) / tpb;\n"
      << "    if (b < rt * nc) {\n      const int t0 = b / rt * tpb;\n      sp3_sbar<D, DG, CG, " << g.off
      << ">(lds, M, n * DG, W, ktab + " << g.ktab_off << ", Sbar + s_ncap * " << g.s_off
      << "LL, r0, b % rt * 128, t0, min(nt, t0 + tpb));\n      return;\n    }\n    b -= rt * nc;\n  }\n";
  }
  o << "}\n";
}

}  // namespace

std::string generate_split_source(const Plan& p) {
  std::ostringstream o;
  o << "\n// ---- split products, K=" << p.K << "\n#define K " << p.K << "\n#define NSH " << p.nsh << "\n#define CXI "
    << p.dim_in << "\n#define CXO " << p.dim_out << "\n"
    << kSplit;
  if (split_plan(p)) emit_split(o, p);
  return o.str();
}

}  // namespace sobek
