// Generator of the moment-form adjoint kernels (device/adjoint.hip): slot groups, the coupling of each
// step as immediates, and the step sequence.
#include <algorithm>
#include <array>
#include <sstream>

#include "adjoint.h"
#include "gen.h"

namespace sobek {

namespace {
const char* kAdjoint =
#include "adjoint_embed.inc"
    ;
}  // namespace

// Slots of a group: a wave forms a slot, and the phi Y planes (12 KiB a step) and two Rb buffers
// (7.5 KiB a slot) share the 160 KiB of LDS.  Six leave a wave's state in its 256 registers (eight spill
// 40 of them: 17 % slower on 64x0e+64x1o+64x1e+64x2e).  An irrep of more than six slots is a group alone.
namespace {
std::vector<AdjGroup> pack_groups(const Plan& p, int block) {
  const int most = 6;
  std::vector<AdjJob> jobs;
  std::vector<int> used(p.in.size(), 0);
  for (auto& q : p.paths) used[q.i_in] = 1;
  for (int a = 0; a < (int)p.in.size(); ++a)
    for (int u0 = 0; used[a] && u0 < p.in[a].mul; u0 += block) jobs.push_back({a, u0, 0});
  auto width = [&](const AdjJob& j) { return std::min(block, p.in[j.a].mul - j.U0) / 16; };
  auto slots = [&](const AdjJob& j) { return 2 * p.in[j.a].l + 1; };
  std::stable_sort(jobs.begin(), jobs.end(), [&](const AdjJob& x, const AdjJob& y) { return slots(x) > slots(y); });
  std::vector<AdjGroup> gs;
  for (const AdjJob& j : jobs) {
    int at = -1;   // the fullest group of this width with room
    for (int i = 0; i < (int)gs.size(); ++i)
      if (gs[i].UT == width(j) && gs[i].slots + slots(j) <= most && (at < 0 || gs[i].slots > gs[at].slots)) at = i;
    if (at < 0) {
      at = (int)gs.size();
      gs.push_back(AdjGroup());
      gs[at].UT = width(j);
    }
    AdjJob k = j;
    k.slot = gs[at].slots;
    gs[at].jobs.push_back(k);
    gs[at].slots += slots(j);
  }
  return gs;
}
}  // namespace

// Channel blocks of 64, or narrower where that packs the slots into fewer steps (each costs a barrier
// and the latency of its products whatever it holds).  A group's steps over m_y are written out, its
// channel tiles are a loop, and the compiler moves loads ahead through what is written out: 16 to 40 steps
// spill up to 81 registers, the 88 of 128x0e+64x1o+64x2e+64x3o in blocks of 16 (eleven groups of one tile)
// 6,970, and its 96 steps in blocks of 64, 24 of them written out, 57.  Backward of 700 receivers, degree 64:
// 3.88 ms and 1.02 ms (per-edge kernels 1.34 ms).  A narrower block is taken up to kWritten only.
std::vector<AdjGroup> adjoint_groups(const Plan& p) {
  const int kWritten = 48, NC = (p.nsh + 1) / 2;
  std::vector<AdjGroup> best;
  int fewest = 0;
  for (int block = 64; block >= 16; block /= 2) {
    std::vector<AdjGroup> gs = pack_groups(p, block);
    int steps = 0;
    for (auto& g : gs) steps += g.UT;
    if (best.empty() || (steps < fewest && (int)gs.size() * NC <= kWritten)) {
      best = gs;
      fewest = steps;
    }
  }
  return best;
}

// Edge time by the per-edge kernel (waves own channel slices, coupling applied to every edge) and this
// one, mean degree 8 / 64 on radius graphs (us):
//   64x0e+64x1o+64x1e+64x2e lmax 3, 3,000 receivers     64 steps   999 / 2,390   789 / 1,814
//   64x0e+32x1o+32x2e+32x3o lmax 3, 6,000 receivers     48 steps 1,627 / 3,718 1,528 / 3,078
//   64x0e+64x1o+64x2e lmax 2, 6,000 receivers           30 steps   930 / 2,046   901 / 1,906
//   128x0e+64x1o lmax 1, 20,000 receivers                8 steps   493 / 1,420   921 / 2,287
// A receiver's first loads, Y and the outputs are a fixed cost that a few steps do not carry, and at
// lmax 1 the coupling that is saved is small.  The line lies at the least that was level; nothing between 8
// and 30 steps was measured.
//
// The choice is the plan's: the order of a kept adjoint state follows from it.  A CU holds one block of this
// kernel and three of the per-edge one, so 513 to 768 receivers are three turns against one, and with two passes
// against one launch few edges do not pay.  Where that shows is a double backward on a kept adjoint state (us,
// per-edge and this; the split products make up for it where Sbar is formed in the call):
//   edge vectors alone, 700 receivers, degree 8   64x0e+64x1o+64x2e 102 / 113, 128x0e+64x1o+64x2e 122 / 129;
//                                                 at 400 receivers 93 / 78, 1,000 196 / 148 (the first plan)
//   x, edge vectors, phi, 64x0e+32x1o+32x2e+32x3o degree 8: 400 receivers 223 / 240, 1,500 731 / 768; degree 28:
//                                                 0.57 to 0.82 of the per-edge time
// Its backward gained more each time: the two together take 0.28 to 0.98 of the time with per-edge kernels and
// the older products (seven plans, 60 to 4,000 receivers, degree 2 to 100).  Per-edge kernels that read the
// order of this one were 1.05 to 1.48 times slower than it there (four-byte LDS stores in their staging), and
// the per-edge order for such graphs would cost the other cotangents up to 1.6 times.
bool adjoint_plan(const Plan& p) {
  if (p.mode != 0 || p.K != 16 || p.lmax < 2 || p.paths.empty() || !p.vec4) return false;
  for (auto& q : p.paths)
    if (p.in[q.i_in].mul % 16) return false;
  for (auto& r : p.in)
    if (r.off % 4) return false;
  int steps = 0;
  for (auto& g : adjoint_groups(p)) steps += g.UT * ((p.nsh + 1) / 2);
  return steps >= 30;
}

namespace {

// What wave w forms in step c: the adjoint-state entries (path, channel block, m_o) it needs and the
// terms (entry, coefficient) of its values.  A wave takes a slot; few slots go by (slot, m_y).
struct Step {
  std::vector<std::array<int, 3>> need;
  struct Val { int slot, y; std::vector<std::pair<int, double>> terms; };
  std::vector<Val> vals;
};

Step adj_step(const Plan& p, const AdjGroup& g, int c, int w) {
  Step s;
  auto entry = [&](int t, int blk, int mo) {
    const std::array<int, 3> e{t, blk, mo};
    for (size_t i = 0; i < s.need.size(); ++i)
      if (s.need[i] == e) return (int)i;
    s.need.push_back(e);
    return (int)s.need.size() - 1;
  };
  const int ny = std::min(2, p.nsh - 2 * c);
  const bool single = g.slots * ny <= 8;
  for (const AdjJob& jb : g.jobs)
    for (int mi = 0; mi < 2 * p.in[jb.a].l + 1; ++mi)
      for (int y = 0; y < ny; ++y) {
        const int slot = jb.slot + mi;
        if ((single ? slot * ny + y : slot) != w) continue;
        Step::Val v{slot, y, {}};
        for (size_t t = 0; t < p.paths.size(); ++t) {
          const Path& q = p.paths[t];
          if (q.i_in != jb.a) continue;
          const PathTerms pt = path_terms(q);
          for (size_t k = 0; k < pt.pairs.size(); ++k)
            if (pt.pairs[k].first == mi)
              for (auto& tm : pt.terms[k])
                if (q.l_sh * q.l_sh + tm.my == 2 * c + y)
                  v.terms.push_back({entry((int)t, jb.U0, pt.pairs[k].second), tm.c});
        }
        s.vals.push_back(v);
      }
  return s;
}

// the adjoint state of step c on channel tile `ut` into sv
void emit_load(std::ostringstream& o, const Plan& p, const AdjGroup& g, int c, const char* ut, const std::string& ind) {
  for (int w = 0; w < 8; ++w) {
    const Step s = adj_step(p, g, c, w);
    if (s.need.empty()) continue;
    o << ind << "if (w == " << w << ") {\n";
    for (size_t i = 0; i < s.need.size(); ++i) {
      const Path& q = p.paths[s.need[i][0]];
      const Group& og = p.groups[q.group];
      o << ind << "  sv[" << i << "] = sba_ld4(Sb + (sb_ncap * " << og.s_off << "LL + row * " << (int64_t)og.d * og.D << "LL + "
        << (int64_t)s.need[i][2] * og.D + q.koff + 16 * s.need[i][1] << ") + 256 * " << ut << ", lo);\n";
    }
    o << ind << "}\n";
  }
}

// Rb of step c from sv, into the buffer at Bn
void emit_produce(std::ostringstream& o, const Plan& p, const AdjGroup& g, int c, const std::string& ind) {
  const int SL = g.slots, PL = 2 * SL * 640;
  for (int w = 0; w < 8; ++w) {
    const Step s = adj_step(p, g, c, w);
    if (s.vals.empty()) continue;
    o << ind << "if (w == " << w << ") {\n";
    for (auto& v : s.vals) {
      o << ind << "  sba_put4(Bn + " << (v.y * SL + v.slot) * 640 << ", " << PL << ", ";
      for (size_t i = 0; i < v.terms.size(); ++i)
        o << (i ? " + " : "") << fl(v.terms[i].second) << "*sv[" << v.terms[i].first << "]";
      o << (v.terms.empty() ? "(sbm_f4){0.f, 0.f, 0.f, 0.f}" : "") << ");\n";
    }
    o << ind << "}\n";
  }
}

std::vector<int> group_cols(const Plan& p, const AdjGroup& g) {
  std::vector<int> cols;
  for (auto& jb : g.jobs)
    for (int m = 0; m < 2 * p.in[jb.a].l + 1; ++m) cols.push_back(p.in[jb.a].off + m * p.in[jb.a].mul + jb.U0);
  return cols;
}

// sender-row slices of a group's channel tile: slot pair s in lanes g >> 1, channels 8 (g & 1) .. + 7
void emit_xload(std::ostringstream& o, const Plan& p, const AdjGroup& g, const char* ut, const std::string& ind) {
  const std::vector<int> cols = group_cols(p, g);
  for (int s = 0; 2 * s < g.slots; ++s) {
    const int c0 = cols[2 * s], c1 = 2 * s + 1 < g.slots ? cols[2 * s + 1] : c0;
    o << ind << "{\n" << ind << "  const float* xs = xr + (g >> 1 ? " << c1 << " : " << c0 << ") + 16 * " << ut << ";\n"
      << ind << "  xv[" << 2 * s << "] = *(const sbm_f4*)xs;\n" << ind << "  xv[" << 2 * s + 1 << "] = *(const sbm_f4*)(xs + 4);\n"
      << ind << "}\n";
  }
}

}  // namespace

std::string generate_adjoint_source(const Plan& p) {
  std::ostringstream o;
  o.precision(17);
  o << kAdjoint;
  const std::vector<AdjGroup> groups = adjoint_groups(p);
  const int NC = (p.nsh + 1) / 2, NG = (int)groups.size();
  int slmax = 0, nsv = 1;
  for (auto& g : groups) {
    slmax = std::max(slmax, g.slots);
    for (int c = 0; c < NC; ++c)
      for (int w = 0; w < 8; ++w) nsv = std::max(nsv, (int)adj_step(p, g, c, w).need.size());
  }
  const int bufb = std::max(3 * 2 * slmax * 640, 4096);   // the finish passes 8 KiB through the buffers
  const int phib = 4 * NC * 3 * 1024;
  o << "template <bool DB>\nSB_DEV void sba_body(char* lds, const int* __restrict__ rowptr, const int* __restrict__ sender,"
       " const float* __restrict__ evec, const float* __restrict__ phi, const float* __restrict__ x,"
       " const float* __restrict__ Sb, const float* __restrict__ evdot, const float* __restrict__ phidot,"
       " float* __restrict__ gphi, float* __restrict__ gevec, float* __restrict__ contrib, int r0, int e0, int flags,"
       " sb_i64 sb_ncap, int sb_r0, int win0, int win1, int accum, int accx) {\n"
       "  const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, g = lane >> 4;\n"
       "  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), mt = w >> 1, hf = w & 1;\n"
       "  const int po = (g >> 1) * 320 + j * 16 + (g & 1) * 8;   // Rb of channel j, q = 4 g .. 4 g + 3\n"
       "  const int il = blockIdx.x;\n"
       "  const int wb = max(rowptr[r0 + il], win0), we = min(rowptr[r0 + il + 1], win1);\n"
       "  char* sR = lds + " << phib << ";\n"
       "  float* sYw = (float*)(lds + " << phib + 2 * bufb << ") + mt * (NSH * 16);\n"
       "  const sb_i64 row = sb_r0 + il;\n"
       "  int buf = 0;\n  const unsigned lo = 64u * j + 16u * g;   // channel j, q = 4 g of an adjoint-state row\n  sbm_f4 sv[" << nsv << "];\n  sbm_f4 xv[" << 2 * ((slmax + 1) / 2) << "];\n"
       "  for (int rb = wb + 64 * (int)blockIdx.y; rb < we; rb += 64 * (int)gridDim.y) {\n"
       "    const int ebase = rb + 16 * mt;\n"
       "    const bool act = ebase < we, valid = ebase + j < we;\n"
       "    const sb_i64 ec = min(ebase + j, we - 1);\n"
       "    const float* xr = x + (sb_i64)sender[ec] * CXI + 8 * (g & 1);\n";
  emit_load(o, p, groups[0], 0, "0", "    ");
  emit_xload(o, p, groups[0], "0", "    ");
  o << "    const float vx = evec[3 * ec], vy = evec[3 * ec + 1], vz = evec[3 * ec + 2];\n"
       "    const float rinv = __builtin_amdgcn_rsqf(vx * vx + vy * vy + vz * vz);\n"
       "    const float ux = vx * rinv, uy = vy * rinv, uz = vz * rinv;\n"
       "    float dx = 0.f, dy = 0.f, dz = 0.f;\n"
       "    if (DB && (flags & 4)) { dx = evdot[3 * ec]; dy = evdot[3 * ec + 1]; dz = evdot[3 * ec + 2]; }\n"
       "    sbm_b8* sPhi = (sbm_b8*)lds + mt * " << NC * 3 * 64 << " + lane;\n"
       "    if (act) {\n"
       "      float Y[NSH], Yd[NSH] = {};\n      sb_sh_eval_L" << p.lmax << "(ux, uy, uz, Y);\n"
       "      if (DB) sb_sh_jvp_L" << p.lmax << "(ux, uy, uz, rinv, dx, dy, dz, Y, Yd);\n"
       "      if (g == 0 && hf == 0) {\n#pragma unroll\n        for (int m = 0; m < NSH; ++m) {\n"
       "          sYw[m * 16 + j] = DB ? Yd[m] : Y[m];\n        }\n      }\n"
       // planes of phi Y (or its tangent): k = 16 (g >> 1) + 8 (g & 1) + i is (m_y 2 c + (g >> 1), q 8 (g & 1) + i)
       "      float ph[8], phd[8];\n      const float* pp = phi + ec * K + 8 * (g & 1);\n"
       "      const float* pd = (DB && (flags & 1)) ? phidot + ec * K + 8 * (g & 1) : pp;\n"
       "#pragma unroll\n      for (int k = 0; k < 8; ++k) { ph[k] = pp[k]; phd[k] = pd[k]; }\n"
       "#pragma unroll\n      for (int c = 0; c < SBA_NC; ++c) {\n        if ((c & 1) == hf) {\n"
       "          const float y0 = Y[2 * c], y1 = 2 * c + 1 < NSH ? Y[2 * c + 1 < NSH ? 2 * c + 1 : 0] : 0.f;\n"
       "          const float d0 = DB ? Yd[2 * c] : 0.f, d1 = DB && 2 * c + 1 < NSH ? Yd[2 * c + 1 < NSH ? 2 * c + 1 : 0] : 0.f;\n"
       "          const float yv = g >> 1 ? y1 : y0, yd = g >> 1 ? d1 : d0;\n          float v[8];\n"
       "#pragma unroll\n          for (int k = 0; k < 8; ++k)\n"
       "            v[k] = !DB ? ph[k] * yv : ((flags & 4) ? ph[k] * yd : 0.f) + ((flags & 1) ? phd[k] * yv : 0.f);\n"
       "          const sbm_p3 s = sbm_split(v);\n"
       "#pragma unroll\n          for (int q = 0; q < 3; ++q) sPhi[(c * 3 + q) * 64] = s.p[q];\n        }\n      }\n    }\n"
       "    sbm_f4 T[SBA_NC];\n#pragma unroll\n    for (int c = 0; c < SBA_NC; ++c) T[c] = (sbm_f4){0.f, 0.f, 0.f, 0.f};\n";
  for (int gi = 0; gi < NG; ++gi) {
    const AdjGroup& g = groups[gi];
    const AdjGroup& gn = groups[(gi + 1) % NG];
    const int SL = g.slots, SH = (SL + 1) / 2;
    const std::vector<int> cols = group_cols(p, g);
    o << "    for (int ut = 0; ut < " << g.UT << "; ++ut) {  // " << SL << " slots\n"
      << "      const bool same = ut + 1 < " << g.UT << ";\n"
      << "      sbm_p3 xp[" << SH << "];\n      sbm_f4 xacc[" << SH << "];\n"
      << "#pragma unroll\n      for (int s = 0; s < " << SH << "; ++s) {\n        xacc[s] = (sbm_f4){0.f, 0.f, 0.f, 0.f};\n"
      << "        float v[8] = {xv[2 * s][0], xv[2 * s][1], xv[2 * s][2], xv[2 * s][3], xv[2 * s + 1][0], xv[2 * s + 1][1],"
         " xv[2 * s + 1][2], xv[2 * s + 1][3]};\n";
    if (SL % 2)
      o << "        if (s == " << SH - 1 << ") {\n#pragma unroll\n          for (int k = 0; k < 8; ++k) v[k] = g >> 1 ? 0.f : v[k];\n        }\n";
    o << "        xp[s] = sbm_split(v);\n      }\n";
    for (int c = 0; c < NC; ++c) {
      const int ny = std::min(2, p.nsh - 2 * c);
      o << "      {  // m_y " << 2 * c << (ny > 1 ? ", " + std::to_string(2 * c + 1) : std::string()) << "\n        char* B = sR + buf * "
        << bufb << ";\n        char* Bn = B + po;\n";
      emit_produce(o, p, g, c, "        ");
      // the next step's adjoint state, and after the last step the next channel tile's sender rows
      if (c + 1 < NC) {
        emit_load(o, p, g, c + 1, "ut", "        ");
      } else {
        o << "        if (same) {\n";
        emit_load(o, p, g, 0, "(ut + 1)", "          ");
        emit_xload(o, p, g, "(ut + 1)", "          ");
        if (gi + 1 < NG) {
          o << "        } else {\n";
          emit_load(o, p, gn, 0, "0", "          ");
          emit_xload(o, p, gn, "0", "          ");
        }
        o << "        }\n";
      }
      o << "        __syncthreads();\n"
        << "        if (act) sba_step<" << SL << ", " << ny << ">(B, j, g, hf, contrib != nullptr, sPhi + " << c * 3 * 64
        << ", xp, xacc, T[" << c << "]);\n        buf ^= 1;\n      }\n";
    }
    o << "      if (valid && act && contrib) {\n        float* cr = contrib + (sb_i64)(ebase + j - e0) * CXI + 16 * ut + 4 * g;\n";
    for (int s = 0; s < SH; ++s) {
      const bool tail = SH + s >= SL;   // the second half of an odd group is one shorter
      o << "        " << (tail ? "if (!hf) " : "") << "{\n          sbm_f4* q = (sbm_f4*)(cr + " << (tail ? std::to_string(cols[s]) : "(hf ? " + std::to_string(cols[SH + s]) + " : " + std::to_string(cols[s]) + ")")
        << ");\n          *q = accx ? *q + xacc[" << s << "] : xacc[" << s << "];\n        }\n";
    }
    o << "      }\n    }\n";
  }
  if (!p.dead_in.empty()) {
    o << "    if (valid && act && contrib && !accx && !hf) {\n      float* cr = contrib + (sb_i64)(ebase + j - e0) * CXI;\n";
    for (int a : p.dead_in)
      o << "      for (int t = g; t < " << p.in[a].dim() << "; t += 4) cr[" << p.in[a].off << " + t] = 0.f;\n";
    o << "    }\n";
  }
  o << "    __syncthreads();\n"
       "    sba_finish<DB>(T, sYw, (float*)sR + mt * 512, lane, hf, act, ec, valid, ux, uy, uz, rinv, dx, dy, dz, phi, phidot,"
       " flags, gphi, gevec, accum);\n"
       "  }\n}\n";
  for (int db = 0; db < 2; ++db)
    o << "extern \"C\" __global__ __launch_bounds__(SBA_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void "
      << (db ? "sobek_adj_dE" : "sobek_adj_E")
      << "(const int* __restrict__ rowptr, const int* __restrict__ sender, const float* __restrict__ evec,"
         " const float* __restrict__ phi, const float* __restrict__ x, const float* __restrict__ Sb,"
         " const float* __restrict__ evdot, const float* __restrict__ phidot, float* __restrict__ gphi,"
         " float* __restrict__ gevec, float* __restrict__ contrib, int r0, int e0, int flags, sb_i64 sb_ncap, int sb_r0,"
         " int win0, int win1, int accum, int accx) {\n"
      << "  __shared__ __attribute__((aligned(128))) char lds[" << phib + 2 * bufb + 4 * p.nsh * 64 << "];\n"
      << "  sba_body<" << (db ? "true" : "false")
      << ">(lds, rowptr, sender, evec, phi, x, Sb, evdot, phidot, gphi, gevec, contrib, r0, e0, flags, sb_ncap, sb_r0,"
         " win0, win1, accum, accx);\n}\n";
  return o.str();
}

}  // namespace sobek
