// The triangle limiter, as a pass of its own (k_limit_tri) and at the end of a stage (k_stage_tri:
// u + 0 (in + dt R(in))), on one block of four triangles, under every order of the block's
// waves.  One triangle after the other has a state u whose pressure is negative at a random node;
// the limiter has to act on it, and on no other, whatever the order.
#include <algorithm>
#include <cstdio>

#include "emulator.hpp"

#include "kernels_tri.hip"

using namespace frsg;

namespace {

int g_bad = 0;

// density 1, momentum 0, energy 2.5; u on triangle `low` with a first chaos mode of 3 in the energy
template <int PD>
void check(bool stage, int filter) {
  constexpr int M = 3, NQ = 4, E = kTriEPB;
  fr_sg_problem P{};
  P.equation = FRSG_EULER2D, P.element = FRSG_ELEM_TRI, P.fr_degree = PD, P.rdim = 2, P.gpc_order = 1, P.nq1d = 2;
  P.gamma = 1.4, P.n_tri = E, P.nx = P.ny = 1;
  for (int32_t& b : P.bc) b = FRSG_BC_OUTFLOW;
  P.filter = filter ? FRSG_FILTER_EXP : FRSG_FILTER_NONE, P.alpha = 0.0, P.s = 2.0;
  std::vector<double> xy;
  std::vector<int32_t> nbr(3 * E, -1), face(3 * E, -1);
  for (int e = 0; e < E; ++e) xy.insert(xy.end(), {0.0, 0.0, 1.0, 0.0, 0.0, 1.0});
  P.tri_xy = xy.data(), P.tri_nbr = nbr.data(), P.tri_nbr_face = face.data();
  HostTables T;
  TriTables R;
  std::string err;
  if (!build_host_tables(P, T, err) || !build_tri_tables(P, R, err)) {
    std::fprintf(stderr, "%s\n", err.c_str());
    std::exit(2);
  }
  tri_filter_tables(P, R, T);
  KParams K{};
  unsigned status = 0;
  double dt = 0.0;
  K.eq = P.equation, K.E = E, K.M = T.M, K.Nq = T.Nq, K.nsp = R.np, K.nfp = R.nfp, K.gamma = P.gamma;
  K.filter = P.filter, K.sensor = FRSG_SENSOR_ALWAYS, K.limiter = 1, K.status = &status, K.dt = &dt;
  K.tab.PhiT = T.PhiT.data(), K.tab.cmax = T.cmax.data(), K.tab.swts = T.swts.data(), K.tab.filt = T.filt.data();
  K.tab.PWT = T.PWT.data();
  K.tri_geo = R.geo.data(), K.tri_nbr = R.nbr.data(), K.tri_rows = R.rows.data();
  for (int i = 0; i < 4; ++i) K.bc[i] = P.bc[i];
  K.tri_Lf = R.Lf.data(), K.tri_V = R.V.data(), K.tri_Vinv = R.Vinv.data();
  if (T.M != M || T.Nq != NQ) std::exit(2);
  const int np = R.np, len = 4 * M * E * np;
  TriPost post;
  post.limit = 1, post.filter = filter;
  const std::vector<double> traces(4 * M * E * 3 * R.nfp, 1.0);  // of the neighbours: there are none
  for (int low = 0; low < E; ++low) {
    std::vector<int> order(TriShape<PD>::RG);
    for (size_t w = 0; w < order.size(); ++w) order[w] = (int)w;
    std::vector<double> first;
    do {
      std::vector<double> u(len, 0.0), in(len, 0.0);
      for (int e = 0; e < E; ++e)
        for (int j = 0; j < np; ++j) {
          auto at = [&](int s, int k) { return ((s * M + k) * E + e) * np + j; };
          u[at(0, 0)] = in[at(0, 0)] = 1.0, u[at(3, 0)] = in[at(3, 0)] = 2.5;
          if (e == low) u[at(3, 1)] = 3.0;
        }
      std::vector<unsigned char> flags(E, 9), filt(E, 9);
      post.flag_lim = flags.data(), post.flag_filt = filt.data();
      gridDim = dim3(1), blockIdx = dim3(0);
      emu::run_block(TriShape<PD>::NT, order, [&] {
        if (stage)
          k_stage_tri<PD, M, NQ>(K, in.data(), u.data(), u.data(), 1.0, 0.0, 0, traces.data(), nullptr, post, TriDt());
        else
          k_limit_tri<PD, M, NQ>(K, u.data(), u.data(), nullptr, post);
      });
      bool ok = status == 0;
      for (int e = 0; e < E; ++e) ok = ok && flags[e] == (e == low);
      if (first.empty()) first = u;
      ok = ok && first == u;
      if (!ok) {
        ++g_bad;
        std::printf("%s, p = %d, filter %d, triangle %d, waves", stage ? "stage" : "pass", PD, filter, low);
        for (int w : order) std::printf(" %d", w);
        std::printf(": limiter flags %d %d %d %d, state %s\n", flags[0], flags[1], flags[2], flags[3],
                    first == u ? "as in the first order" : "differs");
      }
    } while (std::next_permutation(order.begin(), order.end()));
  }
}

}  // namespace

int main() {
  for (int i = 0; i < 4; ++i) {
    check<1>(i & 1, i >> 1);
    check<2>(i & 1, i >> 1);
    check<3>(i & 1, i >> 1);
    check<4>(i & 1, i >> 1);
  }
  if (g_bad) return 1;
  std::printf("limiter decisions independent of the wave order\n");
  return 0;
}
