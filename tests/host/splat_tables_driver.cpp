// Test driver for the tables of the splat's gather form (host-only plan code): builds
// them for the detector named on the command line (nu nv dv/du n_theta ds/du n_s) and
// checks, by visiting every block, row and column, what the kernel relies on: every
// pixel read lies in the copy, a lane's columns meet each image pixel of the block's
// rows exactly once, a set's positions stay within one bin of a column's lower end,
// and sets and blocks hold an even number of rows.  Prints the angles per group.
#include <cstdio>
#include <cstdlib>
#include <set>

#include "plan_host.h"

#define CHECK(c)                                          \
  do {                                                    \
    if (!(c)) {                                           \
      std::printf("line %d: %s\n", __LINE__, #c);         \
      return 1;                                           \
    }                                                     \
  } while (0)

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  dc_grid g{};
  g.nu = std::atoi(argv[1]);
  g.nv = std::atoi(argv[2]);
  g.du = 1.0;
  g.dv = std::atof(argv[3]);
  g.n_theta = std::atoi(argv[4]);
  g.ds = std::atof(argv[5]);
  g.n_s = std::atoi(argv[6]);
  g.nx = g.ny = g.nz = 2;
  g.vx = g.vy = g.vz = 1.0;
  dc_view v{{750, 0, 0}, {-450, 0, 0}, {0, 1, 0}, {0, 0, 1}, {0, 1, 0}};
  const int first[2] = {0, 1};
  dc::HostPlan p;
  std::string err;
  if (dc::plan_tables(&g, &v, 1, first, 1, dc::KernelShape(), &p, &err) != DC_OK) {
    std::printf("%s\n", err.c_str());
    return 1;
  }
  int angles = 0;
  for (size_t a = 0; a < (p.shear_g ? p.shear_groups.size() : 0); ++a) {
    const dc::ShearGroup& gr = p.shear_groups[a];
    const dc::ShearRow* rows = &p.shear_rows[a * dc::kShearPad];
    const int n = gr.col ? g.nv : g.nu, walk = gr.col ? g.nu : g.nv, pitch = n + dc::kShearPad;
    CHECK(gr.k0 == angles && gr.kn >= 1 && gr.kn <= p.shear_g);
    angles += gr.kn;
    CHECK(gr.rows % 2 == 0 && gr.n_first % 2 == 0 && gr.rows <= dc::kShearPad && gr.rows >= 2);
    CHECK(gr.blocks * gr.rows == p.shear_pad_rows[gr.col] && gr.blocks * gr.rows >= walk);
    const int span = n + std::abs(gr.shift), left = std::min(gr.shift, 0);
    const long long last = (long long)p.shear_pad_rows[gr.col] * pitch + dc::kShearPad;
    std::set<long long> seen;
    for (int i = 0; i < gr.rows; ++i) {
      const int off = i < dc::kShearAhead ? gr.first[i] : rows[i - dc::kShearAhead].ahead;
      CHECK(off % 16 == 0 && rows[i].ahead % 16 == 0);
      const int w = (int)std::floor((off / 16 + 0.5 * pitch) / pitch), sigma = w * pitch - off / 16;
      CHECK(w >= 0 && w < gr.rows);
      for (int q = 0; q < gr.kn; ++q) {
        const double rest = w * gr.b[q] - sigma * gr.a[q] - (gr.base[q] - p.ang[3 * (gr.k0 + q) + 2]);
        CHECK(std::fabs(rest - rows[i].rest[q]) < 1e-6);
        CHECK(std::fabs(gr.alpha[q] * rows[i].rho + gr.delta[q] * rows[i].wc - rest) < 1e-6);
        const double lo = gr.lo[i < gr.n_first ? 0 : 1][q];
        CHECK(rest - lo > -1e-6 && rest - lo < 1.0);
      }
      for (int blk = 0; blk < gr.blocks; blk += std::max(1, gr.blocks - 1))
        for (int c = 0; c < span; ++c) {
          const int lp = c + left, l = lp - sigma;
          const long long rec = (long long)blk * gr.rows * pitch + dc::kShearPad + lp + off / 16;
          const long long again = (long long)blk * gr.rows * pitch + dc::kShearPad + lp + rows[i].ahead / 16;
          CHECK(rec >= 0 && rec < last && again >= 0 && again < last);
          CHECK(l >= -dc::kShearPad && l < n + dc::kShearPad);
          if (blk == 0 && l >= 0 && l < n) CHECK(seen.insert((long long)w * n + l).second);
        }
    }
    CHECK((int)seen.size() == gr.rows * n);
  }
  CHECK(p.shear_g == 0 || angles == g.n_theta);
  std::printf("%d\n", p.shear_g);
  return 0;
}
