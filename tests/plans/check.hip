// Host-side check of the library's plans (no GPU): reads "variant op nx ny n" lines
// and, for each, prints the route that a call takes and "bad: ..." where a launch
// exceeds what HIP takes, a slice is empty, or a region that the route uses does not
// lie in the workspace apart from the others.
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/cgh.h"
#include "../../paper_1002_0916_amd/csrc/cgh_internal.h"
#include "../../paper_1002_0916_amd/csrc/contract.h"

using namespace cgh;

namespace {

char* const kBase = (char*)(1 << 20);
std::string bad;
struct Region {
  const char* name;
  int64_t begin, end;
};
std::vector<Region> regions;

void region(const char* name, const void* at, int64_t bytes) {
  if (bytes <= 0) return;
  const int64_t b = (const char*)at - kBase;
  regions.push_back({name, b, b + bytes});
}
void check_regions(const Plan& p) {
  for (size_t i = 0; i < regions.size(); ++i) {
    const Region& r = regions[i];
    if (r.begin < 0 || r.end > (int64_t)p.total || r.begin % 16)
      bad += std::string(" ") + r.name + " outside the workspace";
    for (size_t j = 0; j < i; ++j)
      if (r.begin < regions[j].end && regions[j].begin < r.end)
        bad += std::string(" ") + r.name + " over " + regions[j].name;
  }
}
void launch(const char* name, int64_t blocks, int threads) {
  if (blocks < 1 || blocks * threads > 0xffffffffll) bad += std::string(" launch ") + name;
}
int64_t up(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Pixels and threads of the tile shapes <MI, NJ, WM, KS>, as launched.
const int kRows[] = {128, 64, 64, 64, 32, 32, 64}, kCols[] = {128, 128, 64, 64, 64, 32, 64},
          kThreads[] = {256, 512, 256, 512, 512, 512, 64};

void forward(const Plan& p, const Workspace& w) {
  ContractFwd c{};
  const int64_t pixels = (int64_t)p.nx * p.ny;
  if (!plan_contract_fwd(p, w, c)) {
    printf("direct-form");
    if (p.variant != 1) return;
    region("ytab", w.ytab, (int64_t)p.groups * p.npad * kCompRows * 4);
    region("xtab", w.xtab, w.xtab ? (int64_t)p.fwd_gx * kWave * p.npad * 4 : 0);
    region("xrec", w.xrec, p.npad * kAxisRec * 4);
    return;
  }
  if (c.direct) {
    printf("one-launch");
    launch("direct", up(p.nx, 32) * up(p.ny, 32), 512);
    return;
  }
  const bool f32 = c.mode == kF32;
  const int side = c.shape == kOrdered && f32 ? 32 : 0;
  const int rows = side ? side : kRows[c.shape], cols = side ? side : kCols[c.shape];
  const int64_t tiles = up(p.nx, cols) * up(p.ny, rows);
  const int64_t points = c.chunk ? c.chunk : p.npad, unit = c.shape == kOrdered ? 16 : 64;
  printf("tiles shape %d slices %d passes %lld", c.shape, c.slices, (long long)up(p.npad, points));
  launch("tiles", tiles * c.slices, kThreads[c.shape]);
  launch("tables", points / 16, 256);
  if (c.slices > 1 || c.chunk) launch("sum", up(pixels, 256), 256);
  if ((c.slices - 1) * up(points / unit, c.slices) >= points / unit) bad += " empty slice";
  region("yq", c.yq, points * c.rows_y * (f32 ? 8 : 4));
  region("xq", c.xq, c.xtab ? points * c.cols_x * (f32 ? 8 : 4) : 0);
  region("rec", c.rec, c.xtab ? 0 : points * 20);
  region("amp", c.amp, p.npad * 4);
  region("amax", c.amax, c.amax ? kWave * 4 : 0);
  const int64_t planes = (c.slices > 1 ? c.slices : 0) + (c.chunk ? 1 : 0);
  region("planes", c.planes, planes * pixels * 4);
  if (c.rows_y < p.ny || c.cols_x < p.nx) bad += " tables too small";
}

void backward(const Plan& p, const Workspace& w) {
  ContractAdj c{};
  if (!plan_contract_adj(p, w, c)) {
    printf("direct-form");
    return;
  }
  const int tile = c.direct ? 32 : 128;
  printf("%s groups %d + %d slices %d + %d", c.direct ? "one-launch" : "tiles", c.groups_u,
         c.groups_p, c.slices_u, c.slices_p);
  launch("tiles", up(p.npad, tile) * c.planes, c.direct ? 512 : 256);
  region("partial", c.partial, (int64_t)c.planes * p.npad * 16);
  if (c.direct) return;
  const int64_t stages[2] = {up(p.ny, 32), up(p.nx, 32)};
  if ((c.slices_u - 1) * up(stages[0], c.slices_u) >= stages[0] ||
      (c.slices_p - 1) * up(stages[1], c.slices_p) >= stages[1])
    bad += " empty slice";
  region("gmax", c.gmax, c.gblocks * 4);
  const bool phases = c.mode == kHalfF16x3 || c.mode == kF32;
  auto bytes = [&](int64_t size) {
    return phases ? up(size, 4) * p.npad * 16 : 2 * up(size, 8) * p.npad * 16;
  };
  region("yq", c.yq, c.tab ? bytes(p.ny) : 0);
  region("xq", c.xq, c.tab ? bytes(p.nx) : 0);
  launch("tables", c.gblocks + up(p.npad, 256) * (c.tab ? up(p.ny, 64) + up(p.nx, 64) : 0) + 1, 256);
}

void forward64(const Plan& p, const Workspace& w) {
  if (p.f64_slices == 0) {
    printf("direct-form");
    region("rec64", w.rec64, p.npad * 32);
    return;
  }
  const int64_t tiles = up(p.nx, 64) * up(p.ny, 64), pixels = (int64_t)p.nx * p.ny;
  printf("tiles slices %d passes %lld", p.f64_slices, (long long)up(p.npad, p.f64_chunk));
  launch("tiles", tiles * p.f64_slices, 256);
  region("rec64", w.rec64, p.npad * 32);
  region("tab64", w.tab64, (int64_t)p.f64_chunk * 16 * (up(p.ny, 64) + up(p.nx, 64)) * 64);
  region("planes64", w.planes64, p.f64_slices > 1 ? p.f64_slices * pixels * 8 : 0);
  if ((p.f64_slices - 1) * up(p.f64_chunk / 64, p.f64_slices) >= p.f64_chunk / 64) bad += " empty slice";
}

}  // namespace

int main() {
  int variant, op, nx, ny, table;
  long long n;
  while (scanf("%d %d %d %d %lld %d", &variant, &op, &nx, &ny, &n, &table) == 6) {
    bad.clear();
    regions.clear();
    const Plan p = make_plan(n, nx, ny, variant, op, table != 0);
    const Workspace w = carve(p, kBase);
    if (op == CGH_OP_FORWARD_F64)
      forward64(p, w);
    else if (op == CGH_OP_BACKWARD)
      backward(p, w);
    else
      forward(p, w);
    check_regions(p);
    printf(" bytes %lld%s%s\n", (long long)p.total, bad.empty() ? "" : " bad:", bad.c_str());
  }
  return 0;
}
