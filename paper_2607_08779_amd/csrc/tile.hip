// Matmul for middle token counts (49 <= M, as long as small tiles pay): which tile runs, and
// in how many slices of K (tile_kernels.h describes the kernel).
#include <algorithm>

#include "stream_kernels.h"

namespace ssq {
namespace tile {
hipError_t launch_q2(const stream::StreamArgs& a, int kind, int form);
hipError_t launch_q3(const stream::StreamArgs& a, int kind, int form);
hipError_t launch_q4(const stream::StreamArgs& a, int kind, int form);
}  // namespace tile

namespace {

constexpr int kCUs = 256;
constexpr int kMaxSlices = 6;

// Time of a launch, us: rounds of as many workgroups as run at once, each `start` and `step`
// for every 64 k of its busiest wavefront (the 32 x 32 tile runs two workgroups a CU, which
// share its memory pipe: `busy` more a step when all CUs are busy), and `meet` if slices of K
// meet in the workspace.  Least squares over 62 sizes, W4 g32 signed, 33 to 1024 tokens,
// 256 to 28672 rows: 6 to 9 % rms (32 x 32: 18 %); the tile it picks is within a few percent
// of the fastest one in most.
struct Form {
  int bm, bn, waves, unit_blocks, at_once;
  float start, step, busy, meet;
};
constexpr Form kForms[] = {{32, 32, 8, 4, 512, 3.9f, 2.36f, 2.61f, 0.5f}, {64, 32, 4, 8, 256, 2.7f, 2.29f, 0.0f, 3.3f},
                           {96, 32, 4, 8, 256, 3.1f, 2.86f, 0.0f, 3.8f},  {64, 64, 4, 8, 256, 4.3f, 3.44f, 0.0f, 3.8f},
                           {96, 64, 4, 8, 256, 5.4f, 4.14f, 0.0f, 4.9f},  {128, 64, 4, 4, 256, 5.3f, 5.70f, 0.0f, 6.0f}};

}  // namespace

TilePlan tile_plan(int64_t M, int64_t N, int64_t K, int64_t room) {
  TilePlan best{0, 1, 0.0f};
  for (int f = 0; f < (int)(sizeof(kForms) / sizeof(kForms[0])); ++f) {
    const Form& t = kForms[f];
    const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const int64_t units = (K / 32 + t.unit_blocks - 1) / t.unit_blocks;
    for (int s = 1; s <= kMaxSlices; ++s) {
      const int64_t items = tiles * s;
      if (s > 1 && (items > 300 || K / 32 < 8 * s || kSplitCounterBytes + items * t.bm * t.bn * 4 > room)) break;
      const int64_t rounds = (items + t.at_once - 1) / t.at_once, per = (units + s - 1) / s;
      const float steps = (float)((per + t.waves - 1) / t.waves) * (float)t.unit_blocks / 8.0f;
      // several rounds come out about a tenth longer: 459 tokens on 4480x1024 20.6 for 17.9
      const float us = (rounds > 1 ? 1.1f : 1.0f) * (float)rounds * (t.start + (t.step + t.busy * std::min(1.0f, (float)items / kCUs)) * steps) +
                       (s > 1 ? t.meet : 0.0f);
      if (best.us == 0.0f || us < best.us) best = TilePlan{f, s, us};
    }
  }
  return best;
}

Route tile_route(const TilePlan& plan) {
  return Route{kRouteTile, kForms[plan.form].bm, kForms[plan.form].bn, plan.slices};
}

hipError_t launch_tile_bf16(const TilePlan& plan, const uint16_t* x, int64_t M, const uint8_t* codes,
                            const uint16_t* scales, GroupMeta meta, int64_t N, int64_t K, int group, int q, uint16_t* y,
                            void* workspace, hipStream_t stream) {
  stream::StreamArgs a;
  a.x = x; a.M = M; a.codes = codes; a.scales = scales; a.meta = meta.ptr;
  a.N = N; a.K = K;
  a.gshift = group == 32 ? 0 : group == 64 ? 1 : 2;
  a.slices = plan.slices;
  a.y = y;
  a.partials = plan.slices > 1 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + kSplitCounterBytes) : nullptr;
  a.counters = static_cast<unsigned int*>(workspace);
  a.stream = stream;
  switch (q) {
    case 2: return tile::launch_q2(a, meta.kind, plan.form);
    case 3: return tile::launch_q3(a, meta.kind, plan.form);
    default: return tile::launch_q4(a, meta.kind, plan.form);
  }
}

}  // namespace ssq
