// Matmul for small token counts (3 <= M <= 80): which streaming kernel runs, and how the
// matrix is cut (stream_kernels.h describes the kernels).
#include <algorithm>

#include "stream_kernels.h"

namespace ssq {
namespace stream {
hipError_t launch_rounded_q2(const StreamArgs& a, int kind, int tok, int rt);
hipError_t launch_rounded_q3(const StreamArgs& a, int kind, int tok, int rt);
hipError_t launch_rounded_q4(const StreamArgs& a, int kind, int tok, int rt);
hipError_t launch_exact(const StreamArgs& a, int q, int kind, int tok, int rt);
}  // namespace stream

namespace {

constexpr int kCUs = 256;
constexpr int kMaxSlices = 8;

// ---------------------------------------------------------------------------
// Row tiles per workgroup and slices of K.  A launch takes rounds of 256 workgroups (one per
// CU); a round takes about 3 us, plus 0.5 per row tile, plus the time below for every 8
// units of K (2048 k: one unit per wavefront), and meeting in the workspace 1.9 us.  The
// times are measured with all CUs busy (W4 g32 signed, 4096 RT rows, K = 4096 against 8192,
// us); fewer workgroups share the memory system and take down to 70 % of them.  Most
// choices come out as the smallest RT that makes one round, unsliced: 16 tokens on
// 4096x4096 5.9 us (RT 1; 7.1 with 2), on 14336x4096 12.2 (RT 4, 224 workgroups; 13.3 with
// 2 in two rounds), on 8192x28672 34.9 (RT 4, two slices; 38.7 with RT 2 unsliced).
// ---------------------------------------------------------------------------
struct Form {
  int tok;
  float us[5];          // per RT 1..5, 0: no such kernel
};
constexpr Form kExactForms[] = {{8, {1.40f, 2.68f, 3.66f, 4.92f, 0.0f}}, {16, {1.70f, 3.14f, 4.26f, 5.50f, 0.0f}}};
constexpr Form kRoundedForms[] = {{16, {1.69f, 3.15f, 4.00f, 4.90f, 0.0f}},
                                  {32, {2.74f, 3.81f, 5.49f, 7.26f, 9.51f}},
                                  {48, {3.91f, 5.27f, 0.0f, 9.14f, 0.0f}},
                                  {64, {4.85f, 5.84f, 0.0f, 9.89f, 0.0f}},
                                  {80, {5.66f, 6.78f, 8.86f, 11.1f, 0.0f}}};

template <int Q, int META>
bool fits_qm(int tok, int rt) {
  using namespace stream;
  if (tok == 32 && rt == 5) return stream_fits<Q, META, 32, 5>();
  if (tok == 80 && rt == 4) return stream_fits<Q, META, 80, 4>();
  if (tok == 80 && rt == 3) return !stream_fits<Q, META, 80, 4>();
  static_assert(stream_fits<Q, META, 16, 4>() && stream_fits<Q, META, 32, 4>() && stream_fits<Q, META, 48, 4>() &&
                stream_fits<Q, META, 64, 4>() && stream_fits<Q, META, 80, 3>(), "LDS of the kernels");
  return true;
}
bool rounded_fits(int q, int kind, int tok, int rt) {
  switch (q * 4 + kind) {
    case 8: return fits_qm<2, 0>(tok, rt);
    case 9: return fits_qm<2, 1>(tok, rt);
    case 10: return fits_qm<2, 2>(tok, rt);
    case 12: return fits_qm<3, 0>(tok, rt);
    case 13: return fits_qm<3, 1>(tok, rt);
    case 14: return fits_qm<3, 2>(tok, rt);
    case 16: return fits_qm<4, 0>(tok, rt);
    case 17: return fits_qm<4, 1>(tok, rt);
    default: return fits_qm<4, 2>(tok, rt);
  }
}

struct Cut {
  int rt, slices;
  float us;
};
// `room`: workspace bytes that a sliced launch may use (0: none).
Cut choose(const Form& f, bool exact, int64_t N, int64_t K, int q, int kind, int64_t room) {
  const int64_t tiles = (N + 15) / 16, units = (K / 32 + 7) / 8;
  Cut best{1, 1, 0.0f};
  for (int rt = 1; rt <= 5; ++rt) {
    if (f.us[rt - 1] == 0.0f || (!exact && !rounded_fits(q, kind, f.tok, rt))) continue;
    const int64_t rbs = (tiles + rt - 1) / rt;
    for (int s = 1; s <= kMaxSlices; ++s) {
      const int64_t wgs = rbs * s;
      if (s > 1) {
        const int64_t bytes = kSplitCounterBytes + wgs * rt * ((f.tok + 15) / 16) * 1024;
        if (wgs > kCUs || s > units || bytes > room) break;
      }
      const int64_t per = (units + s - 1) / s;
      const float busy = 0.7f + 0.3f * std::min(1.0f, (float)wgs / kCUs);
      const float us = (float)((wgs + kCUs - 1) / kCUs) * (3.0f + 0.5f * rt + busy * f.us[rt - 1] * (float)((per + 7) / 8)) +
                       (s > 1 ? 1.9f : 0.0f);
      if (best.us == 0.0f || us < best.us) best = Cut{rt, s, us};
    }
  }
  return best;
}

// 3-bit codes at 17 to 32 tokens over 1024 row tiles: the streaming kernel is faster than the one
// cut across small workgroups where its rounds are full (1280 tiles are one round of five a
// workgroup, 1536 two of three) and rows are short or, with zero points or minimums in groups
// of 32 or 64, longer too.  That one / streaming, us, 24 tokens (17 and 32 alike):
//   no metadata, up to 1280 tiles: 18432x1024 13.2 / 9.2, 20480x2048 16.6 / 13.6, 18432x4096
//     28.2 / 24.0, 20480x5120 33.1 / 28.3, 19456x4608 26.2 / 26.5, 17408x5120 26.9 / 27.6, but
//     19456x5632 30.9 / 32.7, 16448x7168 33.1 / 35.4, 20480x8192 40.7 / 42.7;
//   up to 1536: 22016x3072 27.1 / 22.2, 24576x2048 19.6 / 17.3, but 22016x4096 26.1 / 29.2,
//     24576x4096 27.2 / 30.4; more: 28672x2048 19.8 / 21.0, 28672x4096 32.9 / 37.4,
//     32768x3072 27.0 / 29.1;
//   zero points, groups of 32 (minimums alike): 17408x5120 31.4 / 29.0, 20480x6144 39.4 / 35.5,
//     16448x8192 47.8 / 45.2, 24576x6144 49.2 / 45.7, but 18432x12288 64.4 / 66.2, 24576x4096
//     31.7 / 33.0, 28672x4608 43.6 / 45.0, 28672x8192 68.2 / 72.2;
//   groups of 64: 17408x5120 29.7 / 27.9, 20480x6144 37.3 / 34.9, 24576x4096 29.3 / 31.3;
//   groups of 128 as no metadata: 20480x5120 32.9 / 28.0, 16448x8192 42.1 / 43.2.
bool three_bits_stream(int64_t tiles, int64_t K, int64_t weights, int group, int kind) {
  const bool meta = kind != 0 && group < 128 && weights < 190000000;
  if (tiles <= 1280) return K <= 5120 || meta;
  return tiles <= 1536 && (K <= 3072 || (meta && group == 32 && K > 4096));
}

// Large matrices go to the kernels that cut K across many small workgroups (skinny.hip) where
// those measured faster, a workspace given (W4 g32 signed unless said, us, those / these).
// Their time follows the weights; that of these follows rounds of 256 workgroups of up to
// four row tiles, which a matrix of just over 512 or 1024 tiles fills badly.
//   over 1024 tiles, exact from 1.5e8 weights on: 16 tokens on 28672x8192 36.7 / 42.8,
//     24576x8192 33.2 / 36.3, but 28672x4096 26.6 / 23.8; rounded always: 24 tokens on
//     28672x8192 50.2 / 62.1, 28672x4096 31.2 / 34.3, except 3-bit codes at 17 to 32 tokens
//     (three_bits_stream);
//   513 to 1024 tiles, from 1.9e8 weights on: 16 tokens on 13312x16384 39.0 / 44.1 (but
//     13312x12288 30.7 / 31.0); at 17 to 32 tokens from 1.2e8 on, 3-bit codes excepted:
//     32 tokens on 10240x12288 31.6 / 35.6, W2 27.9 / 32.8, W3 40.9 / 41.4, but 13312x8192
//     31.5 / 31.9; two-bit codes on 16384x12288 the other way, 38.2 / 35.4;
//   513 to 590 tiles, rounded (three row tiles on at most 77 % of the CUs), above 16 tokens from 9e7
//     weights on: 18 on W2 8320x13312 30.1 / 36.8, 24 on W4 8411x10752 25.4 / 30.2; below from 1.5e8
//     on: 9 on W3 8768x18304 39.7 / 45.8;
//   exact with zero points or minimums stays here below those sizes, though the others would be
//     faster from 6e7 weights on in groups of 64 and 128 (9 tokens, W2 7296x19456 21.0 / 29.3, 16
//     on W4 16704x6144 23.8 / 30.7) and 8.5e7 in groups of 32 (W2 23808x5632 21.6 / 27.2): their
//     sums cancel the offsets over 16 blocks, not within one, and are ten times as far from 64
//     bits (5.7e-3 of the bf16 outputs off the correctly rounded one for 5.8e-4);
//   exact over a K of one slice (no workspace needed): over 1024 tiles, and from 512 on
//     where groups hold a minimum or zero point: 12 tokens on 28672x2048 10.8 / 13.9,
//     W4 asymmetric on 8192x2048 6.1 / 6.8.
bool blocked_is_faster(int64_t M, int64_t N, int64_t K, int group, int q, int kind, bool exact, bool workspace) {
  const int64_t tiles = (N + 15) / 16, weights = N * K;
  if (exact && K <= 2048) return tiles > 1024 || (kind != 0 && K > 1024 && tiles >= 512);
  if (!workspace || M > kSkinnyMaxM) return false;
  if (tiles <= 512) return false;
  if (!exact && tiles <= 590 && weights >= (M > 16 ? 90000000 : 150000000)) return true;
  if (tiles > 1024) return exact ? weights >= 150000000 : !(q == 3 && M > 16 && three_bits_stream(tiles, K, weights, group, kind));
  if (M > 16 && q != 3 && weights >= 120000000) return q == 4 || tiles < 900;
  return weights >= 190000000 && !(M > 16 && tiles >= 900) && !(q == 2 && tiles >= 900);
}

// More than 32 tokens on more than 512 row tiles: the tiled GEMM (gemm.hip), whose time is that
// of 64 or 80 tokens whatever M is, where it measured faster (us, GEMM / these).
//   at most 70 % of the row tiles of whole rounds in use: W2, 64 tokens on 20480x5120 38.5 /
//     44.5, and from 1.9e8 weights on 34 tokens on 10240x23168 73.4 / 89.2 (but 10240x8192
//     34.1 / 31.5); W4, 64 tokens on 20480x10240 92.5 / 97.3; 80 tokens on 20480x1536 W2
//     17.4 / 23.6, W3 23.6 / 26.8, W4 19.7 / 22.0;
//   over 1024 tiles of short rows, whose second round is all start: 64 tokens W4 on 24896x512 10.2 /
//     19.0, 43 on 28189x1024 14.2 / 18.3, 39 on 29707x1408 18.2 / 21.9 (1792 22.5 / 21.8); up to 48
//     tokens W2 and W3 to K = 896: 41 tokens W2 on 26432x512 9.9 / 16.3, 37 W3 on 22244x896 16.1 /
//     18.3 (but 43 W3 on 19389x1024 15.7 / 13.6), above 48 to 1536: 49 W3 on 25796x1408 23.4 / 25.0;
//   over 64 tokens: W2 in several rounds, 28672x4096 41.1 / 44.8 (16384x4096 28.1 / 23.7);
//     W4 where LDS has no room for four row tiles, from 1.9e8 weights on: 16384x12288
//     89.8 / 98.5 (but 16384x4096 41.8 / 34.2); below K = 1024 W2 and W4: 16384x576 9.7 /
//     10.5 and 10.9 / 14.1.
bool tiled_is_faster(int64_t M, int64_t N, int64_t K, int q, int kind) {
  const int64_t tiles = (N + 15) / 16, weights = N * K;
  if (M <= kSkinnyMaxM || tiles <= 512) return false;
  if (tiles > 1024 && K <= (q == 4 || M > 48 ? 1536 : 896)) return true;
  const int64_t whole = (tiles + 1023) / 1024 * 1024;
  const bool part_filled = 10 * tiles <= 7 * whole;
  if (part_filled) {
    if (q == 2 && (M > 64 || weights >= 190000000 || (M > 48 && tiles > 1024))) return true;
    if (q == 4 && M > 48 && weights >= 190000000) return true;
    if (M > 64 && K < 2048) return true;
  }
  if (M <= 64) return false;
  if (q == 2) return tiles > 1024 || K < 1024;
  return q == 4 && (K < 1024 || (weights >= 190000000 && !rounded_fits(q, kind, 80, 4)));
}

// What runs and its cut.  `have`: workspace bytes (0: none), `aligned`: scales and metadata at
// 16-byte addresses.
struct Choice {
  int kernel;           // kRouteGemm: launch_gemm_bf16
  bool exact;
  int tok;
  Cut cut;
  TilePlan tile;
};
Choice choose_kernel(int64_t M, int64_t N, int64_t K, int group, int q, int kind, bool aligned, int64_t have) {
  // Exact weights: the sizes that allow it, rows of scales and metadata that start 16-byte
  // aligned, and the workspace its layout names (or a K that needs none).
  int64_t exact_bytes = 0;
  Choice c{};
  c.exact = stat_layout_bytes(M, N, K, q, &exact_bytes) && aligned && have >= exact_bytes;
  const Form* form = c.exact ? (M <= 8 ? &kExactForms[0] : &kExactForms[1]) : &kRoundedForms[0];
  if (!c.exact)
    while (form->tok < M) ++form;
  c.tok = form->tok;
  const int64_t named = c.exact ? exact_bytes : M <= kSkinnyMaxM ? split_layout_bytes(M, N, K) : (int64_t)gemm_workspace_bytes(M, N, K);
  const int64_t room = named > 0 && have >= named ? named : 0;
  c.kernel = c.exact ? kRouteExact : kRouteRounded;
  if (blocked_is_faster(M, N, K, group, q, kind, c.exact, room > 0)) {
    c.kernel = c.exact ? kRouteStat : kRouteSplit;
    return c;
  }
  if (tiled_is_faster(M, N, K, q, kind)) {
    c.kernel = kRouteGemm;
    return c;
  }
  c.cut = choose(*form, c.exact, N, K, q, kind, room);
  // Above 48 tokens the tiles of tile.hip, where their estimate is clearly lower and the
  // matrix is not small: 64 tokens on 12288x4096 22.7 here, 20.1 there, 77 tokens on
  // 4096x12288 26.4 / 24.2, but 52 on 4672x1536 7.4 / 8.1 and 67 on 960x25216 20.1 / 21.5.
  if (M > 48 && N * K >= 30000000) {
    c.tile = tile_plan(M, N, K, room);
    if (c.tile.us < 0.9f * c.cut.us) c.kernel = kRouteTile;
  }
  return c;
}

}  // namespace

Route stream_route(int64_t M, int64_t N, int64_t K, int group, int q, int kind, bool aligned, int64_t workspace_bytes) {
  const Choice c = choose_kernel(M, N, K, group, q, kind, aligned, workspace_bytes);
  switch (c.kernel) {
    case kRouteStat: case kRouteSplit: return skinny_route(M, N, K, q, c.exact);
    case kRouteGemm: return gemm_route(M, N, K, q, workspace_bytes);
    case kRouteTile: return tile_route(c.tile);
    default: return Route{c.kernel, c.tok, 16 * c.cut.rt, c.cut.slices};
  }
}

hipError_t launch_stream_bf16(const uint16_t* x, int64_t M, const uint8_t* codes, const uint16_t* scales, GroupMeta meta,
                              int64_t N, int64_t K, int group, int q, uint16_t* y, void* workspace,
                              size_t workspace_bytes, hipStream_t stream) {
  if (M < 3 || M > kStreamMaxM) return hipErrorInvalidValue;
  const bool aligned = reinterpret_cast<uintptr_t>(scales) % 16 == 0 && reinterpret_cast<uintptr_t>(meta.ptr) % 16 == 0;
  const Choice c = choose_kernel(M, N, K, group, q, meta.kind, aligned, workspace != nullptr ? (int64_t)workspace_bytes : 0);
  switch (c.kernel) {
    case kRouteStat: case kRouteSplit:
      return launch_skinny_bf16(x, M, codes, scales, meta, N, K, group, q, y, workspace, c.exact, stream);
    case kRouteGemm:
      return launch_gemm_bf16(x, M, codes, scales, meta, N, K, group, q, y, workspace, workspace_bytes, stream);
    case kRouteTile:
      return launch_tile_bf16(c.tile, x, M, codes, scales, meta, N, K, group, q, y, workspace, stream);
  }
  stream::StreamArgs a;
  a.x = x; a.M = M; a.codes = codes; a.scales = scales; a.meta = meta.ptr;
  a.N = N; a.K = K;
  a.gshift = group == 32 ? 0 : group == 64 ? 1 : 2;
  a.slices = c.cut.slices;
  a.y = y;
  a.partials = c.cut.slices > 1 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + kSplitCounterBytes) : nullptr;
  a.counters = static_cast<unsigned int*>(workspace);
  a.stream = stream;
  if (c.exact) return stream::launch_exact(a, q, meta.kind, c.tok, c.cut.rt);
  switch (q) {
    case 2: return stream::launch_rounded_q2(a, meta.kind, c.tok, c.cut.rt);
    case 3: return stream::launch_rounded_q3(a, meta.kind, c.tok, c.cut.rt);
    default: return stream::launch_rounded_q4(a, meta.kind, c.tok, c.cut.rt);
  }
}

size_t stream_workspace_bytes(int64_t M, int64_t N, int64_t K, int q) {
  // the larger of skinny.hip's two layouts; the kernels here need less
  int64_t exact_bytes = 0;
  const bool ok = stat_layout_bytes(M, N, K, q, &exact_bytes);
  return (size_t)std::max<int64_t>(split_layout_bytes(M, N, K), ok ? exact_bytes : 0);
}

}  // namespace ssq
