// Kernel of the matmul for middle token counts (tile.hip chooses among its tiles):
// y[M,N] = x[M,K] * What[N,K]^T, from 49 tokens on.
//
// App. B.3 of the paper: What[n,k] = s[n,b] (u[n,k] - o[n,b]), each weight formed exactly in
// fp32 and rounded to bf16 once, multiplied by v_mfma_f32_32x32x16_bf16.
//
// Work split.  Tens to hundreds of tokens make too few of the GEMM's 256 x 128 tiles to fill
// the chip, and cutting those along K costs more than the product (4096x4096, 256 tokens: 32
// tiles in 8 slices, 33 MB of partials, 25 us).  Here a workgroup's tile is small (32 TI
// tokens x 32 TC rows) and its W wavefronts split K among themselves: each computes the whole
// tile for every W-th unit of UB blocks, from its own stages in LDS, so the main loop has no
// barrier, an activation is read from LDS once per TC row tiles and a weight is dequantized
// once per TI token tiles; the wavefronts meet in LDS at the end.
//
// A step is 64 k: lanes 0-31 of a wavefront take its first block, lanes 32-63 the second, and
// MFMA j of the step the weights 8j..8j+7 of each lane's block, so that a lane dequantizes
// whole blocks (one scale each).  Operands are read one MFMA slice ahead, activation stages
// are filled by direct-to-LDS loads one or two steps ahead, codes go through registers to LDS
// a unit ahead (whole 64- or 128-byte pieces of a row).
//
// What bounds it: the activations, which enter a CU at about 100 bytes per ns (2 BM K bytes a
// workgroup; 10 of the 28 us of 128 tokens on 12288x4096), partly overlapped with 8 us of
// dequantization and MFMA, and 5 us of start, codes and reduction.  W4 g32 signed, GEMM /
// these, us: 96 tokens on 4096x4096 18.4 / 12.2, 256 tokens 25.4 / 18.1, 128 tokens on
// 12288x4096 38.4 / 28.0, 256 tokens on 1024x4096 23.5 / 9.3.  Tried without gain: a third
// stage where two fit, eight wavefronts for 64-token tiles, K started elsewhere in each
// workgroup.
#pragma once

#include <algorithm>
#include <type_traits>

#include "stream_kernels.h"

namespace ssq {
namespace tile {

using stream::kOutOfRange;
using stream::lds_object;
using stream::lds_ptr_t;
using stream::wave_sync;
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int Q, int META, int TI, int TC, int S, int W>
struct Tile {
  static constexpr int BM = 32 * TI, BN = 32 * TC;
  static constexpr int UB = W > 4 || TI * TC >= 8 ? 4 : 8;                  // 32-k blocks of a unit
  static constexpr int kSteps = UB / 2;
  static constexpr int kStageBytes = BM * 128;                     // 64 k of every token
  static constexpr int kXLoads = kStageBytes / 1024;
  static constexpr int kPieceRows = 256 / (4 * Q * UB);            // rows of codes in 256 bytes
  static constexpr int kCodePitch = Q == 3 ? 12 * UB + 4 : 4 * Q * UB;
  static constexpr int kCodeBytes = BN * kCodePitch;
  static constexpr int kScalePitch = 3 * UB;                       // 2 UB bytes and a spare
  static constexpr int kScaleBytes = BN * kScalePitch;
  static constexpr int kLoads = BN * UB / 64;                      // load instructions of a unit's codes
  static constexpr int kLds = W * (S * kStageBytes + kCodeBytes + kScaleBytes * (META != kMetaNone ? 2 : 1)) + (S > 2 ? 0 : 16) + (META != kMetaNone ? 0 : 16);
};

// Slice J (weights 8J..8J+7) of a block.
template <int Q, int J>
__device__ __forceinline__ bf16x8 dequant_slice(const uint32_t (&d)[Q], const float (&sc)[2], const float (&so)[2],
                                                uint32_t mask, uint32_t mask_hi, uint32_t magic) {
  uint32_t w;
  if constexpr (Q == 4) w = d[J];
  else if constexpr (Q == 2) w = (J & 1) ? d[J >> 1] >> 16 : d[J >> 1];
  else w = J == 0 ? d[0] : J == 1 ? __builtin_amdgcn_alignbit(d[1], d[0], 24)
           : J == 2 ? __builtin_amdgcn_alignbit(d[2], d[1], 16) : d[2] >> 8;
  return stream::dequant8<Q>(w, sc, so, mask, mask_hi, magic);
}

template <int Q, int META, int TI, int TC, int S, int W>
__global__ __launch_bounds__(64 * W) void tile_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
    const void* __restrict__ meta, int M, int N, int K, int gshift, int slices, int chunk, uint16_t* __restrict__ y,
    float* __restrict__ partials, unsigned int* __restrict__ counters) {
  using C = Tile<Q, META, TI, TC, S, W>;
  constexpr int UB = C::UB;
  constexpr int kMetaSize = META == kMetaZp ? 1 : META == kMetaMin ? 2 : 0;
  uint8_t* const xs0 = lds_object<0, W * C::kStageBytes>();
  uint8_t* const xs1 = lds_object<1, W * C::kStageBytes>();
  uint8_t* const xs2 = lds_object<2, (S > 2 ? W * C::kStageBytes : 16)>();
  uint8_t* const cs_all = lds_object<3, W * C::kCodeBytes>();
  uint8_t* const ss_all = lds_object<4, W * C::kScaleBytes>();
  uint8_t* const zs_all = lds_object<5, META != kMetaNone ? W * C::kScaleBytes : 16>();
  auto stage = [&](auto idx) -> uint8_t* {
    constexpr int i = decltype(idx)::value % S;
    return i == 0 ? xs0 : i == 1 ? xs1 : xs2;
  };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Work order: XCD b % 8 takes a run of `chunk` items; an item's K slices are adjacent, then
  // the token tiles of one row tile (which read the same weights).
  const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
  const int b = ((int)blockIdx.x & 7) * chunk + ((int)blockIdx.x >> 3);
  if (b >= tiles_m * tiles_n * slices) return;
  const int slice = b % slices, ti = b / slices;
  const int64_t m0 = (int64_t)(ti % tiles_m) * C::BM, n0 = (int64_t)(ti / tiles_m) * C::BN;
  const int nblk = K / 32;
  const int nu_all = (nblk + UB - 1) / UB, per = (nu_all + slices - 1) / slices;
  const int u_end = std::min(nu_all, (slice + 1) * per);
  const uint32_t row_bytes = (uint32_t)K * Q / 8;
  const uint32_t gpr = (uint32_t)nblk >> gshift;
  const uint32_t rows = (uint32_t)std::min<int64_t>(C::BN, N - n0), toks = (uint32_t)std::min<int64_t>(C::BM, M - m0);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + n0 * row_bytes, rows * row_bytes);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales + n0 * gpr, rows * gpr * 2);
  const uint8_t* const mp = static_cast<const uint8_t*>(meta);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(kMetaSize ? mp + n0 * gpr * kMetaSize : mp,
                                              kMetaSize ? rows * gpr * kMetaSize : 0u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + m0 * K, toks * (uint32_t)K * 2);

  uint8_t* const cs = cs_all + wave * C::kCodeBytes;
  uint8_t* const ss = ss_all + wave * C::kScaleBytes;
  uint8_t* const zs = META != kMetaNone ? zs_all + wave * C::kScaleBytes : zs_all;
  const int r32 = lane & 31, h = lane >> 5;      // MFMA operand row, block of the step

  struct Codes {
    uint32_t d[C::kLoads][Q];
    uint32_t s[C::kLoads], z[C::kLoads];
  };
  // Codes, scales and metadata of unit u: lane -> (row lane / UB, block lane % UB) of 64 / UB
  // rows.  Past the row or slice bit 31 is set, out of every descriptor's range.
  const int lrow = lane / UB, lblk = lane % UB;
  auto issue_c = [&](int u, Codes& t) {
    const int blk = UB * u + lblk;
    const uint32_t past = (blk < nblk) & (u < u_end) ? 0u : kOutOfRange;
#pragma unroll
    for (int i = 0; i < C::kLoads; ++i) {
      const uint32_t row = (uint32_t)(i * (64 / UB) + lrow);
      buffer_block_codes<Q>(rc, (row * row_bytes + (uint32_t)blk * (4 * Q)) | past, 0, t.d[i]);
      const uint32_t gi = row * gpr + (uint32_t)(blk >> gshift);
      t.s[i] = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)((gi * 2) | past), 0, 0);
      if constexpr (META == kMetaZp) t.z[i] = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)(gi | past), 0, 0);
      if constexpr (META == kMetaMin) t.z[i] = __builtin_amdgcn_raw_buffer_load_b16(rz, (int)((gi * 2) | past), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto code_swz = [&](int row) { return (row / C::kPieceRows) & (UB - 1); };
  auto store_codes = [&](const Codes& t) {
#pragma unroll
    for (int i = 0; i < C::kLoads; ++i) {
      const int row = i * (64 / UB) + lrow;
      const uint32_t (&d)[Q] = t.d[i];
      if constexpr (Q == 4) *reinterpret_cast<u32x4*>(cs + row * C::kCodePitch + 16 * (lblk ^ code_swz(row))) = u32x4{d[0], d[1], d[2], d[3]};
      else if constexpr (Q == 2) *reinterpret_cast<u32x2*>(cs + row * C::kCodePitch + 8 * (lblk ^ code_swz(row))) = u32x2{d[0], d[1]};
      else
#pragma unroll
        for (int e = 0; e < 3; ++e) *reinterpret_cast<uint32_t*>(cs + row * C::kCodePitch + 12 * lblk + 4 * e) = d[e];
      *reinterpret_cast<uint16_t*>(ss + row * C::kScalePitch + 2 * lblk) = (uint16_t)t.s[i];
      if constexpr (META != kMetaNone) *reinterpret_cast<uint16_t*>(zs + row * C::kScalePitch + 2 * lblk) = (uint16_t)t.z[i];
    }
  };
  // Activations of a step (two blocks, 64 k) into a stage: lane L of load i fills piece L % 8
  // of token 8 i + L / 8, which holds piece (L % 8) ^ (token / 2 % 8): the 16 lanes that an
  // operand read serves at once then touch every bank once.
  const int xt = lane >> 3;
  const int p0 = (lane & 7) ^ (xt >> 1), p1 = p0 ^ 4;     // pieces of even and odd loads
  const uint32_t x0 = (uint32_t)xt * (uint32_t)K * 2;
  auto issue_x = [&](int u, int st, uint8_t* base, auto firstc, auto lastc) {
    const int blk0 = UB * u + 2 * st;
    const uint32_t a = x0 + (uint32_t)blk0 * 64;
    const uint32_t in0 = (blk0 + (p0 >> 2) < nblk) & (u < u_end) ? 0u : kOutOfRange;
    const uint32_t in1 = (blk0 + (p1 >> 2) < nblk) & (u < u_end) ? 0u : kOutOfRange;
    const uint32_t o0 = (a + 16 * p0) | in0, o1 = (a + 16 * p1) | in1;
#pragma unroll
    for (int i = decltype(firstc)::value; i < decltype(lastc)::value; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(base + wave * C::kStageBytes + i * 1024), 16,
                                               (int)(((i & 1) ? o1 : o0) + (uint32_t)i * 16u * (uint32_t)K), 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x16 acc[TI][TC];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int c = 0; c < TC; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][c][r] = 0.0f;

  const uint32_t mask = opaque_s(stream::code_mask<Q>()), magic = opaque_v(0x64006400u);
  const uint32_t mask_hi = opaque_s(stream::code_mask<Q>() << Q);
  struct Weights {
    uint32_t d[TC][Q];
    uint32_t s[TC], z[TC];
  };
  auto read_codes = [&](int st, Weights& w) {
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int row = 32 * c + r32, blk = 2 * st + h;
      if constexpr (Q == 4) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(cs + row * C::kCodePitch + 16 * (blk ^ code_swz(row)));
        w.d[c][0] = v.x; w.d[c][1] = v.y; w.d[c][2] = v.z; w.d[c][3] = v.w;
      } else if constexpr (Q == 2) {
        const u32x2 v = *reinterpret_cast<const u32x2*>(cs + row * C::kCodePitch + 8 * (blk ^ code_swz(row)));
        w.d[c][0] = v.x; w.d[c][1] = v.y;
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e) w.d[c][e] = *reinterpret_cast<const uint32_t*>(cs + row * C::kCodePitch + 12 * blk + 4 * e);
      }
      w.s[c] = *reinterpret_cast<const uint16_t*>(ss + row * C::kScalePitch + 2 * blk);
      if constexpr (META != kMetaNone) w.z[c] = *reinterpret_cast<const uint16_t*>(zs + row * C::kScalePitch + 2 * blk);
      else w.z[c] = 0u;
    }
  };
  auto read_x = [&](const uint8_t* base, int j, bf16x8 (&a)[TI]) {
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const int t = 32 * i + r32;
      a[i] = *reinterpret_cast<const bf16x8*>(base + wave * C::kStageBytes + t * 128 + (((4 * h + j) ^ ((t >> 1) & 7)) << 4));
    }
  };

  // The wavefront's units: u0, u0 + W, ... (loads past the last move nothing)
  const int u0 = slice * per + wave;
  Codes next;
  issue_c(u0, next);
#pragma unroll
  for (int st = 0; st < S - (S == 3); ++st) issue_x(u0 + st / C::kSteps * W, st % C::kSteps, st == 0 ? xs0 : st == 1 ? xs1 : xs2, std::integral_constant<int, 0>{}, std::integral_constant<int, C::kXLoads>{});
  bf16x8 a[2][TI];
  Weights w;
  if (u0 < u_end) {
    store_codes(next);
    wave_sync();
    issue_c(u0 + W, next);
    read_codes(0, w);
    read_x(xs0, 0, a[0]);
  }

  // Step `st` of unit u from stage P: slice j's successor is read before slice j is
  // dequantized; the last slice first sends the loads that refill the stage, then reads the
  // next step's first operands.
  auto step = [&](int u, auto stc, auto pc) {
    constexpr int st = decltype(stc)::value, P = decltype(pc)::value;
    uint8_t* const cur = stage(pc);
    float sc[TC][2], so[TC][2];
    Weights v = w;
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const float s = f16_bits_to_f32(v.s[c]);
      sc[c][0] = s;
      sc[c][1] = s * (1.0f / (float)(1 << Q));
      so[c][0] = dequant_offset<META, Q>(s, v.z[c]);
      so[c][1] = stream::dequant_offset_hi<META, Q>(s, v.z[c]);
    }
    auto slice_j = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      if constexpr (S == 3) {
        // the stage that the step before read takes the step after next, a quarter of its loads a slice
        constexpr int t = st + 2;
        issue_x(u + t / C::kSteps * W, t % C::kSteps, stage(std::integral_constant<int, P + 2>{}),
                std::integral_constant<int, j * C::kXLoads / 4>{}, std::integral_constant<int, (j + 1) * C::kXLoads / 4>{});
      }
      if constexpr (j < 3) {
        read_x(cur, j + 1, a[(j + 1) & 1]);
        if constexpr (j == 1 && st == C::kSteps - 1) {        // the unit's codes have all been read
          wave_sync();
          store_codes(next);
          wave_sync();
          issue_c(u + 2 * W, next);
        }
        if constexpr (j == 2) read_codes((st + 1) % C::kSteps, w);
      } else {
        __builtin_amdgcn_s_waitcnt(0xC07F);       // the stage's operands are in registers
        if constexpr (S != 3)
          issue_x(u + (st + S) / C::kSteps * W, (st + S) % C::kSteps, cur,
                  std::integral_constant<int, 0>{}, std::integral_constant<int, C::kXLoads>{});
        read_x(stage(std::integral_constant<int, P + 1>{}), 0, a[0]);
      }
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 bq[TC];
#pragma unroll
      for (int c = 0; c < TC; ++c) bq[c] = dequant_slice<Q, j>(v.d[c], sc[c], so[c], mask, mask_hi, magic);
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int c = 0; c < TC; ++c)
          acc[i][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j & 1][i], bq[c], acc[i][c], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    slice_j(std::integral_constant<int, 0>{});
    slice_j(std::integral_constant<int, 1>{});
    slice_j(std::integral_constant<int, 2>{});
    slice_j(std::integral_constant<int, 3>{});
  };
  auto unit = [&](int u, auto pc) {
    constexpr int P = decltype(pc)::value;
    step(u, std::integral_constant<int, 0>{}, std::integral_constant<int, P % S>{});
    step(u, std::integral_constant<int, 1>{}, std::integral_constant<int, (P + 1) % S>{});
    if constexpr (C::kSteps > 2) {
      step(u, std::integral_constant<int, 2>{}, std::integral_constant<int, (P + 2) % S>{});
      step(u, std::integral_constant<int, 3>{}, std::integral_constant<int, (P + 3) % S>{});
    }
  };
  for (int u = u0; u < u_end; u += W) {
    unit(u, std::integral_constant<int, 0>{});
    if constexpr (S == 3) {                       // the stages come round after three units
      if ((u += W) >= u_end) break;
      unit(u, std::integral_constant<int, C::kSteps % 3>{});
      if ((u += W) >= u_end) break;
      unit(u, std::integral_constant<int, 2 * C::kSteps % 3>{});
    }
  }

  // The wavefronts' partial sums meet in LDS in wavefront order, row tile by row tile.
  wait_vmcnt<0>();
  __syncthreads();
  constexpr int kTF = TI * TC * 1024;
  constexpr int kSc1 = 16;
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(partials + (int64_t)ti * slices * kTF, slices > 1 ? (uint32_t)slices * (kTF * 4) : 0u);
  // element quad e of row tile c: token tile e / 256, registers 4 (e / 64 % 4).., lane e % 64
  auto put = [&](int c, int e, const f32x4& v) {
    const int l = e & 63, q4 = (e >> 6) & 3, i = e >> 8;
    const int64_t n = n0 + 32 * c + (l & 31), m = m0 + 32 * i + 8 * q4 + 4 * (l >> 5);
    if (n < N)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (m + r < M) y[(m + r) * N + n] = f32_to_bf16_bits(v[r]);
  };
#pragma unroll
  for (int c = 0; c < TC; ++c) {
    float* const part = reinterpret_cast<float*>(c == 0 ? xs0 : xs1);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<f32x4*>(part + (wave * TI + i) * 1024 + q4 * 256 + 4 * lane) =
            f32x4{acc[i][c][4 * q4], acc[i][c][4 * q4 + 1], acc[i][c][4 * q4 + 2], acc[i][c][4 * q4 + 3]};
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < TC; ++c) {
    const float* const part = reinterpret_cast<const float*>(c == 0 ? xs0 : xs1);
#pragma unroll
    for (int e = tid; e < TI * 256; e += 64 * W) {
      f32x4 v = *reinterpret_cast<const f32x4*>(part + 4 * e);
#pragma unroll
      for (int k = 1; k < W; ++k) v += *reinterpret_cast<const f32x4*>(part + k * TI * 1024 + 4 * e);
      if (slices == 1) put(c, e, v);
      else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rp, (slice * kTF + c * TI * 1024 + 4 * e) * 4, 0, kSc1);
    }
  }
  if (slices == 1) return;
  unsigned int* const arrived = reinterpret_cast<unsigned int*>(cs_all);
  wait_vmcnt<0>();
  __syncthreads();
  if (tid == 0) *arrived = atomicAdd(&counters[ti], 1u);
  __syncthreads();
  if (*arrived != (unsigned int)(slices - 1)) return;
  for (int e = tid; e < TC * TI * 256; e += 64 * W) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < slices; s0 += 4) {
      f32x4 p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        p[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             rp, s0 + i < slices ? ((s0 + i) * kTF + 4 * e) * 4 : (int)kOutOfRange, 0, kSc1));
#pragma unroll
      for (int i = 0; i < 4; ++i) v += p[i];
    }
    put(e / (TI * 256), e % (TI * 256), v);
  }
  if (tid == 0) __hip_atomic_store(&counters[ti], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int Q, int META, int TI, int TC, int S, int W>
hipError_t tile_launch(const stream::StreamArgs& a) {
  using C = Tile<Q, META, TI, TC, S, W>;
  static_assert(C::kLds <= 163840, "LDS of a workgroup");
  static_assert(S == 3 || C::kSteps % S == 0, "stages come round with the units");
  const int64_t items = ((a.M + C::BM - 1) / C::BM) * ((a.N + C::BN - 1) / C::BN) * a.slices;
  const int64_t chunk = (items + 7) / 8;
  tile_kernel<Q, META, TI, TC, S, W><<<dim3((unsigned)(8 * chunk)), 64 * W, 0, a.stream>>>(
      a.x, a.codes, a.scales, a.meta, (int)a.M, (int)a.N, (int)a.K, a.gshift, a.slices, (int)chunk, a.y, a.partials,
      a.counters);
  return hipGetLastError();
}

// The tiles, in the order of tile.hip's table.
template <int Q, int META>
hipError_t tile_form(const stream::StreamArgs& a, int form) {
  switch (form) {
    case 0: return tile_launch<Q, META, 1, 1, 2, 8>(a);
    case 1: return tile_launch<Q, META, 2, 1, 3, 4>(a);
    case 2: return tile_launch<Q, META, 3, 1, 2, 4>(a);
    case 3: return tile_launch<Q, META, 2, 2, 3, 4>(a);
    case 4: return tile_launch<Q, META, 3, 2, 2, 4>(a);
    case 5: return tile_launch<Q, META, 4, 2, 2, 4>(a);
  }
  return hipErrorInvalidValue;
}
template <int Q>
hipError_t tile_q(const stream::StreamArgs& a, int kind, int form) {
  return kind == kMetaNone ? tile_form<Q, kMetaNone>(a, form)
       : kind == kMetaZp ? tile_form<Q, kMetaZp>(a, form) : tile_form<Q, kMetaMin>(a, form);
}

}  // namespace tile
}  // namespace ssq
