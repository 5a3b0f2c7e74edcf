// Kernels of the streaming matmul for small token counts (stream.hip chooses among them):
// y[M,N] = x[M,K] * What[N,K]^T, 3 <= M <= 80.
//
// App. B.3 of the paper: What[n,k] = s[n,b] (u[n,k] - o[n,b]).  With few tokens the product
// is bound by streaming the packed weights; the tokens share each weight through bf16 MFMA
// (v_mfma_f32_16x16x32_bf16).
//
// Work split.  A workgroup of 8 wavefronts owns RT tiles of 16 weight rows and all the
// tokens; its wavefronts take the units of K (256 k: 8 blocks) in turn, each for every row
// of the workgroup, and meet once at the end, in LDS and in wavefront order.  So there is no
// barrier in the main loop, every activation is read by one wavefront of the workgroup and
// serves RT tiles, and a matrix needs no reduction across workgroups: with 256 workgroups
// or fewer (one per CU, RT chosen for it) the launch is one round.  Long rows in few
// workgroups may still be cut into slices that meet in the caller's workspace.
//
// Per unit a wavefront holds its codes and scales in registers (128 contiguous bytes a row
// at q = 4: with 64 a 33 MB read took 7.0 us, with 128 6.3), moves them through a private
// piece of LDS to the MFMA layout, and gets its activations by direct-to-LDS loads, two
// stages ahead.  Loads return in order, so activations are requested before the codes that
// are needed after them.
//
// What bounds it: the activations (M K bytes times two per 16 RT rows through one CU's
// cache port, in the same queue as the codes), then vector work per weight, then the
// launch (2.5 us).  Measured against the kernels that cut every matrix across small
// workgroups, or a 128-row GEMM tile from 33 tokens on (W4 g32 signed, us): 16 tokens on
// 1024x4096 7.8 before, 5.4 now, 4096x4096 8.4 / 6.0, 14336x4096 15.3 / 12.4, 4096x14336
// 15.3 / 14.0; 32 tokens on 4096x4096 11.4 / 7.5; 77 tokens on 12288x4096 37 / 24,
// 4096x14336 30.5 / 27.  Two forms:
//  * exact (q = 2, 4; M <= 16): every weight enters the MFMA exactly.  For block b of row n,
//      sum_k x[m,k] s (u - o) = s * (sum_k x[m,k] (128 + u) - (128 + o) xs[m,b]):
//    OR-ing a code into the bf16 constant 128 (0x4300 | u == 128 + u) takes one v_and_or
//    for two weights, the second term is the accumulator's start value, one more MFMA of the
//    activations against a constant (a zero point starts at -128 xs and takes another with -z
//    for each row tile; the minimum layout starts at -128 xs and adds m xs as -m/128 times
//    that), and one fma per output and block applies the scale.
//  * rounded (every other case): a weight is formed as s (u - o) exactly in fp32 and rounded to
//    bf16 once, so nothing is left to do per output; cheaper from about 32 tokens on.
#pragma once

#include <algorithm>
#include <type_traits>

#include "mfma_dequant.h"
#include "ssq_internal.h"

namespace ssq {
namespace stream {

constexpr uint32_t kOutOfRange = 0x80000000u;   // past every buffer's size: loads return 0
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Shapes of one instantiation: TOK tokens (8 or a multiple of 16), RT tiles of 16 weight rows.
constexpr int kWaves = 8;
template <int Q, int META, int TOK, int RT>
struct Stream {
  static constexpr int MB = (TOK + 15) / 16;
  static constexpr int kRows = 16 * RT;
  static constexpr int XB = MB == 1 ? 4 : MB <= 2 ? 2 : 1;          // 32-k blocks of an activation stage
  static constexpr int kRowBytes = 64 * XB;                        // a token's activations in a stage
  static constexpr int kStageBytes = TOK * kRowBytes;              // one wavefront's stage
  static constexpr int kXLoads = kStageBytes / 1024;
  static constexpr int kSteps = 8 / XB;                            // stages per unit (8 blocks)
  static constexpr int kCodePitch = Q == 3 ? 100 : 32 * Q;         // bytes of a row's codes in a unit
  static constexpr int kTileBytes = 16 * kCodePitch;
  static constexpr int kScalePitch = 24;                           // bytes of a row's 8 binary16 scales + spare
  static constexpr int kScaleBytes = 16 * kScalePitch;
  static constexpr int kTileFloats = MB * 256;                     // a row tile's accumulators
};

// 8 weights s*(u - o) (or s*u + m) in natural order as four bf16 pairs, from 8 codes at bit
// 0 of `w`.  Each field is OR-ed into the mantissa of fp16 1024 where it lies or one field
// higher; one fma per weight forms (1024 + u) s + so[0] or (1024 + 2^q u)(s 2^-q) + so[1],
// exact in fp32 and rounded to bf16 once.
template <int Q>
__device__ __forceinline__ bf16x8 dequant8(uint32_t w, const float (&sc)[2], const float (&so)[2], uint32_t mask,
                                           uint32_t mask_hi, uint32_t magic) {
  if constexpr (Q == 2) w = __builtin_amdgcn_perm(0u, w, 0x0C010C00u);
  if constexpr (Q == 3) w = (w & 0xFFFu) | ((w << 4) & 0x0FFF0000u);
  const uint32_t t = w >> (2 * Q);
  const uint32_t p[4] = {(w & mask) | magic, (w & mask_hi) | magic, (t & mask) | magic, (t & mask_hi) | magic};
  float f[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[i] = __builtin_fmaf(f16_lo(p[i]), sc[i & 1], so[i & 1]);
    f[i + 4] = __builtin_fmaf(f16_hi(p[i]), sc[i & 1], so[i & 1]);
  }
  return __builtin_bit_cast(bf16x8, u32x4{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                                          pack_bf16x2(f[6], f[7])});
}
template <int META, int Q>
__device__ __forceinline__ float dequant_offset_hi(float s, uint32_t meta_bits) {
  constexpr float kBase = (float)(1024 >> Q);
  if constexpr (META == kMetaMin) return __builtin_fmaf(-kBase, s, f16_bits_to_f32(meta_bits));
  const float o = META == kMetaZp ? (float)meta_bits : (float)(1 << (Q - 1));
  return -(kBase + o) * s;
}

// 8 codes of a block as bf16 pairs 128 + u, paired (e0, e4), (e1, e5), (e2, e6), (e3, e7).
// `mask` and `magic` are opaque, so that each pair is one v_and_or_b32 (and_or() may not write
// an MFMA's operand).
template <int Q>
__device__ __forceinline__ bf16x8 code_pairs(uint32_t w, uint32_t mask, uint32_t magic) {
  if constexpr (Q == 2) w = __builtin_amdgcn_perm(0u, w, 0x0C010C00u);   // bytes {b0, 0, b1, 0}
  if constexpr (Q == 3) w = (w & 0xFFFu) | ((w << 4) & 0x0FFF0000u);
  const u32x4 v{(w & mask) | magic, ((w >> Q) & mask) | magic, ((w >> (2 * Q)) & mask) | magic,
                ((w >> (3 * Q)) & mask) | magic};
  return __builtin_bit_cast(bf16x8, v);
}
template <int Q>
constexpr uint32_t code_mask() { return Q == 4 ? 0x000F000Fu : Q == 3 ? 0x00070007u : 0x00030003u; }

// Orders LDS stores of some lanes before loads of others within one wavefront.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// An LDS array of its own (the kernels' stages are distinct objects, see stream_kernel).
template <int I, int BYTES>
__device__ __forceinline__ uint8_t* lds_object() {
  __shared__ __attribute__((aligned(1024))) uint8_t mem[BYTES];
  return mem;
}

template <int Q, int META, int TOK, int RT>
struct Exact {
  static constexpr int kRows = 16 * RT;
  static constexpr int kStageBytes = TOK * 256;                    // 128 k of every token, bf16
  static constexpr int kCodeBytes = 16 * 32 * Q;                   // a unit of a row tile
  static constexpr int kTileBytes = kCodeBytes + 256 + (META != kMetaNone ? 256 : 0);
  static constexpr int kTileFloats = 256;
};

// The exact form (see the top of the file): MB = 1.
template <int Q, int META, int TOK, int RT>
__global__ __launch_bounds__(64 * kWaves) void stream_exact_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
    const void* __restrict__ meta, int M, int N, int K, int gshift, int slices, uint16_t* __restrict__ y,
    float* __restrict__ partials, unsigned int* __restrict__ counters) {
  using S = Exact<Q, META, TOK, RT>;
  constexpr int W = kWaves, MB = 1;
  constexpr int kMetaSize = META == kMetaZp ? 1 : META == kMetaMin ? 2 : 0;
  uint8_t* const xs0 = lds_object<0, W * S::kStageBytes>();
  uint8_t* const xs1 = lds_object<1, W * S::kStageBytes>();
  uint8_t* const cs_all = lds_object<2, W * S::kTileBytes>();
  auto stage_of = [&](auto idx) -> uint8_t* {
    constexpr int i = decltype(idx)::value;
    if constexpr (i == 0) return xs0;
    else if constexpr (i == 1) return xs1;
    else return lds_object<i + 8, W * S::kStageBytes>();
  };

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = (int)blockIdx.x % slices, rb = (int)blockIdx.x / slices;
  const int64_t n0 = (int64_t)rb * S::kRows;
  const int nblk = K / 32;                      // a multiple of 16
  const int nu_all = nblk / 8, per = (nu_all + slices - 1) / slices;
  const int u_end = std::min(nu_all, (slice + 1) * per);
  const uint32_t row_bytes = (uint32_t)K * Q / 8;
  const uint32_t gpr = (uint32_t)nblk >> gshift;
  const uint32_t rows = (uint32_t)std::min<int64_t>(S::kRows, N - n0);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + n0 * row_bytes, rows * row_bytes);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales + n0 * gpr, rows * gpr * 2);
  const uint8_t* const mp = static_cast<const uint8_t*>(meta);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(kMetaSize ? mp + n0 * gpr * kMetaSize : mp,
                                              kMetaSize ? rows * gpr * kMetaSize : 0u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2);

  uint8_t* const cs = cs_all + wave * S::kTileBytes;
  const int n = lane & 15, c = lane >> 4;       // MFMA operand row (or column) and 8-k chunk
  const int lrow = lane >> 3, lpiece = lane & 7;
  struct Codes {
    uint32_t d[RT][2][Q];
    uint32_t s[RT][2], z[RT][2];
  };
  auto issue_c = [&](int u, Codes& t) {
    const int blk = 8 * u + lpiece;
    const uint32_t past = u < u_end ? 0u : kOutOfRange;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t row = (uint32_t)(16 * rt + 8 * h + lrow);
        buffer_block_codes<Q>(rc, (row * row_bytes + (uint32_t)blk * (4 * Q)) | past, 0, t.d[rt][h]);
        const uint32_t gi = row * gpr + (uint32_t)(blk >> gshift);
        t.s[rt][h] = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)((gi * 2) | past), 0, 0);
        if constexpr (META == kMetaZp) t.z[rt][h] = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)(gi | past), 0, 0);
        if constexpr (META == kMetaMin) t.z[rt][h] = __builtin_amdgcn_raw_buffer_load_b16(rz, (int)((gi * 2) | past), 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Activations of k [128 sb, 128 sb + 128) into stage `idx`: four tokens of 256 bytes a load.
  auto issue_x = [&](int sb, auto idx) {
    uint8_t* const st = stage_of(idx) + wave * S::kStageBytes;
#pragma unroll
    for (int j = 0; j < TOK / 4; ++j) {
      const int m = 4 * j + (lane >> 4);
      const int piece = (lane & 15) ^ m;
      const uint32_t off = (((uint32_t)m * (uint32_t)K + (uint32_t)sb * 128 + 8 * piece) * 2) | (sb < 2 * u_end ? 0u : kOutOfRange);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(st + j * 1024), 16, (int)off, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x4 acc[RT][MB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) acc[rt][0] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t mask = opaque_s(code_mask<Q>()), magic = opaque_v(0x43004300u);
  const int am = TOK == 8 ? n & 7 : n;

  // Row tile rt's codes, scales and metadata to this wavefront's LDS buffer (rows of 32q
  // bytes, pieces of one block swizzled so that 16 rows' reads touch every bank once).
  auto store_tile = [&](const Codes& t, int rt) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = 8 * h + lrow;
      const uint32_t (&d)[Q] = t.d[rt][h];
      if constexpr (Q == 4) *reinterpret_cast<u32x4*>(cs + row * 128 + ((lpiece ^ ((row >> 1) & 7)) << 4)) = u32x4{d[0], d[1], d[2], d[3]};
      else *reinterpret_cast<u32x2*>(cs + row * 64 + ((lpiece ^ ((row >> 2) & 7)) << 3)) = u32x2{d[0], d[1]};
      *reinterpret_cast<uint16_t*>(cs + S::kCodeBytes + row * 16 + 2 * lpiece) = (uint16_t)t.s[rt][h];
      if constexpr (META != kMetaNone) *reinterpret_cast<uint16_t*>(cs + S::kCodeBytes + 256 + row * 16 + 2 * lpiece) = (uint16_t)t.z[rt][h];
    }
  };

  // Unit u (P0: its first stage's index): half by half, row tile by row tile; the next
  // tile's codes go to LDS while this one is multiplied.  The next loads go out at the
  // end, activations first: loads return in order, and they are needed first.
  auto unit = [&](int u, Codes& t, auto p0, bool next) {
    constexpr int P0 = decltype(p0)::value;
    auto half = [&](auto sc_) {
      constexpr int s = decltype(sc_)::value;
      wave_sync();
      store_tile(t, 0);
      bf16x8 a[4];
      f32x4 d0[4];
      const uint8_t* const xw = stage_of(std::integral_constant<int, P0 + s>{}) + wave * S::kStageBytes;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(xw + am * 256 + (((4 * j + c) ^ am) << 4));
        constexpr uint32_t kLo = 0x05040100u, kHi = 0x07060302u;
        a[j] = __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_perm(v.z, v.x, kLo), __builtin_amdgcn_perm(v.z, v.x, kHi),
                                                __builtin_amdgcn_perm(v.w, v.y, kLo), __builtin_amdgcn_perm(v.w, v.y, kHi)});
      }
      // -(128 + o) xs[m] in every column (o = 0 where a group has a zero point or a minimum)
      constexpr uint32_t kOff = META != kMetaNone ? 0xC300C300u : 0xC300C300u | ((1u << (Q - 1)) * 0x00010001u);
      const bf16x8 off = __builtin_bit_cast(bf16x8, u32x4{kOff, kOff, kOff, kOff});
#pragma unroll
      for (int j = 0; j < 4; ++j) d0[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], off, zero4, 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        wave_sync();
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int blk = 4 * s + j;
          if constexpr (Q == 4) w[j] = *reinterpret_cast<const uint32_t*>(cs + n * 128 + ((blk ^ ((n >> 1) & 7)) << 4) + 4 * c);
          else w[j] = *reinterpret_cast<const uint16_t*>(cs + n * 64 + ((blk ^ ((n >> 2) & 7)) << 3) + 2 * c);
        }
        const u32x2 sh = *reinterpret_cast<const u32x2*>(cs + S::kCodeBytes + n * 16 + 8 * s);
        u32x2 zh = {0u, 0u};
        if constexpr (META != kMetaNone) zh = *reinterpret_cast<const u32x2*>(cs + S::kCodeBytes + 256 + n * 16 + 8 * s);
        if (rt + 1 < RT) {             // the buffer is free once its reads are queued: LDS serves a wavefront in order
          wave_sync();
          store_tile(t, rt + 1 < RT ? rt + 1 : rt);
        }
        f32x4 d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bf16x8 b = code_pairs<Q>(w[j], mask, magic);
          f32x4 base = d0[j];
          if constexpr (META == kMetaZp) {       // -z: every byte is exact in bf16, as -(128 + z) is not
            const uint32_t zp2 = j < 2 ? zh.x : zh.y;
            const uint32_t zb = __float_as_uint((float)((j & 1) ? (zp2 >> 16) & 0xFFu : zp2 & 0xFFu));
            const uint32_t zz = 0x80008000u | __builtin_amdgcn_perm(0u, zb, 0x03020302u);
            base = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], __builtin_bit_cast(bf16x8, u32x4{zz, zz, zz, zz}), base, 0, 0, 0);
          }
          d[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], b, base, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t sp = j < 2 ? sh.x : sh.y;
          const float sc = (j & 1) ? f16_hi(sp) : f16_lo(sp);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[rt][0][r] = __builtin_fmaf(sc, d[j][r], acc[rt][0][r]);
          if constexpr (META == kMetaMin) {
            const uint32_t mp2 = j < 2 ? zh.x : zh.y;
            const float mm = ((j & 1) ? f16_hi(mp2) : f16_lo(mp2)) * -0.0078125f;   // d0 = -128 xs
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rt][0][r] = __builtin_fmaf(mm, d0[j][r], acc[rt][0][r]);
          }
        }
      }
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, 1>{});
    // every LDS read of the stages has returned: a load that hits the cache could overtake it
    __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    if (next) {
      issue_x(2 * (u + 2 * W), std::integral_constant<int, P0>{});
      issue_x(2 * (u + 2 * W) + 1, std::integral_constant<int, P0 + 1>{});
      issue_c(u + 2 * W, t);
    }
  };

  // Units of this wavefront: u0, u0 + W, ...; two units' loads in flight.
  const int u0 = slice * per + wave;
  Codes c0, c1;
  issue_x(2 * u0, std::integral_constant<int, 0>{});
  issue_x(2 * u0 + 1, std::integral_constant<int, 1>{});
  issue_c(u0, c0);
  issue_x(2 * (u0 + W), std::integral_constant<int, 2>{});
  issue_x(2 * (u0 + W) + 1, std::integral_constant<int, 3>{});
  issue_c(u0 + W, c1);
  int u = u0;
  for (; u + 2 * W < u_end; u += 2 * W) {
    unit(u, c0, std::integral_constant<int, 0>{}, true);
    unit(u + W, c1, std::integral_constant<int, 2>{}, true);
  }
  if (u < u_end) unit(u, c0, std::integral_constant<int, 0>{}, false);
  if (u + W < u_end) unit(u + W, c1, std::integral_constant<int, 2>{}, false);

  // The wavefronts' partial sums meet in LDS row tile by row tile, in wavefront order.
  wait_vmcnt<0>();
  __syncthreads();
  constexpr int kTF = S::kTileFloats;
  constexpr int kSc1 = 16;
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(partials + (int64_t)rb * slices * (RT * kTF), slices > 1 ? (uint32_t)slices * (RT * kTF * 4) : 0u);
  auto put = [&](int rt, int e, float v) {
    const int mb = e >> 8, l = (e & 255) >> 2, r = e & 3;
    const int m = 16 * mb + 4 * (l >> 4) + r;
    const int64_t row = n0 + 16 * rt + (l & 15);
    if (m < M && row < N) y[(int64_t)m * N + row] = f32_to_bf16_bits(v);
  };
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float* const part = reinterpret_cast<float*>((rt & 1) == 0 ? xs0 : xs1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(part + wave * kTF + mb * 256 + 4 * lane) = acc[rt][mb];
    __syncthreads();
    for (int e = tid; e < kTF; e += 64 * W) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) v += part[w * kTF + e];
      if (slices == 1) put(rt, e, v);
      else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rp, ((slice * RT + rt) * kTF + e) * 4, 0, kSc1);
    }
  }
  if (slices == 1) return;
  unsigned int* const arrived = reinterpret_cast<unsigned int*>(cs_all);
  wait_vmcnt<0>();
  __syncthreads();
  if (tid == 0) *arrived = atomicAdd(&counters[rb], 1u);
  __syncthreads();
  if (*arrived != (unsigned int)(slices - 1)) return;
  for (int e = 4 * tid; e < RT * kTF; e += 256 * W) {
    f32x4 v = zero4;
    for (int s0 = 0; s0 < slices; s0 += 4) {
      f32x4 p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        p[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             rp, s0 + i < slices ? ((s0 + i) * (RT * kTF) + e) * 4 : (int)kOutOfRange, 0, kSc1));
#pragma unroll
      for (int i = 0; i < 4; ++i) v += p[i];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) put(e / kTF, e % kTF + r, v[r]);
  }
  if (tid == 0) __hip_atomic_store(&counters[rb], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int Q, int META, int TOK, int RT>
__global__ __launch_bounds__(64 * kWaves) void stream_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
    const void* __restrict__ meta, int M, int N, int K, int gshift, int slices, uint16_t* __restrict__ y,
    float* __restrict__ partials, unsigned int* __restrict__ counters) {
  using S = Stream<Q, META, TOK, RT>;
  constexpr int W = kWaves, XB = S::XB, MB = S::MB;
  constexpr int kMetaSize = META == kMetaZp ? 1 : META == kMetaMin ? 2 : 0;
  // Each activation stage its own LDS object: the compiler then waits for exactly the
  // direct-to-LDS loads of the stage it reads.
  uint8_t* const xs0 = lds_object<0, W * S::kStageBytes>();
  uint8_t* const xs1 = lds_object<1, W * S::kStageBytes>();
  uint8_t* const cs_all = lds_object<2, W * RT * S::kTileBytes>();
  uint8_t* const ss_all = lds_object<3, W * RT * S::kScaleBytes>();
  uint8_t* const zs_all = lds_object<4, META != kMetaNone ? W * RT * S::kScaleBytes : 16>();

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = (int)blockIdx.x % slices, rb = (int)blockIdx.x / slices;
  const int64_t n0 = (int64_t)rb * S::kRows;
  const int nblk = K / 32;
  const int nu_all = (nblk + 7) / 8, per = (nu_all + slices - 1) / slices;
  const int u_end = std::min(nu_all, (slice + 1) * per);
  const uint32_t row_bytes = (uint32_t)K * Q / 8;
  const uint32_t gpr = (uint32_t)nblk >> gshift;
  const uint32_t rows = (uint32_t)std::min<int64_t>(S::kRows, N - n0);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + n0 * row_bytes, rows * row_bytes);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales + n0 * gpr, rows * gpr * 2);
  const uint8_t* const mp = static_cast<const uint8_t*>(meta);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(kMetaSize ? mp + n0 * gpr * kMetaSize : mp,
                                              kMetaSize ? rows * gpr * kMetaSize : 0u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2);

  uint8_t* const cs0 = cs_all + wave * RT * S::kTileBytes;
  uint8_t* const ss0 = ss_all + wave * RT * S::kScaleBytes;
  uint8_t* const zs0 = META != kMetaNone ? zs_all + wave * RT * S::kScaleBytes : zs_all;
  const int n = lane & 15, c = lane >> 4;       // MFMA operand row (or column) and 8-k chunk
  const int lrow = lane >> 3, lpiece = lane & 7;

  struct Codes {
    uint32_t d[RT][2][Q];
    uint32_t s[RT][2], z[RT][2];
  };
  // Codes, scales and metadata of unit u (blocks 8u..8u+7): lane -> (row lane / 8, block
  // lane % 8) of half a row tile, 128 contiguous bytes a row at q = 4.  Past the row bit 31
  // is set, out of every descriptor's range (a select would become a branch around the loads).
  auto issue_c = [&](int u, Codes& t) {
    const int blk = 8 * u + lpiece;
    const uint32_t past = (blk < nblk) & (u < u_end) ? 0u : kOutOfRange;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t row = (uint32_t)(16 * rt + 8 * h + lrow);
        buffer_block_codes<Q>(rc, (row * row_bytes + (uint32_t)blk * (4 * Q)) | past, 0, t.d[rt][h]);
        const uint32_t gi = row * gpr + (uint32_t)(blk >> gshift);
        t.s[rt][h] = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)((gi * 2) | past), 0, 0);
        if constexpr (META == kMetaZp) t.z[rt][h] = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)(gi | past), 0, 0);
        if constexpr (META == kMetaMin) t.z[rt][h] = __builtin_amdgcn_raw_buffer_load_b16(rz, (int)((gi * 2) | past), 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Activations of stage `st` of unit u (XB blocks) into stage object P.  Lane L of load i
  // fills position L % (4 XB) of its token's row, which holds piece pos ^ swizzle(token):
  // 16 lanes that read one piece of 16 tokens then touch every bank once.
  auto swizzle = [&](int m) { return XB == 4 ? (m & 15) : XB == 2 ? ((m >> 1) & 7) : ((m >> 2) & 3); };
  constexpr int kPieces = 4 * XB;
  auto issue_x = [&](int u, int st, auto idx) {
    uint8_t* const base = (decltype(idx)::value == 0 ? xs0 : xs1) + wave * S::kStageBytes;
    const int blk0 = 8 * u + XB * st;
#pragma unroll
    for (int i = 0; i < S::kXLoads; ++i) {
      const int m = (64 / kPieces) * i + lane / kPieces;
      const int piece = (lane % kPieces) ^ swizzle(m);
      const uint32_t past = (blk0 + (piece >> 2) < nblk) & (u < u_end) ? 0u : kOutOfRange;
      const uint32_t off = (((uint32_t)m * (uint32_t)K + (uint32_t)blk0 * 32 + 8 * piece) * 2) | past;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(base + i * 1024), 16, (int)off, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x4 acc[RT][MB];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[rt][mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t mask = opaque_s(code_mask<Q>()), magic = opaque_v(0x64006400u);
  const uint32_t mask_hi = opaque_s(code_mask<Q>() << Q);
  // LDS address of this lane's code bytes: row n, 16-byte pieces XOR-swizzled with n / 2
  // (q = 4; the rows of q = 2 are swizzled alike in 8-byte pieces, q = 3 rows are padded).
  auto code_at = [&](const uint8_t* cs, int blk) -> const uint8_t* {
    if constexpr (Q == 3) return cs + n * S::kCodePitch + 12 * blk;
    else return cs + n * S::kCodePitch + ((blk ^ ((n >> (Q == 4 ? 1 : 2)) & 7)) * (4 * Q));
  };
  auto store_codes = [&](const Codes& t) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint8_t* const cs = cs0 + rt * S::kTileBytes;
        const int row = 8 * h + lrow;
        const uint32_t (&d)[Q] = t.d[rt][h];
        if constexpr (Q == 4) {
          *reinterpret_cast<u32x4*>(cs + row * S::kCodePitch + ((lpiece ^ ((row >> 1) & 7)) << 4)) = u32x4{d[0], d[1], d[2], d[3]};
        } else if constexpr (Q == 2) {
          *reinterpret_cast<u32x2*>(cs + row * S::kCodePitch + ((lpiece ^ ((row >> 2) & 7)) << 3)) = u32x2{d[0], d[1]};
        } else {
#pragma unroll
          for (int i = 0; i < 3; ++i) *reinterpret_cast<uint32_t*>(cs + row * S::kCodePitch + 12 * lpiece + 4 * i) = d[i];
        }
        const int at = rt * S::kScaleBytes + row * S::kScalePitch + 2 * lpiece;
        *reinterpret_cast<uint16_t*>(ss0 + at) = (uint16_t)t.s[rt][h];
        if constexpr (META != kMetaNone) *reinterpret_cast<uint16_t*>(zs0 + at) = (uint16_t)t.z[rt][h];
      }
  };

  // Unit u: its codes from registers to LDS, the next unit's loads into the registers, then
  // stage by stage; a stage's successor but one is requested once its operands are read.
  auto unit = [&](int u, Codes& t) {
    wave_sync();
    store_codes(t);
    wave_sync();
    __builtin_amdgcn_sched_barrier(0);
    issue_c(u + W, t);
    auto step = [&](auto stc) {
      constexpr int st = decltype(stc)::value;
      const uint8_t* const xw = ((st & 1) == 0 ? xs0 : xs1) + wave * S::kStageBytes;
      bf16x8 a[XB][MB];
#pragma unroll
      for (int j = 0; j < XB; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const int m = 16 * mb + n;
          a[j][mb] = *reinterpret_cast<const bf16x8*>(xw + m * S::kRowBytes + (((XB * c + j) ^ swizzle(n)) << 4));
        }
      __builtin_amdgcn_sched_barrier(0);
      // This stage's operands are in registers (waited for: a load that hits the cache could
      // overtake LDS reads still queued): its object takes the stage after the next.
      __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0)
      if constexpr (st + 2 < S::kSteps) issue_x(u, st + 2, std::integral_constant<int, st & 1>{});
      else issue_x(u + W, st + 2 - S::kSteps, std::integral_constant<int, st & 1>{});
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const uint8_t* const cs = cs0 + rt * S::kTileBytes;
        const uint8_t* const sp = ss0 + rt * S::kScaleBytes + n * S::kScalePitch;
        const uint8_t* const zp = zs0 + rt * S::kScaleBytes + n * S::kScalePitch;
          // this lane's 8 XB weights: stage bytes c * XB * Q on, one block's
          const int blk = XB * st + (XB * c) / 4, part = (XB * c) % 4;        // in 8-weight parts
          const uint8_t* const p = code_at(cs, blk) + part * Q;
          uint32_t w[XB];
          if constexpr (Q == 4) {
            if constexpr (XB == 4) { const u32x4 v = *reinterpret_cast<const u32x4*>(p); w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
            else if constexpr (XB == 2) { const u32x2 v = *reinterpret_cast<const u32x2*>(p); w[0] = v.x; w[1] = v.y; }
            else w[0] = *reinterpret_cast<const uint32_t*>(p);
          } else if constexpr (Q == 2) {
            if constexpr (XB == 4) { const u32x2 v = *reinterpret_cast<const u32x2*>(p); w[0] = v.x & 0xFFFFu; w[1] = v.x >> 16; w[2] = v.y & 0xFFFFu; w[3] = v.y >> 16; }
            else if constexpr (XB == 2) { const uint32_t v = *reinterpret_cast<const uint32_t*>(p); w[0] = v & 0xFFFFu; w[1] = v >> 16; }
            else w[0] = *reinterpret_cast<const uint16_t*>(p);
          } else {
            const uint32_t sh = (uint32_t)(part * 3) & 3u;                     // the dwords from the one at or below p
            const uint32_t* const w32 = reinterpret_cast<const uint32_t*>(p - sh);
            if constexpr (XB == 4) {
              const uint32_t v0 = w32[0], v1 = w32[1], v2 = w32[2];
              w[0] = v0; w[1] = __builtin_amdgcn_alignbit(v1, v0, 24); w[2] = __builtin_amdgcn_alignbit(v2, v1, 16); w[3] = v2 >> 8;
            } else {
              const uint32_t v0 = w32[0], v1 = w32[1];
              w[0] = __builtin_amdgcn_alignbit(v1, v0, 8 * sh);
              if constexpr (XB == 2) w[1] = (uint32_t)((((uint64_t)v1 << 32) | v0) >> (8 * sh + 24));
            }
          }
          const float s = f16_bits_to_f32(*reinterpret_cast<const uint16_t*>(sp + 2 * blk));
          const uint32_t zb = META != kMetaNone ? (uint32_t)*reinterpret_cast<const uint16_t*>(zp + 2 * blk) : 0u;
          const float sc[2] = {s, s * (1.0f / (float)(1 << Q))};
          const float so[2] = {dequant_offset<META, Q>(s, zb), dequant_offset_hi<META, Q>(s, zb)};
#pragma unroll
          for (int j = 0; j < XB; ++j) {
            const bf16x8 b = dequant8<Q>(w[j], sc, so, mask, mask_hi, magic);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
              acc[rt][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][mb], b, acc[rt][mb], 0, 0, 0);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    if constexpr (S::kSteps >= 4) { step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{}); }
    if constexpr (S::kSteps >= 8) {
      step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
      step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 7>{});
    }
  };

  // Units of this wavefront: u0, u0 + W, ... (loads past the last move nothing)
  const int u0 = slice * per + wave;
  issue_x(u0, 0, std::integral_constant<int, 0>{});
  issue_x(u0, 1, std::integral_constant<int, 1>{});
  Codes c0;
  issue_c(u0, c0);
  for (int u = u0; u < u_end; u += W) unit(u, c0);

  // The wavefronts' partial sums meet in LDS row tile by row tile, in wavefront order.
  wait_vmcnt<0>();
  __syncthreads();
  constexpr int kTF = S::kTileFloats;
  constexpr int kSc1 = 16;
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(partials + (int64_t)rb * slices * (RT * kTF), slices > 1 ? (uint32_t)slices * (RT * kTF * 4) : 0u);
  auto put = [&](int rt, int e, float v) {
    const int mb = e >> 8, l = (e & 255) >> 2, r = e & 3;
    const int m = 16 * mb + 4 * (l >> 4) + r;
    const int64_t row = n0 + 16 * rt + (l & 15);
    if (m < M && row < N) y[(int64_t)m * N + row] = f32_to_bf16_bits(v);
  };
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float* const part = reinterpret_cast<float*>((rt & 1) == 0 ? xs0 : xs1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(part + wave * kTF + mb * 256 + 4 * lane) = acc[rt][mb];
    __syncthreads();
    for (int e = tid; e < kTF; e += 64 * W) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) v += part[w * kTF + e];
      if (slices == 1) put(rt, e, v);
      else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rp, ((slice * RT + rt) * kTF + e) * 4, 0, kSc1);
    }
  }
  if (slices == 1) return;
  unsigned int* const arrived = reinterpret_cast<unsigned int*>(cs_all);
  wait_vmcnt<0>();
  __syncthreads();
  if (tid == 0) *arrived = atomicAdd(&counters[rb], 1u);
  __syncthreads();
  if (*arrived != (unsigned int)(slices - 1)) return;
  for (int e = 4 * tid; e < RT * kTF; e += 256 * W) {
    f32x4 v = zero4;
    for (int s0 = 0; s0 < slices; s0 += 4) {
      f32x4 p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        p[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                             rp, s0 + i < slices ? ((s0 + i) * (RT * kTF) + e) * 4 : (int)kOutOfRange, 0, kSc1));
#pragma unroll
      for (int i = 0; i < 4; ++i) v += p[i];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) put(e / kTF, e % kTF + r, v[r]);
  }
  if (tid == 0) __hip_atomic_store(&counters[rb], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int Q, int META, int TOK, int RT>
hipError_t exact_launch(const uint16_t* x, int64_t M, const uint8_t* codes, const uint16_t* scales, const void* meta,
                        int64_t N, int64_t K, int gshift, int slices, uint16_t* y, float* partials,
                        unsigned int* counters, hipStream_t stream) {
  const int64_t rbs = (N + 16 * RT - 1) / (16 * RT);
  stream_exact_kernel<Q, META, TOK, RT><<<dim3((unsigned)(rbs * slices)), 64 * kWaves, 0, stream>>>(
      x, codes, scales, meta, (int)M, (int)N, (int)K, gshift, slices, y, partials, counters);
  return hipGetLastError();
}

template <int Q, int META, int TOK, int RT>
hipError_t stream_launch(const uint16_t* x, int64_t M, const uint8_t* codes, const uint16_t* scales, const void* meta,
                         int64_t N, int64_t K, int gshift, int slices, uint16_t* y, float* partials,
                         unsigned int* counters, hipStream_t stream) {
  const int64_t rbs = (N + 16 * RT - 1) / (16 * RT);
  stream_kernel<Q, META, TOK, RT><<<dim3((unsigned)(rbs * slices)), 64 * kWaves, 0, stream>>>(
      x, codes, scales, meta, (int)M, (int)N, (int)K, gshift, slices, y, partials, counters);
  return hipGetLastError();
}


// Whether an instantiation's LDS fits (rows kernels take 160 KB at most).
template <int Q, int META, int TOK, int RT>
constexpr bool stream_fits() {
  using S = Stream<Q, META, TOK, RT>;
  return kWaves * (2 * S::kStageBytes + RT * (S::kTileBytes + S::kScaleBytes * (META != kMetaNone ? 2 : 1))) +
             (META != kMetaNone ? 0 : 16) <= 163840;
}

// What a launch is given (stream.hip fills it in).
struct StreamArgs {
  const uint16_t* x;
  int64_t M;
  const uint8_t* codes;
  const uint16_t* scales;
  const void* meta;
  int64_t N, K;
  int gshift, slices;
  uint16_t* y;
  float* partials;
  unsigned int* counters;
  hipStream_t stream;
};

template <int Q, int META, int TOK, int RT>
hipError_t rounded_rt(const StreamArgs& a) {
  return stream_launch<Q, META, TOK, RT>(a.x, a.M, a.codes, a.scales, a.meta, a.N, a.K, a.gshift, a.slices, a.y,
                                         a.partials, a.counters, a.stream);
}
template <int Q, int META, int TOK>
hipError_t rounded_tok(const StreamArgs& a, int rt) {
  switch (rt) {
    case 1: return rounded_rt<Q, META, TOK, 1>(a);
    case 2: return rounded_rt<Q, META, TOK, 2>(a);
    case 3: if constexpr (TOK <= 32 || !stream_fits<Q, META, TOK, 4>()) return rounded_rt<Q, META, TOK, 3>(a); break;
    case 4: if constexpr (stream_fits<Q, META, TOK, 4>()) return rounded_rt<Q, META, TOK, 4>(a); break;
    case 5: if constexpr (TOK == 32 && stream_fits<Q, META, TOK, 5>()) return rounded_rt<Q, META, TOK, 5>(a); break;
  }
  return hipErrorInvalidValue;
}
template <int Q, int META>
hipError_t rounded_any(const StreamArgs& a, int tok, int rt) {
  switch (tok) {
    case 16: return rounded_tok<Q, META, 16>(a, rt);
    case 32: return rounded_tok<Q, META, 32>(a, rt);
    case 48: return rounded_tok<Q, META, 48>(a, rt);
    case 64: return rounded_tok<Q, META, 64>(a, rt);
    case 80: return rounded_tok<Q, META, 80>(a, rt);
  }
  return hipErrorInvalidValue;
}
template <int Q>
hipError_t rounded_q(const StreamArgs& a, int kind, int tok, int rt) {
  return kind == kMetaNone ? rounded_any<Q, kMetaNone>(a, tok, rt)
       : kind == kMetaZp ? rounded_any<Q, kMetaZp>(a, tok, rt) : rounded_any<Q, kMetaMin>(a, tok, rt);
}

template <int Q, int META, int TOK>
hipError_t exact_tok(const StreamArgs& a, int rt) {
  auto go = [&](auto rtc) {
    return exact_launch<Q, META, TOK, decltype(rtc)::value>(a.x, a.M, a.codes, a.scales, a.meta, a.N, a.K, a.gshift,
                                                            a.slices, a.y, a.partials, a.counters, a.stream);
  };
  switch (rt) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
  }
  return hipErrorInvalidValue;
}
template <int Q, int META>
hipError_t exact_any(const StreamArgs& a, int tok, int rt) {
  return tok == 8 ? exact_tok<Q, META, 8>(a, rt) : tok == 16 ? exact_tok<Q, META, 16>(a, rt) : hipErrorInvalidValue;
}

}  // namespace stream
}  // namespace ssq
