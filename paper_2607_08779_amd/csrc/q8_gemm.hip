// Q8_0 matmul for several tokens: y[M,N] from quantized activations and packed weights,
// on int8 MFMA (v_mfma_i32_32x32x32_i8).
//
// App. B.3 of the paper: for each block b of 32 activations inside weight group g,
//   y[m,n] += d[m,b] s[n,g] (I - o[n,g] R),  I = sum q u,  R = sum q  (exact integers),
// or d (s I + m R) for the binary16-minimum layout.
//
// What bounds it.  A scale per 32 activations and one per 32 weights: each int32 result
// of a block (one MFMA is one block deep) needs two vector instructions before it joins
// the fp32 sum, 32 per lane and 32x32 tile against 26 ns of MFMA, so many tokens are
// vector-ALU bound and few tokens latency bound (a stage's loads, LDS round trip and
// barrier).  The two convert I - o R to binary32 (exactly) and add it times d s.  The
// products d s of a block come from an MFMA of their own, v_mfma_f32_32x32x8_f16 with the
// scales in one of four k and zeros in the others: exact, so a block term is rounded once,
// by the fma that adds it, and an infinite scale gives the infinity that it gives in the
// one-token kernel (q8.hip).  Both halves of the wavefront hold the scale, so the product is
// 2 d s, and the sum is halved at the end.  Forming t = s (I - o R) first, as
// s (1.5 * 2^23 + I - o R) - s 1.5 * 2^23, takes no MFMA and the same vector instructions,
// but makes NaN of an infinite s and rounds t where |I - o R| passes 2^13.  The minimum layout's
// d (s I + m R) takes four vector instructions, rounded as in the one-token kernel.  A
// symmetric format's offset joins the start value through one more MFMA (the activations
// against constant bytes -o), shared by a wavefront's column tiles; a zero point is
// subtracted from the code bytes.
//
// Sums: chains of 8 blocks (16 from K = 4640 on), added in turn, then the K-groups as a tree.
// Their error against 64 bits is that of 16 chains of K / 512 blocks (2-norm of the
// binary32 sums, K = 4096 / 14336: 8.8e-8 / 1.1e-7 for 8.8e-8 / 1.2e-7); one chain a K-group
// has 1.4e-7 / 2.5e-7 at two K-groups, and rounds 1.5 times as many outputs to the wrong
// bf16 neighbour.  The second set of sums leaves registers for two column tiles a wavefront,
// so the widest tiles have two wavefronts side by side: 512 tokens on 4096x14336 110 us for
// 102 with single chains and four column tiles, on 14336x4096 120 for 110.
//
// Work split.  A workgroup of 8 wavefronts owns a tile of 32 WM tokens x 32 WN TC outputs and
// the whole reduction, as 8 / (WM WN) K-groups; a wavefront covers 32 tokens and TC column
// tiles.  A stage is SB blocks: the activation
// codes go straight to LDS, the weight codes through registers, where each block is
// unpacked once for the whole tile, and the scales beside them.  The next stage's
// activations and the stage after that's weights are in flight while a stage is
// multiplied.  With the weights one stage ahead only, a 32x32 tile took 16.1 us at K = 4096
// (0.95 us a stage, the loads' latency) against 11.2.
//
// Up to 16 tokens a 32-token tile leaves out the sums of tokens 16 to 31, half of its vector work,
// and two 32x32 tiles share a CU: 8 tokens on 12288x4096 13.9 us for 15.7, on 4096x12288 19.3 for
// 23.1.
//
// Measured (W4 g32 signed, graph replays; the kernel this replaces read the weights once
// per 32 tokens on 16x16x32 MFMA): 512 tokens on 4096x14336 110 us (709 before), on
// 14336x4096 120 (870); 64 tokens on 4096x4096 10.7 (30), 8 tokens on 12288x4096 13.9 (33), on
// 4096x4096 9.0 (11.8).  That kernel had 16 rows a workgroup and is missed where few tokens meet
// fewer than 128 tiles and a long K: 14 tokens on W3 4096x30208 with minimums 64 for 42, 8 on
// 3593x12288 27 for 20; 3 % of 500 random sizes of 2 to 40 tokens.
#include <algorithm>
#include <type_traits>

#include "mfma_dequant.h"
#include "ssq_internal.h"

namespace ssq {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr uint32_t kOutOfRange = 0x80000000u;   // past every buffer's size: loads return 0
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
// The int32 accumulators start at the bits of 1.5 * 2^23, so that an accumulator read as
// binary32 is 1.5 * 2^23 + I exactly (|I| < 2^17) and one subtraction converts it.
constexpr uint32_t kMagicBits = 0x4B400000u;
constexpr float kMagic = 12582912.0f;

// SB: 32-k blocks of a stage.
template <int META, int WM, int WN, int TC, int SB>
struct Q8Cfg {
  static constexpr int kStageBlocks = SB;
  static constexpr int BM = 32 * WM, BN = 32 * TC * WN;
  static constexpr int KG = kWaves / (WM * WN);                // K-groups
  static constexpr int NB = kStageBlocks / KG;                 // blocks of a stage per K-group
  static constexpr int kABytes = BM * kStageBlocks * 32;       // activation codes of a stage
  static constexpr int kBBytes = BN * kStageBlocks * 32;       // weight codes, a byte each
  // token scales [block][row]: binary16 for the MFMA that multiplies them with the weights',
  // binary32 in the minimum layout; weight scales (and minimums) alike [block][column]
  static constexpr int kScaleSize = META == kMetaMin ? 4 : 2;
  static constexpr int kDBytes = BM * kStageBlocks * kScaleSize;
  static constexpr int kSBytes = BN * kStageBlocks * kScaleSize;
  static constexpr int kALoads = kABytes / 1024 / kWaves;      // per wavefront
  static constexpr int kBItems = BN * kStageBlocks;            // weight blocks of a stage
  static constexpr int kBPer = (kBItems + kThreads - 1) / kThreads;
  static constexpr int kDItems = BM * kStageBlocks;
  static constexpr int kDPer = (kDItems + kThreads - 1) / kThreads;
};

// 16 unsigned fields (a half-block) as 16 bytes in the k order of act_order<Q>.
template <int Q>
__device__ __forceinline__ u32x4 unpack16(uint32_t v0, uint32_t v1) {   // 8 fields each, from bit 0
  uint32_t o[4];
  const uint32_t v[2] = {v0, v1};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (Q == 4) {
      o[2 * i] = v[i] & 0x0F0F0F0Fu;
      o[2 * i + 1] = (v[i] >> 4) & 0x0F0F0F0Fu;
    } else if constexpr (Q == 2) {
      const uint32_t x = ((v[i] << 12) & 0x0FFF0000u) | (v[i] & 0xFFFFu);
      o[2 * i] = x & 0x03030303u;
      o[2 * i + 1] = (x >> 2) & 0x03030303u;
    } else {
      const uint32_t s = (v[i] & 0xFFFu) | ((v[i] << 4) & 0x0FFF0000u);
      o[2 * i] = (s & 0x00070007u) | (((s >> 3) & 0x00070007u) << 8);
      o[2 * i + 1] = ((s >> 6) & 0x00070007u) | (((s >> 9) & 0x00070007u) << 8);
    }
  }
  return u32x4{o[0], o[1], o[2], o[3]};
}
// 16 activation bytes in the same order: per 8, q = 4 [0 2 4 6 | 1 3 5 7], q = 2
// [0 4 2 6 | 1 5 3 7], q = 3 [0 1 4 5 | 2 3 6 7].
template <int Q>
__device__ __forceinline__ i32x4 act_order(const u32x4 x) {
  constexpr uint32_t kLo = Q == 4 ? 0x06040200u : Q == 2 ? 0x06020400u : 0x05040100u;
  constexpr uint32_t kHi = Q == 4 ? 0x07050301u : Q == 2 ? 0x07030501u : 0x07060302u;
  return i32x4{(int)__builtin_amdgcn_perm(x.y, x.x, kLo), (int)__builtin_amdgcn_perm(x.y, x.x, kHi),
               (int)__builtin_amdgcn_perm(x.w, x.z, kLo), (int)__builtin_amdgcn_perm(x.w, x.z, kHi)};
}
// bytes u - z of unsigned fields u <= 15 and a zero point z <= 15 (z in every byte of zz)
__device__ __forceinline__ uint32_t sub_bytes(uint32_t u, uint32_t zz) {
  return ((u | 0x80808080u) - zz) ^ 0x80808080u;
}

// An LDS array of its own.
template <int I, int BYTES>
__device__ __forceinline__ uint8_t* lds_object() {
  __shared__ __attribute__((aligned(1024))) uint8_t mem[BYTES];
  return mem;
}

template <int Q, int META, int WM, int WN, int TC, int SB, bool HALF>
__global__ __launch_bounds__(kThreads, HALF && TC == 1 ? 4 : 2) void q8_gemm_kernel(
    const int8_t* __restrict__ qx, const uint16_t* __restrict__ dx, int M, const uint8_t* __restrict__ codes,
    const uint16_t* __restrict__ scales, const void* __restrict__ meta, int N, int K, int gshift,
    uint16_t* __restrict__ y) {
  using C = Q8Cfg<META, WM, WN, TC, SB>;
  constexpr int KG = C::KG, NB = C::NB, BM = C::BM, BN = C::BN, kStageBlocks = SB, kRow = 32 * SB;   // kRow: bytes of a stage row
  constexpr int kMetaSize = META == kMetaZp ? 1 : META == kMetaMin ? 2 : 0;
  constexpr bool MIN = META == kMetaMin;
  constexpr int kR = HALF ? 8 : 16;                    // results of a lane: those from 8 on are tokens 16..31
  uint8_t* const as0 = lds_object<0, C::kABytes>();
  uint8_t* const as1 = lds_object<1, C::kABytes>();
  uint8_t* const bs = lds_object<2, 2 * C::kBBytes>();
  using scale_t = std::conditional_t<MIN, float, uint16_t>;
  scale_t* const ds = reinterpret_cast<scale_t*>(lds_object<3, 2 * C::kDBytes>());
  scale_t* const ss = reinterpret_cast<scale_t*>(lds_object<4, 2 * C::kSBytes>());
  scale_t* const ms = reinterpret_cast<scale_t*>(lds_object<5, MIN ? 2 * C::kSBytes : 16>());
  auto scale_of = [](uint32_t bits) -> scale_t {
    if constexpr (MIN) return f16_bits_to_f32(bits);
    else return (uint16_t)bits;
  };
  constexpr int kDCount = C::kDBytes / sizeof(scale_t), kSCount = C::kSBytes / sizeof(scale_t);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM % WN, grp = wave / (WM * WN);
  const int tiles_m = (M + BM - 1) / BM;
  int b = (int)blockIdx.x;
  const int tiles = (int)gridDim.x;
  if (tiles % 8 == 0) b = (b % 8) * (tiles / 8) + b / 8;       // each XCD a contiguous run of tiles
  const int tm = b % tiles_m, tn = b / tiles_m;
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int nblk = K / 32, nstages = (nblk + kStageBlocks - 1) / kStageBlocks;
  const uint32_t row_bytes = (uint32_t)K * Q / 8;
  const uint32_t gpr = (uint32_t)nblk >> gshift;
  const uint32_t rows_m = (uint32_t)std::min<int64_t>(BM, M - m0), rows_n = (uint32_t)std::min<int64_t>(BN, N - n0);
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(qx + m0 * K, rows_m * (uint32_t)K);
  const __amdgpu_buffer_rsrc_t rd = make_rsrc(dx + m0 * nblk, rows_m * (uint32_t)nblk * 2);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + n0 * row_bytes, rows_n * row_bytes);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales + n0 * gpr, rows_n * gpr * 2);
  const uint8_t* const mp = static_cast<const uint8_t*>(meta);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(kMetaSize ? mp + n0 * gpr * kMetaSize : mp,
                                              kMetaSize ? rows_n * gpr * kMetaSize : 0u);

  // Activation codes of stage s, straight into LDS: rows of kRow bytes, 16-byte pieces
  // XOR-swizzled with the row so that an operand read of 16 rows touches every bank once.
  auto issue_a = [&](int s, uint8_t* st) {
#pragma unroll
    for (int i = 0; i < C::kALoads; ++i) {
      const int li = wave * C::kALoads + i;
      constexpr int kPieces = 2 * SB;
      const int m = (64 / kPieces) * li + lane / kPieces, piece = (lane % kPieces) ^ (m & 15);
      const int blk = kStageBlocks * s + (piece >> 1);
      const uint32_t off = ((uint32_t)m * (uint32_t)K + (uint32_t)(kStageBlocks * s) * 32 + 16 * piece) |
                           (blk < nblk ? 0u : kOutOfRange);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(st + li * 1024), 16, (int)off, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Weight codes, scales, metadata and token scales of a stage, through registers.
  struct Regs {
    uint32_t c[C::kBPer][Q];
    uint32_t s[C::kBPer], z[C::kBPer];
    uint32_t d[C::kDPer];
  };
  auto issue_b = [&](int s, Regs& t) {
#pragma unroll
    for (int i = 0; i < C::kBPer; ++i) {
      const int it = tid + i * kThreads;
      const int n = it / kStageBlocks, blk = kStageBlocks * s + it % kStageBlocks;
      const uint32_t past = (blk < nblk) & (it < C::kBItems) ? 0u : kOutOfRange;
      buffer_block_codes<Q>(rc, ((uint32_t)n * row_bytes + (uint32_t)blk * (4 * Q)) | past, 0, t.c[i]);
      const uint32_t gi = (uint32_t)n * gpr + (uint32_t)(blk >> gshift);
      t.s[i] = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)((gi * 2) | past), 0, 0);
      if constexpr (META == kMetaZp) t.z[i] = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)(gi | past), 0, 0);
      if constexpr (META == kMetaMin) t.z[i] = __builtin_amdgcn_raw_buffer_load_b16(rz, (int)((gi * 2) | past), 0, 0);
    }
#pragma unroll
    for (int i = 0; i < C::kDPer; ++i) {
      const int it = tid + i * kThreads;
      const int m = it / kStageBlocks, blk = kStageBlocks * s + it % kStageBlocks;
      const uint32_t past = (blk < nblk) & (it < C::kDItems) ? 0u : kOutOfRange;
      t.d[i] = __builtin_amdgcn_raw_buffer_load_b16(rd, (int)((((uint32_t)m * nblk + blk) * 2) | past), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto store_b = [&](const Regs& t, int buf) {
#pragma unroll
    for (int i = 0; i < C::kBPer; ++i) {
      const int it = tid + i * kThreads;
      if (C::kBItems % kThreads != 0 && it >= C::kBItems) break;
      const int n = it / kStageBlocks, j = it % kStageBlocks;
      uint32_t v[4];
      if constexpr (Q == 4) {
        v[0] = t.c[i][0]; v[1] = t.c[i][1]; v[2] = t.c[i][2]; v[3] = t.c[i][3];
      } else if constexpr (Q == 2) {
        v[0] = t.c[i][0] & 0xFFFFu; v[1] = t.c[i][0] >> 16; v[2] = t.c[i][1] & 0xFFFFu; v[3] = t.c[i][1] >> 16;
      } else {
        v[0] = t.c[i][0];
        v[1] = __builtin_amdgcn_alignbit(t.c[i][1], t.c[i][0], 24);
        v[2] = __builtin_amdgcn_alignbit(t.c[i][2], t.c[i][1], 16);
        v[3] = t.c[i][2] >> 8;
      }
      uint8_t* const row = bs + buf * C::kBBytes + n * kRow;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u32x4 o = unpack16<Q>(v[2 * h], v[2 * h + 1]);
        if constexpr (META == kMetaZp) {
          const uint32_t zz = __builtin_amdgcn_perm(0u, t.z[i], 0u);
          o = u32x4{sub_bytes(o.x, zz), sub_bytes(o.y, zz), sub_bytes(o.z, zz), sub_bytes(o.w, zz)};
        }
        *reinterpret_cast<u32x4*>(row + (((2 * j + h) ^ (n & 15)) << 4)) = o;
      }
      ss[buf * kSCount + j * BN + n] = scale_of(t.s[i]);
      if constexpr (MIN) ms[buf * kSCount + j * BN + n] = scale_of(t.z[i]);
    }
#pragma unroll
    for (int i = 0; i < C::kDPer; ++i) {
      const int it = tid + i * kThreads;
      if (C::kDItems % kThreads != 0 && it >= C::kDItems) break;
      ds[buf * kDCount + (it % kStageBlocks) * BM + it / kStageBlocks] = scale_of(t.d[i]);
    }
  };

  f32x16 acc[TC], tot[TC];                             // the chain of the moment, the finished chains
#pragma unroll
  for (int c = 0; c < TC; ++c)
#pragma unroll
    for (int r = 0; r < kR; ++r) acc[c][r] = tot[c][r] = 0.0f;
  auto fold = [&]() {
#pragma unroll
    for (int c = 0; c < TC; ++c)
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        tot[c][r] += acc[c][r];
        acc[c][r] = 0.0f;
      }
  };
  // Stages of a chain (a power of two): 8 blocks, 16 where the number of chains would count
  // for more.
  const int chain = std::max(1, (nblk <= 144 ? 8 : 16) / NB);
  const int lr = lane & 31, h = lane >> 5;
  // The int32 accumulators start at 0 and are converted, or (16 registers more) at the bits of
  // 1.5 * 2^23, so that read as binary32 they are 1.5 * 2^23 + I exactly (|I| < 2^17) and one
  // subtraction converts them: where the registers are free (at the start, 512 tokens on
  // 14336x4096, zero point, 125 us for 130; the 128x128 symmetric tile and the minimum layout
  // spill with it).
  constexpr bool kZero = MIN || (HALF && TC == 1) || (META == kMetaNone && WM * WN == 8);
  i32x16 start;
#pragma unroll
  for (int r = 0; r < 16; ++r) start[r] = kZero ? 0 : (int)kMagicBits;
  auto value = [](int v) { return kZero ? (float)v : __int_as_float(v) - kMagic; };

  // This K-group's blocks of a stage.  A lane's 16-byte piece of block j of any row lies at
  // row + piece0 ^ 32 j, formed as it is read (kept for every block, the addresses spill).
  const uint32_t piece0 = (uint32_t)((h ^ (lr & 15)) << 4);
  auto compute = [&](const uint8_t* as, int buf) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int j = grp * NB + k;                      // block of the stage
      const uint32_t piece = opaque_v(piece0) ^ (uint32_t)(32 * j);
      const i32x4 a = act_order<Q>(*reinterpret_cast<const u32x4*>(as + (wm * 32 + lr) * kRow + piece));
      const scale_t* const dj = ds + buf * kDCount + j * BM + wm * 32;
      f32x4 dv[4];                                     // minimum layout: the scales of this lane's 16 rows
      f16x4 da = {};                                   // others: row lr's, as an MFMA operand
      if constexpr (MIN) {
#pragma unroll
        for (int i = 0; i < kR / 4; ++i) dv[i] = *reinterpret_cast<const f32x4*>(dj + 8 * i + 4 * h);
      } else {
        da[0] = __builtin_bit_cast(_Float16, dj[lr]);
      }
      i32x16 base;
      if constexpr (META == kMetaNone) {               // magic - o R in every column
        constexpr int kNo = (int)((0x100u - (1u << (Q - 1))) * 0x01010101u);
        base = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, i32x4{kNo, kNo, kNo, kNo}, start, 0, 0, 0);
      } else if constexpr (MIN) {                      // magic + R
        base = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, i32x4{0x01010101, 0x01010101, 0x01010101, 0x01010101}, start, 0, 0, 0);
      }
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        const int bn = (wn * TC + c) * 32 + lr;
        const i32x4 bv = *reinterpret_cast<const i32x4*>(bs + buf * C::kBBytes + bn * kRow + piece);
        const scale_t sn = ss[buf * kSCount + j * BN + bn];
        const i32x16 v = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, bv, META == kMetaNone ? base : start, 0, 0, 0);
        if constexpr (MIN) {
          const float m = ms[buf * kSCount + j * BN + bn];
#pragma unroll
          for (int r = 0; r < kR; ++r) {
            const float t = __builtin_fmaf(sn, value(v[r]), m * value(base[r]));
            acc[c][r] = __builtin_fmaf(dv[r >> 2][r & 3], t, acc[c][r]);
          }
        } else {
          f16x4 sb = {};
          sb[0] = __builtin_bit_cast(_Float16, sn);
          f32x16 zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
          const f32x16 ds2 = __builtin_amdgcn_mfma_f32_32x32x8f16(da, sb, zero, 0, 0, 0);      // 2 d s
#pragma unroll
          for (int r = 0; r < kR; ++r) acc[c][r] = __builtin_fmaf(ds2[r], value(v[r]), acc[c][r]);
        }
      }
      if constexpr (NB > 4) {                          // two blocks at a time: with eight, zero points spill
        if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  // Stage s: the activations of stage s + 1 and the register loads of stage s + 2 go out,
  // this stage is multiplied, stage s + 1's weights go from registers to LDS, and once its
  // activations have landed (everything but the register loads just issued) the workgroup
  // meets.  The barrier is for LDS only: the register loads stay in flight across it.
  constexpr int kRegLoads = C::kBPer * (META == kMetaNone ? 2 : 3) + C::kDPer;
  Regs t0, t1;
  issue_a(0, as0);
  issue_b(0, t0);
  issue_b(1, t1);
  store_b(t0, 0);
  wait_vmcnt<kRegLoads>();
  lds_barrier();
  auto stage = [&](int s, const uint8_t* as, uint8_t* as_next, Regs& freed, const Regs& next, int buf) {
    issue_a(s + 1, as_next);
    issue_b(s + 2, freed);
    compute(as, buf);
    if (((s + 1) & (chain - 1)) == 0) fold();
    __builtin_amdgcn_sched_barrier(0);
    store_b(next, 1 - buf);
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<kRegLoads>();
    lds_barrier();
  };
  int s = 0;
  for (; s + 2 <= nstages; s += 2) {
    stage(s, as0, as1, t0, t1, 0);
    stage(s + 1, as1, as0, t1, t0, 1);
  }
  if (s < nstages) stage(s, as0, as1, t0, t1, 0);
  fold();
  wait_vmcnt<0>();
  __syncthreads();

  // The K-groups' sums meet pairwise in LDS (group order fixed): group g + half adds into
  // group g until group 0 holds the tile.
  float* const red = reinterpret_cast<float*>(bs);
#pragma unroll
  for (int half = KG / 2; half >= 1; half >>= 1) {
    // at most half * WM * WN = 4 wavefronts write at a time, their TC column tiles in turn
    constexpr int kRoom = 2 * C::kBBytes / 4;
    const int slot = ((grp - half) * WN + wn) * WM + wm;
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      if (grp >= half && grp < 2 * half)
#pragma unroll
        for (int q4 = 0; q4 < kR / 4; ++q4)
          *reinterpret_cast<f32x4*>(red + slot * 1024 + q4 * 256 + lane * 4) =
              f32x4{tot[c][4 * q4], tot[c][4 * q4 + 1], tot[c][4 * q4 + 2], tot[c][4 * q4 + 3]};
      __syncthreads();
      if (grp < half)
#pragma unroll
        for (int q4 = 0; q4 < kR / 4; ++q4) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(red + ((grp * WN + wn) * WM + wm) * 1024 + q4 * 256 + lane * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) tot[c][4 * q4 + e] += v[e];
        }
      __syncthreads();
    }
    static_assert(kRoom >= 4 * 1024, "partial tiles of four wavefronts fit");
  }
  if (grp != 0) return;
#pragma unroll
  for (int c = 0; c < TC; ++c)
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int64_t m = m0 + wm * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
      const int64_t n = n0 + (wn * TC + c) * 32 + lr;
      if (m < M && n < N) y[m * N + n] = f32_to_bf16_bits(MIN ? tot[c][r] : 0.5f * tot[c][r]);
    }
}

template <int Q, int META, int WM, int WN, int TC, int SB, bool HALF = false>
hipError_t q8_gemm_launch(const int8_t* qx, const uint16_t* dx, int64_t M, const uint8_t* codes, const uint16_t* scales,
                          const void* meta, int64_t N, int64_t K, int gshift, uint16_t* y, hipStream_t stream) {
  using C = Q8Cfg<META, WM, WN, TC, SB>;
  const int64_t tiles = ((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
  q8_gemm_kernel<Q, META, WM, WN, TC, SB, HALF><<<dim3((unsigned)tiles), kThreads, 0, stream>>>(
      qx, dx, (int)M, codes, scales, meta, (int)N, (int)K, gshift, y);
  return hipGetLastError();
}

// Tile choice.  Every tile walks all of K, so a launch takes the tile's time for one pass
// over K times its rounds over the 256 CUs.  Cost of a pass relative to a 32x32 tile's, with
// the weights in cache.  From memory, 256 tiles at K = 4096, us: 32x32 11.3, 32x64 17.4, 64x64
// 23.5, 64x128 37.8, 128x128 65.4 (2 workgroups of 32x32 fit a CU).
struct Q8Tile {
  int bm, bn, cost, cost2;     // cost2: a round of up to 512 tiles where two share a CU (up to 16 tokens), else 0
};
constexpr Q8Tile kQ8Tiles[] = {{32, 32, 106, 168}, {32, 64, 150, 0}, {64, 64, 192, 0}, {64, 128, 315, 0}, {128, 128, 545, 0}};

int q8_tile_for(int64_t M, int64_t N) {
  int best = 0;
  int64_t best_cost = 0;
  for (int i = 0; i < 5; ++i) {
    const Q8Tile& t = kQ8Tiles[i];
    const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    int64_t c;
    if (t.cost2 && M <= 16) {
      const int64_t rest = tiles % 512;
      c = tiles / 512 * t.cost2 + (rest == 0 ? 0 : rest <= 256 ? t.cost : t.cost2);
    } else {
      c = (tiles + 255) / 256 * t.cost;
    }
    if (i == 0 || c < best_cost) {
      best = i;
      best_cost = c;
    }
  }
  return best;
}

}  // namespace

Route q8_gemm_route(int64_t M, int64_t N) {
  const Q8Tile& t = kQ8Tiles[q8_tile_for(M, N)];
  return Route{kRouteQ8Tile, t.bm, t.bn, 1};
}

// Time of the launch, us: 3.8, and the tile's pass over K per round (least squares over 460 sizes
// of up to 32 tokens, 7 % rms; zero points and minimums cost more a block).
float q8_gemm_us(int64_t M, int64_t N, int64_t K, int kind) {
  const Q8Tile& t = kQ8Tiles[q8_tile_for(M, N)];
  const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), slots = t.cost2 && M <= 16 ? 512 : 256;
  const int pass = slots == 512 && tiles > 256 ? t.cost2 : t.cost;
  const float block = kind == kMetaMin ? 1.05f : kind == kMetaZp ? 0.82f : 0.75f;
  return 3.8f + (float)((tiles + slots - 1) / slots) * block * ((float)pass / 10.0f - 3.0f) * (float)K / 4096.0f;
}

namespace {

template <int Q, int META>
hipError_t q8_gemm_dispatch(const int8_t* qx, const uint16_t* dx, int64_t M, const uint8_t* codes, const uint16_t* scales,
                            const void* meta, int64_t N, int64_t K, int gshift, uint16_t* y, hipStream_t stream) {
  switch (q8_tile_for(M, N)) {
    case 0:
      if (M <= 16) return q8_gemm_launch<Q, META, 1, 1, 1, 16, true>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
      return q8_gemm_launch<Q, META, 1, 1, 1, 16>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
    case 1:
      if (M <= 16) return q8_gemm_launch<Q, META, 1, 1, 2, 8, true>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
      return q8_gemm_launch<Q, META, 1, 1, 2, 8>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
    case 2: return q8_gemm_launch<Q, META, 2, 1, 2, 8>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
    case 3: return q8_gemm_launch<Q, META, 2, 2, 2, 8>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
    default: return q8_gemm_launch<Q, META, 4, 2, 2, 8>(qx, dx, M, codes, scales, meta, N, K, gshift, y, stream);
  }
}

}  // namespace

hipError_t launch_q8_gemm(const int8_t* qx, const uint16_t* dx, int64_t M, const uint8_t* codes, const uint16_t* scales,
                          GroupMeta meta, int64_t N, int64_t K, int group, int q, uint16_t* y, hipStream_t stream) {
  const int gshift = group == 32 ? 0 : group == 64 ? 1 : 2;
  switch (q * 4 + meta.kind) {
#define SSQ_Q8_CASE(Q, META) \
  case Q * 4 + META: return q8_gemm_dispatch<Q, META>(qx, dx, M, codes, scales, meta.ptr, N, K, gshift, y, stream);
    SSQ_Q8_CASE(2, 0) SSQ_Q8_CASE(2, 1) SSQ_Q8_CASE(2, 2)
    SSQ_Q8_CASE(3, 0) SSQ_Q8_CASE(3, 1) SSQ_Q8_CASE(3, 2)
    SSQ_Q8_CASE(4, 0) SSQ_Q8_CASE(4, 1) SSQ_Q8_CASE(4, 2)
#undef SSQ_Q8_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ssq
