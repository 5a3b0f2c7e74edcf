// Binary32 matmul: y[M,N] = x[M,K] * What[N,K]^T with binary32 x and y.
//
// App. B.3 of the paper: What[n,k] = s[n,b] (u[n,k] - o[n,b]), or s u + m for the
// binary16-minimum layout.  Every weight is formed exactly as before in binary32 (s (u - o)
// exactly, s u + m rounded once) and multiplied on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 products and sums).
//
// What bounds it: the fp32 MFMA rate for 16 tokens (32 MFMAs of 13 ns per 16 rows x 128 k),
// latency for few rows.  A workgroup owns 16 weight rows and up to 16 tokens; its
// wavefronts take the 128-k super-blocks in turn.  Lane l of an MFMA holds weight row
// l % 16 and 32-weight block l / 16 of the super-block, and MFMA t multiplies weight t of
// each lane's block, so a lane unpacks one whole block and its operand needs no moves;
// the activation operand follows the same assignment.  Activations go straight to LDS
// (512 contiguous bytes a token), codes are loaded four lanes to a row and moved to their
// MFMA lanes with ds_bpermute: a load with a row per lane runs the texture unit at a
// quarter of its rate.  Sums: 32 MFMA steps per super-block in eight chains, then the
// wavefront's super-blocks, then the wavefronts as a tree.
//
// Measured (W4 g32, graph replays; before: a wavefront per row and 4 tokens, each lane
// reading its block's 128 bytes of every token from memory): 8 x 4096 x 4096 10.3 us (60),
// 16 x 4096 x 4096 11.3 (117), 64 x 4096 x 4096 37 (452), 128 x 4096 x 14336 206 (3160).
#include <algorithm>

#include "mfma_dequant.h"
#include "ssq_internal.h"

namespace ssq {
namespace {

constexpr uint32_t kOutOfRange = 0x80000000u;   // past every buffer's size: loads return 0
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kRows = 16, kTokens = 16;

// TOK tokens are staged (4, 8 or 16; the MFMA's other rows repeat them and are dropped), 128
// k of each a stage; as many wavefronts as two stages each leave room for in 160 KB of LDS.
template <int TOK>
struct F32Cfg {
  static constexpr int kStageBytes = TOK * 512;
  static constexpr int kXLoads = TOK / 2;       // two tokens a load
  static constexpr int kMaxWaves = TOK == 16 ? 8 : 16;
};

// The 32 weights of a block in binary32, from its q dwords.
template <int Q, int META>
__device__ __forceinline__ void block_weights(const uint32_t (&d)[Q], float s, uint32_t meta_bits, float (&f)[32]) {
  // fields j and j + 4 of each 8 (8 and 16 bits apart) in the low mantissa bits of fp16 1024
  const uint32_t magic = 0x64006400u;
  const float o = META == kMetaZp ? (float)meta_bits : (float)(1 << (Q - 1));
  const float so = -(1024.0f + o) * s;          // exact: 11-bit by 11-bit
  const float m = META == kMetaMin ? f16_bits_to_f32(meta_bits) : 0.0f;
  auto weight = [&](float b) {                  // b = 1024 + u
    if constexpr (META == kMetaMin) return __builtin_fmaf(b - 1024.0f, s, m);
    else return __builtin_fmaf(b, s, so);
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t w;                                 // 8 fields: 0..3 at bit 0, 4..7 at bit 16
    if constexpr (Q == 4) {
      w = d[i];
    } else if constexpr (Q == 2) {
      const uint32_t h = d[i >> 1] >> (16 * (i & 1));
      w = __builtin_amdgcn_perm(0u, h, 0x0c010c00u);
    } else {
      const uint32_t v = i == 0 ? d[0]
                       : i == 1 ? __builtin_amdgcn_alignbit(d[1], d[0], 24)
                       : i == 2 ? __builtin_amdgcn_alignbit(d[2], d[1], 16)
                                : d[2] >> 8;
      w = (v & 0xFFFu) | ((v << 4) & 0x0FFF0000u);
    }
    constexpr uint32_t kMask = Q == 4 ? 0x000F000Fu : Q == 3 ? 0x00070007u : 0x00030003u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t p = ((w >> (Q * j)) & kMask) | magic;
      f[8 * i + j] = weight(f16_lo(p));
      f[8 * i + j + 4] = weight(f16_hi(p));
    }
  }
}

template <int I, int BYTES>
__device__ __forceinline__ uint8_t* lds_object() {
  __shared__ __attribute__((aligned(1024))) uint8_t mem[BYTES];
  return mem;
}

template <int Q, int META, int TOK>
__global__ __launch_bounds__(64 * F32Cfg<TOK>::kMaxWaves) void matmul_f32_kernel(
    const float* __restrict__ x, int M, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
    const void* __restrict__ meta, int N, int K, int gshift, float* __restrict__ y) {
  using C = F32Cfg<TOK>;
  constexpr int kStageBytes = C::kStageBytes;
  constexpr int kMetaSize = META == kMetaZp ? 1 : META == kMetaMin ? 2 : 0;
  // each stage its own LDS object, so that reading one does not wait for the other's loads
  uint8_t* const xs0 = lds_object<0, C::kMaxWaves * kStageBytes>();
  uint8_t* const xs1 = lds_object<1, C::kMaxWaves * kStageBytes>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = (int)blockDim.x >> 6;
  const int64_t n0 = (int64_t)blockIdx.x * kRows, m0 = (int64_t)blockIdx.y * kTokens;
  const int nblk = K / 32, nsb = (nblk + 3) / 4;
  const uint32_t row_bytes = (uint32_t)K * Q / 8;
  const uint32_t gpr = (uint32_t)nblk >> gshift;
  const uint32_t rows = (uint32_t)std::min<int64_t>(kRows, N - n0);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + n0 * row_bytes, rows * row_bytes);
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(scales + n0 * gpr, rows * gpr * 2);
  const uint8_t* const mp = static_cast<const uint8_t*>(meta);
  const __amdgpu_buffer_rsrc_t rz = make_rsrc(kMetaSize ? mp + n0 * gpr * kMetaSize : mp,
                                              kMetaSize ? rows * gpr * kMetaSize : 0u);
  const uint32_t tokens = (uint32_t)std::min<int64_t>(kTokens, M - m0);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + m0 * K, tokens * (uint32_t)K * 4);

  const int n = lane & 15, c = lane >> 4;
  const int lrow = lane >> 2, lpiece = lane & 3;
  const int perm = (4 * n + c) * 4;             // the lane that loaded (row n, block c), in bytes

  // Activations of super-block sb: 2 tokens of 512 bytes a load, 16-byte pieces XOR-swizzled
  // with the token, so that 16 tokens' reads of one piece touch every bank once.
  auto issue_x = [&](int sb, uint8_t* st) {
#pragma unroll
    for (int i = 0; i < C::kXLoads; ++i) {
      const int m = 2 * i + (lane >> 5);
      const int piece = (lane & 31) ^ (m & 15);
      const uint32_t past = 4 * sb + (piece >> 3) < nblk ? 0u : kOutOfRange;
      const uint32_t off = (((uint32_t)m * (uint32_t)K + (uint32_t)sb * 128 + 4 * piece) * 4) | past;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(st + wave * kStageBytes + i * 1024), 16, (int)off, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  struct Codes {
    uint32_t d[Q];
    uint32_t s, z;
  };
  auto issue_c = [&](int sb, Codes& t) {
    const int blk = 4 * sb + lpiece;
    const uint32_t past = blk < nblk ? 0u : kOutOfRange;
    buffer_block_codes<Q>(rc, ((uint32_t)lrow * row_bytes + (uint32_t)blk * (4 * Q)) | past, 0, t.d);
    const uint32_t gi = (uint32_t)lrow * gpr + (uint32_t)(blk >> gshift);
    t.s = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)((gi * 2) | past), 0, 0);
    t.z = 0u;
    if constexpr (META == kMetaZp) t.z = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)(gi | past), 0, 0);
    if constexpr (META == kMetaMin) t.z = __builtin_amdgcn_raw_buffer_load_b16(rz, (int)((gi * 2) | past), 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  const f32x4 zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 acc = zero4;
  auto step = [&](Codes& t, const uint8_t* st) {
    uint32_t d[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) d[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(perm, (int)t.d[i]);
    const uint32_t sbits = (uint32_t)__builtin_amdgcn_ds_bpermute(perm, (int)t.s);
    const uint32_t zbits = META != kMetaNone ? (uint32_t)__builtin_amdgcn_ds_bpermute(perm, (int)t.z) : 0u;
    float f[32];
    block_weights<Q, META>(d, f16_bits_to_f32(sbits), zbits, f);
    f32x4 a[8];
    const int am = n & (TOK - 1);
    const uint8_t* const row = st + wave * kStageBytes + am * 512;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = *reinterpret_cast<const f32x4*>(row + (((8 * c + i) ^ am) << 4));
    // eight sums of four MFMAs, added as a tree: with one or two sums the chains are 128 or
    // 64 additions long and the error against 64 bits 1.5e-7; with eight 1.0e-7
    f32x4 e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].x, f[4 * i], zero4, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].y, f[4 * i + 1], e[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].z, f[4 * i + 2], e[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].w, f[4 * i + 3], e[i], 0, 0, 0);
    acc += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
  };

  // Super-blocks of this wavefront: wave, wave + W, ... in two slots.
  Codes c0, c1;
  issue_x(wave, xs0);
  issue_c(wave, c0);
  issue_x(wave + W, xs1);
  issue_c(wave + W, c1);
  int sb = wave;
  for (; sb + 2 * W < nsb; sb += 2 * W) {
    step(c0, xs0);
    __builtin_amdgcn_sched_barrier(0);
    issue_x(sb + 2 * W, xs0);
    issue_c(sb + 2 * W, c0);
    step(c1, xs1);
    __builtin_amdgcn_sched_barrier(0);
    issue_x(sb + 3 * W, xs1);
    issue_c(sb + 3 * W, c1);
  }
  if (sb < nsb) step(c0, xs0);
  if (sb + W < nsb) step(c1, xs1);

  // The wavefronts' sums, as a tree: lane l holds D[4 (l/16) + r][l % 16].
  wait_vmcnt<0>();
  __syncthreads();
  float* const part = reinterpret_cast<float*>(xs0);           // a kilobyte a wavefront
  *reinterpret_cast<f32x4*>(part + wave * 256 + 4 * lane) = acc;
  __syncthreads();
  for (int e = tid; e < 256; e += 64 * W) {
    float p[C::kMaxWaves];
#pragma unroll
    for (int w = 0; w < C::kMaxWaves; ++w) p[w] = w < W ? part[w * 256 + e] : 0.0f;
#pragma unroll
    for (int h = C::kMaxWaves / 2; h >= 1; h >>= 1)
#pragma unroll
      for (int w = 0; w < h; ++w) p[w] += p[w + h];
    const float v = p[0];
    const int l = e >> 2;
    const int64_t m = m0 + 4 * (l >> 4) + (e & 3), row = n0 + (l & 15);
    if (m < M && row < N) y[m * N + row] = v;
  }
}

// Up to three tokens of a short matrix: one wavefront per weight row, each lane whole blocks
// on the vector ALU, four chains a block (error against 64 bits at K = 8192 9.7e-8; 1.08e-7 with
// one, 1.07e-7 in the kernel above; the same time).  It spreads 16 rows over four workgroups
// where the kernel above gives them to one, whose MFMAs cost the same for 1 token as for 16.
template <int Q, int META>
__global__ __launch_bounds__(256) void matmul_f32_rows_kernel(
    const float* __restrict__ x, int M, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales,
    const void* __restrict__ meta, int N, int K, int gshift, float* __restrict__ y) {
  constexpr int kMaxTokens = 4;
  const int lane = threadIdx.x & 63;
  const int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const int nblk = K / 32;
  const int64_t row_bytes = (int64_t)K * Q / 8;
  float acc[kMaxTokens] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int j = lane; j < nblk; j += 64) {
    uint32_t d[Q];
    load_block_codes<Q>(codes + n * row_bytes + (int64_t)j * (4 * Q), d);
    const int64_t gi = n * (nblk >> gshift) + (j >> gshift);
    const float s = f16_bits_to_f32(scales[gi]);
    // weight = s*u - s*o, or s*u + m for the minimum layout
    const float so = META == kMetaMin ? f16_bits_to_f32(static_cast<const uint16_t*>(meta)[gi])
                   : META == kMetaZp ? -s * (float)static_cast<const uint8_t*>(meta)[gi]
                                     : -s * (float)(1 << (Q - 1));
    float w[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) w[k] = __builtin_fmaf(s, (float)field<Q>(d, k), so);
#pragma unroll
    for (int t = 0; t < kMaxTokens; ++t) {
      if (t >= M) break;
      const float* xr = x + (int64_t)t * K + (int64_t)j * 32;
      float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 32; ++k) a[k & 3] = __builtin_fmaf(xr[k], w[k], a[k & 3]);
      acc[t] += (a[0] + a[1]) + (a[2] + a[3]);
    }
  }
#pragma unroll
  for (int t = 0; t < kMaxTokens; ++t) {
    const float v = group_sum<64>(acc[t]);
    if (lane == 0 && t < M) y[(int64_t)t * N + n] = v;
  }
}

// Short matrices at 1 to 3 tokens take the rows kernel: 2 x 1024 x 4096 runs in 6.8 us
// against 8.6, 3 x 333 x 1056 in 4.8 against 5.7, 2 x 8 x 32768 in 31 against 47; from M N =
// 4096 on it loses (1 x 4096 x 4096: 12.1 us against 9.8; 4 x 32 x 4096: 10.0 against 8.2).
// One token of more than 4096 rows, a second round of the kernel above (its 16 wavefronts fill a
// CU), takes it too, unless rows are short enough for two workgroups a CU or the rounds are
// many: 4219x8192 21.0 us against 27.3, 5943x4096 14.4 / 18.9, 8842x3840 19.5 / 24.0, 13956x3840
// 28.1 / 36.5, but 4009x512 5.5 / 4.0, 6967x896 9.4 / 6.8, 16252x3456 31.8 / 29.5.
constexpr int64_t kRowsMaxTokens = 3, kRowsMaxOutputs = 3072;
bool rows_kernel(int64_t M, int64_t N, int64_t K) {
  return M <= kRowsMaxTokens && (M * N <= kRowsMaxOutputs || (M == 1 && N > 4096 && N <= 15360 && K > 1152));
}

template <int Q, int META>
hipError_t f32_dispatch(const float* x, int64_t M, const uint8_t* codes, const uint16_t* scales, const void* meta,
                        int64_t N, int64_t K, int gshift, float* y, hipStream_t stream) {
  if (rows_kernel(M, N, K)) {
    matmul_f32_rows_kernel<Q, META><<<dim3((unsigned)((N + 3) / 4)), 256, 0, stream>>>(x, (int)M, codes, scales, meta,
                                                                                     (int)N, (int)K, gshift, y);
    return hipGetLastError();
  }
  const int64_t nsb = (K / 32 + 3) / 4;
  constexpr int64_t kMaxTokens = int64_t(65535) * kTokens;      // the grid's second dimension
  for (int64_t m0 = 0; m0 < M; m0 += kMaxTokens) {
    const int64_t mm = std::min<int64_t>(M - m0, kMaxTokens);
    const dim3 grid((unsigned)((N + kRows - 1) / kRows), (unsigned)((mm + kTokens - 1) / kTokens));
    const unsigned threads = 64 * (unsigned)std::min<int64_t>(mm <= 8 ? 16 : 8, nsb);
    const float* const xm = x + m0 * K;
    float* const ym = y + m0 * N;
    if (mm <= 4)
      matmul_f32_kernel<Q, META, 4><<<grid, threads, 0, stream>>>(xm, (int)mm, codes, scales, meta, (int)N, (int)K, gshift, ym);
    else if (mm <= 8)
      matmul_f32_kernel<Q, META, 8><<<grid, threads, 0, stream>>>(xm, (int)mm, codes, scales, meta, (int)N, (int)K, gshift, ym);
    else
      matmul_f32_kernel<Q, META, 16><<<grid, threads, 0, stream>>>(xm, (int)mm, codes, scales, meta, (int)N, (int)K, gshift, ym);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_matmul_f32(const float* x, int64_t M, const uint8_t* codes, const uint16_t* scales, GroupMeta meta,
                             int64_t N, int64_t K, int group, int q, float* y, hipStream_t stream) {
  const int gshift = group == 32 ? 0 : group == 64 ? 1 : 2;
  switch (q * 4 + meta.kind) {
#define SSQ_F32_CASE(Q, META) \
  case Q * 4 + META: return f32_dispatch<Q, META>(x, M, codes, scales, meta.ptr, N, K, gshift, y, stream);
    SSQ_F32_CASE(2, 0) SSQ_F32_CASE(2, 1) SSQ_F32_CASE(2, 2)
    SSQ_F32_CASE(3, 0) SSQ_F32_CASE(3, 1) SSQ_F32_CASE(3, 2)
    SSQ_F32_CASE(4, 0) SSQ_F32_CASE(4, 1) SSQ_F32_CASE(4, 2)
#undef SSQ_F32_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ssq
