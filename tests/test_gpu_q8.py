"""GPU parity: Q8_0 activation quantization (bit-exact codes and scales) and the
integer-dot matmul (App. B.3) against the CPU oracle (App. C readings)."""
import json
import os

import numpy as np
import pytest
import torch

from oracle import ssq_oracle as O
from paper_2607_08779_amd import ssq, synth
from tests.routes import route
from tests.parity_common import (Guarded, assert_within, log_metric, rel_l2, sample_rows, to_device,
                                 y_to_f64)

pytestmark = pytest.mark.gpu

MODES = [O.SIGNED_SYM, O.UNSIGNED_SYM, O.ASYM, O.ASYM_MIN]


def bf16_bits(a):
    return synth.to_bf16_bits(np.asarray(a, np.float32))


def act_bits(M, K, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    x = rng.standard_t(4, size=(M, K)) * scale
    x[rng.random(x.shape) < 0.01] *= 30
    return bf16_bits(x)


def check_act(xb, tag=""):
    M, K = xb.shape
    g_q, g_d = Guarded((M, K), torch.int8, fill=0x5A), Guarded((M, K // 32), torch.int16, fill=0x5A)
    qx, dx = ssq.ssq_quantize_act_q8(to_device(xb, True), out=(g_q.t, g_d.t))
    torch.cuda.synchronize()
    g_q.check(f"{tag} codes")
    g_d.check(f"{tag} scales")
    with np.errstate(over="ignore"):
        ref = O.quantize_act_q8(O.bf16_bits_to_f32(xb))
    q, d = qx.cpu().numpy(), dx.cpu().numpy().view(np.uint16)
    if not np.array_equal(q, ref.q):
        m, k = np.argwhere(q != ref.q)[0]
        raise AssertionError(f"{tag}: code ({m}, {k}) gpu {q[m, k]} oracle {ref.q[m, k]}")
    if not np.array_equal(d, ref.d):
        m, b = np.argwhere(d != ref.d)[0]
        raise AssertionError(f"{tag}: scale ({m}, {b}) gpu {d[m, b]:#06x} oracle {ref.d[m, b]:#06x}")
    return qx, dx, ref


@pytest.mark.parametrize("M,K", [(1, 32), (1, 4096), (3, 14336), (64, 1024)])
def test_quantize_act_q8_matches_oracle(M, K):
    check_act(act_bits(M, K, seed=M * 7 + K), tag=f"M={M} K={K}")


def test_quantize_act_q8_worked_example_and_edges():
    gold = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "q8_worked_example.json")))
    _, _, ref = check_act(bf16_bits([gold["x"]]), tag="worked example")
    assert ref.q.tolist() == [gold["q"]]
    rng = np.random.default_rng(4)
    rows = [np.zeros(64), -np.zeros(64), rng.standard_normal(64) * 1e-38,   # subnormal d, binary16 0
            rng.standard_normal(64) * 3e7,                                  # binary16 scale overflows
            np.arange(64) - 31.5, np.full(64, -2.75)]
    check_act(bf16_bits(np.stack(rows)), tag="edges")


def check_q8_matmul(w, x_bits, group, q, mode, rows_idx=None, tag="", repeat_rows=None):
    """Oracle-quantized weights and activations on the GPU through ssq_matmul_q8.  The rows of w
    come round until there are `repeat_rows`."""
    N, K = w.shape
    r = O.quantize(w, group, q, mode)
    if repeat_rows is not None:
        at = np.resize(np.arange(N), repeat_rows)
        N = repeat_rows
        r = r._replace(codes=r.codes[at], scales=r.scales[at], zp=None if r.zp is None else r.zp[at],
                       mins=None if r.mins is None else r.mins[at])
    a = O.quantize_act_q8(O.bf16_bits_to_f32(x_bits))
    meta = r.mins if mode == O.ASYM_MIN else r.zp
    dev_meta = None if meta is None else torch.from_numpy(
        meta.view(np.int16) if mode == O.ASYM_MIN else meta).cuda()
    M = x_bits.shape[0]
    g_y = Guarded((M, N), torch.bfloat16)
    y = ssq.ssq_matmul_q8(torch.from_numpy(a.q).cuda(), torch.from_numpy(a.d.view(np.int16)).cuda(),
                          torch.from_numpy(r.codes).cuda(), torch.from_numpy(r.scales.view(np.int16)).cuda(),
                          dev_meta, N, K, group, q, out=g_y.t)
    g_y.check(tag)
    sel = slice(None) if rows_idx is None else rows_idx
    ref = O.matmul_q8(a.q, a.d, r.codes[sel], r.scales[sel], None if r.zp is None else r.zp[sel],
                      r.codes[sel].shape[0], K, group, q, mins=None if r.mins is None else r.mins[sel])
    assert_q8_close(y, ref, sel, tag)


def assert_q8_close(y, ref, sel, tag):
    """Element-wise: the integer terms are exact, so the output carries one bf16 rounding
    (half an ulp, 2^-8 relative) plus binary32 accumulation of the K/32 block terms,
    bounded by 1e-5 of the row's largest output."""
    y_all = y_to_f64(y)
    assert not np.isnan(y_all).any(), f"{tag}: output elements left unwritten"
    got = y_all[:, sel]
    tol = 2.0 ** -8 * np.abs(ref) + 1e-5 * np.abs(ref).max(axis=1, keepdims=True) + 1e-30
    worst = assert_within(got, ref, tol, tag)
    err = rel_l2(got, ref)
    log_metric(test="q8_matmul", tag=tag, rel_l2=err, max_err_over_bound=worst)
    assert err <= 5e-3, f"{tag}: rel L2 {err:.2e}"


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("mode", MODES)
def test_matmul_q8_all_formats(q, group, mode):
    rng = np.random.default_rng(q * 31 + group + mode)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(37, 1024)) * 0.02))
    check_q8_matmul(w, act_bits(2, 1024, seed=q + group), group, q, mode, tag=f"q={q} g={group} m={mode}")


@pytest.mark.parametrize("K", [32, 96, 19200])
def test_matmul_q8_reduction_lengths(K):
    """One block, an odd block count, and 600 blocks (two passes, the second ragged)."""
    rng = np.random.default_rng(K)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(9, K)) * 0.02))
    for q in (2, 3, 4):
        check_q8_matmul(w, act_bits(1, K, seed=K + q), 32, q, O.SIGNED_SYM, tag=f"K={K} q={q}")


@pytest.mark.parametrize("M", [1, 2, 5])
def test_matmul_q8_token_counts(M):
    rng = np.random.default_rng(M)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(70, 2048)) * 0.02))
    check_q8_matmul(w, act_bits(M, 2048, seed=M), 32, 4, O.ASYM, tag=f"M={M}")


def test_q8_pipeline_llama3_8b_down_proj_full_size():
    """4096x14336 at W4 g32, signed: GPU weight quantization, GPU activation
    quantization and the integer matmul against the oracle on sampled rows."""
    spec = synth.llama3_8b_decode().layers["down_proj"]
    wb = synth.weights(spec)
    x = act_bits(1, spec.cols, seed=21, scale=0.5)
    W = to_device(wb, True)
    codes, scales, zp = ssq.ssq_quantize(W, 32, 4, O.SIGNED_SYM)
    qx, dx, a = check_act(x, tag="down_proj activations")
    y = ssq.ssq_matmul_q8(qx, dx, codes, scales, zp, spec.rows, spec.cols, 32, 4)
    torch.cuda.synchronize()
    rows = sample_rows(spec.rows, 64, seed=5)
    r = O.quantize(O.bf16_bits_to_f32(wb[rows]), 32, 4, O.SIGNED_SYM)
    assert np.array_equal(codes.cpu().numpy()[rows], r.codes)
    ref = O.matmul_q8(a.q, a.d, r.codes, r.scales, None, len(rows), spec.cols, 32, 4)
    assert_q8_close(y, ref, rows, "q8 pipeline down_proj")


# ---------------------------------------------------------------------------
# Several tokens: the one-token kernel with a grid row per token (up to 40 tokens of small
# matrices) and the smallest tile.
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("M", [2, 16, 17, 32, 33, 40, 41, 72])
@pytest.mark.parametrize("mode", MODES)
def test_matmul_q8_batched_token_counts(M, mode):
    """Up to 40 tokens the one-token kernel, above 32x32 tiles, two and three of them; 70 rows (a
    ragged last tile) and K = 2016 (63 blocks: a ragged last stage)."""
    assert route(M, 70, 2016, 32, 4, mode, q8=True).kernel == ("q8_gemv" if M <= 40 else "q8_tile")
    rng = np.random.default_rng(M * 5 + mode)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(70, 2016)) * 0.02))
    check_q8_matmul(w, act_bits(M, 2016, seed=M + 100), 32, 4, mode, tag=f"batched M={M} m={mode}")


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
def test_matmul_q8_batched_formats(q, group):
    """Every q and group size at M = 16 with K = 4224: the one-token kernel, a grid row a token."""
    assert route(16, 33, 4224, group, q, O.ASYM, q8=True).kernel == "q8_gemv"
    rng = np.random.default_rng(q * 13 + group)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(33, 4224)) * 0.02))
    for mode in MODES:
        check_q8_matmul(w, act_bits(16, 4224, seed=q + group + mode), group, q, mode,
                        tag=f"batched q={q} g={group} m={mode}")


def test_matmul_q8_batched_long_rows_fall_back():
    """Rows longer than K = 32768 take the one-token kernel per token; same answers."""
    rng = np.random.default_rng(77)
    w = O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(9, 33792)) * 0.02))
    check_q8_matmul(w, act_bits(3, 33792, seed=78), 32, 4, O.SIGNED_SYM, tag="batched K=33792")


@pytest.mark.parametrize("M", [16, 32])
def test_q8_batched_llama3_8b_down_proj_full_size(M):
    """4096x14336 at W4 g32, signed, M tokens in 32x32 tiles, sampled rows."""
    spec = synth.llama3_8b_decode().layers["down_proj"]
    wb = synth.weights(spec)
    x = act_bits(M, spec.cols, seed=31 + M, scale=0.5)
    codes, scales, zp = ssq.ssq_quantize(to_device(wb, True), 32, 4, O.SIGNED_SYM)
    qx, dx, a = check_act(x, tag="batched activations")
    g_y = Guarded((M, spec.rows), torch.bfloat16)
    ssq.ssq_matmul_q8(qx, dx, codes, scales, zp, spec.rows, spec.cols, 32, 4, out=g_y.t)
    g_y.check("batched full size")
    rows = sample_rows(spec.rows, 64, seed=M)
    r = O.quantize(O.bf16_bits_to_f32(wb[rows]), 32, 4, O.SIGNED_SYM)
    assert np.array_equal(codes.cpu().numpy()[rows], r.codes)
    ref = O.matmul_q8(a.q, a.d, r.codes, r.scales, None, len(rows), spec.cols, 32, 4)
    assert_q8_close(g_y.t, ref, rows, f"q8 batched down_proj M={M}")


# ---------------------------------------------------------------------------
# Tiles of the several-token kernel (q8_gemm.hip): 32x32, 32x64, 64x64, 64x128 and 128x128
# outputs, chosen by how many of each cover M x N.
# ---------------------------------------------------------------------------

Q8_TILES = [
    (3, 33, 544),        # too few tokens for a tile: the one-token kernel
    (31, 8225, 288),     # 32x64: the last tile one column; two 256-deep stages, the second one block
    (65, 8161, 800),     # 64x64: two token tiles, the second one row; four stages, the last one block
    (129, 10400, 256),   # 64x128: three token tiles; exactly one stage
    (255, 14305, 1056),  # 128x128: two token tiles, the second short of a row; five stages
]


@pytest.mark.parametrize("M,N,K", Q8_TILES)
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_matmul_q8_tiles(M, N, K, q, mode):
    spec = synth.WeightSpec(N, K, nu=5.0, scale=0.02, outlier_frac=0.001, seed=M + q)
    w = O.bf16_bits_to_f32(synth.weights(spec))
    check_q8_matmul(w, act_bits(M, K, seed=M + mode), 32, q, mode, rows_idx=sample_rows(N, n=40, seed=q),
                    tag=f"tiles {M}x{N}x{K} q={q} m={mode}")


# The same tiles in the other group sizes, and 32x32 with two workgroups a CU.
@pytest.mark.parametrize("tile,M,N,K", [
    ((32, 32), 41, 33, 640),         # two token tiles; two 512-deep stages, the second four blocks
    ((32, 32), 16, 4100, 640),       # half a tile of tokens
    ((32, 32), 16, 17000, 640),      # 532 tiles
    ((32, 64), 13, 8300, 640),       # half a tile of tokens
    ((32, 64), 31, 8225, 384),
    ((64, 64), 65, 8161, 896),
    ((64, 128), 129, 10400, 1152),
    ((128, 128), 255, 14305, 1152),
])
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [64, 128])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_matmul_q8_tile_groups(tile, M, N, K, q, group, mode):
    assert route(M, N, K, group, q, mode, q8=True)[:3] == ("q8_tile", *tile)
    w = O.bf16_bits_to_f32(synth.weights(synth.WeightSpec(min(N, 499), K, nu=5.0, scale=0.02, outlier_frac=0.001, seed=M + q)))
    check_q8_matmul(w, act_bits(M, K, seed=M + mode), group, q, mode, rows_idx=sample_rows(N, n=40, seed=q),
                    tag=f"tiles {M}x{N}x{K} q={q} g={group} m={mode}", repeat_rows=N)


# Few tokens: the one-token kernel with a grid row per token on small or long matrices, and
# the tiles just past its 40 tokens and, half full, on matrices large enough for them.
Q8_FEW = [
    (2, 5, 32),          # one block, a row past the workgroup's four
    (3, 1001, 4128),     # 129 blocks: ragged passes over K
    (16, 130, 8224),     # ragged rows
    (40, 130, 2080),     # its most tokens
    (41, 33, 544),       # 32x32: a ragged tile both ways, two stages, the second one block
    (16, 4100, 544),     # 32x32, half the tokens
    (7, 16900, 544),     # 32x32: 529 tiles, two workgroups a CU
    (12, 8300, 544),     # 32x64, half the tokens
]


@pytest.mark.parametrize("M,N,K", Q8_FEW)
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_matmul_q8_few_tokens(M, N, K, q, mode):
    spec = synth.WeightSpec(N, K, nu=5.0, scale=0.02, outlier_frac=0.001, seed=M + q)
    w = O.bf16_bits_to_f32(synth.weights(spec))
    check_q8_matmul(w, act_bits(M, K, seed=M + mode), 32, q, mode, rows_idx=sample_rows(N, n=40, seed=q),
                    tag=f"few tokens {M}x{N}x{K} q={q} m={mode}")


# ---------------------------------------------------------------------------
# Scales at the ends of binary16: infinities and NaN (a group or block that overflowed) reach
# the output as they do in the product of the separate terms, on both kernels, and subnormal
# scales keep their value.
# ---------------------------------------------------------------------------

def q8_on_gpu(a, r, meta, M, N, K, q, mode):
    dev = None if meta is None else torch.from_numpy(meta.view(np.int16) if mode == O.ASYM_MIN else meta).cuda()
    y = ssq.ssq_matmul_q8(torch.from_numpy(a.q).cuda(), torch.from_numpy(a.d.view(np.int16)).cuda(),
                          torch.from_numpy(r.codes).cuda(), torch.from_numpy(r.scales.view(np.int16)).cuda(), dev,
                          N, K, 32, q)
    return y_to_f64(y)


@pytest.mark.parametrize("M,N", [(1, 40), (17, 40), (41, 40), (70, 40), (16, 4100)])   # one-token kernel; two, three and half 32x32 tiles
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_matmul_q8_infinite_scales(M, N, q, mode):
    K = 1056
    assert route(M, N, K, 32, q, mode, q8=True).kernel == ("q8_gemv" if M in (1, 17) else "q8_tile")
    rng = np.random.default_rng(q + mode)
    r = O.quantize(O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(N, K)) * 0.02)), 32, q, mode)
    a = O.quantize_act_q8(O.bf16_bits_to_f32(act_bits(M, K, seed=M + q)))
    r.scales[1, 3], r.scales[2, 32], r.scales[4, 0] = 0x7C00, 0xFC00, 0x7E00       # +inf, -inf, NaN
    r.scales[6, 5], r.scales[6, 20] = 0x7C00, 0xFC00                               # both signs meet
    if r.mins is not None:
        r.mins[8, 7], r.mins[9, 1] = 0x7C00, 0xFC00
    a.d[M // 2, 4] = 0x7C00
    with np.errstate(invalid="ignore"):
        ref = O.matmul_q8(a.q, a.d, r.codes, r.scales, r.zp, N, K, 32, q, mins=r.mins)
    y = q8_on_gpu(a, r, r.mins if mode == O.ASYM_MIN else r.zp, M, N, K, q, mode)
    assert np.isinf(ref).any() and np.isnan(ref).any() and (M == 1 or np.isfinite(ref).any())
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    fine = np.isfinite(ref)
    if fine.any():
        assert (np.abs(y[fine] - ref[fine]) <= 2.0 ** -8 * np.abs(ref[fine]) + 1e-5 * np.abs(ref[fine]).max()).all()


@pytest.mark.parametrize("M", [1, 17, 41])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_matmul_q8_subnormal_scales(M, mode):
    N, K, q = 40, 1056, 4
    rng = np.random.default_rng(mode)
    r = O.quantize(O.bf16_bits_to_f32(bf16_bits(rng.standard_t(5, size=(N, K)) * 0.02)), 32, q, mode)
    a = O.quantize_act_q8(O.bf16_bits_to_f32(act_bits(M, K, seed=M)))
    r.scales[:] = rng.integers(1, 0x400, size=r.scales.shape)
    a.d[:] = rng.integers(1, 0x400, size=a.d.shape)
    if r.mins is not None:
        r.mins[:] = rng.integers(1, 0x400, size=r.mins.shape)
    ref = O.matmul_q8(a.q, a.d, r.codes, r.scales, r.zp, N, K, 32, q, mins=r.mins)
    y = q8_on_gpu(a, r, r.mins if mode == O.ASYM_MIN else r.zp, M, N, K, q, mode)
    assert (np.abs(y - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * np.abs(ref).max()).all()


# ---------------------------------------------------------------------------
# Binary32 sums of the several-token kernel.  A bf16 output goes to the wrong neighbour where
# the sum's error crosses a midpoint, so the share of such outputs follows the error: a float32
# model of the sums gives 8.8e-8 (2-norm) for chains of 8 blocks at K = 4096 and 1.4e-7 for one
# chain in each of two K-groups, 1.1e-7 and 2.5e-7 at K = 14336.  The bars lie between the
# shares of the two, 7 and 5 standard deviations of the count from them.
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("M,N,K,share", [
    (512, 14336, 4096, 1.25e-4),      # 128x128 tiles, one K-group: 1.0e-4 with short chains, 1.5e-4 without
    (512, 4096, 14336, 1.8e-4),       # 64x128 tiles, two K-groups: 1.2e-4, 2.3e-4
])
def test_matmul_q8_sum_error(M, N, K, share):
    gen = torch.Generator(device="cuda").manual_seed(N)
    w = 0.02 * torch.randn((N, K), generator=gen, device="cuda")
    far = torch.rand((N, K), generator=gen, device="cuda") < 1e-3
    codes, scales, _ = ssq.ssq_quantize(torch.where(far, 20 * w, w).to(torch.bfloat16), 32, 4, O.SIGNED_SYM)
    qx, dx = ssq.ssq_quantize_act_q8(torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16))
    y = ssq.ssq_matmul_q8(qx, dx, codes, scales, None, N, K, 32, 4)
    x64 = (qx.double().view(M, K // 32, 32) * dx.view(torch.float16).double()[..., None]).view(M, K)
    off = 0
    for r in range(0, N, 2048):
        u = torch.stack([codes[r:r + 2048] & 15, codes[r:r + 2048] >> 4], dim=2).double().view(-1, K // 32, 32)
        w64 = ((u - 8) * scales[r:r + 2048].view(torch.float16).double()[..., None]).view(-1, K)
        ref = (x64 @ w64.t()).float().to(torch.bfloat16)
        off += (ref.view(torch.int16) != y[:, r:r + 2048].view(torch.int16)).sum().item()
    log_metric(test="q8_sum_error", M=M, N=N, K=K, share=off / (M * N))
    assert off <= share * M * N, f"{off} of {M * N} outputs ({off / (M * N):.2e}) off the correctly rounded value"
