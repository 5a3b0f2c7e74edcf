"""GPU parity: ssq_matmul (GEMV at M = 1, 2, streaming MFMA kernels at 3 <= M <= 80 and the
kernels of large matrices at 3 <= M <= 32, small tiles and the GEMM above) and
ssq_matmul_f32 against the binary64 CPU oracle.  Where a test is about one kernel it asserts
the library's choice (tests/routes.py).

Every comparison is element-wise (tests/parity_common.py states the bound and its
derivation): one bf16 rounding of the output plus binary32 accumulation slack, plus,
on the MFMA paths that round each dequantized weight to bf16, C_W = 6 times the
standard scale of that rounding; the symmetric and zero-point formats on the MFMA
paths are also held to the exact model x bf16(W_hat)^T.  The binary32 path is held to
1e-5.  The relative L2 bar of the workloads (2e-2 bf16, 1e-3 binary32) is asserted
too.  Every output (and workspace) sits between guard bytes that are checked after
the call, and starts as NaN so an unwritten output fails.
"""
import numpy as np
import pytest
import torch

from oracle import ssq_oracle as O
from paper_2607_08779_amd import ssq, synth
from tests.routes import route
from tests.parity_common import (Guarded, assert_quant_equal, assert_within, bf16_round_f64,
                                 guarded_quant_outputs, log_metric, matmul_error_bound, rel_l2,
                                 sample_rows, to_device, weights_host, widen, y_to_f64)

pytestmark = pytest.mark.gpu

MODES = [O.SIGNED_SYM, O.UNSIGNED_SYM, O.ASYM, O.ASYM_MIN]
TOL_BF16 = 2e-2
TOL_F32 = 1e-3


def quantize_guarded(W, rows, cols, group, q, mode, tag=""):
    """ssq_quantize into guarded buffers; returns the plain tensors after checking the guards."""
    g = guarded_quant_outputs(rows, cols, group, q, mode)
    out = ssq.ssq_quantize(W, group, q, mode, out=tuple(b.t if b is not None else None for b in g))
    for b in g:
        if b is not None:
            b.check(f"{tag} quantize")
    return out


def exact_weight_path(M, K, q, workspace):
    """Whether ssq_matmul runs a batched-decode kernel that keeps every weight exact: q = 2 or
    4, 3 <= M <= 16, K a multiple of 512 and either a workspace or K <= 2048.  The other
    MFMA kernels round s (u - o) to bf16, so these are held to the exact-weight bound."""
    if q not in (2, 4) or not 3 <= M <= 16:
        return False
    return K % 512 == 0 and (workspace or K <= 2048)


def compare_matmul(y, x_real, ref_q, sel, K, group, q, bf16_x, tag, workspace=False):
    """Element-wise comparison of y[:, sel] (a GPU tensor) with the oracle; returns rel L2."""
    M = x_real.shape[0]
    y_ref = O.matmul(x_real, ref_q.codes, ref_q.scales, ref_q.zp, len(sel), K, group, q, mins=ref_q.mins)
    w_hat = O.dequantize(ref_q.codes, ref_q.scales, ref_q.zp, K, group, q, ref_q.mins)
    # batched decode and prefill round W_hat to bf16, except the exact-weight kernels
    rounded = bf16_x and M > 2 and not exact_weight_path(M, K, q, workspace)
    bound, S = matmul_error_bound(x_real, w_hat, y_ref, rounded, f32=not bf16_x)
    y_all = y_to_f64(y)
    assert not np.isnan(y_all).any(), f"{tag}: output elements left unwritten (NaN fill)"
    y_gpu = y_all[:, sel]
    worst = assert_within(y_gpu, y_ref, bound, tag)
    worst_model = None
    if rounded and ref_q.mins is None:
        y_model = np.asarray(x_real, np.float64) @ bf16_round_f64(w_hat).T
        bound_m = 2.0 ** -8 * np.abs(y_model) + 2.0 ** -12 * S
        worst_model = assert_within(y_gpu, y_model, bound_m, f"{tag} (bf16 weight model)")
    err = rel_l2(y_gpu, y_ref)
    log_metric(test=tag, M=M, N=int(ref_q.codes.shape[0]), K=K, q=q, group=group, rel_l2=err,
               max_err_over_bound=worst, max_err_over_model_bound=worst_model,
               dtype="bf16" if bf16_x else "f32")
    tol = TOL_BF16 if bf16_x else TOL_F32
    assert err <= tol, f"{tag}: rel L2 {err:.3e} > {tol}"
    return err


def check_matmul(w_host, x_host, group, q, mode, rows_idx=None, bf16_w=True, bf16_x=True, tag="",
                 workspace=False, repeat=1, need_split=True):
    """Quantize on the GPU, multiply on the GPU, compare with the oracle on rows_idx.
    With workspace=True the split-reduction entry point runs `repeat` times on one
    workspace and every result is checked (need_split=False: shapes whose plan does not
    split run without one)."""
    N, K = w_host.shape
    M = x_host.shape[0]
    W = to_device(w_host, bf16_w)
    codes, scales, zp = quantize_guarded(W, N, K, group, q, mode, tag=tag)
    X = to_device(x_host, bf16_x)
    ws = None
    if workspace:
        nbytes = ssq.ssq_matmul_workspace_size(M, N, K, group, q)
        assert nbytes > 0 or not need_split, "shape chosen to need a split"
        ws = Guarded((nbytes,), torch.uint8, fill=0) if nbytes else None
    sel = np.arange(N) if rows_idx is None else rows_idx
    ref_q = O.quantize(widen(w_host[sel], bf16_w), group, q, mode)
    assert_quant_equal((codes, scales, zp), ref_q, None if rows_idx is None else sel, tag=tag)
    xr = widen(x_host, bf16_x)
    err = None
    for r in range(repeat):          # same workspace, same answer every call
        y = Guarded((M, N), torch.bfloat16 if bf16_x else torch.float32)
        ssq.ssq_matmul(X, codes, scales, zp, N, K, group, q, out=y.t,
                       workspace=None if ws is None else ws.t)
        y.check(f"{tag} y (call {r})")
        if ws is not None:
            ws.check(f"{tag} workspace (call {r})")
        err = compare_matmul(y.t, xr, ref_q, sel, K, group, q, bf16_x, f"{tag} (call {r})",
                             workspace=ws is not None)
    return err


def rand_w(N, K, seed, bf16=True):
    return synth.weights(synth.WeightSpec(N, K, nu=5.0, scale=0.02, outlier_frac=0.001,
                                          seed=seed, bf16=bf16))


# ---------------------------------------------------------------------------
# Small and ragged cases, every format.
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("mode", MODES)
def test_gemv_small_all_formats(q, group, mode):
    w = rand_w(37, 1536, seed=10 * q + group)
    x = synth.activations(1, 1536, seed=q)
    check_matmul(w, x, group, q, mode, tag="gemv 37x1536")


@pytest.mark.parametrize("K", [32, 64, 4096 + 32])
def test_gemv_odd_reduction_lengths(K):
    w = rand_w(9, K, seed=K)
    x = synth.activations(1, K, seed=K)
    for mode in MODES:
        check_matmul(w, x, 32, 4, mode, tag=f"gemv K={K}")


@pytest.mark.parametrize("q,group", [(4, 32), (3, 64), (2, 128)])
def test_gemv_multi_pass_ragged(q, group):
    # K=17408 is 544 blocks: two passes of a 320-thread team, the second one partial.
    K = 17408
    w = rand_w(21, K, seed=q + group)
    x = synth.activations(1, K, seed=5)
    for mode in MODES:
        check_matmul(w, x, group, q, mode, tag=f"gemv multi-pass q={q} g={group}")


@pytest.mark.parametrize("mode", MODES)
def test_gemv_unaligned_metadata(mode):
    """Scales (and zero points) that start off a 16-byte boundary take the per-lane
    load path; the result equals the aligned call bit for bit."""
    N, K = 24, 2048
    w = rand_w(N, K, seed=3)
    codes, scales, zp = ssq.ssq_quantize(to_device(w, True), 32, 4, mode)
    X = to_device(synth.activations(1, K, seed=4), True)
    y_ref = ssq.ssq_matmul(X, codes, scales, zp, N, K, 32, 4)
    s_buf = torch.zeros(scales.numel() + 8, dtype=scales.dtype, device="cuda")
    s_off = s_buf[1:1 + scales.numel()].view(scales.shape)
    s_off.copy_(scales)
    z_off = None
    if zp is not None:
        z_buf = torch.zeros(zp.numel() + 16, dtype=zp.dtype, device="cuda")
        z_off = z_buf[3:3 + zp.numel()].view(zp.shape)
        z_off.copy_(zp)
    assert s_off.data_ptr() % 16 != 0
    y = ssq.ssq_matmul(X, codes, s_off, z_off, N, K, 32, 4)
    torch.cuda.synchronize()
    assert torch.equal(y, y_ref)


@pytest.mark.parametrize("M", [16, 96, 300])
@pytest.mark.parametrize("mode", MODES)
def test_matmul_unaligned_metadata(M, mode):
    """Batched decode and small tiles with scales (and zero points or minimums) that start
    off a 4-byte boundary (offsets of one element): the result equals the aligned call
    bit for bit, with and without the split workspace."""
    N, K = 200, 1056
    w = rand_w(N, K, seed=31)
    codes, scales, zp = ssq.ssq_quantize(to_device(w, True), 32, 4, mode)
    X = to_device(synth.activations(M, K, seed=32), True)
    s_buf = torch.zeros(scales.numel() + 8, dtype=scales.dtype, device="cuda")
    s_off = s_buf[1:1 + scales.numel()].view(scales.shape)
    s_off.copy_(scales)
    z_off = None
    if zp is not None:
        z_buf = torch.zeros(zp.numel() + 16, dtype=zp.dtype, device="cuda")
        z_off = z_buf[3:3 + zp.numel()].view(zp.shape) if zp.dtype == torch.uint8 else \
            z_buf[1:1 + zp.numel()].view(zp.shape)
        z_off.copy_(zp)
    assert s_off.data_ptr() % 4 != 0
    for ws in (None, ssq.ssq_matmul_workspace(M, N, K, 32, 4)):
        y_ref = ssq.ssq_matmul(X, codes, scales, zp, N, K, 32, 4, workspace=ws)
        y = ssq.ssq_matmul(X, codes, s_off, z_off, N, K, 32, 4, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), y_ref.view(torch.int16))


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 128])
@pytest.mark.parametrize("mode", MODES)
def test_tile_ragged_all_formats(q, group, mode):
    # small tiles: M=200, N=300 leave partial 32x32 tiles in both directions; at g=32, K=1056
    # is an odd number of 32-blocks (half of the last 64-deep step is empty)
    K = 1056 if group == 32 else 1152
    assert route(200, 300, K, group, q, mode).kernel == "tile"
    w = rand_w(300, K, seed=7 * q + group)
    x = synth.activations(200, K, seed=q + group)
    check_matmul(w, x, group, q, mode, tag=f"tile 200x300x{K}")


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("mode", MODES)
def test_rounded_all_formats(q, group, mode):
    # streaming, rounded weights: N=45 leaves a partial 16-row tile; K leaves a partial unit of
    # 256 (one, two or four blocks)
    K = {32: 1056, 64: 1088, 128: 1152}[group]
    assert route(7, 45, K, group, q, mode).kernel == "rounded"
    w = rand_w(45, K, seed=3 * q + group + mode)
    x = synth.activations(7, K, seed=q * group)
    check_matmul(w, x, group, q, mode, tag=f"rounded 7x45x{K}")


@pytest.mark.parametrize("M", [2, 15, 16, 17, 31, 32])
def test_rounded_token_counts(M):
    # one and two 16-token MFMA blocks, both partial and full (no workspace: weights rounded;
    # M=2 the GEMV); K=14336 spreads 56 units over 8 wavefronts
    assert M == 2 or route(M, 40, 14336, 32, 4, O.ASYM).kernel == "rounded"
    w = rand_w(40, 14336, seed=M)
    x = synth.activations(M, 14336, seed=M)
    for mode in MODES:
        check_matmul(w, x, 32, 4, mode, tag=f"rounded M={M}")


@pytest.mark.parametrize("K", [32, 64, 128, 4096 + 96])
def test_rounded_short_and_odd_reductions(K):
    # a lone partial unit, a partial last one
    w = rand_w(33, K, seed=K + 1)
    x = synth.activations(16, K, seed=K + 1)
    for mode in MODES:
        check_matmul(w, x, 32, 3, mode, tag=f"rounded K={K}")


@pytest.mark.parametrize("K", [32, 64, 96, 128, 192])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM])
def test_tile_short_reductions(K, mode):
    # small tiles of one unit, not full: most wavefronts have no work
    assert route(200, 300, K, 32, 4, mode).kernel == "tile"
    w = rand_w(300, K, seed=K + mode)
    x = synth.activations(200, K, seed=K)
    check_matmul(w, x, 32, 4, mode, tag=f"tile 200x300x{K}")


@pytest.mark.parametrize("M,N", [(300, 5000), (120, 6000)])       # 256 and 128 tokens a workgroup
@pytest.mark.parametrize("K", [32, 64, 96, 128, 192])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM])
def test_gemm_short_reductions(M, N, K, mode):
    # one to three 64-deep windows per tile: the loads of the window after the last one
    # (issued at the start of the tile, or by the last window) lie past K and read
    # nothing the result uses; signed scales take the two-window start, zero points not
    assert route(M, N, K, 32, 4, mode)[:2] == ("gemm", 256 if M > 128 else 128)
    w = np.ascontiguousarray(np.resize(rand_w(997, K, seed=K + mode), (N, K)))
    x = synth.activations(M, K, seed=K)
    check_matmul(w, x, 32, 4, mode, rows_idx=sample_rows(N, n=64, seed=K), tag=f"gemm {M}x{N}x{K}")


GEMM_FORMS = [      # tokens of a workgroup, split, shape (K per group: an odd number of 64-deep steps' halves)
    (128, False, 102, 4194, {32: 352, 64: 320, 128: 384}),
    (256, False, 131, 8313, {32: 672, 64: 704, 128: 640}),
    (128, True, 106, 2235, {32: 6304, 64: 6336, 128: 6272}),
    (256, True, 409, 882, {32: 9504, 64: 9536, 128: 9472}),
]


@pytest.mark.parametrize("tokens,split,M,N,Ks", GEMM_FORMS)
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_gemm_all_formats(tokens, split, M, N, Ks, q, group, mode):
    # ragged tiles both ways, whole and cut into slices of K
    K = Ks[group]
    r = route(M, N, K, group, q, mode, split)
    assert r[:2] == ("gemm", tokens) and (r.slices > 1) == split
    w = np.ascontiguousarray(np.resize(rand_w(min(N, 499), K, seed=q + group), (N, K)))
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, group, q, mode, rows_idx=sample_rows(N, n=40, seed=q), tag=f"gemm {M}x{N}x{K} q{q} g{group}",
                 workspace=split, repeat=2 if split else 1)


@pytest.mark.parametrize("M", [2, 3, 16, 32, 33, 129])
def test_token_counts_of_every_range(M):
    # GEMV, exact weights, rounded weights, small tiles
    w = rand_w(64, 512, seed=M)
    x = synth.activations(M, 512, seed=M)
    check_matmul(w, x, 32, 4, O.SIGNED_SYM, tag=f"M={M} 64x512")


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", MODES)
def test_tile_split_reduction_ragged(q, mode):
    # 32x32 tiles of 130x200 over K=3104 (97 blocks) in slices of K, the last ending in a unit of
    # one block; three calls on one workspace
    assert route(130, 200, 3104, 32, q, mode, True) == ("tile", 32, 32, 4)
    w = rand_w(200, 3104, seed=q + 10 * mode)
    x = synth.activations(130, 3104, seed=q)
    check_matmul(w, x, 32, q, mode, tag="split 130x200x3104", workspace=True, repeat=3)


@pytest.mark.parametrize("M,N,K", [(2048, 5120, 4096), (2000, 4700, 4096)])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM_MIN])
def test_gemm_split_last_round(M, N, K, mode):
    # more output tiles than CUs (320, and a ragged 296) with a last round less than half
    # full: those tiles (the weight panels from row 4096 on) are cut into K slices
    # through the workspace while the others are computed whole
    assert route(M, N, K, 32, 4, mode, True) == ("gemm", 256, 128, 4)
    w = rand_w(N, K, seed=N + mode)
    x = synth.activations(M, K, seed=M)
    rows = np.concatenate([sample_rows(4096, n=8, seed=1), 4096 + sample_rows(N - 4096, n=40, seed=2)])
    check_matmul(w, x, 32, 4, mode, rows_idx=rows, tag=f"split last round {M}x{N}x{K}", workspace=True,
                 repeat=2)


def test_gemm_output_past_one_gigabyte():
    """A 4096 x 131072 bf16 output (1 GiB): the GEMM stores it with 64-bit addresses rather
    than through a buffer descriptor; sampled rows against the oracle, guards checked."""
    N, K, M = 131072, 512, 4096
    assert route(M, N, K, 32, 4, O.SIGNED_SYM).kernel == "gemm"
    w = rand_w(N, K, seed=17)
    x = synth.activations(M, K, seed=17)
    rows = np.concatenate([sample_rows(N, n=24, seed=5), np.array([N - 129, N - 128, N - 127])])
    check_matmul(w, x, 32, 4, O.SIGNED_SYM, rows_idx=np.unique(rows), tag="gemm 4096x131072x512 (1 GiB y)")


def test_rounded_split_reduction_group_128():
    assert route(64, 160, 8192, 128, 4, O.SIGNED_SYM, True) == ("rounded", 64, 16, 4)
    w = rand_w(160, 8192, seed=5)
    x = synth.activations(64, 8192, seed=5)
    check_matmul(w, x, 128, 4, O.SIGNED_SYM, tag="split 64x160x8192", workspace=True, repeat=2)


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", MODES)
def test_rounded_with_workspace_ragged(q, mode):
    # batched decode with a workspace that its cut leaves alone: N=200 ends in half a row tile,
    # K=3104 in a unit of one block; three calls on one workspace
    assert route(7, 200, 3104, 32, q, mode, True) == ("rounded", 16, 16, 1)
    w = rand_w(200, 3104, seed=q + 10 * mode + 1)
    x = synth.activations(7, 3104, seed=q + 1)
    check_matmul(w, x, 32, q, mode, tag="rounded 7x200x3104", workspace=True, repeat=3)


@pytest.mark.parametrize("M", [3, 16, 17, 32])
@pytest.mark.parametrize("group", [32, 128])
def test_streaming_split_token_counts(M, group):
    # exact weights up to 16 tokens, rounded above, four slices of K
    assert route(M, 300, 8192, group, 4, O.ASYM, True).slices > 1
    w = rand_w(300, 8192, seed=M + group)
    x = synth.activations(M, 8192, seed=M + group)
    for mode in MODES:
        check_matmul(w, x, group, 4, mode, tag=f"streaming split M={M}", workspace=True, repeat=2)


# Exact weights (q = 2, 4; up to 16 tokens; K a multiple of 512).

@pytest.mark.parametrize("M", [5, 16])
@pytest.mark.parametrize("q", [2, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("mode", MODES)
def test_exact_all_formats(M, q, group, mode):
    # N=45: three 16-row tiles, the last one partial.  K=2560: ten units over eight wavefronts;
    # two calls on one workspace
    assert route(M, 45, 2560, group, q, mode, True).kernel == "exact"
    w = rand_w(45, 2560, seed=100 + 7 * q + group + mode + M)
    x = synth.activations(M, 2560, seed=q * group + M)
    check_matmul(w, x, group, q, mode, tag=f"exact {M}x45x2560", workspace=True, repeat=2)


@pytest.mark.parametrize("q", [2, 4])
@pytest.mark.parametrize("M,N,K,workspace", [
    (16, 6400, 4096, True),     # 400 tiles, two a workgroup
    (9, 9600, 6144, True),      # 600 tiles, three a workgroup
    (13, 4100, 3072, True),     # a 4-row last tile and a tile past N
    (16, 2000, 1024, False),    # four units: half of the wavefronts without work
])
def test_exact_row_tiles(q, M, N, K, workspace):
    assert route(M, N, K, 32, q, O.SIGNED_SYM, workspace).kernel == "exact"
    w = rand_w(N, K, seed=N + K + q)
    x = synth.activations(M, K, seed=M + q)
    for mode in (O.SIGNED_SYM, O.ASYM_MIN):
        check_matmul(w, x, 32, q, mode, rows_idx=sample_rows(N, n=48, seed=q), tag=f"exact row tiles {M}x{N}x{K}",
                     workspace=workspace, repeat=2 if workspace else 1, need_split=False)


@pytest.mark.parametrize("M,N,K", [
    (96, 256, 8192), (300, 256, 8192),           # small tiles
    (16, 256, 8192),                             # streaming, exact weights
    (106, 2235, 6272), (409, 882, 9472),         # GEMM, 128 and 256 tokens a workgroup
    (16, 23000, 6656), (24, 18500, 4224),        # large matrices, exact and rounded
])
def test_split_reduction_graph_replay(M, N, K):
    """The split kernels in a HIP graph: the arrival counters reset inside the kernel, so
    every replay (with eager work between) reproduces the first result."""
    assert route(M, N, K, 32, 4, O.SIGNED_SYM, True).slices > 1
    w = np.ascontiguousarray(np.resize(rand_w(min(N, 256), K, seed=8), (N, K)))
    W = to_device(w, True)
    codes, scales, _ = ssq.ssq_quantize(W, 32, 4, O.SIGNED_SYM)
    x_host = synth.activations(M, K, seed=8)
    x = to_device(x_host, True)
    ws = ssq.ssq_matmul_workspace(M, N, K, 32, 4)
    assert ws is not None
    y_eager = ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4, workspace=ws)
    sel = np.arange(N) if N <= 256 else sample_rows(N, n=64, seed=M)
    ref_q = O.quantize(widen(w[sel], True), 32, 4, O.SIGNED_SYM)
    compare_matmul(y_eager, widen(x_host, True), ref_q, sel, K, 32, 4, True, f"graph split M={M}",
                   workspace=True)
    y = torch.empty_like(y_eager)
    ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4, out=y, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4, out=y, workspace=ws)
    for _ in range(4):
        y.zero_()
        graph.replay()
        other = ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), y_eager.view(torch.int16))
        assert rel_l2(y_to_f64(other), y_to_f64(y_eager)) < 1e-2


@pytest.mark.parametrize("M", [1, 3, 5])
@pytest.mark.parametrize("mode", MODES)
def test_f32_path(M, mode):
    spec = synth.small_fp32().layers["w"]
    w = weights_host(spec)
    x = synth.activations(M, 512, seed=1100 + M, bf16=False)
    check_matmul(w, x, 32, 4, mode, bf16_w=False, bf16_x=False, tag=f"f32 256x512 M={M}")


def test_f32_path_other_formats():
    w = synth.weights(synth.WeightSpec(50, 768, nu=4.0, scale=0.02, seed=8, bf16=False))
    x = synth.activations(2, 768, seed=8, bf16=False)
    for q in (2, 3):
        for group in (64, 128):
            check_matmul(w, x, group, q, O.ASYM, bf16_w=False, bf16_x=False, tag="f32 other")


def test_zero_weights_give_zero_output():
    w = np.zeros((16, 256), np.uint16)
    for M in (1, 4):
        x = synth.activations(M, 256, seed=M)
        for mode in MODES:
            W = to_device(w, True)
            codes, scales, zp = ssq.ssq_quantize(W, 32, 4, mode)
            y = ssq.ssq_matmul(to_device(x, True), codes, scales, zp, 16, 256, 32, 4)
            torch.cuda.synchronize()
            assert (y.float() == 0).all()


def test_empty_matmul_is_a_noop():
    codes = torch.zeros((8, 32), dtype=torch.uint8, device="cuda")
    scales = torch.zeros((8, 2), dtype=torch.int16, device="cuda")
    y = ssq.ssq_matmul(torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda"),
                       codes, scales, None, 8, 64, 32, 4)
    assert y.shape == (0, 8)
    y = ssq.ssq_matmul(torch.zeros((3, 64), dtype=torch.bfloat16, device="cuda"),
                       codes, scales, None, 0, 64, 32, 4)
    torch.cuda.synchronize()
    assert y.shape == (3, 0)


@pytest.mark.parametrize("M", [1, 16, 64])
def test_graph_replay_matches_eager(M):
    """ssq_matmul captured in a HIP graph: every replay, with eager work in between,
    equals the eager result bit for bit."""
    N, K = 256, 2048
    w = rand_w(N, K, seed=77)
    W = to_device(w, True)
    codes, scales, _ = ssq.ssq_quantize(W, 32, 4, O.SIGNED_SYM)
    x_host = synth.activations(M, K, seed=M)
    x = to_device(x_host, True)
    y_eager = ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4)
    ref_q = O.quantize(widen(w, True), 32, 4, O.SIGNED_SYM)
    compare_matmul(y_eager, widen(x_host, True), ref_q, np.arange(N), K, 32, 4, True, f"graph M={M}")
    y = torch.empty_like(y_eager)
    ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4, out=y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4, out=y)
    for _ in range(4):
        y.zero_()
        graph.replay()
        scratch = ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4)   # eager work between
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), y_eager.view(torch.int16))
        assert torch.equal(scratch.view(torch.int16), y_eager.view(torch.int16))


# ---------------------------------------------------------------------------
# Full-size workloads (sampled output columns).
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("mode", MODES)
def test_llama3_8b_decode_gemv_full_size(mode):
    wl = synth.llama3_8b_decode()
    for name, spec in wl.layers.items():
        w = weights_host(spec)
        x = synth.activations(1, spec.cols, seed=wl.x_seed)
        check_matmul(w, x, 32, 4, mode, rows_idx=sample_rows(spec.rows, seed=spec.seed),
                     tag=f"decode {name}")


@pytest.mark.parametrize("q", [2, 3])
@pytest.mark.parametrize("group", [32, 64, 128])
def test_llama3_8b_block_gemv_full_size(q, group):
    wl = synth.llama3_8b_block()
    for name in ("q_proj", "k_proj", "gate_proj", "down_proj"):
        spec = wl.layers[name]
        w = weights_host(spec)
        x = synth.activations(1, spec.cols, seed=wl.x_seed)
        for mode in MODES:
            check_matmul(w, x, group, q, mode, rows_idx=sample_rows(spec.rows, n=24, seed=1),
                         tag=f"block {name}")


@pytest.mark.parametrize("M", [512, 2048])
@pytest.mark.parametrize("layer", ["gate_proj", "down_proj"])
def test_prefill_gemm_full_size(M, layer):
    wl = synth.prefill()
    spec = wl.layers[layer]
    w = weights_host(spec)
    x = synth.activations(M, spec.cols, seed=wl.x_seed + M)
    check_matmul(w, x, 32, 4, O.SIGNED_SYM, rows_idx=sample_rows(spec.rows, n=32, seed=M),
                 tag=f"prefill {layer} M={M}")


def test_prefill_gate_split_last_round_full_size():
    """M=2048 on the 14336x4096 gate projection with a workspace: 896 tiles, the last 128
    (rows 12288 on) cut in two K slices."""
    wl = synth.prefill()
    spec = wl.layers["gate_proj"]
    w = weights_host(spec)
    x = synth.activations(2048, spec.cols, seed=wl.x_seed + 2048)
    rows = np.concatenate([sample_rows(12288, n=8, seed=3), 12288 + sample_rows(spec.rows - 12288, n=24, seed=4)])
    check_matmul(w, x, 32, 4, O.SIGNED_SYM, rows_idx=rows, tag="prefill gate_proj M=2048 split last round",
                 workspace=True, repeat=2)


def test_prefill_headline_split_full_size():
    """M=512 on the 4096x14336 down projection through the split-reduction entry point."""
    wl = synth.prefill()
    spec = wl.layers["down_proj"]
    w = weights_host(spec)
    x = synth.activations(512, spec.cols, seed=wl.x_seed + 512)
    check_matmul(w, x, 32, 4, O.SIGNED_SYM, rows_idx=sample_rows(spec.rows, n=32, seed=9),
                 tag="prefill down_proj M=512 split", workspace=True, repeat=2)


@pytest.mark.parametrize("M", [16, 32])
def test_llama3_8b_batched_decode_full_size(M):
    """Batched decode through the split-reduction entry point on every Llama-3-8B
    projection shape, q=4 g=32, sampled rows; both the signed and the Q*_1 layout."""
    wl = synth.llama3_8b_decode()
    for name, spec in wl.layers.items():
        w = weights_host(spec)
        x = synth.activations(M, spec.cols, seed=wl.x_seed + M)
        for mode in (O.SIGNED_SYM, O.ASYM_MIN):
            check_matmul(w, x, 32, 4, mode, rows_idx=sample_rows(spec.rows, n=24, seed=M),
                         tag=f"8b {name} M={M}", workspace=True, repeat=2, need_split=False)


@pytest.mark.parametrize("M,workspace", [(1, False), (16, False), (16, True)])
def test_llama3_70b_matmul_full_size(M, workspace):
    """Every distinct 70B projection shape (q/o 8192x8192, k/v 1024x8192, gate/up
    28672x8192, down 8192x28672) at q=2 g=32, sampled rows."""
    wl = synth.llama3_70b_block()
    for name in ("q_proj", "k_proj", "gate_proj", "down_proj"):
        spec = wl.layers[name]
        w = synth.weights(spec)
        x = synth.activations(M, spec.cols, seed=wl.x_seed + M)
        check_matmul(w, x, 32, 2, O.SIGNED_SYM, rows_idx=sample_rows(spec.rows, n=24, seed=M),
                     tag=f"70b {name} M={M}", workspace=workspace, repeat=2 if workspace else 1, need_split=False)


@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 128])
@pytest.mark.parametrize("mode", MODES)
def test_gemv_two_tokens_all_formats(q, group, mode):
    # M = 2 takes the two-token GEMV: 37 rows (ragged row groups), K = 19200 (two passes)
    w = rand_w(37, 19200, seed=q * 7 + group + mode)
    x = synth.activations(2, 19200, seed=q + group)
    check_matmul(w, x, group, q, mode, tag=f"gemv M=2 q={q} g={group} m={mode}")


@pytest.mark.parametrize("mode", MODES)
def test_gemv_two_tokens_full_size(mode):
    # 4096x14336 at M = 2: seven wavefronts each staging two tokens' activations plus
    # the scales and metadata (the largest LDS of the GEMV), sampled rows
    spec = synth.llama3_8b_decode().layers["down_proj"]
    w = weights_host(spec)
    x = synth.activations(2, spec.cols, seed=77)
    check_matmul(w, x, 32, 4, mode, rows_idx=sample_rows(spec.rows, 48, seed=mode), tag=f"gemv M=2 full m={mode}")


@pytest.mark.parametrize("M,N,K", [
    (1, 3073, 96),      # past the short-matrix kernel: one super-block of three blocks, ragged rows
    (3, 1024, 544),     # its largest three-token matrix
    (1, 4219, 1184),    # its one token past the 4096 rows of a round
    (4, 17, 32),        # one block: one wavefront, three tokens and a row past the tile's 16
    (8, 40, 4256),      # 34 super-blocks over 16 wavefronts (three steps for two of them)
    (9, 33, 2208),      # 16-token stages, 18 super-blocks over 8 wavefronts
    (35, 50, 1056),     # three token tiles, the last of three
])
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_f32_matmul_edges(M, N, K, q, mode):
    w = rand_w(N, K, seed=M + N + q, bf16=False)
    x = synth.activations(M, K, seed=M + mode, bf16=False)
    check_matmul(w, x, 32, q, mode, bf16_w=False, bf16_x=False, tag=f"f32 {M}x{N}x{K}")


def test_f32_rows_sum_error():
    """Sums of the wavefront-per-row kernel against 64 bits (2-norm): a block in one chain of 32
    gives 1.24e-7 here, in four chains a fifth less; either varies by about 1 % over 4219 outputs."""
    N, K = 4219, 8192
    gen = torch.Generator(device="cuda").manual_seed(5)
    codes, scales, _ = ssq.ssq_quantize((0.02 * torch.randn((N, K), generator=gen, device="cuda")).to(torch.bfloat16), 32, 4, O.SIGNED_SYM)
    x = torch.randn((1, K), generator=gen, device="cuda")
    y = ssq.ssq_matmul(x, codes, scales, None, N, K, 32, 4)
    u = torch.stack([codes & 15, codes >> 4], dim=2).double().view(N, K // 32, 32)
    w64 = ((u - 8) * scales.view(torch.float16).double()[..., None]).view(N, K)
    ref = x.double() @ w64.t()
    err = ((y.double() - ref).norm() / ref.norm()).item()
    log_metric(test="f32_rows_sum_error", rel_l2=err)
    assert err <= 1.03e-7, f"rel L2 {err:.3e}"


@pytest.mark.parametrize("M,N,K", [(4, 40, 896), (8, 33, 2432), (17, 50, 1152)])       # 4, 8 and 16 tokens a stage
@pytest.mark.parametrize("q", [2, 3, 4])
@pytest.mark.parametrize("group", [64, 128])
@pytest.mark.parametrize("mode", [O.SIGNED_SYM, O.ASYM, O.ASYM_MIN])
def test_f32_matmul_groups(M, N, K, q, group, mode):
    w = rand_w(N, K, seed=M + N + q, bf16=False)
    x = synth.activations(M, K, seed=M + mode, bf16=False)
    check_matmul(w, x, group, q, mode, bf16_w=False, bf16_x=False, tag=f"f32 {M}x{N}x{K} g{group}")


@pytest.mark.parametrize("M,N,K,workspace", [
    (1, 45, 1536, False), (2, 45, 1536, False),                                    # GEMV
    (5, 45, 1536, False), (16, 4500, 512, False), (9, 45, 2560, True),             # exact weights
    (12, 8192, 2048, False),                                                       # exact, large matrix
    (7, 50, 288, False), (40, 300, 1056, False), (100, 300, 1056, False), (300, 300, 1056, False),
])
@pytest.mark.parametrize("q", [2, 4])
def test_zero_points_past_the_code_range(M, N, K, workspace, q):
    """Any byte is a zero point (a checkpoint's need not lie on the grid that ssq_quantize
    makes): odd ones from 129 on, whose 128 + z has nine significant bits."""
    rng = np.random.default_rng(M + N + q)
    ref_q = O.quantize(widen(rand_w(min(N, 97), K, seed=M + q), True), 32, q, O.ASYM)
    assert N != 8192 or route(M, N, K, 32, q, O.ASYM, workspace).kernel == "stat"
    ref_q.zp[:] = rng.integers(64, 128, size=ref_q.zp.shape) * 2 + 1
    rows = np.resize(np.arange(len(ref_q.zp)), N)
    dev = [torch.from_numpy(np.ascontiguousarray(a[rows])).cuda() for a in (ref_q.codes, ref_q.scales.view(np.int16), ref_q.zp)]
    x = synth.activations(M, K, seed=M)
    ws = ssq.ssq_matmul_workspace(M, N, K, 32, q) if workspace else None
    y = Guarded((M, N), torch.bfloat16)
    ssq.ssq_matmul(to_device(x, True), *dev, N, K, 32, q, out=y.t, workspace=ws)
    y.check("zero points past the code range")
    sel = sample_rows(N, n=64, seed=q)
    part = ref_q._replace(codes=ref_q.codes[rows[sel]], scales=ref_q.scales[rows[sel]], zp=ref_q.zp[rows[sel]])
    compare_matmul(y.t, widen(x, True), part, sel, K, 32, q, True, f"zero points {M}x{N}x{K} q{q}", workspace=workspace)


# ---------------------------------------------------------------------------
# Streaming kernels (3 <= M <= 80): every tile of tokens (8 to 80) and every number of
# 16-row tiles per workgroup, with all of K in a workgroup and in slices, and the large
# matrices that go to the kernels cut across small workgroups instead.
# ---------------------------------------------------------------------------
STREAMING = [
    # exact weights, 8 tokens: 1, 2 (a short last tile), 3 and 4 row tiles a workgroup
    (5, 17, 512, False), (8, 4100, 1536, False), (5, 9000, 1024, False), (3, 12300, 1024, False),
    # 16 tokens: 2 to 4 row tiles, four slices of K, a workspace left alone
    (16, 4500, 512, False), (9, 8200, 512, False), (13, 12500, 512, False), (16, 200, 8192, True),
    (11, 3000, 4608, True),
    # rounded weights; 9 or 17 blocks of K: a unit of one block after one or two full ones
    (7, 50, 288, False), (16, 4097, 544, False), (10, 9000, 800, False), (12, 12500, 800, False), (14, 70, 4128, True),
    (17, 4090, 544, False), (25, 8100, 320, False), (32, 12200, 320, False), (20, 16001, 288, False),
    (31, 20000, 288, False), (24, 1000, 4128, True),
    (33, 4000, 288, False), (48, 7000, 288, False), (40, 16000, 288, False), (40, 300, 8192, True),
    (49, 3000, 288, False), (64, 8100, 544, False), (50, 15000, 288, False), (64, 520, 4128, True),
    (65, 3001, 288, False), (79, 8000, 288, False), (80, 12000, 1056, False), (66, 16000, 1056, False), (70, 16000, 288, False),
    (77, 200, 4352, True), (81, 200, 4352, True),                # 81 tokens: a small tile
    # more than 1024 row tiles: exact in one slice, exact in several, rounded
    (13, 18500, 1024, False), (16, 23000, 6656, True), (24, 18500, 4128, True), (7, 18500, 4128, True),
]
STREAMING_FORMATS = [(2, O.SIGNED_SYM), (3, O.ASYM), (4, O.ASYM_MIN), (4, O.SIGNED_SYM)]


@pytest.mark.parametrize("M,N,K,workspace", STREAMING)
@pytest.mark.parametrize("q,mode", STREAMING_FORMATS)
def test_streaming_tiles(M, N, K, workspace, q, mode):
    w = rand_w(min(N, 997), K, seed=M + N + q)
    w = np.ascontiguousarray(np.resize(w, (N, K)))          # 997 rows, repeated
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, 32, q, mode, rows_idx=sample_rows(N, n=64, seed=q), tag=f"streaming {M}x{N}x{K} q{q}",
                 workspace=workspace, repeat=2 if workspace else 1, need_split=False)


# Several row tiles a workgroup and several slices of K, in every group size: exact weights of 8
# and 16 tokens, rounded ones of 16 to 80.
STREAMING_SLICES = [
    (4, 33, 4608), (4, 1474, 10240), (6, 1608, 14336), (4, 2233, 13824),
    (9, 35, 4608), (11, 1085, 12800), (16, 1232, 12800), (10, 4265, 5632),
    (13, 1396, 8576), (4, 1849, 8320), (8, 4292, 4736),
    (20, 34, 2176), (20, 1482, 4224), (20, 2139, 6272), (23, 4101, 4224), (18, 3478, 8576),
    (35, 33, 2176), (40, 1364, 4224), (33, 1656, 8320),
    (49, 33, 2176), (50, 2168, 2176), (50, 2729, 4224),
    (65, 38, 2176), (66, 1051, 6272), (65, 1399, 10368),
]
SLICE_FORMATS = [(2, 64, O.ASYM), (3, 128, O.SIGNED_SYM), (3, 64, O.ASYM_MIN), (4, 128, O.ASYM), (4, 64, O.SIGNED_SYM), (4, 32, O.ASYM_MIN)]


@pytest.mark.parametrize("M,N,K", STREAMING_SLICES)
@pytest.mark.parametrize("q,group,mode", SLICE_FORMATS)
def test_streaming_slices(M, N, K, q, group, mode):
    r = route(M, N, K, group, q, mode, True)
    assert r.kernel in ("exact", "rounded")
    assert r.slices > 1 or mode != O.SIGNED_SYM       # 80 rows with metadata do not fit the LDS
    w = np.ascontiguousarray(np.resize(rand_w(min(N, 211), K, seed=M + N + q), (N, K)))
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, group, q, mode, rows_idx=sample_rows(N, n=48, seed=q), tag=f"slices {M}x{N}x{K} q{q} g{group}",
                 workspace=True, repeat=2)


# Large matrices (skinny.hip): more than 1024 row tiles, every group size and layout.
LARGE = [
    ("stat", 13, 16500, 1024, False), ("stat", 15, 17203, 9216, True),      # exact: one slice of K, five
    ("split", 7, 16431, 1152, True), ("split", 24, 17408, 7168, True),      # rounded: 16 and 32 tokens
]


LARGE_FORMATS = [(32, O.ASYM), (64, O.SIGNED_SYM), (64, O.ASYM_MIN), (128, O.SIGNED_SYM), (128, O.ASYM), (128, O.ASYM_MIN)]
# 3-bit weights are never exact, and those with metadata may stream at more than 16 tokens
LARGE_CASES = [(*case, q, group, mode) for case in LARGE for q in (2, 3, 4) for group, mode in LARGE_FORMATS
               if q != 3 or (case[0] == "split" and (case[1] <= 16 or group == 128 or mode == O.SIGNED_SYM))]


@pytest.mark.parametrize("kernel,M,N,K,workspace,q,group,mode", LARGE_CASES)
def test_large_matrices(kernel, M, N, K, workspace, q, group, mode):
    r = route(M, N, K, group, q, mode, workspace)
    assert r.kernel == kernel and (r.slices > 1) == workspace
    w = np.ascontiguousarray(np.resize(rand_w(499, K, seed=M + N + q), (N, K)))
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, group, q, mode, rows_idx=sample_rows(N, n=48, seed=q), tag=f"{kernel} {M}x{N}x{K} q{q} g{group}",
                 workspace=workspace, repeat=2 if workspace else 1, need_split=False)


# ---------------------------------------------------------------------------
# Middle token counts: small tiles whose wavefronts split K, 32 x 32 to 128 x 64, unsliced
# and in slices of K; ragged rows and tokens; units of one block, units without work.
# ---------------------------------------------------------------------------
MIDDLE = [
    (81, 300, 1056, False), (83, 500, 8192, True),              # 32 tokens x 32 rows
    (100, 40, 288, False), (160, 2050, 2080, False), (120, 500, 16416, True),    # 64 x 32
    (95, 8100, 1056, False), (190, 600, 4128, True),            # 96 x 32
    (250, 4000, 1056, False), (200, 900, 12288, True),          # 64 x 64
    (350, 4070, 2080, False), (147, 2500, 8224, True),          # 96 x 64
    (300, 4100, 2336, False), (213, 1379, 7680, True),          # 128 x 64
    (64, 9000, 3424, True),                                     # from the streaming range: 64 x 64
    (128, 12200, 1056, False),                                  # past them: the GEMM
]


@pytest.mark.parametrize("M,N,K,workspace", MIDDLE)
@pytest.mark.parametrize("q,group,mode", [(2, 32, O.ASYM), (3, 32, O.SIGNED_SYM), (4, 32, O.ASYM_MIN), (4, 32, O.SIGNED_SYM)])
def test_middle_tiles(M, N, K, workspace, q, group, mode):
    w = rand_w(min(N, 997), K, seed=M + N + q)
    w = np.ascontiguousarray(np.resize(w, (N, K)))
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, group, q, mode, rows_idx=sample_rows(N, n=64, seed=q), tag=f"middle {M}x{N}x{K} q{q}",
                 workspace=workspace, repeat=2 if workspace else 1, need_split=False)


# The same tiles in the other group sizes: K of whole groups, units partly filled.
MIDDLE_GROUPS = [
    (81, 300, 1152, False), (83, 500, 8320, True), (160, 2050, 2176, False), (120, 500, 16512, True),
    (95, 8100, 1152, False), (190, 600, 4224, True), (250, 4000, 1152, False), (200, 900, 12416, True),
    (350, 4070, 2176, False), (147, 2500, 8320, True), (300, 4100, 2432, False), (213, 1379, 7680, True),
]


@pytest.mark.parametrize("M,N,K,workspace", MIDDLE_GROUPS)
@pytest.mark.parametrize("q,group,mode", [(2, 64, O.SIGNED_SYM), (2, 128, O.ASYM_MIN), (3, 64, O.ASYM), (3, 128, O.ASYM_MIN),
                                          (4, 64, O.ASYM_MIN), (4, 128, O.ASYM)])
def test_middle_tiles_groups(M, N, K, workspace, q, group, mode):
    r = route(M, N, K, group, q, mode, workspace)
    assert r.kernel == "tile" and (r.slices > 1) == workspace
    w = np.ascontiguousarray(np.resize(rand_w(min(N, 499), K, seed=M + N + q), (N, K)))
    x = synth.activations(M, K, seed=M + mode)
    check_matmul(w, x, group, q, mode, rows_idx=sample_rows(N, n=48, seed=q), tag=f"middle {M}x{N}x{K} q{q} g{group}",
                 workspace=workspace, repeat=2 if workspace else 1, need_split=False)
