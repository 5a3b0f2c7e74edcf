"""Which kernels the GPU tests reach, asked of the library on the host: every form of the
several-token matmul kernels that a call can reach must be in some test's list, whole and in
slices of K where it has both."""
import functools
import random

import pytest

from oracle import ssq_oracle as O
from tests import test_gpu_matmul as gm, test_gpu_q8 as gq
from tests.routes import route


@functools.lru_cache(None)
def covered():
    seen = set()
    for M, N, K, workspace in gm.STREAMING:
        for q, mode in gm.STREAMING_FORMATS:
            seen.add((q, route(M, N, K, 32, q, mode, workspace)))
    for M, N, K in gm.STREAMING_SLICES:
        for q, group, mode in gm.SLICE_FORMATS:
            seen.add((q, route(M, N, K, group, q, mode, True)))
    for _, M, N, K, workspace in gm.LARGE:
        for q in (2, 3, 4):
            seen.add((q, route(M, N, K, 128, q, O.SIGNED_SYM, workspace)))
    for M, N, K, workspace in gm.MIDDLE + gm.MIDDLE_GROUPS:
        for q in (2, 3, 4):
            seen.add((q, route(M, N, K, 32, q, O.SIGNED_SYM, workspace)))
    for _, split, M, N, Ks in gm.GEMM_FORMS:
        for q in (2, 3, 4):
            seen.add((q, route(M, N, Ks[64], 64, q, O.SIGNED_SYM, split)))
    return {form(q, r) for q, r in seen}


def form(q, r):
    """The compiled kernel, and whether its slices meet in the workspace.  Row tiles of a run of
    the exact kernel for large matrices are a loop, not a form."""
    return q, r.kernel, r.tokens, 0 if r.kernel == "stat" else r.rows, r.slices > 1


def test_every_reachable_form_is_tested():
    rng = random.Random(3)
    reached = {}
    for _ in range(60000):
        M = rng.choice((rng.randint(3, 80), rng.randint(3, 80), rng.randint(81, 2100)))
        N = int(2 ** rng.uniform(4, 15.2))
        K = 512 * rng.randint(1, 56) if rng.random() < 0.5 else 128 * rng.randint(1, 224)
        q, mode = rng.choice((2, 3, 4)), rng.choice((O.SIGNED_SYM, O.ASYM, O.ASYM_MIN))
        r = route(M, N, K, 128, q, mode, rng.random() < 0.8)
        reached.setdefault(form(q, r), (M, N, K, mode))
    missing = {f: s for f, s in reached.items() if f not in covered()}
    assert not missing, missing


@pytest.mark.parametrize("shapes,kernels", [
    (gq.Q8_TILES, ["q8_gemv", "q8_tile 32x64", "q8_tile 64x64", "q8_tile 64x128", "q8_tile 128x128"]),
    (gq.Q8_FEW, ["q8_gemv", "q8_gemv", "q8_gemv", "q8_gemv", "q8_tile 32x32", "q8_tile 32x32", "q8_tile 32x32", "q8_tile 32x64"]),
])
def test_q8_shapes_run_what_their_comments_say(shapes, kernels):
    for (M, N, K), want in zip(shapes, kernels):
        for q in (2, 3, 4):
            r = route(M, N, K, 32, q, O.SIGNED_SYM, q8=True)
            assert (r.kernel if r.kernel == "q8_gemv" else f"{r.kernel} {r.tokens}x{r.rows}") == want, (M, N, K, q)


@pytest.mark.parametrize("N,K,group,mode,kernel", [
    (20480, 5120, 32, O.SIGNED_SYM, "rounded"), (19456, 5632, 32, O.SIGNED_SYM, "split"),
    (24576, 3072, 32, O.SIGNED_SYM, "rounded"), (24576, 4096, 32, O.SIGNED_SYM, "split"),
    (28672, 2048, 32, O.SIGNED_SYM, "split"), (28672, 4096, 32, O.ASYM, "split"),
    (16448, 8192, 32, O.ASYM, "rounded"), (18432, 12288, 32, O.ASYM, "split"),
    (24576, 6144, 32, O.ASYM_MIN, "rounded"), (24576, 4096, 32, O.ASYM, "split"),
    (20480, 6144, 64, O.ASYM, "rounded"), (24576, 4096, 64, O.ASYM, "split"), (16448, 8192, 128, O.ASYM, "split"),
])
@pytest.mark.parametrize("M", [17, 24, 32])
def test_three_bit_rule_follows_its_measurements(M, N, K, group, mode, kernel):
    assert route(M, N, K, group, 3, mode, True).kernel == kernel


# Either side of the lines between kernels, where the rules name measured sizes.
@pytest.mark.parametrize("M,N,K,group,q,mode,kernel", [
    # short rows over 1024 row tiles: the GEMM above 32 tokens
    (64, 24896, 512, 64, 4, O.ASYM, "gemm"), (39, 29707, 1408, 32, 4, O.SIGNED_SYM, "gemm"), (43, 23004, 1792, 32, 4, O.ASYM, "rounded"),
    (41, 26432, 512, 32, 2, O.ASYM, "gemm"), (43, 19389, 1024, 32, 3, O.SIGNED_SYM, "rounded"), (49, 25796, 1408, 32, 3, O.ASYM, "gemm"),
    # just over 512 row tiles, rounded weights
    (18, 8320, 13312, 32, 2, O.ASYM_MIN, "split"), (24, 8411, 10752, 32, 4, O.SIGNED_SYM, "split"), (24, 8411, 9216, 32, 4, O.SIGNED_SYM, "rounded"),
    (9, 8768, 18304, 128, 3, O.SIGNED_SYM, "split"), (9, 8768, 16384, 128, 3, O.SIGNED_SYM, "rounded"),
    # exact weights with metadata: the streaming kernel's sums are closer
    (9, 7296, 19456, 128, 2, O.ASYM, "exact"), (16, 16704, 6144, 128, 4, O.ASYM, "exact"), (9, 16640, 9728, 32, 4, O.ASYM_MIN, "stat"),
])
def test_streaming_rules_follow_their_measurements(M, N, K, group, q, mode, kernel):
    assert route(M, N, K, group, q, mode, True).kernel == kernel


@pytest.mark.parametrize("M,N,K,q,mode,kernel", [
    (22, 257, 6144, 2, O.ASYM_MIN, "q8_gemv"), (4, 2437, 11776, 3, O.SIGNED_SYM, "q8_gemv"), (20, 1024, 1536, 4, O.ASYM, "q8_gemv"),
    (16, 1367, 2688, 2, O.SIGNED_SYM, "q8_gemv"), (8, 4096, 4096, 4, O.SIGNED_SYM, "q8_tile"), (17, 3918, 2048, 3, O.SIGNED_SYM, "q8_tile"),
    (41, 257, 6144, 2, O.ASYM_MIN, "q8_tile"), (1, 4096, 4096, 4, O.SIGNED_SYM, "q8_gemv"),
])
def test_q8_rule_follows_its_measurements(M, N, K, q, mode, kernel):
    assert route(M, N, K, 32, q, mode, q8=True).kernel == kernel
