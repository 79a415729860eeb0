"""LDLQ's candidate search and its products at their edges, against the fp64
oracle, bit for bit: targets on and next to the planes between codewords
(several candidates: the fp64 distances decide, the lowest index on ties),
pairs and targets over many magnitudes, and shapes around the 16-row, 128-row
and 128-column tiles (one to five blocks, odd and even numbers of row blocks).
"""
import numpy as np
import pytest

import oracle
from test_gpu_ldlq import hessian, lib, pairs, run_gpu  # noqa: F401  (lib: fixture that loads the library)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(W, U, A, B, ga):
    got = run_gpu(W, U, A, B, ga)
    ref, _ = oracle.ldlq(W, U, A, B, shared=(ga != 0))
    assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} codes differ"


@pytest.mark.parametrize("N,K", [(16, 128), (16, 256), (48, 384), (144, 512), (128, 640), (272, 640), (112, 256)])
def test_shapes(N, K):
    rng = np.random.default_rng(N * K)
    W = rng.standard_normal((N, K)).astype(np.float32)
    check(W, oracle.ldl_blocks(hessian(rng, K))[0], *pairs(rng, N, K, "row_group"))


@pytest.mark.parametrize("kind", ["same", "axis", "zero", "rank1"])
def test_ties(kind):
    """Every target halfway between codewords, exactly: A = B's grid axes, an
    all-zero A (256 equal codewords) or a rank-one A."""
    rng = np.random.default_rng(5)
    N, K = 32, 256
    W = (rng.integers(-4, 11, (N, K)) / 2).astype(np.float32)
    A = {"same": np.ones((4, 4)), "axis": np.eye(4), "zero": np.zeros((4, 4)),
         "rank1": np.outer([1, 2, -1, 1], [1, 1, 0, 0])}[kind]
    A = np.tile(A.astype(np.float16), (N, K // 128, 1, 1))
    B = np.zeros((N, K // 128, 4), np.float16)
    check(W, np.eye(K), A, B, 0)


@pytest.mark.parametrize("ulps", [0, 1, 40, 4000])
def test_near_ties(ulps):
    """Targets some fp32 steps off the plane between two codewords."""
    rng = np.random.default_rng(ulps)
    N, K = 64, 256
    W = (rng.integers(0, 3, (N, K)) + 0.5).astype(np.float32)
    W = (W + np.float32(2.0 ** -23) * rng.integers(-ulps, ulps + 1, (N, K))).astype(np.float32)
    A = np.tile(np.eye(4, dtype=np.float16), (N, K // 128, 1, 1))
    check(W, np.eye(K), A, np.zeros((N, K // 128, 4), np.float16), 0)


@pytest.mark.parametrize("a,w", [(1.0, 1e-30), (1.0, 1e4), (1e-6, 1.0), (3e-7, 1e-7), (2e4, 1e4), (1.0, 1e20), (1e-3, 3e38)])
def test_magnitudes(a, w):
    """Pair entries near the ends of fp16, targets from far below to far above
    the grid (beyond fp32's squares included)."""
    rng = np.random.default_rng(int(a * 1e7) % 1000 + 1)
    N, K = 32, 384
    W = (rng.standard_normal((N, K)) * w).astype(np.float32)
    A = (rng.uniform(-1, 1, (N, K // 128, 4, 4)) * a).astype(np.float16)
    B = (rng.uniform(-1, 1, (N, K // 128, 4)) * a).astype(np.float16)
    U, _ = oracle.ldl_blocks(hessian(rng, K))
    check(W, U, A, B, 0)


def test_workspace_at_16_bytes():
    """A workspace aligned to 16 bytes and no more, with stale NaNs in it."""
    import paper_2606_10520_amd.unisvq as u
    from test_gpu_ldlq import DEV, dev_half
    rng = np.random.default_rng(21)
    N, K = 48, 640
    W = rng.standard_normal((N, K)).astype(np.float32)
    A, B, ga = pairs(rng, N, K, "row_group")
    U, _ = oracle.ldl_blocks(hessian(rng, K))
    buf = torch.full((u.ldlq_workspace_bytes(N, K) // 8 + 64,), float("nan"), dtype=torch.float64, device=DEV)
    off = (16 - buf.data_ptr()) % 32 // 8  # doubles to an address of 16 modulo 32
    got = u.ldlq(torch.from_numpy(W).to(DEV), torch.from_numpy(U).to(DEV), dev_half(A), dev_half(B), ga,
                 workspace=buf[off:].view(torch.uint8))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.ldlq(W, U, A, B, shared=False)[0])
