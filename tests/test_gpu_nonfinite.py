"""Pairs with infinite or subnormal entries through the kernels that decode
weights on the matrix cores (1 to 7 row blocks per workgroup up to 16 tokens,
17 to 64 tokens, tiled): an infinite entry of A or B makes its own component of
the vectors of its row and group infinite and leaves the other three finite, as
the definition W = A q + B has it."""
import numpy as np
import pytest

import oracle
from paper_2606_10520_amd import workloads as wl
from test_gpu_parity import dev_u16_as_half, dev_x, lib, rel_err, upload_pack, x_as_f64  # noqa: F401  (lib: fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2606_10520_amd.unisvq as u  # noqa: E402

# heights 1, 2, 3 (an absent row block in the last workgroup) and 7 up to 16 tokens
SHAPES = [(1040, 1152), (4112, 1152), (8208, 1152), (25600, 384)]


@pytest.mark.parametrize("M", [2, 8, 24, 64, 100])
@pytest.mark.parametrize("N,K", SHAPES)
def test_infinite_entries(N, K, M):
    """Codes 1 to 3, positive pairs and activations: with an infinite entry (each
    position of A and B once, both signs) a row's sums are infinite, with no
    0 * inf or inf - inf in the definition, and every other row is finite."""
    rng = np.random.default_rng(N + M)
    Q = rng.integers(1, 4, (N, K), dtype=np.uint8)
    A = rng.uniform(0.01, 0.05, (N, K // 128, 4, 4)).astype(np.float16)
    B = rng.uniform(0.01, 0.05, (N, K // 128, 4)).astype(np.float16)
    sign = np.zeros(N)
    for i in range(20):  # row, group, entry, sign
        r, g, s = (i * N) // 20 + i % 16, i % (K // 128), 1.0 if i % 3 else -1.0
        sign[r] = s
        if i < 16:
            A[r, g, i // 4, i % 4] = s * np.inf
        else:
            B[r, g, i - 16] = s * np.inf
    x = rng.uniform(0.5, 1.0, (M, K)).astype(np.float16)
    y = u.gemm(upload_pack(Q, A, B), N, K, torch.from_numpy(x).to("cuda:0"), out_dtype=torch.float32)
    torch.cuda.synchronize()
    got, hit = y.cpu().numpy(), sign != 0
    assert np.array_equal(got[:, hit], np.broadcast_to(sign[hit] * np.inf, (M, hit.sum())))
    assert np.isfinite(got[:, ~hit]).all()


@pytest.mark.parametrize("M", [2, 8, 24, 64, 100])
def test_infinite_entry_of_a_shared_pair(M):
    """One pair per group, an entry of the last one (component 2) infinite: with
    positive activations every sum is +inf."""
    N, K = 272, 640
    rng = np.random.default_rng(M)
    Q = rng.integers(1, 4, (N, K), dtype=np.uint8)
    A = rng.uniform(0.01, 0.05, (K // 128, 4, 4)).astype(np.float16)
    B = rng.uniform(0.01, 0.05, (K // 128, 4)).astype(np.float16)
    A[-1, 2, 1] = np.inf
    pc, pa = u.pack_shared(torch.from_numpy(Q).to("cuda:0"), dev_u16_as_half(A), dev_u16_as_half(B))
    x = torch.from_numpy(rng.uniform(0.5, 1.0, (M, K)).astype(np.float16)).to("cuda:0")
    y = u.gemm_shared(pc, pa, N, K, K // 128, x, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert torch.equal(y, torch.full_like(y, float("inf")))


@pytest.mark.parametrize("M", [2, 8, 24, 64, 100])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_subnormal_entries(dtype, M):
    """Pairs of a few steps of 2^-24, so that every weight is a subnormal fp16
    value or one just above, without rounding: what is left are the fp32 sums
    (at most K + 3 roundings of 2^-24, K = 1152) and, for bf16 activations with
    outliers, the fp16 copy's (below 2^-14 of the row's largest value)."""
    N, K = 1040, 1152
    rng = np.random.default_rng(M)
    Q = rng.integers(0, 4, (N, K), dtype=np.uint8)
    A = (rng.integers(-60, 61, (N, K // 128, 4, 4)) * 2.0 ** -24).astype(np.float16)
    B = (rng.integers(-60, 61, (N, K // 128, 4)) * 2.0 ** -24).astype(np.float16)
    xb = wl.gen_activations(M, K, seed=7, dtype=dtype, outliers=True)
    y = u.gemm(upload_pack(Q, A, B), N, K, dev_x(xb, dtype), out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.matmul(oracle.pack(Q, A, B)[0], N, K, x_as_f64(xb, dtype))
    assert rel_err(y.cpu().numpy(), ref) <= 1e-4
