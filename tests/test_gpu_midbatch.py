"""Batches of 17 to 64 tokens on the kernel of their own, at its edges: every
workgroup height (1, 2, 3, 4 and 6 row blocks) and token tile count, partial
last workgroups, a half packet at the end of K, wavefronts with no packet, one
and several packets each; both activation layouts (f16 row-major, bf16 through
the tiled copy); and the pre-pass that writes that copy, at both of its forms.
Every output element against the fp64 oracle at the small-batch bar (5e-4 of
max|y|: one fp16 rounding of the decoded weight)."""
import numpy as np
import pytest

import oracle
from paper_2606_10520_amd import workloads as wl
from test_gpu_parity import dev_x, lib, rel_err, run_shared, upload_pack, x_as_f64  # noqa: F401  (lib: fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2606_10520_amd.unisvq as u  # noqa: E402

# K = 1152: nine groups, five packets, the last half a packet, three of the
# eight wavefronts without one; heights as the launcher picks them
SETS = {
    "rb1": [(1040, 1152)],
    "rb2": [(4112, 1152)],
    "rb3": [(9168, 1152)],
    "rb4": [(16368, 1152)],
    "rb6": [(11008, 1152), (11008, 1152)],  # four at 49 tokens and more
    "long": [(272, 4224), (48, 11008), (16, 128), (32, 256)],
}


@pytest.mark.parametrize("M", [17, 31, 33, 48, 49, 64])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("which", sorted(SETS))
def test_edges(which, dtype, M):
    probs, refs = [], []
    for i, (N, K) in enumerate(SETS[which]):
        Q, A, B = wl.gen_weights(N, K, seed=310 + i)
        xb = wl.gen_activations(M, K, seed=315 + (0 if which == "rb6" else i), dtype=dtype, outliers=True)
        x = probs[0][3] if which == "rb6" and i else dev_x(xb, dtype)  # (one buffer: one scaled copy)
        probs.append((upload_pack(Q, A, B), N, K, x, None))
        refs.append(oracle.matmul(oracle.pack(Q, A, B)[0], N, K, x_as_f64(xb, dtype)))
    outs = u.gemm_batched(probs, out_dtype=torch.float32)
    again = u.gemm_batched(probs, out_dtype=torch.float32)
    outs16 = u.gemm_batched(probs, out_dtype=torch.float16)
    torch.cuda.synchronize()
    for (pk, N, K, x, _), y, y2, y16, ref in zip(probs, outs, again, outs16, refs):
        assert torch.equal(y, y2), (N, K)
        assert torch.equal(y16, y.to(torch.float16)), (N, K)
        assert rel_err(y.cpu().numpy(), ref) <= 5e-4, (N, K)
        if M <= 32:  # the same kernel and summation order alone
            assert torch.equal(y, u.gemm(pk, N, K, x, out_dtype=torch.float32)), (N, K)


@pytest.mark.parametrize("M", [17, 40, 64])
@pytest.mark.parametrize("per_group", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_shared_pairs(dtype, per_group, M):
    N, K = 2064, 1152
    y, (Q, A, B), xb = run_shared("gemm_shared", N, K, M, K // 128 if per_group else 1, dtype, seed=330)
    ref = oracle.matmul_shared(oracle.pack_codes(Q)[0], N, K, A, B, x_as_f64(xb, dtype))
    assert rel_err(y.cpu().numpy(), ref) <= 5e-4


@pytest.mark.parametrize("M", [17, 100, 511, 512, 513])
@pytest.mark.parametrize("K", [128, 2048, 2176, 8192])
def test_tiled_copy_per_token_scales(M, K):
    """Tokens scaled by powers of two from 2^-100 to 2^100, one of them zero:
    per token the error stays at the bar, whichever form of the pre-pass writes
    the copy (one workgroup per token up to 512 tokens)."""
    N = 32
    rng = np.random.default_rng(M + K)
    Q, A, B = wl.gen_weights(N, K, seed=340)
    base = wl.gen_activations(M, K, seed=341, dtype="bf16")
    x = dev_x(base, "bf16") * torch.from_numpy(np.exp2(rng.integers(-100, 101, (M, 1))).astype(np.float32)).to("cuda:0").bfloat16()
    x[M // 2] = 0
    y = u.gemm(upload_pack(Q, A, B), N, K, x, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.matmul(oracle.pack(Q, A, B)[0], N, K, x.double().cpu().numpy())
    got = y.double().cpu().numpy()
    assert not got[M // 2].any()
    for t in range(M):
        if t != M // 2:
            assert np.abs(got[t] - ref[t]).max() <= 1e-3 * np.abs(ref[t]).max(), t
