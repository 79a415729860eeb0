"""Batches of 17 to 64 tokens on the kernel of their own, at its edges: every
workgroup height (1, 2, 3, 4 and 6 row blocks) and token tile count, partial
last workgroups, a half packet at the end of K, wavefronts with no packet, one
and several packets each; both activation layouts (f16 row-major and copied to
tiles, bf16 through the scaled tiled copy); and the pre-pass that writes that
copy, at both of its forms.  A batch equals its problems alone bit for bit where
both take this kernel (the library's own rule says where).  Every output element against the fp64 oracle at the small-batch bar (5e-4 of
max|y|: one fp16 rounding of the decoded weight)."""
import numpy as np
import pytest

import oracle
from paper_2606_10520_amd import workloads as wl
from test_mid_plan_cpu import plan
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
    "rb6": [(11008, 1152), (11008, 1152)],  # three at 49 tokens and more
    "long": [(272, 4224), (48, 11008), (16, 128), (32, 256)],  # (above 32 tokens the tiled product)
}


def served(shapes, M, dtype):
    """The rule's answer for a batch of (N, K): whether this kernel serves it, and through a copy."""
    room = all(u.gemm_workspace_bytes(N, K, M, torch.float16) >= -(-M // 16) * 16 * K * 2 for N, K in shapes)
    return plan([N for N, _ in shapes], max(K for _, K in shapes), M, dtype, room)


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
        if served(SETS[which], M, dtype)[0] and served([(N, K)], M, dtype)[0]:
            assert torch.equal(y, u.gemm(pk, N, K, x, out_dtype=torch.float32)), (N, K)


# Batches whose f16 activations are copied to tiles: one buffer for three
# problems, a ragged second problem, several packets per wavefront with a half
# one at the end; and one above 32 tokens that is not copied.
COPY_SETS = {
    "qkv": ([(4096, 4096)] * 3, (33, 49, 63)),
    "down": ([(4096, 11008), (272, 4224)], (24, 33, 64)),
    "long": ([(4112, 8320), (1040, 2176)], (32, 48, 50)),
    "rows": ([(2064, 3712)], (33, 34)),
}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("which,M", [(w, m) for w, (_, ms) in sorted(COPY_SETS.items()) for m in ms])
def test_copied_activations(which, M, dtype):
    shapes = COPY_SETS[which][0]
    assert served(shapes, M, dtype) == (True, dtype == "bf16" or which != "rows")
    probs, refs = [], []
    for i, (N, K) in enumerate(shapes):
        one_x = which == "qkv"
        Q, A, B = wl.gen_weights(N, K, seed=350 + i)
        xb = wl.gen_activations(M, K, seed=355 + (0 if one_x else i), dtype=dtype, outliers=True)
        x = probs[0][3] if one_x and i else dev_x(xb, dtype)
        probs.append((upload_pack(Q, A, B), N, K, x, None))
        refs.append(oracle.matmul(oracle.pack(Q, A, B)[0], N, K, x_as_f64(xb, dtype)))
    outs = u.gemm_batched(probs, out_dtype=torch.float32)
    again = u.gemm_batched(probs, out_dtype=torch.float32)
    singles = [u.gemm(pk, N, K, x, out_dtype=torch.float32) for pk, N, K, x, _ in probs]
    torch.cuda.synchronize()
    compared = 0
    for (pk, N, K, x, _), y, y2, y1, ref in zip(probs, outs, again, singles, refs):
        assert torch.equal(y, y2), (N, K)
        assert rel_err(y.cpu().numpy(), ref) <= 5e-4, (N, K)
        if served([(N, K)], M, dtype)[0]:
            compared += 1
            assert torch.equal(y, y1), (N, K)
    assert compared


@pytest.mark.parametrize("per_group", [False, True])
@pytest.mark.parametrize("N,M", [(1024, 24), (4096, 63)])
def test_copied_activations_shared_pairs(N, M, per_group):
    K = 11008
    assert served([(N, K)], M, "f16") == (True, True)
    y, (Q, A, B), xb = run_shared("gemm_shared", N, K, M, K // 128 if per_group else 1, "f16", seed=360)
    ref = oracle.matmul_shared(oracle.pack_codes(Q)[0], N, K, A, B, x_as_f64(xb, "f16"))
    assert rel_err(y.cpu().numpy(), ref) <= 5e-4


# Both sides of the rule's lines where the tiled product takes over: long and
# narrow, 32768 rows, K below 512.
@pytest.mark.parametrize("N,K,M,serves", [(1024, 8192, 48, True), (1008, 8192, 48, False), (32752, 640, 32, True),
                                          (32768, 640, 32, False), (32768, 640, 33, False), (16384, 384, 32, True),
                                          (16400, 384, 32, False), (32768, 1152, 17, True)])
def test_both_sides_of_the_rule(N, K, M, serves):
    for dtype in ("f16", "bf16"):
        assert served([(N, K)], M, dtype)[0] == serves
        Q, A, B = wl.gen_weights(N, K, seed=370)
        xb = wl.gen_activations(M, K, seed=371, dtype=dtype)
        y = u.gemm(upload_pack(Q, A, B), N, K, dev_x(xb, dtype), out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert rel_err(y.cpu().numpy(), oracle.matmul(oracle.pack(Q, A, B)[0], N, K, x_as_f64(xb, dtype))) <= 5e-4


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
