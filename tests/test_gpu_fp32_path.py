"""Single-precision path (fp32 matrix cores) against the fp64 oracle: forward and
backward of fp32 inputs, and the backward of bf16 inputs without a fused instance.

Bounds (2-norm per output): every product and sum is fp32.  A weight's relative error is
that of its logit, an fp32 sum of d products: sqrt(d) 2^-24 |s|, 7e-7 at d = 128 and unit
logits; gradients chain two such sums.  The bounds are three times that, 2e-6 and 4e-6;
one operand rounded to bf16 would give 1e-3.
"""
import numpy as np
import pytest

import oracle
from paper_2609_08443_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sa():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_08443_amd import sa_sketch
    sa_sketch.lib()
    return sa_sketch


def rel(g, r):
    return np.linalg.norm(g.cpu().numpy().astype(np.float64) - r) / max(np.linalg.norm(r), 1e-30)


# prototype counts around a wave's 32 and the workgroups' 64 / 128 / 256 (one part: no
# log-sum-exp pass); users of one token, of whole tiles, empty, and split over ranges
@pytest.mark.parametrize("lengths,H,M,d,dtype,R", [
    ([33, 0, 1, 64], 2, 1, 64, "fp32", 1), ([40, 7], 1, 33, 128, "fp32", 2), ([31, 0, 65], 2, 64, 128, "fp32", 1),
    ([70], 3, 65, 64, "fp32", 1), ([129, 2], 1, 127, 128, "fp32", 3), ([64, 64, 0], 2, 129, 64, "fp32", 1),
    ([50, 300], 1, 255, 64, "fp32", 2), ([90, 33], 2, 257, 128, "fp32", 1), ([45, 0, 77], 1, 385, 64, "fp32", 1),
    ([3000, 12, 4100, 0, 900], 2, 96, 64, "fp32", 2), ([2000, 5, 700], 1, 520, 64, "fp32", 1),
    ([33, 0, 1, 64], 2, 33, 64, "bf16", 2), ([300, 7, 2000], 1, 200, 128, "bf16", 1), ([70, 41], 2, 300, 64, "bf16", 3)])
@pytest.mark.parametrize("want_lse", [True, False])
def test_forward_and_backward(sa, lengths, H, M, d, dtype, R, want_lse):
    w = wl.custom(lengths, H, M, d, dtype, seed=sum(lengths) + M + d, R=R, bwd=True)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, dtype)
    print(f"case {w.name} R={R} lse={want_lse}", flush=True)
    args = dev["K"], dev["V"], dev["P"], dev["offsets"]
    sk, lse = sa.sketch_fwd(*args, w.scale, want_lse=want_lse)
    rs, rl = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], w.scale)
    assert rel(sk, rs) <= 2e-6
    if not want_lse:
        return
    assert rel(lse, rl) <= 2e-7 * max(1.0, d ** 0.5 / 8) + 2e-7
    got = sa.sketch_bwd(*args, dev["dsketch"], lse, w.scale)
    ref = oracle.bwd(host["K"], host["V"], host["P"], host["offsets"], host["dsketch"], w.scale)
    for name, g, r in zip(("dK", "dV", "dP"), got, ref):
        # (M = 1: the weight is 1 whatever the logit; dK and dP are zero)
        if M == 1 and name != "dV":
            assert float(g.abs().max()) <= 1e-4 * float(got[1].abs().max())
        else:
            assert rel(g, r) <= 4e-6, name


# one pass (M <= 256: per-wave maxima combined through LDS) and two (a lane's running maximum)
@pytest.mark.parametrize("M,d", [(64, 64), (129, 64), (256, 128), (300, 64), (640, 64)])
@pytest.mark.parametrize("scale", [0.125, 4.0])
def test_prototypes_out_of_use(sa, M, d, scale):
    """Logits of -inf (prototypes switched off) have weight 0, also where a wave has no
    other.  The bound of unit logits plus that of logits of size scale: sqrt(d) 2^-24 scale
    is 7e-7 scale at d = 128, three times that."""
    w = wl.custom([70, 0, 33], 2, M, d, "fp32", seed=M)
    host = wl.host_tensors(w)
    host["K"][:, :, 0] = np.abs(host["K"][:, :, 0]) + 1.0
    host["P"][:, :32, 0] = -np.inf
    dev = wl.to_device(host, "fp32")
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], scale)
    rs, rl = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], scale)
    assert np.all(np.isfinite(rs)) and not sk[:, :, :32].any()
    assert rel(sk, rs) <= 2e-6 + 2e-6 * scale
    assert rel(lse, rl) <= 2e-6 + 2e-6 * scale


@pytest.mark.parametrize("dtype,H,M,d", [("fp32", 2, 128, 64), ("fp32", 3, 33, 128), ("bf16", 2, 200, 64)])
def test_backward_without_users(sa, dtype, H, M, d):
    """B = 0 with tokens: zero gradients, and nothing written past the workspace (heads begin
    inside a range, so each head's slot is used)."""
    T, code = 1000, sa.SA_FP32 if dtype == "fp32" else sa.SA_BF16
    dt = dict(dtype=torch.float32 if dtype == "fp32" else torch.bfloat16, device="cuda")
    K, V, P = torch.randn(T, H, d, **dt), torch.randn(T, H, d, **dt), torch.randn(H, M, d, **dt)
    n = sa.bwd_workspace_size(0, T, H, M, d, code, 1)
    ws = torch.full((n + 4 * M * d * H,), 77, dtype=torch.uint8, device="cuda")
    out = sa.sketch_bwd(K, V, P, torch.zeros(1, dtype=torch.int64, device="cuda"),
                        torch.empty((0, 1, H, M, d), device="cuda"), torch.zeros(T, H, device="cuda"),
                        None, *(torch.full_like(x, 5.0, dtype=torch.float32) for x in (K, V, P)), workspace=ws)
    for name, g in zip(("dK", "dV", "dP"), out):
        assert not g.any(), name
    assert bool((ws[n:] == 77).all())


# log-sum-exp workgroups of 128 tokens (enough of them for every CU), and of 32 tokens shared by
# four waves, which take tiles of 32 prototypes in turn: some or all idle in the last round
@pytest.mark.parametrize("lengths,H,M,d", [([20000, 3, 0, 13000], 1, 300, 64), ([9000, 7500], 2, 264, 128),
                                           ([70, 0, 33], 2, 288, 64), ([1], 1, 416, 128), ([31, 65], 1, 449, 64)])
def test_log_sum_exp_waves(sa, lengths, H, M, d):
    w = wl.custom(lengths, H, M, d, "fp32", seed=M)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, "fp32")
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], w.scale)
    rs, rl = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], w.scale)
    assert rel(sk, rs) <= 2e-6 and rel(lse, rl) <= 4.9e-7


def test_few_tokens_against_many_prototypes(sa):
    """The log-sum-exp of 64 tokens against 4,096 prototypes is shared by the waves of a workgroup: five
    times as long as the aggregation (15 times with a wave for 32 tokens)."""
    dev = wl.device_tensors(wl.custom([64], 1, 4096, 64, "fp32", seed=1))
    ratio = 1e9
    for _ in range(10):
        sa.profile_enable(True)
        sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"])
        torch.cuda.synchronize()
        t = sa.kernel_times()
        sa.profile_enable(False)
        ratio = min(ratio, t["plain_lse"][1] / t["plain_agg"][1])
    assert ratio <= 7.0, ratio
