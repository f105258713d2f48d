"""One-pass fused forward at every instance, on batches long enough to reach it (short
ones run in two passes), against float64 torch on the same device.

The bounds are those of the other forward tests: normwise 2e-2 per (user, head) for bf16
weights, lse 1e-3 absolute.  Two-pass runs of the same shapes are compared with the same
reference, so that the line between the two paths is covered on both sides.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

INSTANCES = [(m, 64) for m in range(128, 1025, 128)] + [(m, 128) for m in range(128, 513, 128)]


@pytest.fixture(scope="module")
def sa():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_08443_amd import sa_sketch
    sa_sketch.lib()
    return sa_sketch


def reference(K, V, P, off, scale):
    B, (H, M, d) = len(off) - 1, P.shape
    sk = torch.zeros(B, H, M, d, dtype=torch.float64, device=K.device)
    lse = torch.empty(K.shape[0], H, dtype=torch.float64, device=K.device)
    for h in range(H):
        p = P[h].double()
        for b in range(B):
            s = K[off[b]:off[b + 1], h].double() @ p.t() * scale
            lse[off[b]:off[b + 1], h] = torch.logsumexp(s, 1)
            sk[b, h] = torch.softmax(s, 1).t() @ V[off[b]:off[b + 1], h].double()
    return sk, lse


def check(sa, lengths, H, M, d, gain=1.0):
    g = torch.Generator(device="cuda").manual_seed(sum(lengths) + M + d)
    T = sum(lengths)
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    K, V = (torch.randn(T, H, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    P = (torch.randn(H, M, d, generator=g, device="cuda") * d ** -0.5 * gain).to(torch.bfloat16)
    print(f"M={M} d={d} T={T} H={H}", flush=True)
    sk, lse = sa.sketch_fwd(K, V, P, torch.tensor(off, device="cuda"))
    rs, rl = reference(K, V, P, off, d ** -0.5)
    err = (sk.double() - rs).abs().amax(dim=(2, 3)) / rs.abs().amax(dim=(2, 3)).clamp_min(1e-30)
    assert float(err.max()) <= 2e-2
    assert float((lse.double() - rl).abs().max()) <= 1e-3 * max(1.0, float(rl.abs().max()) / 10)
    for b, n in enumerate(lengths):
        if n == 0:
            assert not sk[b].any()


@pytest.mark.parametrize("M,d", INSTANCES)
def test_one_pass_instances(sa, M, d):
    check(sa, [9000, 1, 0, 33, 8001, 64, 127, 3000], 8, M, d)   # 161,808 (head, token) pairs


@pytest.mark.parametrize("M,d", [(128, 64), (1024, 64), (512, 128)])
def test_both_sides_of_the_line(sa, M, d):
    line = 131072 if d == 128 else 65536
    for T in (line // 8 - 1, line // 8, line // 8 + 1):
        check(sa, [T - 40, 40], 8, M, d)
    if M * d <= 8192:   # short batches of the smallest shape stay in one pass
        check(sa, [1023], 8, M, d)
        check(sa, [1024], 8, M, d)


@pytest.mark.parametrize("M,d", [(256, 64), (1024, 64), (512, 128)])
def test_one_pass_loose_bound_exact_maximum(sa, M, d):
    """Logits far below the Cauchy-Schwarz shift (z < 2^-64): the exact-maximum path."""
    H, T = 8, 20000
    g = torch.Generator(device="cuda").manual_seed(M)
    K, V = (torch.randn(T, H, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    P = (torch.randn(H, M, d, generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    # one long prototype, almost opposite to some tokens, makes their shift far too large
    P[:, 0] = (60.0 * torch.randn(H, d, generator=g, device="cuda")).to(torch.bfloat16)
    K[5::97] = -(P[None, :, 0].float() / 60.0).to(torch.bfloat16)
    off = [0, 12000, 12033, T]
    sk, lse = sa.sketch_fwd(K, V, P, torch.tensor(off, device="cuda"))
    rs, rl = reference(K, V, P, off, d ** -0.5)
    err = (sk.double() - rs).abs().amax(dim=(2, 3)) / rs.abs().amax(dim=(2, 3))
    assert float(err.max()) <= 2e-2
    assert float((lse.double() - rl).abs().max()) <= 2e-2   # logits of several hundred


@pytest.mark.parametrize("M", [128, 384])
def test_both_sides_of_the_short_line(sa, M):
    """d = 128 and M no multiple of 256: two passes up to 32,768 (head, token) pairs."""
    for T in (4095, 4096, 4097):
        check(sa, [T - 40, 40], 8, M, 128)
