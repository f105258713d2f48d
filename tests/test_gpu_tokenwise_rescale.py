"""Token-wise forward where a prototype's maximum logit keeps rising along a user's
tokens: by steps below and above the slack after which the running sums are rescaled
(2^8 in weight), within a range and across ranges, with ragged and whole last tiles.

Bound: the token-wise tests' normwise 2e-2 and 1e-3 on lse_m, relative to its size here
(logits up to a few hundred in fp32: 2^-23 |s| each).
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [0.02, 0.5, 6.0, 40.0])
@pytest.mark.parametrize("lengths,M,d", [([32, 64, 1], 128, 64), ([33, 95, 7], 256, 128), ([700, 0, 2100], 128, 128)])
def test_rising_maximum(lengths, M, d, step):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_08443_amd import sa_sketch as sa
    g = torch.Generator(device="cuda").manual_seed(M + d)
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    T = off[-1]
    K = torch.randn(T, 1, d, generator=g, device="cuda")
    P = torch.randn(1, M, d, generator=g, device="cuda") * d ** -0.5
    P[:, :, 0] = P[:, :, 0].abs() + 0.5
    for b, n in enumerate(lengths):   # feature 0 lifts every logit by up to `step` a tile
        ramp = torch.arange(n, device="cuda") // 32
        K[off[b]:off[b + 1], 0, 0] = (ramp % 40) * step * d ** 0.5
    K, P = K.to(torch.bfloat16), P.to(torch.bfloat16)
    V = torch.randn(T, 1, d, generator=g, device="cuda").to(torch.bfloat16)
    sk, lse = sa.sketch_fwd_tokenwise(K, V, P, torch.tensor(off, device="cuda"))
    for b, n in enumerate(lengths):
        if n == 0:
            assert not sk[b].any() and bool(torch.isneginf(lse[b]).all())
            continue
        s = P[0].double() @ K[off[b]:off[b + 1], 0].double().t() * d ** -0.5
        ref = torch.softmax(s, 1) @ V[off[b]:off[b + 1], 0].double()
        rl = torch.logsumexp(s, 1)
        assert float((sk[b, 0].double() - ref).abs().max()) <= 2e-2 * float(ref.abs().max())
        assert float((lse[b, 0].double() - rl).abs().max()) <= 1e-3 * max(1.0, float(rl.abs().max()) / 100)
