"""Fused backward over short token ranges, whose workgroups share the segments by their
number: against the fp64 oracle with fewer and more segments than workgroups, users at and
between range boundaries and without tokens; and its time where every user ends at one.

Bounds as in the other parity tests of the bf16 backward: 2e-2 of each output's largest value.
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


@pytest.mark.parametrize("lengths,H,M,d", [
    ([128] * 9, 1, 128, 64), ([128], 1, 640, 64), ([1], 1, 512, 128), ([300, 0, 84], 3, 256, 64),
    ([128] * 4 + [0] * 40 + [128] * 4, 2, 512, 64), ([5, 0, 130] * 60, 2, 128, 128), ([7] * 700, 1, 128, 64),
    ([33, 1, 64] * 90, 2, 1024, 64), ([128] * 260, 1, 128, 128)])
def test_backward_over_segments(sa, lengths, H, M, d):
    w = wl.custom(lengths, H, M, d, "bf16", seed=sum(lengths) + M + d, R=1, bwd=True)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, "bf16")
    print(f"users={len(lengths)} T={w.T} H={H} M={M} d={d}", flush=True)
    args = dev["K"], dev["V"], dev["P"], dev["offsets"]
    lse = sa.sketch_fwd(*args, w.scale)[1]
    got = sa.sketch_bwd(*args, dev["dsketch"], lse, w.scale)
    ref = oracle.bwd(host["K"], host["V"], host["P"], host["offsets"], host["dsketch"], w.scale)
    for name, g, r in zip(("dK", "dV", "dP"), got, ref):
        assert np.abs(g.cpu().numpy() - r).max() <= 2e-2 * np.abs(r).max(), name


def test_every_xcd_gets_its_share(sa):
    """32 users of 128 tokens in 8 heads are 256 segments, one user's 4,096 in four heads 128: the
    token side takes one round of workgroups for both (two for the first when the grid was dealt
    out by the most segments there can be, and four XCDs got none)."""
    def token_side(lengths, H):
        w = wl.custom(lengths, H, 1024, 64, "bf16", seed=5, R=1, bwd=True)
        dev = wl.device_tensors(w)
        args = dev["K"], dev["V"], dev["P"], dev["offsets"]
        lse = sa.sketch_fwd(*args)[1]
        best = 1e9
        for _ in range(10):
            sa.profile_enable(True)
            sa.sketch_bwd(*args, dev["dsketch"], lse)
            torch.cuda.synchronize()
            times = sa.kernel_times()
            sa.profile_enable(False)
            best = min(best, times["bwd_token"][1])
        return best

    half, full = token_side([4096], 4), token_side([128] * 32, 8)
    print(f"token side {half * 1e3:.1f} and {full * 1e3:.1f} us")
    assert full <= 1.4 * half, (half, full)
