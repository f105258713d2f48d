"""sa_sketch_fwd_noalloc on every route of the forward: bit-identical to sa_sketch_fwd, with and
without lse (whose scratch the two-pass routes then hold)."""
import pytest

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


@pytest.mark.parametrize("lengths,H,M,d,dtype,scope", [
    ([9000, 1, 0, 33, 8001], 8, 256, 64, "bf16", "fused_fwd"), ([9000, 1, 0, 33, 8001], 8, 512, 128, "bf16", "fused_fwd"),
    ([300, 0, 70], 2, 512, 128, "bf16", "split_agg"), ([300, 0, 70], 2, 200, 64, "bf16", "split_agg"),
    ([300, 0, 70], 2, 64, 128, "fp32", "plain_fwd"), ([300, 0, 70], 2, 300, 64, "fp32", "plain_agg"),
    ([34] * 330, 1, 128, 64, "bf16", "split_agg")])
def test_noalloc_routes(sa, lengths, H, M, d, dtype, scope):
    w = wl.custom(lengths, H, M, d, dtype, seed=M + d)
    dev = wl.device_tensors(w)
    args = dev["K"], dev["V"], dev["P"], dev["offsets"], w.scale
    print(f"users={len(lengths)} H={H} M={M} d={d} {dtype}", flush=True)
    sa.profile_enable(True)
    sk, lse = sa.sketch_fwd(*args)
    torch.cuda.synchronize()
    times = sa.kernel_times()
    sa.profile_enable(False)
    assert scope in times
    for want in (True, False):
        got, gl = sa.sketch_fwd_noalloc(*args, want_lse=want)
        assert torch.equal(got, sk) and (torch.equal(gl, lse) if want else gl is None)
        assert torch.equal(sa.sketch_fwd(*args, want_lse=want)[0], sk)
