"""sa_kernel_times: the timed scopes of one call do not overlap, so that they add up to no
more than the call."""
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


@pytest.mark.parametrize("dtype,M,d", [("fp32", 64, 64), ("fp32", 300, 128), ("bf16", 200, 64), ("bf16", 256, 64),
                                       ("bf16", 1024, 128)])
def test_scopes_add_up_to_the_call(sa, dtype, M, d):
    w = wl.custom([20000, 7000, 0, 13000], 1, M, d, dtype, seed=M, R=2, bwd=True)
    dev = wl.device_tensors(w)
    args = dev["K"], dev["V"], dev["P"], dev["offsets"]

    def timed(call, names):
        call()
        torch.cuda.synchronize()
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        sa.profile_enable(True)
        a.record()
        call()
        b.record()
        b.synchronize()
        t = sa.kernel_times()
        sa.profile_enable(False)
        assert names <= set(t) and all(n == 1 for n, _ in t.values()), t
        assert sum(ms for _, ms in t.values()) <= 1.01 * a.elapsed_time(b), (t, a.elapsed_time(b))

    lse = sa.sketch_fwd(*args)[1]
    timed(lambda: sa.sketch_fwd(*args), {"splitL_merge"})
    fused = dtype == "bf16" and M % 128 == 0
    timed(lambda: sa.sketch_bwd(*args, dev["dsketch"], lse),
          {"bwd_token", "bwd_proto"} if fused else {"dY_reduce", "plain_bwd_token", "plain_bwd_proto", "plain_dp_sum"})
