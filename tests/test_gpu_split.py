"""Two-pass forward of bf16 inputs (shapes without a one-pass instance) against the
fp64 oracle: the weights keep fp32 precision, so the bounds are those of
single-precision sums.

A weight's relative error is that of its logit (an fp32 sum of d exact products,
about sqrt(d) 2^-24 |s| for unit logits, 7e-7 at d = 128) plus a few roundings of
2^-24; the errors of different tokens are independent, so the sketch's 2-norm
error stays near that of one weight: 2e-6 is three times it, and half of what
dropping the lowest of the three bf16 parts of a weight would add (2^-18).
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


# prototype counts around a wave's 32, a workgroup's 64 / 128 / 256 and an LDS tile's
# 64; users of one token, of a tile, empty, and split over ranges at both ends
CASES = [
    ([33, 0, 1, 64], 2, 1, 64), ([40, 7], 1, 3, 128), ([95, 32], 2, 33, 64), ([31, 0, 65], 2, 64, 128),
    ([70], 3, 65, 64), ([129, 2], 1, 127, 128), ([64, 64], 2, 129, 64), ([50, 300], 1, 200, 128),
    ([90], 2, 257, 64), ([45, 0, 77], 1, 385, 128), ([5000, 12, 7000, 0, 2500], 2, 640, 128),
    ([300, 1, 4001], 1, 1152, 64), ([2100, 33], 1, 2048, 128), ([100], 1, 4096, 64),
    # 256-, 128- and 64-token workgroups of the log-sum-exp (by their number)
    ([20000, 3, 13000], 2, 200, 64), ([20000, 0, 129], 2, 65, 128),
]


@pytest.mark.parametrize("lengths,H,M,d", CASES)
@pytest.mark.parametrize("want_lse", [True, False])
def test_split_fwd_single_precision(sa, lengths, H, M, d, want_lse):
    w = wl.custom(lengths, H, M, d, "bf16", seed=sum(lengths) + M + d)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, "bf16")
    print(f"case {w.name} lse={want_lse}", flush=True)
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], w.scale, want_lse=want_lse)
    ref, rlse = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], w.scale)
    g = sk.cpu().numpy().astype(np.float64)
    for b, n in enumerate(lengths):
        if n == 0:
            assert np.all(g[b] == 0)
            continue
        assert np.linalg.norm(g[b] - ref[b]) <= 2e-6 * np.linalg.norm(ref[b]), b
    if want_lse:
        assert np.abs(lse.cpu().numpy() - rlse).max() <= 2e-6 * max(1.0, np.abs(rlse).max())


def test_split_fwd_infinite_values(sa):
    """An infinite V reaches exactly its own column, as in a plain sum of products."""
    w = wl.custom([40, 300, 33], 1, 200, 64, "bf16", seed=3)
    host = wl.host_tensors(w)
    host["V"][17, 0, 5] = np.inf
    host["V"][40 + 299, 0, 63] = -np.inf
    host["V"][340 + 2, 0, 0] = np.nan
    dev = wl.to_device(host, "bf16")
    bits = dev["V"].view(torch.int16)
    bits[340 + 2, 0, 0] = 0x7FC0
    g = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], w.scale)[0].cpu().numpy()
    assert np.all(g[0, 0, :, 5] == np.inf) and np.all(g[1, 0, :, 63] == -np.inf) and np.all(np.isnan(g[2, 0, :, 0]))
    for b, (t, j) in enumerate(((17, 5), (339, 63), (342, 0))):
        host["V"][t, 0, j] = 0.0
    ref = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], w.scale)[0]
    for b, j in enumerate((5, 63, 0)):
        keep = [c for c in range(64) if c != j]
        assert np.linalg.norm(g[b, 0][:, keep] - ref[b, 0][:, keep]) <= 2e-6 * np.linalg.norm(ref[b, 0][:, keep])


# A prototype tile with few valid rows (none in some lane) and scales that take a masked
# row's value to -inf, on batches that reach one, two and four waves a token set (by the
# number of 256-token workgroups a head: 256 CUs, 128 and fewer).  The logits are fp32
# sums of size `scale`: sqrt(d) 2^-24 scale = 5e-7 scale each, three times that beside
# the bound of unit scale.
@pytest.mark.parametrize("lengths,H", [([40, 0, 31], 1), ([9000, 0, 24500], 1), ([9000, 33, 24500], 2)])
@pytest.mark.parametrize("M", [1, 3, 4, 33, 36, 68, 100])
@pytest.mark.parametrize("scale", [0.7, 1.0, 4.0])
def test_split_fwd_few_valid_rows_large_scale(sa, lengths, H, M, scale):
    w = wl.custom(lengths, H, M, 64, "bf16", seed=M)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, "bf16")
    print(f"case {w.name} scale={scale}", flush=True)
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], scale)
    ref, rlse = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], scale)
    bound = 2e-6 + 1.5e-6 * scale
    assert np.linalg.norm(sk.cpu().numpy() - ref) <= bound * np.linalg.norm(ref)
    assert np.abs(lse.cpu().numpy() - rlse).max() <= bound * max(1.0, np.abs(rlse).max())


@pytest.mark.parametrize("lengths,M,d", [([70, 33], 200, 64), ([33000], 100, 64), ([70, 33], 640, 128),
                                         ([70, 33], 512, 128)])
@pytest.mark.parametrize("scale", [0.125, 4.0])
def test_split_fwd_prototypes_out_of_use(sa, lengths, M, d, scale):
    """Logits of -inf (prototypes switched off) have weight 0, also where a wave has no other."""
    w = wl.custom(lengths, 1, M, d, "bf16", seed=M)
    host = wl.host_tensors(w)
    host["K"][:, :, 0] = np.abs(host["K"][:, :, 0]) + 1.0
    host["P"][:, 32:64, 0] = -np.inf
    host["K"] = torch.from_numpy(host["K"]).bfloat16().float().numpy()
    dev = wl.to_device(host, "bf16")
    print(f"case {w.name} scale={scale}", flush=True)
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], scale)
    ref, rlse = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], scale)
    assert np.all(np.isfinite(ref)) and not sk[:, :, 32:64].any()
    bound = 2e-2 if (M, d) == (512, 128) else 2e-6 + 1.5e-6 * scale * (d / 64) ** 0.5
    assert np.linalg.norm(sk.cpu().numpy() - ref) <= bound * np.linalg.norm(ref)
    assert np.abs(lse.cpu().numpy() - rlse).max() <= (2e-6 + 3e-6 * scale) * max(1.0, np.abs(rlse).max())


def test_split_fwd_segment_beyond_4_gib(sa):
    """A segment's last tokens lie more than 4 GiB behind its first one (16 ranges of M = 4096
    prototypes hold whole users); float64 torch on the last head."""
    H, M, d, T = 64, 4096, 128, 264_000
    assert sa.fwd_chunk_tokens(1, T, H, M, d, sa.SA_BF16) >= T and T * H * d * 2 > 1 << 32
    g = torch.Generator(device="cuda").manual_seed(4)
    X = torch.empty((T, H, d), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    P = (torch.randn(H, M, d, generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    sk, lse = sa.sketch_fwd(X, X, P, torch.tensor([0, T], device="cuda"))
    x, p = X[:, -1].double(), P[-1].double()
    ref, rl = torch.zeros(M, d, dtype=torch.float64, device="cuda"), []
    for part in x.split(16384):
        s = part @ p.t() * d ** -0.5
        rl.append(torch.logsumexp(s, 1))
        ref += torch.exp(s - rl[-1][:, None]).t() @ part
    assert float((sk[0, -1].double() - ref).norm() / ref.norm()) <= 2e-6
    assert float((lse[:, -1].double() - torch.cat(rl)).abs().max()) <= 2e-6 * float(lse.max())


@pytest.mark.parametrize("M,dtype", [(128, "bf16"), (200, "bf16"), (128, "fp32")])
def test_users_without_tokens_cost_their_zeros(sa, M, dtype):
    """4,000 users without tokens between others (and, in two heads, at each head's end): their zero
    sketches are 0.13 GB a head and right, and the call stays within ten times that of the users with
    tokens alone (a walk over them one at a time took 1.1 ms, 18 times as long)."""
    few = [2000, 300, 1500, 2500, 700, 90, 1800, 1110]

    def timed(lengths):
        w = wl.custom(lengths, 2, M, 64, dtype, seed=1)
        dev = wl.device_tensors(w)
        args = dev["K"], dev["V"], dev["P"], dev["offsets"]
        sk, lse = sa.sketch_fwd(*args)
        ws = torch.empty(sa.fwd_workspace_size(len(lengths), sum(lengths), 2, M, 64, sa._dtype_code(dev["K"])), dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                sa.sketch_fwd(*args, sketch=sk, lse=lse, workspace=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return sk, best

    sk0, t0 = timed(few)
    lengths = few[:4] + [0] * 4000 + few[4:]
    sk1, t1 = timed(lengths)
    assert not sk1[4:4004].any()
    assert float((sk1[:4] - sk0[:4]).norm()) <= 1e-5 * float(sk0[:4].norm())   # (partials added in other groups)
    assert t1 <= 10 * t0, (t0, t1)


# more (pair, column group)s than workgroups of the merge: each takes several column groups
@pytest.mark.parametrize("M,d,dtype", [(1024, 64, "bf16"), (640, 128, "bf16"), (512, 64, "fp32")])
def test_merge_of_many_pairs(sa, M, d, dtype):
    lengths = [5] * 700 + [300, 0, 2500] + [3] * 300
    w = wl.custom(lengths, 1, M, d, dtype, seed=M)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, dtype)
    args = dev["K"], dev["V"], dev["P"], dev["offsets"]
    ref = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], w.scale)[0]
    sk = sa.sketch_fwd(*args, w.scale)[0].cpu().numpy()
    # 2-norm per user: single-precision sums, or weights rounded to bf16 (2^-9 each)
    err = np.linalg.norm((sk - ref).reshape(len(lengths), -1), axis=1)
    assert np.all(err <= (4e-3 if M == 1024 else 2e-6) * np.linalg.norm(ref.reshape(len(lengths), -1), axis=1))


def test_merge_of_unsplit_pairs_is_short(sa):
    """2,048 users none of whom is split: finding that out takes a small part of the aggregation's time
    (a fifth; two thirds with a workgroup for every 1,024 columns)."""
    dev = wl.device_tensors(wl.custom([16] * 2048, 1, 512, 64, "bf16", seed=1))
    ratio = 1e9
    for _ in range(10):
        sa.profile_enable(True)
        sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"])
        torch.cuda.synchronize()
        t = sa.kernel_times()
        sa.profile_enable(False)
        ratio = min(ratio, t["splitL_merge"][1] / t["split_agg"][1])
    assert ratio <= 0.4, ratio


@pytest.mark.parametrize("M", [200, 256])
@pytest.mark.parametrize("scale", [0.0, 1e-39, 1e-38, 1e-30])
def test_split_fwd_vanishing_scale(sa, M, scale):
    """Logits of nothing: every weight 1 / M, also where 1 / scale has no fp32 value.  Bounds as at
    unit scale (bf16 weights of 1 / 200 and 1 / 256: 2^-9)."""
    w = wl.custom([70, 0, 33], 1, M, 64, "bf16", seed=M)
    host = wl.host_tensors(w)
    dev = wl.to_device(host, "bf16")
    sk, lse = sa.sketch_fwd(dev["K"], dev["V"], dev["P"], dev["offsets"], scale)
    ref, rlse = oracle.fwd(host["K"], host["V"], host["P"], host["offsets"], scale)
    assert np.linalg.norm(sk.cpu().numpy() - ref) <= (2e-6 if M == 200 else 2e-3) * np.linalg.norm(ref)
    assert np.abs(lse.cpu().numpy() - rlse).max() <= 2e-6 * np.abs(rlse).max()
