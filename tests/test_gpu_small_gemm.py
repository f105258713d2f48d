"""Single-precision batched product (the fallback of sa_gemm_bf16, and the products of
fp32 STCA) at the edges of its tiles, k groups and load widths, against float64.

Bound: a sum of K exact products (bf16 operands) or rounded ones (fp32) in fp32, at most
(K + 8) 2^-24 sum |a b| whatever the order.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sa():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_08443_amd import sa_sketch
    sa_sketch.lib()
    return sa_sketch


# rows and columns around 32 and 64, k around groups of 4, 8, 4 x 8 and 16 x 8 (four
# waves); the last two have enough 64 x 64 tiles to be cut that way
@pytest.mark.parametrize("M,N,K,batch", [
    (1, 1, 1, 1), (31, 33, 3, 2), (33, 31, 4, 1), (64, 65, 7, 2), (65, 64, 8, 1), (32, 96, 12, 3), (40, 33, 33, 1),
    (96, 32, 100, 1), (33, 34, 130, 2), (70, 129, 136, 1), (64, 64, 300, 1), (257, 130, 36, 60), (129, 193, 140, 45)])
@pytest.mark.parametrize("a_kc,b_kc", [(True, True), (True, False), (False, True), (False, False)])
def test_bf16_operands(sa, M, N, K, batch, a_kc, b_kc):
    g = torch.Generator(device="cuda").manual_seed(M + 7 * N + 31 * K)
    a = torch.randn(batch, M, K, generator=g, device="cuda").to(torch.bfloat16)
    b = torch.randn(batch, K, N, generator=g, device="cuda").to(torch.bfloat16)
    A = a.contiguous() if a_kc else a.transpose(1, 2).contiguous()
    Bt = b.transpose(1, 2).contiguous() if b_kc else b.contiguous()
    c0 = torch.randn(batch, M, N, generator=g, device="cuda")
    print(f"{M}x{N}x{K} batch {batch} {a_kc} {b_kc}", flush=True)
    for acc in (False, True):
        C = c0.clone()
        sa.gemm_bf16(A, (M * K, K, 1) if a_kc else (M * K, 1, M), Bt, (K * N, 1, K) if b_kc else (K * N, N, 1), C,
                     (M * N, N), M, N, K, batch, alpha=0.5, accumulate=acc)
        ref = 0.5 * torch.stack([a[z].double() @ b[z].double() for z in range(batch)]) + (c0.double() if acc else 0)
        mag = 0.5 * torch.stack([a[z].double().abs() @ b[z].double().abs() for z in range(batch)]) + c0.double().abs()
        assert bool(((C.double() - ref).abs() <= (K + 8) * 2.0 ** -24 * mag).all())


# D / h and k off every multiple of four: one value a load; and on them: vectors
@pytest.mark.parametrize("B,R,k,D,h", [(2, 3, 37, 30, 2), (1, 33, 64, 96, 3), (2, 5, 130, 64, 1), (1, 1, 1, 7, 7)])
def test_fp32_stca(sa, B, R, k, D, h):
    g = torch.Generator(device="cuda").manual_seed(D + k)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    Xs, q, dout = rnd(B, k, D), rnd(B, R, D), rnd(B, R, D)
    W = [rnd(D, D) * D ** -0.5 for _ in range(3)]
    out, _ = sa.stca_fwd(Xs, q, *W, h)
    got = sa.stca_bwd(Xs, q, *W, h, dout)
    x = [t.double().requires_grad_() for t in (Xs, q, *W)]
    dh = D // h
    o = []
    for i in range(h):
        s = slice(i * dh, (i + 1) * dh)
        Q, Kk, V = (x[1] @ x[2])[..., s], (x[0] @ x[3])[..., s], (x[0] @ x[4])[..., s]
        o.append(torch.softmax(Q @ Kk.transpose(1, 2).contiguous() * dh ** -0.5, -1) @ V)
    ref = torch.cat(o, -1)
    ref.backward(dout.double())
    names = ("dXs", "dq", "dWq", "dWk", "dWv")
    for name, u, v in [("out", out, ref.detach())] + [(n, got[n], t.grad) for n, t in zip(names, x)]:
        # (k = 1: the weight is 1 whatever the logits, their gradients are zero)
        assert float((u.double() - v).norm()) <= 1e-5 * max(float(v.norm()), float(dout.norm())), name


# the sketch gradient's two contractions in one product: one slab each, three each, a
# ragged last tile, and a contraction length (R h = 24) that takes two products.
# bf16 intermediates in a chain of products: 5.5e-3 measured, four times that allowed
@pytest.mark.parametrize("B,R,k,D,h", [(2, 8, 72, 128, 8), (3, 24, 200, 256, 8), (1, 16, 136, 192, 4), (2, 3, 64, 64, 8)])
def test_bf16_stca_sketch_gradient(sa, B, R, k, D, h):
    g = torch.Generator(device="cuda").manual_seed(D + k + R)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    Xs, q = rnd(B, k, D).to(torch.bfloat16), rnd(B, R, D).to(torch.bfloat16)
    W = [(rnd(D, D) * D ** -0.5).to(torch.bfloat16) for _ in range(3)]
    dout = rnd(B, R, D)
    got = sa.stca_bwd(Xs, q, *W, h, dout)
    x = [t.double().requires_grad_() for t in (Xs, q, *W)]
    dh = D // h
    o = []
    for i in range(h):
        s = slice(i * dh, (i + 1) * dh)
        Q, Kk, V = (x[1] @ x[2])[..., s], (x[0] @ x[3])[..., s], (x[0] @ x[4])[..., s]
        o.append(torch.softmax(Q @ Kk.transpose(1, 2).contiguous() * dh ** -0.5, -1) @ V)
    torch.cat(o, -1).backward(dout.double())
    for name, t in zip(("dXs", "dq", "dWq", "dWk", "dWv"), x):
        assert float((got[name].double() - t.grad).norm()) <= 2.2e-2 * float(t.grad.norm()), name


# enough 64 x 64 tiles for the product through LDS: k of one value, around its slabs of 32, and
# off every multiple of four; rows and columns off the tile
@pytest.mark.parametrize("M,N,K,batch", [(64, 64, 1, 520), (65, 63, 31, 260), (130, 70, 33, 90), (100, 100, 65, 130),
                                         (512, 320, 1030, 16)])
@pytest.mark.parametrize("a_kc,b_kc", [(True, True), (True, False), (False, True), (False, False)])
def test_bf16_operands_tiled(sa, M, N, K, batch, a_kc, b_kc):
    test_bf16_operands(sa, M, N, K, batch, a_kc, b_kc)


def test_layouts_of_large_products_cost_alike(sa):
    """k strided, or contiguous and no multiple of four, through LDS: within 1.6 times the other layout
    (from L2 one value at a time: 2.3 times)."""
    def time(M, N, K, batch, kc):
        A, B = (torch.randn(batch, n * K, device="cuda").to(torch.bfloat16) for n in (M, N))
        C = torch.empty(batch, M, N, device="cuda")
        best = 1e9
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                sa.gemm_bf16(A, (M * K, K, 1) if kc else (M * K, 1, M), B, (K * N, 1, K) if kc else (K * N, N, 1), C,
                             (M * N, N), M, N, K, batch)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    assert time(512, 1024, 160, 32, False) <= 1.6 * time(512, 1024, 160, 32, True)
    assert time(160, 500, 1030, 32, True) <= 1.6 * time(160, 500, 1030, 32, False)
