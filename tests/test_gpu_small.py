"""Dense steps of few rows: sizes at the edges of the tiles (32 rows by 32 columns or units), of the groups of terms and of
the dispatch, against float64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2501_15348_amd import reinc

    c = reinc.Context(64, 1, (16, 16), "gru", 16, "sum", True, arena_bytes=1 << 20)
    yield c
    c.close()


def _bound(a, w, extra=0):
    """Element-wise: at most K rounded fp32 additions and products of the terms, and a few more (scale, bias, parts)."""
    return (2 * a.shape[1] + 8 + extra) * 2.0**-24 * (a.abs() @ w.abs())


# 1024 tiles are the last of the rule (2048 of deep products): 32768 rows by 32 columns are inside, one row more is not
@pytest.mark.parametrize("n,k,m", [(1, 1, 1), (31, 2, 33), (32, 7, 32), (33, 33, 31), (500, 64, 64), (65, 96, 65), (257, 160, 70),
                                   (40, 1433, 16), (97, 513, 129), (3, 1056, 300), (32768, 64, 32), (32769, 64, 32), (65536, 520, 5)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shift", [0, 1])
def test_product_of_few_rows(ctx, n, k, m, bf16, shift):
    import torch

    g = torch.Generator(device="cuda").manual_seed(n * 1009 + k * 31 + m)
    a = torch.randn(n * k + shift, generator=g, device="cuda")
    a = (a.bfloat16() if bf16 else a)[shift:].reshape(n, k)  # (shift 1: rows that are not aligned)
    w = torch.randn(k, m, generator=g, device="cuda")
    rs = torch.rand(n, generator=g, device="cuda") + 0.01
    b = torch.randn(m, generator=g, device="cuda")
    scaled = a.float() * rs[:, None]
    ref = scaled.double() @ w.double() + b.double()
    bound = _bound(scaled.double(), w.double()) + 2.0**-22 * (ref.abs() + b.double().abs())
    out = ctx.gcn_transform(a, w, b, rs, relu=False).double()
    assert bool(((out - ref).abs() <= bound).all())
    out = ctx.gcn_transform(a, w, None, None, relu=True).double()
    ref = (a.double() @ w.double()).clamp(min=0)
    assert bool(((out - ref).abs() <= _bound(a.double(), w.double())).all())


def test_product_of_few_rows_that_are_not_finite(ctx):
    import torch

    a = torch.ones(40, 33, device="cuda")
    rs = torch.ones(40, device="cuda")
    rs[3], a[5, 2], a[39, 32] = float("inf"), float("nan"), float("-inf")
    w = torch.ones(33, 35, device="cuda")
    out = ctx.gcn_transform(a, w, None, rs, relu=False)
    want = torch.full((40, 35), 33.0, device="cuda")
    want[3], want[5], want[39] = float("inf"), float("nan"), float("-inf")
    assert torch.equal(out.nan_to_num(nan=-1.0), want.nan_to_num(nan=-1.0))


# 256 tiles are the last of the rule (all of steps deeper than 512)
@pytest.mark.parametrize("kind", ["gru", "lstm"])
@pytest.mark.parametrize("n,d,h", [(1, 32, 32), (31, 64, 64), (33, 32, 96), (500, 64, 32), (8192, 32, 32), (8193, 32, 32),
                                   (65, 500, 33), (9000, 481, 32), (5, 1030, 1)])
@pytest.mark.parametrize("zero", [False, True])
def test_step_of_few_rows(ctx, kind, n, d, h, zero):
    import torch

    from paper_2501_15348_amd import reinc

    if reinc._rnn_work_bytes(reinc.RNN[kind], n, d, h):
        pytest.skip("a shape of the plane kernels")
    g = torch.Generator(device="cuda").manual_seed(n * 1009 + d * 31 + h)
    gates = 3 if kind == "gru" else 4
    x = torch.randn(n, d, generator=g, device="cuda")
    hp = None if zero else torch.rand(n, h, generator=g, device="cuda") * 2 - 1
    cp = None if zero or kind == "gru" else torch.randn(n, h, generator=g, device="cuda")
    w_i = torch.randn(d, gates * h, generator=g, device="cuda") / d**0.5
    w_h = torch.randn(h, gates * h, generator=g, device="cuda") / h**0.5
    b_i = torch.randn(gates * h, generator=g, device="cuda") * 0.1
    b_h = torch.randn(gates * h, generator=g, device="cuda") * 0.1
    saved = torch.empty(n, 4 * h, device="cuda")
    out, c_out = ctx.rnn_step(kind, x, hp, cp, w_i, w_h, b_i, b_h, saved)
    hd = torch.zeros(n, h, dtype=torch.float64, device="cuda") if zero else hp.double()
    gi, gh = x.double() @ w_i.double() + b_i.double(), hd @ w_h.double() + b_h.double()
    # of a sum; sigmoid has slope 1/4 and tanh 1, and their fast forms are good to 2^-21
    eps = float((_bound(x.double(), w_i.double(), 8) + _bound(hd, w_h.double(), 8)).max()) + 2.0**-20
    u = lambda s, t: s[:, t * h:(t + 1) * h]
    if kind == "gru":
        r, z = torch.sigmoid(u(gi, 0) + u(gh, 0)), torch.sigmoid(u(gi, 1) + u(gh, 1))
        nn = torch.tanh(u(gi, 2) + r * u(gh, 2))
        want, keep = nn + z * (hd - nn), torch.cat([r, z, nn, u(gh, 2)], 1)
        scale = 2 + float(u(gh, 2).abs().max())
    else:
        s = gi + gh
        i, f, c, o = torch.sigmoid(u(s, 0)), torch.sigmoid(u(s, 1)), torch.tanh(u(s, 2)), torch.sigmoid(u(s, 3))
        prev = torch.zeros_like(hd) if zero else cp.double()
        cn = f * prev + i * c
        want, keep = o * torch.tanh(cn), torch.cat([i, f, c, o], 1)
        scale = 2 + float(prev.abs().max())
        assert float((c_out.double() - cn).abs().max()) <= scale * eps
    assert float((saved.double() - keep).abs().max()) <= scale * eps
    assert float((out.double() - want).abs().max()) <= scale * eps
