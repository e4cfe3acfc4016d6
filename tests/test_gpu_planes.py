"""Dense products on two fp16 planes per operand: sizes at the edges of the kernels' tiles and of their dispatch, wide
ranges of magnitudes, and non-finite rows, against float64."""
import numpy as np
import pytest

import oracle
from helpers import RTOL_FP32, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2501_15348_amd import reinc

    c = reinc.Context(64, 1, (16, 16), "gru", 16, "sum", True, arena_bytes=1 << 20)
    yield c
    c.close()


def _prepared(n, k, m):
    from paper_2501_15348_amd import reinc

    return reinc._gcn_work_bytes(n, k, m) > 0


def _bound(a, w):
    """Element-wise bound: each operand is kept to 2^-22, the product of the two remainders (2^-22) is left out, and the
    three partial products of every 16 k values are rounded fp32 additions (plus bias, scale and the exponents)."""
    k = a.shape[1]
    return (3 * 2.0**-22 + (3 * (k / 16 + 1) + 16) * 2.0**-24) * (a.abs() @ w.abs())


# K % 32 != 0: taken at any n; whole tiles and remainders of rows (64 or 32 per block), of columns (32 per tile, 1, 2, 4
# and 8 tiles per pass), of k (padded to 32; one, two and four groups of eight per lane), and the deep products
@pytest.mark.parametrize("n", [1, 31, 64, 65, 193])
@pytest.mark.parametrize("k,m", [(65, 1), (100, 33), (66, 64), (72, 65), (200, 128), (250, 129), (49, 257), (510, 40), (512, 128),
                                 (480, 300), (57, 96), (260, 32)])
@pytest.mark.parametrize("bf16", [False, True])
def test_row_product_edges(ctx, n, k, m, bf16):
    import torch

    assert _prepared(n, k, m)
    g = torch.Generator(device="cuda").manual_seed(n * 1009 + k * 31 + m)
    a = torch.randn(n, k, generator=g, device="cuda") * torch.exp2(torch.randint(-30, 30, (n, 1), generator=g, device="cuda").float())
    a = a.bfloat16() if bf16 else a
    w = torch.randn(k, m, generator=g, device="cuda") * torch.exp2(torch.randint(-20, 20, (1, m), generator=g, device="cuda").float())
    rs = torch.rand(n, generator=g, device="cuda") + 0.01
    b = torch.randn(m, generator=g, device="cuda")
    out = ctx.gcn_transform(a, w, b, rs, relu=False).double()
    scaled = (a.float() * rs[:, None]).double()  # (the scale is applied in fp32)
    ref = scaled @ w.double() + b.double()
    assert bool(((out - ref).abs() <= _bound(scaled, w.double()) + 2.0**-23 * ref.abs()).all())


@pytest.mark.parametrize("n,k,m", [(65536, 256, 256), (65601, 256, 300), (98305, 128, 256), (98304, 224, 129), (65537, 384, 200)])
def test_row_product_of_many_rows(ctx, n, k, m):
    import torch

    assert _prepared(n, k, m) and not _prepared(n // 2, k, m)
    g = torch.Generator(device="cuda").manual_seed(n + k + m)
    a = torch.randn(n, k, generator=g, device="cuda")
    w = torch.randn(k, m, generator=g, device="cuda") / k**0.5
    out = ctx.gcn_transform(a, w, None, None, relu=True).double()
    ref = torch.relu(a.double() @ w.double())
    assert bool(((out - ref).abs() <= _bound(a.double(), w.double())).all())


# from where the prepared form is taken of 65 to 127 columns and of 96 terms: first and ragged row counts, the first and the
# last of those columns, numbers of k-steps that leave the ring of four early or not
@pytest.mark.parametrize("n,k,m", [(16384, 224, 65), (16385, 256, 127), (16447, 320, 97), (16384, 384, 80), (98304, 96, 129)])
@pytest.mark.parametrize("bf16", [False, True])
def test_row_product_where_it_begins_to_pay(ctx, n, k, m, bf16):
    import torch

    first = 16384 if m < 128 else 98304
    assert _prepared(n, k, m) and not _prepared(first - 1, k, m)
    g = torch.Generator(device="cuda").manual_seed(n + k + m)
    a = torch.randn(n, k, generator=g, device="cuda")
    a = a.bfloat16() if bf16 else a
    w = torch.randn(k, m, generator=g, device="cuda") / k**0.5
    b = torch.randn(m, generator=g, device="cuda")
    out = ctx.gcn_transform(a, w, b, None, relu=False).double()
    ref = a.double() @ w.double() + b.double()
    assert bool(((out - ref).abs() <= _bound(a.double(), w.double()) + 2.0**-23 * ref.abs()).all())


# The blocks of a row product depend on its rows, terms, columns and type, its results do not: the last rows of a call of many
# rows are those of a call by themselves, bit for bit.  Both sides of each line between the kernels, least and most of 65 to 128
# columns and of more, ragged rows.
@pytest.mark.parametrize("n,k,m", [(131072, 50, 65), (131073, 50, 65), (131100, 57, 128), (131073, 63, 96), (131072, 72, 97), (131073, 72, 97),
                                   (131073, 65, 128), (131105, 95, 65), (131073, 97, 96), (16385, 193, 65), (131073, 225, 127),
                                   (140000, 200, 128), (16384, 290, 129), (16385, 290, 129), (16417, 383, 200), (16385, 385, 160)])
@pytest.mark.parametrize("bf16", [False, True])
def test_row_products_do_not_depend_on_the_block(ctx, n, k, m, bf16):
    import torch

    assert _prepared(n, k, m) and _prepared(130, k, m)
    g = torch.Generator(device="cuda").manual_seed(n + k + m)
    a = torch.randn(n, k, generator=g, device="cuda")
    a = a.bfloat16() if bf16 else a
    w = torch.randn(k, m, generator=g, device="cuda") / k**0.5
    b, rs = torch.randn(m, generator=g, device="cuda"), torch.rand(n, generator=g, device="cuda") + 0.01
    out = ctx.gcn_transform(a, w, b, rs, relu=True)
    for rows in (slice(0, 130), slice(n - 130, n)):
        part = ctx.gcn_transform(a[rows].clone(), w, b, rs[rows].clone(), relu=True)
        assert torch.equal(out[rows], part), rows
    scaled = (a.float() * rs[:, None]).double()
    ref = torch.relu(scaled @ w.double() + b.double())
    assert bool(((out.double() - ref).abs() <= _bound(scaled, w.double()) + 2.0**-23 * (ref + b.double().abs())).all())


# The kernels with resident weights keep the shapes that they are faster at: rows that are no whole groups of eight for each of
# eight threads, and 224 terms of bf16 rows, whose call has a work area all the same (the type is not known to its size).
def test_row_products_that_keep_the_resident_weights(ctx):
    import torch

    from paper_2501_15348_amd import reinc

    n, k, m = 16400, 224, 96
    assert _prepared(n, k, m) and not any(_prepared(n * i, j, m) for i in (1, 3, 20) for j in (288, 352, 416))
    g = torch.Generator(device="cuda").manual_seed(k)
    a, w = torch.randn(n, k, generator=g, device="cuda"), torch.randn(k, m, generator=g, device="cuda") / k**0.5
    for rows in (a, a.bfloat16()):
        bf16 = rows.dtype == torch.bfloat16
        resident = torch.empty(n, m, device="cuda")
        ptr = reinc._dev_ptr
        ctx._ck(ctx.lib.reinc_gcn_transform(ctx.handle, ptr(rows), int(bf16), n, k, m, None, ptr(w), None, 0, ptr(resident), reinc._stream()))
        out = ctx.gcn_transform(rows, w, None, None, relu=False)
        assert torch.equal(out, resident) == bf16
        ref = rows.double() @ w.double()
        assert bool(((out.double() - ref).abs() <= _bound(rows.double(), w.double())).all())


def _bound_wide(a, w):
    """... where a row or a column spans more than the planes hold: one fp32 chain over k."""
    return _bound(a, w) + a.shape[1] * 2.0**-24 * (a.abs() @ w.abs())


def test_outliers_and_extreme_magnitudes(ctx):
    """One huge value in a row, rows and columns at both ends of the exponent range, denormal and zero rows.  (The bound of
    an element is that of the terms it has: a huge value that meets a zero or a tiny weight leaves none.)"""
    import torch

    g = torch.Generator(device="cuda").manual_seed(3)
    n, k, m = 200, 100, 100
    a = torch.randn(n, k, generator=g, device="cuda")
    a[0, 5] = 1e30
    a[1] *= 1e37 / a[1].abs().max()
    a[2] *= 1e-37
    a[3] = 0.0
    a[4] = 1e-42
    w = torch.randn(k, m, generator=g, device="cuda")
    w[:, 0] *= 1e-30
    w[:, 1] = 0.0
    w[3, 2] = 1e-38
    w[5, 3:60] = 0.0
    w[5, 60:] *= 1e-30
    a[5, 6] = 1e34
    w[6, 4] = 1e-38
    a[:, 7] = torch.where(torch.arange(n, device="cuda") % 3 == 0, 1e-44, 0.0)
    w[7, 8] = 1e30
    out = ctx.gcn_transform(a, w, None, None, relu=False).double()
    ref = a.double() @ w.double()
    assert bool(((out - ref).abs() <= _bound_wide(a.double(), w.double()) + 1e-42).all())


# one feature of another magnitude than the rest (a raw time stamp, a byte count) over weights that make up for it, over
# zero weights (a feature that is not used), over weights that are zero for all but one column, and the mirrored case (one
# tiny row of weights under features that make up for it); whole and ragged tiles, one and several row tiles per wave
@pytest.mark.parametrize("exponent", [16, 24, 30, 40, 100])
@pytest.mark.parametrize("n,k,m,bf16", [(65, 100, 64, False), (33, 260, 40, False), (129, 72, 200, True), (40, 100, 16, False)])
def test_features_of_unequal_magnitudes(ctx, exponent, n, k, m, bf16):
    import torch

    assert _prepared(n, k, m) or m == 16
    f = 2.0**exponent
    for case in ("scaled", "zero", "one column", "tiny weight", "columns"):
        g = torch.Generator(device="cuda").manual_seed(n + exponent)
        a, w = torch.randn(n, k, generator=g, device="cuda"), torch.randn(k, m, generator=g, device="cuda")
        b = torch.randn(m, generator=g, device="cuda")
        if case == "tiny weight":
            a[:, 3] *= 2.0 ** (0.7 * exponent)
            w[3] /= f
        elif case == "columns":  # a column of weights that spans as much, and features that are zero under its large part
            w[:, 5] *= torch.exp2(-exponent * torch.rand(k, generator=g, device="cuda"))
            a[:, w[:, 5].abs() > 0.01] = 0.0
        else:
            a[::2, 3] *= f  # (every other row: the others keep their results bit for bit)
            w[3] = w[3] / f if case == "scaled" else 0.0
            if case == "one column":
                w[3, 7] = 1.0
        a = a.bfloat16() if bf16 else a
        rs = torch.rand(n, generator=g, device="cuda") + 0.01
        out = ctx.gcn_transform(a, w, b, rs, relu=False)
        scaled = (a.float() * rs[:, None]).double()
        ref = scaled @ w.double() + b.double()
        assert bool(((out.double() - ref).abs() <= _bound_wide(scaled, w.double()) + 2.0**-23 * ref.abs()).all()), case
        if case == "zero":
            a[::2] = a[1::2][:1]
            assert torch.equal(ctx.gcn_transform(a, w, b, rs, relu=False)[1::2], out[1::2])


# a few elements far below the rest of their row or column: as many as the lists take (8 and 4), one more, and elements too
# small for them; the outputs that only those elements reach have to be right too
@pytest.mark.parametrize("count", [1, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("exponent", [23, 40, 61, 90])
@pytest.mark.parametrize("n,k,m", [(70, 100, 40), (33, 260, 130), (129, 72, 300)])
def test_few_tiny_elements(ctx, count, exponent, n, k, m):
    import torch

    assert _prepared(n, k, m)
    g = torch.Generator(device="cuda").manual_seed(count + exponent)
    a, w = torch.randn(n, k, generator=g, device="cuda"), torch.randn(k, m, generator=g, device="cuda")
    f = 2.0**-exponent
    low = torch.randperm(k, generator=g, device="cuda")[:count]
    rows = torch.arange(0, n, 3, device="cuda")
    a[rows[:, None], low] *= f
    keep = torch.zeros(k, dtype=torch.bool, device="cuda")
    keep[low] = True
    w[~keep, 1::4] = 0.0  # columns that only meet the rows' tiny elements
    w[low[0], 2::4] *= f  # one tiny element in a column, `count` of them in others
    w[:, 3::4][keep] *= f
    a[1::3, ~keep] = 0.0  # rows that only meet those
    b = torch.randn(m, generator=g, device="cuda") * f
    out = ctx.gcn_transform(a, w, None, None, relu=False).double()
    ref = a.double() @ w.double()
    assert bool(((out - ref).abs() <= _bound_wide(a.double(), w.double())).all())
    out = ctx.gcn_transform(a, w, b, None, relu=True).double()
    assert bool(((out - torch.relu(ref + b.double())).abs() <= _bound_wide(a.double(), w.double()) + 2.0**-23 * b.abs()).all())


def test_non_finite_rows_stay_in_their_rows(ctx):
    import torch

    g = torch.Generator(device="cuda").manual_seed(4)
    a = torch.randn(130, 100, generator=g, device="cuda")
    w = torch.randn(100, 100, generator=g, device="cuda")
    clean = ctx.gcn_transform(a, w, None, None, relu=False)
    bad = a.clone()
    bad[7, 3], bad[70, 99], bad[129, 0] = float("inf"), float("nan"), -float("inf")
    out = ctx.gcn_transform(bad, w, None, None, relu=False)
    rows = torch.tensor([7, 70, 129], device="cuda")
    assert not bool(torch.isfinite(out[rows]).any())
    keep = torch.ones(130, dtype=torch.bool, device="cuda")
    keep[rows] = False
    assert torch.equal(out[keep], clean[keep])


@pytest.mark.parametrize("n,k,m", [(130, 100, 100), (65536, 256, 256)])
def test_infinite_operands_give_what_fp32_products_give(ctx, n, k, m):
    """An infinite row or column of weights gives infinities of the terms' signs (so that ReLU keeps an overflowed row), and
    NaN only where two of them cancel."""
    import torch

    assert _prepared(n, k, m)
    g = torch.Generator(device="cuda").manual_seed(5)
    a, w = torch.randn(n, k, generator=g, device="cuda"), torch.randn(k, m, generator=g, device="cuda")
    a[7, 3], a[70, k - 1], w[5, 9] = float("inf"), -float("inf"), -float("inf")
    ref = a.double() @ w.double()
    out = ctx.gcn_transform(a, w, None, None, relu=False)
    assert torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(out[torch.isinf(ref)].double(), ref[torch.isinf(ref)]) and int(torch.isinf(ref).sum()) > m + n - 4
    keep = ~torch.isnan(ref)
    relu = ctx.gcn_transform(a, w, None, None, relu=True)
    assert torch.equal(torch.isinf(relu[keep]), torch.isinf(torch.relu(ref)[keep])) and bool((relu[keep] >= 0).all())


def test_shapes_that_keep_the_resident_kernels():
    from paper_2501_15348_amd import reinc

    reinc.load_library()
    for n, d, h in ((32767, 128, 128), (100000, 64, 96), (100000, 64, 64), (100000, 64, 128), (100000, 128, 32), (0, 16, 16), (100, 512, 32)):
        assert reinc._rnn_work_bytes(0, n, d, h) == 0, (n, d, h)
    for n, k, m in ((100000, 32, 512), (50, 7, 96), (100000, 31, 64), (100000, 48, 512), (65535, 256, 256), (200000, 384, 128), (200000, 64, 512), (98303, 128, 256), (200000, 128, 128), (0, 100, 100), (50, 513, 64), (50, 100, (1 << 20) + 1)):
        assert reinc._gcn_work_bytes(n, k, m) == 0, (n, k, m)


def _step_errors(ctx, kind, n, d, h, state):
    """Relative errors (2-norm, against float64) of a recurrent step's outputs: its saved gates by name, c and h."""
    import torch

    g = torch.Generator(device="cuda").manual_seed(n + 7 * d + 31 * h)
    kg = 3 if kind == "gru" else 4
    x = torch.randn(n, d, generator=g, device="cuda").relu_()
    hp = torch.tanh(torch.randn(n, h, generator=g, device="cuda")) if state else None
    cp = torch.randn(n, h, generator=g, device="cuda") if state and kind == "lstm" else None
    uniform = lambda fan, *shape: (torch.rand(*shape, generator=g, device="cuda") * 2 - 1) / fan**0.5  # noqa: E731
    wi, wh, bi, bh = uniform(d, d, kg * h), uniform(h, h, kg * h), 0.1 * uniform(1, kg * h), 0.1 * uniform(1, kg * h)
    saved = torch.empty(n, 4 * h, device="cuda")
    h_out, c_out = ctx.rnn_step(kind, x, hp, cp, wi, wh, bi, bh, saved)
    xi, sh = x.double() @ wi.double() + bi.double(), bh.double().expand(n, -1)
    hd, cd = hp.double() if state else 0.0, cp.double() if cp is not None else 0.0
    if state:
        sh = sh + hd @ wh.double()
    part = lambda v, i: v[:, i * h:(i + 1) * h]  # noqa: E731
    if kind == "lstm":
        gi, gf, gg, go = (f(part(xi, i) + part(sh, i)) for i, f in enumerate((torch.sigmoid, torch.sigmoid, torch.tanh, torch.sigmoid)))
        c = gf * cd + gi * gg
        ref, names = dict(i=gi, f=gf, g=gg, o=go, c=c, h=go * torch.tanh(c)), "ifgo"
    else:
        r, z = (torch.sigmoid(part(xi, i) + part(sh, i)) for i in range(2))
        nn = torch.tanh(part(xi, 2) + r * part(sh, 2))
        ref, names = dict(r=r, z=z, n=nn, hn=part(sh, 2), h=(1 - z) * nn + z * hd), ("r", "z", "n", "hn")
    got = dict({name: part(saved, i) for i, name in enumerate(names)}, h=h_out, c=c_out)
    return {name: float((got[name].double() - v).norm() / v.norm()) for name, v in ref.items()}


# hidden units: one tile and a remainder, two tiles, more than four (a second pass), depths up to 512
@pytest.mark.parametrize("kind", ["gru", "lstm"])
@pytest.mark.parametrize("n,d,h,zero_state", [(1, 16, 16, False), (65, 33, 33, False), (129, 100, 64, True), (64, 64, 65, False),
                                              (32769, 128, 128, False), (8192, 60, 64, True), (97, 96, 250, False), (33, 256, 256, False), (70, 1, 31, False),
                                              (40, 300, 40, True)])
def test_recurrent_step_edges(ctx, kind, n, d, h, zero_state):
    import torch

    from paper_2501_15348_amd import reinc

    assert reinc._rnn_work_bytes(reinc.RNN[kind], n, d, h) > 0
    rng = np.random.default_rng(n + 7 * d + 13 * h)
    kg = 3 if kind == "gru" else 4
    x = rng.standard_normal((n, d)).astype(np.float32)
    hp = np.zeros((n, h), np.float32) if zero_state else rng.standard_normal((n, h)).astype(np.float32)
    cp = np.zeros((n, h), np.float32) if zero_state else rng.standard_normal((n, h)).astype(np.float32)
    wi = (rng.standard_normal((d, kg * h)) / np.sqrt(d)).astype(np.float32)
    wh = (rng.standard_normal((h, kg * h)) / np.sqrt(h)).astype(np.float32)
    bi, bh = (rng.standard_normal(kg * h).astype(np.float32) * 0.3 for _ in range(2))
    dev = lambda v: torch.from_numpy(v).cuda()  # noqa: E731
    saved = torch.empty((n, 4 * h), device="cuda")
    h_out, c_out = ctx.rnn_step(kind, dev(x), None if zero_state else dev(hp), None if zero_state or kind == "gru" else dev(cp),
                                dev(wi), dev(wh), dev(bi), dev(bh), saved)
    f = lambda v: v.astype(np.float64)  # noqa: E731
    if kind == "gru":
        ref_h, gates = oracle.gru_cell(f(x), f(hp), f(wi), f(wh), f(bi), f(bh))
    else:
        ref_h, ref_c, gates = oracle.lstm_cell(f(x), f(hp), f(cp), f(wi), f(wh), f(bi), f(bh))
        assert_close(c_out.cpu().numpy(), ref_c, RTOL_FP32, "c")
    assert_close(h_out.cpu().numpy(), ref_h, RTOL_FP32, "h")
    assert_close(saved.cpu().numpy(), np.concatenate(gates, axis=1), RTOL_FP32, "saved gates")


# Each sum of a recurrent step is as close to 64 bits as with the products of all gates together and their cross products first.
# The limits are the relative errors of such a kernel on these very inputs, rounded up in the fourth digit; with one chain of
# main products and the cross products added at its end the listed outputs are 0.3 to 5 % above them.  Wide cells, the least
# units and inputs of a GRU's, and shapes whose chains are too short to gain from it.
@pytest.mark.parametrize("kind,d,h,limits", [
    ("gru", 256, 256, dict(z=5.631e-8, n=1.657e-7, hn=1.170e-7, h=1.092e-7)),
    ("gru", 128, 128, dict(r=5.290e-8, z=5.251e-8, n=1.613e-7, hn=1.036e-7, h=1.052e-7)),
    ("gru", 136, 64, dict(z=4.990e-8, n=1.565e-7, hn=7.868e-8)),
    ("gru", 160, 40, dict(z=5.050e-8, n=1.625e-7, hn=8.508e-8)),
    ("gru", 16, 256, dict(n=1.445e-7, hn=1.171e-7, h=9.902e-8)),
    ("lstm", 256, 256, dict(f=5.624e-8, c=9.367e-8, h=1.506e-7)),
    ("lstm", 128, 128, dict(f=5.235e-8, c=8.601e-8, h=1.453e-7)),
])
def test_sums_of_a_recurrent_step_are_as_close_as_with_all_gates_together(ctx, kind, d, h, limits):
    from paper_2501_15348_amd import reinc

    n = 60000
    assert reinc._rnn_work_bytes(reinc.RNN[kind], n, d, h) > 0
    errors = _step_errors(ctx, kind, n, d, h, state=True)
    for name, limit in limits.items():
        assert errors[name] <= limit, (name, errors[name], limit)


# ... and without a state, where the sums are of the input's terms alone: too few of them, and enough.
@pytest.mark.parametrize("kind,n,d,h,limits", [
    ("lstm", 100000, 16, 100, dict(g=1.388e-7, c=1.483e-7, h=2.888e-7)),
    ("gru", 60000, 33, 200, dict(n=1.525e-7, h=1.598e-7)),
    ("gru", 60000, 100, 100, dict(r=4.724e-8, z=4.769e-8, n=1.591e-7, h=1.660e-7)),
    ("lstm", 60000, 100, 100, dict(i=4.760e-8, f=4.747e-8, g=1.569e-7, c=1.675e-7, h=3.106e-7)),
])
def test_sums_of_a_first_recurrent_step_are_as_close_as_with_all_gates_together(ctx, kind, n, d, h, limits):
    errors = _step_errors(ctx, kind, n, d, h, state=False)
    for name, limit in limits.items():
        assert errors[name] <= limit, (name, errors[name], limit)


# one feature of the input far above the rest over small or zero weights, an input far above the state, and a row of W_h far
# above the rest under a zero state of that unit
@pytest.mark.parametrize("kind", ["gru", "lstm"])
@pytest.mark.parametrize("n,d,h", [(65, 100, 40), (32769, 128, 128), (33, 256, 256)])
@pytest.mark.parametrize("case", ["scaled", "zero", "x over h", "W_h row", "few", "few, zero state"])
def test_recurrent_step_of_unequal_magnitudes(ctx, kind, n, d, h, case):
    import torch

    from paper_2501_15348_amd import reinc

    assert reinc._rnn_work_bytes(reinc.RNN[kind], n, d, h) > 0
    rng = np.random.default_rng(n + d)
    kg = 3 if kind == "gru" else 4
    x, hp, cp = (rng.standard_normal((n, w)).astype(np.float32) for w in (d, h, h))
    wi = (rng.standard_normal((d, kg * h)) / np.sqrt(d)).astype(np.float32)
    wh = (rng.standard_normal((h, kg * h)) / np.sqrt(h)).astype(np.float32)
    bi, bh = (rng.standard_normal(kg * h).astype(np.float32) * 0.3 for _ in range(2))
    f = np.float32(2.0**34)
    if case in ("scaled", "zero"):
        x[::3, 2] *= f
        wi[2] = wi[2] / f if case == "scaled" else 0.0
    elif case == "x over h":
        x *= f
        wi /= f
    elif case == "W_h row":
        wh[3] *= f
        hp[:, 3] = 0.0
    else:  # a few tiny elements: inputs, states, weights of either part
        x[::3, 4:6] /= f
        hp[1::3, 1] /= f
        wi[7, ::2] /= f
        wh[2:4, ::3] /= f
        wi[:, 5], x[:, 3] = 0.0, 0.0
        wi[3, 5] = 1.0  # (with the line above: a column whose input part comes from its tiny terms alone)
        if case == "few, zero state":
            hp[:], cp[:] = 0.0, 0.0
    dev = lambda v: torch.from_numpy(v).cuda()  # noqa: E731
    saved = torch.empty((n, 4 * h), device="cuda")
    state = (None, None) if case == "few, zero state" else (dev(hp), dev(cp) if kind == "lstm" else None)
    h_out, c_out = ctx.rnn_step(kind, dev(x), *state, dev(wi), dev(wh), dev(bi), dev(bh), saved)
    up = lambda v: v.astype(np.float64)  # noqa: E731
    if kind == "gru":
        ref_h, gates = oracle.gru_cell(up(x), up(hp), up(wi), up(wh), up(bi), up(bh))
    else:
        ref_h, ref_c, gates = oracle.lstm_cell(up(x), up(hp), up(cp), up(wi), up(wh), up(bi), up(bh))
        assert np.abs(c_out.cpu().numpy() - ref_c).max() < 2e-5
    # sums of at most 512 terms whose magnitudes add up to about 20: 512 * 2^-24 * 20 < 1e-3 in the worst case, a hundredth
    # of it seen; a lost state or input shows as 0.1 to 1
    assert np.abs(h_out.cpu().numpy() - ref_h).max() < 2e-5
    assert np.abs(saved.cpu().numpy() - np.concatenate(gates, axis=1)).max() < 4e-5


# a loss that is 2^36 times as large for one hidden unit, whose gates take nothing from the other units' weights: the other
# units' gradients come from elements far below the largest of their rows
@pytest.mark.parametrize("rnn", ["gru", "lstm"])
@pytest.mark.parametrize("n,hidden", [(65, 40), (70, 64), (33, 128), (40, 136)])
def test_backward_step_of_unequal_magnitudes(rnn, n, hidden):
    import torch

    from helpers import oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    length = 3
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, 48), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 26)
    ctx.load_sequence(seq)
    ctx.build_deltas(-1)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    target[:, 0] *= 2.0**36
    p = synth.split_params(wl, flat)
    kg = 3 if rnn == "gru" else 4
    mine = np.arange(kg) * hidden  # the columns of unit 0
    p["W_i"][:, mine] = 0.0
    p["W_h"][:, mine] = 0.0
    p["W_h"][0, :] = 0.0
    flat = np.concatenate([p[name].ravel() for name, _ in synth.param_shapes(wl)]).astype(np.float32)
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target).cuda()
    loss, grads = torch.zeros(1, device="cuda"), torch.empty_like(params)
    ctx.forward_window(0, length, params, tgt, loss)
    ctx.backward_window(0, length, params, tgt, grads)
    p = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle_graphs(seq), [oracle_feats(seq, t) for t in range(length)]
    _, ref_h, saved = oracle.forward_window(graphs, feats, p, 1, wl.agg, wl.self_loop, rnn, target.astype(np.float64), keep=True)
    ref = oracle.backward_window(graphs, saved, ref_h, p, 1, wl.agg, wl.self_loop, rnn, target.astype(np.float64))
    got = synth.split_params(wl, grads.cpu().numpy())
    for name in ("W_i", "W_h", "b_i", "b_h"):
        for others in (False, True):
            pick = (lambda v: np.delete(v, mine, axis=-1)) if others else (lambda v: v[..., mine])
            assert_close(pick(got[name]), pick(ref[name]), 1e-3, f"{name}, {'other units' if others else 'unit 0'}")
    ctx.close()


# one backward step per launch: hidden widths around the two block shapes (64 and 128 units), with padded k-steps (three or
# four gates of a width that is no multiple of 32), and on both sides of the widths the kernel takes
@pytest.mark.parametrize("rnn", ["gru", "lstm"])
@pytest.mark.parametrize("n,hidden", [(33, 32), (65, 40), (130, 56), (64, 64), (31, 64), (129, 72), (33, 104), (65, 128), (40, 136), (50, 44)])
def test_backward_step_edges(rnn, n, hidden):
    import torch

    from helpers import GRAD_RTOL_FP32, assert_gradients_close, oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    length = 3
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, 32), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 26)
    ctx.load_sequence(seq)
    ctx.build_deltas(-1)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target).cuda()
    loss, grads = torch.zeros(1, device="cuda"), torch.empty_like(params)
    ctx.forward_window(0, length, params, tgt, loss)
    ctx.backward_window(0, length, params, tgt, grads)
    p = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle_graphs(seq), [oracle_feats(seq, t) for t in range(length)]
    _, ref_h, saved = oracle.forward_window(graphs, feats, p, 1, wl.agg, wl.self_loop, rnn, target, keep=True)
    assert_gradients_close(synth.split_params(wl, grads.cpu().numpy()), saved,
                           lambda sv: oracle.backward_window(graphs, sv, ref_h, p, 1, wl.agg, wl.self_loop, rnn, target),
                           [name for name, _ in synth.param_shapes(wl)], GRAD_RTOL_FP32)
    ctx.close()


# shapes with the recurrent weights in matrix-core form: in the zero state before the window (many rows), in what a node
# batch's placement leaves of the states' array (covered by the batch tests), nowhere (40 rows)
@pytest.mark.parametrize("model", ["stacked", "integrated"])
@pytest.mark.parametrize("rnn,hidden,n", [("gru", 64, 3001), ("lstm", 128, 2500), ("lstm", 64, 40)])
def test_window_weights_are_out_of_the_arenas_way(model, rnn, hidden, n):
    """A forward call that waits on its own stream while the next snapshot is loaded (whose scratch memory and arrays take
    the arena up to the local cache), and a captured one that is replayed after that, give what an undisturbed call gives;
    so does a context whose arena has next to no room left."""
    import torch

    from paper_2501_15348_amd import reinc, synth

    steps = 6
    wl = synth.WORKLOADS["c2"].scaled(n, steps, dims=(64, 64), hidden=hidden, rnn=rnn)
    seq = synth.make_sequence(wl)
    params = torch.from_numpy(synth.make_params(wl, bias_scale=0.2)).cuda()
    if model == "integrated":
        params = params[-(64 + hidden + 2) * (3 if rnn == "gru" else 4) * hidden:].contiguous()
    target = torch.from_numpy(synth.make_target(wl)).cuda()
    xs = [seq.x0]
    for t in range(1, steps):
        x = xs[-1].copy()
        x[seq.feat_rows[t]] = seq.feat_vals[t]
        xs.append(x)

    def load(ctx, t):
        ctx.load_edges(t, *seq.edges[t])
        ctx.load_features_full(t, xs[t])

    def outputs():
        return torch.zeros(1, device="cuda"), torch.zeros(n, hidden, device="cuda"), torch.zeros_like(params)

    def run(ctx, loss, h, grads, backward=True):
        (ctx.forward_window if model == "stacked" else ctx.forward_window_integrated)(0, 4, params, target, loss, h)
        if backward:
            (ctx.backward_window if model == "stacked" else ctx.backward_window_integrated)(0, 4, params, target, grads)

    def context(arena):
        ctx = reinc.Context.for_workload(wl, arena_bytes=arena)
        for t in range(4):
            load(ctx, t)
        return ctx

    ctx = context(1 << 28)
    quiet = outputs()
    run(ctx, *quiet)
    used = (1 << 28) - ctx.arena_free_bytes()
    torch.cuda.synchronize()
    ctx.close()

    # the arena as small as the window calls allow, found by halving: the forward pass takes the same kernels
    low, high, tight = used // 4, 1 << 28, None
    while high - low > 4096:
        size = (low + high) // 2 // 256 * 256
        got, small = outputs(), reinc.Context.for_workload(wl, arena_bytes=size)
        try:
            for t in range(4):
                load(small, t)
            run(small, *got)
            torch.cuda.synchronize()
            high, tight = size, got
        except reinc.ReincError as e:
            assert e.code == reinc.E_NOMEM
            low = size
        finally:
            small.close()
    assert torch.equal(tight[0], quiet[0]) and torch.equal(tight[1], quiet[1])
    assert_close(tight[2].cpu().numpy(), quiet[2].cpu().numpy(), RTOL_FP32, "gradients in the smallest arena")

    ctx = context(1 << 28)
    side = torch.cuda.Stream()
    busy = outputs()
    run(ctx, *outputs(), backward=False)  # (the local cache and the layer-1 sums are made)
    torch.cuda.synchronize()
    graph, replayed = torch.cuda.CUDAGraph(), outputs()
    with torch.cuda.graph(graph):
        run(ctx, *replayed, backward=False)
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)
        run(ctx, *busy, backward=False)
    load(ctx, 4)
    load(ctx, 5)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        (ctx.backward_window if model == "stacked" else ctx.backward_window_integrated)(0, 4, params, target, busy[2])
    torch.cuda.synchronize()
    for a, b in zip(busy, quiet):
        assert torch.equal(a, b)
    for _ in range(3):
        replayed[1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(replayed[0], quiet[0]) and torch.equal(replayed[1], quiet[1])
    assert [ctx.get_snapshot_csr(t)[1].size for t in (4, 5)] == [len(set(zip(*map(np.ndarray.tolist, seq.edges[t])))) for t in (4, 5)]
    ctx.close()


# one profiled launch per timestep of the backward recurrence, whether gate gradients and product share it (64 and 16 units, but
# for the first timestep) or the width is not for that kernel (136, 44)
@pytest.mark.parametrize("hidden,products", [(64, 0), (16, 0), (136, 2), (44, 2)])
def test_profile_counts_launches_of_the_backward_recurrence_once(hidden, products):
    import torch

    from paper_2501_15348_amd import reinc, synth

    wl = synth.WORKLOADS["c3"].scaled(200, 3, dims=(16, 32), hidden=hidden, rnn="gru", mean_degree=4.0)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 26)
    ctx.load_sequence(synth.make_sequence(wl))
    params, tgt = torch.from_numpy(synth.make_params(wl)).cuda(), torch.from_numpy(synth.make_target(wl)).cuda()
    ctx.forward_window(0, 3, params, tgt, torch.zeros(1, device="cuda"))
    ctx.profile_begin(["elem", "gemm_rows"])
    ctx.backward_window(0, 3, params, tgt, torch.empty_like(params))
    seen = {k: v[0] for k, v in ctx.profile_end().items()}
    assert seen["elem"] == 3 and seen["gemm_rows"] == products + 1, seen  # (and W_i^T's, all timesteps at once)
    ctx.close()


# The timesteps of a window in one launch per direction, the backward one with the input's gradient: both sides of each block
# shape's hidden width, parts of a row that are no whole k-steps, more and fewer column tiles of the input than waves, the
# fp32 instructions (GRU 16, LSTM 8), ragged rows; few rows (no room for the forward weights) and more.
@pytest.mark.parametrize("rnn", ["gru", "lstm"])
@pytest.mark.parametrize("n,hidden,top", [(33, 8, 24), (321, 16, 16), (70, 16, 72), (65, 24, 33), (321, 32, 96), (645, 64, 130), (31, 64, 32),
                                          (129, 40, 200), (70, 96, 64), (833, 128, 160), (96, 128, 31), (65, 104, 48)])
def test_steps_of_a_window_in_one_launch(rnn, n, hidden, top):
    import torch

    from helpers import GRAD_RTOL_FP32, assert_gradients_close, oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    length = 4
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, top), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 27)
    ctx.load_sequence(seq)
    ctx.build_deltas(-1)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target).cuda()

    def run(timed):
        out = [torch.zeros(1, device="cuda"), torch.full((n, hidden), 7.0, device="cuda"), torch.empty_like(params)]
        if timed:  # (timestep by timestep)
            ctx.profile_begin(["rnn", "elem", "gemm_rows"])
        ctx.forward_window(0, length, params, tgt, out[0], out[1])
        ctx.backward_window(0, length, params, tgt, out[2])
        if timed:
            ctx.profile_end()
        torch.cuda.synchronize()
        return out

    one, apart = run(False), run(True)
    assert torch.equal(one[0], apart[0]) and torch.equal(one[1], apart[1])  # (the same arithmetic)
    assert_close(one[2].cpu().numpy(), apart[2].cpu().numpy(), RTOL_FP32, "gradients, together and apart")
    p = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle_graphs(seq), [oracle_feats(seq, t) for t in range(length)]
    _, ref_h, saved = oracle.forward_window(graphs, feats, p, 1, wl.agg, wl.self_loop, rnn, target, keep=True)
    assert_close(one[1].cpu().numpy(), ref_h, RTOL_FP32, "h_last")
    assert_gradients_close(synth.split_params(wl, one[2].cpu().numpy()), saved,
                           lambda sv: oracle.backward_window(graphs, sv, ref_h, p, 1, wl.agg, wl.self_loop, rnn, target),
                           [name for name, _ in synth.param_shapes(wl)], GRAD_RTOL_FP32)
    ctx.close()


def _window(n, hidden, top, rnn, length, edges, x, flat, target, keep=None):
    """A window of a stacked model over given edges (one [2, E] array a snapshot) and features of `n` nodes: loss, h_last and, the
    recurrent steps together or (timed) by themselves, gradients; keep: rows of h_last alone, no gradients."""
    import torch

    from paper_2501_15348_amd import reinc

    ctx = reinc.Context(n, length, (16, top), rnn, hidden, "sum", True, arena_bytes=1 << 30)
    for t in range(length):
        ctx.load_edges(t, edges[t][0], edges[t][1])
        ctx.load_features_full(t, x[t][:n])
    ctx.build_deltas(-1)
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target[:n]).cuda()

    def run(timed):
        out = [torch.zeros(1, device="cuda"), torch.full((n, hidden), 7.0, device="cuda"), torch.empty_like(params)]
        if timed:
            ctx.profile_begin(["rnn", "elem", "gemm_rows"])
        ctx.forward_window(0, length, params, tgt, out[0], out[1])
        if keep is None:
            ctx.backward_window(0, length, params, tgt, out[2])
        if timed:
            ctx.profile_end()
        torch.cuda.synchronize()
        return out

    got = run(False)[1][:keep] if keep is not None else (run(False), run(True))
    ctx.close()
    return got


# Recurrent steps gate by gate, in the launch of a window and by themselves: they are taken from 16 385 rows on, seen by the last
# bits of the other rows, which a node without edges more changes (and does not where all gates go together).  Two and four
# waves of columns, one to five tiles of units on them (a fifth is a wave's second), blocks of 32 rows (more than 256 terms),
# products that leave the ring of four early or not, a first step of fewer inputs than the ring has steps; of a GRU from 200 terms,
# 33 inputs and 64 units on.
@pytest.mark.parametrize("rnn,n,hidden,top,by_gate", [
    ("lstm", 16385, 64, 24, True), ("lstm", 16448, 64, 16, True), ("lstm", 16411, 96, 33, True), ("lstm", 16411, 96, 168, True),
    ("lstm", 16391, 128, 31, True), ("lstm", 16447, 128, 160, True), ("lstm", 16385, 160, 40, True), ("lstm", 16420, 160, 120, True),
    ("lstm", 16385, 72, 40, False), ("gru", 16385, 64, 144, True), ("gru", 16448, 64, 194, True), ("gru", 16411, 96, 104, True),
    ("gru", 16391, 128, 160, True), ("gru", 16447, 160, 40, True), ("gru", 16385, 160, 65, True), ("gru", 16385, 64, 96, False),
    ("gru", 16391, 192, 31, False),
])
def test_window_gate_by_gate(rnn, n, hidden, top, by_gate):
    import torch

    from helpers import GRAD_RTOL_FP32, assert_gradients_close
    from paper_2501_15348_amd import synth

    # (at most 8e6 units of layer 1: about two of them are so near zero, 3e-7 of their rms, that rounding switches them, and the
    # gradients are compared under either decision for up to three)
    length, fewer = 2 if top > 160 else 3, 16384
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, top), hidden=hidden, rnn=rnn, mean_degree=2.0)
    rng = np.random.default_rng(n + 7 * hidden + 31 * top)
    edges = [rng.integers(0, fewer, (2, 2 * fewer)).astype(np.int32) for _ in range(length)]
    x = rng.standard_normal((length, n, 16)).astype(np.float32)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    one, apart = _window(n, hidden, top, rnn, length, edges, x, flat, target)
    assert torch.equal(one[0], apart[0]) and torch.equal(one[1], apart[1])  # (the same arithmetic)
    together = _window(fewer, hidden, top, rnn, length, edges, x, flat, target, keep=fewer)
    assert torch.equal(one[1][:fewer], together) != by_gate
    p = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle.graphs_of(edges, n), [v.astype(np.float64) for v in x]
    _, ref_h, saved = oracle.forward_window(graphs, feats, p, 1, "sum", True, rnn, target, keep=True)
    assert_close(one[1].cpu().numpy(), ref_h, RTOL_FP32, "h_last")
    assert_gradients_close(synth.split_params(wl, one[2].cpu().numpy()), saved,
                           lambda sv: oracle.backward_window(graphs, sv, ref_h, p, 1, "sum", True, rnn, target),
                           [name for name, _ in synth.param_shapes(wl)], GRAD_RTOL_FP32)


# A step by itself, gate by gate: one tile of units on one wave of columns (LSTM 32), two and four waves, blocks of 32 rows, ragged
# rows; with and without a state, the state's halves each by itself, and without saved gates, whose results are the same bits.
@pytest.mark.parametrize("kind,n,d,h", [("lstm", 129, 16, 32), ("lstm", 65, 100, 32), ("lstm", 70, 33, 64), ("lstm", 193, 100, 100),
                                        ("lstm", 33, 300, 40), ("lstm", 64, 90, 160), ("gru", 65, 136, 64), ("gru", 129, 152, 49),
                                        ("gru", 70, 330, 64), ("gru", 193, 100, 100), ("gru", 33, 80, 160), ("gru", 31, 300, 200)])
def test_step_gate_by_gate(ctx, kind, n, d, h):
    import torch

    rng = np.random.default_rng(n + 7 * d + 13 * h)
    kg = 3 if kind == "gru" else 4
    draw = lambda *shape: rng.standard_normal(shape).astype(np.float32)  # noqa: E731
    x, hp, cp = draw(n, d), draw(n, h), draw(n, h)
    wi, wh, bi, bh = draw(d, kg * h) / np.float32(d**0.5), draw(h, kg * h) / np.float32(h**0.5), 0.3 * draw(kg * h), 0.3 * draw(kg * h)
    dev = lambda v: None if v is None else torch.from_numpy(v).cuda()  # noqa: E731
    up = lambda v: v.astype(np.float64)  # noqa: E731
    zero = np.zeros((n, h))
    for state in ((hp, cp), (None, None)) + (((None, cp), (hp, None)) if kind == "lstm" else ()):
        h0, c0 = state[0], state[1] if kind == "lstm" else None
        saved = torch.empty((n, 4 * h), device="cuda")
        args = [dev(v) for v in (x, h0, c0, wi, wh, bi, bh)]
        h_out, c_out = ctx.rnn_step(kind, *args, saved)
        bare = ctx.rnn_step(kind, *args, None)
        assert torch.equal(bare[0], h_out) and (kind == "gru" or torch.equal(bare[1], c_out))
        rh, rc = zero if h0 is None else up(h0), zero if c0 is None else up(c0)
        if kind == "gru":
            ref_h, gates = oracle.gru_cell(up(x), rh, up(wi), up(wh), up(bi), up(bh))
        else:
            ref_h, ref_c, gates = oracle.lstm_cell(up(x), rh, rc, up(wi), up(wh), up(bi), up(bh))
            assert_close(c_out.cpu().numpy(), ref_c, RTOL_FP32, "c")
        assert_close(h_out.cpu().numpy(), ref_h, RTOL_FP32, "h")
        assert_close(saved.cpu().numpy(), np.concatenate(gates, axis=1), RTOL_FP32, "saved gates")


# Non-finite inputs, states and weights of a step gate by gate: rows stay by themselves, a column of weights reaches its unit alone.
# An infinite input makes its gates 0, 1 or -1 and 1 by the terms' signs as in fp32 (no NaN out of planes), NaN makes NaN.
@pytest.mark.parametrize("kind,n,d,h", [("lstm", 130, 100, 100), ("lstm", 100, 300, 40), ("gru", 130, 100, 100), ("gru", 100, 136, 64)])
def test_non_finite_values_in_a_step_gate_by_gate(ctx, kind, n, d, h):
    import torch

    g = torch.Generator(device="cuda").manual_seed(n + d)
    kg = 3 if kind == "gru" else 4
    x, hp = torch.randn(n, d, generator=g, device="cuda"), torch.randn(n, h, generator=g, device="cuda")
    cp = torch.randn(n, h, generator=g, device="cuda") if kind == "lstm" else None
    wi = torch.randn(d, kg * h, generator=g, device="cuda") / d**0.5
    wh = torch.randn(h, kg * h, generator=g, device="cuda") / h**0.5
    b = torch.randn(kg * h, generator=g, device="cuda")

    def step(x, wi):
        saved = torch.empty(n, 4 * h, device="cuda")
        return ctx.rnn_step(kind, x, hp, cp, wi, wh, b, b, saved)[0], saved

    clean = step(x, wi)
    bad = x.clone()
    bad[7, 3], bad[70, d - 1], bad[n - 1, 0] = float("inf"), float("nan"), -float("inf")
    out, saved = step(bad, wi)
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[[7, 70, n - 1]] = False
    assert torch.equal(out[keep], clean[0][keep]) and torch.equal(saved[keep], clean[1][keep])
    assert bool(torch.isnan(out[70]).all())
    for row, col, sign in ((7, 3, 1), (n - 1, 0, -1)):
        want = torch.sigmoid(sign * wi[col, :2 * h] * float("inf"))
        assert torch.equal(saved[row, :2 * h], want)
        last = torch.sign(sign * wi[col, 2 * h:3 * h])  # (n, or the LSTM's g)
        assert torch.equal(saved[row, 2 * h:3 * h], last)
    weights = wi.clone()
    weights[5, 9] = float("inf")  # of the first gate, unit 9
    out, saved = step(x, weights)
    others = torch.ones(h, dtype=torch.bool, device="cuda")
    others[9] = False
    assert torch.equal(out[:, others], clean[0][:, others])
    assert torch.equal(saved[:, 9], torch.sigmoid(x[:, 5] * float("inf"))) and not bool(torch.isnan(out[:, 9]).any())


# Inputs as wide as the state: the gradients of W_i and W_h come out of one launch, over one timestep, a batch of them and two
# batches; a slab a wave, four slabs a block inside the output and over its edge, rows that end inside a trip.
@pytest.mark.parametrize("rnn", ["gru", "lstm"])
@pytest.mark.parametrize("n,hidden,length", [(33, 32, 3), (701, 64, 1), (701, 64, 3), (645, 96, 3), (897, 128, 3), (130, 128, 9), (70, 40, 9)])
def test_gradients_of_both_recurrent_weights_in_one_launch(rnn, n, hidden, length):
    import torch

    from helpers import GRAD_RTOL_FP32, assert_gradients_close, oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, hidden), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 28)
    ctx.load_sequence(seq)
    ctx.build_deltas(-1)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target).cuda()
    loss, grads = torch.zeros(1, device="cuda"), torch.empty_like(params)
    ctx.forward_window(0, length, params, tgt, loss)
    ctx.backward_window(0, length, params, tgt, grads)
    p = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle_graphs(seq), [oracle_feats(seq, t) for t in range(length)]
    _, ref_h, saved = oracle.forward_window(graphs, feats, p, 1, wl.agg, wl.self_loop, rnn, target, keep=True)
    assert_gradients_close(synth.split_params(wl, grads.cpu().numpy()), saved,
                           lambda sv: oracle.backward_window(graphs, sv, ref_h, p, 1, wl.agg, wl.self_loop, rnn, target),
                           [name for name, _ in synth.param_shapes(wl)], GRAD_RTOL_FP32)
    ctx.close()


# A backward pass whose scratch holds the prepared W_h^T but not W_i^T keeps the steps that make gate gradients and their
# product with W_h^T together, and multiplies with W_i as it is (a GRU's gate gradients lie 4 H apart, 3 H wide).
@pytest.mark.parametrize("rnn", ["gru", "lstm"])
def test_backward_with_room_for_the_recurrent_weights_alone(rnn):
    import torch

    from paper_2501_15348_amd import reinc, synth

    length, hidden = 3, 64
    wl = synth.WORKLOADS["c3"].scaled(65, length, dims=(16, 512), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    params, tgt = torch.from_numpy(synth.make_params(wl, bias_scale=0.2)).cuda(), torch.from_numpy(synth.make_target(wl)).cuda()

    def run(arena, timed=False):
        ctx = reinc.Context.for_workload(wl, arena_bytes=arena)
        try:
            ctx.load_sequence(seq)
            grads = torch.full_like(params, 7.0)
            ctx.forward_window(0, length, params, tgt, torch.zeros(1, device="cuda"))
            if timed:
                ctx.profile_begin(["elem", "gemm_rows"])
            ctx.backward_window(0, length, params, tgt, grads)
            seen = {k: v[0] for k, v in ctx.profile_end().items()} if timed else {}
            torch.cuda.synchronize()
            return grads, seen
        except reinc.ReincError:
            return None, {}
        finally:
            ctx.close()

    roomy, _ = run(1 << 26)
    low, high = 1 << 18, 1 << 26  # the smallest arena that the pass takes: no room for either
    while high - low > 4096:
        mid = (low + high) // 2 & ~255
        low, high = (low, mid) if run(mid)[0] is not None else (mid, high)
    tight = high + (64 << 10)  # W_h^T takes 48 KiB (GRU) or 64 KiB at most, W_i^T 384 KiB or more, a second timestep 380 KiB
    tight += (16 << 10) if rnn == "lstm" else 0
    plain, _ = run(tight)
    counted, seen = run(tight, True)
    assert seen["elem"] == length and seen["gemm_rows"] == length, seen  # (W_i^T's, one per batch of one timestep)
    for grads in (plain, counted):
        assert_close(grads.cpu().numpy(), roomy.cpu().numpy(), RTOL_FP32, "gradients")


# The backward recurrence is as close to 64 bits as the product of a gate gradient's row with W_i^T by itself (timed passes
# launch it apart), and rows that share a block with wide ones are as close as among their like.  Nodes without edges whose
# features are the unit vectors: layer 1's weight gradient holds the rows of the input's gradient.
@pytest.mark.parametrize("rnn,hidden", [("gru", 8), ("gru", 16), ("gru", 24), ("gru", 32), ("gru", 40), ("gru", 64), ("gru", 128),
                                        ("lstm", 8), ("lstm", 16), ("lstm", 24), ("lstm", 32), ("lstm", 64), ("lstm", 128)])
def test_backward_products_are_as_close_as_those_of_a_launch_each(rnn, hidden):
    import torch

    from helpers import oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    n = 256
    wl = synth.WORKLOADS["c3"].scaled(n, 1, dims=(n, 100), hidden=hidden, rnn=rnn, agg="sum", feat_dtype="fp32", mean_degree=4.0)
    seq = synth.make_sequence(wl)
    seq.edges[0] = (np.zeros(0, dtype=np.int32), np.zeros(0, dtype=np.int32))
    seq.x0 = np.eye(n, dtype=np.float32)
    flat = synth.make_params(wl)
    synth.split_params(wl, flat)["b1"][:] = 1.0  # (every unit of layer 1 is on)
    normal = synth.make_target(wl)
    huge = normal.copy()
    huge[::32, 0] *= 1e19  # the row's other elements are below 2^-60 of it
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 26)
    ctx.load_sequence(seq)
    params = torch.from_numpy(flat).cuda()
    rest = np.arange(n) % 32 != 0

    def error(target, timed):
        tgt, grads = torch.from_numpy(target).cuda(), torch.empty_like(params)
        ctx.forward_window(0, 1, params, tgt, torch.zeros(1, device="cuda"))
        if timed:
            ctx.profile_begin(["elem"])
        ctx.backward_window(0, 1, params, tgt, grads)
        if timed:
            ctx.profile_end()
        q = synth.split_params(wl, flat.astype(np.float64))
        _, ref_h, saved = oracle.forward_window(oracle_graphs(seq), [oracle_feats(seq, 0)], q, 1, "sum", True, rnn, target.astype(np.float64), keep=True)
        ref = oracle.backward_window(oracle_graphs(seq), saved, ref_h, q, 1, "sum", True, rnn, target.astype(np.float64))["W1"][rest]
        got = synth.split_params(wl, grads.cpu().numpy().astype(np.float64))["W1"][rest]
        return np.linalg.norm(got - ref) / np.linalg.norm(ref)

    apart, together, beside_wide = error(normal, True), error(normal, False), error(huge, False)
    ctx.close()
    assert together <= 1.005 * apart, (together, apart)  # (the rms of 24 000 rounded values is known to about 0.5 %)
    assert beside_wide <= 1.05 * together, (beside_wide, together)


# The widest cells whose product with W_i^T keeps three bf16 planes over many rows: by itself, timed or not, from the same
# gate gradients.
@pytest.mark.parametrize("rnn,hidden", [("gru", 32), ("lstm", 16)])
def test_input_gradient_of_few_terms_keeps_its_product(rnn, hidden):
    import torch

    from paper_2501_15348_amd import reinc, synth

    length, n = 8, 8193
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, 40), hidden=hidden, rnn=rnn, mean_degree=2.0)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 28)
    ctx.load_sequence(synth.make_sequence(wl))
    params, tgt = torch.from_numpy(synth.make_params(wl, bias_scale=0.2)).cuda(), torch.from_numpy(synth.make_target(wl)).cuda()
    ctx.forward_window(0, length, params, tgt, torch.zeros(1, device="cuda"))
    grads = []
    for timed in (False, True):
        grads.append(torch.empty_like(params))
        if timed:
            ctx.profile_begin(["elem", "gemm_rows"])
        ctx.backward_window(0, length, params, tgt, grads[-1])
    assert ctx.profile_end()["gemm_rows"][0] == 1  # (all timesteps at once)
    assert torch.equal(grads[0], grads[1])
    ctx.close()


# A GRU's gate gradients take 4 H floats a row: so many more timesteps of a window fit the arena at once (the product with
# W_i^T is launched once per batch of timesteps).
def test_batch_of_timesteps_counts_the_gate_gradients_once():
    import torch

    from paper_2501_15348_amd import reinc, synth

    n, hidden, length = 20000, 64, 4
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, 16), hidden=hidden, rnn="gru", mean_degree=2.0)
    seq = synth.make_sequence(wl)
    params, tgt = torch.from_numpy(synth.make_params(wl)).cuda(), torch.from_numpy(synth.make_target(wl)).cuda()

    def batches(mib):
        ctx = reinc.Context.for_workload(wl, arena_bytes=mib << 20)
        try:
            ctx.load_sequence(seq)
            ctx.forward_window(0, length, params, tgt, torch.zeros(1, device="cuda"))
            ctx.profile_begin(["gemm_rows"])
            ctx.backward_window(0, length, params, tgt, torch.empty_like(params))
            return ctx.profile_end()["gemm_rows"][0]
        except reinc.ReincError:
            return length + 1
        finally:
            ctx.close()

    def smallest(most):  # the smallest arena that needs at most so many batches, in MiB
        low, high = 16, 1024
        while high - low > 1:
            mid = (low + high) // 2
            low, high = (low, mid) if batches(mid) <= most else (mid, high)
        return high

    grown = smallest(1) - smallest(length)  # three timesteps more: gate gradients, three arrays of layer gradients ...
    partials = 3 * n // 256 * (16 + 16 + 1 + hidden + 1) * 3 * hidden * 4  # ... and at most the weight gradients' partial sums
    assert grown <= (3 * n * (4 * hidden + 3 * hidden) * 4 + partials) / 2**20 + 2, grown


# The rare branches of a window's recurrent launches: weights with elements far below the others of their row (wide columns of
# W_h^T and W_i^T, and of the forward weights), input rows with three and with twelve elements far below the row's largest one
# (which meets no weight, so that the others decide), states with elements near 2^-40.  Forward bitwise against a launch per
# step, everything against 64 bits.
@pytest.mark.parametrize("rnn,n,hidden,top", [(rnn, 833, hidden, 48) for rnn in ("gru", "lstm") for hidden in (40, 64, 128)]
                         + [("gru", 16397, 96, 104), ("gru", 16397, 64, 144), ("lstm", 16397, 64, 48), ("lstm", 16397, 160, 48)])  # (gate by gate)
@pytest.mark.parametrize("case", ["columns", "listed", "wide", "state"])
def test_unequal_magnitudes_in_the_steps_of_a_window(rnn, n, hidden, top, case):
    import torch

    from helpers import oracle_feats, oracle_graphs
    from paper_2501_15348_amd import reinc, synth

    length = 4 if n < 16384 else 3
    wl = synth.WORKLOADS["c3"].scaled(n, length, dims=(16, top), hidden=hidden, rnn=rnn, mean_degree=4.0)
    seq = synth.make_sequence(wl)
    ctx = reinc.Context.for_workload(wl, arena_bytes=1 << 27 if n < 16384 else 1 << 30)
    ctx.load_sequence(seq)
    ctx.build_deltas(-1)
    flat, target = synth.make_params(wl, bias_scale=0.2), synth.make_target(wl)
    p = synth.split_params(wl, flat)  # (views)
    p["b1"][:] = np.abs(p["b1"]) + 0.1
    groups = [np.arange(top)]  # columns of layer 1 of like magnitude
    if case == "columns":
        for name, row in (("W_h", 3), ("W_h", hidden - 1), ("W_i", 5), ("W_i", top - 1)):
            p[name][row, 2::7] *= np.float32(2.0**-40)
    elif case == "state":
        unit = 2 * hidden + np.array([1, 7, hidden - 2])  # the candidate gate's columns of three units
        for name in ("W_i", "W_h", "b_i", "b_h"):
            p[name][..., unit] *= np.float32(2.0**-40)
    else:
        few = np.arange(1, 4 if case == "listed" else 13)
        rest = np.arange(few[-1] + 1, top)
        for cols, up in ((np.array([0]), 36), (rest, 20)):
            p["W1"][:, cols] *= np.float32(2.0**up)
            p["b1"][cols] *= np.float32(2.0**up)
        p["W_i"][0] = 0.0
        p["W_i"][rest] *= np.float32(2.0**-20)
        groups = [few, rest]
    params, tgt = torch.from_numpy(flat).cuda(), torch.from_numpy(target).cuda()

    def run(timed):
        out = [torch.zeros(1, device="cuda"), torch.full((n, hidden), 7.0, device="cuda"), torch.empty_like(params)]
        if timed:
            ctx.profile_begin(["rnn", "elem", "gemm_rows"])
        ctx.forward_window(0, length, params, tgt, out[0], out[1])
        ctx.backward_window(0, length, params, tgt, out[2])
        if timed:
            ctx.profile_end()
        torch.cuda.synchronize()
        return out

    one, apart = run(False), run(True)
    ctx.close()
    assert torch.equal(one[0], apart[0]) and torch.equal(one[1], apart[1])
    q = synth.split_params(wl, flat.astype(np.float64))
    graphs, feats = oracle_graphs(seq), [oracle_feats(seq, t) for t in range(length)]
    _, ref_h, saved = oracle.forward_window(graphs, feats, q, 1, wl.agg, wl.self_loop, rnn, target, keep=True)
    ref = oracle.backward_window(graphs, saved, ref_h, q, 1, wl.agg, wl.self_loop, rnn, target)
    assert_close(one[1].cpu().numpy(), ref_h, RTOL_FP32, "h_last")
    for what, grads in (("together", one[2]), ("apart", apart[2])):
        got = synth.split_params(wl, grads.cpu().numpy())
        for name in ("W_h", "b_i", "b_h"):
            assert_close(got[name], ref[name], RTOL_FP32, f"{name}, {what}")
        for cols in groups:
            assert_close(got["W_i"][cols], ref["W_i"][cols], RTOL_FP32, f"W_i, {what}")
            # (a unit of layer 1 near zero may be on in one and off in the other: a few entries of the sums over all rows)
            assert_close(got["W1"][:, cols], ref["W1"][:, cols], 1e-3, f"W1, {what}")
