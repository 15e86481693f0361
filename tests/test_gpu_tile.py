"""The tile form of the GEMM and accumulate kernels (automatic policy): one
workgroup tile of 64 x 64 to 128 x 256, chosen by the product's size, with its
last tiles moved back over their neighbours, the k tail as the first chunk, k
shared among wave groups where tiles are few, and buffer loads of any
alignment.

The bar is that of the GEMM tests (gpu_util.gate): each FP32 addition moves a
result by at most an ulp of a partial sum bounded by N, whatever the order of
the sums, and the wave groups' partial sums add at most three more additions,
within the bar's k + 2 and k + 8 for every k here from 31 on; below that one
group computes the product.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_15152_amd as pkg
import synth
from gpu_util import assert_periodic, device, gate, gate_applies, periodic_batch, to_np

pytestmark = pytest.mark.gpu

GUARD = 64


def _strided(X, pad, offset):
    """X ([batch, r, c]) on the device with rows c + pad apart, starting
    `offset` floats into a buffer."""
    b, r, c = X.shape
    flat = torch.full((b * r * (c + pad) + offset,), float("nan"), device=device())
    view = flat[offset:].view(b, r, c + pad)[:, :, :c]
    view.copy_(X)
    return view


def _output(b, r, c, pad, offset):
    """A NaN output of that kind with guard values around it."""
    flat = torch.full((b * r * (c + pad) + offset + 2 * GUARD,), float("nan"), device=device())
    body = flat[GUARD + offset:GUARD + offset + b * r * (c + pad)].view(b, r, c + pad)
    return flat, body, body[:, :, :c]


def _check_untouched(flat, body, c, offset):
    assert torch.isnan(flat[:GUARD + offset]).all()
    assert torch.isnan(flat[GUARD + offset + body.numel():]).all()
    assert torch.isnan(body[:, :, c:]).all()


# batch, m, n, k, row padding, offset of the bases: tiles moved back by one line
# and by all but one, one tile exactly and one line more, matrices smaller than
# a tile in m, n or both, k of one chunk, one value more or less and of odd and
# even numbers of chunks per wave group (FORMS below has every tile shape)
SHAPES = [
    (1, 64, 64, 66, 0, 0), (3, 65, 65, 65, 0, 0), (2, 127, 129, 95, 0, 1), (1, 63, 200, 97, 3, 2),
    (2, 200, 61, 130, 1, 0), (5, 33, 35, 129, 2, 3), (4, 1, 4, 70, 1, 1), (2, 3, 300, 31, 0, 0),
    (1, 70, 4, 33, 1, 0), (2, 66, 5, 1, 0, 0), (2, 68, 68, 6, 1, 1), (1, 100, 100, 1027, 0, 0),
    (1, 131, 70, 2050, 0, 0), (300, 130, 67, 67, 0, 0), (600, 129, 131, 99, 1, 1),
    (40, 300, 260, 287, 0, 0), (3, 1025, 1000, 161, 1, 0), (8, 1001, 999, 97, 0, 0),
    (1, 1100, 1500, 200, 0, 0), (1, 512, 512, 512, 0, 0), (20, 128, 640, 768, 0, 0)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_products(shape):
    b, m, n, k, pad, offset = shape
    print(f"case tile {shape}", flush=True)
    A, B = synth.gemm_inputs(b, m, n, k, seed=b + m + n + k)
    flat, body, C = _output(b, m, n, pad, offset)
    pkg.sgemm_emu_batched(_strided(A, pad, offset), _strided(B, pad, offset), C)
    _check_untouched(flat, body, n, offset)
    items = sorted({0, b // 2, b - 1})
    ref = oracle.gemm(A[items].numpy(), B[items].numpy())
    gate(to_np(C[items]), ref, k, f"tile {shape}", max_gate=gate_applies(ref))
    # every item against the general kernel, which takes any form of operand:
    # both within the bar's distance of the same exact sums
    general = pkg.sgemm_emu_batched(_strided(A, pad, offset), _strided(B, pad, offset),
                                    policy=pkg.Policy(pkg.FLOW_SPLIT, 1, pkg.TILE_64x64))
    N = torch.bmm(A.abs().to(device()).double(), B.abs().to(device()).double())
    assert bool(((C.double() - general).abs() <= 2 * (k + 2) * 2.0 ** -23 * N).all())


# One ragged product per form of the kernel (rows and columns of the workgroup
# tile, wave groups): tiles moved back in m and n, a k tail, several items, and
# for 64 x 64 a matrix smaller than the tile as well.
FORMS = {(64, 64, 1): [(2, 65, 70, 67), (3, 33, 40, 67)],
         (64, 64, 2): [(1, 65, 70, 515), (2, 33, 40, 515)],
         (64, 64, 4): [(1, 65, 70, 2051), (1, 33, 40, 2050)],
         (128, 64, 1): [(60, 390, 70, 331)], (128, 64, 2): [(60, 130, 70, 331)],
         (128, 128, 1): [(40, 200, 271, 67)], (128, 128, 2): [(60, 130, 141, 701)],
         (128, 256, 1): [(60, 200, 271, 67)]}
ACC_FORMS = {**FORMS, (128, 64, 1): [(60, 390, 70, 330)], (128, 64, 2): [(60, 130, 70, 330)],
             (128, 128, 1): [(40, 200, 270, 67)], (128, 128, 2): [(60, 130, 140, 700)],
             (128, 256, 1): [(40, 130, 700, 33)]}


def _cases(forms):
    return [(f, s) for f, shapes in forms.items() for s in shapes]


def _fid(c):
    return "x".join(map(str, c[0])) + "-" + "x".join(map(str, c[1]))


@pytest.mark.parametrize("case", _cases(FORMS), ids=_fid)
def test_every_form(case):
    form, (b, m, n, k) = case
    print(f"case tile form {case}", flush=True)
    A, B = synth.gemm_inputs(b, m, n, k, seed=3 * m + n + k)
    flat, body, C = _output(b, m, n, 0, 0)
    Ad, Bd = A.to(device()), B.to(device())
    assert pkg.sgemm_emu_launch_form(Ad, Bd, C) == ("gemm_tile_kernel", form)
    pkg.sgemm_emu_batched(Ad, Bd, C)
    _check_untouched(flat, body, n, 0)
    items = sorted({0, b // 2, b - 1})
    ref = oracle.gemm(A[items].numpy(), B[items].numpy())
    gate(to_np(C[items]), ref, k, f"tile form {case}", max_gate=gate_applies(ref))
    general = pkg.sgemm_emu_batched(Ad, Bd, policy=pkg.Policy(pkg.FLOW_SPLIT, 1, pkg.TILE_64x64))
    N = torch.bmm(A.abs().to(device()).double(), B.abs().to(device()).double())
    assert bool(((C.double() - general).abs() <= 2 * (k + 2) * 2.0 ** -23 * N).all())


@pytest.mark.parametrize("k", [70, 1030])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 65520.0, 3e38])
def test_operands_outside_the_split(value, k):
    """A value of A or B whose split is not finite makes its row or column of C
    non-finite, as in the general kernel, and nothing else: not what tiles
    that overlap compute twice, not what the k tail or the wave groups share."""
    m, n = 150, 141
    A, B = synth.gemm_inputs(1, m, n, k, seed=9)
    clean = to_np(pkg.sgemm_emu_batched(A.to(device()), B.to(device())))
    rows, cols = [0, 21, 63, 64, 86, m - 1], [0, 63, 77, 128, n - 1]
    for i, r in enumerate(rows):
        A[0, r, (i * 37 + k - 1) % k] = value  # the k tail among them
    for i, c in enumerate(cols):
        B[0, (i * 29 + k - 1) % k, c] = value
    Ad, Bd = A.to(device()), B.to(device())
    C = to_np(pkg.sgemm_emu_batched(Ad, Bd))
    assert pkg.sgemm_emu_launch_form(Ad, Bd, torch.empty(1, m, n, device=device()))[0] == (
        "gemm_tile_kernel")
    general = to_np(pkg.sgemm_emu_batched(
        Ad, Bd, policy=pkg.Policy(pkg.FLOW_SPLIT, 1, pkg.TILE_64x64)))
    hit = np.zeros((1, m, n), dtype=bool)
    hit[:, rows, :] = True
    hit[:, :, cols] = True
    assert not np.isfinite(C[hit]).any() and not np.isfinite(general[hit]).any()
    assert np.array_equal(C[~hit], clean[~hit])


def test_shared_operands():
    """One A or one B for the whole batch (item stride 0)."""
    A, B = synth.gemm_inputs(6, 150, 170, 203, seed=5)
    dev = device()
    for a, b in ((A, B[0]), (A[0], B)):
        C = to_np(pkg.sgemm_emu_batched(a.to(dev), b.to(dev)))
        an = A.numpy() if a.dim() == 3 else np.repeat(A[:1].numpy(), 6, axis=0)
        bn = B.numpy() if b.dim() == 3 else np.repeat(B[:1].numpy(), 6, axis=0)
        gate(C, oracle.gemm(an, bn), 203, "tile, shared operand")


def test_integers_exact():
    """Small integers: every product and sum is exact in any order (also with
    the k tail and the wave groups' sums), so the result is."""
    g = synth.rng(8)
    A = synth.integer_matrix((2, 150, 1031), g, -8, 8)
    B = synth.integer_matrix((2, 1031, 90), g, -8, 8)
    C = to_np(pkg.sgemm_emu_batched(A.to(device()), B.to(device())))
    ref = np.einsum("bik,bkj->bij", A.numpy().astype(np.int64), B.numpy().astype(np.int64))
    assert np.array_equal(C, ref.astype(np.float32))


# Row pitches (floats) on both sides of the tile kernel's 32-bit offsets: 64
# rows of C reach 2^31 bytes at pitch 2^23 (less a tile's columns).
@pytest.mark.parametrize("ldc", [(1 << 23) - 72, (1 << 23) - 64, 1 << 23])
@pytest.mark.parametrize("k", [320, 319])
def test_far_rows(k, ldc):
    """C rows on both sides of the reach of the tile kernel's offsets: past it
    the calls take the kernels that address with 64-bit pointers (the register
    flow, and for unaligned rows the general kernel)."""
    m, n = 66, 68
    print(f"case tile far rows k={k} ldc={ldc}", flush=True)
    A, B = synth.gemm_inputs(1, m, n, k, seed=6)
    Ad, Bd = A.to(device()), B.to(device())
    buf = torch.full(((m - 1) * ldc + n,), float("nan"), device=device())
    C = buf.as_strided((1, m, n), (0, ldc, 1))
    kernel, _ = pkg.sgemm_emu_launch_form(Ad, Bd, C)
    far = "bgemm_reg_kernel" if k % 4 == 0 else "bgemm_emu_kernel"
    assert kernel == ("gemm_tile_kernel" if ldc < (1 << 23) - 64 else far)
    pkg.sgemm_emu_batched(Ad, Bd, C)
    gate(to_np(C), oracle.gemm(A.numpy(), B.numpy()), k, f"tile, far rows k={k}")
    del buf, C
    torch.cuda.empty_cache()


def test_far_rows_of_large_products():
    """A large product of nearly whole tiles with C rows past the 128 x 256
    tile's 32-bit offsets (its 64-bit stores): outputs sampled on all seams
    and corners, and nothing written between the rows."""
    m, n, k, ldc = 4100, 4300, 2060, (1 << 22) + 4
    print(f"case tile far rows large {m}x{n}x{k} ldc={ldc}", flush=True)
    A, B = synth.gemm_inputs(1, m, n, k, seed=7)
    Ad, Bd = A.to(device()), B.to(device())
    buf = torch.full(((m - 1) * ldc + n,), float("nan"), device=device())
    C = buf.as_strided((1, m, n), (0, ldc, 1))
    assert pkg.sgemm_emu_launch_form(Ad, Bd, C) == ("gemm_tile_kernel", (128, 256, 1))
    pkg.sgemm_emu_batched(Ad, Bd, C)
    body = to_np(C[0].contiguous())
    assert np.isfinite(body).all()
    assert torch.isnan(buf.as_strided((m - 1, 64), (ldc, 1), n)).all()
    assert torch.isnan(buf.as_strided((m - 1, 64), (ldc, 1), ldc - 64)).all()
    g = np.random.default_rng(3)
    rows = np.unique([0, 127, 128, 3971, 3972, 4095, 4096, m - 1, *g.integers(0, m, 12)])
    cols = np.unique([0, 255, 256, 4043, 4044, 4095, 4096, n - 1, *g.integers(0, n, 12)])
    rr, cc = (x.ravel() for x in np.meshgrid(rows, cols, indexing="ij"))
    ref = oracle.dots(A[0].numpy()[rr], np.ascontiguousarray(B[0].numpy()[:, cc].T))
    gate(body[rr, cc], ref, k, "tile, far rows, large")
    del buf, C
    torch.cuda.empty_cache()


@pytest.mark.parametrize("k", [4, 5])
def test_tall_products(k):
    """One item of more 64 x 64 tiles than a launch of the tile kernel holds
    (8,388,607): the calls take the kernels that split it, accumulate and
    unaligned products alike.  P rows checked against the oracle repeat down
    the matrix; every output row must equal its own bitwise."""
    P, n, m = 1021, 4, 64 * 8388607 + 71
    print(f"case tall m={m} n={n} k={k}", flush=True)
    g = synth.rng(40 + k)
    A, B = synth.uniform((P, k), g), synth.uniform((k, n), g)
    Ad, Bd = periodic_batch(A.to(device()), m), B.to(device())
    D = torch.full((m, n), float("nan"), device=device())
    if k == 4:
        pkg.sgemm_emu_batched_acc(Ad, Bd, None, D)
    else:
        pkg.sgemm_emu_batched(Ad, Bd, D)
    ref = {key: v[0] for key, v in oracle.gemm(A[None].numpy(), B[None].numpy()).items()}
    gate(to_np(D[:P]), ref, k, f"tall k={k}", max_gate=False)
    assert_periodic(D, P, "tall rows")
    del Ad, D
    torch.cuda.empty_cache()


ACC_SHAPES = [(1, 64, 64, 96, 0, 0), (2, 65, 66, 67, 1, 1), (3, 130, 63, 300, 0, 0),
              (2, 5, 131, 40, 2, 3), (1, 129, 260, 1000, 0, 0), (300, 140, 70, 64, 0, 0),
              (30, 270, 520, 130, 1, 2), (2, 4, 4, 9, 0, 0), (1, 2050, 1030, 97, 0, 0)]


@pytest.mark.parametrize("case", _cases(ACC_FORMS), ids=_fid)
@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
def test_every_accumulate_form(case, ta, tb):
    form, (b, m, n, k) = case
    _accumulate((b, m, n, k, 1, 0), ta, tb, 0, form)


@pytest.mark.parametrize("shape", ACC_SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("col", [0, 1])
def test_accumulate(shape, ta, tb, col):
    """Every operand and output layout."""
    _accumulate(shape, ta, tb, col)


def _accumulate(shape, ta, tb, col, form=None):
    """C apart, C in place and no C, against the oracle; with `form`, on that
    form of the tile kernel."""
    b, m, n, k, pad, offset = shape
    print(f"case tile acc {shape} ta={ta} tb={tb} col={col}", flush=True)
    g = synth.rng(m + n + k)
    A, B = synth.uniform((b, m, k), g), synth.uniform((b, k, n), g)
    C = synth.uniform((b, m, n), g)
    stored = lambda X, t: X.transpose(1, 2).contiguous() if t else X  # noqa: E731
    Ad = _strided(stored(A, ta), pad, offset)
    Bd = _strided(stored(B, tb), pad, offset)
    Cs = stored(C, col)
    r, c = Cs.shape[1:]
    kw = dict(op_a=ta, op_b=tb, layout=col)
    items = sorted({0, b // 2, b - 1})
    logical = lambda D: to_np(D[items]).transpose(0, 2, 1) if col else to_np(D[items])  # noqa: E731
    an, bn, cn = A[items].numpy(), B[items].numpy(), C[items].numpy()
    ref = oracle.gemm_acc(an, bn, cn)
    flat, body, D = _output(b, r, c, pad, offset)
    Cd = _strided(Cs, pad, offset)
    if form:
        for addend in (Cd, D, None):
            assert pkg.sgemm_emu_acc_launch_form(Ad, Bd, addend, D, **kw) == ("gemm_tile_kernel",
                                                                              form)
    pkg.sgemm_emu_batched_acc(Ad, Bd, Cd, D, **kw)
    _check_untouched(flat, body, c, offset)
    gate(logical(D), ref, k, f"tile acc {shape}", max_gate=gate_applies(ref))
    apart = D.clone()
    D.copy_(Cs)
    pkg.sgemm_emu_batched_acc(Ad, Bd, D, D, **kw)  # in place: the same sums
    _check_untouched(flat, body, c, offset)
    assert torch.equal(D, apart)
    pkg.sgemm_emu_batched_acc(Ad, Bd, None, D, **kw)
    ref0 = oracle.gemm(an, bn)
    gate(logical(D), ref0, k, f"tile acc, no C {shape}", max_gate=gate_applies(ref0))


@pytest.mark.parametrize("shape", [(2, 65, 66, 40), (1, 129, 260, 300)])
def test_addend_extremes(shape):
    """C entries of any size: infinities (an additive mask) stay what they are,
    the largest and lowest FP32 values and 1e30 absorb a product far below half
    their ulp, NaN stays NaN, and every other output is as without them.  The
    kernel written with the fragment interface gives the same on all of them."""
    b, m, n, k = shape
    g = synth.rng(14)
    A, B = synth.uniform((b, m, k), g).to(device()), synth.uniform((b, k, n), g).to(device())
    C = synth.uniform((b, m, n), g).to(device())
    plain = pkg.sgemm_emu_batched_acc(A, B, C)
    top = torch.finfo(torch.float32).max
    values = [float("inf"), float("-inf"), top, -top, 1e30, -1e30, float("nan")]
    Cx = C.clone()
    marked = torch.zeros_like(C, dtype=torch.bool)
    for i, v in enumerate(values):
        Cx[:, i::11, (3 * i)::13] = v
        marked[:, i::11, (3 * i)::13] = True
    fragments = pkg.sgemm_emu_batched_acc(A, B, Cx, shape=pkg.SHAPE_16x16x32)
    D = pkg.sgemm_emu_batched_acc(A, B, Cx)
    assert torch.equal(D[~marked], plain[~marked])
    for X in (D, fragments):
        assert torch.equal(torch.nan_to_num(X[marked], nan=7.0),
                           torch.nan_to_num(Cx[marked], nan=7.0))
        assert torch.equal(torch.isnan(X), torch.isnan(Cx))


def test_in_place_where_tiles_overlap():
    """Tiles moved back over their neighbours read and write only their own
    outputs: D += A B in place gives the same bits every time."""
    g = synth.rng(12)
    A, B = synth.uniform((4, 321, 70), g).to(device()), synth.uniform((4, 70, 333), g).to(device())
    C = synth.uniform((4, 321, 333), g).to(device())
    first = None
    for _ in range(5):
        D = C.clone()
        pkg.sgemm_emu_batched_acc(A, B, D, D)
        first = D if first is None else first
        assert torch.equal(D, first)
