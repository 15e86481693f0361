"""Parity of the batched inclusive scan computed as x^T U with the
upper-triangular all-ones U built from its rule by foreach_ij (Sec. 4.1,
eq. scan-mat), in emulated FP32 (Sec. 4.4), against the scan oracle.

* row counts around the 1 to 4 rows of a wave and the 32 of a short one
  (1, 7, 8, 9, 100) and lengths around the 1024-value block and the 32-value
  segment (1, 31, 33, 1000, 1024, 1025, 3072);
* few long rows in parts, short rows 32 to a block, and their limits;
* integer inputs give the exact running sums; a unit impulse gives a step;
* in place, padded row strides, unaligned bases;
* values outside the range of the split;
* the full-size workload on sampled rows.

Tolerance: an output sums at most 32 split values inside its segment
(accumulated by the matrix instruction), then takes one fused combine of
the two accumulators, the segment offset from a five-level scan of segment
totals and one addition of it, and one carry addition per earlier block of
the row: at most 32 + 9 + len / 1024 roundings of partial sums bounded by
N.  The element-wise bounds of the GEMM tests (gpu_util.gate) are applied
with k = min(len, 64) + 2 ceil(len / 64), which is at least that count.
|Y - YM| <= (k + 2) 2^-23 N and |Y - Y64| <= (k + 8) 2^-23 N, N the running
sum of |x|.  The ratio gate against the plain FP32 running sum is not
applied: on short prefixes that sum is exact by construction.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_15152_amd as pkg
import synth
from gpu_util import (assert_all_finite, assert_periodic, device, gate, gate_repeated, nan_output,
                      periodic_batch, spread_items, to_np)

pytestmark = pytest.mark.gpu


def _k_eff(length):
    return min(length, 64) + 2 * ((length + 63) // 64)


@pytest.mark.parametrize("rows", [1, 7, 8, 9, 100])
@pytest.mark.parametrize("length", [1, 31, 33, 1000, 1024, 1025, 3072])
def test_parity_shapes(rows, length):
    print(f"case scan rows={rows} len={length}", flush=True)
    X = synth.uniform((rows, length), synth.rng(rows * 7 + length))
    Y = to_np(pkg.sgemm_emu_scan(X.to(device())))
    ref = oracle.scan(X.numpy())
    gate(Y, ref, _k_eff(length), f"scan {rows}x{length}", max_gate=False)


# Few long rows are scanned in parts (three launches): the smallest such row
# and the one below it, a last part of one value, of one block and of whole
# blocks, the most rows taken and one more, parts of more than 4 blocks, odd
# lengths (rows off 16-byte alignment).
PART_SHAPES = [(1, 15 * 1024), (1, 15 * 1024 + 1), (3, 16 * 1024 + 1), (2, 17 * 1024),
               (5, 20 * 1024), (511, 15 * 1024 + 5), (512, 15 * 1024 + 5), (2, 100001),
               (300, 65 * 1024 + 3)]


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("shape", PART_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rows_in_parts(shape, in_place):
    rows, length = shape
    print(f"case scan in parts rows={rows} len={length} in_place={in_place}", flush=True)
    X = synth.uniform((rows, length), synth.rng(rows + length))
    Xd = X.to(device())
    Y = Xd if in_place else torch.full((rows, length), float("nan"), device=device())
    pkg.sgemm_emu_scan(Xd, Y)
    ref = oracle.scan(X.numpy())
    gate(to_np(Y), ref, _k_eff(length), f"scan {rows}x{length}", max_gate=False)


@pytest.mark.parametrize("rows,length", [(3, 20 * 1024 + 5), (40, 100001)])
def test_padded_rows_in_parts(rows, length):
    """Row pitches of X and Y that differ, off 16-byte alignment: nothing is
    written between the rows, neither by the totals nor by the parts."""
    X = synth.uniform((rows, length), synth.rng(rows))
    xbuf = torch.full((rows * (length + 5) + 1,), 7.0, device=device())
    Xv = xbuf[1:].view(rows, length + 5)[:, :length]
    Xv.copy_(X)
    ybuf = torch.full((rows * (length + 12) + 3,), 5.0, device=device())
    whole = ybuf[3:].view(rows, length + 12)
    pkg.sgemm_emu_scan(Xv, whole[:, :length])
    gate(to_np(whole[:, :length]), oracle.scan(X.numpy()), _k_eff(length), "scan padded parts",
         max_gate=False)
    assert bool((whole[:, length:] == 5.0).all()) and bool((ybuf[:3] == 5.0).all())
    assert torch.equal(pkg.sgemm_emu_scan(X.to(device())), whole[:, :length])


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 65520.0, -1e30])
@pytest.mark.parametrize("rows", [8, 600])
def test_values_outside_the_split(rows, value):
    """A value whose split is not finite makes its row NaN to the end, whether
    the row is scanned whole (600 rows) or in parts (8 rows, whose totals are
    plain FP32 sums); what lies before its 32-value segment stays as it was.
    65519 is the largest magnitude on the other side, and stays finite."""
    length = 20 * 1024 + 7
    X = synth.uniform((rows, length), synth.rng(31))
    Xx = X.clone()
    at = [0, 100, 4095, 4096, 9000, length - 1]  # 4095: the last value of a part
    for r, j in enumerate(at):
        Xx[r, j] = value
    Xx[len(at), 5000] = 65519.0
    plain = to_np(pkg.sgemm_emu_scan(X.to(device())))
    Y = pkg.sgemm_emu_scan(Xx.to(device()))
    in_place = Xx.to(device())
    pkg.sgemm_emu_scan(in_place, in_place)
    for out in (to_np(Y), to_np(in_place)):
        for r, j in enumerate(at):
            assert np.isnan(out[r, j:]).all(), (r, j, int(np.isfinite(out[r, j:]).sum()))
            assert np.array_equal(out[r, :j - j % 32], plain[r, :j - j % 32])
        assert np.isfinite(out[len(at):]).all()
        assert np.array_equal(out[len(at) + 1:], plain[len(at) + 1:])


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 129, 5000, 600001])
@pytest.mark.parametrize("length", [1, 2, 5, 7, 8, 9, 16, 17, 30, 32, 33])
def test_short_rows(rows, length):
    """Rows of at most one 32-value segment, 32 of them to a block (and the
    first length past it), with padded rows off 16-byte alignment, in place
    too: against the oracle, bit for bit the scan of whole blocks (which rows
    2^24 floats apart still take), nothing written between the rows."""
    print(f"case scan short rows={rows} len={length}", flush=True)
    X = synth.uniform((rows, length), synth.rng(rows + 37 * length))
    pitch = length + 3
    xbuf = torch.full((rows * pitch + 1,), 7.0, device=device())
    Xv = xbuf[1:].view(rows, pitch)[:, :length]
    Xv.copy_(X)
    ybuf = torch.full((rows * (pitch + 1) + 2,), 5.0, device=device())
    Yv = ybuf[2:].view(rows, pitch + 1)[:, :length]
    pkg.sgemm_emu_scan(Xv, Yv)
    some = spread_items(rows, 2000) if rows > 2000 else np.arange(rows)
    ref = oracle.scan(X[some].numpy())
    gate(to_np(Yv[torch.from_numpy(some).to(device())]), ref, _k_eff(length),
         f"scan {rows}x{length}", max_gate=False)
    assert bool((ybuf[2:].view(rows, pitch + 1)[:, length:] == 5.0).all())
    assert bool((ybuf[:2] == 5.0).all())
    kept = Yv.clone()
    pkg.sgemm_emu_scan(Xv, Xv)
    assert torch.equal(Xv, kept)
    assert bool((xbuf[1:].view(rows, pitch)[:, length:] == 7.0).all())
    if rows in (33, 129) and length in (1, 9, 32):
        far = torch.empty((rows - 1) * (1 << 24) + length, device=device())
        Z = far.as_strided((rows, length), (1 << 24, 1))
        Z.copy_(X)
        pkg.sgemm_emu_scan(Z, Z)
        assert torch.equal(Z, kept)
        del far, Z
        torch.cuda.empty_cache()


@pytest.mark.parametrize("length", [3000, 4096])
def test_integer_exact_and_in_place(length):
    X = synth.integer_matrix((70, length), synth.rng(5), -1000, 1000)
    Xd = X.to(device())
    pkg.sgemm_emu_scan(Xd, Xd)
    exact = np.cumsum(X.numpy().astype(np.int64), axis=1)
    assert np.array_equal(to_np(Xd), exact.astype(np.float32))


@pytest.mark.parametrize("length", [300, 2048])
def test_impulse_gives_step(length):
    X = torch.zeros((40, length))
    X[3, 0] = 2.5
    X[39, length - 1] = -1.0
    X[17, 64] = 3.0
    X[20, min(1023, length - 2)] = 0.75
    Y = to_np(pkg.sgemm_emu_scan(X.to(device())))
    expect = np.cumsum(X.numpy().astype(np.float64), axis=1).astype(np.float32)
    assert np.array_equal(Y, expect)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("length,pitch", [(130, 136), (1024, 1040)])
def test_padded_and_unaligned(offset, length, pitch):
    dev = device()
    X = synth.uniform((45, length), synth.rng(6))
    buf = torch.zeros(45 * pitch + offset, device=dev)
    Xv = buf[offset:].view(45, pitch)[:, :length]
    Xv.copy_(X.to(dev))
    Ybuf = torch.full((45, pitch + 4), 5.0, device=dev)
    pkg.sgemm_emu_scan(Xv, Ybuf[:, :length])
    out = to_np(Ybuf)
    gate(out[:, :length], oracle.scan(X.numpy()), _k_eff(length), "scan padded",
         max_gate=False)
    assert np.all(out[:, length:] == 5.0)


def test_unaligned_output_only():
    """X aligned, Y one element off 16-byte alignment."""
    dev = device()
    X = synth.uniform((9, 2048), synth.rng(7)).to(dev)
    ybuf = torch.full((9 * 2048 + 1,), 5.0, device=dev)
    Y = ybuf[1:].view(9, 2048)
    pkg.sgemm_emu_scan(X, Y)
    out = to_np(ybuf)
    assert out[0] == 5.0
    gate(out[1:].reshape(9, 2048), oracle.scan(to_np(X)), _k_eff(2048), "scan unaligned Y",
         max_gate=False)


def test_workload_scan_sampled():
    """The full workload: every output written (NaN beforehand, finite
    after) and 4096 whole rows spread over the batch held to the bar."""
    w = synth.WORKLOADS["scan_2048"]
    print(f"case workload=scan_2048 rows={w.batch} len={w.n}", flush=True)
    (X,) = synth.workload_inputs(w)
    Y = nan_output((w.batch, w.n))
    pkg.sgemm_emu_scan(X.to(device()), Y)
    assert_all_finite(Y, "scan_2048")
    rows = spread_items(w.batch, 4096)
    Ys = to_np(Y[torch.from_numpy(rows).to(Y.device)])
    ref = oracle.scan(X[rows].numpy())
    e = gate(Ys, ref, _k_eff(w.n), "scan_2048", max_gate=False)
    print(f"scan_2048: err {e[0]:.3e} fp32 running sum {e[1]:.3e}")


# A launch holds 2^31 / 256 - 1 workgroups of four waves, a wave 4 whole rows, or
# 128 rows of at most 32 values.
@pytest.mark.parametrize("length,per_wave", [(33, 4), (1, 128)])
def test_rows_past_one_launch(length, per_wave):
    """More rows than one launch holds.  A pool of P rows is checked against the
    oracle and repeated down the rows; the rows on both sides of every launch
    boundary are held to the bar and every output row must equal its pool row
    bitwise."""
    P = 1021
    per_launch = ((1 << 31) // 256 - 1) * 4 * per_wave
    rows = per_launch + 2 * P + 7
    print(f"case scan rows={rows} len={length}", flush=True)
    X = synth.uniform((P, length), synth.rng(99))
    Xd = periodic_batch(X.to(device()), rows)
    Y = torch.full((rows, length), float("nan"), device=device())
    pkg.sgemm_emu_scan(Xd, Y)
    ref = oracle.scan(X.numpy())
    gate(to_np(Y[:P]), ref, _k_eff(length), "scan pool", max_gate=False)
    bounds = range(per_launch, rows, per_launch)
    gate_repeated(Y, ref, P, [r + d for r in bounds for d in (-1, 0, 1)] + [rows - 1],
                  _k_eff(length), "scan, launch boundary")
    assert_periodic(Y, P, "scan rows", slab_items=1 << 26)
    del Xd, Y
    torch.cuda.empty_cache()
