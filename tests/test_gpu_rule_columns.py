"""Rule-built products over the forms of B and C their kernels tell apart: one
or two 32-column blocks per wave, even column counts (8-byte accesses) and odd
ones, a last group of one block, bases and row pitches of any alignment, and
row pitches past the reach of 32-bit byte offsets (64 rows of 2^22 floats).

The bars are those of the Householder and Givens tests: gpu_util.gate with
k = 64 for the dense reflector and k = 2 for the rotation, whose rows sum at
most two nonzero terms.
"""
import pytest
import torch

import oracle
import paper_2308_15152_amd as pkg
import synth
from gpu_util import assert_all_finite, device, gate, nan_output, spread_items, to_np

pytestmark = pytest.mark.gpu

COLUMNS = [1, 2, 16, 31, 32, 33, 34, 63, 64, 65, 78, 96, 97, 98]


def _forms(B, pad, offset):
    """B on the device in rows ncols + pad apart from an offset base, and a
    NaN-filled C of the same form with its whole buffer."""
    b, n, c = B.shape
    size = b * n * (c + pad) + offset + 64
    fb = torch.zeros(size, device=device())
    fc = torch.full((size,), float("nan"), device=device())
    cut = slice(offset, offset + b * n * (c + pad))
    Bv = fb[cut].view(b, n, c + pad)[:, :, :c]
    Bv.copy_(B)
    whole = fc[cut].view(b, n, c + pad)
    return Bv, fc, whole


def _untouched(fc, whole, c, offset):
    assert torch.isnan(fc[:offset]).all() and torch.isnan(fc[offset + whole.numel():]).all()
    assert torch.isnan(whole[:, :, c:]).all()


@pytest.mark.parametrize("pad,offset", [(0, 0), (1, 1), (3, 2)])
@pytest.mark.parametrize("ncols", COLUMNS)
def test_columns(ncols, pad, offset):
    print(f"case rule columns {ncols} pad={pad} offset={offset}", flush=True)
    u, B = synth.householder_inputs(9, 64, ncols, seed=200 + ncols)
    c, s, _ = synth.givens_inputs(9, 64, 1, seed=201 + ncols)
    Bv, fc, whole = _forms(B, pad, offset)
    C = whole[:, :, :ncols]
    ref = oracle.householder(u.numpy(), B.numpy())
    for mode in (pkg.HOUSEHOLDER_RULE, pkg.HOUSEHOLDER_LDS):
        fc.fill_(float("nan"))
        pkg.householder_emu_batched(u.to(device()), Bv, C, mode=mode)
        _untouched(fc, whole, ncols, offset)
        gate(to_np(C), ref, 64, f"householder {ncols} columns", max_gate=False)
    for (i, j), modes in (((5, 37), (pkg.GIVENS_MAP, pkg.GIVENS_EMBEDDED, pkg.GIVENS_LDS)),
                          ((62, 17), (pkg.GIVENS_MAP, pkg.GIVENS_LDS))):
        ref = oracle.givens(i, j, c.numpy(), s.numpy(), B.numpy())
        for mode in modes:
            fc.fill_(float("nan"))
            pkg.givens_emu_batched(i, j, c.to(device()), s.to(device()), Bv, C, mode=mode)
            _untouched(fc, whole, ncols, offset)
            gate(to_np(C), ref, 2, f"givens {ncols} columns", max_gate=False)


@pytest.mark.parametrize("mb", [39, 41])
@pytest.mark.parametrize("ncols", [65, 66, 94, 96, 98, 158])
def test_last_groups(ncols, mb):
    """Batches on both sides of the 40 MB up to which 65 to 96 columns are not
    read in pairs: items over the batch, every output written."""
    batch = mb * 10 ** 6 // (512 * ncols)
    print(f"case rule last group {ncols} batch={batch}", flush=True)
    u, B = synth.householder_inputs(batch, 64, ncols, seed=400 + ncols)
    c, s, _ = synth.givens_inputs(batch, 64, 1, seed=401 + ncols)
    Bd, C = B.to(device()), nan_output((batch, 64, ncols))
    items = spread_items(batch, 40)
    it = torch.from_numpy(items).to(device())
    pkg.householder_emu_batched(u.to(device()), Bd, C)
    assert_all_finite(C, f"householder {ncols} columns")
    gate(to_np(C[it]), oracle.householder(u[items].numpy(), B[items].numpy()), 64,
         f"householder {ncols} columns", max_gate=False)
    for i, j in ((5, 37), (62, 17)):
        C.fill_(float("nan"))
        pkg.givens_emu_batched(i, j, c.to(device()), s.to(device()), Bd, C)
        assert_all_finite(C, f"givens {ncols} columns")
        ref = oracle.givens(i, j, c[items].numpy(), s[items].numpy(), B[items].numpy())
        gate(to_np(C[it]), ref, 2, f"givens {ncols} columns", max_gate=False)


@pytest.mark.parametrize("batch", [2929, 2930, 8192, 8193])
def test_streamed_rows(batch):
    """64 columns on both sides of the 96 MB from which and the 256 MiB up to
    which B is read through the caches: all forms give what a padded call, never streamed, gives."""
    print(f"case rule streamed batch={batch}", flush=True)
    u, B = synth.householder_inputs(batch, 64, 64, seed=500)
    c, s, _ = synth.givens_inputs(batch, 64, 1, seed=501)
    ud, cd, sd, Bd = (x.to(device()) for x in (u, c, s, B))
    padded = torch.empty((batch, 64, 65), device=device())[:, :, :64]
    for call in (lambda C: pkg.householder_emu_batched(ud, Bd, C),
                 lambda C: pkg.givens_emu_batched(5, 37, cd, sd, Bd, C),
                 lambda C: pkg.givens_emu_batched(62, 17, cd, sd, Bd, C)):
        C = nan_output((batch, 64, 64))
        call(C)
        call(padded)
        assert torch.equal(C, padded)
    ref = oracle.givens(62, 17, c[-9:].numpy(), s[-9:].numpy(), B[-9:].numpy())
    gate(to_np(C[-9:]), ref, 2, "givens, streamed", max_gate=False)


@pytest.mark.parametrize("ncols", [24, 65, 70])
@pytest.mark.parametrize("ld", [(1 << 22) - 1, 1 << 22, (1 << 22) + 1])
def test_far_rows(ld, ncols):
    """Row pitches on both sides of the 32-bit reach, on B and on C alone, from
    an odd base: one block, pairs and single columns through 64-bit pointers,
    nothing written between the rows."""
    print(f"case rule far rows ld={ld} ncols={ncols}", flush=True)
    u, B = synth.householder_inputs(1, 64, ncols, seed=300)
    c, s, _ = synth.givens_inputs(1, 64, 1, seed=301)
    dev = device()
    far = torch.full((63 * ld + ncols + 2,), float("nan"), device=dev)
    farv = far.as_strided((1, 64, ncols), (0, ld, 1), 1)
    between = (far.as_strided((64,), (ld,), 0), far.as_strided((64,), (ld,), ncols + 1))
    ref = oracle.householder(u.numpy(), B.numpy())
    refg = oracle.givens(3, 60, c.numpy(), s.numpy(), B.numpy())
    near = torch.empty((1, 64, ncols), device=dev)
    pkg.householder_emu_batched(u.to(dev), B.to(dev), farv)
    gate(to_np(farv), ref, 64, "householder, far C", max_gate=False)
    pkg.givens_emu_batched(3, 60, c.to(dev), s.to(dev), B.to(dev), farv)
    gate(to_np(farv), refg, 2, "givens, far C", max_gate=False)
    assert all(bool(torch.isnan(x).all()) for x in between)
    farv.copy_(B)
    pkg.householder_emu_batched(u.to(dev), farv, near)
    gate(to_np(near), ref, 64, "householder, far B", max_gate=False)
    pkg.givens_emu_batched(3, 60, c.to(dev), s.to(dev), farv, near)
    gate(to_np(near), refg, 2, "givens, far B", max_gate=False)
    del far, farv
    torch.cuda.empty_cache()
