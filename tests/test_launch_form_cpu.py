"""What a call launches, as the host-only queries report it (no GPU: the
addresses are never read): the tile kernel and its form where an automatic
call takes it, the named kernel for a named policy, and one translation unit
per kernel name."""
import ctypes
import pathlib
import re

import pytest

import bench
import paper_2308_15152_amd as pkg

ROOT = pathlib.Path(__file__).resolve().parents[1]
PA, PB, PC, PD = (i << 44 for i in (1, 2, 3, 4))
AUTO, REG = pkg.Policy(), pkg.Policy(pkg.FLOW_REG, 1, pkg.TILE_64x64)


def gemm_form(m, n, k, batch=1, policy=None, lda=None, ldb=None, ldc=None, offset=0):
    """(status, kernel, form) of a packed product (or with the given row
    pitches), its bases `offset` floats off alignment."""
    lda, ldb, ldc = lda or k, ldb or n, ldc or n
    kern, form = ctypes.c_char_p(), (ctypes.c_int * 3)()
    rc = pkg.load().sgemm_emu_launch_form(
        m, n, k, PA + 4 * offset, lda, PB + 4 * offset, ldb, PC + 4 * offset, ldc, batch,
        pkg.Stride(m * lda, k * ldb, m * ldc), None if policy is None else ctypes.byref(policy),
        ctypes.byref(kern), form)
    return rc, (kern.value or b"").decode(), tuple(form)


def acc_form(m, n, k, batch=1, ta=0, tb=0, col=0, c=True, shape=pkg.SHAPE_32x32x16, ec=1, pad=0,
             offset=0):
    lda, ldb, ldd = (max(x, 1) + pad for x in (m if ta else k, k if tb else n, m if col else n))
    st = pkg.Stride4(lda * (k if ta else m), ldb * (n if tb else k), ldd * (n if col else m),
                     ldd * (n if col else m))
    kern, form = ctypes.c_char_p(), (ctypes.c_int * 3)()
    o = 4 * offset
    rc = pkg.load().sgemm_emu_acc_launch_form(
        ta, tb, col, m, n, k, PA + o, lda, PB + o, ldb,
        None if not c else PD + o if c == "D" else PC + o, ldd, PD + o, ldd,
        batch, st, shape, ec, ctypes.byref(kern), form)
    return rc, (kern.value or b"").decode(), tuple(form)


def test_automatic_and_named_products():
    assert gemm_form(1100, 1500, 2000) == (0, "gemm_tile_kernel", (128, 64, 2))
    assert gemm_form(1100, 1500, 2000, policy=AUTO)[1] == "gemm_tile_kernel"
    assert gemm_form(1100, 1500, 2000, policy=REG) == (0, "bgemm_reg_kernel", (64, 64, 1))
    assert gemm_form(8192, 8192, 8192) == (0, "bgemm_big_kernel", (128, 256, 1))
    assert gemm_form(256, 256, 256, 1024) == (0, "bgemm_big_stream_kernel", (256, 128, 1))
    assert gemm_form(0, 4, 4) == (0, "", (0, 0, 0))
    assert gemm_form(-1, 4, 4)[0] == -1
    for m, n, k, batch in ((8192, 8192, 8192, 1), (1100, 1500, 2000, 1), (16, 16, 16, 9)):
        named = pkg.Policy(pkg.FLOW_SPLIT, 1, pkg.TILE_128x128)
        out, kern = pkg.Policy(), ctypes.c_char_p()
        st = pkg.Stride(m * k, k * n, m * n)
        assert pkg.load().sgemm_emu_resolve_policy(m, n, k, PA, k, PB, n, PC, n, batch, st,
                                                   ctypes.byref(named), ctypes.byref(out),
                                                   ctypes.byref(kern)) == 0
        assert gemm_form(m, n, k, batch, policy=named)[1] == kern.value.decode()


def test_accumulate():
    assert acc_form(4096, 4096, 4096, tb=1) == (0, "gemm_tile_kernel", (128, 256, 1))
    assert acc_form(512, 32, 256, batch=500, ta=1) == (0, "gemm_acc_kernel", (64, 64, 1))
    assert acc_form(128, 128, 128, shape=pkg.SHAPE_16x16x32) == (0, "gemm_acc_kernel",
                                                                 (32, 32, 1))
    assert acc_form(128, 128, 128, ec=0)[1] == "gemm_acc_kernel"
    assert acc_form(128, 128, 0)[1] == "gemm_acc_kernel"
    assert acc_form(0, 4, 4) == (0, "", (0, 0, 0))
    assert acc_form(4, 4, 4, ta=2)[0] == -8


@pytest.mark.parametrize("name", sorted(bench.KERNEL_SOURCES))
def test_one_translation_unit_per_kernel(name):
    """A kernel's name stands for the code of one translation unit, the one
    whose hash its counter runs are filed under."""
    csrc = ROOT / "paper_2308_15152_amd" / "csrc"
    named = {f.name for f in csrc.glob("*.hip")
             if re.search(rf"\b{name}\s*\(", re.sub(r"//[^\n]*", "", f.read_text()))
             and "__global__" in f.read_text()}
    macros = {f.name for f in csrc.glob("*.hip")
              if re.search(rf"KERNEL\w*\(\s*{name}\s*\)", f.read_text())}
    assert named | macros == {bench.KERNEL_SOURCES[name]}, (name, named, macros)


def test_items_of_more_tiles_than_a_launch_holds():
    """A launch holds 2^31 / 256 - 1 = 8,388,607 workgroups of 256 threads.  An
    item of more 64 x 64 tiles (narrow matrices take no other) goes to the
    kernels that split it over launches or walk it, as does one of 2^30 rows."""
    last = 64 * 8388607
    for k in (4, 20):
        assert acc_form(last, 4, k)[:2] == (0, "gemm_tile_kernel")
        assert acc_form(last + 1, 4, k)[:2] == (0, "gemm_acc_kernel")
        assert acc_form(4, last, k, ta=1, tb=1, col=1)[:2] == (0, "gemm_tile_kernel")
        assert acc_form(4, last + 1, k, ta=1, tb=1, col=1)[:2] == (0, "gemm_acc_kernel")
    assert gemm_form(last, 4, 5)[:2] == (0, "gemm_tile_kernel")
    assert gemm_form(last + 1, 4, 5)[:2] == (0, "bgemm_emu_kernel")
    assert gemm_form((1 << 30) + 8, 4, 5)[:2] == (0, "bgemm_emu_kernel")
    # wide enough for 128 x 64 tiles, the same rows are fewer tiles
    assert acc_form(last + 1, 64, 4) == (0, "gemm_tile_kernel", (128, 64, 1))


def test_far_rows():
    """Large products of nearly whole tiles keep the 128 x 256 tile however far
    apart C's rows are; operand rows past its 32-bit offsets leave it."""
    shape = (4100, 4300, 2060)
    for ldc in (4300, (1 << 22) - 260, 1 << 22, (1 << 23) + 4, 1 << 30):
        assert gemm_form(*shape, ldc=ldc) == (0, "gemm_tile_kernel", (128, 256, 1)), ldc
    assert gemm_form(*shape, ldb=(1 << 24) - 16)[1] == "gemm_tile_kernel"
    assert gemm_form(*shape, ldb=1 << 24) == (0, "bgemm_reg_kernel", (64, 64, 1))
    assert gemm_form(*shape, ldb=1 << 24, ldc=1 << 23) == (0, "bgemm_reg_kernel", (64, 64, 1))
    # other products with far rows go to the kernels with 64-bit addresses
    assert gemm_form(300, 300, 400, ldc=1 << 23)[1] == "bgemm_reg_kernel"
    assert gemm_form(300, 300, 401, ldc=1 << 23)[1] == "bgemm_emu_kernel"


@pytest.mark.parametrize("m,n,k,batch,apart,in_place", [
    (128, 128, 128, 2304, 0, 1), (128, 128, 128, 2303, 0, 0),   # 9216 tiles of 64 x 64
    (192, 192, 256, 1024, 1, 1), (192, 192, 256, 1023, 0, 0), (192, 192, 257, 1400, 0, 0),
    (192, 224, 128, 1400, 0, 0), (224, 192, 128, 1400, 0, 0), (192, 128, 128, 2100, 1, 1),
    (160, 160, 100, 8000, 0, 0), (224, 96, 128, 1536, 1, 1), (224, 96, 128, 1535, 0, 0),
    (4000, 64, 48, 200, 1, 1), (4000, 64, 47, 200, 0, 0), (95, 64, 100, 8000, 0, 0),
    (96, 64, 100, 8000, 1, 1), (128, 80, 100, 8000, 0, 0)])
def test_accumulate_route_of_transposed_batches(m, n, k, batch, apart, in_place):
    """Large batches of small A^T B products stay on the kernel written with
    the fragment interface, by sizes, by the alignment of D and by whether C is
    D; with B transposed or column-major D they don't."""
    name = ("gemm_tile_kernel", "gemm_acc_kernel")
    assert acc_form(m, n, k, batch, ta=1)[1] == name[apart]
    assert acc_form(m, n, k, batch, ta=1, c=False)[1] == name[apart]
    assert acc_form(m, n, k, batch, ta=1, c="D")[1] == name[in_place]
    for kw in ({"tb": 1}, {"col": 1}, {"pad": 4}, {"offset": 1}):
        assert acc_form(m, n, k, batch, ta=1, c="D", **kw)[1] == "gemm_tile_kernel"
    assert acc_form(m, n, k, batch, c="D")[1] == "gemm_tile_kernel"


@pytest.mark.parametrize("m,n,k,batch,register_flow", [
    (116, 116, 128, 384, True), (116, 116, 128, 383, False),      # 1536 tiles of 64 x 64
    (116, 116, 316, 1000, True), (116, 116, 320, 1000, False), (110, 1024, 316, 100, True),
    (64, 1024, 100, 100, False), (128, 1024, 100, 100, False), (1024, 104, 124, 100, True),
    (2025, 2300, 124, 11, True), (2025, 2300, 128, 11, False), (2025, 2304, 64, 11, False),
    (1000, 300, 88, 186, True), (1000, 300, 88, 187, False), (1000, 302, 88, 40, False),
    (1000, 301, 88, 40, False)])
def test_short_products_left_to_the_register_flow(m, n, k, batch, register_flow):
    """Ragged products of short k that fill the device, with 16-byte rows of B,
    by sizes and by the alignment of C's rows."""
    expect = "bgemm_reg_kernel" if register_flow else "gemm_tile_kernel"
    assert gemm_form(m, n, k, batch)[1] == expect
    if register_flow:
        assert gemm_form(m, n, k, batch) == (0, expect, (128, 128, 1))
        # unaligned operands go to the tile kernel
        assert gemm_form(m, n, k, batch, offset=1)[1] == "gemm_tile_kernel"
