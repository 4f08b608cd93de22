"""GPU parity of the ring kernel (mid-size products, the int16-output update
and convolutions) against the CPU oracle, bit for bit: edges of its tiles and
k-tiles, every row alignment (DMA and register staging), k slices that end
inside a k-tile, the conversion at shifts around its two forms, and the shapes
where the automatic plans take it."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads
from gpu_util import describe_mismatch, gpu_gemm, oracle_gemm
from test_gpu_conv import _check as check_conv
from test_gpu_srs import _check as check_srs

RING = {"i8": ("i8_ring_128x128", "i8_ring_64x128"),
        "i16": ("i16_ring_128x128", "i16_ring_64x64")}


def _ig():
    import paper_2302_07594_amd as ig
    return ig


def _kid(name):
    ig = _ig()
    return [ig.igemm_kernel_name(i) for i in range(ig.igemm_num_kernels())].index(name)


def _check(dt, m, n, k, name, split=-1, pad=(0, 0, 0), offsets=(0, 0, 0), seed=1):
    A, B, C = workloads.random_operands(dt, m, n, k, seed=seed, lda=k + pad[0], ldb=n + pad[1],
                                        ldc=n + pad[2])
    _, got = gpu_gemm(A, B, C, m, n, k, kernel=_kid(name), split=split, offsets=offsets)
    want = oracle_gemm(A, B, C, m, n, k)
    assert np.array_equal(got, want), describe_mismatch(got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (64, 128, 128), (65, 129, 129),
                                   (127, 255, 127), (130, 140, 16), (200, 15, 300),
                                   (129, 260, 1000)], ids=lambda s: "x".join(map(str, s)))
def test_ring_edges(dt, shape):
    """One below, at and above the tiles and the k-tiles; rows and columns
    shorter than the 16 bytes of one load; one to four k slices."""
    for name in RING[dt]:
        for split in (1, 2, 4):
            _check(dt, *shape, name, split=split, seed=sum(shape))


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("off", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("pad", [0, 1, 2, 4])
def test_ring_alignments(dt, off, pad):
    """Every address of A and B modulo the dword and leading dimensions that
    are and are not whole dwords: DMA where both allow it, registers else."""
    for name in RING[dt]:
        _check(dt, 140, 200, 332, name, split=2, pad=(pad, pad, 3), offsets=(off, off, 1),
               seed=7 * off + pad)
        _check(dt, 140, 200, 332, name, split=1, pad=(4, pad, 0), offsets=(0, off, 0), seed=5)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
def test_ring_extreme_values(dt):
    """The types' ends over a k range of the launch limit and beyond it
    (slices), where every partial sum is as large as it can be."""
    info = np.iinfo(np.int8 if dt == "i8" else np.int16)
    for k in (32768, 33000):
        for a, b in ((info.min, info.min), (info.min, info.max), (info.max, info.max)):
            A = np.full((40, k), a, dtype=info.dtype)
            B = np.full((k, 72), b, dtype=info.dtype)
            C = np.full((40, 72), -5, dtype=np.int32)
            want = oracle_gemm(A, B, C, 40, 72, k)
            for name in RING[dt]:
                _, got = gpu_gemm(A, B, C, 40, 72, k, kernel=_kid(name))
                assert np.array_equal(got, want), (name, k, a, b)


# Every int16-output form of the kernel that the automatic plan takes (the calls
# name no ring kernel): operand type, m, n, k and padding of A, B and C -> tile
# shape and staging (1: DMA, 0: registers), asserted by test_ring_srs_plans. The
# last two int8 ones have one workgroup per unit at most and more.
SRS_FORMS = {
    ("i8", 451, 532, 300, (0, 0, 3)): ("i8_ring_64x128", 1),
    ("i8", 451, 530, 300, (1, 0, 3)): ("i8_ring_64x128", 0),
    ("i16", 451, 530, 300, (1, 0, 3)): ("i16_ring_64x64", 0),
    ("i8", 4000, 2044, 644, (0, 0, 1)): ("i8_ring_128x128", 1),
    ("i8", 2000, 2001, 901, (0, 0, 2)): ("i8_ring_128x128", 0),
    ("i8", 4001, 2047, 385, (0, 0, 0)): ("i8_ring_128x128", 0),
    ("i16", 2000, 2040, 333, (0, 1, 2)): ("i16_ring_128x128", 0),
}


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_ring_srs_plans(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    csrc = os.path.join(root, "paper_2302_07594_amd", "csrc")
    exe = str(tmp_path / "srs_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(root, "include"), "-I", csrc,
                    os.path.join(csrc, "igemm_plan.cpp"),
                    os.path.join(root, "tests", "srs_plan_driver.cpp"), "-o", exe], check=True)
    for (dt, m, n, k, pad), (name, vec) in SRS_FORMS.items():
        args = (1 if dt == "i8" else 2, m, n, k, k + pad[0], n + pad[1])
        out = subprocess.run([exe] + [str(x) for x in args], check=True, capture_output=True,
                             text=True).stdout.split()
        assert out[:2] == [name, str(vec)], (args, out)
        if m in (2000, 4001) and dt == "i8":
            assert (int(out[2]) <= 256) == (m == 2000)


@pytest.mark.gpu
@pytest.mark.parametrize("form", SRS_FORMS, ids=lambda f: "-".join(map(str, f[:4])))
def test_ring_srs_forms(form):
    """Ragged in every extent, both sides of each conversion form."""
    from test_gpu_srs import _operands
    dt, m, n, k, pad = form
    A, B, C = _operands(dt, m, n, k, seed=m + k, pad=pad)
    for shift, rnd in ((0, False), (9, True), (16, True), (17, False), (31, True)):
        got = check_srs(A, B, C, m, n, k, 0, shift, rnd)
        assert np.array_equal(got[:, n:], C[:, n:])


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("conv", [(0, 0, False), (0, 1, True), (0, 15, True), (0, 16, False),
                                  (0, 16, True), (0, 17, True), (0, 17, False), (0, 24, True),
                                  (0, 31, True), (0, 32, True), (0, 47, False), (100, 9, True),
                                  (256, 5, False)], ids=str)
def test_ring_srs(dt, conv):
    kc, shift, rnd = conv
    m, n, k = 451, 530, 300
    from test_gpu_srs import _operands
    A, B, C = _operands(dt, m, n, k, seed=40 + shift, pad=(1, 0, 3))
    check_srs(A, B, C, m, n, k, kc, shift, rnd)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("end", ["min", "max"])
def test_ring_srs_extremes(dt, end):
    """Constant operands at the types' ends over the conversion's longest
    block (2^14): shifts on both sides of its two forms."""
    from test_gpu_srs import _operands
    m, n, k = 257, 1030, 1 << 14
    v = int(getattr(np.iinfo(np.int8 if dt == "i8" else np.int16), end))
    A, B, C = _operands(dt, m, n, k, seed=3, lo=v, hi=v)
    for shift, rnd in ((0, False), (16, True), (17, True), (28, True), (29, False)):
        check_srs(A, B, C, m, n, k, 0, shift, rnd)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("case", [
    # n, h, w, c, k, r, s, stride, pad, dil
    (9, 57, 55, 16, 96, 3, 3, (1, 1), (1, 1), (1, 1)),
    (7, 41, 37, 48, 91, 3, 3, (2, 1), (2, 0), (2, 3)),
    (3, 30, 30, 64, 255, 5, 3, (1, 2), (2, 1), (1, 1)),
    (40, 28, 28, 32, 260, 1, 1, (1, 1), (0, 0), (1, 1)),
    (2, 14, 14, 512, 130, 3, 3, (1, 1), (1, 1), (1, 1)),
], ids=lambda c: "x".join(map(str, c[:7])))
def test_ring_conv(dt, case):
    n, h, w, c, k, r, s, stride, pad, dil = case
    check_conv(dt, n, h, w, c, k, r, s, stride, pad, dil, seed=n + c)
    # weights at an odd dword: register staging
    check_conv(dt, n, h, w, c, k, r, s, stride, pad, dil, seed=n + k, w_off=1)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("w_off", [0, 1])
@pytest.mark.parametrize("big", [True, False])
def test_ring_conv_forms(dt, w_off, big):
    """Each tile shape and staging (int8 weights at odd bytes, and int16: through
    registers), whole k and in slices (a deep window alone asks for them)."""
    ig = _ig()
    n, h, c, k = (32, 28, 64, 200) if big else (1, 8, 4112, 256)
    es = 1 if dt == "i8" else 2
    d = ig.conv_desc(n, h, h, c, k, 3, 3, (1, 1), (1, 1), (1, 1))
    want = (RING[dt][0 if big else 1], 1 if dt == "i8" and w_off == 0 else 0)
    for split in (-1, 2):
        p = ig.igemm_conv2d_query_plan(es, d, W=0x10000 + es * w_off, num_cu=256, split=split)
        assert (p["kernel_name"], p["vec_a"]) == want
        assert p["split"] == (2 if split == 2 else 1) or (not big and p["split"] > 16)
        check_conv(dt, n, h, h, c, k, 3, 3, (1, 1), (1, 1), (1, 1), seed=n + w_off, split=split,
                   w_off=w_off)


def test_ring_plan_rules():
    """Where the automatic plans take the ring kernel and how they slice it
    (256 units, aligned buffers), and its 32-bit window limits."""
    ig = _ig()

    def plan(es, m, n, k, **kw):
        p = ig.igemm_query_plan(es, m, n, k, num_cu=256, **kw)
        return p["kernel_name"], p["split"], p["vec_a"]
    assert plan(1, 512, 4096, 4096) == ("i8_ring_64x128", 1, 1)
    assert plan(1, 64, 4096, 4096) == ("i8_ring_64x128", 4, 1)
    assert plan(1, 2048, 4096, 4096) == ("i8_ring_128x128", 1, 1)
    assert plan(1, 1000, 3001, 1777)[0].startswith("i8_ring") and \
        plan(1, 1000, 3001, 1777)[2] == 0
    assert plan(1, 64, 64, 64) == ("i8_ring_64x128", 1, 1)
    assert not plan(1, 146, 501, 801)[0].startswith("i8_ring")    # few tiles, odd rows
    assert not plan(1, 32, 300, 300)[0].startswith("i8_ring")     # few rows
    assert plan(2, 1536, 1536, 1536)[0] == "i16_ring_128x128"
    assert plan(2, 777, 1111, 2049)[0].startswith("i16_ring")
    assert plan(2, 201, 201, 6001)[0] == "i16_ring_64x64"
    assert not plan(2, 2000, 3000, 64)[0].startswith("i16_ring")  # one k-tile
    # one k slice per 32768 at least; an explicit count in units of 64
    assert plan(1, 512, 4096, 40000)[1] >= 2
    p = ig.igemm_query_plan(1, 64, 64, 640, split=10)
    assert p["split"] == 10 and p["k_chunk"] == 64
    # a k range of B beyond 2 GiB is staged through registers; rows of A or C
    # beyond it are refused
    kid = _kid("i8_ring_128x128")
    big = 1 << 20
    assert ig.igemm_query_plan(1, 256, 256, 8192, ldb=big, kernel=kid, split=1)["vec_a"] == 0
    for kw in ({"lda": 1 << 25}, {"ldb": 1 << 25}, {"ldc": 1 << 23}):
        with pytest.raises(ig.IgemmError) as e:
            ig.igemm_query_plan(1, 256, 256, 8192, kernel=kid, **kw)
        assert e.value.status == ig.IGEMM_ENOTSUP
    # convolutions: whole 16-byte channel chunks, from 2^27 multiply-adds
    for es, c in ((1, 16), (2, 8)):
        d = ig.conv_desc(32, 56, 56, c, 128, 3, 3, (1, 1), (1, 1), (1, 1))
        assert "ring" in ig.igemm_conv2d_query_plan(es, d)["kernel_name"]
        d = ig.conv_desc(32, 56, 56, c + 1, 128, 3, 3, (1, 1), (1, 1), (1, 1))
        assert "ring" not in ig.igemm_conv2d_query_plan(es, d)["kernel_name"]


def test_conv_slice_counts_refused():
    """A slice count that is neither -1 nor at least 1 is refused, whichever
    kernel the automatic plan takes: the ring kernel (64 channels, batch 32),
    a fused one (63 channels) or the small-output kernel (batch 1)."""
    ig = _ig()
    for es in (1, 2):
        for n, c in ((32, 64), (32, 63), (1, 64)):
            d = ig.conv_desc(n, 14, 14, c, 256, 3, 3, (1, 1), (1, 1), (1, 1))
            for split in (-1, 1, 3):
                assert ig.igemm_conv2d_query_plan(es, d, split=split)["grid"] > 0
            for split in (0, -2, -5):
                with pytest.raises(ig.IgemmError) as e:
                    ig.igemm_conv2d_query_plan(es, d, split=split)
                assert e.value.status == ig.IGEMM_EINVAL, (es, n, c, split)


@pytest.mark.parametrize("es,m,n,k", [(1, 1200000000, 1, 1), (1, 1200000000, 3, 5),
                                      (1, 1, 1200000000, 1), (1, 1100000000, 1, 3),
                                      (1, 300, 1100000000, 300), (2, 1100000000, 100, 300)])
def test_plans_fit_one_dispatch(es, m, n, k):
    """Work-items of one launch (workgroups times the plan's own threads) are
    counted in 32 bits: products of a billion rows or columns, whose ring
    forms of 512 threads would exceed that, keep a kernel that fits."""
    ig = _ig()
    for base in (0x10000, 0x10001 if es == 1 else 0x10002):
        p = ig.igemm_query_plan(es, m, n, k, base, k, base, n, base, n, num_cu=256)
        assert p["grid"] * p["threads"] < 1 << 32, p
    for name in RING["i8" if es == 1 else "i16"]:
        try:
            p = ig.igemm_query_plan(es, m, n, k, num_cu=256, kernel=_kid(name))
        except ig.IgemmError as e:
            assert e.status == ig.IGEMM_ENOTSUP
            continue
        assert p["grid"] * p["threads"] < 1 << 32, p


def test_ring_slices_over_long_k():
    """Long k over few tiles is sliced until the compute units are busy; tall
    products of a few columns, whose atomic adds cost as much as 16 columns',
    are not sliced beyond what they save."""
    ig = _ig()
    for es in (1, 2):
        for m, n, k in ((64, 64, 262144), (128, 128, 262144)):
            p = ig.igemm_query_plan(es, m, n, k, num_cu=256)
            assert "ring" in p["kernel_name"] and p["grid"] >= 128, (es, m, n, k, p["grid"])
            assert p["split"] * p["k_chunk"] >= k and p["k_chunk"] <= 32768
        for m, n, k in ((100000, 1, 1024), (100000, 1, 256)):
            p = ig.igemm_query_plan(es, m, n, k, num_cu=256)
            assert "ring" in p["kernel_name"] and p["split"] == 1, (es, m, n, k, p["split"])


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
def test_ring_many_slices(dt):
    """The automatic plan's slices of a long k (more than 16, the last one
    shorter) against the oracle."""
    m, n, k = 65, 68, 20004
    p = _ig().igemm_query_plan(1 if dt == "i8" else 2, m, n, k, num_cu=256)
    assert "ring" in p["kernel_name"] and p["split"] > 16
    A, B, C = workloads.random_operands(dt, m, n, k, seed=9)
    _, got = gpu_gemm(A, B, C, m, n, k)
    want = oracle_gemm(A, B, C, m, n, k)
    assert np.array_equal(got, want), describe_mismatch(got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["i8", "i16"])
@pytest.mark.parametrize("r", range(1, 17))
def test_ring_short_edges(dt, r):
    """A last column tile and a last k-tile of 1 to 16 elements (their rows are
    read in one or two pieces), and outputs and k ranges that short."""
    for m, n, k, ld in ((70, 128 + r, 128 + r, 1), (5, r, 300, 0), (66, 130, r, 1)):
        for name in RING[dt]:
            _check(dt, m, n, k, name, split=1, pad=(ld, ld, 2), offsets=(1, 1, 0), seed=r)


@pytest.mark.gpu
@pytest.mark.parametrize("k,kc", [(374, 290), (84, 0), (128, 0), (200, 0)])
def test_ring_edge_tiles_row_by_row(k, kc):
    """Every k row of the edge tiles (rows at odd addresses, more workgroups than
    units): with A one at p alone, the int16 output is row p of B."""
    import torch
    ig = _ig()
    m, n = 2420, 965
    rng = np.random.default_rng(k)
    B = torch.from_numpy(rng.integers(-128, 128, size=(k, 967), dtype=np.int8)).cuda()[:, 2:]
    A = torch.zeros(m, k + 5, dtype=torch.int8, device="cuda")
    C = torch.zeros(m, n, dtype=torch.int16, device="cuda")
    for p in range(k):
        A.zero_()
        A[:, 1 + p] = 1
        C.zero_()
        ig.gemm_srs(A[:, 1:1 + k], B, C, kc=kc)
        assert torch.equal(C, B[p].to(torch.int16).expand(m, n)), p
