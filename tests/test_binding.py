"""The tensor calls' native path against their Python path, over the forms of
arguments that either takes: the same result, or the same exception. (The
Python path is reached with workspace="torch" or an explicit stream, which mean
the same as the defaults.)"""
import numpy as np
import pytest

import workloads


def _ig():
    import paper_2302_07594_amd as ig
    return ig


def test_native_path_leaves_other_arguments_to_python():
    """Without a GPU no tensor is a CUDA tensor: every native function
    declines, and the calls raise what their Python checks raise."""
    import torch
    ig = _ig()
    native = ig._load_native()
    a = torch.zeros(4, 4, dtype=torch.int16)
    c = torch.zeros(4, 4, dtype=torch.int32)
    x = torch.zeros(1, 4, 4, 4, dtype=torch.int16)
    y = torch.zeros(1, 4, 4, 4, dtype=torch.int32)
    assert native.gemm(2, a, a, c, -1, -1) is None
    assert native.gemm(2, None, 3, "c", -1, -1) is None
    assert native.gemm(2, a, a) is None
    assert native.srs(a, a, a, 0, 0, False, -1) is None
    assert native.srs(a, a, a, 1 << 70, 0, False, -1) is None
    assert native.packed_b(2, a, a, 0, 4, 4, c, -1) is None
    assert native.conv2d(x, x, y, (1, 1), (0, 0), (1, 1), -1, -1) is None
    assert native.conv2d(x, x, y, [1, 1], 0, (1, 1), -1, -1) is None
    with pytest.raises(ValueError):
        ig.gemm_i16(a, a, c)
    with pytest.raises(TypeError):
        ig.gemm_i8(a, a, c)
    with pytest.raises(TypeError):
        ig.gemm_srs(a, a, c)
    with pytest.raises(ValueError):
        ig.conv2d(x, x, y)


def _forms(torch):
    """name -> (A, B, C), int16, on the GPU; some of them invalid."""
    rng = np.random.default_rng(5)

    def mk(shape, dt=np.int16):
        return torch.from_numpy(rng.integers(-30000, 30000, size=shape).astype(dt)).cuda()
    m, n, k = 70, 90, 130
    wide = mk((m, 200))
    return {
        "plain": (mk((m, k)), mk((k, n)), mk((m, n), np.int32)),
        "row views": (wide[:, 3:3 + k], mk((k, 101))[:, :n], mk((m, 99), np.int32)[:, 4:4 + n]),
        "one row": (mk((1, k)), mk((k, n)), mk((1, n), np.int32)),
        "one column": (mk((m, k)), mk((k, 7))[:, 2:3], mk((m, 5), np.int32)[:, 1:2]),
        "k = 1": (mk((m, 9))[:, 4:5], mk((1, n)), mk((m, n), np.int32)),
        "expanded rows": (mk((1, k)).expand(m, k), mk((k, n)), mk((m, n), np.int32)),
        "transposed A": (mk((k, m)).t(), mk((k, n)), mk((m, n), np.int32)),
        "transposed C": (mk((m, k)), mk((k, n)), mk((n, m), np.int32).t()),
        "empty k": (mk((m, 0)), mk((0, n)), mk((m, n), np.int32)),
        "empty m": (mk((0, k)), mk((k, n)), mk((0, n), np.int32)),
        "shape mismatch": (mk((m, k)), mk((k + 1, n)), mk((m, n), np.int32)),
        "wrong C type": (mk((m, k)), mk((k, n)), mk((m, n))),
        "C on the host": (mk((m, k)), mk((k, n)), mk((m, n), np.int32).cpu()),
        "3-D A": (mk((1, m, k)), mk((k, n)), mk((m, n), np.int32)),
        "parameter": (torch.nn.Parameter(mk((m, k)), requires_grad=False), mk((k, n)),
                      mk((m, n), np.int32)),
    }


@pytest.mark.gpu
def test_native_and_python_paths_agree():
    import torch
    ig = _ig()

    def outcome(fn, c):
        before = c.clone()
        try:
            fn(c)
        except Exception as e:  # the same type and text on both paths
            assert torch.equal(c, before)
            return type(e), str(e)
        torch.cuda.synchronize()
        return c.cpu().numpy().copy()

    for name, (a, b, c0) in _forms(torch).items():
        def c_like():  # the same form of C with the same contents
            c = torch.empty_strided(c0.shape, c0.stride(), dtype=c0.dtype, device=c0.device)
            return c.copy_(c0)
        for kw in ({}, {"split": 2}, {"kernel": 10 ** 6}):
            got = outcome(lambda c: ig.gemm_i16(a, b, c, **kw), c_like())
            want = outcome(lambda c: ig.gemm_i16(a, b, c, workspace="torch", **kw), c_like())
            assert (got == want) if isinstance(want, tuple) else np.array_equal(got, want), name
        if c0.dtype == torch.int32 and c0.dim() == 2:
            s16 = torch.empty_strided(c0.shape, c0.stride(), dtype=torch.int16, device=c0.device)
            s16.copy_(c0)
            for kw in ({"shift": 5, "round_half_up": True}, {"kc": 64}, {"shift": 99}):
                got = outcome(lambda c: ig.gemm_srs(a, b, c, **kw), s16.clone())
                want = outcome(lambda c: ig.gemm_srs(a, b, c, workspace="torch", **kw),
                               s16.clone())
                assert (got == want) if isinstance(want, tuple) else np.array_equal(got, want), name


@pytest.mark.gpu
@pytest.mark.parametrize("op", ["gemm", "srs"])
def test_native_path_streams_and_workspaces(op):
    """The current stream is the one a call runs on, and a product that packs
    takes its workspace from the allocator, on that stream, eagerly and under
    capture: memory that later work on the stream overwrites must not be in
    use still."""
    import torch
    ig = _ig()
    m, n, k = 2048, 2048, 1536
    A, B, C = workloads.random_operands("i16", m, n, k, seed=8)
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    if op == "gemm":
        need = ig.igemm_query_plan(2, m, n, k, Ad, k, Bd, n, None, n, ncu)["workspace_bytes"]
        C0, call = torch.from_numpy(C).cuda(), ig.gemm_i16
    else:
        C0 = torch.from_numpy(C.astype(np.int16)).cuda()
        need = ig.igemm_srs_query(2, m, n, k, Ad, k, Bd, n, C0, n, 512, ncu)

        def call(a, b, c, **kw):
            return ig.gemm_srs(a, b, c, kc=512, shift=9, round_half_up=True, **kw)
    assert need > 0
    native = ig._load_native()
    c = C0.clone()
    assert (native.gemm(2, Ad, Bd, c, -1, -1) if op == "gemm" else
            native.srs(Ad, Bd, c, 512, 9, True, -1)) == ig.IGEMM_OK   # not left to Python
    want = call(Ad, Bd, C0.clone(), workspace="torch")
    assert torch.equal(c, want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        c = C0.clone()
        for _ in range(3):
            call(Ad, Bd, c)
            torch.full((need // 4 + 4096,), -1, dtype=torch.int32, device="cuda")
    side.synchronize()
    thrice = C0.clone()
    for _ in range(3):
        call(Ad, Bd, thrice, workspace="torch")
    assert torch.equal(c, thrice)
    c = C0.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(Ad, Bd, c)
        torch.full((need // 4 + 4096,), -1, dtype=torch.int32, device="cuda")
    for _ in range(3):
        c.copy_(C0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, want)
        assert torch.equal(call(Ad, Bd, C0.clone()), want)   # eager work between replays


@pytest.mark.gpu
def test_native_path_packed_b_and_transforms():
    """gemm_packed_b gives what the one-call product gives; a batched tensor is
    not taken for a plain one."""
    import torch
    ig = _ig()
    m, n, k = 1100, 1100, 2000
    A, B, C = workloads.random_operands("i16", m, n, k, seed=8)
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    C0 = torch.from_numpy(C).cuda()
    want = ig.gemm_i16(Ad, Bd, C0.clone(), workspace="torch")
    pb = ig.pack_b(Bd)
    assert torch.equal(ig.gemm_packed_b(Ad, pb, C0.clone()), want)
    with pytest.raises(Exception):
        torch.func.vmap(lambda a: ig.gemm_i16(a, Bd, C0.clone()))(Ad[None])


def test_library_builds_without_torch(monkeypatch, tmp_path):
    """The C library needs no torch: without it (or without its headers) the
    binding is left out instead of failing a build whose library is done, and
    a binding counts as current only for the torch it was built against."""
    from paper_2302_07594_amd import build
    lib, binding, stamp = (tmp_path / n for n in ("lib.so", "binding.so", "stamp"))
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "BINDING", str(binding))
    monkeypatch.setattr(build, "STAMP", str(stamp))
    lib.write_bytes(b"")
    binding.write_bytes(b"")
    stamp.write_text(build.source_hash() + "\n")
    assert build.is_current()
    monkeypatch.setattr(build, "torch_version", lambda: "0.0.1")   # another torch
    assert not build.is_current()
    monkeypatch.undo()
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "BINDING", str(binding))
    monkeypatch.setattr(build, "STAMP", str(stamp))
    binding.unlink()
    assert not build.is_current()
    monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    assert not build.is_current()                  # built for a torch that is gone
    build._build_binding(False)                    # nothing to build, no error
    assert not binding.exists()
    stamp.write_text(build.source_hash() + "\n")
    assert build.is_current()
