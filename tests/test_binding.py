"""The native calling side of pb.py against its Python functions: unusual and wrong arguments."""
import os
import shutil
import subprocess
import sys
import textwrap

import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pb():
    from paper_2003_00822_amd import pb as _pb
    _pb.lib()
    return _pb


def test_arguments_that_are_no_gpu_tensors(pb):
    d = pb.pb_desc_init(8, 64, 3)
    t = torch.zeros(64)
    with pytest.raises(TypeError, match="packed must be a CUDA/HIP tensor"):
        pb.pb_unpack(t, d, t)
    with pytest.raises(TypeError, match="X must be a CUDA/HIP tensor"):
        pb.pb_act_prep(d, [1.0], 1, t, stream=0)
    with pytest.raises(TypeError):
        pb.pb_unpack(t, d)                       # an argument missing
    with pytest.raises(TypeError):
        pb.pb_unpack(t, d, t, None, 5)           # one too many


def test_the_library_serves_without_the_extension(tmp_path):
    """A package without `_binding.so` answers size queries and argument errors; the extension is taken up if it is built
    between the import and the first use, and left alone if it is built for another torch."""
    from paper_2003_00822_amd import build
    src = os.path.dirname(build.LIB)
    pkg = tmp_path / "paper_2003_00822_amd"
    pkg.mkdir()
    for f in os.listdir(src):
        if f.endswith(".py"):
            shutil.copy(os.path.join(src, f), pkg)
    os.symlink(build.LIB, pkg / "libpbatch.so")
    code = """
        import os, sys, warnings
        import torch
        what, ext = sys.argv[1:]
        if what == "other torch":
            os.symlink(ext, "paper_2003_00822_amd/_binding.so")
            torch.__version__ = "0.0.1"
        from paper_2003_00822_amd import pb
        assert os.path.realpath(pb.__file__).startswith(os.getcwd())
        if what == "built later":
            os.symlink(ext, "paper_2003_00822_amd/_binding.so")
        with warnings.catch_warnings(record=True) as w:
            warnings.simplefilter("always")
            assert pb.pb_packed_bytes(pb.pb_desc_init(4096, 4096, 8)) == 4096 * 4096
        native = what == "built later"
        assert isinstance(pb.pb_matmul, type(len)) == native, pb.pb_matmul
        assert [x.category for x in w] == ([] if native else [RuntimeWarning])
        try:
            pb.pb_unpack(torch.zeros(4), pb.pb_desc_init(8, 64, 3), torch.zeros(4))
            raise SystemExit("not refused")
        except TypeError as e:
            assert "packed must be a CUDA/HIP tensor" in str(e)
    """
    env = {k: v for k, v in os.environ.items() if k != "PBATCH_LIB"}
    for what in ("missing", "other torch", "built later"):
        ext = pkg / "_binding.so"
        if ext.is_symlink():
            ext.unlink()
        subprocess.run([sys.executable, "-c", textwrap.dedent(code), what, build.BINDING_LIB], check=True, cwd=tmp_path,
                       env=env, timeout=300)


@pytest.mark.gpu
def test_native_and_python_calls_agree(pb):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = torch.randn((50, 300), device="cuda", generator=g)
    X = torch.randn((6, 300), device="cuda", generator=g)
    lin = pb.PackedLinear(W, 5, max_batch=6)
    Y = lin(X)
    want = torch.empty_like(Y)
    # keywords and an explicit stream take the Python function
    pb.pb_matmul(packed=lin.packed, scales=lin.scales, d=lin.desc, bits_used=5, X=X, batch=6, Y=want, workspace=lin.workspace,
                 stream=torch.cuda.current_stream())
    assert torch.equal(Y, want)
    out = torch.empty_like(Y)
    assert lin(X, 5, out) is out and torch.equal(out, Y)
    assert torch.equal(lin(X.reshape(2, 3, 300)), Y) and torch.equal(lin(X[0]), lin(X[:1]))
    assert torch.equal(lin(X, bits_used=3), lin(X, np.int64(3)))
    assert torch.equal(lin(X.t().contiguous().t().clone(memory_format=torch.contiguous_format)), Y)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = lin(X)
    side.synchronize()
    assert torch.equal(on_side, Y)
    with pytest.raises(AssertionError):
        lin(torch.zeros((7, 300), device="cuda"))
    with pytest.raises(ValueError, match="X must be contiguous"):
        pb.pb_matmul(lin.packed, lin.scales, lin.desc, 5, X.t(), 6, Y, lin.workspace)
    with pytest.raises(TypeError, match="Y must have dtype"):
        pb.pb_matmul(lin.packed, lin.scales, lin.desc, 5, X, 6, Y.double(), lin.workspace)
    with pytest.raises(pb.PbError) as e:
        pb.pb_matmul(lin.packed, lin.scales, lin.desc, 6, X, 6, Y, lin.workspace)
    assert e.value.status == pb.PB_EINVAL
    with pytest.raises(pb.PbError):
        lin(X, bits_used=6)
    with pytest.raises(pb.PbError) as e:
        pb.pb_matmul(lin.packed, None, lin.desc, 5, X, 6, Y, lin.workspace)
    assert e.value.status == pb.PB_EINVAL
    torch.cuda.synchronize()


def test_python_functions_have_the_parameters_of_the_header(pb):
    """Names and order, and the argument types that ctypes converts to."""
    import ctypes
    import inspect
    import re
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(root, "include", "pb.h")).read(), flags=re.S)
    assert len(pb._NATIVE) == 13
    for name in pb._NATIVE:
        args = [re.sub(r"\s+", " ", a).strip() for a in re.search(r"\bint %s\(([^)]*)\)" % name, text).group(1).split(",")]
        names = [re.search(r"(\w+)$", a).group(1) for a in args]
        assert list(inspect.signature(pb._PYTHON[name]).parameters) == names, name
        want = [ctypes.POINTER(pb.pb_desc) if "pb_desc *" in a else ctypes.c_void_p if "*" in a else ctypes.c_int for a in args]
        assert getattr(pb.lib(), name).argtypes == want, name


@pytest.mark.gpu
def test_every_entry_point_by_keywords(pb):
    """Keywords and an explicit stream go to the Python functions: the same results as the native calls, all thirteen."""
    import inspect
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    H, I, N, bits, m = 12, 88, 3, 5, 4
    R, C = 4 * H, I + H
    normal = lambda *shape: torch.randn(shape, device="cuda", generator=g)   # noqa: E731
    W, X, bias, h, c = normal(R, C), normal(N, C), normal(R), normal(N, H), normal(N, H)
    W3 = normal(R, 2)
    d, d2 = pb.pb_desc_init(R, C, bits), pb.pb_desc_init(R, 2, 2)
    rows = pb.pb_desc_init_layout(R, C, bits, pb.PB_LAYOUT_ROWMAJOR_V1)
    lin, lin_rows = pb.PackedLinear(W, bits, max_batch=N), pb.PackedLinear(W, bits, max_batch=N, layout=rows.layout)
    prepared = pb.alloc_workspace(rows, N)
    pb.pb_act_prep(rows, X, N, prepared)
    p, s = lin.packed, lin.scales

    def zeros(*shape, dtype=torch.float32):
        return lambda: torch.zeros(shape, dtype=dtype, device="cuda")

    def nbytes(n):
        return zeros(n, dtype=torch.uint8)

    work, codes = nbytes(lin.workspace.numel()), nbytes(p.numel())
    # a callable makes a fresh buffer; the workspace (last but for pb_act_prep) is not a result
    calls = {
        "pb_quantize_pack": [W, R, C, bits, codes, zeros(bits)],
        "pb_quantize_pack_desc": [W, d, codes, zeros(bits)],
        "pb_quantize_pack_mode": [W3, d2, pb.PB_QUANT_SIGN, nbytes(pb.pb_packed_bytes(d2)), zeros(2)],
        "pb_unpack": [p, d, zeros(R, C, dtype=torch.int32)],
        "pb_matmul": [p, s, d, m, X, N, zeros(N, R), work],
        "pb_matmul_static": [p, s, d, m, X, N, zeros(N, R)],
        "pb_matmul_bias_act": [p, s, d, m, X, N, bias, pb.PB_ACT_RELU, zeros(N, R), work],
        "pb_matmul_acc": [p, d, m, X, N, zeros(m, N, R, dtype=torch.int64), work],
        "pb_matmul_acc_pairs": [p, d, m, X, N, zeros(m // 2, N, R, dtype=torch.int64), work],
        "pb_act_prep": [rows, X, N, nbytes(prepared.numel())],
        "pb_matmul_prepared": [lin_rows.packed, lin_rows.scales, rows, m, N, zeros(N, R), prepared],
        "pb_fixed_point": [rows, X, N, zeros(N, C, dtype=torch.int32), work],
        "pb_lstm_cell": [p, s, d, m, X[:, :I].contiguous(), I, h, c, bias, zeros(N, H), zeros(N, H), N, work],
    }
    assert sorted(calls) == sorted(pb._NATIVE)
    side = torch.cuda.Stream()
    for name, args in calls.items():
        print(name, flush=True)
        made = [i for i, a in enumerate(args) if callable(a)]
        keep = [i for i in made if args[i] is not work]
        names = list(inspect.signature(pb._PYTHON[name]).parameters)
        native = [a() if callable(a) else a for a in args]
        getattr(pb, name)(*native)
        side.wait_stream(torch.cuda.current_stream())
        for stream in (torch.cuda.current_stream(), side, side.cuda_stream):
            with torch.cuda.stream(side):
                byname = [a() if callable(a) else a for a in args]
            side.synchronize()
            getattr(pb, name)(stream=stream, **dict(zip(names, byname)))
            torch.cuda.synchronize()
            for i in keep:
                assert native[i].view(torch.uint8).any(), (name, names[i])
                assert torch.equal(native[i], byname[i]), (name, names[i])


@pytest.mark.gpu
def test_computed_attributes_stay_alive(pb):
    """A layer whose tensors are made on access: none of them may share memory with the output."""
    class Computed(pb.PackedLinear):
        pass

    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    W = torch.randn((50, 300), device="cuda", generator=g)
    X = torch.randn((1, 300), device="cuda", generator=g)
    want = pb.PackedLinear(W, 5)(X)
    lin = Computed(W, 5)
    packed, scales, used = lin.packed, lin.scales, []

    def fresh(t):
        t = t.clone()
        used.append(t.data_ptr())
        return t

    Computed.packed = property(lambda self: fresh(packed))
    Computed.scales = property(lambda self: fresh(scales))
    Y = lin(X)
    assert len(used) == 2 and Y.data_ptr() not in used
    assert torch.equal(Y, want)
