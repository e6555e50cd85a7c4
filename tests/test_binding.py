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
