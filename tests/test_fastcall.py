"""The native call path of the Python binding: it takes plain GPU tensors and
integers only, declines everything else, and gives what the ctypes path gives."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2609_16389_amd import _fastcall
from paper_2609_16389_amd import xgemm as xg


def test_declines_what_is_not_plain():
    a = torch.zeros(8, 8, dtype=torch.bfloat16)
    c = torch.zeros(8, 8)
    assert _fastcall.gemm(a, a, c) is None                    # not on a GPU
    assert _fastcall.gemm(a, a, None) is None
    assert _fastcall.bmm(a, a, c) is None and _fastcall.gemv(c, c, c) is None
    assert _fastcall.run(None, 1, 1, 1, None, 1, None, 1, None, 1, 0, 2 ** 80) is None
    assert _fastcall.run(None, 1.0, 1, 1, None, 1, None, 1, None, 1, 0, None) is None
    assert _fastcall.run(None, 1, 1) is None
    # plain integers reach the library
    assert _fastcall.run(None, 1, 1, 1, None, 1, None, 1, None, 1, 0, None) == xg.XGEMM_ERR_INVALID_ARG
    assert xg.xgemm_run_noalloc(None, 1, 1, 1, None, 1, None, 1, None, 1, 0, None) == xg.XGEMM_ERR_INVALID_ARG


@pytest.mark.parametrize("kind", ["missing", "other_torch"])
def test_import_without_a_matching_extension(kind, tmp_path):
    """The extension is an addition: without one built for this torch the
    module warns, loads, and calls the library through ctypes."""
    pkg = os.path.dirname(xg.__file__)
    copy = tmp_path / "paper_2609_16389_amd"
    shutil.copytree(pkg, copy, ignore=shutil.ignore_patterns("__pycache__", "csrc"))
    ext = copy / "_fastcall.so"
    if kind == "missing":
        ext.unlink()
    else:
        tag = b"torch " + torch.__version__.encode()
        data = ext.read_bytes()
        assert tag in data
        ext.write_bytes(data.replace(tag, b"torch 0" + tag[7:]))
    code = ("import warnings\nwith warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always')\n    from paper_2609_16389_amd import xgemm as xg\n"
            "assert any('_fastcall' in str(x.message) for x in w)\n"
            "assert xg.xgemm_run(None, 1, 1, 1, None, 1, None, 1, None, 1, 0, None) == xg.XGEMM_ERR_INVALID_ARG\n"
            "assert '_fastcall.so' not in open('/proc/self/maps').read()\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path)},
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr


@pytest.mark.gpu
def test_same_as_the_other_path():
    g = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randn(70, 136, device="cuda", generator=g).to(torch.float16)[:, :131]
    B = torch.randn(131, 96, device="cuda", generator=g).to(torch.float16)
    s = torch.cuda.current_stream()
    out = torch.full((70, 96), float("nan"), device="cuda")
    ref = xg.gemm(A, B, stream=s)
    assert xg.gemm(A, B, out=out) is out and torch.equal(out, ref)
    assert _fastcall.gemm(A, B, out) == xg.XGEMM_OK           # the handle exists: taken
    A3, B3 = torch.stack([A, A]), torch.stack([B, B])
    out3 = torch.empty(2, 70, 96, device="cuda")
    assert torch.equal(xg.bmm(A3, B3, out=out3), xg.bmm(A3, B3, stream=s))
    x, y = torch.randn(131, device="cuda", generator=g), torch.empty(70, device="cuda")
    Af = A.float()
    assert torch.equal(xg.gemv(Af, x, out=y), xg.gemv(Af, x, stream=s))


@pytest.mark.gpu
def test_errors_are_the_other_paths():
    A = torch.zeros(8, 8, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(8, 8, device="cuda")
    xg.gemm(A, A, out=out)
    with pytest.raises(TypeError):
        xg.gemm(A, A.half(), out=out)
    with pytest.raises(ValueError):
        xg.gemm(A, A, out=out[:4])
    with pytest.raises(ValueError):
        xg.gemm(A.t(), A, out=out)
    with pytest.raises(xg.XgemmError):                        # overlapping rows: refused by the library
        xg.gemm(A.as_strided((8, 8), (4, 1)), A, out=out)
    with pytest.raises(Exception):                            # batched by a transform: no data pointer
        torch.func.vmap(lambda a: xg.gemm(a, A, out=out))(A.expand(2, 8, 8))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        xg.gemm(A, A, out=out)
    torch.cuda.synchronize()
    assert xg.handle(0, side) != xg.handle(0, torch.cuda.current_stream())
