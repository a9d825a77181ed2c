"""The native marshalling only saves host time: without it, or with one that does not fit, the binding works."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2609_38166_amd import binding as B

SCRIPT = """
import warnings
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    from paper_2609_38166_amd import binding as B
    B.lib()
assert any("_marshal" in str(w.message) for w in said), said
d = B.make_dims(2, 4, 2, window=8, n_comp=2)
st = B.State.empty(d, device="cpu")
print(B.leapquant_state_bytes(d)[0], B.LIB_PATH)
for f, n in ((B.leapquant_decode_step, 6), (B.leapquant_decode_step_commit, 6), (B.leapquant_decode_step_general, 7),
             (B.leapquant_window_commit, 0)):
    try:
        f(d, st, *[st.scale] * n)
    except ValueError as e:                     # the Python checks took the call
        assert "device tensor" in str(e), e
    else:
        raise AssertionError(f.__name__)
"""


@pytest.mark.parametrize("kind", ["absent", "unloadable"])
def test_the_binding_works_without_the_extension(tmp_path, kind):
    pkg = os.path.dirname(os.path.abspath(B.__file__))
    to = tmp_path / os.path.basename(pkg)
    to.mkdir()
    for f in ("__init__.py", "binding.py", "synth.py", "libleapquant.so"):
        shutil.copy(os.path.join(pkg, f), to / f)
    if kind == "unloadable":
        (to / "_marshal.so").write_bytes(b"no shared library")
    env = {k: v for k, v in os.environ.items() if k not in ("LEAPQUANT_LIB", "PYTHONPATH")}
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=tmp_path, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert str(to) in r.stdout and int(r.stdout.split()[0]) == 2 * 4 * 128 * 128


def test_an_extension_built_against_another_torch_is_left_alone(monkeypatch):
    B.lib()
    native = B._M
    assert native.torch_version == B.torch.__version__
    monkeypatch.setattr(native, "torch_version", "0.0")
    monkeypatch.setattr(B, "_L", None)
    monkeypatch.setattr(B, "_M", None)
    with pytest.warns(RuntimeWarning, match="_marshal"):
        B.lib()
    assert B._M is not native and B._M.step(0) is None and B._M.commit(0) is None


def test_the_library_is_built_where_the_extension_cannot_be(monkeypatch, tmp_path):
    """build() makes the HIP libraries and warns; an extension of an earlier build does not stay behind."""
    from paper_2609_38166_amd import build as lib_build
    left = tmp_path / "_marshal.so"
    left.write_bytes(b"an earlier build's")
    made = []
    monkeypatch.setattr(lib_build, "MARSHAL_LIB", str(left))
    monkeypatch.setattr(lib_build, "CXX", str(tmp_path / "no-such-compiler"))
    monkeypatch.setattr(lib_build, "_compile", lambda srcs, out, verbose, defines=(): made.append(out))
    with pytest.warns(RuntimeWarning, match="_marshal"):
        assert lib_build.build() == lib_build.LIB
    assert made == [lib_build.LIB, lib_build.BENCH_LIB] and not left.exists()
