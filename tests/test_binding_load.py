"""Loading of the binding's library and of its native calls, on the host: copies
of the package whose shared objects are missing or do not fit."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2609_39859_amd import _binding

HERE = os.path.dirname(os.path.abspath(_binding.__file__))
NAME = os.path.basename(HERE)


def _copy(tmp_path, *objects):
    pkg = tmp_path / NAME
    pkg.mkdir()
    for f in os.listdir(HERE):
        if f.endswith(".py") or f in objects:
            shutil.copy(os.path.join(HERE, f), str(pkg / f))
    return pkg


def _run(tmp_path, code):
    r = subprocess.run([sys.executable, "-c", code], cwd=str(tmp_path), text=True,
                       capture_output=True, env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert r.returncode == 0, r.stderr
    return r.stdout


@pytest.mark.parametrize("other", ["not a library", "other structures"])
def test_native_calls_that_do_not_fit_are_left_out(tmp_path, other):
    """The first use of the library warns, and it and all later ones work."""
    pkg = _copy(tmp_path, "libforkstep.so", "_fastcall.so")
    code = "import warnings, %s._binding as b\n" % NAME
    if other == "not a library":
        (pkg / "_fastcall.so").write_bytes(b"\x7fELF of another interpreter")
    else:
        code += "class Longer(b.ForkSelectArgs): _fields_ = [('more', b._I32)] * 1\n"
        code += "b.ForkSelectArgs = Longer\n"
    code += ("with warnings.catch_warnings(record=True) as w:\n"
             "    warnings.simplefilter('always')\n"
             "    first = b.version()\n"
             "    assert [x.category for x in w] == [RuntimeWarning], w\n"
             "assert b._fast is None and b.version() == first\n")
    _run(tmp_path, code)


def test_arguments_are_checked_before_the_library_is_loaded(tmp_path):
    """Without the library a wrong argument is reported as such."""
    _copy(tmp_path)
    out = _run(tmp_path, """
import torch, %s._binding as b
t = torch.zeros(4, 4)
for call in (lambda: b.top_entropy(t, 1, t), lambda: b.grpo_objective(t, t, t, t, 2, 0.2, t, t, t),
             lambda: b.fork_step_ex(t, t, t, t, t, 1, 0.5, t, t, t, t, B=2, L=2),
             lambda: b.select(t, t, t, t, t, 1, 0.5, t, B=1, L=1), lambda: b.logprob(t, t, t, t)):
    try:
        call()
    except (TypeError, ValueError) as e:
        print(type(e).__name__, e)
""" % NAME)
    assert len(out.splitlines()) == 5 and "GPU" in out
