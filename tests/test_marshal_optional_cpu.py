"""The binding without its C++ half: libcottn.so and binding.py alone make every call, over ctypes.  A _marshal.so that is
not there, or is there and cannot be used, is a warning that says which and why."""
import os
import shutil
import subprocess
import sys

import pytest

import paper_2409_18747_amd.binding as binding

# a refusal of binding.py, and an answer of the library
PROGRAM = """
import sys, warnings
import torch
{before}
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2409_18747_amd.binding as b
print([str(w.message) for w in seen if issubclass(w.category, RuntimeWarning) and "_marshal" in str(w.message)])
assert b.cottn_workspace_bytes(b.OP_BWD_CAUSAL, 1, 2, 4096, 64) > 0
Q = torch.zeros(1, 2, 8, 64, dtype=torch.bfloat16)
try:
    b.cottn_fwd_causal(Q, Q, Q, torch.ones(2))
except ValueError as e:
    assert "must live on the GPU" in str(e), e
else:
    raise AssertionError("accepted")
q = torch.zeros(1, 2, 64)
for call, args in ((b.cottn_bwd_causal, (Q, Q, Q, torch.ones(2), Q[:, :1])), (b.cottn_step, (q, q[:, :1], q, torch.ones(2), q)),
                   (b.cottn_scale_from_m_varlen, (torch.ones(2), torch.ones(1)))):
    try:
        call(*args)
    except (ValueError, TypeError):
        continue
    raise AssertionError("accepted")
"""


def warnings_of(tmp_path, marshal, before=""):
    package = tmp_path / "paper_2409_18747_amd"
    package.mkdir()
    for name in ("__init__.py", "binding.py", "build.py"):
        shutil.copy(os.path.join(os.path.dirname(binding.library_path), name), package / name)
    os.symlink(binding.library_path, package / "libcottn.so")
    if marshal is not None:
        (package / "_marshal.so").write_bytes(marshal)
    done = subprocess.run([sys.executable, "-c", PROGRAM.format(before=before)], cwd=tmp_path, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return done.stdout


@pytest.mark.parametrize("marshal,why", [(None, "is not built"), (b"not a library", "does not load")])
def test_calls_are_made_without_it(tmp_path, marshal, why):
    said = warnings_of(tmp_path, marshal)
    assert why in said and said.count("_marshal.so") >= 1, said
    assert (marshal is None) or "invalid ELF header" in said or "file too short" in said, said


def test_no_warning_with_it(tmp_path):
    with open(os.path.join(os.path.dirname(binding.library_path), "_marshal.so"), "rb") as f:
        assert warnings_of(tmp_path, f.read()).strip() == "[]"


def test_one_built_for_another_torch_is_not_used(tmp_path):
    """It holds the layout of that torch's tensors."""
    with open(os.path.join(os.path.dirname(binding.library_path), "_marshal.so"), "rb") as f:
        said = warnings_of(tmp_path, f.read(), "torch.__version__ = '1.0'")
    assert "_marshal.so was built for torch" in said and "not for torch 1.0" in said, said
