"""binding.py where _native cannot be loaded (not built, or built against another torch): its constants and host-side calls
are there, and only a call that needs the module raises."""
import subprocess
import sys

CODE = """
import sys
sys.modules["paper_2506_10443_amd._native"] = None      # importing it is an ImportError
from paper_2506_10443_amd import binding as B
assert (B.GROUP, B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT) == (64, 34)
for name in B.EXPORTS:
    if name not in ("mnnq_status_string", "mnnq_last_hip_error", "mnnq_version", "mnnq_act_planes_size"):
        assert callable(getattr(B, name)), name
for call in (B.mnnq_pack_weights, B.mnnq_linear_decode_fused, B.mnnq_linear_prefill_f16_o16):
    try:
        call(None, 16, 64, None)
    except RuntimeError as e:
        assert "not built" in str(e) and call.__name__ in str(e)
    else:
        raise AssertionError(call)
print("ok")
"""


def test_import_without_the_native_module():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr
