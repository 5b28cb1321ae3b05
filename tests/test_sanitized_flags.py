"""The host-sanitized driver's build: sanitizers and -O1 in the host pass, the
device pass with the library's own options (CPU only: what hipcc would run)."""
import os
import shlex
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _passes(flags):
    """{target: options} of the compiler's own calls for a source."""
    src = os.path.join(ROOT, "paper_2211_12867_amd", "csrc", "stage.hip")
    r = subprocess.run(["hipcc", "-###", "-x", "hip", "-c", src, "-o", "x.o"] + flags, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    calls = [shlex.split(line) for line in r.stderr.splitlines() if '"-cc1"' in line]
    return {c[c.index("-triple") + 1].split("-")[0]: c for c in calls}


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_device_code_is_the_librarys():
    import importlib.util
    spec = importlib.util.spec_from_file_location("_ic_build",
                                                  os.path.join(ROOT, "paper_2211_12867_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    lib, san = _passes(b.FLAGS), _passes(b.SAN_FLAGS)

    def options(call):                       # without the names of intermediate files
        return [o for o in call if "/tmp/" not in o and not o.startswith("-cuid=")]

    assert options(lib["amdgcn"]) == options(san["amdgcn"])
    assert "-O3" in san["amdgcn"] and not any("sanitize" in o for o in san["amdgcn"])
    host = san["x86_64"]
    assert "-O1" in host and any(o.startswith("-fsanitize=") and "address" in o for o in host)
