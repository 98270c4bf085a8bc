"""The memory kept between preconditioners, on the CPU: the library's own source
over a stand-in for the HIP allocator."""
import re
import subprocess
from pathlib import Path

ROOT = Path(__file__).resolve().parents[1]


def test_kept_buffers(tmp_path):
    exe = tmp_path / "pool_check"
    subprocess.run(["g++", "-std=c++17", "-x", "c++", "-I", str(ROOT / "tests" / "hip_stub"),
                    "-I", str(ROOT / "include"), "-I", str(ROOT / "paper_1809_00828_amd" / "csrc"),
                    str(ROOT / "tests" / "pool_check.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_every_allocation_can_have_the_kept_memory():
    """Device memory is asked for in one file, which gives back what is kept before
    it reports that none is left."""
    csrc = ROOT / "paper_1809_00828_amd" / "csrc"
    direct = [f.name for f in sorted(csrc.iterdir())
              if re.search(r"\bhipMalloc(Async|Managed)?\(", f.read_text())]
    assert direct == ["dev_pool.hip"]
