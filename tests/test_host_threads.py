"""State that launches from several host threads share, under the thread sanitizer (host code only, no GPU)."""
import os
import subprocess

import pytest

from paper_2408_10188_amd import build

MAIN = """
#include <stdint.h>
#include <thread>
namespace mmsp { int cu_count(); int64_t bwd_dkdv_partial_bytes() { return 0; } }
int main() {
  std::thread a([] { mmsp::cu_count(); }), b([] { mmsp::cu_count(); });
  a.join();
  b.join();
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
def test_cu_count_from_two_threads(tmp_path):
    main, exe = tmp_path / "main.hip", tmp_path / "threads"
    main.write_text(MAIN)
    flags = [f for f in build.FLAGS if f != "-O3"]
    built = subprocess.run([build.HIPCC, *flags, "-O1", "-g", "-Xarch_host", "-fsanitize=thread",
                            os.path.join(build.CSRC, "split.hip"), str(main), "-o", str(exe)], capture_output=True, text=True)
    if "clang_rt.tsan" in built.stderr:
        pytest.skip("the compiler has no thread sanitizer runtime")
    assert built.returncode == 0, built.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    if "unexpected memory mapping" in out.stderr:
        pytest.skip("the sanitizer does not run under this kernel's address layout")
    assert "cu_count" not in out.stderr, out.stderr
    assert out.returncode == 0, out.stderr
