"""A launch of few tiles ends in a chain of latencies.  The kernels ask for the running result they add to before they drain their copies and
meet at the last barrier; read off the generated code, because results and most timings do not show the order."""
import os
import re
import subprocess

import pytest

from paper_2408_10188_amd import build


def kernels(asm):
    """{symbol: instruction lines} of an assembly listing."""
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w*_kernel\w*):", line)
        if m:
            name = m[1]
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            out[name].append(line.split(";")[0].strip())
    return out


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
@pytest.mark.parametrize("source,reading", [("fwd_bf16.hip", 2), ("bwd_dq_bf16.hip", 2),    # of these add to a result: one of 4, one of 8 wavefronts
                                            ("bwd_dkdv_bf16.hip", 2)])                    # with and without a mask
def test_running_results_are_read_before_the_last_barrier(tmp_path, source, reading):
    out = tmp_path / "k.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    found = 0
    for name, code in kernels(out.read_text()).items():
        if "reduce" in name:
            continue
        written = max(i for i, line in enumerate(code) if line.startswith("ds_write_b128"))     # the result on its way through LDS
        barrier = max(i for i, line in enumerate(code[:written]) if line.startswith("s_barrier"))
        end = min(i for i, line in enumerate(code) if line.startswith("s_endpgm") and i > written)
        loads = [i for i, line in enumerate(code) if line.startswith("global_load_dwordx4")]
        assert not [i for i in loads if barrier < i < end], name
        found += len([i for i in loads if i < barrier]) >= 8 + 16                                # Q (and dO) or K and V, then the running result
    assert found >= reading
