"""The kernels of a step fuse a multiplication and an addition only where the
source writes fma: compiled with and without the compiler's own contraction
they have the same operations (the step forms have to agree bit for bit)."""
import collections
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2502_16818_amd import build

SOURCES = sorted(s for s, flags in build.EXTRA.items() if "-ffp-contract=off" in flags)


def _operations(src, contract, out):
    flags = [f for f in build.FLAGS + build.EXTRA[src] if not f.startswith("-ffp-contract")]
    subprocess.run([build.hipcc(), "-x", "hip", f"--offload-arch={build.ARCH}", *flags, f"-ffp-contract={contract}",
                    "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    count = collections.Counter()
    for line in out.read_text().splitlines():
        m = re.match(r"\s+v_(fma|fmac|fmamk|fmaak|mul|add|sub|subrev)_(f32|f64)", line)
        if m:   # a subtraction is an addition, whichever operand is negated
            op = "fma" if m[1].startswith("fma") else "mul" if m[1] == "mul" else "add"
            count[op, m[2]] += 1
    return count


@pytest.mark.slow
def test_step_kernels_fuse_only_what_is_written(tmp_path):
    assert {"kernels_stage.hip", "kernels_quad.hip", "kernels_tile.hip", "kernels_march.hip",
            "kernels_step.hip", "kernels_batch.hip"} == set(SOURCES)
    jobs = [(s, c) for s in SOURCES for c in ("off", "fast")]
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        got = dict(zip(jobs, ex.map(lambda j: _operations(*j, tmp_path / f"{j[0]}.{j[1]}.s"), jobs)))
    for s in SOURCES:
        assert got[s, "off"]["fma", "f64"] > 100
        assert got[s, "off"] == got[s, "fast"], s
