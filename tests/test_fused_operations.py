"""The kernels of an FP64 or mixed step fuse a multiplication and an addition only
where the source writes fma: compiled with and without the compiler's own
contraction each has the same operations (the step forms have to agree bit for
bit)."""
import collections
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2502_16818_amd import build

SOURCES = ["kernels_stage.hip", "kernels_quad.hip", "kernels_tile.hip", "kernels_march.hip",
           "kernels_step.hip", "kernels_batch.hip"]


def _operations(src, contract, out):
    """Per kernel, its counts of fused and single operations."""
    flags = [f for f in build.FLAGS + build.EXTRA[src] if not f.startswith("-ffp-contract")]
    subprocess.run([build.hipcc(), "-x", "hip", f"--offload-arch={build.ARCH}", *flags, f"-ffp-contract={contract}",
                    "--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    count, kernel = collections.defaultdict(collections.Counter), None
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            kernel = m[1]
        m = re.match(r"\s+v_(fma|fmac|fmamk|fmaak|mul|add|sub|subrev)_(f32|f64)", line)
        if m:   # a subtraction is an addition, whichever operand is negated
            op = "fma" if m[1].startswith("fma") else "mul" if m[1] == "mul" else "add"
            count[kernel][op, m[2]] += 1
    # k_stage<S, STAGE2, COMP, ..>: the compensated form has no other to agree with
    return {k: c for k, c in count.items() if not re.search(r"k_stageI[fd]Lb[01]ELb1E", k)}


@pytest.mark.slow
def test_step_kernels_fuse_only_what_is_written(tmp_path):
    for s in SOURCES[1:]:
        assert "-ffp-contract=off" in build.EXTRA[s]
    jobs = [(s, c) for s in SOURCES for c in ("off", "fast")]
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        got = dict(zip(jobs, ex.map(lambda j: _operations(*j, tmp_path / f"{j[0]}.{j[1]}.s"), jobs)))
    for s in SOURCES:
        assert sum(c["fma", "f64"] for c in got[s, "off"].values()) > 100, s
        assert got[s, "off"] == got[s, "fast"], s
