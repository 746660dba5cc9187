"""Properties of the compiled forward kernels that decide their speed and that
no output shows, read from the compiler's listing for gfx950 (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2412_12392_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Listing of m3s_kernels.hip: the lines of every kernel by its mangled name."""
    out = str(tmp_path_factory.mktemp("listing") / "kernels.s")
    subprocess.run([build.hipcc(), *build.flags(), "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "m3s_kernels.hip"), "-o", out], check=True, capture_output=True)
    found, name = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"(_Z\w+):", line)
            if m:
                name = m.group(1)
                found[name] = []
            elif line.startswith(".Lfunc_end"):
                name = None
            elif name:
                found[name].append(line)
    return found


def _blocks(lines):
    """Instructions of each basic block."""
    block = []
    for line in lines:
        if re.match(r"\.LBB|; %bb", line):
            yield block
            block = []
        elif re.match(r"\s+[a-z]\w+", line):
            block.append(line.split()[0])
    yield block


def test_global_scan_loads_stay_together(kernels):
    """A candidate's six descriptor loads are neighbours: between them another wave's
    loads evict the line (a quarter to a half of a batch's time)."""
    checked = 0
    for name, lines in kernels.items():
        if "fwd_kernel" not in name or "ILi" not in name:
            continue
        for ops in _blocks(lines):
            loads = [i for i, op in enumerate(ops) if re.match(r"(global|flat)_load_dwordx4", op)]
            dots = sum(op.startswith(("v_fma_f32", "v_fmac_f32")) for op in ops)
            if len(loads) != 6 or dots != 24:
                continue
            checked += 1
            assert loads[-1] - loads[0] == 5, (name, [ops[i] for i in range(loads[0], loads[-1] + 1)])
    assert checked >= 8, checked


def test_matcher_kernels_do_not_spill(kernels):
    """No kernel of the forward keeps vector registers in scratch memory: with the scans of
    three radii inlined twice the multi-level kernels did, and batches of two levels lost 6 to
    15 % to it."""
    scratch = {}
    for name, lines in kernels.items():
        if "fwd" in name:
            scratch[name] = sum("scratch_store" in line for line in lines)
    assert len(scratch) > 20
    assert not any(scratch.values()), {k: v for k, v in scratch.items() if v}
