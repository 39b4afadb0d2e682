"""What the compiler makes of the kernels: an iteration of pasa_rows' key loop must not wait for loads that the next ones need, and no kernel
keeps vector registers in memory.  Compiles, needs no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_01873_amd import build


pytestmark = pytest.mark.skipif(not shutil.which("hipcc") and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


def _assembly(source, tmp_path):
    out = tmp_path / "kernels.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([build.hipcc(), *flags, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def test_no_iteration_waits_for_all_its_loads(tmp_path):
    text = _assembly("pasa_rows.hip", tmp_path)
    names = re.findall(r"^(\S*pasa_rowsI\S*):", text, re.M)
    assert len(names) == 6
    for name in names:
        body = text[text.index("\n" + name + ":"):].split(".Lfunc_end")[0]
        headers = set(re.findall(r"^\.L(BB\d+_\d+):.*Loop Header", body, re.M))
        loops, at = {}, None
        for line in body.splitlines():
            block = re.match(r"(?:\.L(BB\d+_\d+):|; %bb\.\d+:)", line)
            if block:
                of = re.search(r"Header=(BB\d+_\d+)", line)
                at = block.group(1) if block.group(1) in headers else of.group(1) if of else None
            if at is not None:
                loops.setdefault(at, []).append(line)
        key_loops = [lines for lines in loops.values() if sum("v_mfma" in x for x in lines) > 8]
        assert len(key_loops) == 1, name
        waits = [int(n) for x in key_loops[0] for n in re.findall(r"s_waitcnt.*vmcnt\((\d+)\)", x)]
        # four fragments of d = 64 are the fewest that are asked for at a time; the newest ones are needed next time round
        assert waits and min(waits) >= 4, (name, waits)


@pytest.mark.parametrize("source", ["pasa_kernels.hip", "pasa_fwd4.hip", "pasa_rows.hip"])
def test_no_vector_register_is_kept_in_memory(source, tmp_path):
    """pasa_fwd with counters too: the first pass of the adaptive start is one of those."""
    spilled = dict(re.findall(r"\.name: +(\S+)\n(?:(?! +- ).*\n)*? +\.vgpr_spill_count: +(\d+)", _assembly(source, tmp_path)))
    assert any("pasa_" in name for name in spilled) and not any(int(n) for n in spilled.values()), spilled
