"""Checks of the assembly that the compiler makes of the hand-written kernels (no GPU)."""
import os
import re
import subprocess

import pytest

import __graft_entry__ as entry


def _assembly(source, tmp_path):
    command = entry.hipcc_command(str(tmp_path / "kernels.s"))
    flags = [a for a in command if not a.startswith(entry.CSRC) and a not in ("-shared", "-fPIC", "-ldl")]
    res = subprocess.run(flags + ["--offload-device-only", "-S", os.path.join(entry.CSRC, source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return (tmp_path / "kernels.s").read_text()


@pytest.mark.parametrize("source,kernels", [("mfma.hip", 18), ("staged_rows.hip", 8)])
def test_waves_meet_with_no_lds_access_on_its_way(source, kernels, tmp_path):
    """Behind a barrier of these kernels another wave overwrites what was read from LDS before it: a read that is still
    on its way would return the new bytes, and nothing but the wait keeps the instruction that uses it in front."""
    bodies = re.findall(r"^(_ZN8sparsert\w+):.*?$(.*?)^\.Lfunc_end", _assembly(source, tmp_path), re.S | re.M)
    assert len(bodies) == kernels
    for name, body in bodies:
        lines = [l for l in (l.split(";")[0].strip() for l in body.splitlines()) if l]
        barriers = [i for i, l in enumerate(lines) if l == "s_barrier"]
        assert barriers
        for i in barriers:
            while True:
                i -= 1
                assert not lines[i].startswith("ds_") and not lines[i].endswith(":"), (name, lines[i:i + 8])
                if re.match(r"s_waitcnt .*lgkmcnt\(0\)", lines[i]):
                    break


def test_half_results_of_low_tiles_go_straight_to_memory(tmp_path):
    """Tiles of 32 rows and less with rows of C that are no whole 128-byte lines; 32 columns of halves never are."""
    bodies = dict(re.findall(r"^_ZN8sparsert11mfma_kernelI(\w+?)EEEvNS_8MfmaArgsE:.*?$(.*?)^\.Lfunc_end", _assembly("mfma.hip", tmp_path), re.S | re.M))
    assert "ds_write" not in bodies["Li0ELi2ELi2ELi1ELi1ELi2ELi4"] and "ds_write" in bodies["Li0ELi2ELi2ELi2ELi2ELi2ELi4"]
