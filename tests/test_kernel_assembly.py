"""Checks of the assembly that the compiler makes of the hand-written kernels, and of their launch geometry (no GPU)."""
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


def test_half_results_of_small_tiles_go_straight_to_memory(tmp_path):
    """Rows of 32 halves are never whole lines of 128 bytes; a small tile does not earn the barrier and the round trip back."""
    bodies = dict(re.findall(r"^_ZN8sparsert11mfma_kernelI(\w+?)EEEvNS_8MfmaArgsE:.*?$(.*?)^\.Lfunc_end", _assembly("mfma.hip", tmp_path), re.S | re.M))
    assert "ds_write" not in bodies["Li0ELi2ELi2ELi1ELi1ELi2ELi4"] and "ds_write" in bodies["Li0ELi2ELi2ELi2ELi2ELi2ELi4"]


def test_half_results_stay_in_the_caches_for_the_next_layer(tmp_path):
    """Only int32 results, which an element-wise kernel reads next, are stored with the hint that nothing reads them soon;
    whole lines of half results go through to the caches behind the L2, others are stored plainly."""
    bodies = re.findall(r"^_ZN8sparsert11mfma_kernelILi(\d)E\w+:.*?$(.*?)^\.Lfunc_end", _assembly("mfma.hip", tmp_path), re.S | re.M)
    assert len(bodies) == 18
    for dtype, body in bodies:
        stores = re.findall(r"buffer_store\S* (.*)", body)
        assert any(re.search(r"\bnt\b", l) for l in stores) == (dtype == "1")
        assert any(re.search(r"\bsc1\b", l) for l in stores) == (dtype == "0" and "ds_write" in body)
        assert any(not re.search(r"\b(nt|sc1)\b", l) for l in stores)


def _pulled(M, K, N, ldb, esz, tm, tn, per):
    """Bytes of A and B, B in lines of 128 bytes, that the eight XCDs pull with the tiles in parts of `per` along M."""
    m_tiles, n_tiles = -(-M // tm), -(-N // tn)
    order = [(m, n) for m0 in range(0, m_tiles, per) for n in range(n_tiles) for m in range(m0, min(m_tiles, m0 + per))]
    share, total = -(-len(order) // 8), 0
    for x in range(0, len(order), share):
        mine = order[x:x + share]
        total += len({m for m, _ in mine}) * tm * K * esz
        total += 128 * len({line for n in {n for _, n in mine} for k in range(K)
                            for line in range((k * ldb + n * tn) * esz // 128, ((k * ldb + min(N, (n + 1) * tn)) * esz - 1) // 128 + 1)})
    return total


@pytest.mark.parametrize("M,K,N,ldb,esz,tm,tn", [
    (272, 3592, 196, 196, 1, 32, 32), (768, 3072, 1024, 1024, 1, 64, 64), (3072, 768, 1024, 1024, 2, 96, 128), (226, 1768, 128, 128, 2, 32, 32),
    (594, 640, 1142, 1142, 1, 64, 128), (608, 1024, 496, 550, 2, 32, 64), (248, 2696, 640, 640, 1, 32, 32), (147, 1904, 1248, 1248, 1, 32, 32)])
def test_order_of_tiles_pulls_few_bytes(M, K, N, ldb, esz, tm, tn, tmp_path):
    source = tmp_path / "order.cpp"
    source.write_text('#include <cstdio>\n#include "mfma.h"\nint main() { using namespace sparsert;\n'
                      f'    printf("%d", mfma_rows_per_part(kMfmaConfigs[mfma_find({tm}, {tn})], {M}, {K}, {N}, {ldb}, {esz})); }}\n')
    subprocess.run(["g++", "-std=c++17", "-I", entry.CSRC, "-o", str(tmp_path / "order"), str(source)], check=True)
    chosen = int(subprocess.run([str(tmp_path / "order")], capture_output=True, text=True, check=True).stdout)
    least = min(_pulled(M, K, N, ldb, esz, tm, tn, per) for per in {1, -(-M // tm)})
    assert _pulled(M, K, N, ldb, esz, tm, tn, chosen) < 1.05 * least


def test_assembly_that_sets_m0_puts_it_back(tmp_path):
    """s_set_gpr_idx_* write M0, where the compiler may keep an index of its own across the block."""
    blocks = [b for b in re.findall(r";;#ASMSTART(.*?);;#ASMEND", _assembly("blocked_rows.hip", tmp_path), re.S) if "s_set_gpr_idx" in b]
    assert len(blocks) == 2
    for b in blocks:
        lines = [l for l in (l.split(";")[0].strip() for l in b.splitlines()) if l]
        first, last = (next(i for i in order if re.search(r"s_set_gpr_idx|\bm0\b", lines[i])) for order in (range(len(lines)), range(len(lines) - 1, -1, -1)))
        saved = re.fullmatch(r"s_mov_b32 (s\d+), m0", lines[first]).group(1)
        assert lines[last] == f"s_mov_b32 m0, {saved}"
        assert not any(re.search(rf"\b{saved}\b", l) for l in lines[first + 1:last])


def test_the_multiply_add_ceiling_is_the_fast_form(tmp_path):
    """Multiply-adds of the ceiling kernel read vector registers only, as those of the kernels held against it; a scalar operand halves their rate."""
    command = entry.ceilings_command(str(tmp_path / "ceilings.s"))
    flags = [a for a in command if not a.startswith(entry.CSRC) and a not in ("-shared", "-fPIC")]
    subprocess.run(flags + ["--offload-device-only", "-S", os.path.join(entry.CSRC, "ceilings.hip")], check=True, capture_output=True)
    body = re.search(r"^_ZN\w*fma_kernel\w*:.*?$(.*?)^\.Lfunc_end", (tmp_path / "ceilings.s").read_text(), re.S | re.M).group(1)
    mads = re.findall(r"v_(?:fma|fmac|pk_fma)_f32\S* (.*)", body)
    assert len(mads) == 32 and all(re.fullmatch(r"v\d+(, v\d+)+", m.split(";")[0].strip()) for m in mads)
