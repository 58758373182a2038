"""The code generator's output, checked statically on the host: every memory access of every
generated block stays inside its buffer, no register is used before its load has been waited
for (see asm_check.py).  Runs over the executor variants, storage types, convolution, batch,
leading dimensions and a randomised grid - with no GPU."""
import os
import re

import numpy as np
import pytest
from hypothesis import HealthCheck, given, settings, strategies as st

import asm_check
from paper_2008_11849_amd import sparsert as sp, synth

ESZ = {np.dtype(np.float32): (4, 4), np.dtype(np.float16): (2, 2), np.dtype(np.int8): (1, 4)}


def _generated(csr, N, tmp_path, **opts):
    """Host-only plan with the generated kernel; returns (assembly text, plan info)."""
    path = os.path.join(str(tmp_path), "kernel.s")
    os.environ["SPARSERT_DUMP_ASM"] = path
    try:
        plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, csr.M, csr.K, N, host_only=True, kernel=sp.KERNEL_SPEC, **opts)
    finally:
        del os.environ["SPARSERT_DUMP_ASM"]
    info = plan.info()
    plan.destroy()
    return open(path).read(), info


def _clean(csr, N, tmp_path, **opts):
    text, info = _generated(csr, N, tmp_path, **opts)
    esz, osz = ESZ[csr.vals.dtype]
    problems, stats = asm_check.check(text, info, esz, osz)
    assert not problems, problems[:5]
    return info, stats


def _csr(dtype, M, K, sparsity, seed):
    return synth.int8_csr(M, K, sparsity, seed) if dtype == np.int8 else synth.uniform_csr(M, K, sparsity, seed, dtype=dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.int8])
@pytest.mark.parametrize("opts", [dict(spec_rows=1), dict(spec_rows=7, spec_tiles=2), dict(spec_rows=16, spec_ksplit=2),
                                  dict(spec_rows=24, spec_ksplit=8), dict(spec_rows=200, spec_ksplit=8), dict(spec_rows=210, spec_ksplit=8), dict(spec_rows=9, spec_depth=3),
                                  dict(spec_rows=5, spec_swizzle=True), dict(spec_rows=8, spec_lanes=16, spec_ksplit=4), dict()])
@pytest.mark.parametrize("N", [1, 49, 64, 196, 300])
def test_direct_and_k_split_blocks_stay_in_bounds(dtype, opts, N, tmp_path):
    csr = _csr(dtype, 210, 333, 0.9, N)
    info, stats = _clean(csr, N, tmp_path, **opts)
    esz, osz = ESZ[np.dtype(dtype)]
    # the checker saw the far corner of both matrices: the last row of B and of C are reached
    assert stats["max_out_end"] == 210 * N * osz
    assert stats["max_in_end"] <= 333 * N * esz and stats["loads"] > 0 and stats["stores"] >= 210



@pytest.mark.parametrize("M,K,N,batch,opts,on", [(2314, 520, 688, 1, {}, 1), (2314, 520, 688, 4, {}, 0), (2314, 520, 688, 1, dict(spec_depth=16), 0),
                                                 (768, 3072, 256, 1, {}, 0), (300, 300, 196, 1, {}, 0)])
def test_long_blocks_touch_their_code_ahead(M, K, N, batch, opts, on, tmp_path):
    csr = synth.uniform_csr(M, K, 0.856, 3)
    info, _ = _clean(csr, N, tmp_path, batch=batch, **opts)
    assert info["spec_mode"] == sp.SPEC_DIRECT and bool(info["spec_prefetch"]) == bool(on)


@pytest.mark.parametrize("dtype,M,K,N,sparsity,img,on", [
    (np.float32, 384, 1008, 2209, 0.818, 47, 0), (np.float16, 408, 1152, 2704, 0.85, 52, 0), (np.int8, 392, 1152, 2601, 0.835, 51, 0),
    (np.float16, 2173, 560, 3968, 0.919, 0, 0), (np.int8, 3584, 216, 3400, 0.803, 0, 0), (np.float16, 1258, 780, 728, 0.821, 0, 1),
    (np.int8, 1420, 942, 888, 0.852, 0, 1), (np.float32, 2759, 320, 1307, 0.8, 0, 1)])
def test_what_touching_code_ahead_slows_down_does_not(dtype, M, K, N, sparsity, img, on):
    """Convolutions, half and int8 products in few parts: long blocks and much code, and slower for the touches all the same."""
    csr = synth.int8_csr(M, K, sparsity, 3) if dtype == np.int8 else synth.uniform_csr(M, K, sparsity, 3, dtype=dtype)
    info = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, M, K, N, host_only=True, kernel=sp.KERNEL_SPEC, **(dict(conv=(K // 9, img, img)) if img else {})).info()
    assert info["spec_mode"] == sp.SPEC_DIRECT and info["spec_rows"] > 50 and info["spec_code_bytes"] > 720000
    assert bool(info["spec_prefetch"]) == bool(on)


def test_the_touches_can_be_switched_off():
    """A caller that runs one plan alone, whose code stays in the caches, gets the plan without them and no other change."""
    csr = synth.uniform_csr(2314, 520, 0.856, 3)
    on, off, plain = ({k: p.info()[k] for k in p.info()} for p in (sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 2314, 520, 688, host_only=True, **o)
                                                                   for o in ({}, dict(spec_prefetch=-1), dict(spec_depth=16))))
    assert on["spec_prefetch"] > 0 and off["spec_prefetch"] == 0
    assert {k for k in on if on[k] != off[k]} <= {"spec_prefetch", "spec_code_bytes"} and off["spec_code_bytes"] == plain["spec_code_bytes"]
    half = synth.uniform_csr(1024, 1024, 0.8, 3, dtype=np.float16)   # a plan without generated code stays one
    assert sp.inspect(half.row_ptr, half.col_idx, half.vals, 1024, 1024, 512, host_only=True, spec_prefetch=-1).info()["spec_mode"] == sp.SPEC_MFMA
    with pytest.raises(sp.SparseRTError):
        sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 2314, 520, 688, host_only=True, spec_prefetch=-2)


def test_code_prefetch_is_checked(tmp_path):
    csr = synth.uniform_csr(300, 500, 0.8, 2)
    text, info = _generated(csr, 130, tmp_path, spec_rows=96, spec_ksplit=2, spec_prefetch=1)
    problems, stats = asm_check.check(text, info, 4, 4)
    assert not problems and stats["prefetch_loads"] >= 2 and info["spec_prefetch"] == stats["prefetch_loads"]   # blocks of more than 8 KiB
    off, info2 = _generated(csr, 130, tmp_path, spec_rows=96, spec_ksplit=2)
    assert asm_check.check(off, info2, 4, 4) == ([], dict(stats, prefetch_loads=0)) and info2["spec_prefetch"] == 0
    # a prefetch whose offset runs ahead of its mask would read past the block: the checker sees it
    bad = text.replace("global_load_dword v2, v4, s[18:19] offset:128", "global_load_dword v2, v4, s[18:19] offset:256", 1)
    assert any("not covered by its length mask" in p for p in asm_check.check(bad, info, 4, 4)[0])


def test_code_prefetch_stops_at_the_end_of_its_block(tmp_path):
    """Also where blocks are moved apart: what lies between them is never run."""
    csr = synth.uniform_csr(1024, 1024, 0.9, 4)
    text, info = _generated(csr, 832, tmp_path, spec_rows=54, spec_ksplit=8, spec_prefetch=1)
    gap = {int(l.split()[1]) for l in text.splitlines() if ".space" in l}
    assert len(gap) == 1 and min(gap) > 0 and asm_check.check(text, info, 4, 4)[0] == []
    bad = text.replace("\ts_sub_u32 s55, s55, 0x%x\n" % min(gap), "", 1)
    assert any("bytes apart" in p for p in asm_check.check(bad, info, 4, 4)[0])


@pytest.mark.parametrize("N,vec,dtype", [(64, 2, np.float16), (130, 2, np.float16), (64, 4, np.int8), (260, 4, np.int8)])
@pytest.mark.parametrize("ks", [1, 4])
def test_packed_columns_stay_in_bounds(N, vec, dtype, ks, tmp_path):
    _clean(_csr(dtype, 100, 200, 0.85, 5), N, tmp_path, spec_rows=12, spec_vec=vec, spec_ksplit=ks)


@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.int8])
@pytest.mark.parametrize("waves", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("K", [5, 128, 129, 515])
def test_lds_staged_blocks_stay_in_bounds(waves, K, dtype, tmp_path):
    csr = _csr(dtype, 90, K, 0.8, K)
    info, stats = _clean(csr, 130, tmp_path, spec_rows=6, spec_mode=sp.SPEC_LDS, spec_tiles=waves)
    assert stats["lds"] > 0 and stats["max_lds_end"] <= info["spec_lds_bytes"]


@pytest.mark.parametrize("M,K,N,sparsity,rows,waves", [
    (90, 515, 130, 0.8, 6, 4), (33, 129, 64, 0.9, 40, 2), (40, 300, 64, 0.99, 3, 16),   # a last chunk of 3, 1 and 44 rows
    (90, 1000, 130, 0.999, 6, 8),                                                        # chunks without a nonzero of the block
    (64, 128, 64, 0.9, 8, 4),                                                            # one chunk
    (2048, 1024, 4035, 0.97, 0, 0)])                                                     # the default shape
def test_lds_staged_waves_agree_on_which_buffer_is_read(M, K, N, sparsity, rows, waves, tmp_path):
    opts = dict(spec_rows=rows, spec_tiles=waves, spec_mode=sp.SPEC_LDS) if rows else {}
    text, info = _generated(synth.uniform_csr(M, K, sparsity, 3), N, tmp_path, **opts)
    assert info["spec_mode"] == sp.SPEC_LDS
    chunk = min(128, 32 * info["spec_tiles"])
    for block in re.split(r"\n\.Lg\d+:", text)[1:]:
        lines, barriers, in_flight, staging = [l.strip() for l in block.splitlines()], 0, 0, {}
        for l in lines:
            if l == "s_barrier":        # chunk `barriers` is read from here on, and the one after it written to the other buffer
                assert in_flight == 0
                barriers += 1
            m = re.match(r"s_waitcnt lgkmcnt\((\d+)\)", l)
            if m:
                in_flight = min(in_flight, int(m.group(1)))
                staging = {r: n for r, n in staging.items() if n < in_flight}
            m = re.match(r"ds_(read|write)_b\d+ .*offset:(\d+)", l)
            if m:
                which = int(m.group(2)) // (chunk * 256)
                assert which == ((barriers - 1) & 1 if m.group(1) == "read" else barriers & 1), l
                staging = {r: n + 1 for r, n in staging.items()}
                in_flight += 1
                if m.group(1) == "write":
                    first, last = re.search(r", v\[(\d+):(\d+)\]", l).groups()
                    staging.update({r: 0 for r in range(int(first), int(last) + 1)})
            m = re.match(r"buffer_load_dword v(\d+),", l)
            if m:                       # not over words that may still be on their way into LDS
                assert int(m.group(1)) not in staging, l
        assert barriers == -(-K // chunk)


@pytest.mark.parametrize("ldb,ldc,batch", [(0, 0, 3), (136, 0, 1), (0, 4096, 1), (200, 264, 2)])
def test_leading_dimensions_and_batches_stay_in_bounds(ldb, ldc, batch, tmp_path):
    N = 130
    csr = synth.uniform_csr(77, 150, 0.9, 2)
    for opts in (dict(spec_rows=8), dict(spec_rows=16, spec_ksplit=4), dict(spec_rows=8, spec_mode=sp.SPEC_LDS, spec_tiles=4)):
        info, stats = _clean(csr, N, tmp_path, ldb=ldb, ldc=ldc, batch=batch, **opts)
        assert stats["max_out_end"] == (76 * (ldc or N) + N) * 4      # the extent of one matrix of the batch
        assert stats["max_in_end"] <= (149 * (ldb or N) + N) * 4


@pytest.mark.parametrize("Cin,Cout,H,W", [(3, 5, 1, 1), (4, 6, 2, 3), (16, 24, 14, 14), (6, 10, 9, 13), (8, 4, 56, 56)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16, np.int8])
def test_convolution_blocks_stay_in_bounds(Cin, Cout, H, W, dtype, tmp_path):
    csr, _ = synth.conv_weights_csr(Cout, Cin, 0.7, H + W)
    if dtype == np.int8:
        csr = synth.CSR(csr.M, csr.K, csr.row_ptr, csr.col_idx, synth.quantise_weights(csr.vals))
    else:
        csr = synth.CSR(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals.astype(dtype))
    for opts in (dict(spec_rows=3), dict(spec_rows=4, spec_ksplit=4), dict(batch=4)):
        info, stats = _clean(csr, H * W, tmp_path, conv=(Cin, H, W), **opts)
        esz = ESZ[np.dtype(dtype)][0]
        # a tap at the bottom right of the last channel reaches the end of the padded descriptor, never beyond
        assert stats["max_in_end"] <= (Cin * H * W + 2 * (W + 1)) * esz


def test_the_checker_catches_planted_mistakes(tmp_path):
    """The checker itself: one edit of a clean kernel per property it guards."""
    csr = synth.uniform_csr(64, 200, 0.9, 1)
    text, info = _generated(csr, 100, tmp_path, spec_rows=16, spec_ksplit=4)
    assert asm_check.check(text, info, 4, 4)[0] == []
    lines = text.splitlines()

    def edited(find, replace_with, nth=0):
        idx = [i for i, l in enumerate(lines) if find(l)][nth]
        out = list(lines)
        out[idx] = replace_with(out[idx])
        return "\n".join(out)

    import re
    # a row offset one row past the end of B
    t = edited(lambda l: l.startswith("\ts_mov_b32 s62, "), lambda l: "\ts_mov_b32 s62, 0x%x" % (200 * 100 * 4))
    assert any("operand" in p for p in asm_check.check(t, info, 4, 4)[0])
    # a wait that lets one more load stay in flight than the code assumes
    t = edited(lambda l: "s_waitcnt vmcnt(" in l, lambda l: re.sub(r"vmcnt\((\d+)\)", lambda m: "vmcnt(%d)" % (int(m.group(1)) + 1), l))
    assert any("in flight" in p for p in asm_check.check(t, info, 4, 4)[0])
    # an LDS offset beyond the exchange area
    t = edited(lambda l: l.startswith("\tds_write_"), lambda l: re.sub(r"offset:\d+", "offset:%d" % info["spec_lds_bytes"], l))
    assert any("group segment" in p for p in asm_check.check(t, info, 4, 4)[0])
    # a register above the allocation
    t = edited(lambda l: l.startswith("\tv_fmac_f32"), lambda l: re.sub(r"v_fmac_f32_e32 v\d+", "v_fmac_f32_e32 v255", l))
    assert any("next_free_vgpr" in p for p in asm_check.check(t, info, 4, 4)[0])
    # a store below the start of C's last row ... moved past the end of C
    t = edited(lambda l: l.startswith("\tbuffer_store_dword"), lambda l: l, 0)
    idx = [i for i, l in enumerate(lines) if l.startswith("\tbuffer_store_dword")][0]
    out = list(lines)
    out[idx - 1] = re.sub(r"0x[0-9a-f]+", "0x%x" % (64 * 100 * 4), out[idx - 1])
    assert any("result" in p for p in asm_check.check("\n".join(out), info, 4, 4)[0])
    # a block that runs into the next one
    idx = [i for i, l in enumerate(lines) if l.strip() == "s_endpgm"][2]
    out = list(lines)
    out[idx] = "\ts_nop 0"
    assert any("does not end" in p for p in asm_check.check("\n".join(out), info, 4, 4)[0])


@settings(max_examples=60, deadline=None, suppress_health_check=[HealthCheck.function_scoped_fixture])
@given(M=st.integers(1, 130), K=st.integers(1, 400), N=st.integers(1, 330), sparsity=st.sampled_from([0.0, 0.5, 0.9, 0.99]),
       rows=st.sampled_from([0, 1, 3, 8, 31, 96]), ks=st.sampled_from([0, 1, 2, 4, 8]), mode=st.sampled_from([1, 1, 2]),
       dtype=st.sampled_from([np.float32, np.float16, np.int8]), swizzle=st.booleans(), seed=st.integers(0, 99), prefetch=st.booleans())
def test_random_generated_kernels_are_clean(M, K, N, sparsity, rows, ks, mode, dtype, swizzle, seed, prefetch, tmp_path):
    csr = _csr(dtype, M, K, sparsity, seed)
    opts = dict(spec_rows=rows, spec_ksplit=ks, spec_mode=mode, spec_swizzle=swizzle, spec_prefetch=int(prefetch))
    if mode == sp.SPEC_LDS:
        opts["spec_ksplit"] = 0
    try:
        text, info = _generated(csr, N, tmp_path, **opts)
    except sp.SparseRTError as e:
        assert e.status in (sp.EINVAL, sp.EUNSUPPORTED)   # a refusal is fine, a broken kernel is not
        return
    problems, _ = asm_check.check(text, info, *ESZ[np.dtype(dtype)])
    assert not problems, (opts, problems[:5])


def _deal(text):
    """The prologue from the load of the kernel's arguments on."""
    body = [l.strip() for l in text[:text.index("\n.Ltable:")].splitlines()]
    return body[next(i for i, l in enumerate(body) if l.startswith("s_load_dwordx4 s[4:7]")) + 1:]


def _dealt(prologue, x, y, z):
    """(column tile, code block, problem) that the prologue computes for a workgroup of the launch."""
    s, scc = {"s2": x, "s3": y, "s52": z}, False
    value = lambda tok: s[tok] if tok in s else int(tok, 0)
    ops = {"s_and_b32": lambda a, b: (a & b, a & b != 0), "s_lshr_b32": lambda a, b: (a >> b, a >> b != 0), "s_min_u32": lambda a, b: (min(a, b), a <= b),
           "s_add_u32": lambda a, b: (a + b & 0xFFFFFFFF, a + b > 0xFFFFFFFF), "s_sub_u32": lambda a, b: (a - b & 0xFFFFFFFF, a < b),
           "s_mul_i32": lambda a, b: (a * b & 0xFFFFFFFF, scc), "s_mul_hi_u32": lambda a, b: (a * b >> 32, scc)}   # result, condition bit
    for l in prologue:
        op, _, rest = l.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op in ops:
            s[args[0]], scc = ops[op](value(args[1]), value(args[2]))
        elif op == "s_mov_b32":
            s[args[0]] = value(args[1])
        elif op == "s_cmp_eq_u32":
            scc = value(args[0]) == value(args[1])
        elif op == "s_cselect_b32":
            s[args[0]] = value(args[1] if scc else args[2])
        else:
            assert op.startswith("v_"), l
            return s["s2"], s["s3"], s["s52"]


@pytest.mark.parametrize("M,K,N,batch,mask,opts,moved", [
    (1024, 1024, 771, 1, "uniform", dict(), True),                                         # 13 column tiles; blocks in parts
    (1024, 2000, 320, 1, "uniform", dict(spec_rows=48, spec_ksplit=2), True),              # the last part has fewer blocks
    (1000, 2000, 30, 5, "uniform", dict(spec_rows=24, spec_ksplit=4), True),               # one tile, five problems
    (640, 2000, 577, 1, "uniform", dict(spec_rows=32, spec_tiles=2), True),                # workgroups of two adjacent tiles
    (400, 2000, 700, 3, "uniform", dict(spec_mode=sp.SPEC_LDS, spec_rows=12, spec_tiles=4), True),
    (64, 4096, 330, 1, "uniform", dict(spec_rows=64, spec_ksplit=8), False),               # one block: launch order costs the least
    (512, 512, 771, 1, "skewed", dict(spec_rows=1, spec_ksplit=4), False),                 # long rows first
])
def test_every_tile_and_block_is_dealt_to_one_workgroup(M, K, N, batch, mask, opts, moved, tmp_path):
    csr = synth.uniform_csr(M, K, 0.9, 4) if mask == "uniform" else synth.skewed_csr(M, K, 0.9, 4)
    text, info = _generated(csr, N, tmp_path, batch=batch, **opts)
    lds, n_tiles = info["spec_mode"] == sp.SPEC_LDS, -(-N // info["spec_lanes"])
    tiles = n_tiles if lds or info["spec_ksplit"] > 1 else -(-n_tiles // info["spec_tiles"])
    blocks = -(-info["spec_groups"] // info["spec_tiles"]) if lds else info["spec_groups"]
    ids = [(x, y, z) for z in range(batch) for y in range(blocks) for x in range(tiles)]
    prologue = _deal(text)
    got = [_dealt(prologue, *i) for i in ids]
    assert sorted(got) == sorted(ids)
    assert (got != ids) == moved
    if moved:   # what an XCD touches, a byte of code counted three times
        touched = lambda work: sum(len({(t, z) for t, _, z in work[x::8]}) * K * info["spec_lanes"] * 4 + 3 * len({b for _, b, _ in work[x::8]}) * info["spec_code_bytes"] / blocks
                                   for x in range(8))
        assert touched(got) < 0.95 * touched(ids)
        lines = [len(b.splitlines()) for b in re.split(r"\n\.Lg\d+:", text)[1:]]
        waves = len(lines) // blocks
        of_block = [sum(lines[b * waves:(b + 1) * waves]) for b in range(blocks)]   # and what a compute unit runs, 32 to an XCD
        busiest = lambda work: max(sum(of_block[b] for _, b, _ in work[x::8][cu::32]) for x in range(8) for cu in range(32))
        assert busiest(got) < 1.05 * busiest(ids)


@pytest.mark.parametrize("M,K,N,opts", [
    (47, 891, 2116, dict(spec_rows=6, spec_ksplit=8)),     # 34 workgroups to an XCD, rows of very different lengths
    (184, 306, 2500, dict(spec_rows=7, spec_tiles=4))])    # 33 or 34, no K split
def test_workgroups_stay_in_launch_order_where_a_compute_unit_would_get_more_code(M, K, N, opts, tmp_path):
    text, _ = _generated(synth.skewed_csr(M, K, 0.9, 4), N, tmp_path, **opts)
    assert _deal(text)[0].startswith("v_")   # no scalar arithmetic on the workgroup ids


@pytest.mark.parametrize("rows,gap", [(54, True), (36, False), (100, False)])
def test_code_blocks_do_not_lie_a_multiple_of_8_kib_apart(rows, gap, tmp_path):
    csr = synth.uniform_csr(1024, 1024, 0.9, 4)
    text, info = _generated(csr, 832, tmp_path, spec_rows=rows, spec_ksplit=8)
    spaces = {l.strip() for l in text.splitlines() if ".space" in l}
    assert len(spaces) == 1 and (int(spaces.pop().split()[1]) > 0) == gap
    between = info["spec_code_bytes"] / (8 * info["spec_groups"])
    assert 1900 < between % 8192 < 6300


@pytest.mark.parametrize("M,K,N,rows", [(1024, 1024, 832, 44), (80, 512, 3136, 80)])   # 1.5 KB from the multiple; 59 KB of code
def test_code_blocks_stay_where_they_are_fetched_as_fast(M, K, N, rows, tmp_path):
    text, info = _generated(synth.uniform_csr(M, K, 0.879 if M == 80 else 0.9, 4), N, tmp_path, spec_rows=rows, spec_ksplit=8)
    assert {l.strip().split()[1] for l in text.splitlines() if ".space" in l} == {"0"}
    off = info["spec_code_bytes"] / (8 * info["spec_groups"]) % 8192
    assert 6100 < off < 7900 or off < 2048
