"""Properties of the compiled kernels that no result shows: the gfx950 code inside the built library is disassembled (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> list of (mnemonic, operands), of all kernels whose mangled name matches the pattern asked for"""
    from paper_2507_14811_amd import binding, build

    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(binding.LIB_PATH):
        build.build_library(verbose=False)
    d = tmp_path_factory.mktemp("code")
    shutil.copy(binding.LIB_PATH, d / "l.so")
    subprocess.run([OBJDUMP, "--offloading", "l.so"], cwd=d, check=True, stdout=subprocess.DEVNULL)
    objects = sorted(d.glob("l.so.*gfx950*"))
    assert objects

    def select(pattern):
        out = {}
        for o in objects:
            names = [n for n in subprocess.run([OBJDUMP, "-t", str(o)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
                     if re.search(pattern, n) and "." not in n]
            if not names:
                continue
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), str(o)], check=True,
                                  stdout=subprocess.PIPE, text=True).stdout
            for m in re.finditer(r"^[0-9a-f]+ <(_Z\w+)>:\n(.*?)(?=^\s*$|\Z)", text, re.S | re.M):
                out[m.group(1)] = [tuple((line.split("//")[0].split(None, 1) + [""])[:2]) for line in m.group(2).splitlines() if line.strip()]
        return out

    return select


def test_up_projection_requests_all_before_it_waits(kernels):
    """With y_q: the wave's share of Lu, its T values and sixteen pieces of y_q are requested in this order before the first wait, and nothing up to the
    barrier waits for y_q (the wait for Lu counts on exactly sixteen younger loads)."""
    built = set()
    for name, code in kernels("lowrank_up_kernel").items():
        bf16, rank, cpl, mode, yq = map(int, re.search(r"Lb([01])ELi(\d+)ELi(\d)ELNS_6LrModeE(\d)ELb([01])E", name).groups())
        first = max(i for i, (op, _) in enumerate(code) if op == "global_load_lds_dwordx4") + 1
        loads, waits = [], []
        for op, args in code[first:]:
            if op == "s_barrier":
                break
            if op.startswith("global_load"):
                loads.append((op, len(waits)))
            if op == "s_waitcnt" and "vmcnt" in args:
                waits.append(int(re.search(r"vmcnt\((\d+)\)", args).group(1)))
        assert [n for _, n in loads] == [0] * len(loads), (name, "a load behind a wait")
        assert [op for op, _ in loads[:rank // 8]] == ["global_load_dwordx4"] * (rank // 8), name
        assert [op for op, _ in loads[rank // 8:]] == ["global_load_dwordx%d" % cpl] * (16 if yq else 0), name
        assert min(waits) == (16 if yq else 0), (name, waits)
        built.add((bf16, cpl, mode, yq))
    # those that the launch chooses from: past the caches on four columns per lane and with a y_q only, bf16 y never y_q alone
    assert built == {(b, *k) for b in (0, 1) for k in ((4, 2, 1), (4, 0, 1), (2, 0, 1), (4, 0, 0), (2, 0, 0))} | {(0, 4, 1, 1)}


def test_raw_sums_are_stored_sixteen_bytes_at_a_time(kernels):
    """Tile kernel, one K-segment: per 32 x 32 block four 16-byte stores of fp32 and two of bf16 results, whole tiles and ragged ones, and twice four
    of the raw sums."""
    seen = 0
    for name, code in kernels(r"seglinear_mfma_kernelI(Li\d+E){7}Lb[01]ELb0E").items():
        bm, bn, wm, wn = map(int, re.search(r"kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name).groups())
        blocks = (bm // wm // 32) * (bn // wn // 32)
        assert sum(op == "global_store_dwordx4" for op, _ in code) >= 20 * blocks, name
        seen += 1
    assert seen >= 17                                      # nine tiles, eight of them with a polarity split


def test_tile_constants_come_sixteen_bytes_at_a_time(kernels):
    """Tile kernel, several K-segments: a block column's scales are four 16-byte loads wherever the tile lies, in the flush between K-segments (two
    copies where one polarity-split segment shares its registers) as in the last one, which has the biases too, for fp32 and for bf16.
    Eight waves with a running sum next to two accumulator sets alone leave the ragged tiles between K-segments to single loads."""
    seen = 0
    for name, code in kernels(r"seglinear_mfma_kernelILi(64ELi(128|192)E|128ELi256ELi2ELi4E)(Li\d+E)*Lb[01]ELb1ELb[01]ELb0ELb0E").items():
        bn, wn = (int(re.findall(r"Li(\d+)E", name)[i]) for i in (1, 3))
        dual, _, share = (f == "1" for f in re.findall(r"Lb([01])E", name)[:3])
        mid = 16 if share else 4 if dual and wn == 4 else 8
        assert sum(op == "global_load_dwordx4" for op, _ in code) == (32 + mid) * (bn // wn // 32), name
        seen += 1
    assert seen == 9


def test_refilling_k_loop_waits_for_its_ring_only(kernels):
    """Tile kernel, rings of three stages and more, per-token steps: between the barrier of a stage and the end of the loop nothing waits for a
    vector load (a wait for one of the flush's own would drain the ring in every stage)."""
    loops = 0
    for name, code in kernels(r"seglinear_mfma_kernelI(Li\d+E){4}Li[34]E(Li\d+E)*(Lb[01]E){3}Lb1ELb0E").items():
        for i, (op, _) in enumerate(code):
            if op != "s_barrier":
                continue
            end = next(j for j in range(i, len(code)) if code[j][0].startswith("s_cbranch"))
            body = code[i:end]
            if sum(op == "global_load_lds_dwordx4" for op, _ in body) >= 6 and sum(op.startswith("v_mfma") for op, _ in body) >= 8:
                loops += 1
                assert not [a for op, a in body if op == "s_waitcnt" and re.search(r"vmcnt\((?!63)", a)], name
    assert loops >= 5 * 4


def test_three_column_pieces_are_stored_as_three(kernels):
    """Tiles of 192 columns taken in turn: a lane's three columns (bf16: six of two rows' three) go out as twelve bytes; as the compiler's sixteen
    they would run into the next lane's."""
    seen = 0
    for name, code in kernels("seglinear_pair_kernelILi192E").items():
        stores = [op for op, _ in code if op.startswith("global_store_dword")]
        assert "global_store_dwordx3" in stores and "global_store_dwordx4" not in stores, name
        seen += 1
    assert seen == 6
