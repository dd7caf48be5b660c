"""What hand-written waits assume about the compiled kernels, read from the library that was built here: a count of loads in flight is
right only while the compiler issues exactly those loads, in that order."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_10443_amd import binding as B
from paper_2506_10443_amd.build import hipcc

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))), "lib", "llvm", "bin")
if not os.path.isdir(LLVM):
    LLVM = "/opt/rocm/llvm/bin"


def _run(*cmd, cwd=None):
    return subprocess.run(cmd, check=True, capture_output=True, text=True, cwd=cwd).stdout


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """Instructions of the kernels whose mangled name matches a pattern: {name: [instruction, ...]}."""
    if not os.path.exists(B.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    where = tmp_path_factory.mktemp("objects")
    shutil.copy(B.LIB_PATH, where / "lib.so")
    _run(os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so", cwd=where)      # (writes the parts beside the file)
    objects = [str(where / f) for f in sorted(os.listdir(where)) if f.endswith("gfx950")]
    symbols = {o: re.findall(r" FUNC .* (_Z\w+)$", _run(os.path.join(LLVM, "llvm-readelf"), "-sW", o), re.M) for o in objects}

    def kernels(pattern):
        out = {}
        for o, names in symbols.items():
            names = sorted({n for n in names if re.search(pattern, n)})
            if not names:
                continue
            text = _run(os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--no-leading-addr",
                        "--disassemble-symbols=" + ",".join(names), o)
            for name, body in re.findall(r"^<(_Z\w+)>:\n(.*?)(?=^<_Z|\Z)", text, re.S | re.M):
                out[name] = [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
        assert out, pattern
        return out

    def registers(pattern):
        """{name: (vector registers, spilled ones)} of the same kernels."""
        out = {}
        for o in objects:
            notes = _run(os.path.join(LLVM, "llvm-readelf"), "--notes", o)
            for entry in notes.split("  - .agpr_count:")[1:]:
                value = lambda key: re.search(r"\.%s:\s+(\S+)" % key, entry).group(1)
                if re.search(pattern, value("name")):
                    out[value("name")] = (int(value("vgpr_count")), int(value("vgpr_spill_count")))
        assert out, pattern
        return out

    kernels.registers = registers
    return kernels


def test_wide_fp6_ring_counts_its_own_loads(code):
    """prefill6_wide_kernel waits for a stage with vmcnt(39): the 3 direct loads of one stage and the 36 loads of two chunks' weights and
    scales are younger.  The direct loads follow the barrier one after the other, ahead of anything else that the loop loads or contracts,
    and a turn of the loop loads 3 + 18 times."""
    for name, ins in code(r"prefill6_wide_kernel").items():
        at = [i for i, x in enumerate(ins) if x.startswith("s_waitcnt vmcnt(39)")]
        assert len(at) == 1, name
        barrier = next(i for i in range(at[0], len(ins)) if ins[i].startswith("s_barrier"))
        after = [x for x in ins[barrier:] if re.match(r"buffer_load|v_mfma", x)]
        assert all(x.startswith("buffer_load_dwordx4") and x.endswith("lds") for x in after[:3]), (name, after[:4])
        assert not after[3].endswith("lds")
        # the loop: the only backward branch across the barrier
        end = next(i for i in range(barrier, len(ins)) if re.match(r"s_cbranch|s_branch", ins[i]))
        first = max(i for i in range(barrier) if re.match(r"s_barrier", ins[i]))
        back = [x for x in ins[first:end] if x.startswith("buffer_load")]
        assert len(back) == 3 + 18, (name, len(back))
        assert sum(x.endswith("lds") for x in back) == 3


def test_last_row_tile_of_few_tokens_requests_nothing(code):
    """few_resident_kernel: ahead of the last barrier (of a workgroup's last row tile) stands a stretch without any load - the launches
    of one row tile per workgroup must not pay for the next one's.  The loop's barrier is the other one."""
    for name, ins in code(r"few_resident_kernel").items():
        barriers = [i for i, x in enumerate(ins) if x.startswith("s_barrier")]
        assert len(barriers) == 2, (name, len(barriers))
        loads = [i for i, x in enumerate(ins) if x.startswith("buffer_load")]
        assert loads and max(loads) < barriers[0], (name, max(loads), barriers)


def test_second_pass_over_the_row_reads_nothing(code):
    """Fused one-token kernels with float minima (nibble planes: the packed axis runs over the row twice): behind the barrier of the row's
    maximum the row is read in one place only, the loop for what the registers do not hold.  A second read, for the row's second
    pass, would wait for all weights."""
    for name, ins in code(r"13decode_kernelILi\d+ELi\d+ELi\d+ELi1ELb[01]ELb1E").items():
        barriers = [i for i, x in enumerate(ins) if x.startswith("s_barrier")]
        row = [x for x in ins[barriers[0]:barriers[1]] if "load_dwordx4" in x and not x.endswith(" nt")]
        assert len(row) == 1, (name, row)


def test_registers_follow_the_share_of_a_wave(code):
    """Fused one-token call, sixteen waves per row tile: a kernel for every share of five to ten chunks, none of which spills - a spilled
    scale is stored behind a wait for all weights, which the form is there to avoid."""
    for mode in (B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT):
        for chunks in range(65, 161):
            waves, ks, unroll, prefetch = B.mnnq_plan_debug(2, 1, 48, 128 * chunks, mode)[:4]
            assert (waves, ks, unroll, prefetch) == (16, 16, -(-chunks // 16), 0), chunks
    kernels = code.registers(r"13decode_kernelILi16ELi16ELi([5-9]|10)ELi1ELb0ELb[01]ELb0E")
    assert len(kernels) == 12
    for name, (vector, spilled) in kernels.items():
        assert spilled == 0 and vector <= 128, (name, vector, spilled)
