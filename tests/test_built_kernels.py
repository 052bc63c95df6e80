"""What the built library's gfx950 code of the tiled GEMM looks like (no GPU: the disassembly of the code built here)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def tile_kernels(tmp_path_factory):
    """Mangled name -> list of instruction texts, of every gemm_tile_kernel instance."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not found")
    so = os.path.join(ROOT, "paper_2602_01274_amd", "libpacer.so")
    if not os.path.exists(so):
        import __graft_entry__ as g
        g.build()
    tmp = tmp_path_factory.mktemp("isa")
    shutil.copy(so, tmp / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    obj = next(f for f in os.listdir(tmp) if f.endswith("gfx950"))
    out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], cwd=tmp, check=True, capture_output=True, text=True).stdout
    kernels, cur = {}, None
    for line in out.splitlines():
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            cur = kernels.setdefault(m[1], []) if "gemm_tile_kernel" in m[1] else None
        elif cur is not None and line.strip():
            cur.append(line.split("//")[0].strip())
    assert len(kernels) > 30
    return kernels


def test_weights_that_one_block_reads_pass_the_cache(tile_kernels):
    """Up to 32 rows a weight byte belongs to one block, and its load is non-temporal: loaded as data to keep, the weights
    displace from L2 what the next kernels read (attention at 20 rows, 700 keys 12.4 us against 9.0, embedding 7.7 against 5.8).
    With several row groups the blocks share weights through L2, and no load is."""
    for name, ins in tile_kernels.items():
        rt = int(re.search(r"gemm_tile_kernelILi\d+ELi(\d+)E", name)[1])
        loads = [i for i in ins if i.startswith("global_load_lds")]
        nt = [i for i in loads if i.endswith(" nt")]
        assert loads and (0 < len(nt) < len(loads) if rt == 2 else not nt), name


def test_direct_loads_take_m0_from_the_compiler(tile_kernels):
    """The loads into LDS take their LDS address from m0.  No asm text writes that register behind the compiler's back: it is
    an operand, so each load has an instruction of the compiler's before it that sets m0, and the wait state."""
    csrc = os.path.join(ROOT, "paper_2602_01274_amd", "csrc")
    for f in os.listdir(csrc):
        for text in re.findall(r'"((?:[^"\\]|\\.)*)"', open(os.path.join(csrc, f)).read()):
            assert not re.search(r"\bs_\w+ m0\b", text), (f, text)
    for name, ins in tile_kernels.items():
        fresh = False                                  # m0 set since the last load
        for prev, x in zip(ins, ins[1:]):
            fresh = fresh or bool(re.match(r"s_\w+ m0, ", x))
            if x.startswith("global_load_lds"):
                assert fresh and prev == "s_nop 0", name
                fresh = False
