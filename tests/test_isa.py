"""The instructions of the built library, where a compiler's choice decides
whether a kernel is right."""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2511_22510_amd import build as B

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
STORE = re.compile(r"\s*(buffer|global|flat|scratch)_store_dwordx[34]\s+(.*)")


def _registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]", operand) or re.match(r"([va])(\d+)()", operand)
    return {(m[1], i) for i in range(int(m[2]), int(m[3] or m[2]) + 1)} if m else set()


def _overwritten(lines):
    """(wide stores, those with a scalar offset, those whose data an instruction
    writes in the two wait states behind them)."""
    stores, scalar, late, open_ = 0, [], [], []
    kernel = ""
    for line in lines:
        if line.endswith(">:\n"):
            kernel, open_ = line.strip(), []
        is_store = "_store_dwordx" in line
        if not (is_store or open_):
            continue
        text = line.split("//")[0].strip()
        name, _, rest = text.partition(" ")
        if not rest and not name.startswith("s_"):
            continue
        ops = [o.strip() for o in rest.split(",")]
        if name.startswith(("s_endpgm", "s_branch", "s_setpc")):   # what follows is reached from elsewhere
            open_ = []
            continue
        if name.startswith("v_"):
            late += [(kernel, s, text) for s, data, _ in open_ if data & _registers(ops[0])]
        waits = 1 + (int(ops[0], 0) if name == "s_nop" else 0)
        open_ = [(s, d, w + waits) for s, d, w in open_ if w + waits < 2]
        m = STORE.match(line) if is_store else None
        if m:
            stores += 1
            if m[1] == "buffer" and re.match(r"s\d+", ops[3]):
                scalar.append((kernel, text))
            open_.append((text, _registers(ops[0] if m[1] == "buffer" else ops[1]), 0))
    return stores, scalar, late


def test_scan_sees_an_overwritten_store():
    bad = ["<k>:\n", "\tbuffer_store_dwordx4 v[10:13], v125, s[28:31], s0 offen // 0\n", "\tv_cndmask_b32_e64 v11, v37, 0, s[2:3] // 0\n"]
    assert _overwritten(bad)[0] == 1 and len(_overwritten(bad)[1]) == 1 and len(_overwritten(bad)[2]) == 1
    good = ["<k>:\n", "\tbuffer_store_dwordx4 v[10:13], v125, s[28:31], 0 offen // 0\n", "\ts_nop 1 // 0\n", bad[2]]
    assert _overwritten(good) == (1, [], [])


def test_wide_stores_keep_their_data(tmp_path):
    """A store wider than 64 bits reads its data registers after its issue: two
    wait states lie between it and an instruction that writes them.  (The
    compiler leaves them out for buffer stores with a scalar offset.)"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(B.OUT):
        B.build()
    lib = tmp_path / "lib.so"
    lib.symlink_to(B.OUT)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL)
    objects = [str(f) for f in sorted(tmp_path.glob("lib.so.*gfx950"))]
    assert objects

    def scan(path):
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], stdout=subprocess.PIPE,
                              text=True) as p:
            found = _overwritten(p.stdout)
        assert p.returncode == 0
        return found

    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        found = list(ex.map(scan, objects))
    assert sum(f[0] for f in found) > 1000
    assert not [x for f in found for x in f[1]]
    assert not [x for f in found for x in f[2]]
