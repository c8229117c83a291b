"""The one-lane operator hands products from site to site through LDS, one
direction after the other through the same array. A lane's read of its
neighbour's product has to come before that neighbour stores the next
direction's: every direction but the last ends with a workgroup barrier, or
with a wavefront one where the products stay in the wavefront (4^4 blocks).
Without it the result hangs on the order in which the compiler happens to emit
a load and a store of different lanes, so the unoptimised code is looked at.
"""
import os
import re
import subprocess

from paper_1204_5463_amd import build as B


def _functions(tmp_path):
    out = tmp_path / "k_dslash.ll"
    flags = [f for f in B.COMMON if f not in ("-O3", "-fPIC")]
    subprocess.run([B.HIPCC, "-O1"] + flags + ["--cuda-device-only", "-Xclang", "-disable-llvm-passes", "-emit-llvm",
                   "-S", os.path.join(B.CSRC, "k_dslash.hip"), "-o", str(out)], check=True, capture_output=True)
    for m in re.finditer(r"^define [^\n]*@(\w+)\([^\n]*\n(.*?)^\}", out.read_text(), flags=re.M | re.S):
        yield m.group(1), m.group(2)


def test_every_direction_ends_with_a_barrier(tmp_path):
    seen = set()
    for name, body in _functions(tmp_path):
        # dw::(anonymous namespace)::blk_dir<MU, BS, ...> and blk_dir16
        m = re.match(r"_ZN2dw12_GLOBAL__N_1(?:7blk_dir|9blk_dir16)ILi(\d)ELi(\d)E", name)
        if not m:
            continue
        mu, bs = int(m.group(1)), int(m.group(2))
        calls = [c for c in re.findall(r"call [^\n]*@([\w.]+)\(", body) if not c.startswith("llvm.lifetime")]
        wave = "_ZN2dw12_GLOBAL__N_18blk_syncILb1EEEvv"
        group = "_ZN2dw12_GLOBAL__N_18blk_syncILb0EEEvv"
        if mu < 3:
            assert calls[-1] == (wave if bs == 4 else group), name
        seen.add((mu, bs, "blk_dir16" in name))
    assert seen == {(mu, bs, p) for mu in range(4) for bs in (0, 4) for p in (False, True)}
