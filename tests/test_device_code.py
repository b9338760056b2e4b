"""Checks of the device code as the compiler sees it, on its LLVM IR (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2602_20217_amd import build as B


def _device_ir(src, tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "device.ll")
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-emit-llvm", "-S",
                    os.path.join(B.CSRC, src), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_lds_loads_in_asm_name_their_array(tmp_path):
    """The compiler places LDS arrays and sees their use through their addresses
    only.  So a global-to-LDS load written as an asm block takes its target from the
    address of an LDS array (a byte offset alone is right only while that array
    lies at 0, and leaves the compiler an array that nothing writes), and holds the
    wait states that the compiler does not insert there: five between a vector
    write of the scalar base and the load, the move to m0 being one of them."""
    ir = _device_ir("attention.hip", tmp_path)
    seen = 0
    for body in re.split(r"^define ", ir, flags=re.M)[1:]:
        defs = dict(re.findall(r"^  (%[\w.]+) = (.*)$", body, flags=re.M))
        for asm, args in re.findall(r'asm sideeffect "([^"]*global_load_lds[^"]*)", "[^"]*"\((.*)\)',
                                    body):
            seen += 1
            assert int(re.search(r"s_nop (\d+)", asm).group(1)) >= 3, asm
            text = args.split(", ", 2)[2]  # the target
            left, done = re.findall(r"%[\w.]+", text), set()
            while left:  # and everything it is computed from
                v = left.pop()
                if v in done:
                    continue
                done.add(v)
                text += defs.get(v, "")
                left += re.findall(r"%[\w.]+", defs.get(v, ""))
            assert "ptrtoint (ptr addrspace(3) @" in text, (asm, args)
    assert seen > 0


def test_split_sums_take_rows_at_any_float_address(tmp_path):
    """Residual rows in and rows or logits out are the caller's, at any float's
    address, whichever way a batched product is split; only the partial sums lie in
    the workspace.  (The GPU tolerates a 16-byte access there, so no result shows a
    kernel that claims 16-byte alignment of them.)"""
    ir = _device_ir("gemm.hip", tmp_path)
    bodies = [b for b in re.split(r"^define ", ir, flags=re.M)[1:]
              if "k_splitk_reduce" in b.split("\n", 1)[0]]
    assert len(bodies) == 2  # plain and with a residual
    for body in bodies:
        body = body.split("\n}", 1)[0]
        stores = re.findall(r"store .* ptr addrspace\(1\) %\S+, align (\d+)", body)
        assert stores and set(stores) == {"4"}, stores
        loads = re.findall(r"= load <4 x float>, ptr addrspace\(1\) %\S+, align (\d+)", body)
        resid = "ILi1E" in body.split("\n", 1)[0]  # EPI_RESID
        assert ("4" in loads) == resid, loads
