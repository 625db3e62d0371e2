"""Register budgets that the comments of the kernels rely on, read from the metadata of the built library: a kernel that
needs more runs fewer wavefronts per SIMD, without any other sign of it."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2203_17189_amd as P

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (registers, spilled vector registers)} of every gfx950 code object in the library."""
    data = open(os.path.join(os.path.dirname(P.__file__), "libt5mi.so"), "rb").read()
    out, tmp = {}, tmp_path_factory.mktemp("code_objects")
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        q = m.start() + 32
        for i in range(struct.unpack_from("<Q", data, m.start() + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, q)
            target = data[q + 24:q + 24 + n]
            q += 24 + n
            if b"gfx950" not in target or not size:
                continue
            elf = tmp / f"{m.start()}_{i}.elf"
            elf.write_bytes(data[m.start() + off:m.start() + off + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
            for k in notes.split("- .agpr_count:")[1:]:
                f = {x: re.search(rf"\.{x}:\s+(\S+)", k).group(1) for x in ("name", "vgpr_count", "vgpr_spill_count")}
                out[f["name"]] = (int(f["vgpr_count"]), int(f["vgpr_spill_count"]))
    assert len(out) > 100
    return out


# kernel and template arguments (pattern of the mangled name), wavefronts per SIMD that its 512 registers must allow;
# none of these spills more than two registers
WAVES = [("attn_fwd_f32_kernelILi32ELi[124]ELb1", 3), ("attn_fwd_f32_kernelILi64ELi[124]ELb1", 2),
         ("attn_bwd_(dq|dkv)_f32_kernelILi(32ELi[124]|64ELi4)E", 2),
         ("attn_(fwd|bwd_dq|bwd_dkv)_f32_kernelILi(32|64)E", 1),
         ("attn_bwd_dkv_mfma_kernelILi64ELb0ELb0ELb0ELb1E", 3), ("attn_bwd_dkv_mfma_kernelILi64E", 2),
         ("attn_bwd_dq_mfma_kernelILi64ELb[01]ELb[01]ELb0E", 3), ("attn_fwd_mfma_kernel", 2),
         # dropout: three with the causal mask and the window of diagonals, else two
         ("attn_bwd_dq_mfma_kernelILi64ELb1ELb1ELb1ELb1E", 3), ("attn_bwd_dq_mfma_kernel", 2),
         ("attn_bwd_dkv_pipe_kernelILi64E", 2), ("attn_bwd_dkv_pipe_kernel", 1)]


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
@pytest.mark.parametrize("name,waves", WAVES, ids=lambda v: str(v))
def test_wavefronts_per_simd(kernels, name, waves):
    found = {k: v for k, v in kernels.items() if re.search(name, k)}
    assert found
    for k, (regs, spilled) in found.items():
        assert 512 // (-(-regs // 8) * 8) >= waves and spilled <= 2, (k, regs, spilled)
