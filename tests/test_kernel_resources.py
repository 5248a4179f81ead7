"""Register budget of the built kernels, read from the metadata the compiler
wrote into the library: no kernel keeps anything in scratch memory or spills a
vector register.  A reload from scratch waits for every vector memory access in
flight, the update's parameter loads and stores among them."""
import os
import re
import subprocess

import bench
from paper_2606_27153_amd.build import LIB_PATH

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def _kernels(tmp_path):
    with open(LIB_PATH, "rb") as f:
        lib = f.read()
    out = {}
    # the device code objects are ELF images (machine type AMDGPU, 224) inside the host library
    for at in (m.start() for m in re.finditer(b"\x7fELF", lib)):
        if int.from_bytes(lib[at + 18:at + 20], "little") != 224:
            continue
        path = tmp_path / f"{at}.co"
        path.write_bytes(lib[at:])
        notes = subprocess.run([READELF, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
        for part in notes.split(".agpr_count:")[1:]:   # the first key of each kernel's map
            name = re.search(r"\.name: +(\S+)", part.split(".private_segment_fixed_size:")[0].split(".max_flat")[-1])
            val = {k: int(re.search(rf"\.{k}: +(\d+)", part).group(1))
                   for k in ("private_segment_fixed_size", "vgpr_spill_count", "vgpr_count")}
            out[name.group(1)] = val
    return out


def test_no_kernel_spills(tmp_path):
    kernels = _kernels(tmp_path)
    assert sum("ns_gemm_kernel" in k for k in kernels) == 16     # two operand types, four stages, plain and PAD
    assert any("ns_tile_kernel" in k for k in kernels) and any("momentum_kernel" in k for k in kernels)
    bad = {k: v for k, v in kernels.items() if v["private_segment_fixed_size"] or v["vgpr_spill_count"]}
    assert not bad, bad


def test_profile_summaries_name_every_kernel(tmp_path):
    # the summaries' names of the kernels come from their mangled names
    keys = {k: bench.kernel_key(k) for k in _kernels(tmp_path)}
    assert not {k for k, v in keys.items() if v.startswith("other")}, keys
    assert sorted(v for k, v in keys.items() if "ns_gemm_kernel" in k) == sorted(
        2 * [f"{s}:{e}_t256" for s in ("gram", "poly", "bx", "symm") for e in ("bf16", "f16")])
