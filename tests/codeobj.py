"""What the compiler recorded for the kernels of the built library (the metadata
of the code objects in libuot.so): static LDS, registers, spills."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1607_05816_amd", "libuot.so")
LLVM = "/opt/rocm/llvm/bin"


def available():
    return os.path.exists(LIB) and os.path.exists(LLVM + "/llvm-readelf")


def kernels(tmp_path):
    """symbol -> dict(lds, vgprs, spilled); vgprs: accumulation registers included."""
    fat, obj = str(tmp_path / "fat"), str(tmp_path / "obj")
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, LIB, str(tmp_path / "copy")],
                   check=True)
    with open(fat, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(b"\x7fELF", data):
        with open(obj, "wb") as f:
            f.write(data[m.start():])
        notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", obj], capture_output=True, text=True).stdout
        for k in notes.split(".agpr_count")[1:]:
            def num(key):
                return int(re.search(r"\.%s:\s+(\d+)" % key, k).group(1))

            out[re.search(r"\.name:\s+(\S+)", k).group(1)] = dict(
                lds=num("group_segment_fixed_size"), vgprs=num("vgpr_count"), spilled=num("vgpr_spill_count"))
    assert out
    return out
