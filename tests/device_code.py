"""The gfx950 code objects of the built library, for the tests that read
their metadata and assembly (no GPU needed)."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2404_13811_amd", "libmrcm.so")
LLVM = "/opt/rocm/llvm/bin"


def available():
    return os.path.exists(LIB) and all(
        os.path.exists(os.path.join(LLVM, t)) for t in ("llvm-objdump", "llvm-readelf"))


def code_objects(tmp):
    """Paths of the library's code objects, extracted into the folder tmp."""
    so = shutil.copy(LIB, os.path.join(str(tmp), "lib.so"))
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", so], check=True,
                   stdout=subprocess.DEVNULL)
    return sorted(os.path.join(str(tmp), f) for f in os.listdir(str(tmp)) if f.endswith("gfx950"))


def metadata(obj):
    """Text of the code object's notes (the kernels' resource metadata)."""
    return subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], check=True,
                          capture_output=True, text=True).stdout


def assembly(obj):
    """Its instructions, one a line, without addresses and encodings."""
    return subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn",
                           "--no-leading-addr", obj], check=True, capture_output=True, text=True).stdout
