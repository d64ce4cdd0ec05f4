"""csrc/cubic_search.hip built for the CPU, its lanes as fibers (tests/emulate/): what a wave does with sums that
no checked chain has, and whole calls against the oracle, with pages behind every buffer that cannot be touched.
Nothing here needs a GPU; that the same kernels run right there is for the tests marked so."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_12499_amd", "csrc")
EMULATE = os.path.join(ROOT, "tests", "emulate")


def replaced(text, pattern, by, count=1):
    out, found = re.subn(pattern, lambda _: by, text, flags=re.S)
    assert found == count, f"{pattern!r} found {found} times"
    return out


def sources(tmp_path):
    """The header and the kernels with their inline assembly, and the array that stands for dynamic LDS, replaced."""
    header = open(os.path.join(CSRC, "ckpt_internal.h")).read()
    header = replaced(header, r'\.\./\.\./include/ckpt\.h', os.path.join(ROOT, "include", "ckpt.h"))
    header = replaced(header, r'    asm\("s_nop 1.*?"\+v"\(v\)\);\n    return [^;]*;', "    return emu::min_u32(v);")
    (tmp_path / "ckpt_internal.h").write_text(header)
    kernels = open(os.path.join(CSRC, "cubic_search.hip")).read()
    kernels = replaced(kernels, r'extern __shared__ [^;]*search_lds\[\];', "#define search_lds emu::dynamic_lds")
    kernels = replaced(kernels, r'    uint32_t r;\n    asm\("v_cndmask_b32[^;]*;\n    return r;', "    return (mask >> emu::lane()) & 1 ? on : off;")
    assert "asm(" not in kernels and "asm volatile" not in kernels
    (tmp_path / "cubic_search.cpp").write_text(kernels)


def test_the_search_on_the_cpu(tmp_path):
    sources(tmp_path)
    exe = str(tmp_path / "search_driver")
    cmd = ["g++", "-O2", "-std=c++17", "-w", "-fopenmp", "-I", EMULATE, "-I", str(tmp_path), "-o", exe,
           os.path.join(EMULATE, "search_driver.cpp"), os.path.join(EMULATE, "fibers.cpp")]
    subprocess.run(["gcc", "-O2", "-fopenmp", "-c", os.path.join(ROOT, "oracle", "ckpt_oracle.c"), "-o", str(tmp_path / "oracle.o")],
                   check=True)
    subprocess.run(cmd + [str(tmp_path / "oracle.o")], check=True)
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300,
                       env=dict(os.environ, OMP_NUM_THREADS="4"))
    assert p.returncode == 0 and "search_driver ok" in p.stdout, p.stdout[-4000:]
