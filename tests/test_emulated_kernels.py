"""Kernels of csrc/ built for the CPU, their lanes as fibers (tests/emulate/): whole calls against the oracle, with
pages behind every buffer that cannot be touched; what a wave of the cubic search does with sums that no checked chain
has; LDS limits under two host threads.  Nothing here needs a GPU; that the same kernels run right there is for the
tests marked so."""
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


def run(cmd, **kw):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, **kw)
    assert p.returncode == 0, f"{' '.join(cmd)}\n{p.stdout[-4000:]}"
    return p.stdout


def source(name, tmp_path):
    """csrc/<name>.hip for the CPU: the array that stands for dynamic LDS replaced, and inline assembly."""
    text = open(os.path.join(CSRC, name + ".hip")).read()
    kind, lds = re.search(r"extern __shared__ __align__\(16\) ([\w ]+?) (\w+)\[\];", text).groups()
    text = replaced(text, r"extern __shared__ [^;]*;", f"#define {lds} (({kind} *)emu::dynamic_lds)")
    if name == "cubic_search":
        text = replaced(text, r"    uint32_t r;\n    asm\(\"v_cndmask_b32[^;]*;\n    return r;", "    return (mask >> emu::lane()) & 1 ? on : off;")
    assert "asm" not in text
    (tmp_path / (name + ".cpp")).write_text(text)
    header = open(os.path.join(CSRC, "ckpt_internal.h")).read()
    header = replaced(header, r"\.\./\.\./include/ckpt\.h", os.path.join(ROOT, "include", "ckpt.h"))
    header = replaced(header, r"    asm\(\"s_nop 1.*?\"\+v\"\(v\)\);\n    return [^;]*;", "    return emu::min_u32(v);")
    (tmp_path / "ckpt_internal.h").write_text(header)
    return str(tmp_path / (name + ".cpp"))


def run_driver(driver, sources, tmp_path):
    """The driver under tests/emulate/ with these sources of csrc/ and the oracle."""
    run(["gcc", "-O2", "-fopenmp", "-c", os.path.join(ROOT, "oracle", "ckpt_oracle.c"), "-o", str(tmp_path / "oracle.o")])
    exe = str(tmp_path / driver)
    run(["g++", "-O2", "-std=c++17", "-w", "-fopenmp", "-I", EMULATE, "-I", str(tmp_path), "-o", exe,
         os.path.join(EMULATE, driver + ".cpp"), os.path.join(EMULATE, "fibers.cpp"), *sources, str(tmp_path / "oracle.o")])
    out = run([exe], timeout=300, env=dict(os.environ, OMP_NUM_THREADS="4"))
    assert driver + " ok" in out, out


def test_the_search_on_the_cpu(tmp_path):
    source("cubic_search", tmp_path)  # (the driver includes it: it also calls what has no entry point)
    run_driver("search_driver", [], tmp_path)


def test_the_evaluations_on_the_cpu(tmp_path):
    run_driver("eval_driver", [source("eval_peak", tmp_path), source("eval_timeline", tmp_path)], tmp_path)
