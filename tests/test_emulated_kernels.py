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
    if name == "solve_linear":
        text = ring_in_c(text)
        # (the lanes of a row read the step together, before one of them marks it)
        text = replaced(text, r"        const int step = nxt\[cur\];\n", "        const int step = nxt[cur];\n        (void)emu::ballot(true);\n")
        linear_headers(tmp_path)
    assert "asm" not in text
    (tmp_path / (name + ".cpp")).write_text(text)
    header = open(os.path.join(CSRC, "ckpt_internal.h")).read()
    header = replaced(header, r"\.\./\.\./include/ckpt\.h", os.path.join(ROOT, "include", "ckpt.h"))
    header = replaced(header, r"    asm\(\"s_nop 1.*?\"\+v\"\(v\)\);\n    return [^;]*;", "    return emu::min_u32(v);")
    (tmp_path / "ckpt_internal.h").write_text(header)
    return str(tmp_path / (name + ".cpp"))


def ring_in_c(text):
    """linear_ring_wave's assembly as what it does, lane by lane (its ballots only ask whether any lane goes on, and what
    it moves to scalar registers is the same in all lanes); the assembly itself is for the GPU tests."""
    begin, end = text.index("__device__ __forceinline__ void linear_ring_wave"), text.index("__global__ __launch_bounds__(kWave) void linear_ring_kernel")
    ring = text[begin:end].replace("__builtin_amdgcn_readfirstlane", "")
    ring = replaced(ring, r"__builtin_amdgcn_ballot_w64\(low != 0\) != 0", "low != 0")
    ring = replaced(ring, r"__builtin_amdgcn_ballot_w64\(p3\) != 0", "p3")
    ring = replaced(ring, r"__attribute__\(\(address_space\(3\)\)\) uint32_t \*LdsPtr", "uint32_t *LdsPtr")
    ring = replaced(ring, r"    const uint32_t lane_base =[^;]*;\n", "")
    ring = replaced(ring, r"return \(LdsPtr\)\(uintptr_t\)[^;]*;", "return &ring[kPlaneM][(pos & kSlotMask) / kStep][lane];")
    ring = replaced(ring, r"            uint32_t ad, e, t0;\n            uint64_t sv, sv2, sv3;\n            asm volatile\(.*?\);  // \(s_and_saveexec writes SCC\)", """
            for (int moves = 0; Ti + Rc >= Ac; ++moves) {
                if (moves > kRing) emu::stop("the crossover runs around the ring");
                pt += kStep;
                Tpt = Ac - Mc; Jpt = Jc; Rp = Rc;
                Mc = Ac = kNone;
                if (pt == hd) continue;
                const LdsPtr candidate = entry(pt + kStep);
                Mc = candidate[0]; Ac = candidate[kA]; Jc = candidate[kGJ];
                const uint32_t above = (hd - pt) / kStep - 1, mirrors[] = {Ghd, G1, G2, G3};
                Rc = di8;
                for (uint32_t k = 0; k < above; ++k) Rc = max(Rc, k < 4 ? mirrors[k] : entry(hd - k * kStep)[kGJ]);
                Rc >>= 8;
            }""")
    ring = replaced(ring, r"                uint32_t ad;\n                uint64_t sv;\n                asm volatile\(.*?\);  // \(s_and_saveexec writes SCC\)", """
                for (int drops = 0; Mhd >= Mi; ++drops) {
                    if (drops > kRing) emu::stop("the queue runs around the ring");
                    Gacc = max(Gacc, Ghd);
                    hd -= kStep;
                    Mhd = entry(hd)[0]; Ghd = entry(hd)[kGJ];
                }""")
    ring = replaced(ring, r"asm volatile\(\"s_nop 4[^;]*;", "mp[(int64_t)i * pstride] = (uint8_t)step; (void)rowbase;")
    ring = replaced(ring, r"    asm volatile\(\"s_waitcnt[^;]*;\n", "")
    text = text[:begin] + ring + text[end:]
    return replaced(text, r"typedef uint32_t u32x32 [^;]*;", "typedef std::array<uint32_t, 32> u32x32;")


def linear_headers(tmp_path):
    wave = open(os.path.join(CSRC, "linear_wave.h")).read()
    wave = replaced(wave, r'extern "C" __device__ int ckpt_write_lane[^;]*;',
                    "inline int ckpt_write_lane(int v, int lane, int old) { return emu::lane() == lane ? v : old; }")
    wave = replaced(wave, r'    double r;\n    asm\("v_max_f64[^;]*;\n    return r;', "    return a > b ? a : b;")
    wave = replaced(wave, r'    double r;\n    asm\("v_min_f64[^;]*;\n    return r;', "    return a < b ? a : b;")
    rows = open(os.path.join(CSRC, "linear_rows.h")).read()
    rows = replaced(rows, r'extern "C" __device__ double ckpt_update_dpp\(.*?;',
                    "inline double ckpt_update_dpp(double old, double v, int control, int rows, int, bool) { return emu::dpp(old, v, control, rows); }")
    assert "asm" not in wave + rows
    (tmp_path / "linear_wave.h").write_text(wave)
    (tmp_path / "linear_rows.h").write_text(rows)


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


def test_the_search_with_a_row_of_lanes_per_chain_on_the_cpu(tmp_path):
    source("cubic_search", tmp_path)
    run_driver("rows_driver", [], tmp_path)


def test_the_linear_solver_on_the_cpu(tmp_path):
    source("solve_linear", tmp_path)  # (the driver includes it, and launches the forms one by one)
    run_driver("linear_driver", [], tmp_path)


def test_the_evaluations_on_the_cpu(tmp_path):
    run_driver("eval_driver", [source("eval_peak", tmp_path), source("eval_timeline", tmp_path)], tmp_path)
