"""Host-side logic shared with the kernels, compiled with g++ (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rank_order_is_a_permutation(tmp_path):
    exe = str(tmp_path / "order_key_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined",
                           os.path.join(ROOT, "tests", "cpp", "order_key_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr


def test_bench_flop_count_matches_the_step():
    """The bench's algorithmic flop count is the sum of the step's products:
    2N^3 + N^3 (basis change) + 2N^2 M + (q n_it - 1) 2N^3 (folded spectrum) +
    N^3 (overlap) + N^3/3 (Cholesky) + N^3 (triangular solve) + 2N^3 (Rayleigh
    quotients) + 2N^3 (back-rotation) = 19.33 N^3 + 2 N^2 M for q = 2, n_it = 3
    and 13.33 N^3 + 2 N^2 M for q = 1."""
    import importlib.util
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    for n, M in ((8192, 512), (2048, 512), (256, 128)):
        n3 = float(n) ** 3
        assert abs(bench.algorithmic_flops(n, M, 2, 3) - (58.0 / 3.0 * n3 + 2.0 * n * n * M)) <= 1e-9 * n3
        assert abs(bench.algorithmic_flops(n, M, 1, 3) - (40.0 / 3.0 * n3 + 2.0 * n * n * M)) <= 1e-9 * n3
    assert abs(bench.algorithmic_flops(8192, 512, 2, 3) - 1.07e13) <= 0.01e13


def test_pair_solver_lds_handover_has_barriers():
    """The pair solver's Jacobi sweeps and Newton's iteration share their LDS.
    Waves drift apart between barriers, so the hand-over must wait for every
    wave's last reads of the old contents before it writes and for all writes
    before anyone reads, Newton's LDS must be reached in no other way, and the
    sweeps must wait again where Newton's iteration has refused."""
    import re
    src = open(os.path.join(ROOT, "paper_1502_07806_amd", "csrc", "eigh_jacobi.hip")).read()
    src = re.sub(r"//[^\n]*", "", src)
    body = src[src.index("__device__ bool solve_pair("):src.index("__device__ inline void solve_block(")]
    m = re.search(r"auto hand_over = \[&\]\(.*?\) \{\n(.*?)\n  \};\n", body, re.S)
    statements = [t.strip() for t in m.group(1).strip().split("\n") if t.strip()]
    assert statements[0] == "__syncthreads();" and statements[-1] == "__syncthreads();"
    rest = body.replace(m.group(0), "")
    uses = re.findall(r"[^\n]*PL\.newton\b[^\n]*", rest)
    assert len(uses) == 1 and "newton_pair(" in uses[0], uses
    assert re.search(r"newton = false;\s*__syncthreads\(\);", rest)


def test_bench_traffic_belongs_to_the_named_kernel():
    """The FP64 roofline names the folded-spectrum polynomial's whole product and
    takes its HBM bytes from that kernel's entry of the recorded traffic."""
    import json
    import re
    bench = open(os.path.join(ROOT, "bench.py")).read()
    key = re.search(r'EPI_POLY>[^\n]*\n\s*kernel_key = "(\w+)_n%d"', bench).group(1)
    epi = re.search(r"EPI_POLY = (\d+)", open(os.path.join(ROOT, "paper_1502_07806_amd", "csrc", "common.h")).read()).group(1)
    traffic = json.load(open(os.path.join(ROOT, "profiles", "traffic.json")))
    assert traffic[key + "_n8192"]["kernel"].startswith("gemm_f64_dl<true, false, %s," % epi)
