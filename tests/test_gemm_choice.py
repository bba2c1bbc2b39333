"""The choices that the launchers make on the host (csrc/nm_gemm_choice.h, csrc/nm_rows_choice.h): the values of the debug
switch NM_GEMM_CFG and what each configuration requires of a product, and the rows that one launch of the LayerNorm kernel
can hold, in a C++ driver of its own (CPU); and products under a forced configuration whose requirements they do not meet,
against the oracle (GPU)."""
import os
import shutil
import subprocess
import sys

import pytest

from test_gpu_conv import CHAIN_CASES, CHAIN_LINES_CASES, LARGE_TILE_CASES
from test_gpu_parity import STAGED_CASES
from test_sanitizers import SAN, _run

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_choices_on_the_host(tmp_path):
    exe = str(tmp_path / "choice_driver")
    _run(["g++", "-std=c++17", *SAN, "-Wall", "-Werror", "-I", "paper_2305_14405_amd/csrc", "tests/sanitize/choice_driver.cpp", "-o", exe], exe)


def _configurations(tmp_path, kind, products):
    exe = str(tmp_path / "choice_driver")
    _run(["g++", "-std=c++17", *SAN, "-Wall", "-Werror", "-I", "paper_2305_14405_amd/csrc", "tests/sanitize/choice_driver.cpp", "-o", exe], exe)
    out = subprocess.run([exe, kind, *(str(v) for p in products for v in p)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.endswith("SANITIZE_OK\n"), out.stdout + out.stderr
    return [int(v) for v in out.stdout.split()[:-1]]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_large_convolutions_reach_every_configuration(tmp_path):
    """The cases that compare the tile kernel's epilogues for convolutions with the oracle do take that kernel, and between them
    each of its configurations, with rows gathered from the image and with plain ones."""
    products = []
    for B, H, W, Cin, Cout, k, stride, pad, tile in LARGE_TILE_CASES:
        Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
        products.append((B * Ho * Wo, Cout, k * k * Cin, Cin))
    assert _configurations(tmp_path, "relu", products) == [c[8] for c in LARGE_TILE_CASES]
    reached = {(c[8], c[5] > 1 or c[6] > 1) for c in LARGE_TILE_CASES}
    assert reached == {(tile, gathered) for tile in (2, 5, 6, 7, 8, 9, 10, 11) for gathered in (False, True)}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_staged_products_reach_every_configuration(tmp_path):
    """Likewise the register-staged kernel's cases: each configuration with operands aligned to 16, 4 and 1 bytes."""
    products = [(M, N, K, 16 if K % 16 == 0 else 4 if K % 4 == 0 else 1) for M, N, K, tile in STAGED_CASES]
    assert _configurations(tmp_path, "staged", products) == [c[3] for c in STAGED_CASES]
    reached = {(c[3], p[3]) for c, p in zip(STAGED_CASES, products) if c[3] >= 0}
    assert reached == {(tile, align) for tile in range(4) for align in (16, 4, 1)}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_chained_convolutions_are_one_kernel(tmp_path):
    """The cases that compare two chained convolutions with the steps by themselves are one kernel, each of those built among them; few
    positions, a second turn that is nearly empty and channels that it is not built for are not."""
    assert _configurations(tmp_path, "chain", CHAIN_CASES) == [1] * len(CHAIN_CASES)
    assert {(K, N2) for M, K, N1, N2 in CHAIN_CASES} == {(64, 64), (64, 128), (128, 128)}
    others = [(300, 64, 256, 64), (33000, 64, 256, 64), (70000, 128, 512, 128), (50003, 128, 512, 64), (50003, 64, 320, 64), (50003, 64, 256, 256), (50003, 128, 1024, 128)]
    assert _configurations(tmp_path, "chain", others) == [0] * len(others)
    # tables that are no ReLU: later, by measured times
    assert _configurations(tmp_path, "chain_lines", CHAIN_LINES_CASES) == [1] * len(CHAIN_LINES_CASES)
    slower = [(5000, 64, 256, 64), (8000, 64, 256, 64), (36000, 64, 256, 64), (5000, 64, 256, 128), (20000, 64, 512, 64), (131072, 64, 512, 64), (45000, 64, 768, 64)]
    assert _configurations(tmp_path, "chain_lines", slower) == [0] * len(slower)


# A program of its own: the switch is read once per process.
PRODUCT = """
import sys, numpy as np, torch
from oracle import oracle as O
from paper_2305_14405_amd import binding as nm
M, N, K, nseg, per_column = (int(v) for v in sys.argv[1:])
g = np.random.default_rng(M + N + K)
A, W = (g.integers(-127, 128, s, dtype=np.int64).astype(np.int8) for s in ((M, K), (N, K)))
bias = g.standard_normal(N).astype(np.float32)
alpha = np.full(N, 3.0 / (70 * 70 * np.sqrt(K)), np.float32) * (1 + g.random(N)).astype(np.float32) if per_column else None
scale = float(np.float32(3.0 / (70 * 70 * np.sqrt(K))))
dev = lambda a: None if a is None else torch.from_numpy(a).to("cuda:0")
ot = O.build_table(O.F_GELU, -8.0, 8.0, nseg) if nseg else None
dt = nm.nm_tables_from_arrays([("gelu", -8.0, 8.0, nseg, 0)], [ot.k], [ot.b]) if nseg else None
q = torch.full((M, N), 77, dtype=torch.int8, device="cuda:0")
args = [dev(A), dev(W), dev(bias), dev(alpha)]
nm.nm_gemm_pwl(args[0], args[1], bias=args[2], alpha=scale, alpha_vec=args[3], tables=dt, table_idx=0 if nseg else -1, out_inv_scale=30.0, out_q=q)
torch.cuda.synchronize()
want = O.gemm_pwl(A, W, bias=bias, alpha=scale, alpha_vec=alpha, table=ot, out_inv_scale=30.0)
assert np.array_equal(q.cpu().numpy(), want["q"])
print("PRODUCT_OK")
"""


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,M,N,K,nseg,per_column", [
    ("tile3", 1500, 768, 384, 0, 0),      # three slices, a ring of three stages: one slice too few
    ("relu11", 1200, 912, 192, 0, 1),     # slices of 128 bytes, one and a half of them
    ("direct0", 64, 128, 3072, 4096, 0),  # rings and table together beyond LDS
    ("tile3", 1500, 768, 512, 64, 0),   # one that the configuration does take
    # tables that slots do not take
    ("tile0", 700, 1024, 272, 1500, 0), ("tile1", 700, 1008, 384, 300, 0), ("tile4", 500, 1008, 384, 600, 0), ("tile8", 300, 1008, 304, 2100, 0),
    # K in whole chunks but not whole slices, every remainder
    ("tile0", 700, 1024, 272, 128, 0), ("tile1", 700, 1008, 416, 0, 0), ("tile2", 700, 1008, 688, 64, 0), ("tile3", 500, 1008, 576, 0, 0),
    ("tile4", 500, 1008, 336, 100, 0), ("tile5", 500, 1008, 752, 0, 0), ("tile6", 500, 1008, 480, 64, 0), ("tile7", 300, 1008, 400, 300, 0),
    ("tile8", 300, 1008, 304, 0, 0), ("direct0", 100, 260, 400, 64, 0), ("direct3", 100, 260, 80, 0, 0), ("direct5", 100, 260, 1104, 64, 0)])
def test_forced_configuration_keeps_results(cfg, M, N, K, nseg, per_column):
    run = subprocess.run([sys.executable, "-c", PRODUCT, *map(str, (M, N, K, nseg, per_column))], capture_output=True, text=True, cwd=ROOT,
                         env=dict(os.environ, NM_GEMM_CFG=cfg, PYTHONPATH=ROOT), timeout=100)
    assert run.returncode == 0 and "PRODUCT_OK" in run.stdout, (run.stdout[-1000:], run.stderr[-3000:])


# The kernels of one layer, counted as the nodes of its captured graph, and its result.
LAYER = """
import ctypes, hashlib, torch
from paper_2305_14405_amd import binding as nm
import workloads as W
DEV = "cuda:0"
tables = nm.nm_build_tables([("gelu", -8.0, 8.0, 64), ("exp", -16.0, 0.0, 64), ("recip", 1.0, 128.0, 64), ("rsqrt", 1e-3, 64.0, 64)])
g = torch.Generator(device=DEV).manual_seed(3)
codes = lambda *s: torch.randint(-100, 101, s, generator=g, device=DEV).to(torch.int8)
real = lambda n, m=0.0: torch.randn(n, generator=g, device=DEV) * 0.1 + m
hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
s = torch.cuda.Stream()
for B, S, H in ((24, 128, 512), (1, 128, 768), (1, 64, 128)):   # the QKV projection with attention, a LayerNorm with FFN1, a narrow layer's block kernel
    act = dict(q=0.1, k=0.1, v=0.1, p=1.0 / 127, ctx=0.05, ln1=5.0 / 127, ffn1=0.1, out=5.0 / 127)
    p = W.with_scales(dict(B=B, S=S, H=H, heads=H // 64, F=4 * H, s_x=5.0 / 127, s_wqkv=1e-3, s_wo=1e-3, s_w1=1e-3, s_w2=1e-3, eps1=1e-5, eps2=1e-5), act)
    F = 4 * H
    w = dict(Wqkv=codes(3 * H, H), bqkv=real(3 * H), Wo=codes(H, H), bo=real(H), W1=codes(F, H), b1=real(F), W2=codes(H, F), b2=real(H),
             gamma1=real(H, 1.0), beta1=real(H), gamma2=real(H, 1.0), beta2=real(H))
    desc = nm.make_layer_desc(p, w, tables)
    x, y = codes(B * S, H), torch.empty((B * S, H), dtype=torch.int8, device=DEV)
    ws = torch.empty(nm.nm_encoder_layer_workspace(desc), dtype=torch.uint8, device=DEV)
    nm.nm_encoder_layer(desc, x, y, None, ws)
    torch.cuda.synchronize()
    graph, nodes, stream = ctypes.c_void_p(), ctypes.c_size_t(), ctypes.c_void_p(s.cuda_stream)
    assert hip.hipStreamBeginCapture(stream, 1) == 0   # (thread local)
    nm.nm_encoder_layer(desc, x, y, None, ws, stream=s)
    assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0 and hip.hipGraphDestroy(graph) == 0
    print(nodes.value, hashlib.md5(y.cpu().numpy().tobytes()).hexdigest())
"""


@pytest.mark.gpu
def test_switches_reach_the_products_that_layers_fuse():
    """With either debug switch a layer's products are kernels of their own, seven of them, and its result is the same."""
    def run(**switch):
        out = subprocess.run([sys.executable, "-c", LAYER], capture_output=True, text=True, cwd=ROOT, env=dict(os.environ, PYTHONPATH=ROOT, **switch), timeout=100)
        assert out.returncode == 0, out.stdout + out.stderr
        return [line.split() for line in out.stdout.splitlines()[-3:]]
    plain = run()
    assert [n for n, _ in plain] == ["6", "6", "3"]
    for switch in (dict(NM_GEMM_GENERIC="1"), dict(NM_GEMM_CFG="direct1")):
        assert run(**switch) == [["7", result] for _, result in plain]
