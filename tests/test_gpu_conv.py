"""GPU parity of the convolution path (nm_conv2d_pwl, pooling) and of the residual CNN built
from it, element by element against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest
import torch

from paper_2305_14405_amd import binding as nm
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def relu_tables(oracle):
    ot = oracle.relu_table()
    dt = nm.nm_tables_from_arrays([("relu", -8.0, 8.0, 2, 0)], [ot.k], [ot.b])
    return ot, dt


def rand_i8(g, shape, lim=127):
    return g.integers(-lim, lim + 1, shape, dtype=np.int64).astype(np.int8)


CASES = [  # B, H, W, Cin, Cout, kh, kw, stride, pad   (route)
    (2, 14, 14, 64, 64, 3, 3, 1, 1),      # gathered operand, 64-byte slices, narrow output
    (2, 14, 14, 128, 128, 3, 3, 1, 1),    # gathered operand, 128-byte slices
    (3, 15, 13, 128, 192, 3, 3, 2, 1),    # stride 2, odd sizes, N not a tile multiple
    (2, 16, 16, 256, 512, 1, 1, 2, 0),    # strided 1x1 projection shortcut
    (1, 9, 9, 192, 96, 3, 3, 1, 1),       # Cin % 128 != 0 -> 64-byte slices on the wide tile
    (2, 12, 12, 256, 64, 1, 1, 1, 0),     # plain matrix route, narrow output
    (4, 8, 8, 64, 256, 1, 1, 1, 0),       # plain matrix route
    (2, 20, 20, 3, 64, 7, 7, 2, 3),       # stem: patch matrix in the workspace
    (2, 9, 11, 12, 20, 3, 3, 1, 1),       # odd channel counts: patch matrix, unaligned GEMM
    (1, 5, 5, 64, 64, 5, 5, 1, 2),        # filter as large as the image
    (33, 7, 7, 64, 64, 3, 3, 1, 1),       # many images, tile edge in M
    (2, 11, 11, 64, 48, 3, 3, 1, 1),      # gathered operand, fewer than 64 output channels
    (2, 10, 10, 128, 100, 3, 3, 1, 1),    # output channels not a multiple of 16 (no 16-byte row stores)
    (1, 30, 30, 64, 72, 1, 1, 3, 0),      # stride 3
    (1, 29, 31, 192, 136, 5, 5, 1, 2),    # long filters over few positions: small tiles of eight wavefronts
    (1, 28, 30, 64, 136, 7, 7, 1, 3),     # the same, fewer slices
    (1, 29, 31, 64, 208, 2, 2, 1, 0),     # the other small tiles beyond 16x32: 32x32,
    (3, 29, 31, 64, 400, 2, 2, 1, 0),     # 32x64 with four wavefronts,
    (2, 44, 46, 64, 72, 3, 3, 1, 1),      # with eight,
    (1, 59, 61, 64, 136, 3, 3, 1, 1),     # 48x64
    (2, 44, 46, 64, 400, 2, 2, 1, 0),     # and 64x64
]


@pytest.mark.parametrize("B,H,W,Cin,Cout,kh,kw,stride,pad", [
    (1, 1, 1, 3, 16, 3, 3, 1, 1), (1, 1, 2, 2, 16, 3, 3, 1, 1), (2, 33, 35, 3, 64, 7, 7, 2, 3), (1, 17, 16, 4, 48, 3, 8, 1, 0),
    (3, 50, 61, 1, 16, 4, 5, 4, 2), (1, 40, 19, 2, 32, 9, 2, 3, 5), (2, 5, 5, 3, 64, 1, 3, 2, 0),
    (2, 70, 150, 3, 64, 4, 8, 4, 2), (3, 19, 68, 4, 16, 2, 8, 4, 0), (1, 68, 65, 1, 32, 4, 6, 4, 1),   # stride 4: patches of 68 columns
    # up to 1024 workgroups of 16x16 positions pack the filter themselves, beyond a kernel does
    (256, 17, 20, 3, 16, 3, 3, 1, 1), (257, 17, 20, 3, 16, 3, 3, 1, 1), (1025, 5, 7, 1, 48, 2, 8, 1, 3), (1030, 9, 6, 4, 16, 5, 4, 2, 2),
    (513, 40, 9, 2, 32, 9, 1, 1, 0), (600, 9, 33, 3, 64, 7, 7, 2, 3)])
@pytest.mark.parametrize("table", ["relu", None])
def test_conv2d_few_channels_int8_output(oracle, B, H, W, Cin, Cout, kh, kw, stride, pad, table):
    """The kernel for at most four input channels: the word that holds the tensor's last pixel, images smaller
    than a word, padding on every side, each channel count, tile edges in both directions."""
    g = np.random.default_rng(B * 7 + H + Cin + kh)
    x, w = rand_i8(g, (B, H, W, Cin)), rand_i8(g, (Cout, kh, kw, Cin), 60)
    Ho, Wo = oracle.conv_out_hw(H, W, kh, kw, stride, pad)
    K = kh * kw * Cin
    alpha_vec = ((3.0 / (35 * 70 * np.sqrt(K))) * (1 + g.random(Cout))).astype(np.float32)
    bias = (0.3 * g.standard_normal(Cout)).astype(np.float32)
    ot, dt = relu_tables(oracle)
    want = oracle.conv2d_pwl(x, w, stride, pad, bias=bias, alpha_vec=alpha_vec, table=ot if table else None, out_inv_scale=20.0)
    dx, dw, db, da = dev(x), dev(w), dev(bias), dev(alpha_vec)
    oq = torch.full((B, Ho, Wo, Cout), 77, dtype=torch.int8, device=DEV)
    d = nm.make_conv_desc(dx, dw, stride, pad, bias=db, alpha_vec=da, tables=dt if table else None, table_idx=0 if table else -1,
                          out_inv_scale=20.0, out_q=oq)
    ws = torch.empty(max(nm.nm_conv2d_workspace(d), 256), dtype=torch.uint8, device=DEV)
    nm.nm_conv2d_pwl(d, ws)
    assert np.array_equal(host(oq), want["q"])


@pytest.mark.parametrize("B,H,W,Cin,Cout,kh,kw,stride,pad", CASES)
def test_conv2d_all_outputs(oracle, B, H, W, Cin, Cout, kh, kw, stride, pad):
    g = np.random.default_rng(B * 7 + H + Cin + kh)
    x = rand_i8(g, (B, H, W, Cin), 60)
    w = rand_i8(g, (Cout, kh, kw, Cin), 60)
    Ho, Wo = oracle.conv_out_hw(H, W, kh, kw, stride, pad)
    K = kh * kw * Cin
    alpha_vec = ((3.0 / (35 * 35 * np.sqrt(K))) * (1 + g.random(Cout))).astype(np.float32)
    bias = (0.3 * g.standard_normal(Cout)).astype(np.float32)
    resid = rand_i8(g, (B, Ho, Wo, Cout))
    ot, dt = relu_tables(oracle)
    kw_ = dict(stride=stride, pad=pad, bias=bias, alpha_vec=alpha_vec, resid_scale=0.01, out_inv_scale=30.0)
    r = oracle.conv2d_pwl(x, w, resid=resid, table=ot, **kw_)
    oq = torch.empty((B, Ho, Wo, Cout), dtype=torch.int8, device=DEV)
    of = torch.empty((B, Ho, Wo, Cout), dtype=torch.float32, device=DEV)
    oa = torch.empty((B, Ho, Wo, Cout), dtype=torch.int32, device=DEV)
    # device copies stay referenced until the kernels have run (the descriptor holds raw pointers)
    dx, dw, db, dav, dres = dev(x), dev(w), dev(bias), dev(alpha_vec), dev(resid)
    dkw = dict(stride=stride, pad=pad, bias=db, alpha_vec=dav, out_inv_scale=30.0)
    d = nm.make_conv_desc(dx, dw, resid=dres, resid_scale=0.01, tables=dt, table_idx=0, out_q=oq, out_f32=of,
                          dbg_acc=oa, **dkw)
    ws = torch.empty(max(256, nm.nm_conv2d_workspace(d)), dtype=torch.uint8, device=DEV)
    nm.nm_conv2d_pwl(d, ws)
    assert np.array_equal(host(oa), r["acc"]), "accumulators"
    assert np.array_equal(host(of).view(np.uint32), r["y"].view(np.uint32)), "fp32 output"
    assert np.array_equal(host(oq), r["q"]), "int8 output"
    assert (r["q"] == 0).mean() > 0.1 and (r["q"] > 0).mean() > 0.1
    # the int8-only forms the network uses: with table (no residual), and plain (no table)
    kw2 = dict(kw_)
    kw2.pop("resid_scale")
    for table in (ot, None):
        r2 = oracle.conv2d_pwl(x, w, table=table, want_acc=False, **kw2)
        oq2 = torch.empty_like(oq)
        d2 = nm.make_conv_desc(dx, dw, tables=dt, table_idx=0 if table is not None else -1, out_q=oq2, **dkw)
        nm.nm_conv2d_pwl(d2, ws)
        assert np.array_equal(host(oq2), r2["q"]), f"int8-only, table={table is not None}"


# B, H, W, Cin, Cout, k, stride, pad, and the tile kernel's configuration (choose_relu in csrc/nm_gemm_choice.h; that each case
# takes it is shown in test_gemm_choice.py): each of them with rows gathered and with plain ones
LARGE_TILE_CASES = [
    (27, 40, 40, 64, 48, 3, 1, 1, 10), (13, 31, 29, 192, 96, 3, 1, 1, 9), (7, 39, 35, 128, 112, 3, 1, 1, 7), (1, 90, 93, 128, 128, 3, 1, 2, 7),
    (3, 61, 63, 384, 400, 1, 2, 0, 8), (2, 35, 37, 512, 432, 1, 1, 0, 7), (1, 60, 61, 1024, 304, 1, 1, 0, 7), (2, 40, 41, 128, 528, 1, 1, 0, 9),
    (5, 43, 41, 64, 208, 1, 1, 0, 9), (3, 50, 51, 192, 240, 1, 1, 0, 9), (31, 30, 30, 64, 64, 1, 1, 0, 10), (9, 45, 41, 128, 112, 2, 1, 0, 7),
    (1, 111, 113, 256, 240, 3, 1, 1, 11), (9, 45, 42, 512, 144, 1, 1, 0, 2), (9, 37, 35, 128, 272, 2, 1, 0, 2), (3, 59, 57, 512, 144, 1, 1, 0, 5),
    (11, 45, 43, 512, 272, 1, 2, 0, 5), (5, 56, 59, 384, 80, 1, 1, 0, 6), (9, 41, 44, 384, 400, 1, 2, 0, 6), (1, 46, 44, 384, 496, 1, 1, 0, 8),
    (3, 61, 63, 1664, 144, 1, 1, 0, 11), (5, 77, 75, 256, 304, 3, 2, 1, 11), (5, 65, 63, 192, 240, 3, 2, 1, 9)]


@pytest.mark.parametrize("B,H,W,Cin,Cout,k,stride,pad,tile", LARGE_TILE_CASES)
def test_conv2d_large_tile_kernel(oracle, B, H, W, Cin, Cout, k, stride, pad, tile):
    """Convolutions whose outputs are large enough for the tile kernel: gathered rows (64- and 128-byte slices, several taps
    per slice count, strides, padding wider than needed) and plain ones of one, two, three and more slices; partly filled
    row and column tiles; a ReLU, a table of two other lines, none, and a residual.  The results sit between guards."""
    g = np.random.default_rng(B + H + Cin + Cout)
    x, w = rand_i8(g, (B, H, W, Cin), 60), rand_i8(g, (Cout, k, k, Cin), 60)
    Ho, Wo = oracle.conv_out_hw(H, W, k, k, stride, pad)
    assert B * Ho * Wo * Cout >= (1700000 if k * k * Cin <= 256 or Cout <= 64 else 1000000)   # below: the small-tile kernel
    alpha_vec = ((3.0 / (35 * 35 * np.sqrt(k * k * Cin))) * (1 + g.random(Cout))).astype(np.float32)
    bias = (0.3 * g.standard_normal(Cout)).astype(np.float32)
    ot, dt = relu_tables(oracle)
    ot2 = oracle.build_table(oracle.F_GELU, -1.0, 3.0, 2)
    dt2 = nm.nm_tables_from_arrays([("gelu", -1.0, 3.0, 2, 0)], [ot2.k], [ot2.b])
    dx, dw, db, dav = dev(x), dev(w), dev(bias), dev(alpha_vec)
    n = B * Ho * Wo * Cout
    resid = rand_i8(g, (B, Ho, Wo, Cout)) if k == 1 and stride == 1 else None
    dres = dev(resid)
    for tab, dtab, res in ((ot, dt, False), (ot2, dt2, False), (None, None, False), (ot, dt, True)):
        if res and resid is None:
            continue
        rk = dict(resid=resid, resid_scale=0.01) if res else {}
        want = oracle.conv2d_pwl(x, w, stride=stride, pad=pad, bias=bias, alpha_vec=alpha_vec, table=tab, out_inv_scale=30.0,
                                 want_acc=False, **rk)["q"]
        buf = torch.full((n + 256,), 77, dtype=torch.int8, device=DEV)
        oq = buf[128:128 + n].view(B, Ho, Wo, Cout)
        dk = dict(resid=dres, resid_scale=0.01) if res else {}
        d = nm.make_conv_desc(dx, dw, stride=stride, pad=pad, bias=db, alpha_vec=dav, tables=dtab, table_idx=-1 if tab is None else 0,
                              out_inv_scale=30.0, out_q=oq, **dk)
        ws = torch.empty(max(256, nm.nm_conv2d_workspace(d)), dtype=torch.uint8, device=DEV)
        nm.nm_conv2d_pwl(d, ws)
        assert np.array_equal(host(oq), want), (tab is not None, res)
        edge = host(buf)
        assert np.all(edge[:128] == 77) and np.all(edge[128 + n:] == 77)


@pytest.mark.parametrize("B,H,W,Cc,k,stride,pad", [(2, 112, 112, 64, 3, 2, 1), (3, 9, 10, 5, 3, 2, 1), (1, 8, 8, 12, 2, 2, 0),
                                                     (3, 9, 11, 48, 3, 1, 2), (5, 7, 8, 16, 2, 3, 1), (2, 13, 9, 80, 5, 2, 3), (1, 1, 1, 16, 1, 1, 0),
                                                     (2, 4, 3, 32, 4, 3, 3)])
def test_maxpool(oracle, B, H, W, Cc, k, stride, pad):
    x = rand_i8(np.random.default_rng(H), (B, H, W, Cc))
    want = oracle.maxpool_i8(x, k, stride, pad)
    y = torch.empty(want.shape, dtype=torch.int8, device=DEV)
    dx = dev(x)
    nm.nm_maxpool_i8(dx, y, k, stride, pad)
    assert np.array_equal(host(y), want)


@pytest.mark.parametrize("B,HW,C", [(5, 49, 2048), (3, 10, 30), (2, 64, 12), (64, 49, 2048), (1, 1, 4)])
def test_avgpool(oracle, B, HW, C):
    """Global average pooling: four channels per thread where C allows, one otherwise; position counts
    with and without a tail behind the groups of eight."""
    x = rand_i8(np.random.default_rng(B + HW + C), (B, HW, C))
    alpha = float(np.float32(0.013 / HW))
    want = oracle.avgpool_i8(x, alpha, 55.0)
    q = torch.full((B + 1, C), 77, dtype=torch.int8, device=DEV)
    f = torch.empty((B, C), dtype=torch.float32, device=DEV)
    dx = dev(x)
    nm.nm_avgpool_i8(dx, alpha, 55.0, out_q=q, out_f32=f)
    assert np.array_equal(host(f).view(np.uint32), want["y"].view(np.uint32))
    assert np.array_equal(host(q)[:B], want["q"]) and np.all(host(q)[B] == 77)
    q2 = torch.empty((B, C), dtype=torch.int8, device=DEV)
    nm.nm_avgpool_i8(dx, alpha, 55.0, out_q=q2)     # int8 output alone
    assert np.array_equal(host(q2), want["q"])


def test_conv_validation_and_empty():
    dt = nm.nm_build_tables([("relu", -8.0, 8.0, 2)])
    x = torch.zeros((1, 8, 8, 3), dtype=torch.int8, device=DEV)
    w = torch.zeros((4, 3, 3, 3), dtype=torch.int8, device=DEV)
    o = torch.zeros((1, 8, 8, 4), dtype=torch.int8, device=DEV)
    d = nm.make_conv_desc(x, w, 1, 1, tables=dt, table_idx=0, out_q=o)
    need = nm.nm_conv2d_workspace(d)
    assert need == 64 * 64 + 4 * 64  # patch matrix and filter rows, K = 27 padded to 64
    with pytest.raises(nm.NmError) as ei:
        nm.nm_conv2d_pwl(d, None)
    assert ei.value.status == nm.NM_ERR_WORKSPACE
    d.stride = 0
    with pytest.raises(nm.NmError) as ei:
        nm.nm_conv2d_workspace(d)
    assert ei.value.status == nm.NM_ERR_INVALID_ARG


def run_resnet_gpu(p, dt, batch_tensor=None):
    """The network of the workload generator on the GPU: one C-ABI call per operation."""
    cur = {"x": dev(p["x"]) if batch_tensor is None else batch_tensor}
    B = cur["x"].shape[0]
    out = {}
    keep = []
    for op in p["graph"]:
        n = op["name"]
        if op["op"] == "conv":
            Ho = op["Ho"]
            y = torch.empty((B, Ho, Ho, op["Cout"]), dtype=torch.int8, device=DEV)
            wt, bi, av = dev(p["w"][n]), dev(p["bias"][n]), dev(p["alpha_vec"][n])
            keep += [wt, bi, av]
            d = nm.make_conv_desc(cur[op["src"]], wt, op["stride"], op["pad"], bias=bi, alpha_vec=av,
                                  resid=cur[op["resid"]] if op["resid"] else None,
                                  resid_scale=p["resid_scale"][n], tables=dt, table_idx=0 if op["relu"] else -1,
                                  out_inv_scale=p["inv_s"][n], out_q=y)
            ws = torch.empty(max(256, nm.nm_conv2d_workspace(d)), dtype=torch.uint8, device=DEV)
            keep.append(ws)
            nm.nm_conv2d_pwl(d, ws)
            cur[op["dst"]] = y
        elif op["op"] == "maxpool":
            y = torch.empty((B, op["Ho"], op["Ho"], op["C"]), dtype=torch.int8, device=DEV)
            nm.nm_maxpool_i8(cur[op["src"]], y, op["k"], op["stride"], op["pad"])
            cur[op["dst"]] = y
        elif op["op"] == "avgpool":
            y = torch.empty((B, op["C"]), dtype=torch.int8, device=DEV)
            nm.nm_avgpool_i8(cur[op["src"]].view(B, -1, op["C"]), p["alpha"][n], p["inv_s"][n], out_q=y)
            cur[op["dst"]] = y
        elif op["op"] == "fc":
            y = torch.empty((B, op["Cout"]), dtype=torch.float32, device=DEV)
            wt, bi = dev(p["w"][n]), dev(p["bias"][n])
            keep += [wt, bi]
            nm.nm_gemm_pwl(cur[op["src"]], wt, bias=bi, alpha=p["alpha"][n], out_f32=y)
            out["logits"] = y
    torch.cuda.synchronize()  # every buffer in `keep` stays alive until the kernels have run
    out["tensors"] = cur
    return out


@pytest.mark.parametrize("name", ["resnet_odd", "resnet_tiny"])
def test_resnet_every_tensor(oracle, name):
    p = W.resnet_params(name, 0)
    ot, dt = relu_tables(oracle)
    want = oracle.resnet_forward(p, keep=True)
    got = run_resnet_gpu(p, dt)
    for k, v in want["tensors"].items():
        assert np.array_equal(host(got["tensors"][k]), v), f"{name}: tensor {k}"
    assert np.array_equal(host(got["logits"]).view(np.uint32), want["logits"].view(np.uint32)), "logits"


def test_resnet50_full_size_layers_batch4(oracle):
    """The real ResNet-50 layer shapes (224 x 224 input) on four images: every tensor exact."""
    p = W.resnet_params("resnet50", 0, batch=4)
    ot, dt = relu_tables(oracle)
    want = oracle.resnet_forward(p, keep=True)
    got = run_resnet_gpu(p, dt)
    for k, v in want["tensors"].items():
        assert np.array_equal(host(got["tensors"][k]), v), f"resnet50: tensor {k}"
    assert np.array_equal(host(got["logits"]).view(np.uint32), want["logits"].view(np.uint32)), "logits"


def test_resnet50_batch64_launch_configuration(oracle):
    """The configuration bench.py times (batch 64: other tile choices than small batches take):
    every tensor of the network and the logits, all 64 images, against the oracle (~10 s of oracle
    time).  Two images are copies of others, which must give identical results as well."""
    p = W.resnet_params("resnet50", 0, batch=64)
    p["x"] = p["x"].copy()
    p["x"][63] = p["x"][0]
    p["x"][37] = p["x"][1]
    ot, dt = relu_tables(oracle)
    want = oracle.resnet_forward(p, keep=True)
    got = run_resnet_gpu(p, dt)
    for k, v in want["tensors"].items():
        assert np.array_equal(host(got["tensors"][k]), v), f"resnet50 batch 64: tensor {k}"
    logits = host(got["logits"])
    assert np.array_equal(logits.view(np.uint32), want["logits"].view(np.uint32))
    assert np.array_equal(logits[63], logits[0]) and np.array_equal(logits[37], logits[1])


def test_cnn_run_matches_oracle_network(oracle):
    """nm_cnn_run (the whole network as one call over a list of steps) on resnet_tiny."""
    p = W.resnet_params("resnet_tiny", 0)
    ot, dt = relu_tables(oracle)
    want = oracle.resnet_forward(p, keep=True)
    B = p["B"]
    cur = {"x": dev(p["x"])}
    ops, keep = [], []
    for op in p["graph"]:
        n = op["name"]
        if op["op"] == "conv":
            y = torch.empty((B, op["Ho"], op["Ho"], op["Cout"]), dtype=torch.int8, device=DEV)
            wt, bi, av = dev(p["w"][n]), dev(p["bias"][n]), dev(p["alpha_vec"][n])
            keep += [wt, bi, av]
            ops.append(nm.cnn_op_conv(nm.make_conv_desc(
                cur[op["src"]], wt, op["stride"], op["pad"], bias=bi, alpha_vec=av,
                resid=cur[op["resid"]] if op["resid"] else None, resid_scale=p["resid_scale"][n], tables=dt,
                table_idx=0 if op["relu"] else -1, out_inv_scale=p["inv_s"][n], out_q=y)))
            cur[op["dst"]] = y
        elif op["op"] == "maxpool":
            y = torch.empty((B, op["Ho"], op["Ho"], op["C"]), dtype=torch.int8, device=DEV)
            ops.append(nm.cnn_op_maxpool(cur[op["src"]], y, op["k"], op["stride"], op["pad"]))
            cur[op["dst"]] = y
        elif op["op"] == "avgpool":
            y = torch.empty((B, op["C"]), dtype=torch.int8, device=DEV)
            ops.append(nm.cnn_op_avgpool(cur[op["src"]].view(B, -1, op["C"]), p["alpha"][n], p["inv_s"][n], out_q=y))
            cur[op["dst"]] = y
        else:
            logits = torch.empty((B, op["Cout"]), dtype=torch.float32, device=DEV)
            wt, bi = dev(p["w"][n]), dev(p["bias"][n])
            keep += [wt, bi]
            ops.append(nm.cnn_op_gemm(nm.make_gemm_desc(cur[op["src"]], wt, bias=bi, alpha=p["alpha"][n], out_f32=logits)))
    ws = torch.empty(max(256, nm.nm_cnn_workspace(ops)), dtype=torch.uint8, device=DEV)
    nm.nm_cnn_run(ops, ws)
    for k, v in want["tensors"].items():
        assert np.array_equal(host(cur[k]), v), f"nm_cnn_run: tensor {k}"
    assert np.array_equal(host(logits).view(np.uint32), want["logits"].view(np.uint32))
    bad = nm.CnnOp()
    bad.kind = 9
    with pytest.raises(nm.NmError) as ei:
        nm.nm_cnn_run([bad], ws)
    assert ei.value.status == nm.NM_ERR_INVALID_ARG


# two neighbouring steps: H, Cin, then (Cout, k, stride, ReLU) of each on the same image, and how the second one is tied to the first
@pytest.mark.parametrize("B,H,Cin,first,second,tie", [
    (1, 28, 128, (128, 3, 2, True), (512, 1, 2, False), ""),        # a residual block's 3x3 convolution and its projection
    (1, 14, 64, (64, 3, 1, True), (256, 1, 1, False), ""), (3, 15, 64, (52, 1, 1, False), (36, 5, 1, True), ""),
    (1, 7, 512, (512, 3, 1, True), (2048, 1, 2, False), ""), (2, 30, 192, (136, 3, 1, False), (68, 2, 1, False), ""),
    (5, 28, 128, (128, 3, 2, True), (512, 1, 2, False), ""), (1, 9, 64, (64, 3, 1, True), (30, 1, 1, False), ""),
    (1, 14, 128, (128, 3, 1, True), (64, 3, 1, True), "chain"),     # the second reads the first's result,
    (1, 14, 128, (128, 3, 1, True), (128, 1, 1, True), "image"),    # writes over its image,
    (1, 14, 128, (128, 3, 1, True), (128, 1, 1, True), "result")])  # or over its result
def test_neighbouring_convolutions(oracle, B, H, Cin, first, second, tie):
    """nm_cnn_run on two convolutions: as one launch where neither touches what the other writes, one after the other where it does."""
    g = np.random.default_rng(H + Cin)
    ot, dt = relu_tables(oracle)
    x = rand_i8(g, (B, H, H, Cin), 60)
    dx = dev(x)
    ops, keep, want, ys, src, dsrc = [], [], [], [], x, dx
    for n, (cout, k, stride, relu) in enumerate((first, second)):
        w, bias = rand_i8(g, (cout, k, k, Cin), 60), g.standard_normal(cout).astype(np.float32)
        alpha = (1e-3 * (1 + g.random(cout))).astype(np.float32)
        r = oracle.conv2d_pwl(src, w, stride, k // 2, bias=bias, alpha_vec=alpha, table=ot if relu else None, out_inv_scale=9.0)
        want.append(r["q"])
        y = torch.full(r["q"].shape, 77, dtype=torch.int8, device=DEV)
        if n == 1 and tie == "image": y = dx
        if n == 1 and tie == "result": y = ys[0]
        ys.append(y)
        d = [dev(w), dev(bias), dev(alpha)]
        keep += d
        ops.append(nm.cnn_op_conv(nm.make_conv_desc(dsrc, d[0], stride, k // 2, bias=d[1], alpha_vec=d[2], tables=dt, table_idx=0 if relu else -1,
                                                    out_inv_scale=9.0, out_q=y)))
        if tie == "chain": src, dsrc, Cin = r["q"], y, cout
    if tie == "image":
        ops = ops[:1] + [nm.cnn_op_conv(nm.make_conv_desc(ys[0], keep[3], 1, 0, bias=keep[4], alpha_vec=keep[5], tables=dt, table_idx=0, out_inv_scale=9.0, out_q=dx))]
        want[1] = oracle.conv2d_pwl(want[0], host(keep[3]), 1, 0, bias=host(keep[4]), alpha_vec=host(keep[5]), table=ot, out_inv_scale=9.0)["q"]
    nm.nm_cnn_run(ops, torch.empty(256, dtype=torch.uint8, device=DEV))
    for n in (0, 1):
        if not (n == 0 and tie == "result"): assert np.array_equal(host(ys[n]), want[n]), f"step {n}"


@pytest.mark.parametrize("B,H,W,form", [
    (3, 56, 56, "relu"), (9, 31, 33, "relu"), (1, 1, 8193, "relu"), (1, 8200, 1, "relu"), (4100, 1, 2, "relu"), (911, 3, 3, "relu"), (22, 55, 57, "relu"),
    (3, 53, 59, "lines"), (3, 53, 59, "nonfinite"), (3, 53, 59, "scalar"), (3, 53, 59, "none"), (6, 53, 59, "none"), (1, 1, 16385, "none")])
def test_3x3_convolutions_of_64_channels(oracle, B, H, W, form):
    """Stride 1, a border of 1, from 8192 positions on (16384 without a table): images of one row, one column, fewer pixels than a block; a last block that is not
    full; more than one turn of the wavefronts (22 x 55 x 57); any two-segment table, none, columns whose sums are infinite or NaN."""
    g = np.random.default_rng(B + H + W)
    ot, tables = relu_tables(oracle)
    if form == "lines":
        k, b = np.float32([0.125, 1.0]), np.float32([0.1, -0.3])
        tables, ot.k[:], ot.b[:] = nm.nm_tables_from_arrays([("relu", -8.0, 8.0, 2, 0)], [k], [b]), k, b
    x, w = rand_i8(g, (B, H, W, 64)), rand_i8(g, (64, 3, 3, 64))
    bias, alpha = g.standard_normal(64).astype(np.float32), (5e-5 * (1 + g.random(64))).astype(np.float32)
    if form == "nonfinite": bias[[3, 40]], alpha[50] = (np.nan, np.inf), 3e38
    if form == "scalar": bias = alpha = None
    table = form != "none"
    dx, dw, db, da = (dev(v) for v in (x, w, bias, alpha))
    y = torch.full((B * H * W + 64, 64), 77, dtype=torch.int8, device=DEV)   # 64 rows behind the result stay as they are
    nm.nm_conv2d_pwl(nm.make_conv_desc(dx, dw, 1, 1, bias=db, alpha=6e-5, alpha_vec=da, tables=tables, table_idx=0 if table else -1, out_inv_scale=30.0,
                                       out_q=y[:B * H * W].view(B, H, W, 64)), torch.empty(256, dtype=torch.uint8, device=DEV))
    want = oracle.conv2d_pwl(x, w, 1, 1, bias=bias, alpha=6e-5, alpha_vec=alpha, table=ot if table else None, out_inv_scale=30.0)["q"]
    got = host(y)
    assert np.array_equal(got[:B * H * W].reshape(want.shape), want) and (got[B * H * W:] == 77).all()


# positions (a last block of 32 that is not full, a second turn of the wavefronts) and channels of a widening and a narrowing convolution
# that are one kernel (tests/test_gemm_choice.py holds them to its rule); forms at the smallest of each kernel
CHAIN_CASES = [(5037, 64, 256, 64), (5037, 64, 256, 128), (50003, 128, 256, 128), (25089, 64, 512, 64), (100003, 64, 256, 64), (70003, 64, 256, 128),
               (131041, 128, 512, 128)]
CHAIN_LINES_CASES = [(12551, 64, 256, 64), (58003, 64, 256, 128), (62003, 128, 256, 128)]   # with tables that are no ReLU


@pytest.mark.parametrize("M,K,N1,N2,form", [(*c, "relu") for c in CHAIN_CASES] + [
    (*c, form) for c in CHAIN_CASES[:3] for form in ("lines", "nonfinite", "scalar")] + [(*c, "lines") for c in CHAIN_LINES_CASES] + [
    (5037, 64, 256, 64, form) for form in ("over_x", "over_shortcut", "over_result", "over_bias", "apart")])
def test_chained_convolutions(oracle, M, K, N1, N2, form):
    """nm_cnn_run on a 1x1 convolution with a shortcut and the 1x1 one behind it gives what the two steps by themselves give, to the
    bit: any two-segment table, columns that make a sum infinite or NaN, no bias, buffers that one step reads and the other writes."""
    g = np.random.default_rng(M + K + N1 + N2)
    if form == "lines": tables = nm.nm_tables_from_arrays([("relu", -8.0, 8.0, 2, 0)], [np.float32([0.125, 1.0])], [np.float32([0.1, -0.3])])
    else: tables = relu_tables(oracle)[1]
    x, w1, w2, r = rand_i8(g, (M, 1, 1, K)), rand_i8(g, (N1, 1, 1, K)), rand_i8(g, (N2, 1, 1, N1)), rand_i8(g, (M, 1, 1, N1))
    bias = [g.standard_normal(n).astype(np.float32) for n in (N1, N2)]
    alpha = [(a * (1 + g.random(n))).astype(np.float32) for a, n in ((1e-4, N1), (4e-5, N2))]
    if form == "nonfinite":
        bias[0][[3, 77]] = np.nan, np.inf
        alpha[0][200], bias[1][17], alpha[1][60] = 3e38, -np.inf, np.nan
    if form == "over_result": w2[:] = 0   # (rows of the second product read what others of it have written: its codes are those of its bias)

    def run(call):
        dx, dr, d1, d2 = dev(x), dev(r), dev(w1), dev(w2)
        db, da = [dev(v) if form != "scalar" else None for v in bias], [dev(v) if form != "scalar" else None for v in alpha]
        y1, y2 = (torch.full((M, 1, 1, n), 77, dtype=torch.int8, device=DEV) for n in (N1, N2))
        if form == "over_x": y2 = dx
        if form == "over_shortcut": y1 = dr
        if form == "over_result": y2 = y1.view(-1)[M * N2:2 * M * N2].view(M, 1, 1, N2)
        if form == "over_bias":   # of the second step, in what the first one writes
            db[1] = y1.view(-1)[-4 * N2:].view(torch.float32)
        src = y1.clone() if form == "apart" else y1   # the second step reads something else
        ops = [nm.cnn_op_conv(nm.make_conv_desc(dx, d1, 1, 0, bias=db[0], alpha=2e-4, alpha_vec=da[0], resid=dr, resid_scale=0.01, tables=tables, table_idx=0,
                                                out_inv_scale=30.0, out_q=y1)),
               nm.cnn_op_conv(nm.make_conv_desc(src, d2, 1, 0, bias=db[1], alpha=6e-5, alpha_vec=da[1], tables=tables, table_idx=0, out_inv_scale=25.0, out_q=y2))]
        call(ops)
        return host(y1), host(y2)

    ws = torch.empty(256, dtype=torch.uint8, device=DEV)
    got = run(lambda ops: nm.nm_cnn_run(ops, ws))
    want = run(lambda ops: (nm.nm_cnn_run(ops[:1], ws), nm.nm_cnn_run(ops[1:], ws)))
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert 0.1 < np.mean(got[0] != 0) and len(np.unique(got[0])) > 20
    if form == "over_result":   # the second result lies whole over the first
        own = np.unique(got[1].reshape(M, N2), axis=0)
        assert len(own) == 1 and len(np.unique(own)) > 10 and np.array_equal(got[0].reshape(-1)[M * N2:2 * M * N2].reshape(got[1].shape), got[1])
    if form == "relu" and M < 10000:
        ot = oracle.relu_table()
        q1 = oracle.conv2d_pwl(x, w1, 1, 0, bias=bias[0], alpha_vec=alpha[0], resid=r, resid_scale=0.01, table=ot, out_inv_scale=30.0)["q"]
        q2 = oracle.conv2d_pwl(q1, w2, 1, 0, bias=bias[1], alpha_vec=alpha[1], table=ot, out_inv_scale=25.0)["q"]
        assert np.array_equal(got[0], q1) and np.array_equal(got[1], q2)


def test_conv2d_unaligned_operands_take_the_patch_matrix_route(oracle):
    """A 64-channel convolution whose image or filter pointer is not 16-byte aligned cannot use the
    gathered loader: it needs a workspace and still matches the oracle."""
    g = np.random.default_rng(77)
    B, H, Wd, Cin, Cout = 2, 10, 9, 64, 80
    x = rand_i8(g, (B, H, Wd, Cin), 50)
    w = rand_i8(g, (Cout, 3, 3, Cin), 50)
    ot, dt = relu_tables(oracle)
    av = np.full(Cout, 2e-4, np.float32)
    r = oracle.conv2d_pwl(x, w, stride=1, pad=1, alpha_vec=av, table=ot, out_inv_scale=20.0, want_acc=False)
    raw = torch.zeros(x.size + 32, dtype=torch.int8, device=DEV)
    raw[8:8 + x.size] = dev(x).view(-1)            # data starts 8 bytes after an aligned address
    dx = raw[8:8 + x.size].view(B, H, Wd, Cin)
    dw, dav = dev(w), dev(av)
    oq = torch.empty((B, H, Wd, Cout), dtype=torch.int8, device=DEV)
    d = nm.make_conv_desc(dx, dw, 1, 1, alpha_vec=dav, tables=dt, table_idx=0, out_inv_scale=20.0, out_q=oq)
    need = nm.nm_conv2d_workspace(d)
    assert need == B * H * Wd * 576 + Cout * 576
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    nm.nm_conv2d_pwl(d, ws)
    assert np.array_equal(host(oq), r["q"])
    # aligned again: no workspace
    d2 = nm.make_conv_desc(dev(x), dw, 1, 1, alpha_vec=dav, tables=dt, table_idx=0, out_inv_scale=20.0, out_q=oq)
    assert nm.nm_conv2d_workspace(d2) == 0
