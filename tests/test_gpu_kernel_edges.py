"""The kernels' own edges: sizes at which a dispatch rule changes sides or a tile is partly filled,
against the CPU oracle (codes, scales and integer sums bit for bit)."""
import math
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2503_06545_amd import binding as qc
from paper_2503_06545_amd import synth
from test_gpu_parity import RTOL, assert_outputs_close, bits_equal, dev, host_f64, random_x, run_asym_case, run_linear_case

pytestmark = pytest.mark.gpu


def kernel_of(M, K, N, bits, **which):
    """The GEMM kernel a linear takes: "few", "resident" or "ring" with its tile's tokens, "split" and "kept"."""
    plan = qc.linear_plan(M, K, N, bits, **which)
    return plan["kernel"] + (f" {plan['tokens']}" if plan["kernel"] == "ring" else "") + " split" * plan["split"] + " kept" * plan["kept"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K", [(1, 16), (9, 112), (8, 128), (7, 144), (9, 2032), (9, 2048), (9, 2064),
                                 (5, 6144), (5, 6160), (4609, 2048), (4610, 2048)])
def test_row_quantizers_at_the_edges_of_their_column_slices(M, K, dtype):
    """Eight lanes take 128 columns of a row per step, a wavefront one, three or nine steps: a last
    step that is partly or wholly past the row, and both sides of K = 2048, K = 6144 and
    M K = 8192 * 1152, where the number of steps changes."""
    rng = np.random.default_rng(M * 10007 + K)
    x = random_x(rng, M, K, dtype)
    q_ref, s_ref = oracle.quant_act(x)
    a_ref = oracle.quant_act_asym(x)
    qx, sx = qc.quant_act_t(dev(x))
    qa = qc.quant_act_asym_t(dev(x))
    torch.cuda.synchronize()
    assert bits_equal(sx.cpu().numpy(), s_ref) and np.array_equal(qx.cpu().numpy(), q_ref)
    assert np.array_equal(qa[0].cpu().numpy(), a_ref[0])
    assert bits_equal(qa[1].cpu().numpy(), a_ref[1]) and bits_equal(qa[2].cpu().numpy(), a_ref[2])
    if K % 16 == 0:
        r_ref = oracle.quant_act_rot(x, 16, 8)
        qr, sr = qc.quant_act_t(dev(x), 8, 16)
        assert bits_equal(sr.cpu().numpy(), r_ref[1]) and np.array_equal(qr.cpu().numpy(), r_ref[0])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,rot_block", [(1, 16, 16), (9, 32, 32), (3, 64, 64), (9, 144, 16), (8, 160, 32), (7, 192, 64),
                                           (9, 2016, 32), (3, 2112, 64), (2, 4640, 32), (2, 6208, 64), (1, 9184, 32)])
def test_rotated_rows_that_end_within_a_group(M, K, rot_block, dtype):
    """A group of 128 columns that the row fills in part: what lies past the row takes no part in the maximum,
    although the row's last elements, here its largest, are loaded in its place; with one, three
    and nine groups a lane."""
    rng = np.random.default_rng(M * 10007 + K + rot_block)
    x = random_x(rng, M, K, "f32")
    x[:, -rot_block:] = 0.0
    x[:, -4:] = 100.0 * rng.standard_normal((M, 4))
    if dtype == "bf16":
        x = synth.to_bf16_bits(x.astype(np.float32))
    q_ref, s_ref = oracle.quant_act_rot(x, rot_block, 8)
    qx, sx = qc.quant_act_t(dev(x), 8, rot_block)
    assert bits_equal(sx.cpu().numpy(), s_ref) and np.array_equal(qx.cpu().numpy(), q_ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,rot_block", [(147473, 64, 32), (73729, 128, 16), (73731, 128, 128), (36865, 256, 64), (24577, 384, 128),
                                           (18433, 512, 16), (8, 6272, 128), (3, 9216, 16)])
def test_rotated_rows_shorter_than_a_wavefronts_columns(M, K, rot_block, dtype):
    """Rows on three and nine groups a lane, of which one, two, all or one of the next slice are the row's: the first and
    the last rows against the oracle."""
    rng = np.random.default_rng(M + K + rot_block)
    x = random_x(rng, min(M, 40), K, dtype)
    X = dev(x).repeat(-(-M // len(x)), 1)[:M].contiguous()
    q_ref, s_ref = oracle.quant_act_rot(x, rot_block, 8)
    qx, sx = qc.quant_act_t(X, 8, rot_block)
    torch.cuda.synchronize()
    n = len(x)
    assert bits_equal(sx[:n].cpu().numpy(), s_ref) and np.array_equal(qx[:n].cpu().numpy(), q_ref)
    assert torch.equal(sx[n:], sx[:-n]) and torch.equal(qx[n:], qx[:-n])


@pytest.mark.parametrize("scheme", ["token", "rot", "asym"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 416, 448, 480, 512])
def test_rows_streamed_without_the_columns_past_their_end(K, dtype, scheme):
    """Non-temporal loads on rows that leave a third or more of their wavefronts' columns empty, and on the shortest that do
    not (256, 512; of 416 binary32 is whole lines): the first rows against the oracle, the others, with a remainder of three, against those."""
    M = (180 << 20) // ((5 if dtype == "f32" else 3) * K) // 40 * 40 + 3
    assert qc.linear_plan(M, K, 64, x=dtype, scheme=scheme)["nt_loads"] == (K * (4 if dtype == "f32" else 2) % 128 == 0)
    rng = np.random.default_rng(K)
    x = random_x(rng, 40, K, dtype)
    X = dev(x).repeat(-(-M // 40), 1)[:M].contiguous()
    if scheme == "asym":
        got, want = qc.quant_act_asym_t(X, 8), oracle.quant_act_asym(x, 8)
    else:
        rot = 32 if scheme == "rot" else 0
        got, want = qc.quant_act_t(X, 8, rot), oracle.quant_act_rot(x, rot, 8) if rot else oracle.quant_act(x, 8)
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert np.array_equal(g[:40].cpu().numpy(), w)
        assert torch.equal(g[40:], g[:-40])


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N", [
    (1, 16, 1), (2, 9216, 40), (3, 6144, 33), (16, 1536, 4100), (16, 1552, 70), (17, 1152, 128), (31, 1280, 2050),
    (32, 1296, 100), (33, 192, 4100), (100, 1152, 4100), (255, 320, 2048), (256, 64, 2050), (512, 208, 2047),
    (1024, 64, 1024), (1025, 64, 1024), (300, 1000, 131), (1024, 64, 64), (1000, 320, 4), (1001, 1000, 132)])
def test_qlinear_on_few_tokens_at_the_edges_of_its_tiles(M, K, N, bits):
    """Both sides of every change of tile (16 x 32, 32 x 32, 32 x 64, 64 x 64, then the ring kernel), in one launch
    and in two, row counts below a power of two; every quantizer, every output type, channel counts of every store width."""
    rng = np.random.default_rng(M * 31 + K * 7 + N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    assert qc.qc_debug_gemm_kernel(M, K, N, bits) == (3 if M < 1025 else 1)
    x = random_x(rng, M, K, "bf16")
    run_linear_case(x, W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(random_x(rng, M, K, "f32"), W, None, bits, "gelu_erf", "f32", act_bits=6, check_acc=False)
    if K % 16 == 0:
        run_linear_case(x, W, b, bits, "none", "f32", rot_block=16, check_acc=False)
        run_asym_case(x, W, b, bits, "none", "bf16")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,K,N,shift", [(2, 1152, 1152, 0), (64, 1152, 1152, 0), (256, 1152, 1152, 0), (100, 1152, 640, 0),
                                         (64, 1152, 1152, 16), (64, 1152, 1152, -16), (33, 1000, 1000, 0), (64, 1152, 64, 1)])
def test_qlinear_on_few_tokens_over_its_own_input(M, K, N, shift, dtype):
    """Y over X, wholly or shifted by some rows, gives what a Y of its own gives: every block of the
    one-launch form reads tokens that another block's output would have replaced."""
    assert qc.qc_debug_gemm_kernel(M, K, N, 8) == 3
    rng = np.random.default_rng(M + K + N + shift)
    pw = qc.pack_weight_t(dev((rng.standard_normal((N, K)) * 0.02).astype(np.float32)), 8)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    off = 64 * 1152                                   # room for Y on either side
    buf = torch.zeros(off + max(M * K, M * N) + off, dtype=t, device="cuda")
    X = buf[off:off + M * K].view(M, K)
    at = off + shift * N
    Y = buf[at:at + M * N].view(M, N)
    for _ in range(5):
        x = dev(random_x(rng, M, K, dtype))
        X.copy_(x)
        want = qc.qlinear_t(x, pw, None, "none", dtype)
        got = qc.qlinear_t(X, pw, None, "none", dtype, Y=Y)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N", [
    (3, 8, 40), (5, 7, 33), (13, 10, 200), (16, 1530, 70), (16, 1538, 70), (16, 3070, 95), (16, 3074, 40), (1, 24580, 33),
    (2, 24570, 1), (17, 1152, 4100), (48, 1538, 2050), (130, 1000, 1282), (144, 1540, 1282), (250, 1152, 2049), (256, 3068, 2046),
    (272, 1030, 1920), (257, 1152, 4081), (700, 1152, 1281), (505, 1154, 2033), (519, 1151, 1921)])
def test_qlinear_in_one_launch_at_the_edges_of_its_shapes(M, K, N, bits):
    """Every tile of the one-launch form, both counts of wavefronts, one step of pairs of a row and a group and
    three, the longest rows each takes and one group more; ragged rows of any remainder, of less
    than 16 B too, row counts that are no power of two, a last tile with one live row and odd channels."""
    rng = np.random.default_rng(M * 31 + K * 7 + N + bits)
    K += K % 2 if bits == 4 else 0
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    run_linear_case(random_x(rng, M, K, "bf16"), W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(random_x(rng, M, K, "f32"), W, None, bits, "none", "f32", act_bits=6)


@pytest.mark.parametrize("scheme", ["token", "rot16", "rot32", "rot64", "rot128", "asym", "tensor"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,N,bits,act_bits", [
    (1, 128, 33, 8, 8), (3, 384, 40, 4, 6), (16, 1536, 100, 8, 8), (16, 1664, 70, 4, 8), (13, 1152, 4099, 8, 4), (17, 1152, 2050, 4, 8),
    (130, 640, 1282, 8, 6), (48, 2944, 2049, 8, 8), (256, 1152, 1153, 8, 8), (250, 3072, 1200, 4, 4), (300, 512, 1792, 8, 8), (64, 144, 1000, 8, 8)])
def test_one_launch_and_two_are_the_same_for_every_quantizer(scheme, dtype, M, K, N, bits, act_bits):
    """Codes, scales, corrections and outputs, bit for bit: a Y that begins in X's last bytes has the quantizer and
    the GEMM go out one after the other."""
    rot = int(scheme[3:]) if scheme.startswith("rot") else 0
    if rot and K % rot:
        rot = 16
    rng = np.random.default_rng(M * 31 + K * 7 + N + act_bits)
    x = dev(random_x(rng, M, K, dtype))
    pw = qc.pack_weight_t(dev((rng.standard_normal((N, K)) * 0.02).astype(np.float32)), bits, rot)
    bias, sums = dev((rng.standard_normal(N) * 0.01).astype(np.float32)), qc.weight_row_sums_t(pw)
    make = {"asym": qc.qlinear_asym_workspace_t, "tensor": qc.qlinear_tensor_workspace_t}.get(scheme, qc.qlinear_workspace_t)

    def call(X, Y, workspace, **kw):
        if scheme == "asym":
            return qc.qlinear_asym_t(X, pw, sums, bias, workspace=workspace, Y=Y, act_bits=act_bits, **kw)
        if scheme == "tensor":
            return qc.qlinear_tensor_t(X, pw, bias, workspace=workspace, Y=Y, act_bits=act_bits, **kw)
        return qc.qlinear_t(X, pw, bias, workspace=workspace, Y=Y, act_bits=act_bits, rot_block=rot, **kw)

    for out, t, epi in (("bf16", torch.bfloat16, "gelu_tanh"), ("f32", torch.float32, "none"), ("f32", torch.float32, "gelu_erf")):
        got, left = [], []
        for over in (False, True):
            x_bytes = x.numel() * x.element_size()
            at = (x_bytes + 15) // 16 * 16 - 16 if over else (x_bytes + 255) // 256 * 256
            buf = torch.zeros(at + M * N * 4 + 256, dtype=torch.uint8, device="cuda")
            X = buf[:x_bytes].view(x.dtype).view(M, K)
            X.copy_(x)
            Y = buf[at:at + M * N * torch.empty(0, dtype=t).element_size()].view(t).view(M, N)
            ws = make(M, K, N)
            ws.fill_(0x7f)
            call(X, Y, ws, epi=epi, out=out)
            got.append(Y.clone())
            left.append(qc.debug_workspace_act_asym_t(ws, M, K, act_bits) if scheme == "asym" else qc.debug_workspace_act_t(ws, M, K))
        assert torch.equal(*got)
        for a, b in zip(*left):
            assert torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a, b.view(torch.int32) if b.dtype == torch.float32 else b)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("N", [129, 130, 132, 136])
def test_qlinear_ring_kernel_on_ragged_tokens_and_channels(N, bits):
    """The kernel that streams its weights, on tiles of 192 tokens: partial tiles in both directions, channel counts of
    every store width."""
    M, K = 16421, 64
    assert kernel_of(M, K, N, bits, out="f32") == kernel_of(M, K, N, bits, epi="gelu_tanh") == "ring 192"
    rng = np.random.default_rng(100 * bits + N)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    run_linear_case(random_x(rng, M, K, "f32"), W, b, bits, "none", "f32")
    run_linear_case(random_x(rng, M, K, "bf16"), W, b, bits, "gelu_tanh", "bf16", check_acc=False)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,bf16,f32,asym", [
    (5505, 192, 130, "ring 128", "ring 128", "ring 128"), (16384, 64, 129, "ring 128", "ring 128", "ring 128"),
    (16385, 64, 129, "ring 192", "ring 192", "ring 192"), (21889, 64, 257, "ring 128", "ring 128 kept", "ring 128"),
    (21249, 320, 512, "ring 128", "ring 128 kept", "ring 128"), (21250, 64, 511, "ring 128", "ring 128 kept", "ring 128"),
    (26001, 64, 512, "ring 128", "ring 128 kept", "ring 128"), (7501, 400, 1156, "ring 128", "ring 192 kept", "ring 128"),
    (16300, 448, 1003, "ring 128", "ring 256 kept", "ring 128"), (25001, 2064, 129, "ring 256", "ring 256", "ring 256")])
def test_qlinear_ring_kernel_at_every_tile_height(M, K, N, bf16, f32, asym, bits):
    """From a few tiles to several per CU, whose heights the launcher chooses by how they spread; with
    32-bit output also both kinds of store (through the caches from 15 or 24 MB on); an asymmetric one."""
    assert kernel_of(M, K, N, bits, epi="gelu_tanh") == bf16 and kernel_of(M, K, N, bits, out="f32") == f32
    assert kernel_of(M, K, N, bits, epi="gelu_erf", scheme="asym") == asym
    rng = np.random.default_rng(M + N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    x = random_x(rng, M, K, "bf16")
    run_linear_case(x, W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(x, W, None, bits, "none", "f32", check_acc=False)
    run_asym_case(x, W, b, bits, "gelu_erf", "bf16")


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,bf16,f32,i32", [(1100, 64, 1000 + r, "ring 128", "ring 128", "ring 128") for r in range(8)]
                         + [(2200, 64, 2048 + r, "ring 192", "ring 192 kept", "ring 192") for r in range(8)]
                         + [(25000, 2064, 129 + r, "ring 256", "ring 256", "ring 256") for r in range(8)]
                         + [(16300, 448, 1000 + r, "ring 256", "ring 256 kept", "ring 256") for r in range(8)]
                         + [(5700, 64, 1536, "ring 128", "ring 128 kept", "ring 128"), (4300, 64, 1920, "ring 128", "ring 128 kept", "ring 128")]
                         + [(32700, 64, 3448 + r, "resident", "ring 256 kept" if r % 4 == 0 else "ring 128 kept", "resident") for r in (0, 1, 4, 7)]
                         + [(16300, 832, 6896 + r, "resident", "resident", "resident") for r in (0, 3)]
                         + [(262145, 64, 513, "ring 192", None, None), (137000, 448, 1003, "ring 256", None, None)])   # bf16 of more than 256 MB
def test_qlinear_many_tiles_stay_inside_their_output(M, K, N, bf16, f32, i32, bits):
    """Every remainder of N by 8 in the kernels for more than a few tokens, at every height of the ring's tiles, all types of
    output and both kinds of store, rows that are no multiple of 16 B beyond the cache's size too: every row against the
    oracle's (they repeat), nothing written on either side of Y."""
    period = 251
    for out, kernel in (("bf16", bf16), ("f32", f32), ("i32", i32)):
        assert kernel is None or kernel_of(M, K, N, bits, out=out) == kernel
    rng = np.random.default_rng(100 * N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    x = random_x(rng, period, K, "bf16")
    qw, sw = oracle.quant_weight(W, bits)
    ref = oracle.qlinear(x, qw, sw, b, 0, 8)
    X = dev(x).repeat(-(-M // period), 1)[:M].contiguous()
    pw, pad = qc.pack_weight_t(dev(W), bits), 4096
    for out, t, fill, kernel in (("bf16", torch.bfloat16, -7.0, bf16), ("f32", torch.float32, -7.0, f32), ("i32", torch.int32, -7, i32)):
        if kernel is None:
            continue
        buf = torch.full((M * N + 2 * pad,), fill, dtype=t, device="cuda")
        Y = qc.qlinear_t(X, pw, None if out == "i32" else dev(b), "none", out, Y=buf[pad:pad + M * N].view(M, N))
        torch.cuda.synchronize()
        if out == "i32":
            assert np.array_equal(Y[:period].cpu().numpy(), ref["acc"])
        else:
            want = oracle.bf16_bits_to_f64(oracle.round_bf16_bits(ref["y"])) if out == "bf16" else ref["y"]
            assert_outputs_close(host_f64(Y[:period]), want, RTOL[out])
        assert torch.equal(Y[period:], Y[:-period])
        assert bool((buf[:pad] == fill).all()) and bool((buf[pad + M * N:] == fill).all())


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N", [(1100, 1001), (2200, 2050), (50000, 129)])
@pytest.mark.parametrize("K", [200, 1000, 1160])
def test_qlinear_ring_kernel_ragged_k_with_a_poisoned_workspace(K, M, N, bits):
    """K no multiple of 16 or of the stage: what the quantizer leaves unwritten of the last columns meets
    zero weights, at several tile heights and in both halves of a split reduction."""
    wanted = {1100: ("ring 128 split" if bits == 4 and K > 200 else "ring 128"), 2200: "ring 192", 50000: "ring 128" if K == 200 else "ring 256"}[M]
    assert kernel_of(M, K, N, bits, out="i32") == wanted
    rng = np.random.default_rng(K + M + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    qw, _ = oracle.quant_weight(W, bits)
    pw = qc.pack_weight_t(dev(W), bits)
    for dtype in ("bf16", "f32"):
        x = random_x(rng, M, K, dtype)
        ws = qc.qlinear_workspace_t(M, K, N)
        ws.fill_(0x7f)
        acc = qc.qlinear_t(dev(x), pw, None, "none", "i32", workspace=ws)
        assert np.array_equal(acc.cpu().numpy(), oracle.gemm_i32(oracle.quant_act(x)[0], qw))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,w8,w4", [(1100, 4608, 1000, "ring 128 split", "ring 128 split"), (2200, 4608, 2050, "ring 192", "ring 256 split"),
                                         (1100, 2304, 1003, "ring 128 split", "ring 128 split"), (2200, 1152, 2049, "ring 192", "ring 192"),
                                         (6500, 2304, 899, "ring 256", "ring 256 split")])
def test_qlinear_ring_kernel_long_reductions(M, K, N, w8, w4, bits):
    """Every tile height at the reductions it is taken for, split and whole, symmetric, rotated and asymmetric codes."""
    for which in (dict(epi="gelu_tanh"), dict(out="f32", scheme="rot"), dict(out="f32", epi="gelu_erf", scheme="asym")):
        assert kernel_of(M, K, N, bits, **which).replace(" kept", "") == (w8 if bits == 8 else w4)
    rng = np.random.default_rng(M + K + N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    x = random_x(rng, M, K, "bf16")
    run_linear_case(x, W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(x, W, b, bits, "none", "f32", rot_block=64, act_bits=6)
    run_asym_case(x, W, b, bits, "gelu_erf", "f32")


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N", [(4033, 64, 1152), (4081, 192, 1146), (4097, 400, 1151), (4225, 64, 1152), (4225, 208, 1025),
                                   (4352, 64, 1148)])
def test_qlinear_ring_kernel_on_tiles_of_192_tokens(M, K, N, bits):
    """The height between the two, whose wavefronts of 48 tokens begin and end inside the panels of 64 the
    codes lie in: last tiles of 1, 49 and 65 live tokens, one that ends past the padded tokens (4225),
    and nothing written on either side of Y."""
    assert kernel_of(M, K, N, bits, epi="gelu_tanh") == kernel_of(M, K, N, bits, scheme="asym") == "ring 192"
    assert kernel_of(M, K, N, bits, epi="gelu_erf", out="f32") == "ring 192" and kernel_of(M, K, N, bits, out="f32") == "ring 192 kept"
    rng = np.random.default_rng(M + K + N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    x = random_x(rng, M, K, "bf16")
    run_linear_case(x, W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(x, W, None, bits, "gelu_erf", "f32", check_acc=False)
    run_asym_case(x, W, b, bits, "none", "bf16")
    pw, pad = qc.pack_weight_t(dev(W), bits), 4096
    for out, t in (("bf16", torch.bfloat16), ("f32", torch.float32)):
        want = qc.qlinear_t(dev(x), pw, dev(b), "none", out)
        buf = torch.full((M * N + 2 * pad,), -7.0, dtype=t, device="cuda")
        got = qc.qlinear_t(dev(x), pw, dev(b), "none", out, Y=buf[pad:pad + M * N].view(M, N))
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert bool((buf[:pad] == -7.0).all()) and bool((buf[pad + M * N:] == -7.0).all())


@pytest.mark.parametrize("M,K,N,bits", [(1025, 768, 1152, 4), (2001, 960, 1030, 4), (2047, 720, 2045, 4), (1281, 2304, 1148, 8), (2545, 2480, 1023, 8),
                                        (1281, 2480, 1027, 4), (3716, 2304, 1153, 4), (3841, 2480, 1146, 4)])
def test_qlinear_ring_kernel_split_in_two_halves_of_the_reduction(M, K, N, bits):
    """Few tiles of 128 tokens (the first six) and, with 4-bit weights, of 256: the shortest reductions it is taken for, halves
    of the same and of different length, last tiles of 1 token, and nothing written on either side of Y."""
    kernel = f"ring {128 if M < 3000 else 256} split"
    assert kernel_of(M, K, N, bits, epi="gelu_tanh") == kernel_of(M, K, N, bits, scheme="asym") == kernel
    assert kernel_of(M, K, N, bits, epi="gelu_erf", out="f32") == kernel_of(M, K, N, bits, out="f32") == kernel
    rng = np.random.default_rng(M + K + N + bits)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    b = (rng.standard_normal(N) * 0.01).astype(np.float32)
    x = random_x(rng, M, K, "bf16")
    run_linear_case(x, W, b, bits, "gelu_tanh", "bf16")
    run_linear_case(x, W, None, bits, "gelu_erf", "f32", check_acc=False)
    run_asym_case(x, W, b, bits, "none", "bf16")
    pw, pad = qc.pack_weight_t(dev(W), bits), 4096
    for out, t in (("bf16", torch.bfloat16), ("f32", torch.float32)):
        want = qc.qlinear_t(dev(x), pw, dev(b), "none", out)
        buf = torch.full((M * N + 2 * pad,), -7.0, dtype=t, device="cuda")
        got = qc.qlinear_t(dev(x), pw, dev(b), "none", out, Y=buf[pad:pad + M * N].view(M, N))
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert bool((buf[:pad] == -7.0).all()) and bool((buf[pad + M * N:] == -7.0).all())


def test_qlinear_ragged_rows_beyond_the_last_level_cache():
    """bf16 output of more than 256 MB whose rows are no multiple of 16 B: non-temporal stores at any alignment."""
    M, K, N = 262145, 64, 513
    rng = np.random.default_rng(513)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    run_linear_case(random_x(rng, M, K, "bf16"), W, None, 8, "none", "bf16", check_acc=False)


@pytest.mark.parametrize("M,N,epi,kernel", [(220001, 500, "gelu_tanh", "ring 256"), (220001, 501, "none", "ring 192"),
                                            (136701, 768, "gelu_tanh", "ring 256 kept"), (136701, 769, "none", "ring 256 kept"),
                                            (136701, 771, "gelu_erf", "ring 256 kept"), (138001, 764, "none", "ring 256")])
def test_qlinear_f32_output_of_any_size_through_the_caches(M, N, epi, kernel):
    """A short reduction whose f32 output of more than 400 MB stays on its way through the caches, where it is 16 times
    the codes, and on both sides of that: every row against the oracle's (they repeat)."""
    K, period = 64, 251
    assert 4 * M * N > 400 << 20 and kernel_of(M, K, N, 8, epi=epi, out="f32") == kernel
    rng = np.random.default_rng(N)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    x = random_x(rng, period, K, "bf16")
    qw, sw = oracle.quant_weight(W, 8)
    ref = oracle.qlinear(x, qw, sw, np.zeros(N, np.float32), {"none": oracle.EPI_NONE, "gelu_tanh": oracle.EPI_GELU_TANH, "gelu_erf": oracle.EPI_GELU_ERF}[epi], 8)
    Y = qc.qlinear_t(dev(x).repeat(-(-M // period), 1)[:M].contiguous(), qc.pack_weight_t(dev(W), 8), None, epi, "f32")
    torch.cuda.synchronize()
    assert_outputs_close(host_f64(Y[:period]), ref["y"], RTOL["f32"])
    assert torch.equal(Y[period:], Y[:-period])


@pytest.mark.parametrize("n", [1, 4, 1023 * 4, 1024 * 4 + 1, 16 * 4096, 16 * 4096 + 5, 48 * 4096 - 1, 48 * 4096, 3 << 17, (3 << 17) + 1, 1 << 19, (1 << 19) + 1, 170 * 4096 + 5,
                               (12 << 20) // 8, (12 << 20) // 8 + 1])
def test_reductions_on_both_sides_of_the_one_launch_form(n):
    """Up to 393216 elements the block that sees all partial sums finishes (16 blocks, more of them where
    each would have more than two chunks); beyond that a second launch does.  The workspace holds
    arbitrary bytes, then what the call before left in it."""
    rng = np.random.default_rng(n)
    cur, prev = rng.standard_normal(n).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    ref = np.asarray(oracle.latent_delta(cur, prev), np.float64)
    ws = torch.randint(0, 256, (qc.qc_latent_delta_workspace_bytes(n),), dtype=torch.uint8, device="cuda")
    c, p = dev(cur), dev(prev)
    first = qc.latent_delta_t(c, p, workspace=ws).cpu().numpy()
    assert np.all(np.abs(first - ref) <= 1e-5 * np.abs(ref))
    for _ in range(3):
        assert bits_equal(qc.latent_delta_t(c, p, workspace=ws).cpu().numpy(), first)
    other = qc.latent_delta_t(p, c, workspace=ws).cpu().numpy()
    ref = np.asarray(oracle.latent_delta(prev, cur), np.float64)
    assert np.all(np.abs(other - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("n", [32 * 4096, 32 * 4096 + 1, 3 << 17, (3 << 17) + 1, 128 * 4096, 3 << 18])
def test_latent_delta_in_one_launch_of_many_blocks(n):
    """Up to the 48 blocks that the largest input of the one-launch form has, then two launches."""
    rng = np.random.default_rng(n)
    cur, prev = rng.standard_normal(n).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    ref = np.asarray(oracle.latent_delta(cur, prev), np.float64)
    ws = torch.randint(0, 256, (qc.qc_latent_delta_workspace_bytes(n),), dtype=torch.uint8, device="cuda")
    for _ in range(4):
        got = qc.latent_delta_t(dev(cur), dev(prev), workspace=ws).cpu().numpy()
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("count", [1, 4, 5, 8])
@pytest.mark.parametrize("n", [32 * 2048 + 3, 3 << 15, (3 << 15) + 1])
def test_variation_on_both_sides_of_its_one_launch_form(n, count):
    rng = np.random.default_rng(n + count)
    cur, prevs = rng.standard_normal(n).astype(np.float32), [rng.standard_normal(n).astype(np.float32) for _ in range(count)]
    ref = np.asarray(oracle.cumulative_variation(cur, prevs), np.float64)
    ws = torch.randint(0, 256, (qc.qc_cumulative_variation_workspace_bytes(n, count),), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        got = qc.cumulative_variation_t(dev(cur), [dev(p) for p in prevs], workspace=ws).cpu().numpy()
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


def test_reductions_into_their_own_workspace():
    """Outputs inside the workspace, at its start or at the check word of a block's record, are what
    outputs elsewhere are: no block may spoil a check that is an output by then.  (The two forms add the
    same 64-bit sums in another order: a unit in the last place of the rounding to 32 bits, 1.2e-7.)"""
    rng = np.random.default_rng(8)
    a, b = (dev(rng.standard_normal(65536).astype(np.float32)) for _ in range(2))
    m = dev(rng.standard_normal((16, 2048)).astype(np.float32))
    for call, out, floats, bytes_ in (
            (lambda **k: qc.latent_delta_t(a, b, **k), "out3", 3, qc.qc_latent_delta_workspace_bytes(65536)),
            (lambda **k: qc.layer_similarity_t(a, b, **k), "out4", 4, qc.qc_layer_similarity_workspace_bytes(65536)),
            (lambda **k: qc.frame_gradient_norm_t(m, **k), "out2", 2, qc.qc_frame_gradient_norm_workspace_bytes(16, 2048)),
            (lambda **k: qc.cumulative_variation_t(a, [b, a], **k), "out", 3, qc.qc_cumulative_variation_workspace_bytes(65536, 2))):
        ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        want = call(workspace=ws).cpu()
        for at in (0, 8, 16, 24, bytes_ // 2, bytes_ - 4 * floats):
            inside = ws[at:at + 4 * floats].view(torch.float32)
            for _ in range(10):
                assert torch.allclose(call(workspace=ws, **{out: inside}).cpu(), want, rtol=1e-6, atol=0), (out, at)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("count", [1, 4, 5, 7, 8])
def test_variation_stays_in_its_workspace(count, large):
    """As many elements as the one-launch form takes, and two launches with 256 blocks or nearly, on a
    workspace of exactly the stated size with guard bytes behind it."""
    n = (12 << 20) // (4 * (count + 1)) if large else 3 << 15
    rng = np.random.default_rng(count)
    cur = rng.standard_normal(n).astype(np.float32)
    prevs = rng.standard_normal((count, n)).astype(np.float32)
    ref = np.asarray(oracle.cumulative_variation(cur, prevs), np.float64)
    size = qc.qc_cumulative_variation_workspace_bytes(n, count)
    buf = torch.full((size + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    got = qc.cumulative_variation_t(dev(cur), [dev(p) for p in prevs], workspace=buf[:size]).cpu().numpy()
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))
    assert bool((buf[size:] == 0x5a).all())


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, 3_698_757, 256 * 16384 + 5])
def test_similarity_on_both_sides_of_its_change_of_threads(n):
    rng = np.random.default_rng(n)
    a = rng.standard_normal(n).astype(np.float32)
    b = (a + 0.5 * rng.standard_normal(n)).astype(np.float32)
    got = qc.layer_similarity_t(dev(a), dev(b)).cpu().numpy()
    ref = np.asarray(oracle.layer_similarity(a, b), np.float64)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("dtype,n,one_launch", [("f32", 9 << 15, True), ("f32", 1 << 19, True), ("f32", (1 << 19) + 1, False), ("f32", 634887, False),
                                                ("f32", 653550, False), ("bf16", 5 << 18, True), ("bf16", (5 << 18) + 1, False)])
def test_similarity_in_one_launch_and_in_two(dtype, n, one_launch):
    """Which form a size takes shows in the workspace: one launch ends with zeros in its blocks' check words, every fourth
    of 64 at most; two leave three sums a block, none of them zero.  A used workspace and one of arbitrary bytes."""
    rng = np.random.default_rng(n)
    a = rng.standard_normal(n).astype(np.float32)
    b = (a + 0.5 * rng.standard_normal(n)).astype(np.float32)
    if dtype == "bf16":
        a, b = synth.to_bf16_bits(a), synth.to_bf16_bits(b)
    ref = np.asarray(oracle.layer_similarity(a, b), np.float64)
    ws = torch.randint(1, 256, (qc.qc_layer_similarity_workspace_bytes(n),), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        got = qc.layer_similarity_t(dev(a), dev(b), workspace=ws).cpu().numpy()
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))
        checks = ws.view(torch.int64)[3:4 * 64:4].cpu()
        zeros = int((checks == 0).sum())
        assert zeros == min(64, -(-n // (8192 if dtype == "f32" else 16384))) if one_launch else zeros == 0


@pytest.mark.parametrize("extra", [0, 1, 9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_launch_limits_of_similarity_and_gradient(dtype, extra):
    """The largest inputs of the one-launch form and the smallest beyond it, ragged ones among them."""
    rng = np.random.default_rng(extra)
    size = 4 if dtype == "f32" else 2
    n = (1 << 19 if dtype == "f32" else 5 << 18) + extra
    a, b = rng.standard_normal(n).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    m = rng.standard_normal((2, (1 << 20) // size + extra)).astype(np.float32)
    if dtype == "bf16":
        a, b, m = (synth.to_bf16_bits(t) for t in (a, b, m))
    for _ in range(2):
        got = qc.layer_similarity_t(dev(a), dev(b)).cpu().numpy()
        ref = np.asarray(oracle.layer_similarity(a, b), np.float64)
        assert np.all(np.abs(got[1:3] - ref[1:3]) <= 1e-5 * np.abs(ref[1:3]))
        # <a, b> of independent inputs is small against its terms: their rounding is what it is off by
        assert abs(got[0] - ref[0]) <= 1e-5 * math.sqrt(ref[1] * ref[2]) and abs(got[3] - ref[3]) <= 1e-5
        got = qc.frame_gradient_norm_t(dev(m)).cpu().numpy()
        ref = np.asarray(oracle.frame_gradient(m), np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("frames,inner", [(2, 1), (1, 4099), (3, 5), (17, 4096), (300, 5461), (1025, 1024), (40, 40001), (2049, 1288), (4097, 1027)])
def test_frame_gradient_slabs(frames, inner, dtype):
    """The blocks share the map in stretches of whole wavefronts' packs: fewer packs than a stretch, last
    stretches that are partial or empty, whole chunks and remainders, frames at every alignment."""
    rng = np.random.default_rng(frames * 7 + inner)
    m = rng.standard_normal((frames, inner)).astype(np.float32)
    if dtype == "bf16":
        m = synth.to_bf16_bits(m)
    got = qc.frame_gradient_norm_t(dev(m)).cpu().numpy()
    ref = np.asarray(oracle.frame_gradient(m), np.float64)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("frames,inner", [(2, 4), (2, 7), (3, 5), (2, 33), (16, 4099)])
def test_frame_gradient_is_rounded_once(frames, inner, dtype):
    """The squares of the binary32 differences are exact in binary64 and summed there: the result is off by
    its rounding to 32 bits, 2^-24 at most (and some 2^-52 for each term)."""
    for seed in range(20):
        m = np.random.default_rng(seed).standard_normal((frames, inner)).astype(np.float32)
        if dtype == "bf16":
            bits = synth.to_bf16_bits(m)
            m = oracle.bf16_bits_to_f64(bits).astype(np.float32)
        got = float(qc.frame_gradient_norm_t(dev(bits if dtype == "bf16" else m))[0])
        d = (m[1:] - m[:-1]).astype(np.float64)
        assert abs(got - float((d * d).sum())) <= (2.0 ** -24 + 1e-10) * float((d * d).sum())


def test_one_launch_reductions_replay_from_a_graph():
    """A replayed launch carries the same arguments as the time before, the number that marks its
    partial sums included: every replay has to form its result from its own inputs."""
    rng = np.random.default_rng(3)
    n, inner = 65536, 4099
    a, b = (torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda() for _ in range(2))
    m = torch.from_numpy(rng.standard_normal((16, inner)).astype(np.float32)).cuda()
    # the graph's workspaces are the graph's alone: between two replays nothing else writes a record there
    # that would take the place of the earlier replay's
    graphs, eager = ([torch.randint(0, 256, (16384,), dtype=torch.uint8, device="cuda") for _ in range(4)] for _ in range(2))
    outs = [torch.zeros(k, device="cuda") for k in (3, 4, 2, 4)]

    def step(ws, outs):
        qc.latent_delta_t(a, b, workspace=ws[0], out3=outs[0])
        qc.layer_similarity_t(a, b, workspace=ws[1], out4=outs[1])
        qc.frame_gradient_norm_t(m, workspace=ws[2], out2=outs[2])
        qc.cumulative_variation_t(a, [b, a, b], workspace=ws[3], out=outs[3])

    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        step(graphs, outs)
    for k in range(6):
        a.copy_(torch.from_numpy(rng.standard_normal(n).astype(np.float32)))
        m.mul_(1.0 + k)
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        want = [torch.zeros_like(o) for o in outs]
        step(eager, want)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(outs, want)), k
        ref = np.asarray(oracle.latent_delta(a.cpu().numpy(), b.cpu().numpy()), np.float64)
        assert np.all(np.abs(outs[0].cpu().numpy() - ref) <= 1e-5 * np.abs(ref))


@pytest.mark.parametrize("M,K,N,fused", [(1, 49152, 100, True), (1, 49154, 100, False), (1, 49152, 8224, True), (1, 49154, 8224, False),
                                         (1, 49152, 16500, True), (2, 24576, 100, True), (2, 24578, 8224, False), (1, 40960, 8224, True),
                                         (1, 40961, 8224, True), (1, 24576, 100, True), (2, 20480, 8224, True), (16, 1536, 8192, True), (32, 1280, 16384, True)])
def test_qlinear_on_few_tokens_with_the_longest_rows(M, K, N, fused):
    """The longest rows the one-launch form takes on tiles of 32, 64 and 128 channels, which need the most LDS (140 KiB), and
    the shortest that it does not, against quantization and GEMM as two calls."""
    assert qc.linear_plan(M, K, N)["fused"] == fused
    X = torch.randn(M, K, device="cuda").bfloat16()
    pw = qc.pack_weight_t(torch.randn(N, K, device="cuda"), 8)
    ws = qc.qlinear_workspace_t(M, K, N)
    got = qc.qlinear_t(X, pw, None, "none", "i32", workspace=ws)
    want, stream = torch.empty_like(got), torch.cuda.current_stream().cuda_stream
    ws.fill_(0x7f)
    assert qc.qc_qlinear_quant(X.data_ptr(), qc.QC_BF16, M, K, ws.data_ptr(), ws.numel(), stream) == qc.QC_OK
    assert qc.qc_qlinear_gemm(ws.data_ptr(), ws.numel(), M, K, pw.blob.data_ptr(), pw.scale.data_ptr(), 8, N, None,
                              qc.QC_EPI_NONE, want.data_ptr(), qc.QC_OUT_I32_ACC, stream) == qc.QC_OK
    assert torch.equal(got, want)


def test_few_token_kernel_with_much_lds_captured_first():
    """The 64 x 64 tile sums its wavefronts in 70 KB of LDS, which its first launch has to ask for: also
    when that launch is being captured, in a process that has launched nothing of it yet."""
    here = os.path.dirname(os.path.abspath(__file__))
    code = f"import sys; sys.path[:0] = [{os.path.dirname(here)!r}, {here!r}]; import test_gpu_kernel_edges as t; t.capture_the_largest_tile()"
    subprocess.run([sys.executable, "-c", code], check=True, timeout=100)


def capture_the_largest_tile():
    M, K, N = 1000, 192, 1000
    assert qc.qc_debug_gemm_kernel(M, K, N, 8) == 3
    rng = np.random.default_rng(64)
    x = dev(random_x(rng, M, K, "bf16"))
    for bits in (8, 4):
        pw = qc.pack_weight_t(dev((rng.standard_normal((N, K)) * 0.02).astype(np.float32)), bits)
        ws, Y = qc.qlinear_workspace_t(M, K, N), torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            qc.qlinear_t(x, pw, workspace=ws, Y=Y)
        for _ in range(3):
            Y.fill_(0)
            ws.fill_(0)
            graph.replay()
            torch.cuda.synchronize()
            got = Y.clone()
            assert torch.equal(got, qc.qlinear_t(x, pw))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K", [(1, 7), (32, 1024), (33, 1000), (8192, 1024), (8193, 1024)])
def test_tensor_scale_at_the_edges_of_its_slabs(M, K, dtype):
    """One slab exactly, one and a little, 256 slabs (bf16) exactly and more; the largest magnitude last."""
    rng = np.random.default_rng(M + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[-1, -1] = -9.0
    x = synth.to_bf16_bits(x) if dtype == "bf16" else x
    q_ref, s_ref = oracle.quant_act_tensor(x)
    qx, sx = qc.quant_act_tensor_t(dev(x))
    torch.cuda.synchronize()
    assert bits_equal(sx.cpu().numpy(), np.asarray(s_ref, np.float32).reshape(1)) and np.array_equal(qx.cpu().numpy(), q_ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tensor", [False, True])
@pytest.mark.parametrize("M,K", [(2, 1152), (64, 1000), (9, 2048), (9, 2064), (5, 6160), (3, 9216), (40, 1009)])
def test_nan_spoils_no_code_but_its_own(M, K, tensor, dtype):
    """A NaN beside the largest magnitude of its row: the scales and all other codes are those of the
    input with zeros in the NaNs' place, in the row kernels, their ragged form, the one-launch linear
    and the pass for the tensor's maximum."""
    rng = np.random.default_rng(M * 13 + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    cols = rng.integers(0, K // 2, M) * 2
    x[np.arange(M), cols + 1] = -30.0 - np.arange(M)
    x = synth.to_bf16_bits(x) if dtype == "bf16" else x.view(np.uint32)
    nans = np.array([0x7fc0, 0xffff, 0x7f81, 0xffc0], np.uint32)[np.arange(M) % 4] << (0 if dtype == "bf16" else 16)
    clean, bad = x.copy(), x.copy()
    clean[np.arange(M), cols] = 0
    bad[np.arange(M), cols] = nans.astype(x.dtype)
    if dtype == "f32":
        clean, bad = clean.view(np.float32), bad.view(np.float32)
    q_ref, s_ref = oracle.quant_act_tensor(clean) if tensor else oracle.quant_act(clean)
    s_ref = np.broadcast_to(np.asarray(s_ref, np.float32), (M,))
    here = np.zeros((M, K), bool)
    here[np.arange(M), cols] = True

    pw = qc.pack_weight_t(dev((rng.standard_normal((40, K)) * 0.02).astype(np.float32)), 8)
    make, call = ((qc.qlinear_tensor_workspace_t, qc.qlinear_tensor_t) if tensor else (qc.qlinear_workspace_t, qc.qlinear_t))
    ws = make(M, K, 40)
    call(dev(bad), pw, workspace=ws)
    qx, sx = qc.debug_workspace_act_t(ws, M, K)
    assert bits_equal(sx.cpu().numpy(), s_ref) and np.array_equal(qx.cpu().numpy()[~here], q_ref[~here])
    if K % 16 == 0:
        qx, sx = qc.quant_act_tensor_t(dev(bad)) if tensor else qc.quant_act_t(dev(bad))
        assert bits_equal(np.broadcast_to(sx.cpu().numpy(), (M,)), s_ref)
        assert np.array_equal(qx.cpu().numpy()[~here], q_ref[~here])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K", [(3, 1), (37, 7), (9, 127), (9, 129), (4099, 1000), (9, 2049), (5, 6145), (3, 9215), (2, 9217)])
def test_ragged_rows_in_the_fragment_layout(M, K, dtype):
    """Row lengths that are no multiple of 16: rows at every alignment, partial last pieces, both sides
    of each change of the number of steps; per token and with one scale for the tensor."""
    rng = np.random.default_rng(M * 7 + K)
    x = random_x(rng, M, K, dtype)
    xd = dev(x)
    for tensor in (False, True):
        q_ref, s_ref = oracle.quant_act_tensor(x) if tensor else oracle.quant_act(x)
        W = np.ones((8, K), np.float32)
        pw = qc.pack_weight_t(dev(W), 8)
        if tensor:
            ws = qc.qlinear_tensor_workspace_t(M, K, 8)
            ws.fill_(0x7f)
            acc = qc.qlinear_tensor_t(xd, pw, out="i32", workspace=ws)
        else:
            ws = qc.qlinear_workspace_t(M, K, 8)
            ws.fill_(0x7f)
            assert qc.qc_qlinear_quant(xd.data_ptr(), qc.QC_BF16 if dtype == "bf16" else qc.QC_F32, M, K, ws.data_ptr(),
                                       ws.numel(), torch.cuda.current_stream().cuda_stream) == qc.QC_OK
            acc = None
        qx, sx = qc.debug_workspace_act_t(ws, M, K)
        torch.cuda.synchronize()
        assert np.array_equal(qx.cpu().numpy(), q_ref)
        assert bits_equal(sx.cpu().numpy(), np.broadcast_to(np.asarray(s_ref, np.float32), (M,)))
        if acc is not None:
            assert np.array_equal(acc.cpu().numpy(), np.repeat(127 * q_ref.astype(np.int64).sum(axis=1)[:, None], 8, axis=1))
