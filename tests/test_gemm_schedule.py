"""Host logic of the GEMM stage: which of its two kernels a problem takes, and the static schedule
of the one that keeps its weight tile in LDS (every round exactly once, evenly dealt, a block
seldom changing its channel tile).  No GPU needed."""
import collections

import pytest

from paper_2503_06545_amd import binding as qc

BLOCKS = 256


def all_rounds(M, N):
    return [qc.gemm_schedule(M, N, b) for b in range(BLOCKS)]


@pytest.mark.parametrize("M,N", [(131072, 3456), (131072, 4608), (131072, 1152), (65536, 4608), (16384, 3456),
                                 (80037, 3401), (700, 392), (1, 1), (4096, 128), (100000, 129), (9000, 7000),
                                 (513, 5000)])
def test_every_round_is_dealt_exactly_once(M, N):
    n_tiles, chunks = -(-N // 128), -(-(-(-M // 256) * 256) // 512)
    seen = collections.Counter(r for rounds in all_rounds(M, N) for r in rounds)
    assert set(seen) == {(nt, c) for nt in range(n_tiles) for c in range(chunks)}
    assert set(seen.values()) == {1}


def test_block_out_of_range_and_bad_sizes_are_rejected():
    assert qc.qc_debug_gemm_schedule(1024, 128, BLOCKS, None, 0) == -1
    assert qc.qc_debug_gemm_schedule(1024, 128, -1, None, 0) == -1
    assert qc.qc_debug_gemm_schedule(0, 128, 0, None, 0) == -1
    assert qc.qc_debug_gemm_schedule(1024, 128, 0, None, -1) == -1


@pytest.mark.parametrize("M,N", [(131072, 3456), (131072, 4608), (65536, 4608)])
def test_paper_shapes_are_dealt_evenly_and_keep_their_channel_tile(M, N):
    rounds = all_rounds(M, N)
    counts = [len(r) for r in rounds]
    assert max(counts) == min(counts) == (N // 128) * (M // 512) // BLOCKS
    # a block changes its weight tile a handful of times at most
    changes = [sum(1 for a, b in zip(r, r[1:]) if a[0] != b[0]) for r in rounds]
    assert max(changes) <= 6 and sorted(changes)[len(changes) // 2] <= 1
    # at any step the blocks of one XCD (block b runs on XCD b % 8) read few distinct chunks:
    # what the XCD's L2 holds
    for xcd in range(8):
        mine = [rounds[b] for b in range(xcd, BLOCKS, 8)]
        for step in range(0, counts[0], 5):
            assert len({r[step][1] for r in mine}) <= 8


def test_which_problems_take_the_resident_kernel():
    # hidden 1152 (short reduction): QKV, fc1 and the out-projection at full size; not a token
    # count that leaves a block fewer than 6 rounds
    assert qc.qc_debug_gemm_kernel(131072, 1152, 3456, 8) == 2
    assert qc.qc_debug_gemm_kernel(131072, 1152, 4608, 8) == 2
    assert qc.qc_debug_gemm_kernel(131072, 1152, 4608, 4) == 2
    assert qc.qc_debug_gemm_kernel(65536, 1152, 4608, 8) == 2
    assert qc.qc_debug_gemm_kernel(131072, 1152, 1152, 8) == 2
    assert qc.qc_debug_gemm_kernel(32768, 1152, 3456, 8) == 2
    assert qc.qc_debug_gemm_kernel(16384, 1152, 3456, 8) == 1
    assert qc.qc_debug_gemm_kernel(16384, 1152, 4608, 8) == 1
    # fc2: a 128 x 4608 weight tile does not fit in LDS with 8-bit codes, nor with 4-bit ones
    assert qc.qc_debug_gemm_kernel(131072, 4608, 1152, 8) == 1
    assert qc.qc_debug_gemm_kernel(131072, 4608, 1152, 4) == 1
    # 4-bit codes fit up to K = 2304
    assert qc.qc_debug_gemm_kernel(131072, 2304, 4608, 4) == 2
    assert qc.qc_debug_gemm_kernel(131072, 2304, 4608, 8) == 1
    assert qc.qc_debug_gemm_kernel(131072, 2305, 4608, 4) == 0      # odd K with 4 bits
    assert qc.qc_debug_gemm_kernel(0, 1152, 4608, 8) == 0


def test_which_problems_take_the_few_token_kernel():
    """While tiles of 64 x 64 leave at most one block per CU.  A group of 128 channels is cut by every
    eighth: both of its 64-channel tiles have a channel of the output as soon as five do."""
    for N, tiles in ((1, 1), (4, 1), (5, 2), (32, 2), (64, 2), (128, 2), (129, 3), (132, 3), (133, 4), (1152, 18)):
        most = 64 * (256 // tiles)
        for K in (64, 1152, 4608):
            assert qc.qc_debug_gemm_kernel(most, K, N, 8) == 3, (N, K)
            assert qc.qc_debug_gemm_kernel(most + 1, K, N, 8) != 3, (N, K)


def test_the_plan_of_a_linear_agrees_with_the_kernel_it_takes():
    for M, K, N, bits in ((2, 1152, 6912, 8), (1000, 64, 1000, 8), (4099, 1000, 1301, 8), (16384, 1152, 3456, 8), (131072, 1152, 3456, 4)):
        which = {1: "ring", 2: "resident", 3: "few"}[qc.qc_debug_gemm_kernel(M, K, N, bits)]
        assert qc.linear_plan(M, K, N, bits)["kernel"] == which
    assert qc.linear_plan(2, 1152, 6912) == {"kernel": "few", "tokens": 16, "split": False, "kept": False, "fused": True,
                                             "nt_loads": False, "nt_stores": False}
    assert qc.linear_plan(65536, 1152, 4608, epi="gelu_erf")["kernel"] == "ring"      # the epilogue decides too
    assert qc.linear_plan(131072, 1152, 3456, out="i32")["kernel"] == "resident"
    assert qc.linear_plan(131072, 768, 4608, out="f32")["kernel"] == "ring"           # and the output's type
    assert qc.linear_plan(1024, 4608, 1152)["split"] and qc.linear_plan(1024, 4608, 1152)["tokens"] == 128
    assert qc.linear_plan(8192, 1152, 1152, out="f32")["kept"] and not qc.linear_plan(1200, 1152, 1152, out="f32")["kept"]
    for bad in (dict(M=0), dict(K=0), dict(bits=3), dict(K=1153, bits=4), dict(K=1000, scheme="rot"), dict(K=1000, scheme="asym")):
        with pytest.raises(qc.QcError):
            qc.linear_plan(**{"M": 4096, "K": 1152, "N": 1152, **bad})


MB = 1 << 20


@pytest.mark.parametrize("x", ["bf16", "f32"])
@pytest.mark.parametrize("scheme", ["token", "rot", "asym"])
def test_which_quantizers_load_past_the_caches(x, scheme):
    """Whole lines of 128 B from 160 MB of input and codes on, other rows, whose shared lines would be fetched twice, from
    256 MB; the codes are stored past the caches from 288 MB of them on."""
    size = 3 if x == "bf16" else 5
    for K, from_mb in ((1152, 160), (4608, 160), (544, 256), (1200, 256), (1552, 256), (2576, 256)):
        if x == "f32" and K == 544:
            continue                                   # 17 whole lines
        for mb, loads in ((from_mb - 8, False), (from_mb + 8, True), (280, True)):
            plan = qc.linear_plan(mb * MB // (size * K), K, 56, x=x, scheme=scheme)
            assert plan["nt_loads"] == loads and not plan["nt_stores"], (K, mb)
        plan = qc.linear_plan(300 * MB // K, K, 1152, x=x, scheme=scheme)
        assert plan["nt_stores"] and plan["nt_loads"] == (from_mb == 160)
    for M, K, N in ((105713, 544, 56), (26425, 2576, 45), (39840, 1552, 1152)):
        assert not qc.linear_plan(M, K, N)["nt_loads"]
    assert qc.linear_plan(65536, 1152, 4608, epi="gelu_tanh")["nt_loads"]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,x,most", [(32, 4096, "bf16", 2816), (67, 1152, "f32", 2816), (10, 4096, "bf16", 4864), (1, 4096, "f32", 49152),
                                        (256, 1200, "f32", 3072), (687, 565, "f32", 2060), (687, 565, "bf16", 3072), (991, 46, "f32", 1784),
                                        (1091, 92, "f32", 3072), (2687, 122, "f32", 3072), (100, 2048, "f32", 3072), (640, 1152, "f32", 1152), (800, 1152, "f32", 1152)])
def test_the_longest_rows_that_are_quantized_in_the_launch_of_the_gemm(M, N, x, most, bits):
    assert qc.linear_plan(M, most, N, bits, x=x)["fused"]
    assert not qc.linear_plan(M, most + 2, N, bits, x=x)["fused"]
    if (M, x) == (687, "f32"):   # where the quantizer alone costs more, one launch goes on a little
        assert qc.linear_plan(M, 2592, N, bits, x=x, scheme="asym")["fused"]
        assert not qc.linear_plan(M, 2608, N, bits, x=x, scheme="asym")["fused"]


@pytest.mark.parametrize("bits,M,K,N,tokens", [
    (8, 12000, 3072, 576, 256), (8, 6400, 4608, 1152, 256), (8, 1775, 4608, 4608, 256), (8, 2767, 4528, 2797, 256),   # one tile of 256 to a CU
    (8, 6400, 1536, 1152, 128), (8, 6400, 1152, 1152, 128), (8, 5120, 4608, 1152, 192), (8, 7390, 1152, 1152, 192)])
def test_heights_of_tiles_that_are_one_or_two_to_a_cu(bits, M, K, N, tokens):
    plan = qc.linear_plan(M, K, N, bits)
    assert plan["kernel"] == "ring" and not plan["split"] and plan["tokens"] == tokens


@pytest.mark.parametrize("M,K,N,epi,out,tokens,kept", [
    (2850, 1152, 4608, "gelu_erf", "f32", 256, False), (3649, 352, 3456, "gelu_erf", "f32", 256, False),
    (11670, 1152, 1152, "gelu_erf", "f32", 256, False), (2850, 1152, 4608, "gelu_erf", "bf16", 128, False),
    (800, 1152, 4608, "none", "f32", 128, False), (10535, 1152, 1152, "gelu_tanh", "f32", 128, True)])
def test_heights_of_tiles_whose_f32_output_goes_past_the_caches(M, K, N, epi, out, tokens, kept):
    plan = qc.linear_plan(M, K, N, epi=epi, out=out)
    assert (plan["kernel"], plan["tokens"], plan["kept"]) == ("ring", tokens, kept)


@pytest.mark.parametrize("scheme,bits,M,K,N,x,tokens", [
    ("asym", 8, 37714, 256, 3456, "f32", 256), ("asym", 8, 11666, 1152, 4608, "bf16", 256), ("token", 8, 11666, 1152, 4608, "bf16", 192),
    ("asym", 4, 11666, 1152, 4608, "bf16", 192), ("asym", 8, 2478, 1152, 3456, "bf16", 192), ("asym", 8, 4096, 1152, 1152, "bf16", 192), ("asym", 8, 9843, 4608, 1152, "bf16", 192)])
def test_heights_of_tiles_with_a_zero_point(scheme, bits, M, K, N, x, tokens):
    plan = qc.linear_plan(M, K, N, bits, x=x, scheme=scheme)
    assert plan["kernel"] == "ring" and plan["tokens"] == tokens


@pytest.mark.parametrize("M,K,N,epi,kept", [
    (57258, 192, 4608, "none", True), (150000, 576, 2304, "none", True), (150000, 577, 2304, "none", False),
    (57258, 192, 4608, "gelu_erf", True), (88010, 384, 3984, "gelu_erf", True), (97902, 576, 3984, "gelu_erf", False),
    (33000, 576, 3984, "gelu_erf", True), (34000, 576, 3984, "gelu_erf", False), (220001, 64, 500, "none", False), (137000, 64, 768, "none", True)])
def test_short_reductions_whose_f32_output_of_any_size_stays_in_the_caches(M, K, N, epi, kept):
    assert qc.linear_plan(M, K, N, epi=epi, out="f32")["kept"] == kept


@pytest.mark.parametrize("scheme,bits,M,K,N,kernel", [("asym", 8, 81720, 768, 3456, "resident"), ("asym", 8, 90440, 688, 3984, "resident"),
                                                      ("asym", 8, 81720, 576, 3456, "ring"), ("asym", 4, 81720, 768, 3456, "ring"),
                                                      ("token", 8, 81720, 768, 3456, "ring"), ("token", 8, 81720, 784, 3456, "resident")])
def test_which_short_reductions_with_f32_output_keep_their_weights_resident(scheme, bits, M, K, N, kernel):
    assert qc.linear_plan(M, K, N, bits, out="f32", scheme=scheme)["kernel"] == kernel
