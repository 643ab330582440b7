"""Every tile shape of the LDS-tiled GEMM (Eq. 3 over K + k), forced one at a
time through the library's tuning entry point, against the oracle's float64
GEMM: max |dY| <= 1e-3 max |Y|.  Covers row-major activation scales at rows that
start on dwords (K + k a multiple of 128) and at any byte, ragged M, N and K + k,
row and feature tiles cut by the operand edges, steps fewer than the pipeline's
stages and every remainder of them, and grouped calls with empty experts."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import prquant as pq                               # noqa: E402
from paper_2609_22106_amd import inputs                        # noqa: E402
from tests.gpu_util import assert_gemm_close, dev, host, say   # noqa: E402

pytestmark = pytest.mark.gpu

SHAPE_IDS = (0, 1, 2, 3)   # 256x256, 256x128, 128x128, 256x320


def _lib():
    from paper_2609_22106_amd import build, prq  # noqa: F401  (prq loads torch first)
    lib = ctypes.CDLL(build.PROBE_LIB)
    P, I = ctypes.c_void_p, ctypes.c_int
    lib.prq_tune_gemm_tile.argtypes = [P, P, I, P, I, P, P, I, I, P, I, P]
    lib.prq_tune_gemm_tile.restype = I
    return lib


def _run(shape, Aq, Asc, Wq, Wsc, off=None, E=1):
    from paper_2609_22106_amd import prq
    M, N, K_aug = Aq.shape[0], Wq.shape[-2], Aq.shape[1] * 2
    A, As = dev(Aq), dev(Asc)
    W = prq.prq_pack_weight(dev(Wq), dev(Wsc))
    Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    offd = dev(off) if off is not None else None
    rc = _lib().prq_tune_gemm_tile(A.data_ptr(), As.data_ptr(), M,
                                   offd.data_ptr() if offd is not None else None, E,
                                   W.Wp.data_ptr(), W.Wps.data_ptr(), N, K_aug, Y.data_ptr(),
                                   shape, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, rc
    torch.cuda.synchronize()
    return host(Y)


DENSE = [(300, 384, 1024),    # scale rows on dwords, ragged rows
         (513, 272, 1152),    # dwords, ragged rows and features (272 = 17 tiles of 16)
         (40, 512, 9984),     # dwords, the down_proj reduction length, one row tile
         (257, 272, 1088),    # scale rows at any byte (1088 = 8.5 steps of 128)
         (130, 144, 4192),    # any byte, 32.75 steps
         (17, 48, 96),        # any byte, one partial step (fewer steps than stages)
         (64, 256, 256)]      # dwords, two steps


@pytest.mark.parametrize("M,N,K_aug", DENSE)
@pytest.mark.parametrize("shape", SHAPE_IDS)
def test_tile_shape_dense(shape, M, N, K_aug):
    rng = np.random.default_rng(M * 131 + N * 7 + K_aug + shape)
    Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
    Wq, Wsc = inputs.random_mxfp4(rng, N, K_aug)
    say("tile shape case:", shape, M, N, K_aug)
    assert_gemm_close(_run(shape, Aq, Asc, Wq, Wsc), pq.gemm(Aq, Asc, Wq, Wsc),
                      f"shape {shape} {M}x{N}x{K_aug}")


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("shape", SHAPE_IDS)
def test_tile_shape_step_remainders(shape, packed):
    """One to nine K steps: fewer than the stages, whole groups of them, and every
    remainder after one and two groups; the last step whole and partial."""
    from paper_2609_22106_amd import prq
    from tests.packing import pack_rows
    M, N = 130, 144
    for K_aug in (96, 128, 224, 256, 384, 480, 512, 608, 640, 768, 896, 1024, 1056, 1152):
        rng = np.random.default_rng(K_aug + shape)
        Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
        Wq, Wsc = inputs.random_mxfp4(rng, N, K_aug)
        W = prq.prq_pack_weight(dev(Wq), dev(Wsc))
        A, As = (map(dev, pack_rows(Aq, Asc)) if packed else (dev(Aq), dev(Asc)))
        Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        say("tile step remainder case:", shape, packed, K_aug)
        assert _split_lib().prq_tune_gemm_tile_split(
            A.data_ptr(), As.data_ptr(), M, W.Wp.data_ptr(), W.Wps.data_ptr(), N, K_aug, Y.data_ptr(),
            shape, 1, int(packed), None, 0, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert_gemm_close(host(Y), pq.gemm(Aq, Asc, Wq, Wsc), f"shape {shape} packed {packed} K_aug {K_aug}")


GROUPED = [([0, 300, 0, 5, 260], 272, 1024),   # dwords
           ([3, 0, 17, 1, 0], 48, 1088),       # any byte
           ([0, 0, 200], 128, 832)]            # any byte, the expert reduction length


@pytest.mark.parametrize("counts,N,K_aug", GROUPED)
@pytest.mark.parametrize("shape", SHAPE_IDS)
def test_tile_shape_grouped(shape, counts, N, K_aug):
    rng = np.random.default_rng(sum(counts) * 17 + N + K_aug + shape)
    E, M = len(counts), sum(counts)
    off = inputs.routed_offsets(counts)
    Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
    Wq, Wsc = inputs.random_mxfp4(rng, (E, N), K_aug)
    say("tile shape grouped case:", shape, counts, N, K_aug)
    Y = _run(shape, Aq, Asc, Wq, Wsc, off=off, E=E)
    assert_gemm_close(Y, pq.grouped_gemm(Aq, Asc, off, Wq, Wsc),
                      f"grouped shape {shape} {counts} {N}x{K_aug}")


def _split_lib():
    from paper_2609_22106_amd import build, prq  # noqa: F401
    lib = ctypes.CDLL(build.PROBE_LIB)
    P, I = ctypes.c_void_p, ctypes.c_int
    lib.prq_tune_gemm_tile_split.argtypes = [P, P, I, P, P, I, I, P, I, I, I, P, ctypes.c_size_t,
                                             P]
    lib.prq_tune_gemm_tile_split.restype = I
    return lib


# (M, N, K_aug, splits): split ranges of unequal length, more splits than
# whole 4-step groups, a last range of one step, ragged rows and features.
SPLIT = [(300, 272, 1024, 3),      # 8 steps -> 3 + 3 + 2
         (513, 144, 9984, 8),      # 78 steps -> 10 x 7 + 8
         (40, 512, 4192, 4),       # 33 steps -> 9 + 9 + 9 + 6 (scale rows at any byte)
         (129, 64, 1152, 9),       # 9 steps -> one step each
         (64, 256, 640, 2)]        # 5 steps -> 3 + 2


@pytest.mark.parametrize("M,N,K_aug,splits", SPLIT)
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("shape", SHAPE_IDS)
def test_tile_split_k(shape, packed, M, N, K_aug, splits):
    """The tile GEMM split along K (partial sums in the workspace, added to Y in
    a fixed order by the reduction): within the tolerance of the oracle, and
    bit-identical over two calls (deterministic)."""
    from paper_2609_22106_amd import prq
    from tests.packing import pack_rows
    rng = np.random.default_rng(M * 3 + N + K_aug + splits)
    Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
    Wq, Wsc = inputs.random_mxfp4(rng, N, K_aug)
    W = prq.prq_pack_weight(dev(Wq), dev(Wsc))
    A, As = (map(dev, pack_rows(Aq, Asc)) if packed else (dev(Aq), dev(Asc)))
    ws = torch.full((max(splits - 1, 1) * M * N,), float("nan"), dtype=torch.float32, device="cuda")
    outs = []
    for _ in range(2):
        Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        say("tile split case:", shape, packed, M, N, K_aug, splits)
        rc = _split_lib().prq_tune_gemm_tile_split(
            A.data_ptr(), As.data_ptr(), M, W.Wp.data_ptr(), W.Wps.data_ptr(), N, K_aug,
            Y.data_ptr(), shape, splits, int(packed), ws.data_ptr(), ws.numel() * 4,
            torch.cuda.current_stream().cuda_stream)
        assert rc == 0, rc
        torch.cuda.synchronize()
        outs.append(host(Y))
    np.testing.assert_array_equal(outs[0], outs[1])
    assert_gemm_close(outs[0], pq.gemm(Aq, Asc, Wq, Wsc),
                      f"split shape {shape} packed {packed} {M}x{N}x{K_aug} / {splits}")


# Planned calls (row-major, packed) without room for a split: one region and two;
# Y on both sides of the size up to which it is stored non-temporally (7 million values); the narrowest N,
# fewer rows than a tile, more tiles than several rounds; N no multiple of a tile.
PLANNED = [(66, 16, 1056), (70, 13824, 640), (300, 1936, 1312), (1220, 4096, 288), (1222, 4096, 288),
           (1708, 4096, 288), (1710, 4096, 288), (1537, 9728, 416), (2500, 9728, 288), (4096, 6144, 160), (6000, 4112, 160), (8200, 272, 544)]


@pytest.mark.parametrize("M,N,K_aug", PLANNED)
@pytest.mark.parametrize("packed", [True, False])
def test_planned_call_equals_forced_shape(packed, M, N, K_aug):
    """Every tile shape adds a row's products in the same order, so an unsplit
    planned call gives the bits of the 128 x 128 shape forced over all columns
    (itself checked against the oracle above), wherever the planner cuts N."""
    from paper_2609_22106_amd import prq
    from tests.packing import pack_rows
    rng = np.random.default_rng(M + N + K_aug)
    Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
    Wq, Wsc = inputs.random_mxfp4(rng, N, K_aug)
    W = prq.prq_pack_weight(dev(Wq), dev(Wsc))
    A, As = (map(dev, pack_rows(Aq, Asc)) if packed else (dev(Aq), dev(Asc)))
    want, got = (torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    stream = torch.cuda.current_stream().cuda_stream
    say("planned case:", packed, M, N, K_aug)
    rc = _split_lib().prq_tune_gemm_tile_split(A.data_ptr(), As.data_ptr(), M, W.Wp.data_ptr(),
                                               W.Wps.data_ptr(), N, K_aug, want.data_ptr(), 2, 1,
                                               int(packed), 0, 0, stream)
    assert rc == 0, rc
    call = prq._gemm_packed if packed else prq._gemm
    assert call(A.data_ptr(), As.data_ptr(), M, W.Wp.data_ptr(), W.Wps.data_ptr(), N, K_aug,
                got.data_ptr(), None, 0, stream) == 0
    torch.cuda.synchronize()
    assert not torch.isnan(want).any()
    assert torch.equal(want, got)


# (counts, N, K_aug, CUs): experts of exactly a wide tile's 160 rows, one more and
# one fewer, of a row, empty first and last; tiles cut by the lead of a shared
# 16-row block; N below, at and past the 256 columns; steps below and past the four
# stages; fewer workgroups than tiles (8 CUs) and more.
WIDE = [([0, 160, 161, 159, 1, 0], 256, 832, 8), ([3, 157, 320, 5, 330], 240, 544, 256),
        ([17, 0, 0, 500, 31, 16, 144, 176, 20, 40], 528, 416, 8), ([1], 16, 32, 256),
        ([40] * 70, 272, 1056, 16)]


@pytest.mark.parametrize("counts,N,K_aug,cus", WIDE)
def test_wide_persistent_grouped(counts, N, K_aug, cus):
    """The persistent grouped kernel's 160 x 256 tiles: the bits of its 128 x 128
    tiles (both add a row's products in K order) and the oracle's product."""
    from paper_2609_22106_amd import build, prq
    from tests.packing import pack_rows
    rng = np.random.default_rng(sum(counts) + N)
    E, M = len(counts), sum(counts)
    off = inputs.routed_offsets(counts)
    Aq, Asc = inputs.random_mxfp4(rng, M, K_aug)
    Wq, Wsc = inputs.random_mxfp4(rng, (E, N), K_aug)
    W = prq.prq_pack_weight(dev(Wq), dev(Wsc))
    A, As = map(dev, pack_rows(Aq, Asc))
    do = dev(off)
    lib = ctypes.CDLL(build.PROBE_LIB)
    P, I = ctypes.c_void_p, ctypes.c_int
    lib.prq_tune_grouped_gemm_tile_packed.argtypes = [P, P, I, P, I, P, P, I, I, P, I, I, P]
    out = []
    for shape in (4, 5):
        Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        say("wide grouped case:", shape, counts[:8], N, K_aug, cus)
        assert lib.prq_tune_grouped_gemm_tile_packed(
            A.data_ptr(), As.data_ptr(), M, do.data_ptr(), E, W.Wp.data_ptr(), W.Wps.data_ptr(), N,
            K_aug, Y.data_ptr(), shape, cus, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        out.append(host(Y))
    np.testing.assert_array_equal(out[0].view(np.uint32), out[1].view(np.uint32))
    assert_gemm_close(out[1], pq.grouped_gemm(Aq, Asc, off, Wq, Wsc), f"wide {N}x{K_aug}")
