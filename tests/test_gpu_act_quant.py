"""prq_quant_act (fused inverse scale, permutation gather, MXFP4 quantize and
online tail copy) against the oracle: codes and scale bytes bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import prquant as pq                       # noqa: E402
from paper_2609_22106_amd import inputs                # noqa: E402
from tests.golden import load_hand_blocks              # noqa: E402
from tests.gpu_util import dev, host, replay_us, say              # noqa: E402

pytestmark = pytest.mark.gpu


def _pos(inv, perm):
    """Inverse scales in position order, inv_s[perm[p]] (per group when 2-D)."""
    if perm is None:
        return inv
    return np.take_along_axis(np.asarray(inv), np.asarray(perm).astype(np.int64), axis=-1)


def _gpu_quant(X_bits, K, k, inv=None, perm=None, offsets=None, G=1, ld=None):
    from paper_2609_22106_amd import prq
    M = X_bits.shape[0]
    if ld is not None and ld != K:
        Xp = np.zeros((M, ld), np.uint16)
        Xp[:, :K] = X_bits
        Xd = dev(Xp)
    else:
        Xd = dev(X_bits)
    Aq, Asc = prq.prq_quant_act(Xd, K, k, None if inv is None else dev(_pos(inv, perm)),
                                None if perm is None else dev(perm),
                                None if offsets is None else dev(offsets), G)
    torch.cuda.synchronize()
    return host(Aq), host(Asc)


def _check(X_bits, K, k, inv, perm, what, **kw):
    say("act_quant case:", what, X_bits.shape, "k =", k)
    Aq, Asc = _gpu_quant(X_bits, K, k, inv, perm, **kw)
    rq, rs = pq.quant_act(X_bits, inv, perm, k)
    np.testing.assert_array_equal(Asc, rs, err_msg=f"{what}: scales")
    np.testing.assert_array_equal(Aq, rq, err_msg=f"{what}: codes")


def test_tiny_workload():
    c = inputs.tiny_case()
    art = pq.prepare(c.W, c.Xcal, 0.5, 64)
    _check(c.X, 1024, 64, art["inv_scale"], art["perm"], "tiny 16x1024 k64")


@pytest.mark.parametrize("M", [1, 3, 17, 257, 1000])
def test_ragged_rows(M):
    c = inputs.make_dense("r", N=64, K=1024, M=M, T=32, k_tail=64, n_out=8, out_scale=40.0,
                          heavy_tail=False, seed=M)
    art = pq.prepare(c.W, c.Xcal, 0.5, 64)
    _check(c.X, 1024, 64, art["inv_scale"], art["perm"], f"M={M}")


# (at least 1025 rows or more than 1024 x 768 channels: fewer are the few-rows kernel's)
@pytest.mark.parametrize("K,k,M", [(768, 64, 1131), (2048, 64, 389), (4096, 96, 200), (4160, 160, 197),
                                   (6144, 64, 131), (9728, 224, 85), (12320, 288, 66), (16384, 512, 67)])
def test_many_row_kernel_shapes(K, k, M):
    """The many-row kernel at every units-per-thread count (K/8 over 512
    threads: 1 with several rows per pass, 1, 2, 3, 4 and the largest K),
    ragged row counts, random permutation and scales."""
    rng = np.random.default_rng(K + M)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K)) * 3).astype(np.float32))
    perm = rng.permutation(K).astype(np.int32)
    inv = rng.uniform(0.05, 8.0, K).astype(np.float32)
    _check(X, K, k, inv, perm, f"K={K} k={k} M={M}")


def test_few_row_kernel_grouped():
    """Grouped rows through the few-rows kernel (at most 64 rows): a workgroup's
    row range crosses experts, empty experts included."""
    rng = np.random.default_rng(13)
    E, K, k = 6, 768, 64
    counts = [3, 0, 20, 1, 0, 9]
    off = inputs.routed_offsets(counts)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((int(off[-1]), K)) * 3).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(E)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (E, K)).astype(np.float32)
    say("act_quant case: grouped few rows", counts)
    Aq, Asc = _gpu_quant(X, K, k, inv, perm, offsets=off, G=E)
    rq, rs = pq.quant_act_grouped(X, inv, perm, off, k)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)


@pytest.mark.parametrize("M", [1, 5, 48, 64])
def test_few_row_kernel_largest_rows(M):
    """K = 16384 (four staged rows of 32 KiB per workgroup at 64 rows)."""
    rng = np.random.default_rng(M)
    K, k = 16384, 512
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K)) * 3).astype(np.float32))
    perm = rng.permutation(K).astype(np.int32)
    inv = rng.uniform(0.05, 8.0, K).astype(np.float32)
    _check(X, K, k, inv, perm, f"K=16384 M={M}")


def test_many_row_kernel_grouped_two_units_per_thread():
    rng = np.random.default_rng(12)
    E, K, k = 4, 4160, 160
    counts = [60, 0, 130, 9]
    off = inputs.routed_offsets(counts)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((int(off[-1]), K)) * 2).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(E)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (E, K)).astype(np.float32)
    say("act_quant case: grouped K=4160", counts)
    Aq, Asc = _gpu_quant(X, K, k, inv, perm, offsets=off, G=E)
    rq, rs = pq.quant_act_grouped(X, inv, perm, off, k)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)


def test_no_scale_no_perm_k0():
    rng = np.random.default_rng(4)
    X = inputs.f32_to_bf16_bits(rng.standard_normal((33, 512)).astype(np.float32) * 3)
    _check(X, 512, 0, None, None, "identity k0")


def test_whole_row_is_tail():
    """k = K: every block is copied once more."""
    c = inputs.make_dense("t", N=32, K=256, M=9, T=8, k_tail=256, n_out=2, seed=3)
    art = pq.prepare(c.W, c.Xcal, 0.5, 256)
    _check(c.X, 256, 256, art["inv_scale"], art["perm"], "k = K")


def test_random_permutation_and_scales():
    rng = np.random.default_rng(9)
    K = 2048
    X = inputs.f32_to_bf16_bits((rng.standard_normal((40, K)) * 5).astype(np.float32))
    perm = rng.permutation(K).astype(np.int32)
    inv = rng.uniform(0.01, 20.0, K).astype(np.float32)
    _check(X, K, 96, inv, perm, "random perm")


@pytest.mark.parametrize("K,M", [(96, 2), (1056, 31), (4192, 64), (9728, 17)])
def test_few_row_kernel_staged_row_pads(K, M):
    """The few-rows kernel copies each row whole into LDS in 1 KiB pieces: rows
    whose byte length is not a multiple of 1 KiB (the last piece partly past
    the row), strided rows (ld = K + 32), 1 to 4 rows per workgroup."""
    rng = np.random.default_rng(K + M)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K)) * 3).astype(np.float32))
    perm = rng.permutation(K).astype(np.int32)
    inv = rng.uniform(0.05, 8.0, K).astype(np.float32)
    k = 32
    say("act_quant case: staged row pads", K, M)
    Aq, Asc = _gpu_quant(X, K, k, inv, perm, ld=K + 32)
    rq, rs = pq.quant_act(X, inv, perm, k)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)


def test_strided_rows():
    c = inputs.tiny_case()
    art = pq.prepare(c.W, c.Xcal, 0.5, 64)
    _check(c.X, 1024, 64, art["inv_scale"], art["perm"], "ld 1056", ld=1056)


def test_hand_blocks_and_edge_values():
    """The hand-derived blocks (rounded to bf16), subnormals, signed zeros,
    huge values and exact E2M1 ties, with no scaling or permutation."""
    blocks = [b["values"] for b in load_hand_blocks()]
    rng = np.random.default_rng(1)
    ties = np.array([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, 7.0, -0.25, -2.5, 6.0, -6.0] * 2
                    + [7.9, -7.9, 0.0, -0.0, 2.0 ** -130, -(2.0 ** -133), 3e38, -3e38], np.float32)
    extra = [np.concatenate([ties, rng.standard_normal(32 - ties.size % 32 if ties.size % 32 else 0)
                             .astype(np.float32)])]
    row = np.concatenate(blocks + extra)
    row = row[: row.size // 32 * 32]
    X = inputs.f32_to_bf16_bits(np.stack([row, -row, row * 0.75, row * np.float32(2.0 ** -120)]))
    K = X.shape[1]
    _check(X, K, 64, None, None, "hand blocks")


def test_full_decode_rows(c1_art):
    c, art = c1_art
    _check(c.X, 9728, 256, art["inv_scale"], art["perm"], "9728 k256 M=64")


def test_full_prefill_rows_sampled(c1_art):
    """8192 rows through the kernel; 256 sampled rows checked against the oracle."""
    _, art = c1_art
    c = inputs.down_proj_prefill()
    Aq, Asc = _gpu_quant(c.X, 9728, 256, art["inv_scale"], art["perm"])
    rows = np.sort(np.random.default_rng(0).choice(c.X.shape[0], 256, replace=False))
    rows = np.unique(np.concatenate([rows, [0, c.X.shape[0] - 1]]))
    rq, rs = pq.quant_act(c.X[rows], art["inv_scale"], art["perm"], 256)
    np.testing.assert_array_equal(Asc[rows], rs)
    np.testing.assert_array_equal(Aq[rows], rq)


def test_grouped_experts_with_empty_groups():
    rng = np.random.default_rng(2)
    E, K, k = 6, 768, 64
    counts = [5, 0, 70, 1, 0, 33]
    off = inputs.routed_offsets(counts)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((int(off[-1]), K)) * 4).astype(np.float32))
    perms, invs = [], []
    for e in range(E):
        c = inputs.make_dense("g", N=32, K=K, M=1, T=16, k_tail=k, n_out=4, seed=100 + e)
        a = pq.prepare(c.W, c.Xcal, 0.5, k)
        perms.append(a["perm"])
        invs.append(a["inv_scale"])
    perm, inv = np.stack(perms), np.stack(invs)
    say("act_quant case: grouped", counts)
    Aq, Asc = _gpu_quant(X, K, k, inv, perm, offsets=off, G=E)
    rq, rs = pq.quant_act_grouped(X, inv, perm, off, k)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)


# (K, k, M, groups): both sides of the line between the few-rows and the many-rows
# kernels (1024 rows; 1024 x 768 channels), rows past the last 16-row block's
# start filled by several workgroups (one to fifteen of them), more groups than a
# wave has lanes, most of them empty, and the most groups there can be.
LINE = [(768, 64, 1024, 1), (768, 64, 1025, 1), (32, 32, 1024, 1), (32, 0, 1039, 1), (2560, 64, 307, 1),
        (2560, 64, 310, 1), (768, 64, 1024, 128), (768, 32, 1031, 300), (768, 64, 200, 65),
        (2048, 96, 385, 70), (64, 32, 1300, 4096), (64, 32, 90, 4096)]


@pytest.mark.parametrize("K,k,M,G", LINE)
def test_kernel_choice_padding_and_group_search(K, k, M, G):
    from paper_2609_22106_amd import prq
    from tests.packing import pack_rows
    rng = np.random.default_rng(K + M + G)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K)) * 3).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(G)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (G, K)).astype(np.float32)
    off = None
    if G > 1:   # a few crowded groups, the first and the last row's among empty ones
        at = np.sort(rng.choice(np.arange(1, G - 1), 5, replace=False))
        off = inputs.routed_offsets(np.bincount(rng.choice(at, M), minlength=G))
        rq, rs = pq.quant_act_grouped(X, inv, perm, off, k)
    else:
        perm, inv = perm[0], inv[0]
        rq, rs = pq.quant_act(X, inv, perm, k)
    say("act_quant case: line", K, k, M, G)
    Aq, Asc = _gpu_quant(X, K, k, inv, perm, offsets=off, G=G)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)
    cb, sb = prq.prq_packed_act_bytes(M, K + k)
    out = prq.PackedAct(torch.full((cb,), 0x5A, dtype=torch.uint8, device="cuda"),
                        torch.full((sb,), 0xA5, dtype=torch.uint8, device="cuda"), M, K + k)
    prq.prq_quant_act_packed(dev(X), K, k, dev(_pos(inv, perm)), dev(perm), out=out,
                             group_offsets=None if off is None else dev(off), G=G)
    torch.cuda.synchronize()
    ep, es = pack_rows(rq, rs)
    np.testing.assert_array_equal(host(out.Aps), es)
    np.testing.assert_array_equal(host(out.Ap), ep)


@pytest.mark.parametrize("packed", [False, True])
def test_group_search_in_many_groups(packed):
    """The most groups there can be cost about as much as one load's worth of them
    (measured 1.07 times): the search does not look at all of them (3.5 to 4 times)."""
    from paper_2609_22106_amd import prq
    M, K, k = 64, 768, 64
    X = torch.randn(M, K, device="cuda").bfloat16()
    us = []
    for G in (64, 4096):
        off = dev(inputs.routed_offsets(np.bincount(np.arange(M) * (G // M), minlength=G)))
        inv = torch.ones(G, K, device="cuda")
        perm = torch.arange(K, dtype=torch.int32, device="cuda").repeat(G, 1)
        call = prq.prq_quant_act_packed if packed else prq.prq_quant_act
        us.append(replay_us(lambda: call(X, K, k, inv, perm, group_offsets=off, G=G)))
    say("group search us:", packed, us)
    assert us[1] < 1.8 * us[0]


# (K, k, M, G, ld): the copies of several short rows a stage: one unit a row, a
# stage not filled by whole rows, the longest row; rows of the last pass missing;
# strided rows; groups changing inside a pass.
SHORT = [(32, 32, 700, 1, 32), (768, 64, 333, 1, 768), (768, 64, 331, 7, 776), (1440, 96, 258, 1, 1472),
         (1440, 0, 200, 90, 1440), (2016, 32, 130, 3, 2016)]


@pytest.mark.parametrize("K,k,M,G,ld", SHORT)
def test_short_row_copy_kernel(K, k, M, G, ld):
    """act_quant_short_kernel forced (the tuning entry; AUTO takes it for larger
    calls): packed, and row-major in several passes a workgroup and in one."""
    import ctypes
    from paper_2609_22106_amd import build, prq
    from tests.packing import pack_rows
    rng = np.random.default_rng(K + M + G)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, ld)) * 3).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(G)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (G, K)).astype(np.float32)
    off = inputs.routed_offsets(np.bincount(rng.integers(0, G, M), minlength=G))
    rq, rs = pq.quant_act_grouped(X[:, :K], inv, perm, off, k)
    lib = ctypes.CDLL(build.PROBE_LIB)
    P, I, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64
    lib.prq_tune_act_quant_packed.argtypes = [P, L, I, I, I, P, P, P, I, P, P, I, I, P]
    dX, di, dp, do = dev(X), dev(_pos(inv, perm)), dev(perm), dev(off)
    stream = torch.cuda.current_stream().cuda_stream
    say("short rows case:", K, k, M, G, ld)
    cb, sb = prq.prq_packed_act_bytes(M, K + k)
    Ap = torch.full((cb,), 0x5A, dtype=torch.uint8, device="cuda")
    Aps = torch.full((sb,), 0xA5, dtype=torch.uint8, device="cuda")
    assert lib.prq_tune_act_quant_packed(dX.data_ptr(), ld, M, K, k, di.data_ptr(), dp.data_ptr(),
                                         do.data_ptr() if G > 1 else None, G, Ap.data_ptr(),
                                         Aps.data_ptr(), 5, 7, stream) == 0
    torch.cuda.synchronize()
    ep, es = pack_rows(rq, rs)
    np.testing.assert_array_equal(host(Aps), es)
    np.testing.assert_array_equal(host(Ap), ep)
    for cus in (7, 256):
        Aq, Asc = _forced_rows(X, K, k, _pos(inv, perm), perm, off if G > 1 else None, G, 5, cus)
        np.testing.assert_array_equal(Asc, rs)
        np.testing.assert_array_equal(Aq, rq)


def _forced_rows(X, K, k, inv_pos, perm, off, G, kernel, cus):
    """Row-major codes and scales by a forced kernel with workgroups for `cus` CUs."""
    import ctypes
    from paper_2609_22106_amd import build
    lib = ctypes.CDLL(build.PROBE_LIB)
    P, I, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64
    lib.prq_tune_act_quant.argtypes = [P, L, I, I, I, P, P, P, I, P, P, I, I, P]
    M = X.shape[0]
    Aq = torch.full((M, (K + k) // 2), 0x5A, dtype=torch.uint8, device="cuda")
    Asc = torch.full((M, (K + k) // 32), 0xA5, dtype=torch.uint8, device="cuda")
    dX, di, dp = dev(X), dev(inv_pos), dev(perm)
    do = None if off is None else dev(off)
    assert lib.prq_tune_act_quant(dX.data_ptr(), X.shape[1], M, K, k, di.data_ptr(), dp.data_ptr(),
                                  None if do is None else do.data_ptr(), G, Aq.data_ptr(), Asc.data_ptr(),
                                  kernel, cus, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return host(Aq), host(Asc)


# (K, k, M, CUs): one to four units a thread and several rows a pass, each in at least
# five passes or rows a workgroup (stages reused), a ragged last one.
MANY_ROWS = [(32, 0, 1500, 1), (768, 64, 133, 4), (1440, 96, 91, 3), (2048, 32, 97, 5), (4096, 96, 70, 3),
             (4160, 160, 97, 4), (7136, 32, 50, 2), (9728, 224, 65, 3), (12320, 288, 33, 2), (16384, 512, 35, 2)]


@pytest.mark.parametrize("kernel,K,k,M,cus", [(q, *c) for q in (2, 3, 5) for c in MANY_ROWS
                                              if q != 5 or c[0] < 2048])
@pytest.mark.parametrize("G", [1, 6])
def test_many_row_kernels_row_major(kernel, G, K, k, M, cus):
    """Row-major output of each many-rows kernel (2: staged through registers, 3: rows
    copied, 5: short rows copied), forced, with groups changing between passes and
    inside them, empty ones among them."""
    rng = np.random.default_rng(K + M + G)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K + 8)) * 3).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(G)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (G, K)).astype(np.float32)
    off = inputs.routed_offsets(np.bincount(rng.choice([0, 1, 1, 3, 5, 5, 5], M) if G > 1 else np.zeros(M, int),
                                            minlength=G))
    say("many rows case:", kernel, G, K, k, M, cus)
    Aq, Asc = _forced_rows(X, K, k, _pos(inv, perm), perm, off if G > 1 else None, G, kernel, cus)
    rq, rs = pq.quant_act_grouped(X[:, :K], inv, perm, off, k)
    np.testing.assert_array_equal(Asc, rs)
    np.testing.assert_array_equal(Aq, rq)


@pytest.mark.parametrize("M", [7100, 7300])
@pytest.mark.parametrize("packed", [False, True])
def test_grouped_short_rows_on_both_sides_of_the_copy_kernels_line(packed, M):
    """5.5 million channels: below it rows are staged through registers, from it on they
    are copied (grouped calls as an expert prefill makes them)."""
    from paper_2609_22106_amd import prq
    from tests.packing import pack_rows
    K, k, G = 768, 64, 40
    rng = np.random.default_rng(M)
    X = inputs.f32_to_bf16_bits((rng.standard_normal((M, K)) * 3).astype(np.float32))
    perm = np.stack([rng.permutation(K) for _ in range(G)]).astype(np.int32)
    inv = rng.uniform(0.1, 4.0, (G, K)).astype(np.float32)
    off = inputs.routed_offsets(np.bincount(rng.integers(0, G - 1, M), minlength=G))
    rq, rs = pq.quant_act_grouped(X, inv, perm, off, k)
    say("short rows line case:", packed, M)
    if packed:
        A = prq.prq_quant_act_packed(dev(X), K, k, dev(_pos(inv, perm)), dev(perm), group_offsets=dev(off), G=G)
        torch.cuda.synchronize()
        ep, es = pack_rows(rq, rs)
        np.testing.assert_array_equal(host(A.Aps), es)
        np.testing.assert_array_equal(host(A.Ap), ep)
    else:
        Aq, Asc = _gpu_quant(X, K, k, inv, perm, offsets=off, G=G)
        np.testing.assert_array_equal(Asc, rs)
        np.testing.assert_array_equal(Aq, rq)
