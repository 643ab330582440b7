"""The offline evaluation calls (Algorithm 1's alpha search and the y-NRMSE of
one configuration) on the device path against the oracle: errors to the
float32-accumulation level (the reference product is float32 on the device,
float64 in the oracle) and the same selected alpha."""
import numpy as np
import pytest

pytest.importorskip("torch")

from oracle import prquant as pq                       # noqa: E402
from paper_2609_22106_amd import inputs                # noqa: E402
from tests.gpu_util import say                         # noqa: E402

pytestmark = pytest.mark.gpu

RTOL = 1e-4


@pytest.mark.parametrize("scale_search", [False, True])
def test_alpha_search_matches_oracle(scale_search):
    from paper_2609_22106_amd import prq
    c = inputs.tiny_case()
    alphas = [0.0, 0.25, 0.5, 0.75, 1.0]
    say("evaluate case: alpha search tiny, E8M0-W", scale_search)
    best, errs = prq.prq_search_alpha(c.W, c.Xcal, alphas, 64, scale_search=scale_search)
    ref_best, ref_errs = pq.search_alpha(c.W, c.Xcal, alphas, 64, scale_search=scale_search)
    say("errors", np.round(errs, 5), "oracle", np.round(ref_errs, 5))
    np.testing.assert_allclose(errs, ref_errs, rtol=RTOL)
    order = np.sort(ref_errs)
    if order[1] - order[0] > 4 * RTOL * order[0]:
        assert best == alphas[ref_best]


def test_evaluate_on_held_out_rows_matches_oracle():
    from paper_2609_22106_amd import prq
    c = inputs.make_dense("h", N=256, K=2048, M=96, T=128, k_tail=64, n_out=10, seed=21)
    for mode, k in (("smooth", 64), ("smooth", 0), ("none", 0)):
        say("evaluate case:", mode, k)
        got = prq.prq_evaluate_nrmse(c.W, c.Xcal, c.X, 0.5, k, mode)
        y, _ = pq.prquant_forward(c.X, c.W, c.Xcal, 0.5, k, mode)
        want = pq.nrmse(y, pq.reference_product(c.X, c.W))
        assert abs(got - want) <= RTOL * want, (mode, k, got, want)


def test_ablation_grid_matches_oracle():
    """The device-path ablation grid against the oracle's on a small shape."""
    from paper_2609_22106_amd import ablation
    c = inputs.make_dense("a", N=128, K=1024, M=64, T=64, k_tail=64, n_out=8, seed=31)
    got = ablation.run_grid(c.X, c.W, c.Xcal, 0.5, 64)
    want = pq.ablation_grid(c.X, c.W, c.Xcal, 0.5, 64)
    say("ablation grid", {k: round(v, 5) for k, v in got.items()}, "w/o Perm (oracle)",
        round(want["w/o Perm"], 5))
    for name, v in got.items():
        assert abs(v - want[name]) <= RTOL * want[name], (name, v, want[name])


def test_ablation_grid_full_down_proj_matches_stored_oracle():
    """The full 9728 -> 2560 workload (512 evaluation rows) against the oracle
    values written by tests/golden/make_ablation_down_proj.py."""
    import json
    import os
    from paper_2609_22106_amd import ablation
    with open(os.path.join(os.path.dirname(__file__), "golden", "ablation_down_proj.json")) as f:
        want = json.load(f)["y_nrmse"]
    c = inputs.down_proj_prefill()
    say("evaluate case: ablation grid, full down_proj")
    got = ablation.run_grid(c.X[:512], c.W, c.Xcal, c.alpha, c.k_tail)
    for name, v in got.items():
        assert abs(v - want[name]) <= RTOL * want[name], (name, v, want[name])


# (N, K, k, T): one block; a 64-row tile and a remainder; more rows than a maxima
# workgroup's share; the whole row as tail; the longest row; the layer shape.
DEVICE_PREPARE = [(16, 32, 32, 1), (80, 1056, 0, 7), (1104, 352, 64, 300), (48, 256, 256, 16),
                  (32, 16384, 512, 9), (2560, 9728, 256, 64)]


@pytest.mark.parametrize("N,K,k,T", DEVICE_PREPARE)
@pytest.mark.parametrize("search", [False, True])
def test_device_construction_equals_host_prepare(N, K, k, T, search):
    """The construction the alpha search runs on the device against prq_prepare:
    maxima, column errors, permutation, codes and scale bytes, bit for bit; zero
    columns (equal errors, lowest scale codes) and tiny and large columns among
    them."""
    import ctypes
    import torch
    from paper_2609_22106_amd import build, prq
    from tests.gpu_util import dev, host
    rng = np.random.default_rng(N + K + k)
    W = rng.standard_normal((N, K)).astype(np.float32) * 0.02
    X = rng.standard_normal((T, K)).astype(np.float32)
    W[:, rng.random(K) < 0.05] = 0.0
    W[:, rng.random(K) < 0.05] *= 1e-30
    W[:, rng.random(K) < 0.05] *= 1e30
    W[:, :32] *= 1e-37          # a block whose values fall below the smallest scale
    X[:, rng.random(K) < 0.05] = 0.0
    W, X = inputs.f32_to_bf16_bits(W), inputs.f32_to_bf16_bits(X)
    want = prq.prq_prepare(W, X, 0.5, k, with_col_err=True, scale_search=search)
    lib = ctypes.CDLL(build.PROBE_LIB)
    dW, dX = dev(W.view(np.int16)), dev(X.view(np.int16))
    sc, inv = dev(want["scale"]), dev(want["inv_scale"])
    new = lambda n, t: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    mx, err, rank, perm = new(2 * K, torch.int32), new(K, torch.float64), new(K, torch.int32), new(K, torch.int32)
    sp, ip = new(K, torch.float32), new(K, torch.float32)
    Wq, Wsc = new(N * (K + k) // 2, torch.uint8), new(N * (K + k) // 32, torch.uint8)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    say("device construction case:", N, K, k, T, search)
    st = lib.prq_tune_prepare_device(p(dW), N, K, p(dX), T, k, int(search), p(sc), p(inv), p(mx), p(err),
                                     p(rank), p(perm), p(sp), p(ip), p(Wq), p(Wsc),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    m = host(mx).view(np.uint32).reshape(2, K)
    np.testing.assert_array_equal(m[0] >> 16, (X & 0x7FFF).max(0))
    np.testing.assert_array_equal(m[1] >> 16, (W & 0x7FFF).max(0))
    np.testing.assert_array_equal(host(err), want["col_err"])
    np.testing.assert_array_equal(host(perm), want["perm"])
    np.testing.assert_array_equal(host(ip), want["inv_scale_pos"])
    np.testing.assert_array_equal(host(Wsc).reshape(N, -1), want["Wsc"])
    np.testing.assert_array_equal(host(Wq).reshape(N, -1), want["Wq"])


def test_alpha_search_scales_and_errors_follow_prepare():
    """The search's error of each candidate against the same export made by
    prq_prepare and evaluated through the device calls: the same Y, so the same
    error up to the float32 order of the reference product (2e-7 measured; 2e-6)."""
    import torch
    from paper_2609_22106_amd import prq
    from tests.gpu_util import dev, host
    c = inputs.make_dense("s", N=208, K=1312, M=8, T=100, k_tail=96, n_out=9, seed=5)
    alphas = [0.9, 0.0, 0.45]
    for mode in ("smooth", "act_only", "none"):
        _, errs = prq.prq_search_alpha(c.W, c.Xcal, alphas, 96, scale_mode=mode)
        ref = pq.reference_product(c.Xcal, c.W)
        for a, got in zip(alphas, errs):
            art = prq.prq_prepare(c.W, c.Xcal, a, 96, scale_mode=mode)
            Aq, Asc = prq.prq_quant_act(dev(c.Xcal.view(np.int16)), 1312, 96, dev(art["inv_scale_pos"]),
                                        dev(art["perm"]))
            y = prq.prq_gemm(Aq, Asc, prq.prq_pack_weight(dev(art["Wq"]), dev(art["Wsc"])))
            torch.cuda.synchronize()
            want = pq.nrmse(host(y).astype(np.float64), ref)
            say("search error", mode, a, got, want)
            assert abs(got - want) <= 2e-6 * want


def test_search_over_many_alphas():
    """More candidates than are taken together, and many: each one's error is the
    one it has in a search of its own."""
    from paper_2609_22106_amd import prq
    c = inputs.make_dense("many", N=16, K=64, M=8, T=5, k_tail=32, n_out=2, seed=9)
    for n in (65, 70000):
        alphas = np.linspace(0.0, 1.0, n)
        say("many alphas case:", n)
        best, errs = prq.prq_search_alpha(c.W, c.Xcal, alphas, 32)
        assert best == alphas[int(np.argmin(errs))]
        for i in np.unique(np.concatenate([[0, 63, 64, n - 1], np.arange(0, n, max(1, n // 7))])):
            assert prq.prq_search_alpha(c.W, c.Xcal, alphas[i:i + 1], 32)[1][0] == errs[i], i
