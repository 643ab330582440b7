"""Performance cases of the MXFP4 + tail-residual hot path on one MI355X.

A case is one pass of work that a program built on this package has it do,
through the public calls of ``paper_2609_22106_amd.prq``:

* ``step``: a decode step's down-projections, ``layers`` of them with their own
  weights, each quantize + GEMM of up to 64 rows, captured once into a HIP graph
  and replayed (how a serving loop runs launch-bound work);
* ``linear``: quantize + GEMM of one linear at prefill rows, called eagerly;
* ``experts_step`` / ``experts``: the same for the routed rows of a mixture of
  experts, decode (captured) and prefill (eager);
* ``swiglu``: the offline-copy form, SiLU(gate) * up quantized as it is formed,
  then the GEMM;
* ``search``: the offline alpha search of one layer, from host arrays;
* ``pack``: laying out exported weights for the GEMM.

``packed`` picks the packed activation calls (the layout the GEMM copies in whole
kilobytes) or the row-major ones.  Weights, perms, scales and output buffers are
what such a program keeps; activations and routing are seeded draws with the
outlier channels of ``paper_2609_22106_amd.inputs``.
"""
import math

import numpy as np
import torch

from paper_2609_22106_amd import prq

DEV = "cuda"
BLOCK = 32
OUTLIERS, OUTLIER_SCALE = 0.005, 30.0
T_CAL = 64                                    # rows behind the activation maxima
# out features, in features, tail: the decoder linears this repository benchmarks,
# and two generic odd ones (K + k not a multiple of 128; N not of 128)
SHAPES = ((2560, 9728, 256), (4096, 2560, 64), (1024, 2560, 64), (2560, 4096, 96), (9728, 2560, 64),
          (1936, 5216, 128), (3376, 3104, 64))
EXPERTS = 128
EXPERT_SHAPES = ((2048, 768, 64), (1536, 1024, 32), (1040, 1440, 96))


def listed():
    return [
        # one sequence decoding: 24 layers' down-projections, row-major calls
        dict(name="decode step 1 row", kind="step", M=1, N=2560, K=9728, k=256, packed=False, layers=24),
        # a batch of 40 sequences decoding (an odd number of row blocks), packed calls
        dict(name="decode step 40 rows", kind="step", M=40, N=2560, K=9728, k=256, packed=True, layers=24),
        # 64 tokens decoding through 4 expert layers: weight streaming
        dict(name="expert decode 64 tokens", kind="experts_step", tokens=64, N=2048, K=768, k=64,
             packed=False, layers=4),
        # one chunk of a chunked prefill
        dict(name="prefill chunk 512 rows", kind="linear", M=512, N=2560, K=9728, k=256, packed=True),
        # a ragged prompt through the row-major pair, K + k not a multiple of 128
        dict(name="ragged prompt 1537 rows", kind="linear", M=1537, N=2560, K=4096, k=96, packed=False),
        # a prompt through a wide short-K projection (gate / up): the output is most of the bytes
        dict(name="wide projection 4096 rows", kind="linear", M=4096, N=9728, K=2560, k=64, packed=True),
        # a long prompt's down-projection: the largest matrix product
        dict(name="down projection 8192 rows", kind="linear", M=8192, N=2560, K=9728, k=256, packed=True),
        # a 4096-token prompt through the experts
        dict(name="expert prefill 4096 tokens", kind="experts", tokens=4096, N=2048, K=768, k=64,
             packed=True),
        # the gated activation of a long prompt (offline copy), then the down-projection
        dict(name="gated activation 8192 rows", kind="swiglu", M=8192, N=2560, K=9984, packed=True),
        # the same row-major, a short ragged prompt
        dict(name="gated activation 333 rows", kind="swiglu", M=333, N=2560, K=4192, packed=False),
        # calibrating one layer: three candidate alphas on 256 calibration rows
        dict(name="alpha search 3 candidates", kind="search", N=2560, K=9728, k=256, T=256, alphas=3),
        # loading a layer of experts
        dict(name="pack expert weights", kind="pack", E=128, N=2048, K=832),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("step", "linear", "linear", "experts_step", "experts", "swiglu", "search", "pack"))
    N, K, k = rng.choice(SHAPES)
    if kind == "step":
        return dict(kind=kind, M=_log_int(rng, 1, 64), N=N, K=K, k=k, packed=rng.random() < 0.5,
                    layers=rng.randint(8, 24))
    if kind == "linear":
        most = min(8192, 8192 * 2560 * 9984 // (N * (K + k)))
        return dict(kind=kind, M=_log_int(rng, 65, most), N=N, K=K, k=k, packed=rng.random() < 0.5)
    if kind in ("experts_step", "experts"):
        N, K, k = rng.choice(EXPERT_SHAPES)
        if kind == "experts_step":
            return dict(kind=kind, tokens=_log_int(rng, 8, 256), N=N, K=K, k=k, packed=rng.random() < 0.3,
                        layers=rng.randint(2, 4))
        return dict(kind=kind, tokens=_log_int(rng, 512, 4096), N=N, K=K, k=k, packed=rng.random() < 0.7)
    if kind == "swiglu":
        most = min(8192, 8192 * 2560 * 9984 // (N * (K + k)))
        return dict(kind=kind, M=_log_int(rng, 1, most), N=N, K=K + k, packed=rng.random() < 0.5)
    if kind == "search":
        return dict(kind=kind, N=N, K=K, k=k, T=_log_int(rng, 16, 256), alphas=rng.randint(1, 3))
    N, K, k = rng.choice(SHAPES + EXPERT_SHAPES)
    E = _log_int(rng, 1, max(1, 128 * 2048 * 832 // (N * (K + k))))
    return dict(kind="pack", E=E, N=N, K=K + k)


# ------------------------------------------------------------------- inputs ---
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + stream)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _activations(g, rows, K, out_idx):
    """N(0, 1) with heavy-tailed (Student-t, 3 degrees) outlier channels, as bf16."""
    x = _randn(g, rows, K)
    n = out_idx.numel()
    if n:
        t = _randn(g, rows, n) / (_randn(g, 3, rows, n).square().mean(0)).sqrt()
        x[:, out_idx] = OUTLIER_SCALE * t
    return x.bfloat16()


def _outliers(g, K):
    return torch.randperm(K, generator=g, device=DEV)[: int(round(OUTLIERS * K))].sort().values


def _mx(x):
    """MXFP4 of float32 rows [..., K]: (packed codes [..., K/2], scale codes [..., K/32])."""
    b = x.reshape(*x.shape[:-1], -1, BLOCK)
    e = (b.abs().amax(-1).contiguous().view(torch.int32) >> 23) & 0xFF
    sc = (e - 2).clamp_(min=0)
    t = b * ((254 - sc) << 23).view(torch.float32).unsqueeze(-1)
    a = t.abs()
    idx = torch.zeros(b.shape, dtype=torch.uint8, device=x.device)
    for bound, open_ in ((0.25, True), (0.75, False), (1.25, True), (1.75, False), (2.5, True),
                         (3.5, False), (5.0, True)):
        idx += (a > bound) if open_ else (a >= bound)
    idx |= torch.signbit(b).to(torch.uint8) << 3
    idx = idx.reshape(*x.shape[:-1], -1, 2)
    return idx[..., 0] | (idx[..., 1] << 4), sc.to(torch.uint8)


_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _deq(q, sc, dtype=torch.float64):
    lut = torch.tensor(_E2M1 + tuple(-v for v in _E2M1), dtype=dtype, device=q.device)
    v = torch.stack((lut[(q & 15).long()], lut[(q >> 4).long()]), -1).reshape(*q.shape[:-1], -1, BLOCK)
    v = torch.ldexp(v, sc.to(torch.int32).unsqueeze(-1) - 127)
    return v.reshape(*q.shape[:-1], -1)


class _Layer:
    """One exported linear: scales, tail permutation and augmented weight codes."""

    def __init__(self, g, N, K, k):
        self.out_idx = _outliers(g, K)
        W = (0.02 * _randn(g, N, K)).bfloat16().float()
        cal = _activations(g, T_CAL, K, self.out_idx).float()
        s = (cal.abs().amax(0).double() / W.abs().amax(0).double()).sqrt().float()
        hard = torch.zeros(K, dtype=torch.bool, device=DEV)
        hard[torch.argsort(s, descending=True, stable=True)[:k]] = True
        every = torch.arange(K, device=DEV)
        perm = torch.cat((every[~hard], every[hard]))
        Wt = (W * s)[:, perm]
        q, sc = _mx(Wt)
        if k:
            r = Wt[:, K - k:] - _deq(q[:, (K - k) // 2:].contiguous(), sc[:, (K - k) // BLOCK:], torch.float32)
            rq, rsc = _mx(r)
            q, sc = torch.cat((q, rq), 1), torch.cat((sc, rsc), 1)
        self.Wq, self.Wsc = q.contiguous(), sc.contiguous()
        self.perm = perm.int()
        self.inv_pos = (1.0 / s)[perm].contiguous()


def _layer_inputs(case, seed, layer):
    """(exported linear, X) of one layer of a step or linear case."""
    g = _gen(seed, layer)
    L = _Layer(g, case["N"], case["K"], case["k"])
    return L, _activations(g, case["M"], case["K"], L.out_idx)


def _routing(case, seed, layer):
    """Rows per expert of tokens routed to 8 distinct uniform experts: offsets [E + 1]."""
    g = torch.Generator()
    g.manual_seed(7919 * seed + layer)
    picks = torch.rand(case["tokens"], EXPERTS, generator=g).topk(8, dim=1).indices
    off = torch.zeros(EXPERTS + 1, dtype=torch.int32)
    off[1:] = torch.bincount(picks.flatten(), minlength=EXPERTS).cumsum(0)
    return off


def _expert_inputs(case, seed, layer):
    g = _gen(seed, 100 + layer)
    off = _routing(case, seed, layer)
    Ls = [_Layer(g, case["N"], case["K"], case["k"]) for _ in range(EXPERTS)]
    rows = off.diff().tolist()
    X = torch.cat([_activations(g, r, case["K"], L.out_idx) for r, L in zip(rows, Ls)])
    return Ls, off, X


def _gated_inputs(case, seed):
    g = _gen(seed, 0)
    K, out = case["K"], _outliers(_gen(seed, 1), case["K"])
    gate = _randn(g, case["M"], K).bfloat16()
    up = _activations(g, case["M"], K, out)
    Wq, Wsc = _mx(0.14 * _randn(g, case["N"], K))
    return gate, up, Wq.contiguous(), Wsc


def _random_codes(case, seed):
    g = _gen(seed, 0)
    E, N, K = case["E"], case["N"], case["K"]
    q = torch.randint(0, 256, (E, N, K // 2), generator=g, device=DEV, dtype=torch.uint8)
    s = torch.randint(118, 126, (E, N, K // BLOCK), generator=g, device=DEV, dtype=torch.uint8)
    return q, s


def _search_inputs(case, seed):
    """Host arrays: W [N, K], calibration rows [T, K] (bf16 bits), candidate alphas."""
    g = _gen(seed, 0)
    W = (0.02 * _randn(g, case["N"], case["K"])).bfloat16()
    X = _activations(g, case["T"], case["K"], _outliers(g, case["K"]))
    host = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    return host(W), host(X), [0.5, 0.7, 0.3][: case["alphas"]]


# ---------------------------------------------------------------------- run ---
def _act_buffers(packed, M, K_aug):
    if packed:
        cb, sb = prq.prq_packed_act_bytes(M, K_aug)
        return prq.PackedAct(torch.empty(cb, dtype=torch.uint8, device=DEV),
                             torch.empty(sb, dtype=torch.uint8, device=DEV), M, K_aug)
    return (torch.empty((M, K_aug // 2), dtype=torch.uint8, device=DEV),
            torch.empty((M, K_aug // BLOCK), dtype=torch.uint8, device=DEV))


def _pair(A):
    return (A.Ap, A.Aps) if isinstance(A, prq.PackedAct) else A


class _Linear:
    """A linear's kept weight, scales, buffers and workspace, and its call."""

    def __init__(self, L, X, k, packed):
        self.X, self.k, self.packed = X, k, packed
        self.M, self.K = X.shape
        self.W = prq.prq_pack_weight(L.Wq, L.Wsc)
        self.inv, self.perm = L.inv_pos, L.perm
        self.A = _act_buffers(packed, self.M, self.W.K_aug)
        self.Y = torch.empty((self.M, self.W.N), dtype=torch.float32, device=DEV)
        self.ws = _workspace(self.M, self.W, packed)

    def __call__(self):
        if self.packed:
            prq.prq_quant_act_packed(self.X, self.K, self.k, self.inv, self.perm, out=self.A)
            prq.prq_gemm_packed(self.A, self.W, Y=self.Y, workspace=self.ws)
        else:
            prq.prq_quant_act(self.X, self.K, self.k, self.inv, self.perm, Aq=self.A[0], Asc=self.A[1])
            prq.prq_gemm(self.A[0], self.A[1], self.W, Y=self.Y, workspace=self.ws)


def _workspace(M, W, packed):
    n = (prq.prq_gemm_packed_workspace_bytes if packed else prq.prq_gemm_workspace_bytes)(M, W.N, W.K_aug)
    return torch.zeros(n, dtype=torch.uint8, device=DEV) if n else None


class _Experts:
    def __init__(self, Ls, off, X, k, packed):
        self.X, self.k, self.packed = X, k, packed
        self.M, self.K = X.shape
        self.off = off.to(DEV)
        self.W = prq.prq_pack_weight(torch.stack([L.Wq for L in Ls]), torch.stack([L.Wsc for L in Ls]))
        self.inv = torch.stack([L.inv_pos for L in Ls])
        self.perm = torch.stack([L.perm for L in Ls])
        self.A = _act_buffers(packed, self.M, self.W.K_aug)
        self.Y = torch.empty((self.M, self.W.N), dtype=torch.float32, device=DEV)

    def __call__(self):
        E = self.W.E
        if self.packed:
            prq.prq_quant_act_packed(self.X, self.K, self.k, self.inv, self.perm, out=self.A,
                                     group_offsets=self.off, G=E)
            prq.prq_grouped_gemm_packed(self.A, self.off, self.W, Y=self.Y)
        else:
            prq.prq_quant_act(self.X, self.K, self.k, self.inv, self.perm, group_offsets=self.off, G=E,
                              Aq=self.A[0], Asc=self.A[1])
            prq.prq_grouped_gemm(self.A[0], self.A[1], self.off, self.W, Y=self.Y)


class _Gated:
    def __init__(self, gate, up, Wq, Wsc, packed):
        self.gate, self.up, self.packed = gate, up, packed
        self.W = prq.prq_pack_weight(Wq, Wsc)
        M = gate.shape[0]
        self.A = _act_buffers(packed, M, self.W.K_aug)
        self.Y = torch.empty((M, self.W.N), dtype=torch.float32, device=DEV)
        self.ws = _workspace(M, self.W, packed)

    def __call__(self):
        prq.prq_swiglu_quant(self.gate, self.up, self.W.K_aug, packed=self.packed, out=self.A)
        if self.packed:
            prq.prq_gemm_packed(self.A, self.W, Y=self.Y, workspace=self.ws)
        else:
            prq.prq_gemm(self.A[0], self.A[1], self.W, Y=self.Y, workspace=self.ws)


class _Captured:
    """Layers of a decode step in one HIP graph."""

    def __init__(self, layers):
        self.layers = layers
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):        # once eagerly before the capture
            for f in layers:
                f()
        torch.cuda.current_stream().wait_stream(side)
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            for f in layers:
                f()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _Captured([_Linear(*_layer_inputs(case, seed, i), case["k"], case["packed"])
                          for i in range(case["layers"])])
    if kind == "linear":
        return _Linear(*_layer_inputs(case, seed, 0), case["k"], case["packed"])
    if kind == "experts_step":
        return _Captured([_Experts(*_expert_inputs(case, seed, i), case["k"], case["packed"])
                          for i in range(case["layers"])])
    if kind == "experts":
        return _Experts(*_expert_inputs(case, seed, 0), case["k"], case["packed"])
    if kind == "swiglu":
        return _Gated(*_gated_inputs(case, seed), case["packed"])
    if kind == "search":
        return (case["k"],) + _search_inputs(case, seed)
    return _random_codes(case, seed)


def run(state):
    if isinstance(state, _Captured):
        state.graph.replay()
        return {"Y": [f.Y for f in state.layers], "A0": list(_pair(state.layers[0].A))}
    if isinstance(state, (_Linear, _Experts, _Gated)):
        state()
        return {"Y": state.Y, "A": list(_pair(state.A))}
    if isinstance(state[0], int):
        k, W, X, alphas = state
        best, err = prq.prq_search_alpha(W, X, alphas, k)
        return {"best": best, "nrmse": err}
    W = prq.prq_pack_weight(*state)
    return {"codes": W.Wp, "scales": W.Wps}


# ------------------------------------------------------------ floor and rule ---
def work(case):
    kind = case["kind"]
    if kind == "pack":
        codes = case["E"] * case["N"] * (case["K"] / 2 + case["K"] / 32)
        return {"bytes": 2 * codes, "flops": 0}
    if kind == "search":
        # host arrays in once; the reference product and, per alpha, the quantized one
        N, K, k, T, n = (case[x] for x in ("N", "K", "k", "T", "alphas"))
        return {"bytes": 2 * (N * K + T * K) + 8 * n, "flops": 2 * T * N * (K + n * (K + k))}
    N, K, k = case["N"], case["K"], case.get("k", 0)
    weight = N * (K + k) * (0.5 + 1 / 32)
    if kind in ("experts_step", "experts"):
        M, used = 8 * case["tokens"], EXPERTS * (1 - (1 - 8 / EXPERTS) ** case["tokens"])
        fixed = used * (weight + 8 * K)
    else:
        M, fixed = case["M"], weight + (0 if kind == "swiglu" else 8 * K)
    rows = M * ((4 if kind == "swiglu" else 2) * K + (K + k) * (0.5 + 1 / 32) + 4 * N)
    n = case.get("layers", 1)
    return {"bytes": n * (fixed + rows), "flops": n * 2.0 * M * N * (K + k)}


def tolerance(case):
    # codes and scale bytes are whole values and stay the same; Y and the error
    # norms are float32 sums, in any order (measured against 64 bits: Y below
    # 2e-16, its products fit the sum exactly where the scales lie close; norms
    # 5e-8; another order of a 10,000-term sum: 2e-7)
    if case["kind"] == "pack":
        return "exact"
    return {"rel": 1e-6, "max": 2e-5}


# ------------------------------------------------------------------- oracle ---
def _pad_to(t, dim, n, value):
    if t.shape[dim] == n:
        return t
    shape = list(t.shape)
    shape[dim] = n - t.shape[dim]
    return torch.cat((t, torch.full(shape, value, dtype=t.dtype, device=t.device)), dim)


def _lay_out(q, sc):
    """[..., R, K/2] codes and [..., R, K/32] scales in the 16-row, 128-element block layout, flat."""
    R, steps = q.shape[-2], -(-q.shape[-1] // 64)
    B, Q = -(-R // 16), -(-steps // 4)
    q = _pad_to(_pad_to(q, -1, steps * 64, 0), -2, B * 16, 0)
    sc = _pad_to(_pad_to(sc, -1, Q * 16, 127), -2, B * 16, 127)
    q = q.reshape(-1, B, 16, steps, 4, 16).permute(0, 1, 3, 4, 2, 5)
    sc = sc.reshape(-1, B, 16, Q, 4, 4).permute(0, 1, 3, 5, 2, 4)
    return q.reshape(-1), sc.reshape(-1)


def _quantized(X, inv_pos, perm, k):
    z = X.float()[:, perm.long()] * inv_pos
    q, sc = _mx(z)
    K = z.shape[1]
    return (torch.cat((q, q[:, (K - k) // 2:]), 1) if k else q,
            torch.cat((sc, sc[:, (K - k) // BLOCK:]), 1) if k else sc)


def _out_act(q, sc, packed):
    return list(_lay_out(q, sc)) if packed else [q, sc]


def _product(q, sc, Wq, Wsc):
    return torch.cat([_deq(q[i:i + 4096], sc[i:i + 4096]) @ _deq(Wq, Wsc).T for i in range(0, max(1, len(q)), 4096)])


def _exact_linear(L, X, k):
    q, sc = _quantized(X, L.inv_pos, L.perm, k)
    return _product(q, sc, L.Wq, L.Wsc), q, sc


def _exact_experts(Ls, off, X, k):
    off = off.tolist()
    parts = [_exact_linear(L, X[off[e]:off[e + 1]], k) for e, L in enumerate(Ls) if off[e] < off[e + 1]]
    return tuple(torch.cat(p) for p in zip(*parts))


def _exact_silu(x):
    """SiLU of bf16 values by the documented float32 sequence, one rounding an operation (on the
    CPU, over every bf16 value, then looked up)."""
    f = torch.arange(65536, dtype=torch.int32).to(torch.int16).view(torch.bfloat16).float()
    f = torch.where(f.isfinite(), f, torch.zeros_like(f))
    c = lambda h: torch.tensor(float.fromhex(h), dtype=torch.float32)  # noqa: E731
    a = (-f).clamp(-104.0, 89.0)
    n = (a * c("0x1.715476p+0")).round()
    r = (a - n * c("0x1.62e4p-1")) - n * c("0x1.7f7d1cp-20")
    p = c("0x1.6c16c2p-10").expand_as(r)
    for h in ("0x1.111112p-7", "0x1.555556p-5", "0x1.555556p-3", "0x1p-1", "0x1p+0", "0x1p+0"):
        p = p * r
        p = p + c(h)
    e = torch.ldexp(p.double(), n.double()).float()
    return (f / (1.0 + e)).to(x.device)[x.contiguous().view(torch.int16).long() & 0xFFFF]


def _exact_search(case, seed):
    """Algorithm 1's search in 64 bits: y-NRMSE of every candidate, and the best."""
    W, X, alphas = _search_inputs(case, seed)
    k = case["k"]
    up = lambda a: torch.from_numpy(a.view(np.int16)).to(DEV).view(torch.bfloat16)  # noqa: E731
    W, Xb = up(W).float(), up(X)
    K = W.shape[1]
    ref = Xb.double() @ W.double().T
    errs = []
    for alpha in alphas:
        a = Xb.float().abs().amax(0).double().clamp(min=1e-5).cpu().tolist()
        b = W.abs().amax(0).double().clamp(min=1e-5).cpu().tolist()
        s = torch.tensor([math.pow(x, alpha) / math.pow(y, 1.0 - alpha) for x, y in zip(a, b)],
                         dtype=torch.float64).float().to(DEV)
        Ws = W * s
        d = (Ws - _deq(*_mx(Ws), torch.float32)).double()
        order = torch.argsort(-d.square().sum(0), stable=True)
        hard = torch.zeros(K, dtype=torch.bool, device=DEV)
        hard[order[:k]] = True
        every = torch.arange(K, device=DEV)
        perm = torch.cat((every[~hard], every[hard]))
        Wt = Ws[:, perm]
        q, sc = _mx(Wt)
        main = _deq(q, sc, torch.float32)
        if k:
            rq, rsc = _mx(Wt[:, K - k:] - main[:, K - k:])
            q, sc = torch.cat((q, rq), 1), torch.cat((sc, rsc), 1)
        aq, asc = _quantized(Xb, (1.0 / s)[perm], perm, k)
        y = _product(aq, asc, q, sc)
        errs.append(float((y - ref).norm() / ref.norm()))
    return {"best": alphas[int(np.argmin(errs))], "nrmse": np.array(errs, dtype=np.float64)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "pack":
        codes, scales = _lay_out(*_random_codes(case, seed))
        return {"codes": codes, "scales": scales}
    if kind == "search":
        return _exact_search(case, seed)
    if kind in ("step", "experts_step"):
        Y, A0 = [], None
        for i in range(case["layers"]):
            y, q, sc = (_exact_linear(*_layer_inputs(case, seed, i), case["k"]) if kind == "step"
                        else _exact_experts(*_expert_inputs(case, seed, i), case["k"]))
            Y.append(y)
            A0 = A0 or _out_act(q, sc, case["packed"])
        return {"Y": Y, "A0": A0}
    if kind == "swiglu":
        gate, up, Wq, Wsc = _gated_inputs(case, seed)
        q, sc = _mx(_exact_silu(gate) * up.float())
        return {"Y": _product(q, sc, Wq, Wsc), "A": _out_act(q, sc, case["packed"])}
    y, q, sc = (_exact_linear(*_layer_inputs(case, seed, 0), case["k"]) if kind == "linear"
                else _exact_experts(*_expert_inputs(case, seed, 0), case["k"]))
    return {"Y": y, "A": _out_act(q, sc, case["packed"])}
