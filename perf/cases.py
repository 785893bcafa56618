"""The work that a user of this library has it do, as cases to be timed through the public entry points.

A case is one synchronisation step of Algorithm 1, or one half of it: the workers' lines (`Qsl.compress`,
`Qsl.compress_diff`, `Qsl.error_update`) and the master's (`Qsl.aggregate`).  Four kinds:

    round    the whole step for R workers held on one GPU, as the training loop of `algorithm1.py` and `bench.py` do it
    worker   one worker per GPU: it compresses its own vector, then adds up its own and its peers' messages itself
    update   the messages first, the error memory later from the messages (`error_update`), as where the send is not
             allowed to wait for the update
    master   a parameter server's side alone: many workers' messages into the model

A step changes the state in place, as in training: the error memory is carried on, the round number advances.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1906_02367_amd import binding as B
from paper_1906_02367_amd import workloads as W

RESNET50 = 25_557_032
QUANTIZERS = {"qsgd": B.QSGD, "sign_l1": B.SIGN_L1, "sign_l2": B.SIGN_L2, "fp32": B.FP32,
              "qsgd_scaled": B.QSGD_SCALED, "sign_l3": B.SIGN_L3, "sign_l4": B.SIGN_L4}
OPERATOR_SEED = 190602367


def _case(name, **kw):
    c = dict(kind="round", d=RESNET50, R=8, table="one", segments=1, rule="share", share=0.001, cap=0, sparsifier="top",
             quantizer="qsgd", s=16, source="delta", profile="coordinate")
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the paper's convex experiment (softmax regression on 784 features and 10 classes, 15 workers, k = 40, 4-bit QSGD):
        # the smallest calls, where launches and host calls are all there is
        _case("softmax_15_workers", d=7850, R=15, rule="cap", cap=40, s=15, source="models"),
        # TopK-SGD (no quantiser) on a model of a million parameters, an odd size, with the error update on its own
        _case("million_top1pct_fp32", kind="update", d=1_000_003, R=4, share=0.01, quantizer="fp32"),
        # the headline: ResNet-50's vector, 8 workers, Top_k of 0.1 % and QSGD with 16 levels
        _case("resnet50_top0.1pct_qsgd16"),
        # the same operator as deployed, one worker per GPU, Delta formed from the models, eight messages added up
        _case("resnet50_one_of_8_models", kind="worker", source="models"),
        # Rand_k of 1 % with 2-level QSGD: the random choice and many selected entries
        _case("resnet50_rand1pct_qsgd2", sparsifier="rand", share=0.01, s=2),
        # piecewise operator over 160 tensors of log-uniform sizes, sign quantiser
        _case("layerwise160_top0.1pct_sign", R=4, table="loguniform", segments=160, quantizer="sign_l1", s=1, profile="tensor"),
        # the paper's own ResNet-50 setting: every tensor on its own with k_t = min(d_t, 1000), SignTop_k
        _case("resnet50_per_tensor_k1000", table="resnet50", segments=161, rule="cap", cap=1000, quantizer="sign_l1", s=1,
              profile="tensor"),
        # the largest vectors: 2^28 coordinates, four workers, very sparse, 8-bit levels
        _case("large_top0.01pct_qsgd256", d=1 << 28, R=4, share=0.0001, s=256, profile="student"),
        # the comparison schemes without sparsification: EF-signSGD and EF-QSGD, messages without indices
        _case("resnet50_ef_sign", R=2, rule="all", quantizer="sign_l1", s=1),
        _case("resnet50_ef_qsgd15", R=2, rule="all", s=15),
        # a dense Top_k: a tenth of the coordinates, sign quantiser
        _case("resnet50_top10pct_sign", R=4, share=0.1, quantizer="sign_l1", s=1),
        # a parameter server with 32 workers' per-tensor messages
        _case("master_32_messages", kind="master", R=32, table="resnet50", segments=161, rule="cap", cap=1000,
              quantizer="sign_l1", s=1, profile="tensor"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "round", "worker", "update", "master"])
    R = {"round": rng.choice([1, 2, 3, 4, 5, 8, 12, 15]), "worker": rng.randint(2, 16), "update": rng.randint(1, 8),
         "master": round(_log(rng, 2, 64))}[kind]
    rows = 1 if kind == "worker" else R
    d = round(_log(rng, 2000, min(3.0e7, 1.0e8 / rows))) | (rng.random() < 0.7)
    c = _case(None, kind=kind, d=int(d), R=R, source=rng.choice(["delta", "delta", "models"]) if kind in ("round", "worker") else "delta")
    what = rng.random()
    if what < 0.12:                               # every coordinate kept, messages without indices
        c.update(rule="all", quantizer=rng.choice(["sign_l1", "sign_l2", "qsgd", "qsgd"]))
    elif what < 0.27:                             # Rand_k
        c.update(sparsifier="rand", share=_log(rng, 1e-3, 0.05), quantizer=rng.choice(["qsgd", "sign_l1"]))
    elif what < 0.6:                              # Top_k on the whole vector, from very sparse to dense
        c.update(share=_log(rng, 2e-4, 0.25), quantizer=rng.choice(["qsgd", "qsgd", "qsgd_scaled", "sign_l1", "sign_l2", "fp32"]))
    else:                                         # Top_k tensor by tensor
        if rng.random() < 0.3 and rows <= 3:
            c.update(table="resnet50", segments=161, d=RESNET50)
        else:
            c.update(table="loguniform", segments=rng.randint(2, max(3, min(300, c["d"] // 400))))
        c.update(rule=rng.choice(["share", "cap"]), share=_log(rng, 5e-4, 0.05), cap=rng.choice([100, 1000, 1000, 2500]),
                 quantizer=rng.choice(["sign_l1", "sign_l1", "qsgd", "fp32"]), profile="tensor")
    c["s"] = rng.choice([1, 2, 3, 4, 7, 15, 15, 16, 63, 255, 256]) if c["quantizer"].startswith("qsgd") else 1
    return c


def _plan(case):
    """Segment offsets and k of every segment."""
    d = case["d"]
    if case["table"] == "resnet50":
        sizes = np.array(W.resnet50_tensor_sizes(), dtype=np.int64)
    elif case["table"] == "loguniform":
        off, _ = W.segment_table(d, case["segments"], 64.0, max(256.0, 2.4e6 * d / RESNET50))
        sizes = np.diff(off.astype(np.int64))
    else:
        sizes = np.array([d], dtype=np.int64)
    off = np.zeros(sizes.size + 1, dtype=np.uint64)
    off[1:] = np.cumsum(sizes).astype(np.uint64)
    if case["rule"] == "all":
        k = sizes
    elif case["rule"] == "cap":
        k = np.minimum(sizes, case["cap"])
    else:
        k = np.maximum(1, np.ceil(sizes * case["share"] - 1e-9).astype(np.int64))
    return off, k.astype(np.uint32)


class _Vectors:
    """The workers' error memories and updates: heavy-tailed scales that stay the same over workers (one per coordinate, or
    one per tensor), a part that the workers share and a part of their own; every row a function of (seed, worker)."""

    def __init__(self, case, seed, off, device):
        self.case, self.seed, self.device = case, int(seed), device
        d = case["d"]
        g = self._gen(0)
        if case["profile"] == "tensor":
            per = torch.exp(2.0 * torch.randn(off.size - 1, generator=g, device=device))
            self.sigma = torch.repeat_interleave(per, torch.from_numpy(np.diff(off.astype(np.int64))).to(device))
        else:
            a = 1.0 if case["profile"] == "student" else 2.0
            self.sigma = torch.empty(d, device=device).normal_(generator=g).mul_(a).exp_()
        self.sigma.mul_(0.01)
        self.shared = torch.empty(d, device=device).normal_(generator=g).mul_(self.sigma)

    def _gen(self, n):
        g = torch.Generator(device=self.device)
        g.manual_seed((self.seed * 4099 + n) % (1 << 62))
        return g

    def row(self, w, m, delta):
        """Fills worker w's memory and update."""
        g = self._gen(1 + w)
        delta.normal_(generator=g)
        if self.case["profile"] == "student":     # Student-t with 3 degrees of freedom
            chi, z = torch.zeros_like(delta), torch.empty_like(delta)
            for _ in range(3):
                z.normal_(generator=g)
                chi.addcmul_(z, z)
            delta.div_(chi.div_(3.0).sqrt_())
        delta.mul_(self.sigma).add_(self.shared).mul_(math.sqrt(0.5))
        m.normal_(generator=g).mul_(self.sigma)

    def model(self):
        return torch.empty(self.case["d"], device=self.device).normal_(generator=self._gen(100_003)).mul_(0.05)


def _operator(case, off, k, max_workers, device):
    flags = B.FLAG_DENSE_FORMAT if case["rule"] == "all" else 0
    return B.Qsl(case["d"], off, k, case["s"], B.TOPK if case["sparsifier"] == "top" else B.RANDK,
                 QUANTIZERS[case["quantizer"]], OPERATOR_SEED, max_workers, flags=flags, device=device)


def prepare(case, seed):
    device = torch.device("cuda")
    d, R, kind = case["d"], case["R"], case["kind"]
    off, k = _plan(case)
    vec = _Vectors(case, seed, off, device)
    st = {"case": case, "t": 0, "x": vec.model()}
    if kind == "master":                          # the messages of R workers, compressed eight at a time
        n = min(R, 8)
        st["q"] = _operator(case, off, k, R, device)
        st["msg"] = st["q"].new_msg(R)
        src = _operator(case, off, k, n, device)
        m, delta = torch.empty(n, d, device=device), torch.empty(n, d, device=device)
        for w0 in range(0, R, n):
            c = min(n, R - w0)
            for i in range(c):
                vec.row(w0 + i, m[i], delta[i])
            src.compress(m[:c], delta[:c], m[:c], w0, 0, st["msg"][w0:w0 + c])
        torch.cuda.synchronize()
        return st
    rows = 1 if kind == "worker" else R
    m, delta = torch.empty(rows, d, device=device), torch.empty(rows, d, device=device)
    for w in range(rows):
        vec.row(w, m[w], delta[w])
    st["q"] = _operator(case, off, k, rows, device)
    st["msg"] = st["q"].new_msg(R)
    st["bits"] = torch.zeros(rows, dtype=torch.int64, device=device)
    st["m"], st["delta"] = m, delta
    if case["source"] == "models":                # the local models after the local step; Delta = x - xhat
        st["xhat"] = torch.sub(st["x"].unsqueeze(0), delta)
        del st["delta"]
    if kind == "worker":                          # the peers' messages of this round, as they came in
        src = _operator(case, off, k, 1, device)
        pm, pd = torch.empty(1, d, device=device), torch.empty(1, d, device=device)
        for w in range(1, R):
            vec.row(w, pm[0], pd[0])
            src.compress(pm, pd, pm, w, 0, st["msg"][w:w + 1])
        st["update"] = torch.empty(d, device=device)
    elif case["source"] == "models":
        st["update"] = torch.empty(d, device=device)
    if kind == "update":
        st["v"] = torch.empty_like(m)
    torch.cuda.synchronize()
    return st


def run(state):
    case, q, msg = state["case"], state["q"], state["msg"]
    kind, R = case["kind"], case["R"]
    if kind == "master":                          # x <- x - (1/R) sum_r g^(r)
        q.aggregate(msg, state["x"], -1.0 / R, accumulate=True)
        return {"x": state["x"]}
    t = state["t"]
    state["t"] = t + 1
    m, bits = state["m"], state["bits"]
    if kind == "update":
        q.compress(m, state["delta"], state["v"], 0, t, msg, bits)
        q.error_update(m, state["delta"], msg)
        return {"m": m, "msg": msg, "bits": bits}
    mine = msg[:1] if kind == "worker" else msg
    if case["source"] == "models":
        q.compress_diff(m, state["x"], state["xhat"], m, 0, t, mine, bits)
    else:
        q.compress(m, state["delta"], m, 0, t, mine, bits)
    if "update" in state:                         # the update itself, for an optimizer of the program's own
        q.aggregate(msg, state["update"], 1.0 / R)
        return {"m": m, "msg": msg, "bits": bits, "x": state["update"]}
    q.aggregate(msg, state["x"], -1.0 / R, accumulate=True)
    return {"m": m, "msg": msg, "bits": bits, "x": state["x"]}


def _entries(case):
    """(entries of one message, bits of one message): QSGD sends at most about s sqrt(k) of k entries."""
    off, k = _plan(case)
    d, L = case["d"], k.size
    qsgd = case["quantizer"].startswith("qsgd")
    if case["rule"] == "all":
        w = (int(case["s"]).bit_length() + 1) if qsgd else 32 if case["quantizer"] == "fp32" else 1
        return d, 32 + 32 * L + d * w
    kk = k.astype(np.float64)
    n = float(np.minimum(kk, case["s"] * np.sqrt(kk)).sum()) if qsgd else float(kk.sum())
    w = (int(case["s"] - 1).bit_length() + 1) if qsgd else 32 if case["quantizer"] == "fp32" else 1
    return n, 32 + 32 * L + n * (max(1, int(d - 1).bit_length()) + w)


def work(case):
    d, R, kind = case["d"], case["R"], case["kind"]
    n, bits = _entries(case)
    rows = {"worker": 1, "master": 0}.get(kind, R)
    by = 12.0 * rows * d + rows * bits / 8        # m and Delta read, m written; the messages written
    if case["source"] == "models":
        by += 4.0 * d                             # the master's model
    if kind == "update":
        return {"bytes": by, "flops": 2.0 * rows * d}
    by += R * bits / 8                            # the messages read
    touched = min(float(d), R * n)
    by += 4.0 * d if (kind == "worker" or case["source"] == "models") else 8.0 * touched
    return {"bytes": by, "flops": 2.0 * rows * d + R * n}


def tolerance(case):
    """Messages, error memory and model are defined to the bit: every operation that decides an output is one IEEE operation,
    norms are exact sums, messages are added in list order."""
    return "exact"


def _random_words(idx, worker, rnd, stream, seed):
    """Philox4x32-10 (Salmon et al., SC'11): the random words of the coordinates idx (int64), as int64 in [0, 2^32)."""
    mask = 0xFFFFFFFF
    c0 = idx >> 2
    c1 = torch.full_like(c0, worker)
    c2 = torch.full_like(c0, rnd & mask)
    c3 = torch.full_like(c0, ((rnd >> 32) | (stream << 30)) & mask)
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57          # the low 64 bits of the products, wrapped into int64
        c0, c1, c2, c3 = (((p1 >> 32) & mask) ^ c1 ^ k0), p1 & mask, (((p0 >> 32) & mask) ^ c3 ^ k1), p0 & mask
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    j = idx & 3
    return torch.where(j == 0, c0, torch.where(j == 1, c1, torch.where(j == 2, c2, c3)))


def _decoded(case, off, k, v, worker):
    """g = Q Comp_k(v) of one worker at round 0, in 64 bits; v is float64 [d]."""
    g = torch.zeros_like(v)
    dev, s, quant = v.device, case["s"], case["quantizer"]
    for l in range(k.size):
        a, b, kl = int(off[l]), int(off[l + 1]), int(k[l])
        part = v[a:b]
        if kl == b - a:
            idx = torch.arange(a, b, device=dev)
        elif case["sparsifier"] == "top":
            idx = a + torch.topk(part.abs(), kl, sorted=False).indices
        else:
            i = torch.arange(a, b, device=dev)
            key = (_random_words(i, worker, 0, 0, OPERATOR_SEED) << 31) - i
            idx = a + torch.topk(key, kl, sorted=False).indices
        x = v[idx]
        if quant == "fp32":
            g[idx] = x
        elif quant.startswith("sign"):
            m = int(quant[-1])
            c = float((x.abs() ** m).sum()) ** (1.0 / m) / kl
            g[idx] = torch.where(x < 0, -c, c).to(v.dtype)
        else:
            norm = float(x.norm())
            if norm > 0:
                t = (x.abs() / norm * s).clamp(max=float(s))
                u = (_random_words(idx, worker, 0, 1, OPERATOR_SEED) >> 8).to(v.dtype) * 2.0 ** -24
                level = t.floor() + (u < t - t.floor())
                sent = norm if quant == "qsgd" else norm / (1 + min(kl / s ** 2, math.sqrt(kl) / s))
                g[idx] = torch.where(x < 0, -level, level) * (sent / s)
    return g


def exact(case, seed):
    device = torch.device("cuda")
    d, R, kind = case["d"], case["R"], case["kind"]
    off, k = _plan(case)
    if R * k.size > 40_000:
        return None
    vec = _Vectors(case, seed, off, device)
    x = vec.model()
    m, delta = torch.empty(d, device=device), torch.empty(d, device=device)
    rows = {"worker": 1, "master": 0}.get(kind, R)
    new_m = torch.empty(rows, d, dtype=torch.float64, device=device) if rows else None
    total = torch.zeros(d, dtype=torch.float64, device=device)
    for w in range(R):
        vec.row(w, m, delta)
        if case["source"] == "models" and w < rows:
            v = m.double() + (x.double() - torch.sub(x, delta).double())
        else:
            v = m.double() + delta.double()
        g = _decoded(case, off, k, v, w)
        if w < rows:
            new_m[w] = v - g
        total += g
    if kind == "update":
        return {"m": new_m, "msg": None, "bits": None}
    if kind == "worker" or case["source"] == "models":
        return {"m": new_m, "msg": None, "bits": None, "x": total / R}
    after = x.double() - total / R
    return {"x": after} if kind == "master" else {"m": new_m, "msg": None, "bits": None, "x": after}
