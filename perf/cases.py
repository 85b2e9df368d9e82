"""What the library is timed on: training steps, predictions, a model merge and an
elastic round, over the sizes that the package's own workloads span.

A case is a dict of plain values.  ``kind`` says what one pass is:

* ``step``: one ``asgd_train_step`` on a device-resident batch (forward, backward and
  update).  The outputs are the change of every parameter since ``prepare`` and the
  batch's loss; they are read from the model when somebody looks at them, as a program
  reads its weights at a checkpoint and not after each step.
* ``predict``: one ``asgd_predict_topk``: the ids and their logits.
* ``merge``: one ``asgd_merge`` of some replicas with momentum and broadcast: the
  parameters of the new global model and of the first replica.
* ``round``: one ``asgd_elastic_round`` with the virtual clock, which makes its
  schedule a function of the inputs: the global model's change and the round's record.

Batches come from ``synth.generate`` (lognormal row lengths, Zipf feature and label ids,
normalised rows).  The models of the first three kinds hold weights of a trained
model's scale (logits that differ by units, biases of their own) and not the first
step's, whose logits are all about zero.
"""
import math

import numpy as np
import torch

import paper_2110_07029_amd as asgd
from paper_2110_07029_amd import synth

H = asgd.HIDDEN
# With the weights of _weights: large enough that a step's change of a weight stands far above the
# weight's rounding, small enough that thousands of steps on one batch stay finite.
LR = 0.25
NAMES = ("W1", "b1", "Wh", "bh", "W2", "b2")
WHICH = {"W1": asgd.ASGD_PARAM_W1, "b1": asgd.ASGD_PARAM_B1, "Wh": asgd.ASGD_PARAM_WH,
         "bh": asgd.ASGD_PARAM_BH, "W2": asgd.ASGD_PARAM_W2, "b2": asgd.ASGD_PARAM_B2}


def _step(name, features, labels, rows, nnz, row_labels, bf16=True, extra=False, stored=False):
    return {"name": name, "kind": "step", "features": features, "labels": labels, "rows": rows, "nnz": nnz,
            "row_labels": row_labels, "bf16": bf16, "extra": extra, "stored": stored}


def listed():
    return [
        # The package's four workloads at their own batch sizes.  tiny is the smallest call:
        # fp32 operands, a model that fits the caches, a step of launches and latency.
        _step("tiny step", 5_000, 1_000, 128, 20.0, 2.0, bf16=False),
        _step("mid step", 100_000, 30_000, 256, 75.0, 4.0),
        _step("wide-feature step", 782_585, 205_443, 128, 330.0, 74.0),
        _step("wide-label step", 135_909, 670_091, 256, 77.0, 4.5),
        # The largest batch of the elastic configuration, and a size in between, as the
        # batch-size scaling of Alg. 1 leaves it: any whole number of rows.
        _step("wide-label step b_max", 135_909, 670_091, 1_024, 77.0, 4.5),
        _step("wide-label step ragged", 135_909, 670_091, 611, 77.0, 4.5),
        # The options: a second hidden layer (on a short last batch), and the output layer
        # that stores its logits.
        _step("mid step two layers", 100_000, 30_000, 203, 75.0, 4.0, extra=True),
        _step("wide-label step stored logits", 135_909, 670_091, 256, 77.0, 4.5, stored=True),
        # Prediction: a small request, and the evaluation of held-out rows after a round
        # (the largest call: 16,384 rows is the most that one takes).
        {"name": "predict small", "kind": "predict", "features": 100_000, "labels": 30_000, "rows": 50, "nnz": 75.0,
         "k": 5, "bf16": True},
        {"name": "predict evaluation", "kind": "predict", "features": 135_909, "labels": 670_091, "rows": 16_384,
         "nnz": 77.0, "k": 1, "bf16": True},
        # The merge of Alg. 2 and a whole round (steps of changing batch sizes, the norms of
        # the perturbation's gate, the merge, the broadcast) with the configuration's 4 replicas.
        {"name": "merge", "kind": "merge", "features": 135_909, "labels": 670_091, "replicas": 4},
        {"name": "elastic round", "kind": "round", "features": 135_909, "labels": 670_091, "nnz": 77.0,
         "row_labels": 4.5, "replicas": 4, "b_min": 64, "b_max": 512, "megabatch": 12_288, "rows": 8_192},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step",) * 6 + ("predict",) * 2 + ("merge", "round"))
    features, labels = _log(rng, 5_000, 782_585), _log(rng, 1_000, 670_091)
    nnz, row_labels = round(rng.uniform(20, 330), 1), round(math.exp(rng.uniform(math.log(2), math.log(74))), 1)
    if kind == "step":
        bf16 = rng.random() < 0.8
        # fp32 operands are for small models here (the tiny workload's)
        labels = labels if bf16 else _log(rng, 1_000, 30_000)
        rows = _log(rng, 16, 1_024 if bf16 else 512)
        out = _step("", features, labels, rows, nnz, row_labels, bf16=bf16, extra=rng.random() < 0.2,
                    stored=rng.random() < 0.1)
        del out["name"]
        return out
    if kind == "predict":
        return {"kind": kind, "features": features, "labels": labels, "rows": _log(rng, 1, 8_192), "nnz": nnz,
                "k": rng.randint(1, 8), "bf16": rng.random() < 0.9}
    if kind == "merge":
        return {"kind": kind, "features": features, "labels": labels, "replicas": rng.randint(2, 4)}
    b_max = 8 * _log(rng, 8, 64)
    return {"kind": kind, "features": features, "labels": labels, "nnz": nnz, "row_labels": row_labels,
            "replicas": rng.randint(2, 4), "b_min": max(1, b_max // 8), "b_max": b_max,
            "megabatch": 16 * b_max + rng.randint(0, b_max), "rows": 4_096}


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _data(case, seed):
    n = case["nnz"]
    # rows of n entries on average: short rows vary by Poisson's law, others are lognormal
    w = synth.Workload("case", case["features"], case["labels"], case["rows"], case["rows"], LR, True,
                       "poisson" if n < 25 else "lognormal", n if n < 25 else math.log(n) - 0.32,
                       0.0 if n < 25 else 0.8, 5_000, 1.05, "uniform", "poisson",
                       max(case.get("row_labels", 1.0) - 1.0, 0.0), 1.2, 0)
    return synth.generate(w, seed=seed)


def _weights(case, seed):
    """Weights of a trained model's scale, on the GPU: |H1| about 4, logits that differ by units."""
    F, L = case["features"], case["labels"]
    r = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda scale, *shape: torch.randn(*shape, generator=r, device="cuda") * scale  # noqa: E731
    out = {"W1": normal(0.5, F, H), "b1": normal(0.1, H)}
    if case.get("extra"):
        out.update(Wh=normal(0.12, H, H), bh=normal(0.1, H))
    out.update(W2=normal(0.15, L, H), b2=normal(0.3, L))
    return out


class _Model:
    """A model handle that is freed with its last user."""

    def __init__(self, case, rows, nnz, lnnz, seed=0):
        self.h = None
        self.F, self.L, self.extra = case["features"], case["labels"], bool(case.get("extra"))
        self.h = asgd.asgd_model_init(
            self.F, self.L, rows, max(nnz, 1), max(lnnz, 1), gemm_bf16=case.get("bf16", True), seed=seed,
            stream=torch.cuda.current_stream(), extra_hidden_layers=int(self.extra),
            flags=asgd.ASGD_UNFUSED_OUTPUT if case.get("stored") else 0)

    def set(self, weights):
        for k, v in weights.items():
            asgd.asgd_model_set_params(self.h, WHICH[k], v.cpu().numpy())
        return self

    def __del__(self):
        if self.h:
            asgd.asgd_model_free(self.h)


def _read(handle, F, L, name):
    shape = {"W1": (F, H), "b1": (H,), "Wh": (H, H), "bh": (H,), "W2": (L, H), "b2": (L,)}[name]
    return asgd.asgd_model_get_params(handle, WHICH[name], shape)


class _Later(dict):
    """Outputs that live in the library's own buffers, read when they are looked at."""

    def __init__(self, keys, get):
        super().__init__((k, None) for k in keys)
        self.get_now = get

    def __getitem__(self, key):
        return self.get_now(key)


# ---------------------------------------------------------------------------------------
# one state per kind
# ---------------------------------------------------------------------------------------
class _StepState:
    def __init__(self, case, seed):
        self.case, self.seed = case, seed
        ds = _data(case, seed)
        B = case["rows"]
        self.data = dx, dy = asgd.DeviceCSR(ds.x), asgd.DeviceCSR(ds.y)
        self.x, self.y = dx.batch(0, B), dy.batch(0, B)
        self.model = _Model(case, B, ds.x.nnz, ds.y.nnz).set(_weights(case, seed))
        self.keys = [k for k in NAMES if self.model.extra or k not in ("Wh", "bh")] + ["loss"]

    def get(self, key):
        m = self.model
        if key == "loss":
            return asgd.asgd_model_last_loss(m.h)
        before = _weights(self.case, self.seed)[key].cpu().numpy()
        return _read(m.h, m.F, m.L, key) - before

    def run(self):
        asgd.asgd_train_step(self.model.h, self.x, self.y, LR)
        return _Later(self.keys, self.get)


class _PredictState:
    def __init__(self, case, seed):
        ds = _data(case, seed)
        B, self.k = case["rows"], case["k"]
        self.data = asgd.DeviceCSR(ds.x)
        self.x = self.data.batch(0, B)
        self.model = _Model(case, B, ds.x.nnz, 1).set(_weights(case, seed))
        self.ids = torch.empty((B, self.k), dtype=torch.int32, device="cuda")
        self.scores = torch.empty((B, self.k), dtype=torch.float32, device="cuda")

    def run(self):
        asgd.asgd_predict_topk(self.model.h, self.x, self.k, self.ids, self.scores)
        return {"ids": self.ids, "scores": self.scores}


GAMMA = 0.9


def _merge_models(case, seed):
    """Weights of the global model, the one before it and the replicas, one after the other."""
    for k in range(case["replicas"] + 2):
        yield _weights(case, seed * 32 + k)


def _alpha(case, seed):
    a = np.random.default_rng(seed).uniform(0.5, 1.5, case["replicas"])
    return (a / a.sum()).astype(np.float32)


class _MergeState:
    def __init__(self, case, seed):
        self.case = case
        self.models = [_Model(case, 8, 64, 64).set(w) for w in _merge_models(case, seed)]
        self.alpha = [float(a) for a in _alpha(case, seed)]
        self.keys = [who + "." + k for who in ("global", "replica") for k in ("W1", "b1", "W2", "b2")]

    def get(self, key):
        who, name = key.split(".")
        m = self.models[0 if who == "global" else 2]
        return _read(m.h, m.F, m.L, name)

    def run(self):
        h = [m.h for m in self.models]
        asgd.asgd_merge(h[0], h[1], h[2:], self.alpha, GAMMA, True)
        return _Later(self.keys, self.get)


class _RoundState:
    def __init__(self, case, seed):
        self.e = None
        self.case, self.seed = case, seed
        n, b_max = case["replicas"], case["b_max"]
        ds = _data(case, seed)
        ipx, ipy = np.asarray(ds.x.indptr), np.asarray(ds.y.indptr)
        most = lambda ip: int(np.max(ip[b_max:] - ip[:-b_max]))  # noqa: E731
        self.data = dx, dy = asgd.DeviceCSR(ds.x), asgd.DeviceCSR(ds.y)
        self.x, self.y = dx.batch(0, case["rows"]), dy.batch(0, case["rows"])
        self.ipx, self.ipy = ipx.astype(np.int32), ipy.astype(np.int32)
        model = asgd.asgd_config(n_features=case["features"], n_labels=case["labels"], hidden=H, max_batch=b_max,
                                 max_nnz=most(ipx), max_label_nnz=most(ipy), gemm_bf16=1)
        c = asgd.asgd_elastic_config()
        c.n_replicas, c.b_min, c.b_max, c.beta, c.lr, c.gamma = n, case["b_min"], b_max, case["b_min"] / 2.0, LR, GAMMA
        c.weight_mode, c.perturb, c.pert_thr, c.delta = asgd.ASGD_WEIGHTS_ALG2, 1, 0.1, 0.1
        c.megabatch, c.dispatch, c.clock = case["megabatch"], asgd.ASGD_DISPATCH_DYNAMIC, asgd.ASGD_CLOCK_VIRTUAL
        c.c0, c.c1, c.c2 = 1e-4, 2e-6, 2e-8
        for i, v in enumerate((1.0, 1.3, 1.6, 2.0)[:n]):
            c.slow[i] = v
        self.streams = [torch.cuda.Stream() for _ in range(n)]
        self.e = asgd.asgd_elastic_create(c, model, seed, self.streams, torch.cuda.current_stream())
        self.keys = ["W1", "b1", "W2", "b2", "u", "samples", "b_next", "cursor", "schedule"]

    def get(self, key):
        if key not in WHICH:
            v = self.log[key]
            return np.array(v[:self.case["replicas"]] if key in ("u", "samples", "b_next") else v, dtype=np.int64)
        F, L = self.case["features"], self.case["labels"]
        first = _Model(self.case, 1, 1, 1, seed=self.seed)  # the models that every replica started from
        return _read(asgd.asgd_elastic_model(self.e, -1), F, L, key) - _read(first.h, F, L, key)

    def run(self):
        self.log = asgd.asgd_elastic_round(self.e, self.x, self.y, self.ipx, self.ipy)
        return _Later(self.keys, self.get)

    def __del__(self):
        if self.e:
            asgd.asgd_elastic_free(self.e)


def prepare(case, seed):
    return {"step": _StepState, "predict": _PredictState, "merge": _MergeState,
            "round": _RoundState}[case["kind"]](case, seed)


def run(state):
    return state.run()


# ---------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------
def _distinct(features, draws):
    """Distinct ids among `draws` draws of the generator's Zipf law, on average."""
    p = np.arange(1, features + 1, dtype=np.float64) ** -1.05
    return float(-np.expm1(draws * np.log1p(-p / p.sum())).sum())


def _step_work(F, L, B, nnz, row_labels, extra):
    N, M = B * nnz, B * row_labels
    # every parameter the step writes is read and written once: W2, b2 and the touched rows of
    # W1; the batch's entries (id and value; label id) are read once
    params = L * (H + 1) + _distinct(F, N) * H + H + (H * H + H if extra else 0)
    # Z, dH and dW2 over all labels; the first layer forward and its gradient
    return {"bytes": 8.0 * params + 8.0 * N + 4.0 * M + 8.0 * B,
            "flops": 6.0 * B * H * L + 4.0 * N * H + (6.0 * B * H * H if extra else 0.0)}


def work(case):
    F, L = case["features"], case["labels"]
    P = (F + L) * H + H + L
    if case["kind"] == "step":
        return _step_work(F, L, case["rows"], case["nnz"], case["row_labels"], case["extra"])
    if case["kind"] == "predict":
        B, N = case["rows"], case["rows"] * case["nnz"]
        return {"bytes": 4.0 * L * (H + 1) + 4.0 * _distinct(F, N) * H + 8.0 * N + 8.0 * B * case["k"],
                "flops": 2.0 * B * H * L + 2.0 * N * H}
    n = case["replicas"]
    merge = 4.0 * P * ((n + 2) + (n + 1))  # reads replicas, global and previous; writes global and replicas
    if case["kind"] == "merge":
        return {"bytes": merge, "flops": 2.0 * (n + 1) * P}
    steps = case["megabatch"] / (0.8 * case["b_max"])
    one = _step_work(F, L, case["megabatch"] / steps, case["nnz"], case["row_labels"], False)
    return {"bytes": steps * one["bytes"] + merge + 4.0 * n * P, "flops": steps * one["flops"] + 2.0 * (2 * n + 1) * P}


def tolerance(case):
    if case["kind"] == "merge":
        return {"rel": 1e-6}  # float64 sums rounded once: 3.5e-8 from the exact result
    if not case.get("bf16", True):
        # fp32 sums: a step's change of W1 is 1.2e-4 from the exact one (the rounding of the
        # weights themselves), logits 1e-6
        return {"rel": 5e-4 if case["kind"] == "step" else 1e-5, "max": 0.05, "differ": 0.01}
    # bf16 operands: logits are up to 7e-4 from the exact ones, a step's change up to 3.5e-3;
    # ids differ where two logits are closer than that
    return {"rel": 0.003 if case["kind"] == "predict" else 0.01, "max": 0.5, "differ": 0.01}


# ---------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------
def _entries(csr):
    ip = torch.from_numpy(np.asarray(csr.indptr)).cuda()
    row = torch.repeat_interleave(torch.arange(csr.n_rows, device="cuda"), ip[1:] - ip[:-1])
    val = None if csr.values is None else torch.from_numpy(csr.values).cuda().double()
    return row, torch.from_numpy(csr.indices).cuda().long(), val


def _first_layer(w, x, B):
    row, col, val = _entries(x)
    return w["b1"].expand(B, H).clone().index_add_(0, row, val[:, None] * w["W1"][col])


def _exact_step(case, seed):
    w = {k: v.double() for k, v in _weights(case, seed).items()}
    ds, B = _data(case, seed), case["rows"]
    a1 = _first_layer(w, ds.x, B)
    h = h1 = a1.clamp(min=0)
    if case["extra"]:
        a2 = h1 @ w["Wh"].T + w["bh"]
        h = a2.clamp(min=0)
    z = torch.addmm(w["b2"], h, w["W2"].T)
    row, lab, _ = _entries(ds.y)
    share = (1.0 / torch.bincount(row, minlength=B).double())[row]
    lse = torch.logsumexp(z, 1)
    loss = (lse.sum() - (share * z[row, lab]).sum()) / B
    z.sub_(lse[:, None]).exp_()
    z.index_put_((row, lab), -share, accumulate=True)
    dz = z.div_(B)
    g = {"W2": dz.T @ h, "b2": dz.sum(0)}
    d = dz @ w["W2"]
    if case["extra"]:
        d = d * (a2 > 0)
        g.update(Wh=d.T @ h1, bh=d.sum(0))
        d = d @ w["Wh"]
    d = d * (a1 > 0)
    g["b1"] = d.sum(0)
    row, col, val = _entries(ds.x)
    g["W1"] = torch.zeros_like(w["W1"]).index_add_(0, col, val[:, None] * d[row])
    return dict({k: -LR * v for k, v in g.items()}, loss=float(loss))


def _exact_predict(case, seed):
    w = {k: v.double() for k, v in _weights(case, seed).items()}
    ds, B = _data(case, seed), case["rows"]
    h = _first_layer(w, ds.x, B).clamp(min=0)
    top = [torch.addmm(w["b2"], part, w["W2"].T).topk(case["k"], 1).values for part in h.split(2_048)]
    return {"ids": None, "scores": torch.cat(top)}


def _exact_merge(case, seed):
    out = None
    for k, w in enumerate(_merge_models(case, seed)):
        c = GAMMA if k == 0 else -GAMMA if k == 1 else float(_alpha(case, seed)[k - 2])
        w = {n: c * v.double() for n, v in w.items()}
        out = w if out is None else {n: out[n].add_(v) for n, v in w.items()}
    return {who + "." + k: v for who in ("global", "replica") for k, v in out.items()}


def exact(case, seed):
    if case["kind"] == "round":
        return None  # dozens of dependent steps
    return {"step": _exact_step, "predict": _exact_predict, "merge": _exact_merge}[case["kind"]](case, seed)
