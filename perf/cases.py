"""Timed cases of the Tsetlin machine library: what a program does with it, through its public entry points.

Training comes as whole epochs or batches of Algorithm 1, inference as predictions, class sums and clause
outputs, and a resumed session as loading automata, binding the data and saving again.  The machines are the
repository's workloads (noisy XOR, image-like, text-like, planted conjunctions at reduced clause count,
regression) and what lies between them.

Training is timed in its reproducible form: `tm_feedback_step` on a snapshot of the tallies, then
`tm_sync_tallies`, then the next snapshot - the kernels of `tm_fit_epoch`, with results that do not depend on
how the clauses happen to be scheduled.  One case runs `tm_fit_epoch` on the live tallies.  Inputs are drawn
on the GPU from the seed alone; machines that a case needs trained are trained by `prepare`, reproducibly.
"""
import math

import torch

from paper_2009_04861_amd import binding as B


def listed():
    return [
        # the paper's worked example: a machine of 20 clauses, where an epoch is one clause's chain of feedback
        dict(name="xor_epoch", kind="epoch", data="xor", m=2, n=10, o=12, N=100, T=15, s=3.9, q=5000, pre=4),
        # tabular regression at the paper's setting T = n, in its settled state (a few percent error)
        dict(name="regression_epoch", kind="epoch", data="regression", m=1, n=1280, o=256, N=128, T=1280, s=1.5, q=13911, pre=4),
        # the low end of clause scaling: about one clause per SIMD, every gate open
        dict(name="image_epoch_100", kind="epoch", data="image", m=10, n=100, o=784, N=128, T=80, s=10.0, q=60000, pre=2),
        # the headline machine under steady feedback load (T = 0.8 n keeps the gates open)
        dict(name="image_epoch_2000", kind="epoch", data="image", m=10, n=2000, o=784, N=128, T=1600, s=10.0, q=60000, pre=1),
        # the headline step on a settled machine: live epoch, tally pre-calculation, test predictions
        dict(name="image_step", kind="step", data="image", m=10, n=2000, o=784, N=128, T=50, s=10.0, q=60000, pre=8, q_test=10000),
        # bag-of-words documents, 10,000 words: two launches' worth of documents
        dict(name="text_batch", kind="epoch", data="text", m=2, n=10000, o=10000, N=128, T=8000, s=2.0, q=3328, pre=2),
        # the widest clauses: 20,000 sparse features, one launch's worth of examples
        dict(name="planted_batch", kind="epoch", data="planted", m=2, n=8192, o=20000, N=128, T=5000, s=5.0, q=832, pre=3),
        # test-set predictions of the headline machine, with a kept workspace
        dict(name="image_predict", kind="predict", data="image", m=10, n=2000, o=784, N=128, T=50, s=10.0, q=10000, pre=8),
        # one request of a serving loop: a single example, no workspace of its own
        dict(name="image_predict_one", kind="predict_static", data="image", m=10, n=2000, o=784, N=128, T=50, s=10.0, q=1, pre=8),
        # scoring a document collection
        dict(name="text_class_sums", kind="class_sums_ws", data="text", m=2, n=10000, o=10000, N=128, T=8000, s=2.0, q=25000, pre=2),
        # which clauses fire for which example (interpretation of a trained machine), from the include masks
        dict(name="image_clause_outputs", kind="clause_outputs", data="image", m=10, n=2000, o=784, N=128, T=50, s=10.0, q=10000, pre=8),
        # a session resumed from saved automata: load, bind the training data (tallies included), save
        dict(name="image_resume", kind="resume", data="image", m=10, n=2000, o=784, N=128, T=50, s=10.0, q=60000, pre=8),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Most (clause, example, literal word) triples of a drawn case - those of the listed training cases; a triple is far
# cheaper in inference - and most (example, literal word) pairs one clause walks in a training pass.
MOST_TRAIN, MOST_INFER, MOST_WALK = 1.5e10, 1.0e11, 6.0e6


def draw(rng):
    kind = rng.choice(["epoch"] * 6 + ["step", "predict", "predict", "predict_static", "class_sums_ws", "class_sums", "clause_outputs", "resume"])
    if kind == "step":  # live epochs are compared on a settled machine of the headline's kind
        n = 2 * rng.randint(500, 1000)
        return dict(kind=kind, data="image", m=10, n=n, o=rng.randint(600, 1000), N=128, T=n // 40, s=10.0,
                    q=rng.randint(30000, 60000), pre=8, q_test=_log_uniform(rng, 100, 10000))
    o = _log_uniform(rng, 12, 20000)
    n = max(10, _log_uniform(rng, 10, 10000) & ~1)
    data, m = ("xor", 2) if o < 24 else ("image", rng.choice([2, 3, 5, 10])) if o < 2500 else (rng.choice(["text", "planted"]), 2)
    if data == "image" and o % 16 == 0 or (data == "image" and rng.random() < 0.2):
        data, m, o = "regression", 1, (o + 15) // 16 * 16
    s = 1.5 if data == "regression" else rng.choice([2.0, 3.9, 5.0, 10.0, 25.0])
    q = _log_uniform(rng, 500, 60000) if kind in ("epoch", "resume") else _log_uniform(rng, 1, 30000)
    most = MOST_TRAIN if kind == "epoch" else MOST_INFER
    words = 2 * ((o + 31) // 32)
    while m * n * max(q, 500) * words > most and n > 100:
        n = max(100, (n // 2) & ~1)
    while m * n * q * words > most or (kind == "epoch" and q * words > MOST_WALK):
        q //= 2
    if kind == "predict_static":
        # what the static workspace holds: lists of every clause, rows of every literal
        n = min(n, 2 * (2 ** 21 // (m * max(128, o // 4)) // 2) or 2)
        q = min(q, 2048)
    T = n if data == "regression" else max(2, int(n * rng.choice([0.8, 0.025])))
    return dict(kind=kind, data=data, m=m, n=n, o=o, N=rng.choice([100, 128, 128]), T=T, s=s, q=max(1, q), pre=3)


# ---- inputs -------------------------------------------------------------------------------------------------

def _pack(bits, Wf):
    """bool [q][o] -> int32 [q][Wf], feature k in bit k % 32 of word k / 32."""
    q, o = bits.shape
    pad = torch.zeros((q, Wf * 32), dtype=torch.bool, device=bits.device)
    pad[:, :o] = bits
    out = torch.empty((q, Wf), dtype=torch.int32, device=bits.device)
    weights = torch.ones(32, dtype=torch.int64, device=bits.device) << torch.arange(32, device=bits.device)
    for a in range(0, q, 8192):
        words = (pad[a:a + 8192].view(-1, Wf, 32).to(torch.int64) * weights).sum(2)
        out[a:a + 8192] = torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32)
    return out


def _task(case, seed):
    """A learning task of the case's kind: function q, label noise -> (packed features, labels int32)."""
    dev = torch.device("cuda", 0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    m, o, Wf = case["m"], case["o"], (case["o"] + 31) // 32

    def rand(*shape):
        return torch.rand(shape, generator=gen, device=dev)

    def randint(hi, *shape):
        return torch.randint(0, hi, shape, generator=gen, device=dev)

    if case["data"] == "xor":
        def more(q, noise):
            x = rand(q, o) < 0.5
            y = (x[:, 0] ^ x[:, 1]) ^ (rand(q) < (0.4 if noise else 0.0))
            return _pack(x, Wf), y.to(torch.int32)
    elif case["data"] == "image":  # one prototype per class, a tenth of the pixels flipped
        proto = rand(m, o) < 0.2
        def more(q, noise):
            y = randint(m, q)
            return _pack(proto[y] ^ (rand(q, o) < 0.1), Wf), y.to(torch.int32)
    elif case["data"] == "text":  # word presence falls with rank, about 150 words a document, 200 marker words a class
        base = torch.arange(1, o + 1, device=dev, dtype=torch.float32) ** -1.1
        scale = 1.0
        for _ in range(60):
            scale *= (min(150, o / 8) / torch.clamp(base * scale, max=1.0).sum().item()) ** 0.9
        p = torch.clamp(base * scale, max=1.0).repeat(m, 1)
        markers = 50 + torch.randperm(min(o, 5000) - 50, generator=gen, device=dev)[:200 * m].view(m, 200)
        p.scatter_(1, markers, torch.clamp(3.0 * p.gather(1, markers), max=1.0))
        def more(q, noise):
            y = randint(m, q)
            x = torch.empty((q, o), dtype=torch.bool, device=dev)
            for a in range(0, q, 8192):
                x[a:a + 8192] = rand(min(8192, q - a), o) < p[y[a:a + 8192]]
            return _pack(x, Wf), y.to(torch.int32)
    elif case["data"] == "planted":  # 64 hidden conjunctions of three literals, combined by majority
        feats, plain = randint(o, 64, 3), rand(64, 3) < 0.5
        def more(q, noise):
            x = torch.empty((q, o), dtype=torch.bool, device=dev)
            for a in range(0, q, 4096):
                x[a:a + 4096] = rand(min(4096, q - a), o) < 0.05
            hits = (x[:, feats] == plain).all(2).sum(1)
            return _pack(x, Wf), (hits >= hits.median()).to(torch.int32)
    else:  # 16 thermometer bits for each of o / 16 uniform columns
        cols = o // 16
        def more(q, noise):
            u = rand(q, cols)
            f = 0.4 * torch.exp(-((u[:, 0] - 0.55) / 0.18) ** 2) + 0.25 * u[:, 1 % cols] + 0.2 * (u[:, 2 % cols] > 0.5) * u[:, 3 % cols] \
                + 0.15 * u[:, 4 % cols] * u[:, 5 % cols]
            f = torch.clamp(f + (0.03 * torch.randn(q, generator=gen, device=dev) if noise else 0.0), 0.0, 1.0)
            cuts = (torch.arange(16, device=dev) + 0.5) / 16
            return _pack((u[:, :, None] > cuts).reshape(q, o), Wf), torch.round(f * case["T"]).to(torch.int32)
    more.gen = gen
    return more


def _snapshot_of_settled_regression(y, T, gen):
    """Tallies of a regression machine whose error is a few percent of the target range."""
    off = 0.055 * T * torch.randn(y.shape, generator=gen, device=y.device)
    return torch.round(y + off).to(torch.int32).view(-1, 1).contiguous()


def _epoch(tm, state):
    """One reproducible epoch: Algorithm 1 on the snapshot, tallies recomputed, the next snapshot taken."""
    B.tm_set_epoch(tm.h, state["epoch"])
    state["epoch"] += 1
    B.tm_feedback_step(tm.h, state["snapshot"], 0, tm.q)
    B.tm_sync_tallies(tm.h)
    B.tm_get_tallies(tm.h, state["tallies"])
    if not state["fixed"]:
        state["snapshot"], state["tallies"] = state["tallies"], state["snapshot"]
        return state["snapshot"]
    return state["tallies"]


def prepare(case, seed):
    regression = case["data"] == "regression"
    tm = B.TsetlinMachine(case["m"], case["n"], case["o"], case["N"], case["T"], case["s"], 1000003 + seed, regression=regression)
    start = tm.get_ta_state()
    tm.state_buf.zero_()  # the buffer's padding too, which nothing writes
    tm.set_ta_state(start)
    del start
    more = _task(case, seed)
    trains = case["kind"] in ("epoch", "step", "resume")
    q_train = case["q"] if trains else min(60000, int(MOST_TRAIN / (tm.C * 2 * tm.Wf)), 4000 if case["data"] in ("text", "planted") else 60000)
    X, y = more(max(64, q_train) if not trains else q_train, True)
    tm.bind_train(X, y)
    state = dict(tm=tm, kind=case["kind"], epoch=0, fixed=regression, tallies=tm.tallies(), snapshot=tm.tallies())
    if regression:
        state["snapshot"] = _snapshot_of_settled_regression(y, case["T"], more.gen)
    for _ in range(case["pre"]):
        _epoch(tm, state)
    q = case.get("q_test", case["q"])
    if case["kind"] == "resume":
        state["saved"] = tm.get_ta_state()
        state["loaded"] = torch.empty_like(state["saved"])
    elif case["kind"] != "epoch":
        state["X"] = more(q, False)[0]
        state["pred"] = torch.empty(q, dtype=torch.int32, device=tm.dev)
        state["sums"] = torch.empty((q, tm.m), dtype=torch.int32, device=tm.dev)
        if case["kind"] == "clause_outputs":
            state["bits"] = torch.empty((tm.C, (q + 31) // 32), dtype=torch.int32, device=tm.dev)
        elif case["kind"] in ("predict", "class_sums_ws", "step"):
            state["ws"] = torch.empty(B.tm_infer_ws_bytes(tm.cfg, q), dtype=torch.uint8, device=tm.dev)
    if case["kind"] == "step":
        B.tm_set_epoch(tm.h, state["epoch"])
    return state


def run(state):
    tm, kind = state["tm"], state["kind"]
    if kind == "epoch":
        return _epoch(tm, state), tm.state_buf
    if kind == "step":
        B.tm_fit_epoch(tm.h)
        B.tm_sync_tallies(tm.h)
        B.tm_predict_ws(tm.h, state["X"], state["pred"], state["sums"], state["ws"])
        return state["pred"], tm.state_buf
    if kind == "predict":
        B.tm_predict_ws(tm.h, state["X"], state["pred"], state["sums"], state["ws"])
        return state["pred"], state["sums"]
    if kind == "predict_static":
        B.tm_predict_static(tm.h, state["X"], state["pred"])
        return state["pred"]
    if kind == "class_sums_ws":
        B.tm_class_sums_ws(tm.h, state["X"], state["sums"], state["ws"])
        return state["sums"]
    if kind == "class_sums":
        B.tm_class_sums(tm.h, state["X"], state["sums"])
        return state["sums"]
    if kind == "clause_outputs":
        B.tm_clause_outputs(tm.h, state["X"], state["bits"])
        return state["bits"]
    B.tm_set_ta_state(tm.h, state["saved"])
    B.tm_bind_train(tm.h, tm.X, tm.y, tm.ws)
    B.tm_get_ta_state(tm.h, state["loaded"])
    B.tm_get_tallies(tm.h, state["tallies"])
    return state["tallies"], state["loaded"]


def work(case):
    """Bytes: inputs and state read once, outputs and updated state written once.  Operations: one per clause and example."""
    C, Wf, q, m = case["m"] * case["n"], (case["o"] + 31) // 32, case["q"], case["m"]
    examples, masks, automata = q * Wf * 4, C * 2 * Wf * 4, C * 2 * Wf * 36
    sums, outputs = q * m * 4, C * ((q + 31) // 32) * 4
    kind, pairs = case["kind"], C * q
    if kind == "epoch":      # previous outputs are read and rewritten, and so are the automata
        return {"bytes": examples + 4 * q + 2 * automata + 3 * sums + 2 * outputs, "flops": pairs}
    if kind == "step":       # a settled machine moves few of its automata: its masks have to be read
        qt = case["q_test"]
        return {"bytes": examples + 4 * q + 2 * masks + 3 * sums + 2 * outputs + qt * Wf * 4 + qt * 4 * (m + 1), "flops": pairs + C * qt}
    if kind == "clause_outputs":
        return {"bytes": examples + masks + outputs, "flops": pairs}
    if kind == "resume":     # automata in and out as bytes, data, tallies, previous outputs
        return {"bytes": 2 * C * 2 * case["o"] + 2 * automata + examples + 4 * q + 2 * sums + outputs, "flops": pairs}
    return {"bytes": examples + masks + sums + (4 * q if kind == "predict" else 0), "flops": pairs}


def tolerance(case):
    # Integer work throughout.  Only the live epoch depends on which clause happens to act first: two runs of one build
    # differ in a few bytes per thousand of the automata.
    return {"differ": 0.008} if case["kind"] == "step" else "exact"
