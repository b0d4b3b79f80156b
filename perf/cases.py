"""What the speed of this library is measured on.

Every case is a call, or a burst of calls, that a program built on the library makes again and
again through the public binding: train steps on a filled replay, batches sampled for a learner
of the program's own, and experiences added.  The network and replay sizes are those of the
benchmark and the tests (the paper-shaped 27-256-256-30 network, the paper's own dueling network
27-128-(512+512)-(1+30), the wide mixed-precision network 27-1024-1024-30, a replay of 1,000,000
experiences, 84x84x4 byte frames) or generic ones around them.  States and rewards are normal
deviates, actions uniform, terminals rare, as in the benchmark.

Kinds of cases
  train   `count` consecutive train steps in one call, on a full replay, each adding `appends`
          experiences (count = 1: the call an acting-and-learning loop makes per frame); outputs:
          weights, gradients of the last step, Adam moments
  sample  one batch drawn, gathered and unpacked; outputs: the batch and its slot numbers
  append  `rows` experiences added in one call; outputs: the ring's rows
"""
import math

import numpy as np
import torch

from paper_1801_03138_amd import binding as B
from paper_1801_03138_amd import synth

_DTYPE = {"f32": B.RP_F32, "bf16": B.RP_BF16, "u8": B.RP_U8}
_BYTES = {"f32": 4, "bf16": 2, "u8": 1}


def _train(**kw):
    case = dict(kind="train", dtype="f32", capacity=1_000_000, D=27, H=256, G=256, A=30, batch=128,
                count=32, appends=1, host=False, target=0, dueling=False, distinct=False, opt="adam",
                loss="huber")
    case.update(kw)
    return case


def _sample(**kw):
    case = dict(kind="sample", dtype="f32", layout="pair", capacity=1_000_000, D=27, batch=32,
                distinct=False)
    case.update(kw)
    return case


def _append(**kw):
    case = dict(kind="append", dtype="f32", layout="pair", capacity=1_000_000, D=27, rows=2000, host=True)
    case.update(kw)
    return case


def listed():
    return [
        # The loop of one actor that learns as it plays: a frame comes from the host, one step is made.
        _train(name="act_and_learn_b32", batch=32, count=1, host=True),
        # The headline: the paper-shaped network at the paper's batch, experiences already on the GPU.
        _train(name="paper_shaped_b128"),
        # The same network on a large, uneven batch, as learners fed by many actors use it.
        _train(name="paper_shaped_b1000", batch=1000, count=8, appends=8),
        # The paper's own network: shared layer, value and advantage streams, frozen target network.
        _train(name="paper_network_b128", H=128, G=1024, target=10_000, dueling=True),
        # A wider fp32 network with a target network and more inputs and actions than one tile.
        _train(name="f32_512_b512", D=50, H=512, G=512, A=40, batch=512, count=8, appends=4, target=10_000),
        # The wide mixed-precision network: the largest step.
        _train(name="bf16_1024_b4096", dtype="bf16", capacity=4_000_000, H=1024, G=1024, batch=4096, count=16,
               appends=64),
        # The paper's own network in mixed precision on a larger batch.
        _train(name="bf16_paper_network_b512", dtype="bf16", H=128, G=1024, batch=512, count=8, appends=4,
               target=10_000, dueling=True),
        # The smallest sample call: what a learner outside the library asks for per update.
        _sample(name="sample_b32"),
        # A whole epoch's worth of experiences in one call.
        _sample(name="sample_b65536", batch=65_536),
        # Batches without duplicates, as the paper's in-RAM replay draws them.
        _sample(name="sample_distinct_b8192", batch=8192, distinct=True),
        # Large states: 84x84x4 byte frames stored once, unpacked to floats.
        _sample(name="frames_b256", dtype="u8", layout="chain", capacity=200_000, D=84 * 84 * 4, batch=256),
        # The paper's update block: 2000 experiences from host memory.
        _append(name="append_host_2000"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "f32", "f32", "bf16", "bf16", "sample", "sample", "frames", "append"])
    if kind in ("f32", "bf16"):
        two = rng.random() < 0.35
        H = rng.choice([64, 128, 128, 192]) if two else 64 * rng.randint(1, 8 if kind == "f32" else 16)
        G = rng.choice([256, 512, 768, 1024]) if two else H
        count = _log_int(rng, 1, 32 if kind == "f32" else 16)
        return _train(dtype=kind, capacity=_log_int(rng, 20_000, 1_000_000), D=_log_int(rng, 4, 96), H=H, G=G,
                      A=_log_int(rng, 2, 64),
                      batch=_log_int(rng, 16, 2048) if kind == "f32" else _log_int(rng, 64, 4096), count=count,
                      appends=_log_int(rng, 1, 64), host=rng.random() < 0.3,
                      target=rng.choice([0, 10_000]), dueling=rng.random() < 0.3,
                      distinct=rng.random() < 0.15, opt=rng.choice(["adam", "adam", "sgd"]),
                      loss=rng.choice(["huber", "mse"]))
    if kind == "sample":
        distinct = rng.random() < 0.4
        return _sample(dtype=rng.choice(["f32", "bf16", "u8"]), capacity=_log_int(rng, 100_000, 1_000_000),
                       D=_log_int(rng, 4, 64), batch=_log_int(rng, 16, 65_536), distinct=distinct)
    if kind == "frames":
        dtype = rng.choice(["u8", "u8", "f32"])
        return _sample(dtype=dtype, layout="chain", capacity=_log_int(rng, 2_000, 50_000),
                       D=_log_int(rng, 500, 28_224 if dtype == "u8" else 14_112), batch=_log_int(rng, 4, 256))
    layout = rng.choice(["pair", "pair", "chain"])
    return _append(dtype=rng.choice(["f32", "bf16", "u8"]), layout=layout, D=_log_int(rng, 4, 64),
                   rows=_log_int(rng, 1, 65_536), host=rng.random() < 0.5)


# ------------------------------------------------------------------------------------- inputs
def _experiences(gen, n, case, actions):
    """n experiences on the GPU, structure of arrays."""
    D, dt = case["D"], case["dtype"]
    chain = case.get("layout") == "chain"

    def states():
        if dt == "u8":
            return torch.randint(0, 256, (n, D), dtype=torch.uint8, device="cuda", generator=gen)
        x = torch.randn((n, D), device="cuda", generator=gen)
        return x.to(torch.bfloat16) if dt == "bf16" else x
    s = states()
    s_next = None if chain else states()
    a = torch.randint(0, actions, (n,), dtype=torch.int32, device="cuda", generator=gen)
    r = torch.randn(n, device="cuda", generator=gen)
    term = (torch.rand(n, device="cuda", generator=gen) < 0.005).to(torch.uint8)
    return s, s_next, a, r, term


def _fill(ring, gen, case, actions):
    left, D = case["capacity"], case["D"]
    piece = max(1, min(left, 64 * 1024 * 1024 // D))
    while left:
        n = min(piece, left)
        ring.append(*_experiences(gen, n, case, actions))
        left -= n


def _to_host(rows):
    def one(t):
        if t is None:
            return None
        if t.dtype == torch.bfloat16:
            return t.view(torch.int16).cpu().numpy().view(np.uint16)
        return t.cpu().numpy()
    return tuple(one(t) for t in rows)


def _take(rows, lo, hi):
    return tuple(None if x is None else x[lo:hi] for x in rows)


_WINDOWS = 4   # bursts of new experiences that a state holds and hands over in turn


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    layout = B.RP_CHAIN if case.get("layout") == "chain" else B.RP_PAIR
    kind = case["kind"]
    actions = case.get("A", 30)
    ring = B.Replay(case["capacity"], case["D"], _DTYPE[case["dtype"]], layout, seed=seed,
                    max_append=64 if kind == "sample" else 4096,
                    distinct=case.get("distinct", False))
    _fill(ring, gen, case, actions)
    state = {"kind": kind, "ring": ring, "at": 0}
    if kind == "sample":
        state["batch"] = case["batch"]
        state["out"] = ring.alloc_batch(case["batch"])
    elif kind == "append":
        n = case["rows"]
        rows = _experiences(gen, _WINDOWS * n, case, actions)
        rows = _to_host(rows) if case["host"] else rows
        state["windows"] = [_take(rows, k * n, k * n + n) for k in range(_WINDOWS)]
    else:
        H, G, D, O = case["H"], case["G"], case["D"], actions + (1 if case["dueling"] else 0)
        trainer = B.Trainer(
            ring, H, actions, case["batch"], param_dtype=_DTYPE[case["dtype"]],
            loss=B.RP_HUBER if case["loss"] == "huber" else B.RP_MSE,
            opt=B.RP_ADAM if case["opt"] == "adam" else B.RP_SGD, appends_per_step=case["appends"], lr=1e-4,
            target_sync=case["target"], dueling=case["dueling"], hidden2=0 if G == H else G,
            init_params=synth.init_params(D, H, O, seed, hidden2=None if G == H else G))
        n = case["count"] * case["appends"]
        rows = _experiences(gen, _WINDOWS * n, case, actions)
        rows = _to_host(rows) if case["host"] else rows
        state["windows"] = [_take(rows, k * n, k * n + n) for k in range(_WINDOWS)]
        state["trainer"] = trainer
        state["count"] = case["count"]
        # The trainer's arrays in the caller's own workspace: weights, gradients, first and second
        # moments, each padded to whole 32-wide tiles and, with the dueling head, followed by the
        # head's own parameters (the padded output layer in front of them is then scratch).
        Dp, Ap = (D + 31) // 32 * 32, (actions + 31) // 32 * 32
        body = Dp * H + H + H * G + G
        padded = body + G * Ap + Ap
        parts = [(0, body), (padded, padded + (G + 1) * O)] if case["dueling"] else [(0, padded)]
        pitch = (4 * parts[-1][1] + 255) // 256 * 256
        # Gradients of the last step, except in mixed precision under Adam: there they depend on
        # how the roundings of the burst's earlier steps fell, and the moments say the same.
        names = {"weights": 0}
        if case["dtype"] == "f32" or case["opt"] == "sgd":
            names["gradients"] = 1
        if case["opt"] == "adam":
            names.update(m=2, v=3)
        state["out"] = {name: [trainer.workspace[256 + k * pitch + 4 * lo:256 + k * pitch + 4 * hi].view(torch.float32)
                               for lo, hi in parts] for name, k in names.items()}
    torch.cuda.synchronize()
    return state


# --------------------------------------------------------------------------------- one pass
def run(state):
    at = state["at"]
    state["at"] = at + 1
    if state["kind"] == "sample":
        state["ring"].sample_gather(at, state["batch"], out=state["out"])
        return state["out"]
    rows = state["windows"][at % _WINDOWS]
    if state["kind"] == "append":
        state["ring"].append(*rows)
        return state["ring"].storage
    if state["count"] == 1:
        state["trainer"].step(*rows)
    else:
        state["trainer"].steps(state["count"], *rows)
    return state["out"]


# ------------------------------------------------------------- what a pass cannot do without
def work(case):
    D, e = case["D"], _BYTES[case["dtype"]]
    if case["kind"] == "append":
        states = (1 if case["layout"] == "chain" else 2) * D * e
        return {"bytes": case["rows"] * 2 * (states + 12), "flops": 0}
    if case["kind"] == "sample":
        out = 4 if case["dtype"] == "u8" else e
        return {"bytes": case["batch"] * (2 * D * (e + out) + 12 + 12 + 4), "flops": 0}
    H, G, A, n = case["H"], case["G"], case["A"], case["batch"]
    O = A + (1 if case["dueling"] else 0)
    params = D * H + H + H * G + G + G * O + O
    # forward on s and s'; backward: weight gradients of the first two layers, the error of the
    # first, and the last layer's share, whose error has one entry per experience (an output and,
    # with the dueling head, what it spreads over the others)
    flops = 2 * n * (2 * (D * H + H * G + G * O) + (D * H + H * G) + H * G + 2 * G)
    # weights and moments once in and once out, gradients out, every sampled row in, new rows in and out
    moved = params * 4 * (7 if case["opt"] == "adam" else 3)
    rows = case["count"] * (n + 2 * case["appends"]) * (2 * D * e + 12)
    return {"bytes": moved + rows, "flops": case["count"] * flops}


def tolerance(case):
    if case["kind"] != "train":
        return "exact"          # bytes are moved, not computed with
    # Four times what the layer-by-layer step, whose sums run in another order, was seen to differ
    # by after two bursts.  A single step differs by 2e-7 in fp32; what grows over a burst is
    # Adam's quotient where a gradient is lost in its own rounding, and units on a ReLU kink.
    if case["dtype"] == "f32":
        return {"rel": 2e-3, "max": 0.15}
    return {"rel": 2.5e-2, "max": 0.8}
