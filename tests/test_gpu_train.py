"""GPU parity of train_step against the CPU oracle, teacher-forced: before each compared
step the oracle is given the GPU's own state (weights, Adam moments, t), both take one step
on the same sampled batch, and Q-values, targets, loss, gradients and new weights are compared.

Tolerances (written here as the test of record; rtol = 1e-5 for fp32, 2e-2 for the bf16
mixed-precision path; "close" means |x - y| <= rtol * max(|x|, |y|) + rtol * max|ref|):
 1. Q(s,.), Q(s',.), targets, loss: close at rtol.
 2. The update rule, with no slack: the oracle's update rule (oracle.opt_apply) is fed the GPU's
    OWN gradient, moments and t; the GPU's new weights and moments must be close at 1e-5 (both
    precisions: the update runs on fp32 master weights), and the weight change itself must
    agree to 1e-3 of the largest change.
 3. Gradients, end to end: gradients are linear in clip(delta), delta = y - Q(s,a) being a
    difference of two quantities that each carry the Q tolerance, so in fp32 their bound is
    10 x rtol (Adam m: 10 x, v: 20 x); bf16: 2 x (m 2 x, v 4 x).  A wrong index, sign or operand
    in the backward pass is off by O(1), far outside either.
 4. Updated weights, end to end (GPU weights against the oracle's weights from the oracle's own
    gradient): close at rtol, for Adam plus a slack for the one ill-conditioned spot of the
    rule: where a gradient is no larger than its own tolerance d (item 3), Adam's quotient
    m^ / (sqrt(v^) + eps) can move by 2 d / (sqrt(v^) + eps), each factor contributing once, and by
    no more than 2 in any case, so the slack is 2 lr min(1, 2 d / (sqrt(v^) + eps)).  Item 2 is
    the check of the rule itself; this one only ties the two ends together.
 5. The ReLU derivative is a step function: where a hidden pre-activation lies within the
    rounding error of its own fp32 sum of zero (|z| <= 16 * 2^-24 * (sum_k |h_k w_k| + |b|)), the
    two sides may land on different sides of the kink, and that unit of that sample then enters
    the backward pass on one side only.  A unit of layer 1 can only change column j of dW1 and
    db1[j]; a unit k of layer 2 column k of dW2, db2[k] and (through dZ1) all of dW1, db1.  On an
    fp32 step whose gradients disagree AND whose forward pass (oracle side) has such a unit, the
    entries a kink can reach are left out and everything else (always dW3, db3; dW2, db2 except
    the kink's columns; dW1, db1 when only layer 1 has kinks) is compared as usual, as are the
    moments and weights of those entries.  Such steps are counted in Pair.kink_steps, and every
    test ends with the check that they stayed rare (at most 1 + compared steps / 100).
"""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
from paper_1801_03138_amd import synth

pytestmark = pytest.mark.gpu

F32_RTOL, BF16_RTOL = 1e-5, 2e-2


@pytest.fixture(scope="module")
def B():
    from paper_1801_03138_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return binding


_PAIRS = []


@pytest.fixture(autouse=True)
def _kink_budget():
    """Every test ends with the check that steps excused for a ReLU kink stayed rare."""
    _PAIRS.clear()
    yield
    for pr in _PAIRS:
        assert pr.kink_steps <= 1 + pr.compared // 100, (
            "ReLU kinks are rare: %d in %d compared steps is a backward bug" % (pr.kink_steps, pr.compared))
    _PAIRS.clear()


def assert_close(got, ref, rtol, what, slack=0.0):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    assert got.shape == ref.shape, what
    assert np.isfinite(got).all(), what
    scale = np.abs(ref).max() if ref.size else 0.0
    err = np.abs(got - ref)
    bound = rtol * np.maximum(np.abs(got), np.abs(ref)) + rtol * scale + slack
    worst = int(np.argmax(err - bound))
    assert (err <= bound).all(), (what, worst, got.ravel()[worst], ref.ravel()[worst], scale)


class Pair:
    """A GPU replay + trainer and the oracle ring it is compared with."""

    def __init__(self, B, *, capacity, D, H, A, batch, burn_in, seed, dtype="f32", loss="huber",
                 opt="adam", lr=1e-4, appends=1, use_graph=True, max_append=4096, layered=False,
                 target_sync=0, distinct=False, dueling=False, H2=0):
        self.B, self.D, self.H, self.A, self.batch, self.seed = B, D, H, A, batch, seed
        self.H2 = H2 or H                       # width of the second hidden layer
        self.bf16 = dtype == "bf16"
        self.target_sync = target_sync
        self.distinct = distinct
        sd = B.RP_BF16 if self.bf16 else B.RP_F32
        self.gpu_ring = B.Replay(capacity, D, sd, B.RP_PAIR, burn_in=burn_in, seed=seed,
                                 max_append=max_append, distinct=distinct)
        self.ref_ring = oracle.Ring(capacity, D, oracle.BF16 if self.bf16 else oracle.F32,
                                    oracle.PAIR, burn_in=burn_in)
        self.p0 = synth.init_params(D, H, A + (1 if dueling else 0), seed, hidden2=self.H2)
        f = np.float32
        self.hyper = dict(lr=f(lr), gamma=f(0.99), beta1=f(0.9), beta2=f(0.999), eps=f(1e-8))
        self.trainer = B.Trainer(self.gpu_ring, H, A, batch, param_dtype=sd,
                                 loss=B.RP_HUBER if loss == "huber" else B.RP_MSE,
                                 opt=B.RP_ADAM if opt == "adam" else B.RP_SGD,
                                 appends_per_step=appends, use_graph=use_graph, layered=layered,
                                 target_sync=target_sync, dueling=dueling, init_params=self.p0, hidden2=H2,
                                 **{k: float(v) for k, v in self.hyper.items()})
        self.cfg = oracle.make_cfg(D, H, A, batch,
                                   loss=oracle.HUBER if loss == "huber" else oracle.MSE,
                                   opt=oracle.ADAM if opt == "adam" else oracle.SGD,
                                   bf16=int(self.bf16), dueling=int(dueling), hidden2=H2,
                                   **{k: float(v) for k, v in self.hyper.items()})
        self.rtol = BF16_RTOL if self.bf16 else F32_RTOL
        self.kink_steps = 0
        self.compared = 0
        self.dueling = dueling
        _PAIRS.append(self)

    def kink_reach(self, p, S):
        """Boolean mask over the parameter vector: the gradient entries that a hidden unit lying
        within its fp32 rounding error of the ReLU kink (from parameters p on states S, float64)
        can change; None when there is no such unit."""
        D, H, G = self.D, self.H, self.H2
        O = self.A + (1 if self.dueling else 0)
        p = np.asarray(p, np.float64)
        W1, b1 = p[:D * H].reshape(D, H), p[D * H:D * H + H]
        o = D * H + H
        W2, b2 = p[o:o + H * G].reshape(H, G), p[o + H * G:o + H * G + G]
        u = 16.0 * 2.0 ** -24
        z1 = S @ W1 + b1
        k1 = (np.abs(z1) <= u * (np.abs(S) @ np.abs(W1) + np.abs(b1))).any(axis=0)
        h1 = np.maximum(z1, 0.0)
        z2 = h1 @ W2 + b2
        k2 = (np.abs(z2) <= u * (h1 @ np.abs(W2) + np.abs(b2))).any(axis=0)
        if not k1.any() and not k2.any():
            return None
        mW1, mb1 = np.zeros((D, H), bool), np.zeros(H, bool)
        mW2, mb2 = np.zeros((H, G), bool), np.zeros(G, bool)
        mW1[:, k1] = True
        mb1[k1] = True
        if k2.any():
            mW2[:, k2] = True
            mb2[k2] = True
            mW1[:], mb1[:] = True, True
        return np.concatenate([mW1.ravel(), mb1, mW2.ravel(), mb2, np.zeros(G * O + O, bool)])

    def append_only(self, part, device_src=True):
        self.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
        if device_src:
            d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda()
                 for k, v in part.items()}
            self.gpu_ring.append(d["s"], d["s_next"], d["a"], d["r"], d["term"])
            torch.cuda.synchronize()
        else:
            self.gpu_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])

    def states_f64(self, x):
        return (synth.bf16_bits_to_f32(x) if self.bf16 else x).astype(np.float64)

    def step(self, part, compare):
        """Append `part` on both sides and take one train step; returns the GPU status."""
        tr = self.trainer
        if compare:
            p, (m, v, t, step) = tr.params(), tr.opt_state()
            tgt = tr.target() if self.target_sync else None
        self.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
        status = tr.step(part["s"], part["s_next"], part["a"], part["r"], part["term"])
        if not compare:
            return status
        idx = self.ref_ring.sample(self.seed, step, self.batch, distinct=self.distinct)
        if idx is None:
            assert status == self.B.RP_SKIPPED_BURN_IN
            assert np.array_equal(tr.params(), p)
            return status
        assert status == 0
        s, sn, a, r, term = self.ref_ring.gather(idx)
        ref = oracle.train_step(self.cfg, p, m, v, t, self.states_f64(s), self.states_f64(sn), a,
                                r, term, target=tgt)
        last = tr.last()
        assert np.array_equal(last["idx"], idx)
        rt = self.rtol
        assert_close(last["Q"], ref.Q, rt, "Q(s,.)")
        assert_close(last["Qn"], ref.Qn, rt, "Q(s',.)")
        assert_close(last["y"], ref.y, rt, "targets")
        # delta = y - q is a difference of O(1) numbers: bound it on that scale
        assert np.abs(last["delta"] - ref.delta).max() <= 2 * rt * max(1.0, np.abs(ref.y).max(),
                                                                      np.abs(ref.Q).max())
        assert_close([last["loss"]], [ref.loss], rt, "loss")
        self.compared += 1
        g_got = tr.grads()
        new_p = tr.params()
        m2, v2, t2, step2 = tr.opt_state()
        assert step2 == step + 1
        # the update rule on the GPU's own gradient: no slack (item 2 of the module docstring)
        own_p, own_m, own_v, own_t = oracle.opt_apply(self.cfg, p, m, v, t, g_got)
        assert_close(new_p, own_p, F32_RTOL, "update rule applied to the GPU's own gradient")
        du = np.abs((new_p.astype(np.float64) - p) - (own_p - p.astype(np.float64)))
        assert (du <= 1e-3 * np.abs(own_p - p).max() + 2.0 ** -22 * np.abs(p)).all(), "weight change"
        if self.cfg.opt == oracle.ADAM:
            assert t2 == t + 1 == own_t
            assert_close(m2, own_m, F32_RTOL, "Adam m from the GPU's own gradient")
            assert_close(v2, own_v, F32_RTOL, "Adam v from the GPU's own gradient")
        # end to end against the oracle's own backward pass
        g_rt = 10 * rt if not self.bf16 else 2 * rt
        keep = slice(None)
        try:
            assert_close(g_got, ref.grads, g_rt, "gradients")
        except AssertionError:
            reach = None if self.bf16 else self.kink_reach(p, self.states_f64(s))
            if reach is None:
                raise
            # a hidden unit on the ReLU kink (item 5): what it can reach is left out
            self.kink_steps += 1
            keep = ~reach
            assert_close(g_got[keep], ref.grads[keep], g_rt, "gradients a ReLU kink cannot reach")
        slack = 0.0
        if self.cfg.opt == oracle.ADAM:
            d = g_rt * np.maximum(np.abs(g_got), np.abs(ref.grads)) + g_rt * np.abs(ref.grads).max()
            v_hat = np.asarray(ref.v, np.float64) / (1.0 - float(self.hyper["beta2"]) ** ref.t)
            lr, eps = float(self.hyper["lr"]), float(self.hyper["eps"])
            slack = (2.0 * lr * np.minimum(1.0, 2.0 * d / (np.sqrt(v_hat) + eps)))[keep]
        assert_close(new_p[keep], ref.params[keep], rt, "updated weights", slack)
        if self.target_sync:
            # the frozen copy is exactly the old one, or exactly the new weights when a sync is due
            want = oracle.target_after_step(tgt, new_p, t + 1, self.target_sync)
            assert np.array_equal(tr.target().astype(np.float64), want), "target network"
        if self.cfg.opt == oracle.ADAM:
            assert t2 == ref.t
            assert_close(m2[keep], ref.m[keep], 10 * rt if not self.bf16 else 2 * rt, "Adam m")
            assert_close(v2[keep], ref.v[keep], 20 * rt if not self.bf16 else 4 * rt, "Adam v")
        else:
            # the update itself, on its own scale
            assert_close((new_p.astype(np.float64) - p)[keep], (ref.params - p.astype(np.float64))[keep],
                         1e-3 if not self.bf16 else 4 * rt, "weight update")
        return status


@pytest.mark.parametrize("layered", [False, True])
def test_tiny_config_all_100_steps(B, layered):
    """Ring 1024, 27-64-64-8, batch 32, SGD 1e-3, burn-in 256, one append per step."""
    rows = synth.experiences(4096, 27, 8, 0.01, seed=0)
    pr = Pair(B, capacity=1024, D=27, H=64, A=8, batch=32, burn_in=256, seed=0, opt="sgd", lr=1e-3,
              layered=layered)
    assert pr.trainer.kernels_per_step() == (15 if layered else 2)
    executed = 0
    for k in range(4096):
        part = synth.take(rows, k, k + 1)
        if executed < 100:
            st = pr.step(part, compare=True)
            assert st == (B.RP_SKIPPED_BURN_IN if k + 1 < 256 else 0)
            executed += st == 0
        else:
            pr.append_only(part, device_src=False)
    assert executed == 100
    assert pr.gpu_ring.state() == pr.ref_ring.state() == (0, 1024, 4096)
    g, o = pr.gpu_ring.read_rows(0, 1024), pr.ref_ring.read(0, 1024)
    assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(g, o))


@pytest.mark.parametrize("layered", [False, True])
@pytest.mark.parametrize("loss,opt", [("huber", "adam"), ("mse", "sgd"), ("mse", "adam")])
def test_small_net_every_loss_and_optimizer(B, loss, opt, layered):
    """Batch 50 is not a multiple of the row kernel's four experiences per workgroup; a ring of
    128 with 3 appends per step makes sampled slots coincide with slots being overwritten."""
    rows = synth.experiences(300, 11, 5, 0.2, seed=4)
    pr = Pair(B, capacity=128, D=11, H=64, A=5, batch=50, burn_in=20, seed=9, loss=loss, opt=opt,
              lr=1e-3, appends=3, layered=layered)
    for k in range(0, 300, 3):
        pr.step(synth.take(rows, k, k + 3), compare=True)


@pytest.mark.parametrize("layered", [False, True])
def test_graph_and_direct_launch_agree_bitwise(B, layered):
    """200 steps in one call, which a trainer that records runs makes in those and one that does not
    kernel by kernel."""
    rows = synth.experiences(200, 27, 30, 0.05, seed=2)
    outs = []
    for use_graph in (True, False):
        pr = Pair(B, capacity=150, D=27, H=64, A=30, batch=64, burn_in=10, seed=3,
                  use_graph=use_graph, layered=layered)
        assert pr.trainer.steps(200, *(rows[k] for k in synth.FIELDS)) == 191
        for lo in (0, 100):
            part = synth.take(rows, lo, lo + 100)
            pr.ref_ring.append(*(part[k] for k in synth.FIELDS))
        outs.append((pr.trainer.params(), pr.trainer.last()["loss"], pr.trainer.opt_state()))
        assert pr.gpu_ring.state() == pr.ref_ring.state()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1] == outs[1][1]
    assert outs[0][2][2:] == outs[1][2][2:] == (191, 191)


def test_paper_shaped_config_sampled_steps(B):
    """Capacity 1e6, 27-256-256-30, batch 128, Adam 1e-4, burn-in 50,000, 10,000 steps."""
    rows = synth.experiences(60_000, 27, 30, 0.005, seed=0)
    pr = Pair(B, capacity=1_000_000, D=27, H=256, A=30, batch=128, burn_in=50_000, seed=0)
    pr.append_only(synth.take(rows, 0, 49_999))
    compared = {0, 1, 2, 10, 100, 1000, 9999}
    for k in range(10_000):
        st = pr.step(synth.take(rows, 49_999 + k, 50_000 + k), compare=k in compared)
        assert st == 0
    assert pr.trainer.opt_state()[2:] == (10_000, 10_000)
    assert pr.gpu_ring.state() == pr.ref_ring.state() == (59_999, 59_999, 59_999)
    assert pr.trainer.kernels_per_step() == 2
    # every streamed experience landed in its slot although thousands of steps were in flight
    g, o = pr.gpu_ring.read_rows(49_000, 10_999), pr.ref_ring.read(49_000, 10_999)
    assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(g, o))


def test_paper_network_at_paper_size(B):
    """The paper's own network (27-128-(512+512)-(1+30), dueling head, target network synced every
    10,000 updates) on the paper-shaped replay (capacity 1e6, batch 128, burn-in 50,000), the
    configuration the bench times: a compared step, 1,000 steps queued by one call (recorded runs),
    then two more compared steps; ring and counters exact."""
    rows = synth.experiences(52_000, 27, 30, 0.005, seed=0)
    pr = Pair(B, capacity=1_000_000, D=27, H=128, H2=1024, A=30, batch=128, burn_in=50_000, seed=0,
              dueling=True, target_sync=10_000)
    tr = pr.trainer
    pr.append_only(synth.take(rows, 0, 49_999))
    assert pr.step(synth.take(rows, 49_999, 50_000), compare=True) == 0
    new = synth.take(rows, 50_000, 51_000)
    d = {k: torch.from_numpy(x).cuda() for k, x in new.items()}
    assert tr.steps(1000, d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 1000
    pr.ref_ring.append(new["s"], new["s_next"], new["a"], new["r"], new["term"])
    for k in (51_000, 51_001):
        assert pr.step(synth.take(rows, k, k + 1), compare=True) == 0
    assert tr.opt_state()[2:] == (1003, 1003)
    assert pr.gpu_ring.state() == pr.ref_ring.state() == (51_002, 51_002, 51_002)
    assert tr.kernels_per_step() == 6


@pytest.mark.parametrize("dtype,layered,device_src", [("f32", False, True), ("f32", True, True),
                                                      ("bf16", False, True), ("f32", False, False),
                                                      ("bf16", False, False), ("f32", True, False)])
def test_many_steps_in_flight(B, dtype, layered, device_src):
    """train_steps with device or host arrays: 3000 steps queued without a sync, 2 appends each,
    into a ring that wraps; the ring must end up exactly as the oracle's and the counters must add
    up.  (Two-kernel fp32 step, layered step, and the MFMA step whose first kernel appends and
    gathers; host arrays travel through the ring of pinned slots, eight steps per graph launch.)"""
    n_steps, per = 3000, 2
    rows = synth.experiences(n_steps * per, 27, 30, 0.05, seed=21, state_dtype=dtype)
    pr = Pair(B, capacity=4096, D=27, H=64, A=30, batch=64, burn_in=100, seed=5, appends=per,
              layered=layered, dtype=dtype)
    d = rows
    if device_src:
        d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in rows.items()}
    done = pr.trainer.steps(n_steps, d["s"], d["s_next"], d["a"], d["r"], d["term"])
    for lo in range(0, n_steps * per, 4096):
        part = synth.take(rows, lo, min(lo + 4096, n_steps * per))
        pr.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
    assert done == n_steps - 49          # the first 49 steps end below the burn-in of 100
    assert pr.trainer.opt_state()[2:] == (done, done)
    assert pr.gpu_ring.state() == pr.ref_ring.state()
    g, o = pr.gpu_ring.read_rows(0, 4096), pr.ref_ring.read(0, 4096)
    assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(g, o))
    # and the next step still matches the oracle
    extra = synth.experiences(per, 27, 30, 0.05, seed=22, state_dtype=dtype)
    assert pr.step(extra, compare=True) == 0


@pytest.mark.parametrize("dtype,H,H2,layered,device_src", [
    ("f32", 64, 0, False, True), ("f32", 64, 0, False, False), ("bf16", 128, 0, False, True),
    ("f32", 64, 0, True, True), ("f32", 320, 0, False, True), ("f32", 320, 0, False, False),
    ("f32", 128, 1024, False, True), ("f32", 128, 1024, False, False),
    ("bf16", 128, 1024, False, True), ("bf16", 192, 64, False, False)])
def test_steps_in_flight_equal_steps_synchronised_one_by_one(B, dtype, H, H2, layered, device_src):
    """The argument block of the kernel that consumes a step's new experiences is rewritten in
    the recorded graph before every launch, while earlier launches of the same graph may still be
    running.  2,000 steps queued without any synchronisation (32 or 8 steps per graph launch) must
    leave exactly the state that the same 2,000 steps leave when the device is synchronised after
    every single step (launched kernel by kernel): ring, weights, moments, counters and the last
    step's sampled slots, bit for bit.  Two-kernel step (device and host arrays), MFMA step,
    layered step, fp32 MFMA step (whose recorded runs gather a step's batch in the launch of
    the step before it; device and host arrays), the paper's network with a dueling head on
    that step (where the same launch also holds the product dZ1), and two hidden widths with a
    dueling head in mixed precision."""
    # (the queued side makes the 2,000 steps in calls of these lengths, so that recorded runs of
    # every length, single steps and the hand-over from one run to the next all occur)
    n_steps, per = 2000, 2
    calls = [1, 2, 3, 5, 7, 13, 31, 33, 64, 70, 24, 56, 15]
    calls.append(n_steps - sum(calls))
    rows = synth.experiences(n_steps * per, 27, 30, 0.05, seed=51, state_dtype=dtype)
    outs = []
    for one_by_one in (False, True):
        pr = Pair(B, capacity=1500, D=27, H=H, H2=H2, A=30, batch=64, burn_in=100, seed=5, appends=per,
                  layered=layered, dtype=dtype, target_sync=9, dueling=H2 != 0)
        d = rows
        if device_src:
            d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda()
                 for k, v in rows.items()}
        tr = pr.trainer
        if one_by_one:
            done = 0
            for k in range(n_steps):
                lo, hi = k * per, (k + 1) * per
                done += tr.step(d["s"][lo:hi], d["s_next"][lo:hi], d["a"][lo:hi], d["r"][lo:hi],
                                d["term"][lo:hi]) == 0
                torch.cuda.synchronize()
        else:
            done, at = 0, 0
            for n in calls:
                lo, hi = at * per, (at + n) * per
                done += tr.steps(n, d["s"][lo:hi], d["s_next"][lo:hi], d["a"][lo:hi], d["r"][lo:hi],
                                 d["term"][lo:hi])
                at += n
        assert done == n_steps - 49
        last = tr.last()
        outs.append((tr.params(), tr.target(), tr.opt_state(), last["idx"], last["loss"], last["Q"],
                     pr.gpu_ring.state(), pr.gpu_ring.read_rows(0, 1500)))
    a, b = outs
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), "weights / target network"
    assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1]), "Adam moments"
    assert a[2][2:] == b[2][2:] == (n_steps - 49, n_steps - 49)
    assert np.array_equal(a[3], b[3]) and a[4] == b[4] and np.array_equal(a[5], b[5])
    assert a[6] == b[6]
    assert all(np.array_equal(x.view(np.uint8), y.view(np.uint8)) for x, y in zip(a[7], b[7]))


@pytest.mark.parametrize("H,layered,kernels", [(192, False, 2), (320, False, 7), (320, True, 15)])
def test_other_widths_agree_with_oracle(B, H, layered, kernels):
    """Widths that leave lanes idle in the row kernel (192) or exceed it (320: one MFMA product
    per kernel, or one plain kernel per layer, tiles with ragged edges); batch 130, ring that wraps."""
    rows = synth.experiences(900, 27, 30, 0.05, seed=12)
    pr = Pair(B, capacity=500, D=27, H=H, A=30, batch=130, burn_in=300, seed=4, appends=2,
              layered=layered)
    assert pr.trainer.kernels_per_step() == kernels
    for k in range(0, 900, 2):
        pr.step(synth.take(rows, k, k + 2), compare=(k % 50 == 0) or k >= 880)
    assert pr.gpu_ring.state() == pr.ref_ring.state()


@pytest.mark.parametrize("D,H,A,batch,target_sync,dueling", [
    (27, 256, 30, 513, 0, False), (60, 128, 9, 771, 0, False), (27, 64, 30, 600, 0, True),
    (27, 128, 30, 514, 4, False), (40, 256, 5, 512, 0, False)])
def test_batches_beyond_one_workgroup_per_compute_unit(B, D, H, A, batch, target_sync, dueling):
    """The row kernel takes two experiences per workgroup up to batch 512 and four beyond (and
    always four with a target network): batches on both sides of that limit, ragged against 2
    and against 4, on both widths of the first layer."""
    rows = synth.experiences(1400, D, A, 0.05, seed=41)
    pr = Pair(B, capacity=1200, D=D, H=H, A=A, batch=batch, burn_in=800, seed=9, appends=3,
              target_sync=target_sync, dueling=dueling)
    assert pr.trainer.kernels_per_step() == 2
    pr.append_only(synth.take(rows, 0, 1000))
    for k in range(8):
        assert pr.step(synth.take(rows, 1000 + 3 * k, 1003 + 3 * k), compare=True) == 0
    assert pr.gpu_ring.state() == pr.ref_ring.state()


def test_wide_state_and_action_sets(B):
    """D = 60 and A = 64 fill the row kernel's 64-wide limits; D = 70 takes one product per kernel."""
    for D, A, kernels in ((60, 64, 2), (70, 40, 7)):
        rows = synth.experiences(400, D, A, 0.05, seed=13)
        pr = Pair(B, capacity=300, D=D, H=128, A=A, batch=37, burn_in=50, seed=6, appends=1)
        assert pr.trainer.kernels_per_step() == kernels
        for k in range(400):
            pr.step(synth.take(rows, k, k + 1), compare=(k % 40 == 0) or k >= 395)


def test_terminal_rows_and_out_of_range_actions_are_safe(B):
    rows = synth.experiences(64, 27, 8, 1.0, seed=6)       # every experience terminal
    pr = Pair(B, capacity=64, D=27, H=64, A=8, batch=32, burn_in=64, seed=1, opt="sgd", lr=1e-3,
              appends=64)
    pr.step(rows, compare=True)
    last = pr.trainer.last()
    assert np.array_equal(last["y"], pr.ref_ring.gather(last["idx"])[3])


def test_mixed_precision_small(B):
    """bf16 matrix inputs, fp32 accumulation and master weights, on a net that spans several tiles."""
    rows = synth.experiences(600, 27, 30, 0.05, seed=7, state_dtype="bf16")
    pr = Pair(B, capacity=512, D=27, H=128, A=30, batch=200, burn_in=100, seed=2, dtype="bf16",
              appends=4)
    for k in range(0, 600, 4):
        pr.step(synth.take(rows, k, k + 4), compare=(k % 40 == 0) or k >= 560)


@pytest.mark.parametrize("D,H,A,batch", [(40, 64, 40, 7), (31, 192, 33, 130), (32, 64, 3, 513)])
def test_mixed_precision_other_shapes(B, D, H, A, batch):
    """Shapes off the tuned path of the MFMA step: states and action sets that need a second
    32-wide tile (and no spare column for the bias trick), a batch below one tile and batches
    that end inside a tile, a single 64-wide hidden tile."""
    rows = synth.experiences(400, D, A, 0.05, seed=17, state_dtype="bf16")
    pr = Pair(B, capacity=256, D=D, H=H, A=A, batch=batch, burn_in=100, seed=3, dtype="bf16",
              appends=2)
    assert pr.trainer.kernels_per_step() == 8
    for k in range(0, 400, 2):
        pr.step(synth.take(rows, k, k + 2), compare=(k % 60 == 0) or k >= 392)
    assert pr.gpu_ring.state() == pr.ref_ring.state()


def test_mixed_precision_layered_agrees(B):
    """The one-kernel-per-layer bf16 step stays available behind RP_TRAIN_LAYERED."""
    rows = synth.experiences(300, 27, 30, 0.05, seed=19, state_dtype="bf16")
    pr = Pair(B, capacity=256, D=27, H=128, A=30, batch=96, burn_in=100, seed=3, dtype="bf16",
              appends=2, layered=True)
    assert pr.trainer.kernels_per_step() == 15
    for k in range(0, 300, 2):
        pr.step(synth.take(rows, k, k + 2), compare=(k % 60 == 0) or k >= 292)


def test_wide_config_first_steps(B):
    """Capacity 4e6 (bf16 states), 27-1024-1024-30, batch 4096, 64 appends per step, Adam."""
    oracle.set_threads(16)
    try:
        rows = synth.experiences(200_000, 27, 30, 0.005, seed=0, state_dtype="bf16")
        pr = Pair(B, capacity=4_000_000, D=27, H=1024, A=30, batch=4096, burn_in=0, seed=0,
                  dtype="bf16", appends=64, max_append=64)
        pr.append_only(synth.take(rows, 0, 199_808))
        for k in range(3):
            lo = 199_808 + 64 * k
            assert pr.step(synth.take(rows, lo, lo + 64), compare=True) == 0
    finally:
        oracle.set_threads(1)


def test_burn_in_skips_training_but_appends(B):
    rows = synth.experiences(12, 5, 3, 0.1, seed=8)
    pr = Pair(B, capacity=16, D=5, H=64, A=3, batch=4, burn_in=10, seed=0, appends=2)
    for k in range(0, 12, 2):
        st = pr.step(synth.take(rows, k, k + 2), compare=True)
        assert st == (B.RP_SKIPPED_BURN_IN if k + 2 < 10 else 0)
    assert pr.trainer.opt_state()[2:] == (2, 2)


def test_trainer_rejects_bad_configurations(B):
    ring = B.Replay(64, 5)
    p = synth.init_params(5, 64, 3)
    with pytest.raises(B.ReplayError):
        B.Trainer(ring, 50, 3, 4, init_params=synth.init_params(5, 50, 3))      # hidden % 64
    with pytest.raises(B.ReplayError):
        B.Trainer(ring, 64, 3, 4, param_dtype=B.RP_BF16, init_params=p)        # dtype mismatch
    with pytest.raises(B.ReplayError):
        B.Trainer(ring, 64, 3, 4, appends_per_step=10**6, init_params=p)
    chain = B.Replay(64, 5, B.RP_F32, B.RP_CHAIN)
    with pytest.raises(B.ReplayError):
        B.Trainer(chain, 64, 3, 4, init_params=p)


@pytest.mark.parametrize("dtype,H,layered", [("f32", 64, False), ("f32", 320, False),
                                             ("bf16", 128, False), ("bf16", 128, True)])
def test_step_on_a_given_batch_matches_the_oracle(B, dtype, H, layered):
    """train_step_batch: the caller's batch instead of a sampled one, on each kind of step."""
    D, A, batch = 27, 30, 70
    rows = synth.experiences(batch, D, A, 0.1, seed=31, state_dtype=dtype)
    pr = Pair(B, capacity=64, D=D, H=H, A=A, batch=batch, burn_in=0, seed=1, dtype=dtype,
              appends=0, layered=layered)
    tr = pr.trainer
    d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda()
         for k, v in rows.items()}
    for k in range(3):
        p, (m, v, t, step) = tr.params(), tr.opt_state()
        assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
        ref = oracle.train_step(pr.cfg, p, m, v, t, pr.states_f64(rows["s"]),
                                pr.states_f64(rows["s_next"]), rows["a"], rows["r"], rows["term"])
        last = tr.last()
        assert np.array_equal(last["idx"], np.arange(batch))
        assert_close(last["Q"], ref.Q, pr.rtol, "Q(s,.)")
        assert_close(last["Qn"], ref.Qn, pr.rtol, "Q(s',.)")
        assert_close([last["loss"]], [ref.loss], pr.rtol, "loss")
        assert_close(tr.params(), ref.params, pr.rtol, "updated weights")
        assert tr.opt_state()[2:] == (t + 1, step + 1)
    assert pr.gpu_ring.state() == (0, 0, 0)


def test_in_ram_replay_trains_on_the_same_batches_as_the_device_replay(B):
    """The in-RAM comparison system (host sampling, host gather, per-step copy) and the
    device-resident replay draw the same slots and run the same step: identical weights."""
    D, H, A, batch, cap, burn = 27, 64, 30, 48, 300, 100
    rows = synth.experiences(700, D, A, 0.05, seed=41)
    p0 = synth.init_params(D, H, A, 5)
    ring = B.Replay(cap, D, burn_in=burn, seed=9)
    tr_dev = B.Trainer(ring, H, A, batch, appends_per_step=2, init_params=p0)
    done_dev = tr_dev.steps(350, rows["s"], rows["s_next"], rows["a"], rows["r"], rows["term"])
    # the in-RAM side needs a trainer only for the step itself: its replay stays empty
    idle = B.Replay(8, D, seed=9)
    tr_ram = B.Trainer(idle, H, A, batch, appends_per_step=0, init_params=p0)
    ram = B.InRamReplay(cap, D, batch, burn_in=burn, seed=9)
    done_ram = ram.train_steps(tr_ram, 350, 2, rows["s"], rows["s_next"], rows["a"], rows["r"],
                               rows["term"])
    torch.cuda.synchronize()
    assert done_dev == done_ram == 350 - 49
    assert ram.state() == (700 % cap, cap, 700, done_ram)
    assert np.array_equal(tr_dev.params(), tr_ram.params())
    assert tr_dev.last()["loss"] == tr_ram.last()["loss"]
    # and one more step of it against the oracle
    ref_ring = oracle.Ring(cap, D, burn_in=burn)
    for lo in range(0, 700, 100):
        part = synth.take(rows, lo, lo + 100)
        ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
    p, (m, v, t, _) = tr_ram.params(), tr_ram.opt_state()
    assert ram.train_step(tr_ram) == 0
    s, sn, a, r, term = ref_ring.gather(ref_ring.sample(9, done_ram, batch))
    cfg = oracle.make_cfg(D, H, A, batch, loss=oracle.HUBER, opt=oracle.ADAM,
                          lr=float(np.float32(1e-4)), gamma=float(np.float32(0.99)),
                          beta1=float(np.float32(0.9)), beta2=float(np.float32(0.999)),
                          eps=float(np.float32(1e-8)))
    ref = oracle.train_step(cfg, p, m, v, t, s, sn, a, r, term)
    assert_close(tr_ram.last()["Q"], ref.Q, F32_RTOL, "Q(s,.)")
    assert_close(tr_ram.params(), ref.params, F32_RTOL, "updated weights")


@pytest.mark.parametrize("dtype,H,batch,layered,kernels", [
    ("f32", 64, 50, False, 2), ("f32", 64, 50, True, 18), ("f32", 256, 128, False, 2),
    ("bf16", 128, 200, False, 11), ("bf16", 64, 256, False, 8), ("bf16", 128, 96, True, 18)])
def test_frozen_target_network(B, dtype, H, batch, layered, kernels):
    """Q(s', .) from a frozen copy of the weights, synced every 7th update (Deep Q-Network Model):
    the small fp32 step with the target's forward pass in workgroups of its own, the layered step, and the
    MFMA step with the S' rows in the same launches (batch 256) or in launches of their own
    (batch 200)."""
    rows = synth.experiences(400, 27, 30, 0.05, seed=23, state_dtype=dtype)
    pr = Pair(B, capacity=256, D=27, H=H, A=30, batch=batch, burn_in=100, seed=3, dtype=dtype,
              appends=2, layered=layered, target_sync=7, lr=1e-3)
    assert pr.trainer.kernels_per_step() == kernels
    assert np.array_equal(pr.trainer.target(), pr.trainer.params())
    synced = 0
    for k in range(0, 400, 2):
        before = pr.trainer.target()
        pr.step(synth.take(rows, k, k + 2), compare=(k % 10 == 0) or k >= 380)
        synced += not np.array_equal(before, pr.trainer.target())
    assert synced == (200 - 49) // 7
    # a target set by hand is used as it is
    other = synth.init_params(27, H, 30, 99)
    pr.trainer.set_target(other)
    assert np.array_equal(pr.trainer.target(), other)
    pr.step(synth.experiences(2, 27, 30, 0.05, seed=24, state_dtype=dtype), compare=True)


@pytest.mark.parametrize("D,H,A,batch,distinct,dueling", [
    (27, 256, 30, 128, False, False),    # the paper-shaped step
    (60, 128, 9, 1030, False, False),    # wide states, 258 threes of workgroups (more than compute units), ragged
    (27, 64, 30, 131, True, True),       # the extra workgroup that draws the next step's slots, ragged; dueling head
    (5, 192, 64, 3, False, False),       # two groups of workgroups, the second with one row; widest action set
])
def test_target_network_in_workgroups_of_its_own(B, D, H, A, batch, distinct, dueling):
    """Two-kernel step with a frozen target network: the states s' go through the target
    network in workgroups of their own, which pass max_a Q_target(s', a) to the workgroups that
    hold s (through a table filled a step ahead, or inside the same launch).  Q(s', .), targets,
    TD errors and the update against the oracle on every step, across several syncs; then a batch
    given by the caller."""
    rows = synth.experiences(1700, D, A, 0.1, seed=61)
    pr = Pair(B, capacity=1500, D=D, H=H, A=A, batch=batch, burn_in=1100, seed=13, appends=4,
              target_sync=3, distinct=distinct, dueling=dueling, lr=1e-3)
    assert pr.trainer.kernels_per_step() == 2
    pr.append_only(synth.take(rows, 0, 1200))
    for k in range(12):
        assert pr.step(synth.take(rows, 1200 + 4 * k, 1204 + 4 * k), compare=True) == 0
    assert pr.gpu_ring.state() == pr.ref_ring.state()
    tr = pr.trainer
    given = synth.experiences(batch, D, A, 0.1, seed=62)
    d = {k: torch.from_numpy(v).cuda() for k, v in given.items()}
    p, (m, v, t, step), tgt = tr.params(), tr.opt_state(), tr.target()
    assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
    ref = oracle.train_step(pr.cfg, p, m, v, t, pr.states_f64(given["s"]), pr.states_f64(given["s_next"]),
                            given["a"], given["r"], given["term"], target=tgt)
    last = tr.last()
    assert_close(last["Q"], ref.Q, pr.rtol, "Q(s,.)")
    assert_close(last["Qn"], ref.Qn, pr.rtol, "Q_target(s',.)")
    assert_close(last["y"], ref.y, pr.rtol, "targets")
    assert_close([last["loss"]], [ref.loss], pr.rtol, "loss")


@pytest.mark.parametrize("capacity", [5000, 70])
def test_target_values_computed_a_step_ahead(B, capacity):
    """Two-kernel step with a target network: workgroups of a step's launch send the NEXT step's
    sampled states s' through the target network and leave max_a Q_target(s', a) in a table; the
    next step takes them from there unless something changed in between.  Every step against the
    oracle, and for experience 0 of each step where its value came from: the table, except after
    a step that synced the target network, for a row that the step's own append wrote, after an
    append from outside, after train_set_target, after a step on a given batch, and on the first
    step.  With 70 slots for batches of 64 most groups of four mix both sources."""
    D, H, A, batch, per, sync = 27, 64, 30, 64, 2, 6
    rows = synth.experiences(400, D, A, 0.1, seed=81)
    pr = Pair(B, capacity=capacity, D=D, H=H, A=A, batch=batch, burn_in=64, seed=17, appends=per,
              target_sync=sync, lr=1e-3)
    tr = pr.trainer
    pr.append_only(synth.take(rows, 0, 64))
    at = [64]

    def step_and_source(expect_table):
        head = pr.gpu_ring.state()[0]
        assert pr.step(synth.take(rows, at[0], at[0] + per), compare=True) == 0
        at[0] += per
        slot0 = int(tr.last()["idx"][0])
        own_append = (slot0 - head) % capacity < per
        t_after = tr.opt_state()[2]
        assert tr.target_from_table() == (expect_table and not own_append), (at[0], slot0, head)
        return t_after % sync != 0       # whether the step after this one may use the table

    ok = step_and_source(False)                      # first step: nothing in the table
    for _ in range(20):                              # three syncs on the way
        ok = step_and_source(ok)
    pr.append_only(synth.take(rows, at[0], at[0] + 3)); at[0] += 3
    ok = step_and_source(False)                      # experiences added from outside
    ok = step_and_source(ok)
    tr.set_target(synth.init_params(D, H, A, 77))
    ok = step_and_source(False)                      # target network replaced from outside
    ok = step_and_source(ok)
    given = synth.experiences(batch, D, A, 0.1, seed=82)
    d = {k: torch.from_numpy(v).cuda() for k, v in given.items()}
    assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
    ok = step_and_source(False)                      # a step on a given batch in between
    for _ in range(8):
        ok = step_and_source(ok)
    assert pr.gpu_ring.state() == pr.ref_ring.state()


@pytest.mark.parametrize("seed,distinct,dueling,cap,per", [
    (1, False, False, 90, 3), (2, False, True, 90, 3), (3, True, False, 90, 3),
    (4, False, False, 50, 30)])    # a ring shorter than two appends: the next append laps into this one's rows
def test_target_network_under_a_random_sequence_of_calls(B, seed, distinct, dueling, cap, per):
    """Whatever happens between two train steps, the step after it must use the target network
    and the rows as they are then: a seeded random sequence of train steps, steps on given
    batches, appends from outside, new target networks, rewound counters and runs of steps
    queued without a synchronisation, every compared step against the oracle (ring of 90
    slots, batch 37: ragged groups, rows that the steps' own appends overwrite)."""
    D, H, A, batch = 27, 64, 30, 37
    rng = np.random.default_rng(1000 + seed)
    rows = synth.experiences(12000, D, A, 0.1, seed=90 + seed)
    pr = Pair(B, capacity=cap, D=D, H=H, A=A, batch=batch, burn_in=40, seed=seed, appends=per,
              target_sync=int(rng.choice([2, 4, 7])), distinct=distinct, dueling=dueling, lr=1e-3)
    tr = pr.trainer
    at = [0]

    def take(n):
        part = synth.take(rows, at[0], at[0] + n)
        at[0] += n
        return part

    pr.append_only(take(min(60, cap)))
    for _ in range(70):
        op = rng.choice(["step", "step", "step", "batch", "append", "target", "rewind", "run"])
        if op == "step":
            assert pr.step(take(per), compare=True) == 0
        elif op == "batch":
            given = synth.experiences(batch, D, A, 0.1, seed=int(rng.integers(1 << 30)))
            d = {k: torch.from_numpy(v).cuda() for k, v in given.items()}
            assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
        elif op == "append":
            pr.append_only(take(int(rng.integers(1, 8))))
        elif op == "target":
            tr.set_target(synth.init_params(D, H, A + (1 if dueling else 0), int(rng.integers(1 << 30))))
        elif op == "rewind":
            p, (m, v, t, step) = tr.params(), tr.opt_state()
            tr.set_state(p, m, v, max(0, t - int(rng.integers(0, 3))), step + int(rng.integers(0, 3)))
        else:
            n = int(rng.integers(2, 12))
            part = take(n * per)
            for j in range(n):
                one = synth.take(part, j * per, (j + 1) * per)
                pr.ref_ring.append(one["s"], one["s_next"], one["a"], one["r"], one["term"])
            assert tr.steps(n, part["s"], part["s_next"], part["a"], part["r"], part["term"]) == n
    assert pr.step(take(per), compare=True) == 0
    assert pr.gpu_ring.state() == pr.ref_ring.state()


def test_a_hand_over_that_never_arrives_ends_the_wait_and_is_reported(B):
    """The wait of a workgroup for its partner is bounded.  With the waiting side told to look for
    a launch number that nobody sends (a host-side switch: every kernel still runs to its end)
    and a limit of 20 microseconds, the steps finish, the read-back calls report RP_ESTATE, and
    after train_set_state and with the pairing restored the trainer agrees with the oracle again."""
    rows = synth.experiences(400, 27, 30, 0.1, seed=71)
    pr = Pair(B, capacity=300, D=27, H=64, A=30, batch=50, burn_in=100, seed=2, appends=2, target_sync=5)
    tr = pr.trainer
    pr.append_only(synth.take(rows, 0, 200))
    assert pr.step(synth.take(rows, 200, 202), compare=True) == 0
    p, (m, v, t, step) = tr.params(), tr.opt_state()
    tr.set_handoff_wait(ticks=2000, break_pairing=True)
    d = {k: torch.from_numpy(x).cuda() for k, x in synth.take(rows, 202, 210).items()}
    assert tr.steps(4, d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 4
    torch.cuda.synchronize()
    with pytest.raises(B.ReplayError) as err:
        tr.last()
    assert err.value.status == B.RP_ESTATE and "hand-over" in str(err.value)
    with pytest.raises(B.ReplayError):
        tr.opt_state()
    # back to a known state (the ring took the eight rows; the oracle's ring follows)
    part = synth.take(rows, 202, 210)
    pr.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
    tr.set_handoff_wait(ticks=0, break_pairing=False)
    tr.set_state(p, m, v, t, step + 4)
    tr.last()
    for k in range(210, 230, 2):
        assert pr.step(synth.take(rows, k, k + 2), compare=True) == 0


@pytest.mark.parametrize("dtype,H,layered", [("f32", 64, False), ("f32", 64, True), ("bf16", 128, False),
                                             ("f32", 320, False)])
def test_train_step_with_batches_without_duplicates(B, dtype, H, layered):
    """RP_DISTINCT replay under each kind of train step (two-kernel, layered, MFMA mixed precision,
    fp32 MFMA: the last two draw inside their append + gather kernel, one lane per row or, with
    sixteen lanes per row, as a team); with burn-in 10 and batch 40 the first steps are refused
    until 40 experiences are held."""
    rows = synth.experiences(300, 27, 30, 0.05, seed=29, state_dtype=dtype)
    pr = Pair(B, capacity=128, D=27, H=H, A=30, batch=40, burn_in=10, seed=8, dtype=dtype,
              appends=2, layered=layered, distinct=True)
    executed = 0
    for k in range(0, 300, 2):
        st = pr.step(synth.take(rows, k, k + 2), compare=(k % 20 == 0) or k >= 290)
        assert st == (B.RP_SKIPPED_BURN_IN if k + 2 < 40 else 0)
        executed += st == 0
        if st == 0:
            assert len(set(pr.trainer.last()["idx"].tolist())) == 40 or k % 20
    assert executed == 150 - 19
    assert pr.gpu_ring.state() == pr.ref_ring.state()


def test_without_duplicates_slots_drawn_ahead(B):
    """The two-kernel step draws the next step's slots while a step runs, for the ring size the
    next step is expected to see.  Whatever happens between two steps, the slots are those of
    the step's own (seed, step, size): consecutive steps (drawn ahead), appends from outside
    between steps while the ring fills (size differs from the expected one: drawn again), steps
    in a full ring, and a step after one that was refused."""
    rows = synth.experiences(700, 27, 30, 0.05, seed=31)
    pr = Pair(B, capacity=256, D=27, H=64, A=30, batch=48, burn_in=10, seed=12, appends=1,
              distinct=True)
    at = 0
    for k in range(40):                      # refused until 48 experiences are held
        assert pr.step(synth.take(rows, at, at + 1), compare=True) == B.RP_SKIPPED_BURN_IN
        at += 1
    pr.append_only(synth.take(rows, at, at + 20)); at += 20
    for k in range(60):
        assert pr.step(synth.take(rows, at, at + 1), compare=True) == 0
        at += 1
        if k % 7 == 3 and k < 40:            # the ring grows behind the trainer's back
            n = 1 + k % 5
            pr.append_only(synth.take(rows, at, at + n), device_src=bool(k % 2)); at += n
    for n in (200, 100):                                          # full, wrapped
        pr.append_only(synth.take(rows, at, at + n)); at += n
    for k in range(20):
        assert pr.step(synth.take(rows, at, at + 1), compare=True) == 0
        at += 1
        assert len(set(pr.trainer.last()["idx"].tolist())) == 48
    assert pr.gpu_ring.state() == pr.ref_ring.state()


@pytest.mark.parametrize("dtype,H,batch,layered,target_sync,kernels,A", [
    ("f32", 64, 50, False, 0, 2, 30), ("f32", 64, 50, True, 0, 16, 30), ("f32", 128, 33, False, 5, 2, 30),
    ("f32", 128, 33, True, 5, 19, 30),
    ("f32", 256, 130, False, 3, 2, 32), ("f32", 64, 7, False, 0, 2, 2), ("f32", 128, 64, False, 4, 2, 5),
    ("f32", 64, 50, False, 0, 3, 40), ("f32", 128, 33, False, 5, 3, 64),
    ("bf16", 128, 200, False, 0, 9, 30), ("bf16", 64, 256, False, 5, 9, 30),
    ("bf16", 128, 96, True, 0, 16, 30)])
def test_dueling_head(B, dtype, H, batch, layered, target_sync, kernels, A):
    """Q = V + A - mean A with a value stream and an advantage stream (Deep Q-Network Model), on
    every kind of step, alone and together with the frozen target network.  In the two-kernel
    step the weights kernel itself updates a head of up to 32 actions; wider heads get a kernel
    of their own."""
    rows = synth.experiences(300, 27, A, 0.05, seed=37, state_dtype=dtype)
    pr = Pair(B, capacity=256, D=27, H=H, A=A, batch=batch, burn_in=60, seed=6, dtype=dtype,
              appends=2, layered=layered, target_sync=target_sync, dueling=True, lr=1e-3)
    assert pr.trainer.kernels_per_step() == kernels
    assert len(pr.trainer.params()) == 27 * H + H + H * H + H + H * (A + 1) + A + 1
    for k in range(0, 300, 2):
        pr.step(synth.take(rows, k, k + 2), compare=(k % 20 == 0) or k >= 290)
    # weights between the two streams never move, and the mean over actions of Q is the value V
    p0, p1 = pr.p0, pr.trainer.params()
    oW3 = 27 * H + H + H * H + H
    W3a, W3b = (x[oW3:oW3 + H * (A + 1)].reshape(H, A + 1) for x in (p0, p1))
    assert np.array_equal(W3a[H // 2:, 0], W3b[H // 2:, 0]) and np.array_equal(W3a[:H // 2, 1:], W3b[:H // 2, 1:])
    assert not np.array_equal(W3a[:H // 2, 0], W3b[:H // 2, 0])


@pytest.mark.parametrize("D,H,H2,A,batch,target_sync,dueling,opt,loss,kernels", [
    (27, 128, 1024, 30, 128, 6, True, "adam", "huber", 6),     # the paper's network
    (27, 128, 1024, 30, 130, 4, True, "adam", "huber", 6),     # ... on a batch that ends inside a tile
    (27, 128, 512, 30, 64, 0, False, "sgd", "mse", 6),
    (50, 128, 192, 6, 40, 0, False, "adam", "mse", 6),          # 64 padded inputs into 128 units
    (40, 64, 512, 30, 77, 3, False, "adam", "huber", 6),       # 64 inputs after padding, first layer of 64
    (27, 64, 192, 40, 33, 3, True, "adam", "mse", 7),          # head wider than one tile: a kernel of its own
    (27, 128, 512, 40, 48, 3, True, "adam", "huber", 7),       # ... after the launch that holds the dZ1 product
    (70, 320, 64, 5, 50, 0, False, "adam", "huber", 7),
    (27, 512, 512, 30, 256, 5, False, "adam", "huber", 7),
    (9, 1024, 128, 3, 17, 0, True, "sgd", "huber", 7),
])
def test_two_hidden_widths_on_mfma(B, D, H, H2, A, batch, target_sync, dueling, opt, loss, kernels):
    """fp32 networks the two-kernel step does not take, one MFMA product per kernel: two hidden
    layers of different widths, foremost the paper's own network (Deep Q-Network Model: shared
    layer 128, value and advantage stream 512 each, i.e. 27-128-1024-(1+30), frozen target
    network), wide layers, wide states, K splits (contractions of 256 and more) and ragged batches."""
    rows = synth.experiences(700, D, A, 0.05, seed=61)
    pr = Pair(B, capacity=400, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=300, seed=7, appends=2,
              target_sync=target_sync, dueling=dueling, opt=opt, loss=loss, lr=1e-3)
    assert pr.trainer.kernels_per_step() == kernels
    n_params = D * H + H + H * H2 + H2 + H2 * (A + dueling) + A + dueling
    assert len(pr.trainer.params()) == n_params
    for lo in (0, 250):                       # 500 experiences into 400 slots: the ring wraps
        pr.append_only(synth.take(rows, lo, lo + 250))
    for k in range(500, 700, 2):
        assert pr.step(synth.take(rows, k, k + 2), compare=(k % 20 == 0) or k >= 690) == 0
    assert pr.gpu_ring.state() == pr.ref_ring.state()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_two_hidden_widths_layer_by_layer(B, dtype):
    """The plain one-kernel-per-layer step, behind RP_TRAIN_LAYERED, takes two widths as well."""
    rows = synth.experiences(300, 27, 30, 0.05, seed=62, state_dtype=dtype)
    pr = Pair(B, capacity=256, D=27, H=64, H2=128, A=30, batch=40, burn_in=100, seed=3, dtype=dtype,
              appends=2, layered=True, target_sync=5, dueling=True, lr=1e-3)
    assert pr.trainer.kernels_per_step() == 19
    for k in range(0, 300, 2):
        pr.step(synth.take(rows, k, k + 2), compare=(k % 30 == 0) or k >= 290)


def test_paper_network_step_on_a_given_batch_and_without_appends(B):
    """The paper's network with no new experiences per step (sample and gather in a kernel of
    their own) and on a caller-provided batch."""
    D, H, H2, A, batch = 27, 128, 1024, 30, 70
    rows = synth.experiences(400, D, A, 0.1, seed=63)
    pr = Pair(B, capacity=300, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=0, seed=1, appends=0,
              dueling=True, target_sync=2, lr=1e-3)
    assert pr.trainer.kernels_per_step() == 6
    pr.append_only(synth.take(rows, 0, 300))
    empty = synth.take(rows, 0, 0)
    for k in range(4):
        assert pr.step(empty, compare=True) == 0
    tr = pr.trainer
    d = {k: torch.from_numpy(v).cuda() for k, v in synth.take(rows, 300, 300 + batch).items()}
    part = synth.take(rows, 300, 300 + batch)
    for k in range(3):
        p, (m, v, t, step), tgt = tr.params(), tr.opt_state(), tr.target()
        assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
        ref = oracle.train_step(pr.cfg, p, m, v, t, part["s"].astype(np.float64),
                                part["s_next"].astype(np.float64), part["a"], part["r"], part["term"],
                                target=tgt)
        last = tr.last()
        assert_close(last["Q"], ref.Q, pr.rtol, "Q(s,.)")
        assert_close(last["Qn"], ref.Qn, pr.rtol, "Q(s',.)")
        assert_close([last["loss"]], [ref.loss], pr.rtol, "loss")
        own_p, _, _, _ = oracle.opt_apply(pr.cfg, p, m, v, t, tr.grads())
        assert_close(tr.params(), own_p, F32_RTOL, "update rule applied to the GPU's own gradient")
        assert_close(tr.grads(), ref.grads, 10 * pr.rtol, "gradients")


def _random_configs(n, seed, two_widths_bf16=False):
    """Seeded draw of step configurations: every kind of step (two-kernel fp32, MFMA mixed
    precision, layered), shapes on and off the tile sizes, both losses and optimizers, with and
    without the frozen target network, the dueling head and batches without duplicates."""
    rng = np.random.default_rng(seed)
    out = []
    for k in range(n):
        dtype = "bf16" if rng.random() < 0.4 else "f32"
        H = int(rng.choice([64, 128, 192, 256, 320]))
        if dtype == "bf16":
            H = int(rng.choice([64, 128, 192]))
        if two_widths_bf16:
            dtype, H = "bf16", int(rng.choice([64, 128, 192]))
        H2 = int(rng.choice([0, 0, 64, 128, 320])) if dtype == "f32" else 0
        if two_widths_bf16:
            H2 = int(rng.choice([w for w in (64, 128, 320) if w != H]))
        D = int(rng.integers(1, 70))
        A = int(rng.integers(1, 70))
        batch = int(rng.choice([1, 2, 5, 31, 64, 100, 128, 129, 257]))
        appends = int(rng.choice([0, 1, 3, 17]))
        capacity = int(rng.choice([300, 512, 1000]))
        distinct = bool(rng.random() < 0.3) and batch <= 128
        out.append(dict(dtype=dtype, H=H, H2=H2, D=D, A=A, batch=batch, appends=appends, capacity=capacity,
                        loss=str(rng.choice(["huber", "mse"])), opt=str(rng.choice(["adam", "sgd"])),
                        layered=bool(rng.random() < 0.25), target_sync=int(rng.choice([0, 0, 3])),
                        dueling=bool(rng.random() < 0.3) and A >= 2, distinct=distinct,
                        seed=int(rng.integers(0, 1000))))
    return out


@pytest.mark.parametrize("c", _random_configs(64, 20261127) + _random_configs(16, 20261204, True), ids=lambda c: "-".join(
    "%s" % c[k] for k in ("dtype", "D", "H", "H2", "A", "batch", "appends", "opt", "loss")))
def test_random_configurations(B, c):
    """Twelve teacher-forced steps of a randomly drawn configuration, after a prefill that wraps
    the ring when the capacity is small; and the same twelve made by one call on a second trainer, in
    recorded runs, which must leave the same bits behind."""
    n_pre, steps, per = c["capacity"] + 57, 12, c["appends"]
    rows = synth.experiences(n_pre + steps * max(1, per), c["D"], c["A"], 0.05, seed=c["seed"], state_dtype=c["dtype"])
    ends = []
    for one_call in (False, True):
        pr = Pair(B, capacity=c["capacity"], D=c["D"], H=c["H"], H2=c["H2"], A=c["A"], batch=c["batch"], burn_in=40,
                  seed=c["seed"], dtype=c["dtype"], loss=c["loss"], opt=c["opt"], lr=1e-3,
                  appends=per, layered=c["layered"], target_sync=c["target_sync"],
                  distinct=c["distinct"], dueling=c["dueling"])
        for lo in range(0, n_pre, 200):
            pr.append_only(synth.take(rows, lo, min(lo + 200, n_pre)))
        if one_call:
            new = synth.take(rows, n_pre, n_pre + steps * per)
            assert pr.trainer.steps(steps, *(new[k] for k in synth.FIELDS)) == steps
        else:
            for at in range(n_pre, n_pre + steps * per, per) if per else [n_pre] * steps:
                assert pr.step(synth.take(rows, at, at + per), compare=True) == 0
        tr = pr.trainer
        last, (m, v, t, step) = tr.last(), tr.opt_state()
        ends.append([tr.params(), tr.grads(), tr.target(), m, v, last["Q"], last["Qn"], last["y"], last["idx"],
                     np.array([t, step]), np.array([last["loss"]]), np.array(pr.gpu_ring.state()),
                     *pr.gpu_ring.read_rows(0, c["capacity"])])
    for k, (a, b) in enumerate(zip(*ends)):
        assert np.array_equal(a, b), k


def test_paper_network_free_running_through_recorded_runs(B, capsys):
    """The paper's network (27-128-(512+512)-(1+30), dueling head, target network synced every 20
    updates) for 50 consecutive steps made by ONE train_steps call, i.e. in recorded runs of 32,
    16 and 2 steps, whose steps gather the next step's batch in their own launches: no teacher
    forcing, the oracle (fp64) carries its own weights, moments and target network from the same
    start.  Sampled slots of the last step, step counts and the sync schedule must agree exactly,
    the weights and the target network within a loose drift bound (see the test below)."""
    D, H, H2, A, batch, n_steps, sync = 27, 128, 1024, 30, 128, 50, 20
    oracle.set_threads(16)
    try:
        rows = synth.experiences(2000 + n_steps, D, A, 0.01, seed=5)
        pr = Pair(B, capacity=4096, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1000, seed=3,
                  target_sync=sync, dueling=True, lr=1e-4)
        pr.append_only(synth.take(rows, 0, 2000))
        tr = pr.trainer
        assert tr.kernels_per_step() == 6
        p = tr.params().astype(np.float64)
        tgt = tr.target().astype(np.float64)
        m, v, t, step = tr.opt_state()
        m, v = np.asarray(m, np.float64), np.asarray(v, np.float64)
        new = synth.take(rows, 2000, 2000 + n_steps)
        d = {k: torch.from_numpy(x).cuda() for k, x in new.items()}
        assert tr.steps(n_steps, d["s"], d["s_next"], d["a"], d["r"], d["term"]) == n_steps
        for k in range(n_steps):
            part = synth.take(rows, 2000 + k, 2001 + k)
            pr.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
            idx = pr.ref_ring.sample(pr.seed, step + k, batch)
            s_, sn_, a_, r_, term_ = pr.ref_ring.gather(idx)
            ref = oracle.train_step(pr.cfg, p, m, v, t + k, s_.astype(np.float64), sn_.astype(np.float64),
                                    a_, r_, term_, target=tgt)
            p, m, v = ref.params, ref.m, ref.v
            tgt = oracle.target_after_step(tgt, p, t + k + 1, sync)
        assert pr.gpu_ring.state() == pr.ref_ring.state()
        assert np.array_equal(tr.last()["idx"], idx)
        assert tr.opt_state()[2:] == (t + n_steps, step + n_steps)
        scale = np.abs(p).max()
        drift = float(np.abs(tr.params().astype(np.float64) - p).max() / scale)
        drift_t = float(np.abs(tr.target().astype(np.float64) - tgt).max() / scale)
        with capsys.disabled():
            print("\npaper network, 50 free-running steps in recorded runs: max |w_gpu - w_oracle| / max |w| = "
                  "%.2e (target network %.2e)" % (drift, drift_t))
        assert drift <= 1e-4 and drift_t <= 1e-4
        # the target network is the weights as they were after update 40, not the current ones
        assert np.abs(tr.target() - tr.params()).max() > 0
    finally:
        oracle.set_threads(1)


def test_paper_shaped_free_running_drift(B, capsys):
    """100 consecutive steps with no teacher forcing: the GPU (fp32) and the oracle (fp64) each
    carry their own weights and Adam moments from the same start.  The drift of the weights is
    reported; it is only loosely bounded, because a ReLU or an argmax that switches on one side
    first makes the two trajectories part for good (beyond a few hundred steps nothing is pinned)."""
    oracle.set_threads(16)
    try:
        rows = synth.experiences(50_200, 27, 30, 0.005, seed=0)
        pr = Pair(B, capacity=1_000_000, D=27, H=256, A=30, batch=128, burn_in=50_000, seed=0)
        pr.append_only(synth.take(rows, 0, 49_999))
        tr = pr.trainer
        p = tr.params().astype(np.float64)
        m, v, t, step = tr.opt_state()
        m, v = np.asarray(m, np.float64), np.asarray(v, np.float64)
        curve = {}
        for k in range(100):
            part = synth.take(rows, 49_999 + k, 50_000 + k)
            pr.ref_ring.append(part["s"], part["s_next"], part["a"], part["r"], part["term"])
            assert tr.step(part["s"], part["s_next"], part["a"], part["r"], part["term"]) == 0
            idx = pr.ref_ring.sample(pr.seed, step + k, pr.batch)
            s, sn, a, r, term = pr.ref_ring.gather(idx)
            ref = oracle.train_step(pr.cfg, p, m, v, t + k, s.astype(np.float64), sn.astype(np.float64),
                                    a, r, term)
            p, m, v = ref.params, ref.m, ref.v
            if k + 1 in (1, 2, 5, 10, 20, 50, 100):
                got = tr.params().astype(np.float64)
                curve[k + 1] = float(np.abs(got - p).max() / np.abs(p).max())
        with capsys.disabled():
            print("\nfree-running drift, max |w_gpu - w_oracle| / max |w|: " +
                  ", ".join("step %d: %.2e" % kv for kv in curve.items()))
        assert curve[1] <= 2e-5
        assert curve[100] <= 1e-2
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("D,H,H2,A,batch,target_sync,dueling", [
    # weight-gradient tiles: the batch's steps of four rows over eight wavefronts, T in flight
    (27, 64, 0, 8, 1, 0, False), (27, 64, 0, 8, 3, 0, True), (27, 64, 0, 8, 33, 0, False),
    (27, 64, 0, 8, 64, 0, True), (27, 64, 0, 30, 65, 0, False),
    (27, 64, 0, 30, 127, 0, True), (27, 64, 0, 30, 129, 0, False), (27, 64, 0, 30, 255, 3, True),
    (27, 64, 0, 30, 257, 0, False), (27, 64, 0, 30, 514, 0, True),
    # products in 32 x 32 tiles: K of 2, 4, 12, 18 and 36 groups of 16 over four and eight wavefronts,
    # rows that end inside a tile, two parts, the dZ1 product in tiles of its own
    (40, 512, 576, 40, 520, 2, False), (27, 192, 1024, 30, 150, 0, True), (33, 256, 320, 5, 401, 3, False),
    # ... of 2 groups, of 4 and of 6, in all three products
    (27, 1024, 64, 30, 70, 0, False), (60, 256, 64, 8, 33, 3, True), (90, 512, 64, 5, 45, 0, False),
])
def test_fp32_tile_edges(B, D, H, H2, A, batch, target_sync, dueling):
    """The fp32 steps' tiled kernels where a batch, a contraction or a launch ends inside a tile or a
    round of loads; tolerances of the other fp32 cases (the sums are fp32, in another order)."""
    rows = synth.experiences(batch + 120, D, A, 0.05, seed=71)
    pr = Pair(B, capacity=batch + 60, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, appends=3,
              target_sync=target_sync, dueling=dueling, lr=1e-3)
    for lo in (0, batch + 60):                # more than the ring holds: it wraps
        pr.append_only(synth.take(rows, lo, min(lo + batch + 60, batch + 90)))
    for k in range(batch + 90, batch + 120, 3):
        assert pr.step(synth.take(rows, k, k + 3), compare=(k % 2 == 0) or k >= batch + 114) == 0


@pytest.mark.parametrize("D,H,H2,A,batch,target_sync,dueling,opt", [
    (27, 128, 1024, 30, 130, 4, True, "adam"),      # the paper's network, a batch that ends inside a tile
    (27, 128, 1024, 30, 512, 4, True, "adam"),      # ... both networks' rows in one launch
    (40, 64, 192, 40, 65, 0, False, "sgd"),         # a second block of 32 actions
    (9, 256, 64, 3, 64, 3, False, "adam"),          # second layer the narrower
    (27, 64, 256, 30, 5, 3, True, "adam"),          # batches below 64
    (27, 64, 128, 30, 40, 5, True, "adam"),
    (27, 128, 64, 30, 63, 0, False, "adam"),
    (70, 320, 448, 70, 200, 3, True, "adam"),       # stripes of each layer beyond the other, wide states
])
def test_two_hidden_widths_mixed_precision_on_mfma(B, D, H, H2, A, batch, target_sync, dueling, opt):
    """Mixed precision with two hidden widths in the step of one width's networks; tolerances of the
    other mixed-precision cases."""
    rows = synth.experiences(batch + 150, D, A, 0.05, seed=72, state_dtype="bf16")
    pr = Pair(B, capacity=batch + 60, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, dtype="bf16",
              appends=3, target_sync=target_sync, dueling=dueling, opt=opt, lr=1e-3)
    assert pr.trainer.kernels_per_step() == (8 if batch % 128 == 0 or not target_sync else 11) + dueling
    for lo in (0, batch + 60):                # more than the ring holds: it wraps
        pr.append_only(synth.take(rows, lo, min(lo + batch + 60, batch + 90)))
    for k in range(batch + 90, batch + 150, 3):
        assert pr.step(synth.take(rows, k, k + 3), compare=(k % 2 == 0) or k >= batch + 140) == 0


@pytest.mark.parametrize("H,H2,batch,kernels", [(64, 128, 64, 8), (128, 512, 1024, 5)])
def test_output_gradient_keeps_fp32_in_mixed_precision(B, H, H2, batch, kernels):
    """The output layer's gradient in mixed precision contracts bf16 activations with dL/dQ in fp32: three
    bf16 parts that add up to it exactly.  Weights and states are small whole numbers here, so that the
    activations are exact in bf16, and as many experiences as there are actions have one of their own each
    (the others have TD errors and activations of zero), so that an entry of dW3 (and of db3) is one
    product: the sum of three exact ones, two roundings at most.  Two parts, without the last one, miss
    that bound by far in either array."""
    D, A = 27, 64
    rng = np.random.default_rng(73)
    W1 = rng.integers(-1, 2, (D, H)).astype(np.float32)
    W2 = np.zeros((H, H2), np.float32)
    for k in range(H2):
        W2[rng.choice(H, 3, replace=False), k] = rng.choice([-1, 1], 3)
    W3 = rng.standard_normal((H2, A)).astype(np.float32)
    p0 = np.concatenate([W1.ravel(), np.zeros(H), W2.ravel(), np.zeros(H2), W3.ravel(), np.zeros(A)]).astype(np.float32)
    s = rng.integers(0, 4, (batch, D)).astype(np.float32)
    h1 = np.maximum(s @ W1, 0)
    h2 = np.maximum(h1 @ W2, 0).astype(np.float64)
    assert h1.max() <= 256 and h2.max() <= 256          # whole numbers that bf16 holds
    rows = synth.experiences(batch, D, A, 0.05, seed=73, state_dtype="bf16")
    rows["s"], rows["a"] = synth.f32_to_bf16_bits(s), rng.permutation(batch).astype(np.int32) % A
    own = np.sort(rng.choice(batch, A, replace=False))  # (spread over the batch: its chunks, halves and lanes)
    if batch > A:
        own[-1] = batch - 1
        rows["a"][own] = rng.permutation(A)
        rest = np.setdiff1d(np.arange(batch), own)
        rows["s"][rest], rows["r"][rest], rows["term"][rest], h2[rest] = 0, 0, 1, 0
    ring = B.Replay(64, D, B.RP_BF16, seed=5)
    tr = B.Trainer(ring, H, A, batch, param_dtype=B.RP_BF16, loss=B.RP_MSE, opt=B.RP_SGD, appends_per_step=0, lr=1e-3,
                   init_params=p0, hidden2=H2)
    d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in rows.items()}
    assert tr.kernels_per_step() == kernels
    assert tr.step_batch(d["s"], d["s_next"], d["a"], d["r"], d["term"]) == 0
    g = -tr.last()["delta"] / np.float32(batch)         # dL/dQ(s_i, a_i); the batch is a power of two: exact
    assert (np.delete(g, own) == 0).all() and (g[own] != 0).all()
    hi = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(g))
    two_parts = hi + synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(g - hi))

    def gradients(x):
        dW3, db3 = np.zeros((H2, A)), np.zeros(A)
        dW3[:, rows["a"][own]] = h2[own].T * x[own].astype(np.float64)
        db3[rows["a"][own]] = x[own]
        return dW3.ravel(), db3

    got = tr.grads()[-(H2 * A + A):]
    for x, want, without in zip((got[:H2 * A], got[H2 * A:]), gradients(g), gradients(two_parts)):
        bound = 2.0 ** -23 * np.abs(want)
        assert (np.abs(x - want) <= bound).all()
        assert (np.abs(without - want) > 8 * bound).any()


@pytest.mark.parametrize("D,H,H2,A,batch", [
    (27, 64, 64, 5, 1),           # one row of the first slice
    (31, 64, 64, 33, 63),         # last column of the first layer's tile the bias; a second block of actions
    (32, 192, 192, 3, 65),        # the bias behind the padded states; one row of the second slice
    (33, 64, 128, 32, 129),       # states beyond one tile; a row beyond the padding of 128
    (27, 128, 192, 30, 257),
    (64, 320, 320, 64, 191),      # widths that end inside a tile of 128
    (27, 128, 128, 30, 1000),     # (in the large steps' launches) several chunks, the last one ragged
    (27, 128, 1024, 30, 1000),    # several splits, the last one ends inside a slice
    (33, 128, 768, 30, 1100),     # ... two blocks of states
])
def test_mixed_precision_gradients_over_ragged_batches(B, D, H, H2, A, batch):
    """The weight gradients contract over the batch in slices of 64 rows of the batch-major activations
    and errors; tolerances of the other mixed-precision cases."""
    rows = synth.experiences(batch + 60, D, A, 0.05, seed=74, state_dtype="bf16")
    pr = Pair(B, capacity=batch + 30, D=D, H=H, H2=H2 if H2 != H else 0, A=A, batch=batch, burn_in=1, seed=5,
              dtype="bf16", appends=1, opt="sgd", lr=1e-3)
    assert pr.trainer.kernels_per_step() == (5 if batch >= 576 and H2 <= 512 else 8)
    pr.append_only(synth.take(rows, 0, batch + 30))
    for k in range(batch + 30, batch + 36):
        assert pr.step(synth.take(rows, k, k + 1), compare=True) == 0


@pytest.mark.parametrize("batch", [1, 65, 130, 1100])   # (the last one in the large steps' launches)
def test_mixed_precision_gradients_ignore_the_next_states_of_terminals(B, batch):
    """The rows of S' lie behind those of S in the activations: where every experience is terminal, what
    they hold, infinities included, changes no bit of the gradients."""
    D, H, A = 27, 128, 6
    rows = synth.experiences(batch + 1, D, A, 0.05, seed=75, state_dtype="bf16")
    rows["term"][:] = 1
    grads = []
    for bits in (0x0000, 0x7F80):
        rows["s_next"][:] = bits
        ring = B.Replay(batch + 1, D, B.RP_BF16, burn_in=1, seed=3)
        tr = B.Trainer(ring, H, A, batch, param_dtype=B.RP_BF16, opt=B.RP_SGD, appends_per_step=1, lr=1e-3,
                       init_params=synth.init_params(D, H, A, 3))
        assert tr.kernels_per_step() == (5 if batch == 1100 else 8)
        args = [rows[k] for k in ("s", "s_next", "a", "r", "term")]
        ring.append(*(x[:batch] for x in args))
        assert tr.step(*(x[batch:] for x in args)) == 0
        grads.append(tr.grads())
    assert np.isfinite(grads[0]).all() and np.array_equal(grads[0], grads[1])


@pytest.mark.parametrize("H,H2,batch,target_sync,kernels", [
    (512, 0, 512, 3, 8),     # second layer 64 tiles of 128 x 64, the most that go in tiles of 32 columns
    (512, 0, 576, 0, 5),     # (in the large steps' launches, as is the next)
    (512, 0, 1040, 0, 5),
    (64, 192, 37, 3, 11),    # both networks in launches of their own, rows that end inside a tile
    (128, 576, 448, 0, 8),   # 63 tiles
    (128, 576, 512, 3, 8),   # 72 of them, in tiles of 128 x 128; 30 x 16 rows of output layer in tiles of 16 ...
    (64, 1088, 530, 3, 11),  # ... rows that end inside one; seventeen 64-wide slices
])
def test_mixed_precision_products_with_few_tiles(B, H, H2, batch, target_sync, kernels):
    """Both sides of the rule that sends the second layer of small steps to tiles of 32 columns with a split
    contraction; tolerances of the other mixed-precision cases.  (Both sides for the first layer's error:
    test_mixed_precision_steps_with_many_states_or_actions.)"""
    D, A = 27, 30
    rows = synth.experiences(batch + 60, D, A, 0.05, seed=76, state_dtype="bf16")
    pr = Pair(B, capacity=batch + 30, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, dtype="bf16",
              appends=1, target_sync=target_sync, lr=1e-3)
    assert pr.trainer.kernels_per_step() == kernels
    pr.append_only(synth.take(rows, 0, batch + 30))
    for k in range(batch + 30, batch + 34):
        assert pr.step(synth.take(rows, k, k + 1), compare=True) == 0


@pytest.mark.parametrize("D,H,H2,A,batch,target_sync,dueling", [
    (27, 576, 192, 30, 1030, 0, False),   # widths and a batch that end inside tiles of 128 x 128
    (33, 1024, 64, 40, 600, 3, True),     # (small form: two blocks of states and of actions are too much here)
    (33, 512, 64, 40, 1100, 3, True),     # one slice of contraction; two blocks of states and of actions
    (96, 512, 320, 3, 1100, 0, False),    # three blocks of states, the bias behind the last
    (27, 64, 64, 5, 8300, 0, False),      # 256 x 128 tiles, more rows of them than rows of workgroups
    (31, 1024, 64, 33, 9000, 0, True),
    (9, 64, 512, 6, 577, 3, True),        # few tiles, a batch above the rule's line; a row of two steps a wavefront
    (27, 64, 1088, 30, 1537, 0, False),   # rows wider than the output layer's kernel holds at a time
    (27, 128, 512, 30, 640, 3, False),    # both networks' rows in one launch of the first two layers; two slices of H1
    (64, 192, 256, 30, 1600, 0, False),   # three slices, the fewest that are requested inside the loop; 64 states
    (20, 2112, 64, 30, 600, 0, False),    # first layer too wide for that launch
])
def test_mixed_precision_backward_in_two_launches(B, D, H, H2, A, batch, target_sync, dueling):
    """Large steps: output layer, TD errors and the second layer's error in one launch, all gradients and the first
    layer's error in another; tolerances of the other mixed-precision cases."""
    oracle.set_threads(16)
    try:
        rows = synth.experiences(batch + 60, D, A, 0.05, seed=79, state_dtype="bf16")
        pr = Pair(B, capacity=batch + 30, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, dtype="bf16",
                  appends=1, target_sync=target_sync, dueling=dueling, lr=1e-3)
        # gather, first two layers (one launch each for wide states or a wide first layer; another for a target network's
        # rows that share a tile with the others), head, gradients, update; the dueling head's update
        forward = (1 if D <= 64 and H <= 2048 else 2) * (2 if target_sync and batch % 128 else 1)
        assert pr.trainer.kernels_per_step() == (11 if batch == 600 and H == 1024 else 4 + forward) + dueling
        pr.append_only(synth.take(rows, 0, batch + 30))
        for k in range(batch + 30, batch + 34):
            assert pr.step(synth.take(rows, k, k + 1), compare=True) == 0
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("D,H,H2,A,batch,appends,target_sync,dueling,distinct,opt", [
    (27, 256, 0, 30, 1030, 3, 0, False, False, "adam"),     # tiles of 128 x 128
    (27, 128, 512, 30, 640, 1, 3, True, False, "adam"),     # both networks in one launch
    (50, 256, 128, 40, 1100, 17, 3, True, True, "adam"),    # in two, no duplicates; two blocks of states and of actions
    (96, 320, 0, 5, 1540, 1, 0, False, True, "sgd"),        # the first layer in a launch of its own
    (27, 1024, 0, 30, 4000, 64, 0, False, False, "adam"),   # tiles of 256 x 128 and of 128 x 256
    (27, 64, 64, 8, 8300, 0, 4, False, False, "sgd"),       # several groups and row tiles a workgroup
])
def test_recorded_runs_of_large_steps_equal_single_steps(B, D, H, H2, A, batch, appends, target_sync, dueling, distinct, opt):
    """Large steps in recorded runs, where the update's launch also gathers the next step's batch, leave the bits of the
    same steps made one by one, each with a synchronisation; and a second recorded run those of the first."""
    n, cap = 11, batch + 300
    rows = synth.experiences(cap + n * max(appends, 1), D, A, 0.05, seed=83, state_dtype="bf16")
    ends = []
    for how in ("run", "run", "steps"):
        pr = Pair(B, capacity=cap, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, dtype="bf16", appends=appends,
                  target_sync=target_sync, dueling=dueling, distinct=distinct, opt=opt, lr=1e-3)
        tr = pr.trainer
        assert tr.kernels_per_step() <= 6 + dueling             # (eight and more in the small form)
        for lo in range(0, cap, 4096):
            pr.append_only(synth.take(rows, lo, min(lo + 4096, cap)))
        new = synth.take(rows, cap, cap + n * appends)
        if how == "run":
            assert tr.steps(n, *(new[k] for k in synth.FIELDS)) == n
        else:
            for k in range(n):
                assert tr.step(*(new[f][k * appends:(k + 1) * appends] for f in synth.FIELDS)) == 0
                torch.cuda.synchronize()
        last, (m, v, t, step) = tr.last(), tr.opt_state()
        ends.append([tr.params(), tr.grads(), tr.target(), m, v, last["Q"], last["Qn"], last["y"], last["idx"],
                     np.array([t, step]), np.array([last["loss"]]), np.array(pr.gpu_ring.state()), *pr.gpu_ring.read_rows(0, cap)])
    assert np.isfinite(ends[0][0]).all()
    for other in ends[1:]:
        for k, (a, b) in enumerate(zip(ends[0], other)):
            assert np.array_equal(a, b), k


@pytest.mark.parametrize("D,H,H2,A,batch,target_sync,dueling,kernels", [
    (27, 512, 0, 30, 1100, 3, False, 6),      # the large form, in two blocks of rows
    (27, 512, 0, 256, 1100, 3, False, 11),    # ... eight blocks of actions: the small one, the first layer's error tiled
    (256, 512, 0, 30, 1100, 0, True, 9),      # ... eight blocks of states
    (96, 512, 0, 64, 1100, 0, False, 6),      # some of either: the large one, the first layer in a launch of its own
    (200, 64, 128, 100, 1540, 0, False, 8),   # a large batch, few tiles
    (300, 64, 0, 130, 8300, 0, False, 6),     # many more slices of batch than of states and actions
])
def test_mixed_precision_steps_with_many_states_or_actions(B, D, H, H2, A, batch, target_sync, dueling, kernels):
    """Both sides of the rule that takes networks with many states or actions from the large steps' launches, which
    walk them 32 at a time, to those of small steps; tolerances of the other mixed-precision cases."""
    oracle.set_threads(16)
    try:
        rows = synth.experiences(batch + 40, D, A, 0.05, seed=82, state_dtype="bf16")
        pr = Pair(B, capacity=batch + 30, D=D, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=5, dtype="bf16",
                  appends=1, target_sync=target_sync, dueling=dueling, lr=1e-3)
        assert pr.trainer.kernels_per_step() == kernels
        pr.append_only(synth.take(rows, 0, batch + 30))
        for k in range(batch + 30, batch + 34):
            assert pr.step(synth.take(rows, k, k + 1), compare=True) == 0
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("H,batch,kernels", [
    (128, 1100, 5),      # tiles of 128 x 128, the batch ends inside one
    (64, 8300, 5),       # of 256 x 128
    (64, 70, 8),         # a launch for each layer
])
def test_infinite_state_in_the_last_row_of_the_batch(B, H, batch, kernels):
    """The contraction over the batch goes in whole tiles of rows; what stands in for the rows beyond the batch
    contributes nothing, whatever the last row holds.  All weights are positive here and the last experience's
    state has an infinite entry d: its TD error is minus infinity, its Huber slope one and its dZ1 positive and
    finite, so that row d of dW1 is infinite, not NaN, and the other rows and the bias are finite."""
    D, A, d = 27, 6, 3
    p0 = np.abs(synth.init_params(D, H, A, 81))
    rows = synth.experiences(batch, D, A, 0.05, seed=81, state_dtype="bf16")
    rows["s"][-1, d] = 0x7F80
    dev = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in rows.items()}
    ring = B.Replay(64, D, B.RP_BF16, seed=1)
    tr = B.Trainer(ring, H, A, batch, param_dtype=B.RP_BF16, opt=B.RP_SGD, lr=1e-3, appends_per_step=0, init_params=p0)
    assert tr.kernels_per_step() == kernels
    assert tr.step_batch(*(dev[k] for k in ("s", "s_next", "a", "r", "term"))) == 0
    dW1, db1 = tr.grads()[:D * H].reshape(D, H), tr.grads()[D * H:D * H + H]
    assert np.isposinf(dW1[d]).all()
    assert np.isfinite(np.delete(dW1, d, axis=0)).all() and np.isfinite(db1).all()


@pytest.mark.parametrize("bias", [None, np.inf, 3.4e38, -np.inf])
@pytest.mark.parametrize("D,H2,batch", [
    (27, 128, 640),       # tiles of 128 x 128
    (64, 128, 577),       # ... two blocks of states, a batch that ends inside a tile
    (27, 2048, 1600),     # tiles of 128 x 256
])
def test_first_layer_of_large_steps_is_that_of_small_ones(B, D, H2, batch, bias):
    """Large steps form the first layer inside the launch of the second, small ones in a launch of its own; both round
    the same fp32 sum to bf16.  Here W2 passes the first layer's units on and W3 picks one for each action, so that
    the Q-values are those units, and equal bit for bit.  With `bias` one unit has a bias that is not finite, or is
    finite and rounds to infinity in bf16: what the network makes of it (NaNs among it) is the same too."""
    H, A, part = 128, 32, 64
    rng = np.random.default_rng(80)
    p0 = synth.init_params(D, H, A, 80, hidden2=H2)
    o = D * H
    if bias is not None:
        p0[o + 5] = bias
    W2, W3 = np.zeros((H, H2), np.float32), np.zeros((H2, A), np.float32)
    W2[np.arange(H), np.arange(H)] = 1
    W3[rng.permutation(H)[:A], np.arange(A)] = 1
    p0[o + H:] = np.concatenate([W2.ravel(), np.zeros(H2), W3.ravel(), np.zeros(A)])
    rows = synth.experiences(batch, D, A, 0.05, seed=80, state_dtype="bf16")
    d = {k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in rows.items()}
    q, kernels = [], []
    for n in (batch, part):
        ring = B.Replay(64, D, B.RP_BF16, seed=1)
        tr = B.Trainer(ring, H, A, n, param_dtype=B.RP_BF16, opt=B.RP_SGD, lr=1e-3, appends_per_step=0, init_params=p0,
                       hidden2=H2 if H2 != H else 0)
        kernels.append(tr.kernels_per_step())
        got = {"Q": np.empty((batch, A), np.float32), "Qn": np.empty((batch, A), np.float32)}
        for lo in list(range(0, batch - n, n)) + [batch - n]:
            tr.set_state(p0, None, None, 0, 0)
            assert tr.step_batch(*(d[k][lo:lo + n].contiguous() for k in ("s", "s_next", "a", "r", "term"))) == 0
            for k in got:
                got[k][lo:lo + n] = tr.last()[k]
        q.append(got)
    assert kernels == [5, 8]
    for k in ("Q", "Qn"):
        assert np.array_equal(q[0][k], q[1][k], equal_nan=True), k
        assert (bias == np.inf or bias == 3.4e38) != np.isfinite(q[0][k]).all(), k


@pytest.mark.parametrize("dtype,H,H2,batch,n", [
    ("bf16", 8192, 64, 131_200, 100),    # H1, which the second layer reads, is 4.3 GB
    ("bf16", 64, 8192, 262_200, 100),    # so is dZ2, which the first layer's error is formed from
    ("f32", 512, 8192, 524_300, 20),     # H2 is 34 GB, in 8.4 million tiles: more than one row of workgroups
])
def test_very_large_operands(B, dtype, H, H2, batch, n):
    """Products whose operand is larger than 32-bit byte offsets reach, or whose launch has more threads
    than a row of workgroups may have.  The batch is a block of n
    experiences over and over and, last, another block, whose rewards are so large that it makes up
    most of the gradients; 4 GiB is not a whole number of blocks of rows, so that a row that is taken
    from an offset that wrapped around is another experience's.  Every repetition of the block must
    give the same Q-values, the two blocks' Q-values and the gradients (a weighted sum of the two
    blocks'; in fp32 what no unit on a ReLU kink can reach) are the oracle's, at the tolerances of the
    other cases of the type."""
    D, A = 27, 30
    bf16, copies = dtype == "bf16", batch // n - 1
    rtol, g_rtol = (BF16_RTOL, 2 * BF16_RTOL) if bf16 else (F32_RTOL, 10 * F32_RTOL)
    p0 = synth.init_params(D, H, A, 7, hidden2=H2)
    st = B.RP_BF16 if bf16 else B.RP_F32
    ring = B.Replay(64, D, st, seed=1)
    tr = B.Trainer(ring, H, A, batch, param_dtype=st, loss=B.RP_MSE, opt=B.RP_SGD, lr=1e-3, appends_per_step=0,
                   use_graph=False, init_params=p0, hidden2=H2)
    blocks = [synth.experiences(n, D, A, 0.1, seed=k, state_dtype=dtype) for k in (77, 78)]
    blocks[1]["r"] *= np.float32(1e5)
    dev = [{k: torch.from_numpy(v.view(np.int16) if v.dtype == np.uint16 else v).cuda() for k, v in b.items()}
           for b in blocks]
    given = {k: torch.cat([dev[0][k].repeat((copies,) + (1,) * (dev[0][k].dim() - 1)), dev[1][k]]) for k in dev[0]}
    assert tr.step_batch(given["s"], given["s_next"], given["a"], given["r"], given["term"]) == 0
    last, g = tr.last(), tr.grads()
    cfg = oracle.make_cfg(D, H, A, n, loss=oracle.MSE, opt=oracle.SGD, lr=1e-3, gamma=float(np.float32(0.99)),
                          bf16=int(bf16), hidden2=H2)
    want, keep = 0.0, np.ones(len(g), bool)
    oracle.set_threads(16)
    for b, at, weight in ((blocks[0], slice(0, n), copies * n / batch), (blocks[1], slice(batch - n, batch), n / batch)):
        s, sn = ((synth.bf16_bits_to_f32(b[k]) if bf16 else b[k]).astype(np.float64) for k in ("s", "s_next"))
        ref = oracle.train_step(cfg, p0, None, None, 0, s, sn, b["a"], b["r"], b["term"])
        assert_close(last["Q"][at], ref.Q, rtol, "Q(s,.)")
        assert_close(last["Qn"][at], ref.Qn, rtol, "Q(s',.)")
        want = want + weight * ref.grads
        reach = None if bf16 else Pair.kink_reach(SimpleNamespace(D=D, H=H, H2=H2, A=A, dueling=False), p0, s)
        if reach is not None:
            keep &= ~reach
    oracle.set_threads(1)
    assert keep.mean() > 0.9
    for name in ("Q", "Qn"):
        rows = last[name][:copies * n].reshape(copies, n, A)
        assert (rows == rows[0]).all(), name
    for lo, hi in ((0, D * H + H), (D * H + H, D * H + H + H * H2 + H2), (D * H + H + H * H2 + H2, len(g))):
        if keep[lo:hi].any():
            assert_close(g[lo:hi][keep[lo:hi]], want[lo:hi][keep[lo:hi]], g_rtol, "gradients of one layer")


@pytest.mark.parametrize("appends,distinct", [(2, False), (2, True), (0, False), (0, True)])
@pytest.mark.parametrize("dtype,H,H2,batch,layered,target_sync,dueling,A", [
    ("bf16", 128, 0, 64, False, 0, False, 30), ("bf16", 128, 0, 130, False, 3, True, 30),
    ("bf16", 64, 192, 128, False, 3, True, 40), ("bf16", 64, 128, 40, True, 3, True, 30),
    ("bf16", 256, 0, 1100, False, 3, True, 30), ("bf16", 2112, 64, 640, False, 0, False, 30),
    ("f32", 64, 0, 32, False, 3, True, 40), ("f32", 128, 1024, 64, False, 3, True, 30),
    ("f32", 320, 0, 64, False, 0, False, 30), ("f32", 64, 0, 32, True, 0, True, 30)])
def test_launch_count_with_and_without_recorded_runs(B, dtype, H, H2, batch, layered, target_sync, dueling, A,
                                                     appends, distinct):
    """A trainer that records runs of steps counts the launches of a step as it records them; one that
    does not gives the same number."""
    counts = [Pair(B, capacity=max(300, batch + 30), D=27, H=H, H2=H2, A=A, batch=batch, burn_in=1, seed=1, dtype=dtype, appends=appends,
                   layered=layered, target_sync=target_sync, dueling=dueling, distinct=distinct,
                   use_graph=use_graph).trainer.kernels_per_step() for use_graph in (True, False)]
    assert counts[0] == counts[1]
