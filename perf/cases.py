"""The work that a user of this library has it do, as measurable cases.

Every case goes through the public calls of ``paper_1912_06680_amd`` (the
``o5_*`` bindings, or ``PPOStep`` for a whole optimizer step).  Kinds:

step     one whole optimizer step (``PPOStep.run``): GAE, sample cut, LSTM
         forward, heads and PPO loss, truncated BPTT, Adam
lstm     LSTM forward over T steps and its truncated BPTT (fp32 or bf16, with
         or without the input gradient)
rollout  one environment step of B environments: LSTM step without saved
         gates, heads, action filters, Gumbel-max draw
heads    policy and value heads, PPO loss and its gradient (optional
         unit-selection head, action filters, parameter-head mask; the
         gradient of the hidden state as a matrix or in factored form)
input    the LSTM's input side: observation normalisation, pre-LSTM layer
         with the cross-hero pool, and the layer's backward pass
rewards  reward post-processing, GAE and the cut into samples
adam     the optimizer over a flat parameter vector
"""
import math

import numpy as np
import torch

from paper_1912_06680_amd import o5, synth
from paper_1912_06680_amd.step import PARAM_ORDER, PPOStep

DEV = "cuda"
HEADS = "30,8,32,4"          # the four heads of the synthetic configurations
HEADS_UNITS = "30,189,32,4"  # with the paper's 189 units to select from


def listed():
    return [
        # the smallest whole step, fp32: parity runs and smoke tests; launches and latency
        {"name": "step_tiny_f32", "kind": "step", "dtype": "f32", "T": 16, "B": 8, "D": 64, "H": 128, "L": 16, "S": 8,
         "heads": "8"},
        # the benchmark's step: 2048 samples x 16 steps on the 4096-unit LSTM
        {"name": "step_full_bf16", "kind": "step", "dtype": "bf16", "T": 16, "B": 2048, "D": 4096, "H": 4096, "L": 256,
         "S": 128, "heads": HEADS},
        # mid-size training in full precision (debugging a policy, ablations)
        {"name": "lstm_mid_f32", "kind": "lstm", "dtype": "f32", "T": 16, "B": 256, "D": 1024, "H": 1024, "dx": False},
        # the same in bf16: small GEMMs, the chip half idle
        {"name": "lstm_mid_bf16", "kind": "lstm", "dtype": "bf16", "T": 16, "B": 256, "D": 1024, "H": 1024, "dx": False},
        # the paper's per-GPU minibatch (120 samples x 5 heroes) with the input
        # gradient that a trained pre-LSTM layer needs; B is no multiple of a tile
        {"name": "lstm_600_bf16", "kind": "lstm", "dtype": "bf16", "T": 16, "B": 600, "D": 4096, "H": 4096, "dx": True},
        # rollout inference for a small pool of environments: bound by the weights
        {"name": "rollout_60", "kind": "rollout", "dtype": "bf16", "B": 60, "D": 4096, "H": 4096, "heads": HEADS,
         "avail": True},
        # rollout inference for 4,096 environments: bound by the matrix units
        {"name": "rollout_4096", "kind": "rollout", "dtype": "bf16", "B": 4096, "D": 4096, "H": 4096, "heads": HEADS,
         "avail": False},
        # the loss at the paper's head sizes with unit selection, filters and masks
        {"name": "heads_units_9600", "kind": "heads", "dtype": "bf16", "N": 9600, "H": 4096, "heads": HEADS_UNITS,
         "unit_d": 128, "avail": True, "mask": True, "factored": True},
        # the trained input side at the paper's per-GPU minibatch
        {"name": "input_600_bf16", "kind": "input", "dtype": "bf16", "T": 16, "B": 600, "Do": 4096, "D": 4096},
        # advantages of a small rollout (13 games): latency
        {"name": "rewards_13", "kind": "rewards", "L": 256, "G": 13, "T": 16},
        # advantages of the paper's 2.9M-timestep batch
        {"name": "rewards_1152", "kind": "rewards", "L": 256, "G": 1152, "T": 16},
        # the optimizer over every parameter of the 4096-unit policy
        {"name": "adam_full", "kind": "adam", "n": 134541387, "bf16": True},
    ]


# ------------------------------------------------------------------ draws


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, hi=4096):
    return 64 * max(1, min(hi // 64, _log_int(rng, 1, hi // 64)))


def _heads_text(rng, units):
    if units:
        return "%d,%d,%d,%d" % (rng.randint(4, 40), rng.randint(20, 200), rng.randint(4, 90), rng.randint(2, 8))
    return ",".join(str(rng.randint(2, 48)) for _ in range(rng.randint(1, 6)))


def _cost(c):
    """A rough time in microseconds, to keep draws below the largest listed case."""
    w = work(c)
    rate = 20e6 if c.get("dtype") == "f32" else 0.9e9
    launches = 8 * 4 * c.get("T", 1) if c["kind"] in ("step", "lstm") else 60
    return w["flops"] / rate + w["bytes"] / 3.5e6 + launches


def _draw_any(rng):
    kind = rng.choice(("step", "lstm", "lstm", "rollout", "heads", "input", "rewards", "adam"))
    dtype = rng.choice(("bf16", "bf16", "f32"))
    if kind == "step":
        T = rng.choice((4, 8, 16))
        S, J = _log_int(rng, 1, 130), _log_int(rng, 1, 16)
        return {"kind": kind, "dtype": dtype, "T": T, "B": S * J, "D": _width(rng), "H": _width(rng), "L": T * J,
                "S": S, "heads": _heads_text(rng, False)}
    if kind == "lstm":
        return {"kind": kind, "dtype": dtype, "T": rng.choice((1, 4, 8, 15, 16)), "B": _log_int(rng, 1, 2048),
                "D": _width(rng), "H": _width(rng), "dx": rng.random() < 0.4}
    if kind == "rollout":
        return {"kind": kind, "dtype": dtype, "B": _log_int(rng, 1, 4096), "D": _width(rng), "H": _width(rng),
                "heads": _heads_text(rng, False), "avail": rng.random() < 0.5}
    if kind == "heads":
        unit = rng.random() < 0.4
        return {"kind": kind, "dtype": dtype, "N": _log_int(rng, 16, 32768), "H": _width(rng),
                "heads": _heads_text(rng, unit), "unit_d": rng.choice((32, 64, 128)) if unit else 0,
                "avail": rng.random() < 0.5, "mask": rng.random() < 0.5,
                "factored": dtype == "bf16" and rng.random() < 0.6}
    if kind == "input":
        return {"kind": kind, "dtype": dtype, "T": rng.choice((1, 8, 16)), "B": 5 * _log_int(rng, 1, 408),
                "Do": _width(rng), "D": _width(rng)}
    if kind == "rewards":
        T = rng.choice((8, 16))
        return {"kind": kind, "L": T * rng.randint(1, 256 // T), "G": _log_int(rng, 1, 4000), "T": T}
    return {"kind": "adam", "n": _log_int(rng, 10000, 134541387), "bf16": rng.random() < 0.7}


def draw(rng):
    most = _cost(listed()[1])
    while True:
        c = _draw_any(rng)
        if _cost(c) <= most:
            return c


# ----------------------------------------------------------------- inputs


class _Rand:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.g, device=DEV) * std

    def uniform(self, *shape, bound=1.0):
        return (torch.rand(shape, generator=self.g, device=DEV) * 2 - 1) * bound

    def flag(self, *shape, p):
        return (torch.rand(shape, generator=self.g, device=DEV) < p).to(torch.uint8)

    def action(self, N, heads):
        return torch.stack([torch.randint(0, n, (N,), generator=self.g, device=DEV, dtype=torch.int32) for n in heads],
                           1).contiguous()


def _heads(c):
    return tuple(int(n) for n in c["heads"].split(","))


def _et(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _dt(c):
    return o5.O5_BF16 if c["dtype"] == "bf16" else o5.O5_F32


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def _ws(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _prepare_step(c, r):
    cfg = synth.Config("perf", B=c["B"], T=c["T"], D=c["D"], H=c["H"], head_sizes=_heads(c), L=c["L"], S=c["S"],
                       done_p=0.002, state_std=0.1, dtype=c["dtype"])
    st = PPOStep(cfg, device=DEV)
    st.p32.copy_(r.uniform(st.n_params, bound=c["H"] ** -0.5))
    st.sync_bf16()
    st.x.copy_(r.normal(c["T"], c["B"], c["D"]))
    st.h0.copy_(r.normal(c["B"], c["H"], std=0.1))
    st.c0.copy_(r.normal(c["B"], c["H"], std=0.1))
    st.rewards.copy_(r.normal(c["L"], c["S"]))
    st.dones.copy_(r.flag(c["L"], c["S"], p=0.002))
    st.values.copy_(r.normal(c["L"] + 1, c["S"], std=0.2))
    st.act.copy_(r.action(st.N, _heads(c)))
    # the behaviour policy's log-probability: near-uniform heads, some drift
    st.logp_old.copy_(r.normal(st.N, std=0.1) - math.log(np.prod([float(n) for n in _heads(c)])))
    return {"st": st}


def _run_step(c, s):
    st = s["st"]
    st.run()
    return {"stats": st.stats, "grads": {k: st.G[k] for k in PARAM_ORDER}, "p": st.p32, "m": st.m, "v": st.v}


def _lstm_inputs(c, r, T):
    et, B, D, H = _et(c), c["B"], c["D"], c["H"]
    w = H ** -0.5
    return {"x": r.normal(T, B, D).to(et), "Wx": r.uniform(4 * H, D, bound=w).to(et),
            "Wh": r.uniform(4 * H, H, bound=w).to(et), "b": r.uniform(4 * H, bound=w),
            "h0": r.normal(B, H, std=0.1), "c0": r.normal(B, H, std=0.1)}


def _prepare_lstm(c, r):
    et, T, B, D, H = _et(c), c["T"], c["B"], c["D"], c["H"]
    s = _lstm_inputs(c, r, T)
    s["reset"] = r.flag(T, B, p=0.01)
    s["dh"] = r.normal(T, B, H, std=1e-3)
    s["h"], s["c"] = torch.empty((T, B, H), dtype=et, device=DEV), _f32(T, B, H)
    s["gates"] = torch.empty((T, B, 4 * H), dtype=et, device=DEV)
    s["dWx"], s["dWh"], s["db"] = _f32(4 * H, D), _f32(4 * H, H), _f32(4 * H)
    s["dx"] = torch.empty((T, B, D), dtype=et, device=DEV) if c["dx"] else None
    s["ws"] = _ws(max(o5.o5_lstm_fwd_workspace_bytes(_dt(c), T, B, D, H),
                      o5.o5_lstm_bptt_workspace_bytes(_dt(c), T, B, D, H)))
    return s


def _run_lstm(c, s):
    dt, dims = _dt(c), (c["T"], c["B"], c["D"], c["H"])
    o5.o5_lstm_fwd(dt, *dims, s["x"], s["Wx"], s["Wh"], s["b"], s["h0"], s["c0"], s["reset"], s["h"], s["c"],
                   s["gates"], s["ws"])
    o5.o5_lstm_bptt(dt, *dims, s["x"], s["Wx"], s["Wh"], s["h0"], s["c0"], s["reset"], s["h"], s["c"], s["gates"],
                    s["dh"], None, None, s["dWx"], s["dWh"], s["db"], s["dx"], s["ws"])
    out = {k: s[k] for k in ("h", "c", "gates", "dWx", "dWh", "db")}
    if c["dx"]:
        out["dx"] = s["dx"]
    return out


def _avail(r, N, heads, p):
    """Action filters: each logit available with probability p, the first of each head always."""
    a = r.flag(N, sum(heads), p=p)
    o = 0
    for n in heads:
        a[:, o] = 1
        o += n
    return a


def _prepare_rollout(c, r):
    B, H, heads = c["B"], c["H"], _heads(c)
    s = _lstm_inputs(c, r, 1)
    A1 = sum(heads) + 1
    s["Wp"], s["bp"] = r.uniform(A1, H, bound=H ** -0.5).to(_et(c)), r.uniform(A1, bound=H ** -0.5)
    s["avail"] = _avail(r, B, heads, 0.7) if c["avail"] else None
    s["h"], s["c"] = torch.empty((1, B, H), dtype=_et(c), device=DEV), _f32(1, B, H)
    s["act"] = torch.empty((B, len(heads)), dtype=torch.int32, device=DEV)
    s["logp"], s["value"] = _f32(B), _f32(B)
    s["ws"] = _ws(o5.o5_lstm_fwd_workspace_bytes(_dt(c), 1, B, c["D"], H))
    s["sws"] = _ws(o5.o5_policy_sample_workspace_bytes(_dt(c), B, H, heads))
    return s


def _run_rollout(c, s):
    dt, B, H = _dt(c), c["B"], c["H"]
    o5.o5_lstm_fwd(dt, 1, B, c["D"], H, s["x"], s["Wx"], s["Wh"], s["b"], s["h0"], s["c0"], None, s["h"], s["c"], None,
                   s["ws"])
    o5.o5_policy_sample(dt, B, H, _heads(c), s["h"], s["Wp"], s["bp"], 7, 3, s["act"], s["logp"], s["value"], s["sws"],
                        avail=s["avail"])
    return {k: s[k] for k in ("h", "c", "act", "logp", "value")}


UNIT_HEAD = 1  # the head that selects a unit


def _prepare_heads(c, r):
    N, H, heads, d, et = c["N"], c["H"], _heads(c), c["unit_d"], _et(c)
    A1 = sum(heads) + 1
    w = H ** -0.5
    s = {"h": (torch.sigmoid(r.normal(N, H)) * torch.tanh(r.normal(N, H, std=0.7))).to(et),
         "Wp": r.uniform(A1, H, bound=w).to(et), "bp": r.uniform(A1, bound=w), "act": r.action(N, heads),
         "adv": r.normal(N), "ret": r.normal(N),
         "mask": r.flag(N, len(heads), p=0.8) if c["mask"] else None}
    s["avail"] = None
    n_av = [float(n) for n in heads]
    if c["avail"]:
        s["avail"] = _avail(r, N, heads, 0.7)
        # actions were drawn from the available logits
        o = 0
        for k, n in enumerate(heads):
            ok = torch.gather(s["avail"][:, o:o + n], 1, s["act"][:, k:k + 1].long())[:, 0] != 0
            s["act"][:, k] = torch.where(ok, s["act"][:, k], torch.zeros_like(s["act"][:, k]))
            o += n
        n_av = [1 + 0.7 * (n - 1) for n in n_av]
    each = torch.tensor([math.log(n) for n in n_av], device=DEV)
    lp = -(each * s["mask"].float()).sum(1) if c["mask"] else -each.sum().expand(N)
    s["logp_old"] = (lp + r.normal(N, std=0.1)).contiguous()
    s["unit"], s["unit_t"] = None, None
    if d:
        t = {"Wq": r.uniform(d, H, bound=w).to(et), "bq": r.uniform(d, bound=w),
             "E": torch.empty((N, heads[UNIT_HEAD], d), dtype=et, device=DEV),
             "dWq": _f32(d, H), "dbq": _f32(d)}
        t["E"].copy_(r.normal(N, heads[UNIT_HEAD], d, std=0.3))
        s["unit_t"] = t
        s["unit"] = o5.unit_head(UNIT_HEAD, d, t["Wq"], t["bq"], t["E"], t["dWq"], t["dbq"])
    s["stats"], s["dWp"], s["dbp"] = _f32(8), _f32(A1, H), _f32(A1)
    if c["factored"]:
        s["ld"] = o5.o5_ppo_head_grad_ld(H, heads, s["unit"])
        s["P"] = torch.empty((N, s["ld"]), dtype=torch.bfloat16, device=DEV)
        s["W"] = torch.empty((H, s["ld"]), dtype=torch.bfloat16, device=DEV)
    else:
        s["dh"] = _f32(N, H)
    s["ws"] = _ws(o5.o5_ppo_loss_grad_workspace_bytes(_dt(c), N, H, heads, s["unit"]))
    return s


def _run_heads(c, s):
    args = (_dt(c), c["N"], c["H"], _heads(c), s["h"], s["Wp"], s["bp"], s["act"], s["logp_old"], s["adv"], s["ret"],
            s["mask"], 0.2, 1.0, 0.01, s["stats"])
    if c["factored"]:
        o5.o5_ppo_loss_grad_factored(*args, s["P"], s["W"], s["ld"], s["dWp"], s["dbp"], s["ws"], avail=s["avail"],
                                     unit=s["unit"])
    else:
        o5.o5_ppo_loss_grad(*args, s["dh"], s["dWp"], s["dbp"], s["ws"], avail=s["avail"], unit=s["unit"])
    out = {k: s[k] for k in ("stats", "dWp", "dbp") + (("P", "W") if c["factored"] else ("dh",))}
    if s["unit_t"]:
        out["dWq"], out["dbq"] = s["unit_t"]["dWq"], s["unit_t"]["dbq"]
    return out


def _prepare_input(c, r):
    et, T, B, Do, D = _et(c), c["T"], c["B"], c["Do"], c["D"]
    N = T * B
    # a running summary of earlier observations of the same distribution
    n0 = 65536.0
    stats = torch.stack([torch.full((Do,), n0, device=DEV), torch.full((Do,), 1.0, device=DEV),
                         torch.full((Do,), 4.0 * n0, device=DEV)]).double()
    return {"obs": r.normal(N, Do, std=2.0) + 1.0, "stats": stats.contiguous(),
            "W": r.uniform(D, Do, bound=Do ** -0.5).to(et), "b": r.uniform(D, bound=Do ** -0.5),
            "dx": r.normal(N, D, std=1e-3).to(et),
            "o": torch.empty((N, Do), dtype=et, device=DEV), "y": _f32(N, D),
            "x": torch.empty((N, D), dtype=et, device=DEV), "dW": _f32(D, Do), "db": _f32(D),
            "ws": _ws(max(o5.o5_obs_normalize_workspace_bytes(N, Do),
                          o5.o5_prelstm_bwd_workspace_bytes(_dt(c), T, B, Do, D)))}


def _run_input(c, s):
    dt, dims = _dt(c), (c["T"], c["B"], c["Do"], c["D"])
    o5.o5_obs_normalize(dt, c["T"] * c["B"], c["Do"], s["obs"], s["stats"], 5.0, 1e-8, s["o"], s["ws"])
    o5.o5_prelstm_fwd(dt, *dims, s["o"], s["W"], s["b"], s["y"], s["x"])
    o5.o5_prelstm_bwd(dt, *dims, s["o"], s["y"], s["dx"], s["dW"], s["db"], s["ws"])
    return {k: s[k] for k in ("stats", "o", "y", "x", "dW", "db")}


GAMMA, LAM, TAU = 0.998, 0.95, 0.3


def _prepare_rewards(c, r):
    L, G, T = c["L"], c["G"], c["T"]
    S = 10 * G
    B = S * (L // T)
    u = torch.rand((L, S), generator=r.g, device=DEV)
    start = torch.rand((1, G), generator=r.g, device=DEV) * 60.0
    step = synth.STEP_MINUTES * torch.arange(L, device=DEV, dtype=torch.float32)[:, None]
    return {"shaped": r.normal(L, S), "outcome": (u < 0.01).float() - (u > 0.99).float(),
            "game_time": (start + step).contiguous(), "v": r.normal(L + 1, S, std=0.5), "done": r.flag(L, S, p=0.002),
            "stats": torch.zeros(3, dtype=torch.float64, device=DEV), "r": _f32(L, S), "adv": _f32(L, S),
            "ret": _f32(L, S), "adv_s": _f32(T, B), "ret_s": _f32(T, B),
            "reset": torch.empty((T, B), dtype=torch.uint8, device=DEV),
            "ws": _ws(o5.o5_reward_process_workspace_bytes(L, G))}


def _run_rewards(c, s):
    L, G, T = c["L"], c["G"], c["T"]
    S = 10 * G
    o5.o5_reward_process(L, G, s["shaped"], s["outcome"], s["game_time"], TAU, 0.6, 10.0, 1e-8, s["stats"], s["r"],
                         s["ws"])
    o5.o5_gae(L, S, s["r"], s["v"], s["done"], GAMMA, LAM, s["adv"], s["ret"])
    o5.o5_segments_to_samples(L, S, T, s["adv"], s["ret"], s["done"], s["adv_s"], s["ret_s"], s["reset"])
    return {k: s[k] for k in ("stats", "r", "adv", "ret", "adv_s", "ret_s", "reset")}


ADAM = (5e-5, 0.9, 0.999, 1e-8, 5.0)  # learning rate, betas, epsilon, clip


def _prepare_adam(c, r):
    n = c["n"]
    g = r.normal(n, std=1e-4)
    return {"p": r.uniform(n, bound=0.0156), "m": r.normal(n, std=3e-5), "v": 1e-8 * (0.2 + r.uniform(n).abs()),
            "g": g, "pb": torch.empty(n, dtype=torch.bfloat16, device=DEV) if c["bf16"] else None, "step": 100}


def _run_adam(c, s):
    s["step"] += 1
    o5.o5_adam_step(c["n"], s["p"], s["m"], s["v"], s["g"], s["pb"], *ADAM, s["step"])
    out = {k: s[k] for k in ("p", "m", "v")}
    if c["bf16"]:
        out["pb"] = s["pb"]
    return out


_PREPARE = {"step": _prepare_step, "lstm": _prepare_lstm, "rollout": _prepare_rollout, "heads": _prepare_heads,
            "input": _prepare_input, "rewards": _prepare_rewards, "adam": _prepare_adam}
_RUN = {"step": _run_step, "lstm": _run_lstm, "rollout": _run_rollout, "heads": _run_heads, "input": _run_input,
        "rewards": _run_rewards, "adam": _run_adam}


def prepare(case, seed):
    return {"case": case, "data": _PREPARE[case["kind"]](case, _Rand(seed))}


def run(state):
    return _RUN[state["case"]["kind"]](state["case"], state["data"])


# ------------------------------------------------------------ work, bounds


def work(case):
    c = case
    kind = c["kind"]
    e = 4 if c.get("dtype") == "f32" else 2
    if kind == "step":
        T, B, D, H, heads = c["T"], c["B"], c["D"], c["H"], _heads(c)
        N, A1 = T * B, sum(heads) + 1
        n = 4 * H * (D + H + 1) + A1 * (H + 1)
        flops = 4.0 * N * 4 * H * (D + H) + 2.0 * (N - B) * 4 * H * H + 6.0 * N * H * A1
        # p, m, v in and out, the gradient and the bf16 weights out; the inputs
        by = n * (28.0 + (2 if e == 2 else 0)) + e * N * D + 8.0 * B * H + 9.0 * N + N * (4 * len(heads) + 4)
    elif kind == "lstm":
        T, B, D, H = c["T"], c["B"], c["D"], c["H"]
        N = T * B
        flops = 4.0 * N * 4 * H * (D + H) + 2.0 * (N - B) * 4 * H * H + (2.0 * N * 4 * H * D if c["dx"] else 0.0)
        by = (e * N * D * (2 if c["dx"] else 1) + (e + 4.0) * 4 * H * (D + H + 1) + 8.0 * B * H
              + N * H * (5.0 * e + 4 + 4) + N)
    elif kind == "rollout":
        B, D, H, A1 = c["B"], c["D"], c["H"], sum(_heads(c)) + 1
        flops = 2.0 * B * 4 * H * (D + H) + 2.0 * B * A1 * H
        by = e * (B * D + 4.0 * H * (D + H) + A1 * H + B * H) + 12.0 * B * H + (B * A1 if c["avail"] else 0)
    elif kind == "heads":
        N, H, heads, d = c["N"], c["H"], _heads(c), c["unit_d"]
        A1 = sum(heads) + 1
        lin = A1 + (d - heads[UNIT_HEAD] if d else 0)
        flops = 2.0 * N * H * lin * (2 if c["factored"] else 3) + (4.0 * N * heads[UNIT_HEAD] * d if d else 0.0)
        by = (e * (N * H + A1 * H) + 4.0 * A1 * H + N * (12 + 4 * len(heads)) + (N * A1 if c["avail"] else 0)
              + (N * len(heads) if c["mask"] else 0))
        by += 4.0 * (N + H) * lin if c["factored"] else 4.0 * N * H
        by += (e + 4.0) * d * H + e * N * heads[UNIT_HEAD] * d if d else 0.0
    elif kind == "input":
        N, Do, D = c["T"] * c["B"], c["Do"], c["D"]
        flops = 4.0 * N * D * Do
        by = N * Do * (4.0 + e) + N * D * (4.0 + 2 * e) + D * Do * (e + 4.0) + 48.0 * Do
    elif kind == "rewards":
        L, G = c["L"], c["G"]
        flops = 30.0 * L * G * 10
        # shaped, outcome, values, done in; r, advantages and returns in both layouts, reset out; game time
        by = L * G * 10 * (4.0 * 3 + 1 + 4.0 * 5 + 1) + 4.0 * L * G
    else:
        flops = 15.0 * c["n"]
        by = c["n"] * (30.0 if c["bf16"] else 28.0)
    return {"bytes": by, "flops": flops}


def tolerance(case):
    """About four times the largest error that the path shows against 64 bits
    (fp32 sums in another order; bf16: the rounding of the stored hidden
    state, gates and gate gradients, carried through the steps)."""
    kind = case["kind"]
    if kind == "rewards":
        return {"rel": 2e-6, "max": 1e-3}
    if kind == "adam":
        # the bf16 copy: a parameter one fp32 ulp off may round to the neighbour
        return {"rel": 2e-5, "max": 1e-2} if case["bf16"] else {"rel": 4e-7, "max": 1e-4}
    if case["dtype"] == "f32":
        if kind == "rollout":
            return {"rel": 6e-6, "max": 1e-2, "differ": 1e-3}
        return {"rel": 1e-5, "max": 1e-2}
    if kind == "rollout":
        # a hidden state rounded to its neighbour can turn a close draw
        return {"rel": 1e-2, "max": 0.99, "differ": 1e-2}
    if kind == "heads":
        # the (hi, lo) pair: a gradient one fp32 ulp off may split at the neighbour
        return {"rel": 3e-4, "max": 5e-1}
    if kind == "step":
        # a row whose ratio lies on the clip's edge gains or loses its gradient
        return {"rel": 2e-2, "max": 0.99}
    return {"rel": 1e-2, "max": 3e-1}


# ---------------------------------------------- the same in 64 bits, plainly


def _lstm64(s, T, want_grads, dh=None, want_dx=False):
    """h, c, gates [T, ...] and, given dL/dh, the gradients."""
    x, Wx, Wh, b = s["x"].double(), s["Wx"].double(), s["Wh"].double(), s["b"].double()
    reset = s.get("reset")
    h, c = s["h0"].double(), s["c0"].double()
    H = h.shape[1]
    hs, cs, gs, hp, cp = [], [], [], [], []
    for t in range(T):
        if reset is not None:
            keep = (reset[t] == 0).double()[:, None]
            h, c = h * keep, c * keep
        hp.append(h)
        cp.append(c)
        a = x[t] @ Wx.t() + h @ Wh.t() + b
        i, f, g, o = (torch.sigmoid(a[:, :H]), torch.sigmoid(a[:, H:2 * H]), torch.tanh(a[:, 2 * H:3 * H]),
                      torch.sigmoid(a[:, 3 * H:]))
        c = f * c + i * g
        h = o * torch.tanh(c)
        hs.append(h)
        cs.append(c)
        gs.append(torch.cat([i, f, g, o], 1))
    out = {"h": torch.stack(hs), "c": torch.stack(cs), "gates": torch.stack(gs)}
    if not want_grads:
        return out
    dWx, dWh, db = torch.zeros_like(Wx), torch.zeros_like(Wh), torch.zeros_like(b)
    dx = [None] * T
    rec, dc = torch.zeros_like(h), torch.zeros_like(h)
    for t in range(T - 1, -1, -1):
        i, f, g, o = gs[t][:, :H], gs[t][:, H:2 * H], gs[t][:, 2 * H:3 * H], gs[t][:, 3 * H:]
        d = dh[t].double() + rec
        tc = torch.tanh(cs[t])
        dct = dc + d * o * (1 - tc * tc)
        dG = torch.cat([dct * g * i * (1 - i), dct * cp[t] * f * (1 - f), dct * i * (1 - g * g),
                        d * tc * o * (1 - o)], 1)
        dWx += dG.t() @ x[t]
        dWh += dG.t() @ hp[t]
        db += dG.sum(0)
        if want_dx:
            dx[t] = dG @ Wx
        rec, dc = dG @ Wh, dct * f
        if reset is not None:
            keep = (reset[t] == 0).double()[:, None]
            rec, dc = rec * keep, dc * keep
    out.update({"dWx": dWx, "dWh": dWh, "db": db})
    if want_dx:
        out["dx"] = torch.stack(dx)
    return out


def _gae64(r, v, done):
    L = r.shape[0]
    adv, carry = torch.zeros_like(r), torch.zeros_like(r[0])
    for t in range(L - 1, -1, -1):
        nd = (done[t] == 0).double()
        carry = r[t] + GAMMA * nd * v[t + 1] - v[t] + GAMMA * LAM * nd * carry
        adv[t] = carry
    return adv, adv + v[:L]


def _cut(a, T):
    L, S = a.shape
    return a.view(L // T, T, S).permute(1, 2, 0).reshape(T, -1)


def _cut_reset(done, T):
    d = _cut((done != 0).to(torch.uint8), T)
    return torch.cat([torch.zeros_like(d[:1]), d[:-1]])


def _heads64(h, Wp, bp, heads, act, lpo, adv, ret, mask=None, avail=None, unit=None):
    N, A = h.shape[0], sum(heads)
    z = h @ Wp.t() + bp
    if unit is not None:
        q = h @ unit["Wq"].double().t() + unit["bq"].double()
    dz = torch.zeros_like(z)
    logpi, ent, keep = torch.zeros_like(adv), torch.zeros_like(adv), []
    o = 0
    for k, n in enumerate(heads):
        zk = z[:, o:o + n]
        if unit is not None and k == UNIT_HEAD:
            zk = (q[:, None, :] * unit["E"].double()).sum(2)
        if avail is not None:
            zk = zk.masked_fill(avail[:, o:o + n] == 0, -math.inf)
        lp = torch.log_softmax(zk, 1)
        p = lp.exp()
        ek = -torch.where(p > 0, p * lp, torch.zeros_like(p)).sum(1)
        m = torch.ones_like(adv) if mask is None else (mask[:, k] != 0).double()
        onehot = torch.nn.functional.one_hot(act[:, k].long(), n).double()
        logpi += m * torch.gather(lp, 1, act[:, k:k + 1].long())[:, 0]
        ent += m * ek
        keep.append((o, n, m, onehot, p, torch.where(p > 0, lp, torch.zeros_like(p)), ek))
        o += n
    ratio = torch.exp(logpi - lpo)
    surr = torch.minimum(ratio * adv, ratio.clamp(1 - 0.2, 1 + 0.2) * adv)
    err = z[:, A] - ret
    flow = torch.where(adv >= 0, ratio <= 1.2, ratio >= 0.8)
    gl = torch.where(flow, -ratio * adv / N, torch.zeros_like(adv))
    for o, n, m, onehot, p, lp, ek in keep:
        dz[:, o:o + n] = m[:, None] * (gl[:, None] * (onehot - p) + 0.01 / N * p * (lp + ek[:, None]))
    dz[:, A] = 2 * err / N
    pg, vf, en = -surr.mean(), (err * err).mean(), ent.mean()
    stats = torch.stack([pg + vf - 0.01 * en, pg, vf, en, ((ratio - 1).abs() > 0.2).double().mean(),
                         (torch.expm1(logpi - lpo) - (logpi - lpo)).mean(), ratio.mean(), torch.zeros_like(pg)])
    out = {"stats": stats}
    dq = None
    if unit is not None:
        o, n = sum(heads[:UNIT_HEAD]), heads[UNIT_HEAD]
        dq = (dz[:, o:o + n, None] * unit["E"].double()).sum(1)
        dz[:, o:o + n] = 0
        out["dWq"], out["dbq"] = dq.t() @ h, dq.sum(0)
    out["dWp"], out["dbp"], out["dh"] = dz.t() @ h, dz.sum(0), dz @ Wp
    if unit is not None:
        out["dh"] = out["dh"] + dq @ unit["Wq"].double()
    return out


def exact(case, seed):
    c = case
    kind = c["kind"]
    s = prepare(c, seed)["data"]
    if kind == "step":
        st = s["st"]
        T, heads = c["T"], _heads(c)
        adv, ret = _gae64(st.rewards.double(), st.values.double(), st.dones)
        W = {k: st.W[k].double() for k in ("Wx", "Wh", "Wp")}
        d = {"x": st.x, "Wx": W["Wx"], "Wh": W["Wh"], "b": st.P["b"], "h0": st.h0, "c0": st.c0,
             "reset": _cut_reset(st.dones, T)}
        h = _lstm64(d, T, False)["h"].reshape(T * c["B"], c["H"])
        hd = _heads64(h, W["Wp"], st.P["bp"].double(), heads, st.act, st.logp_old.double(),
                      _cut(adv, T).reshape(-1), _cut(ret, T).reshape(-1))
        g = _lstm64(d, T, True, hd["dh"].view(T, c["B"], c["H"]))
        return {"stats": hd["stats"], "grads": {"Wx": g["dWx"], "Wh": g["dWh"], "b": g["db"], "Wp": hd["dWp"],
                                                "bp": hd["dbp"]}, "p": None, "m": None, "v": None}
    if kind == "lstm":
        return _lstm64(s, c["T"], True, s["dh"], c["dx"])
    if kind == "rollout":
        out = _lstm64(s, 1, False)
        value = out["h"][0] @ s["Wp"][-1].double() + s["bp"][-1].double()
        return {"h": out["h"], "c": out["c"], "act": None, "logp": None, "value": value}
    if kind == "heads":
        if c["unit_d"] and c["N"] * _heads(c)[UNIT_HEAD] * c["unit_d"] > 1 << 30:
            return None
        out = _heads64(s["h"].double(), s["Wp"].double(), s["bp"].double(), _heads(c), s["act"],
                       s["logp_old"].double(), s["adv"].double(), s["ret"].double(), s["mask"], s["avail"],
                       s["unit_t"])
        dh = out.pop("dh")
        if c["factored"]:
            out["P"], out["W"] = None, None
        else:
            out["dh"] = dh
        return out
    if kind == "input":
        N, D = c["T"] * c["B"], c["D"]
        x = s["obs"].double()
        n0, m0, q0 = s["stats"]
        mean, var = x.mean(0), x.var(0, unbiased=False)
        n = n0 + N
        d = mean - m0
        stats = torch.stack([n, m0 + d * N / n, q0 + var * N + d * d * n0 * N / n])
        o = ((x - stats[1]) / torch.sqrt(stats[2] / n + 1e-8)).clamp(-5, 5)
        ob = o.to(_et(c)).double()
        y = torch.relu(ob @ s["W"].double().t() + s["b"].double())
        P = D // 4
        yg = y.view(N // 5, 5, D)
        xg = yg.clone()
        top, win = yg[:, :, :P].max(1)
        xg[:, :, :P] = top[:, None, :]
        first = (yg[:, :, :P] == top[:, None, :]).to(torch.uint8).argmax(1)  # the first replica attaining it
        dx = s["dx"].double().view(N // 5, 5, D)
        dp = dx.clone()
        dp[:, :, :P] = 0
        dp[:, :, :P].scatter_(1, first[:, None, :], dx[:, :, :P].sum(1, keepdim=True))
        dp = (dp * (yg > 0)).reshape(N, D)
        return {"stats": stats, "o": o, "y": y, "x": xg.reshape(N, D), "dW": dp.t() @ ob, "db": dp.sum(0)}
    if kind == "rewards":
        L, G, T = c["L"], c["G"], c["T"]
        w = 0.6 ** (s["game_time"].double() / 10.0)
        rho = (s["shaped"].double().view(L, G, 10) * w[:, :, None] + s["outcome"].double().view(L, G, 10)).view(L, G, 2, 5)
        team = rho.mean(3, keepdim=True)
        z = ((1 - TAU) * rho + TAU * team - team.flip(2)).reshape(L, 10 * G)
        n, mean = float(z.numel()), z.mean()
        m2 = ((z - mean) ** 2).sum()
        r = z / torch.sqrt(m2 / n + 1e-8)
        adv, ret = _gae64(r, s["v"].double(), s["done"])
        # (the running mean of zero-sum rewards is rounding noise about zero: it has no value to compare with)
        return {"stats": None, "r": r, "adv": adv, "ret": ret, "adv_s": _cut(adv, T), "ret_s": _cut(ret, T),
                "reset": None}
    lr, b1, b2, eps, k = ADAM
    step = s["step"] + 1
    p, m, v, g = (s[q].double() for q in ("p", "m", "v", "g"))
    v = b2 * v + (1 - b2) * g * g
    vh = (v / (1 - b2 ** step)).sqrt()
    m = b1 * m + (1 - b1) * torch.minimum(torch.maximum(g, -k * vh), k * vh)
    p = p - lr * (m / (1 - b1 ** step)) / (vh + eps)
    out = {"p": p, "m": m, "v": v}
    if c["bf16"]:
        out["pb"] = p
    return out
