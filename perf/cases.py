"""The calls whose speed matters to a user of this package, as measurable cases.

Every case goes through the public entry points of `paper_1805_08899_amd.binding` the way a training loop or a
decoder calls them: buffers, descriptor and workspace are kept by the program, inputs are resident on the GPU, results
land in the program's own buffers.

Kinds of case:
  train     forward and backward of the attention layer on one batch (echo_attn_fwd, echo_attn_bwd)
  infer     forward alone, as in scoring or evaluating a batch
  step      one decoder step of a search: one query per hypothesis against its keys (echo_attn_step_fwd)
  sentence  a decoder's training pass over one batch of sentences, one query at a time: every step forward, every step's
            query gradient in reverse order, then the key-side gradients once (echo_attn_fwd with Tq = 1,
            echo_attn_step_bwd_query, echo_attn_steps_bwd_keys)
  lstm      forward and backward of the LSTM cell's non-linear block (echo_lstm_cell_fwd, echo_lstm_cell_bwd)
  dropout   forward and backward of dropout with the one-bit feature map (echo_dropout_fwd, echo_dropout_bwd)
"""
import math

import torch

from paper_1805_08899_amd import binding as eb


def _attn(kind, name, B, Tq, Tk, H, Dv, dtype, key_lo, scale=0.5):
    return {"name": name, "kind": kind, "B": B, "Tq": Tq, "Tk": Tk, "H": H, "Dv": Dv, "dtype": dtype,
            "key_lo": key_lo, "scale": scale}


def listed():
    return [
        # the five workloads of workloads.py ---------------------------------------------------------------------
        # a toy model, a unit test, the last odd bucket of an epoch: latency and launches are all there is
        _attn("train", "train_tiny_f32", 4, 6, 7, 16, 16, "f32", 1),
        # the translation model's layer at its usual batch and sentence length (the headline benchmark)
        _attn("train", "train_nmt_f32", 64, 50, 50, 512, 512, "f32", 10),
        # the batch and sentence length that the saved memory makes room for
        _attn("train", "train_large_batch_f32", 128, 100, 100, 512, 512, "f32", 20),
        # long sequences of a wider model
        _attn("train", "train_long_f32", 32, 300, 300, 1024, 1024, "f32", 150, 0.3),
        # the wider model with its activations stored in bf16
        _attn("train", "train_wide_bf16", 128, 50, 50, 1024, 1024, "bf16", 5),
        # a bucket of uneven source and target lengths in a model whose width is no power of two
        _attn("train", "train_ragged_f32", 37, 61, 83, 300, 300, "f32", 9),
        # scoring a large batch of sentence pairs, forward only
        _attn("infer", "infer_large_batch_bf16", 256, 60, 60, 512, 512, "bf16", 10),
        # one step of a beam search: 16 sentences with a beam of 5
        _attn("step", "beam_step_f32", 80, 1, 100, 512, 512, "f32", 20),
        # the recurrent decoder's training pass at the translation model's shapes: 50 steps, 50 keys
        _attn("sentence", "decoder_sentence_f32", 64, 50, 50, 512, 512, "f32", 10),
        # one LSTM cell of the translation model, and the cells of a long unrolled or very large batch
        {"name": "lstm_cell_nmt", "kind": "lstm", "B": 128, "H": 512},
        {"name": "lstm_cell_large", "kind": "lstm", "B": 16384, "H": 1024},
        # dropout over the activations of a large layer
        {"name": "dropout_64Mi", "kind": "dropout", "n": 1 << 26, "p": 0.1},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# The tanh evaluations (B Tq Tk H, masked ones included) of the largest listed case, halved: shapes that take the
# slower paths (H not a multiple of four) then still cost less than that case.
_MOST_TANH = 32 * 300 * 300 * 1024 // 2


def draw(rng):
    kind = rng.choice(["train"] * 5 + ["infer"] * 2 + ["step"] * 2 + ["sentence"] + ["lstm"] * 2 + ["dropout"] * 2)
    if kind == "lstm":
        while True:
            c = {"kind": kind, "B": _log_int(rng, 1, 16384), "H": _log_int(rng, 16, 2048)}
            if rng.random() < 0.75:                          # hidden sizes are rarely odd
                c["H"] = (c["H"] + 3) // 4 * 4
            if c["B"] * c["H"] <= 16384 * 1024:
                return c
    if kind == "dropout":
        return {"kind": kind, "n": _log_int(rng, 1 << 10, 1 << 26), "p": rng.choice([0.1, 0.2, 0.3, 0.5])}
    while True:
        dtype = rng.choice(["f32", "f32", "bf16"])
        Tk = _log_int(rng, 4, 400)
        H = _log_int(rng, 32, 1024)
        if rng.random() < 0.75:
            H = (H + 3) // 4 * 4
        Dv = (H + 3) // 4 * 4 if rng.random() < 0.5 else (_log_int(rng, 16, 1024) + 3) // 4 * 4
        if kind == "step":
            B, Tq = _log_int(rng, 1, 512), 1
        elif kind == "sentence":
            B, Tq = _log_int(rng, 1, 128), _log_int(rng, 4, 60)
            Tk = min(Tk, 128)
        else:
            B, Tq = _log_int(rng, 1, 256), max(1, int(round(Tk * rng.uniform(0.6, 1.4))))
        key_lo = max(1, int(round(Tk * rng.choice([0.1, 0.2, 0.5, 1.0]))))
        if B * Tq * Tk * H <= _MOST_TANH:
            c = _attn(kind, "", B, Tq, Tk, H, Dv, dtype, key_lo)
            del c["name"]
            return c


# ---- inputs and buffers --------------------------------------------------------------------------------------------

class _State:
    """What the program keeps for one case: inputs, output buffers, descriptor, workspace."""


def _normal(gen, scale, *shape):
    return torch.randn(*shape, generator=gen, device="cuda") * scale


def _prepare_attn(case, gen):
    s = _State()
    B, Tq, Tk, H, Dv, dt = (case[k] for k in ("B", "Tq", "Tk", "H", "Dv", "dtype"))
    store = torch.bfloat16 if dt == "bf16" else torch.float32
    scale = case["scale"]
    s.Qp = _normal(gen, scale, B, Tq, H).to(store)
    s.Kp = _normal(gen, scale, B, Tk, H).to(store)
    s.V = _normal(gen, scale, B, Tk, Dv).to(store)
    if dt == "bf16":                                          # as in workload 4: a peaky softmax
        s.v = _normal(gen, scale, H).to(store)
    else:
        s.v = (torch.rand(H, generator=gen, device="cuda") * 2 - 1) / math.sqrt(H)
    s.key_len = torch.randint(case["key_lo"], Tk + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    f32 = dict(dtype=torch.float32, device="cuda")
    s.desc = eb.make_desc(B, Tq, Tk, H, Dv, dt)
    if case["kind"] == "sentence":
        s.desc_step = eb.make_desc(B, 1, Tk, H, Dv, dt)
        s.dC = _normal(gen, 1.0, B, Tq, Dv)
        # the decoder's own per-step tensors: queries as they come from its state, gradients as they come from its loss
        s.q = [s.Qp[:, t].contiguous() for t in range(Tq)]
        s.dc = [s.dC[:, t].contiguous() for t in range(Tq)]
        # what the steps write, one row per step (rows start 16-byte aligned)
        s.c_all, s.p_all, s.dq_all = (torch.zeros(Tq, (B * n + 3) // 4 * 4, **f32) for n in (Dv, Tk, H))
        s.c = [row[:B * Dv].view(B, 1, Dv) for row in s.c_all]
        s.p = [row[:B * Tk].view(B, 1, Tk) for row in s.p_all]
        s.dq = [row[:B * H].view(B, 1, H) for row in s.dq_all]
        s.p_by_sample = s.p_all[:, :B * Tk].view(Tq, B, Tk).transpose(0, 1)
        s.P = torch.empty(B, Tq, Tk, **f32)
        s.dKp, s.dV, s.dv = torch.empty(B, Tk, H, **f32), torch.empty(B, Tk, Dv, **f32), torch.empty(H, **f32)
        s.ds_rows = torch.empty(eb.echo_attn_steps_ds_bytes(s.desc), dtype=torch.uint8, device="cuda")
        ws = max(eb.echo_attn_fwd_workspace_bytes(s.desc_step), eb.echo_attn_bwd_workspace_bytes(s.desc), 16)
        s.ws = torch.empty(ws, dtype=torch.uint8, device="cuda")
        return s
    s.C, s.P = torch.empty(B, Tq, Dv, **f32), torch.empty(B, Tq, Tk, **f32)
    if case["kind"] == "step":
        return s
    ws = eb.echo_attn_fwd_workspace_bytes(s.desc)
    if case["kind"] == "train":
        s.dC = _normal(gen, 1.0, B, Tq, Dv)
        s.dQp, s.dKp = torch.empty(B, Tq, H, **f32), torch.empty(B, Tk, H, **f32)
        s.dV, s.dv = torch.empty(B, Tk, Dv, **f32), torch.empty(H, **f32)
        ws = max(ws, eb.echo_attn_bwd_workspace_bytes(s.desc))
    s.ws = torch.empty(max(ws, 16), dtype=torch.uint8, device="cuda")
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "lstm":
        s = _State()
        s.B, s.H = case["B"], case["H"]
        s.Gx, s.Gh = _normal(gen, 1.0, s.B, 4 * s.H), _normal(gen, 1.0, s.B, 4 * s.H)
        s.c_prev, s.dh, s.dc = (_normal(gen, 1.0, s.B, s.H) for _ in range(3))
        s.h, s.c, s.dc_prev = (torch.empty_like(s.c_prev) for _ in range(3))
        s.a, s.da = torch.empty_like(s.Gx), torch.empty_like(s.Gx)
    elif kind == "dropout":
        s = _State()
        s.n, s.p, s.seed = case["n"], case["p"], seed
        s.x, s.dy = _normal(gen, 1.0, s.n), _normal(gen, 1.0, s.n)
        s.y, s.dx = torch.empty_like(s.x), torch.empty_like(s.x)
        s.bits = torch.empty(eb.echo_dropout_mask_words(s.n), dtype=torch.int32, device="cuda")
    else:
        s = _prepare_attn(case, gen)
    s.kind = kind
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------

def _run_train(s, st):
    eb.check(eb.echo_attn_fwd(s.desc, s.Qp, s.Kp, s.V, s.v, s.key_len, s.C, s.P, s.ws, stream=st), "echo_attn_fwd")
    eb.check(eb.echo_attn_bwd(s.desc, s.dC, s.P, s.Qp, s.Kp, s.V, s.v, s.key_len, s.dQp, s.dKp, s.dV, s.dv, s.ws,
                              stream=st), "echo_attn_bwd")
    return {"context": s.C, "P": s.P, "dQp": s.dQp, "dKp": s.dKp, "dV": s.dV, "dv": s.dv}


def _run_infer(s, st):
    eb.check(eb.echo_attn_fwd(s.desc, s.Qp, s.Kp, s.V, s.v, s.key_len, s.C, s.P, s.ws, stream=st), "echo_attn_fwd")
    return {"context": s.C, "P": s.P}


def _run_step(s, st):
    eb.check(eb.echo_attn_step_fwd(s.desc, s.Qp, s.Kp, s.V, s.v, s.key_len, s.C, s.P, stream=st), "echo_attn_step_fwd")
    return {"context": s.C, "P": s.P}


def _run_sentence(s, st):
    steps = len(s.q)
    for t in range(steps):
        eb.check(eb.echo_attn_fwd(s.desc_step, s.q[t], s.Kp, s.V, s.v, s.key_len, s.c[t], s.p[t], s.ws, stream=st),
                 "echo_attn_fwd")
    for t in reversed(range(steps)):
        eb.check(eb.echo_attn_step_bwd_query(s.desc_step, t, steps, s.dc[t], s.p[t], s.q[t], s.Kp, s.V, s.v, s.key_len,
                                             s.dq[t], s.ds_rows, stream=st), "echo_attn_step_bwd_query")
    s.P.copy_(s.p_by_sample)                                  # [B, steps, Tk], as the call for the sentence takes it
    eb.check(eb.echo_attn_steps_bwd_keys(s.desc, s.dC, s.P, s.Qp, s.Kp, s.v, s.key_len, s.ds_rows, s.dKp, s.dV, s.dv,
                                         s.ws, stream=st), "echo_attn_steps_bwd_keys")
    return {"context": s.c_all, "P": s.P, "dQp": s.dq_all, "dKp": s.dKp, "dV": s.dV, "dv": s.dv}


def _run_lstm(s, st):
    eb.check(eb.echo_lstm_cell_fwd(s.B, s.H, s.Gx, s.Gh, s.c_prev, s.h, s.c, s.a, stream=st), "echo_lstm_cell_fwd")
    eb.check(eb.echo_lstm_cell_bwd(s.B, s.H, s.dh, s.dc, s.a, s.c_prev, s.da, s.dc_prev, stream=st),
             "echo_lstm_cell_bwd")
    return {"h": s.h, "c": s.c, "a": s.a, "da": s.da, "dc_prev": s.dc_prev}


def _run_dropout(s, st):
    eb.check(eb.echo_dropout_fwd(s.x, s.n, s.p, s.seed, 0, s.y, s.bits, stream=st), "echo_dropout_fwd")
    eb.check(eb.echo_dropout_bwd(s.dy, s.bits, s.n, s.p, s.dx, stream=st), "echo_dropout_bwd")
    return {"y": s.y, "bits": s.bits, "dx": s.dx}


_RUN = {"train": _run_train, "infer": _run_infer, "step": _run_step, "sentence": _run_sentence, "lstm": _run_lstm,
        "dropout": _run_dropout}


def run(state):
    return _RUN[state.kind](state, torch.cuda.current_stream())


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "lstm":
        n = case["B"] * case["H"]
        # forward reads Gx, Gh, c_prev and writes h, c, a; backward reads dh, dc, a, c_prev and writes da, dc_prev
        return {"bytes": 4 * n * (9 + 6 + 7 + 5), "flops": 60 * n}
    if kind == "dropout":
        return {"bytes": 2 * (8 * case["n"] + case["n"] // 8), "flops": 2 * case["n"]}
    B, Tq, Tk, H, Dv = (case[k] for k in ("B", "Tq", "Tk", "H", "Dv"))
    e = 2 if case["dtype"] == "bf16" else 4
    L = (case["key_lo"] + Tk) / 2                             # mean number of valid keys
    tanh = B * Tq * L * H
    # rows of masked keys need not be read; outputs are written whole
    k_in, v_in, q_in, p, c = B * L * H * e, B * L * Dv * e, B * Tq * H * e, B * Tq * Tk * 4, B * Tq * Dv * 4
    fwd = {"bytes": k_in + v_in + q_in + H * e + p + c, "flops": 9 * tanh + 2 * B * Tq * L * Dv}
    if kind in ("infer", "step"):
        return fwd
    bwd = {"bytes": c + B * Tq * L * 4 + k_in + v_in + q_in + 4 * (B * Tq * H + B * Tk * H + B * Tk * Dv + H),
           "flops": 18 * tanh + 4 * B * Tq * L * Dv}
    if kind == "sentence":                                    # keys and values pass through once per step and direction
        fwd["bytes"] += (Tq - 1) * (k_in + v_in)
        bwd["bytes"] += Tq * (k_in + v_in) - v_in + 2 * p
    return {k: fwd[k] + bwd[k] for k in fwd}


def tolerance(case):
    if case["kind"] == "dropout":
        return "exact"                                        # whole bits, and one rounded product per element
    if case["kind"] != "lstm" and case["dtype"] == "bf16":
        # fp32 arithmetic on bf16 inputs; v of order one makes scores of order ten out of sums whose terms add up to
        # hundreds in magnitude, so the exponentials carry a few 1e-5
        return {"rel": 3e-5}
    return {"rel": 1e-5}
