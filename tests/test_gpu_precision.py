"""Rounding errors of the scores where a careless order of the same operations would lose digits, against float64 with a bound
that counts the roundings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -24                                                # half a unit in the last place, relative


def _check_probabilities(P, S, H, terms, sums, key_len, name):
    """P against the softmax of the float64 scores S [B, Tq, Tk].  A score is off by at most U (10 terms + n sums): `terms` = sum of
    |v| over the entries whose tanh is rounded at all, 10 U its error (exponent 3 U |x| with |x| (1 - tanh^2) <= 0.45, exponential
    and reciprocal one ulp each, the sum with one and the final subtraction half an ulp, the last three doubled by 2 r); `sums` = sum
    of |v tanh|, n the additions that a term passes through.  The softmax: its own exponent, exponential, sum and division."""
    n = H / 64 + 10
    worst = 0.0
    for b, L in enumerate(key_len):
        s = S[b, :, :L] - S[b, :, :L].max(-1, keepdims=True)
        e = np.exp(s)
        ref = e / e.sum(-1, keepdims=True)
        err_s = U * (10 * terms + n * sums[b, :, :L].max())
        bound = 2 * err_s + U * (2 * np.abs(s) + L / 64 + 20)
        on = ref > 1e-25
        off = np.abs(np.log(P[b, :, :L].astype(np.float64)[on] / ref[on])) / bound[on]
        worst = max(worst, off.max())
    print(f"{name}: largest error / bound {worst:.3f}", flush=True)
    assert worst <= 1, (name, worst)


STEPS = [
    # name, B, Tk, H, entry point: one batch of rows and columns, several, rows of fewer than four elements, few keys in eight waves, four blocks a
    # sample
    ("one_batch", 3, 20, 48, "step"),
    ("several_batches", 2, 150, 600, "step"),
    ("narrow_rows", 3, 40, 3, "step"),
    ("few_keys", 3, 6, 45, "step"),
    ("four_blocks", 3, 20, 48, "fwd"),
]


@pytest.mark.parametrize("case", STEPS, ids=[c[0] for c in STEPS])
def test_step_scores_of_operands_that_cancel(case):
    """Queries of a few thousand against keys that cancel them up to order one, and terms that cancel to exactly zero under weights
    a thousand times those of the others: the error must follow q + k and v tanh."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb
    name, B, Tk, H, entry = case
    print("step precision", case, flush=True)
    rng = np.random.default_rng(5 + H)
    q = ((2048 + 1500 * rng.random((B, 1, H))) * rng.choice([-1, 1], (B, 1, H))).astype(np.float32)
    k = (0.7 * rng.standard_normal((B, Tk, H)) - q).astype(np.float32)
    v = (0.3 * rng.standard_normal(H)).astype(np.float32)
    exact = np.arange(H) >= (H + 1) // 2                      # these columns add nothing
    k[:, :, exact] = -q[:, :, exact]
    v[exact] *= 1000
    key_len = np.full(B, Tk, dtype=np.int32)
    key_len[0] = max(1, Tk - 3)
    t = np.tanh(q.astype(np.float64) + k)                     # [B, Tk, H]
    S = (t * v).sum(-1)[:, None, :]
    sums = np.abs(t * v).sum(-1)[:, None, :]
    terms = float(np.abs(v[~exact]).sum())

    up = lambda x: torch.from_numpy(x).cuda()
    V = torch.randn(B, Tk, 8, device="cuda")
    ctx, P = torch.empty(B, 1, 8, device="cuda"), torch.full((B, 1, Tk), float("nan"), device="cuda")
    desc = eb.make_desc(B, 1, Tk, H, 8, "f32")
    st = torch.cuda.current_stream()
    if entry == "step":
        eb.check(eb.echo_attn_step_fwd(desc, up(q), up(k), V, up(v), up(key_len), ctx, P, stream=st))
    else:
        ws = torch.empty(eb.echo_attn_fwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        eb.check(eb.echo_attn_fwd(desc, up(q), up(k), V, up(v), up(key_len), ctx, P, ws, stream=st))
    _check_probabilities(P.cpu().numpy(), S, H, terms, sums, key_len, name)


@pytest.mark.parametrize("shape", [(2, 40, 70, 1001), (40, 64, 66, 1001), (3, 20, 20, 1001)],
                         ids=["four_rows", "eight_rows", "row_mode"])
def test_forward_scores_of_small_terms_at_odd_h(shape):
    """Equal weights and tanh terms of a few hundredths: the scores are small against sum_h v / (exp(2 (q + k)) + 1), half of sum |v|.
    Added over the lanes, sums of that size are rounded at 250 to 500 (1.5e-5 per addition); with the constant half taken off per
    lane first, what is left are roundings of the terms (about 3 U each, sqrt(1001) of them) and of sums up to 8 within a lane
    (half a unit 4.8e-7 each, sqrt(500) of them in all), doubled: 2 (6e-6 + 6e-6) if all errors were at their limits, and about half of
    that as a root mean square."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb
    B, Tq, Tk, H = shape
    print("odd H precision", shape, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    q, k = (0.02 * torch.randn(B, T, H, generator=g, device="cuda") for T in (Tq, Tk))
    v, V = torch.ones(H, device="cuda"), torch.randn(B, Tk, 4, generator=g, device="cuda")
    key_len = torch.full((B,), Tk, dtype=torch.int32, device="cuda")
    ctx, P = torch.empty(B, Tq, 4, device="cuda"), torch.empty(B, Tq, Tk, device="cuda")
    desc = eb.make_desc(B, Tq, Tk, H, 4, "f32")
    ws = torch.empty(eb.echo_attn_fwd_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    eb.check(eb.echo_attn_fwd(desc, q, k, V, v, key_len, ctx, P, ws, stream=torch.cuda.current_stream()))
    off = torch.stack([P[b].double().log() - torch.tanh(q[b].double()[:, None] + k[b].double()).sum(-1) for b in range(min(B, 4))])
    rms = float((off - off.mean(-1, keepdim=True)).square().mean().sqrt())
    print(f"root mean square of the score errors {rms:.2e}", flush=True)
    assert rms <= 1.2e-5, rms


# recomputation with up to 25 rows per lane, one pass over the rows (two lane groups and one) and two
LARGE = [
    # name, B, Tq, Tk, H, Dv, dtype
    ("two_groups", 57, 100, 100, 512, 16, "f32"),
    ("two_groups_bf16", 64, 72, 72, 512, 16, "bf16"),
    ("one_group", 30, 150, 90, 1024, 16, "f32"),
    ("two_passes", 30, 240, 60, 1024, 16, "f32"),
]


def _gradients_in_float64(dC, P, Q, K, V, v, key_len):
    """dQp, dKp and dv from the given P, sample by sample."""
    import torch
    B, Tq, H = Q.shape
    out = {"dQp": [], "dKp": [], "dv": 0.0}
    for b in range(B):
        L = int(key_len[b])
        p, q, k = P[b, :, :L].double(), Q[b].double(), K[b, :L].double()
        dP = dC[b].double() @ V[b, :L].double().t().contiguous()
        dS = (p * (dP - (p * dP).sum(1, keepdim=True)))[:, :, None]
        t = torch.tanh(q[:, None] + k)
        g = dS * (1 - t * t) * v.double()
        out["dQp"].append(g.sum(1))
        dk = g.new_zeros(K.shape[1], H)
        dk[:L] = g.sum(0)
        out["dKp"].append(dk)
        out["dv"] = out["dv"] + (dS * t).sum((0, 1))
    return {k: torch.stack(x) if k != "dv" else x for k, x in out.items()}


class _Backward:
    """Inputs and buffers of a backward whose columns `hit` have weight zero, so that what stands there has no part in P."""

    def __init__(self, case):
        import torch
        from paper_1805_08899_amd import binding as eb
        name, self.B, self.Tq, self.Tk, self.H, self.Dv, dt = case
        g = torch.Generator(device="cuda")
        g.manual_seed(23)
        store = torch.bfloat16 if dt == "bf16" else torch.float32
        draw = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
        self.Q, self.K = ((0.5 * draw(self.B, T, self.H)).to(store) for T in (self.Tq, self.Tk))
        self.V, self.dC = draw(self.B, self.Tk, self.Dv).to(store), draw(self.B, self.Tq, self.Dv)
        self.v = (draw(self.H) / self.H ** 0.5).to(store)
        self.hit = torch.arange(5, self.H, 64, device="cuda")           # one column of every block's 64
        self.v[self.hit] = 0
        self.key_len = torch.full((self.B,), self.Tk, dtype=torch.int32, device="cuda")
        self.key_len[::3] = self.Tk - 5
        self.desc, new = eb.make_desc(self.B, self.Tq, self.Tk, self.H, self.Dv, dt), lambda *s: torch.empty(*s, device="cuda")
        self.P, self.C = new(self.B, self.Tq, self.Tk), new(self.B, self.Tq, self.Dv)
        self.dQ, self.dK, self.dV, self.dv = new(*self.Q.shape), new(*self.K.shape), new(*self.V.shape), new(self.H)
        need = max(eb.echo_attn_fwd_workspace_bytes(self.desc), eb.echo_attn_bwd_workspace_bytes(self.desc), 16)
        self.ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        eb.check(eb.echo_attn_fwd(self.desc, self.Q, self.K, self.V, self.v, self.key_len, self.C, self.P, self.ws,
                                  stream=torch.cuda.current_stream()))

    def put(self, what):
        """Entries beyond the factor limit in the columns `hit` of every sample."""
        if what == "queries":
            self.Q[:, self.Tq // 2, self.hit] = 44.0
        else:
            self.K[:, 1, self.hit] = -44.0

    def run(self):
        import torch
        from paper_1805_08899_amd import binding as eb
        eb.check(eb.echo_attn_bwd(self.desc, self.dC, self.P, self.Q, self.K, self.V, self.v, self.key_len, self.dQ, self.dK, self.dV,
                                  self.dv, self.ws, stream=torch.cuda.current_stream()))

    def errors(self):
        """Error of each gradient relative to its norm, over the columns that hold ordinary entries."""
        import torch
        ref = _gradients_in_float64(self.dC, self.P, self.Q, self.K, self.V, self.v, self.key_len)
        on = torch.ones(self.H, dtype=torch.bool, device="cuda")
        on[self.hit] = False
        self.run()
        got = {"dQp": self.dQ, "dKp": self.dK, "dv": self.dv}
        return {k: float((got[k].double() - r)[..., on].norm() / r[..., on].norm()) for k, r in ref.items()}


@pytest.mark.parametrize("what", ["queries", "keys"])
@pytest.mark.parametrize("case", LARGE, ids=[c[0] for c in LARGE])
def test_large_entries_add_no_error(case, what):
    """Entries beyond the factor limit send their neighbours' evaluations through the exponential of the sum: one rounding of the
    exponent in place of two roundings of exponentials and one of a product, and the same sums in the same order, so the error
    against float64 stays what it is without them.  1.25 times: the ratio of two root mean squares over at least 448 columns strays by
    1 / sqrt(448), 5 %."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    print("large entries", case, what, flush=True)
    run = _Backward(case)
    without = run.errors()
    run.put(what)
    withal = run.errors()
    print({k: f"{without[k]:.2e} -> {withal[k]:.2e}" for k in without}, flush=True)
    assert all(withal[k] <= 1.25 * without[k] for k in without), (without, withal)


def _best_time(run):
    """Milliseconds of one backward, the best of eight short measurements."""
    import torch
    times = []
    for _ in range(8):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        run.run()
        a.record()
        for _ in range(5):
            run.run()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / 5)
    return min(times)


@pytest.mark.parametrize("what", ["queries", "keys"])
@pytest.mark.parametrize("case", LARGE, ids=[c[0] for c in LARGE])
def test_large_entries_cost_little(case, what):
    """What an evaluation costs more there is an exponential and an addition beside a reciprocal and five plain instructions: at most
    1.6 times the backward (an eighth or less of the time lies elsewhere).  Twice: for the noise of a short measurement; evaluations one by
    one from memory took 3 to 6 times."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    print("time with large entries", case, what, flush=True)
    run = _Backward(case)

    without = _best_time(run)
    run.put(what)
    withal = _best_time(run)
    print(f"{1e3 * without:.1f} -> {1e3 * withal:.1f} us", flush=True)
    assert withal <= 2 * without, (without, withal)


PRE = [
    # name, B, Tq, Tk, Dv, dtype: up to 64, 128 and more keys on split operands
    ("64_keys", 70, 60, 60, 516, "f32"),
    ("64_keys_bf16", 70, 60, 60, 516, "bf16"),
    ("128_keys", 40, 100, 100, 516, "f32"),
    ("300_keys", 20, 300, 300, 260, "f32"),
]


def _backward(B, Tq, Tk, Dv, dt, change=None, change_P=None):
    """P and the gradients of a batch of full samples; change(dC, V) and change_P(P) edit them before the backward pass."""
    import torch
    from paper_1805_08899_amd import binding as eb
    H = 32
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    store = torch.bfloat16 if dt == "bf16" else torch.float32
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v, V = (x.to(store) for x in (rand(B, Tq, H), rand(B, Tk, H), rand(H), rand(B, Tk, Dv)))
    dC = rand(B, Tq, Dv)
    key_len = torch.full((B,), Tk, dtype=torch.int32, device="cuda")
    out = {n: torch.empty(*s, device="cuda") for n, s in (("C", (B, Tq, Dv)), ("P", (B, Tq, Tk)), ("dQp", (B, Tq, H)), ("dKp", (B, Tk, H)),
                                                          ("dV", (B, Tk, Dv)), ("dv", (H,)))}
    desc = eb.make_desc(B, Tq, Tk, H, Dv, dt)
    ws = torch.empty(max(16, eb.echo_attn_fwd_workspace_bytes(desc), eb.echo_attn_bwd_workspace_bytes(desc)), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream()
    eb.check(eb.echo_attn_fwd(desc, q, k, V, v, key_len, out["C"], out["P"], ws, stream=st))
    if change:
        change(dC, V)
    if change_P:
        change_P(out["P"])
    eb.check(eb.echo_attn_bwd(desc, dC, out["P"], q, k, V, v, key_len, out["dQp"], out["dKp"], out["dV"], out["dv"], ws, stream=st))
    torch.cuda.synchronize()
    return {n: x.cpu() for n, x in out.items()}, dC.cpu(), V.cpu(), q.cpu(), k.cpu(), v.cpu()


def _errors_of_products(out, dC, V, q, k, v):
    """Relative errors of dV and dQp of the first four samples against float64."""
    import torch
    P, dC, V, q, k, v = (x[:4].double() if x.dim() > 1 else x.double() for x in (out["P"], dC, V, q, k, v))
    rel = lambda got, ref: float((got.double() - ref).norm() / ref.norm())
    e_dv = rel(out["dV"][:4], P.transpose(1, 2) @ dC)
    dP = dC @ V.transpose(1, 2)
    dS = P * (dP - (P * dP).sum(-1, keepdim=True))
    dQ = torch.stack([(dS[b, :, :, None] * (1 - torch.tanh(q[b, :, None] + k[b, None]) ** 2)).sum(1) * v for b in range(4)])
    return e_dv, rel(out["dQp"][:4], dQ)


FEW = [
    # on 51 to 100 blocks of 32 rows, 200 of wide value rows
    ("300_keys_100_blocks", 10, 300, 300, 260, "f32"),
    ("300_keys_100_blocks_bf16", 10, 300, 300, 260, "bf16"),
    ("300_keys_200_blocks", 20, 300, 300, 516, "f32"),
    ("150_keys_52_blocks", 26, 64, 150, 132, "f32"),
]


@pytest.mark.parametrize("case", PRE + FEW, ids=[c[0] for c in PRE + FEW])
def test_split_products_are_no_worse_than_fp32_ones(case):
    """The same samples where the products are fp32 ones: up to 128 keys four of them alone, which make fewer than 64 blocks of 32 rows, in fp32
    storage, which holds bf16 values as they are; beyond, all of them with masked keys up to 516 or, where up to 200 blocks ran in parts
    before they ran on split operands, four of them alone, which still do (on one chain of products the errors were 1.6 times those of the
    parts).  Queries and keys are zero, so that dKp[j] = v
    sum_i dS[i,j] shows dP.  The errors are root mean squares over 15 thousand elements for dV, which are 1 % apart by chance, but 240 and more for
    dKp, 5 %: 3 and 15 % allowed.  (dV over 60 rows 1.1e-7 against 1.4e-7.)"""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    from paper_1805_08899_amd import binding as eb
    name, B, Tq, Tk, Dv, dt = case
    print("split and fp32 products", case, flush=True)
    H = 32
    g = torch.Generator(device="cuda")
    g.manual_seed(29)
    V = torch.randn(B, Tk, Dv, generator=g, device="cuda").to(torch.bfloat16 if dt == "bf16" else torch.float32)
    dC = torch.randn(B, Tq, Dv, generator=g, device="cuda")
    P = torch.softmax(torch.randn(B, Tq, Tk, generator=g, device="cuda"), -1)
    errors = {}
    for form in ("split", "fp32"):
        n, keys = (4, Tk) if form == "fp32" and (Tk <= 128 or case in FEW) else (B, Tk if form == "split" else 516)
        store = dt if form == "split" else "f32"
        kind = torch.bfloat16 if store == "bf16" else torch.float32
        zero = lambda *s: torch.zeros(*s, dtype=kind, device="cuda")
        q, k, v = zero(n, Tq, H), zero(n, keys, H), zero(H) + 1
        values, p_in = zero(n, keys, Dv), torch.zeros(n, Tq, keys, device="cuda")
        values[:, :Tk], p_in[:, :, :Tk] = V[:n], P[:n]
        key_len = torch.full((n,), Tk, dtype=torch.int32, device="cuda")
        dQ, dK, dV, dv = (torch.empty(*s, device="cuda") for s in ((n, Tq, H), (n, keys, H), (n, keys, Dv), (H,)))
        desc = eb.make_desc(n, Tq, keys, H, Dv, store)
        ws = torch.empty(max(16, eb.echo_attn_bwd_workspace_bytes(desc)), dtype=torch.uint8, device="cuda")
        eb.check(eb.echo_attn_bwd(desc, dC[:n].contiguous(), p_in, q, k, values, v, key_len, dQ, dK, dV, dv, ws,
                                  stream=torch.cuda.current_stream()))
        torch.cuda.synchronize()
        p, c, x = (t[:4].cpu().double() for t in (P, dC, V))
        dP = c @ x.transpose(1, 2)
        want = (p * (dP - (p * dP).sum(-1, keepdim=True))).sum(1)
        rel = lambda got, ref: float((got.cpu().double() - ref).norm() / ref.norm())
        errors[form] = rel(dV[:4, :Tk], p.transpose(1, 2) @ c), rel(dK[:4, :Tk, 0], want)
    print(name, {f: [f"{e:.2e}" for e in v] for f, v in errors.items()}, flush=True)
    for split, fp32, most in zip(errors["split"], errors["fp32"], (1.03, 1.15)):
        assert split <= most * fp32, errors


@pytest.mark.parametrize("case", PRE, ids=[c[0] for c in PRE])
def test_error_of_products_of_split_operands(case):
    """dV = P^T dC and, through dQp, dP = dC V^T as six products of bf16 parts.  dV, a sum of n terms: six roundings of the partial sum per 16
    terms, each off by U / sqrt(3) of it (root mean square), the partial sums sqrt(1/2) of the result on average: U sqrt(n / 16), twice that
    allowed; fp32 products without parts, 16 roundings per 16 terms, would be at 1.6.  dQp also has the roundings of the recomputation; 2e-6
    is what its own tests allow."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    name, B, Tq, Tk, Dv, dt = case
    print("split operands", case, flush=True)
    out, dC, V, q, k, v = _backward(B, Tq, Tk, Dv, dt)
    e_dv, e_dq = _errors_of_products(out, dC, V, q, k, v)
    print(f"{name}: dV {e_dv:.2e}, dQp {e_dq:.2e}", flush=True)
    assert e_dv <= 2 * U * (Tq / 16 + 1) ** 0.5, e_dv
    assert e_dq <= 2e-6, e_dq


@pytest.mark.parametrize("what", ["gradients", "values", "probabilities", "one_key"])
@pytest.mark.parametrize("case", PRE, ids=[c[0] for c in PRE])
def test_small_operands_lose_no_digits(case, what):
    """Operands of 1e-35 and below: their bf16 parts are below what bf16 holds, unless they are scaled.  Bounds of
    test_error_of_products_of_split_operands; all scales are powers of two, and the results stay normal numbers."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    name, B, Tq, Tk, Dv, dt = case
    print("small operands", case, what, flush=True)
    scales = {"gradients": (-119, 8, 0), "values": (90, -119, 0)}.get(what, (0, 0, -115))           # of dC, V, P

    def change(dC, V):
        dC.mul_(2.0 ** scales[0])
        V.mul_(2.0 ** scales[1])

    def change_P(P):
        (P[:, :, 1] if what == "one_key" else P).mul_(2.0 ** scales[2])

    out, dC, V, q, k, v = _backward(B, Tq, Tk, Dv, dt, change, change_P)
    dv_bound = 2 * U * (Tq / 16 + 1) ** 0.5
    if what == "one_key":
        want = out["P"][:, :, 1:2].double().transpose(1, 2) @ dC.double()
        e_dv = float((out["dV"][:, 1:2].double() - want).norm() / want.norm())
    else:
        e_dv, e_dq = _errors_of_products(out, dC, V, q, k, v)
    print(f"{name} {what}: dV {e_dv:.2e}", flush=True)
    assert e_dv <= dv_bound, e_dv
    if what in ("gradients", "values"):
        print(f"dQp {e_dq:.2e}", flush=True)
        assert e_dq <= 2e-6, e_dq


@pytest.mark.parametrize("case", PRE, ids=[c[0] for c in PRE])
def test_operands_that_do_not_split(case):
    """Infinities and the largest finite numbers have no bf16 parts: an infinite dC makes its column of dV infinite, and its row of dQp and
    the sample's dKp no numbers, as in fp32; the largest finite dC gives the fp32 products; everything else stays what it was."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    name, B, Tq, Tk, Dv, dt = case
    print("operands that do not split", case, flush=True)
    plain = _backward(B, Tq, Tk, Dv, dt)[0]
    top = float(np.finfo(np.float32).max)
    i, d = Tq - 1, Dv - 3

    def change(dC, V):
        dC[0, i, d] = float("inf")
        V[0, :, d] = 1.0                                      # (after the forward pass: only the backward pass sees it)
        dC[1, i, d] = top
        V[1, :, d] = 0.0

    out, dC = _backward(B, Tq, Tk, Dv, dt, change)[:2]
    assert torch.isinf(out["dV"][0, :, d]).all()
    rest = torch.ones(Dv, dtype=torch.bool)
    rest[d] = False
    for b in (0, 1):
        assert torch.allclose(out["dV"][b][:, rest], plain["dV"][b][:, rest], rtol=0, atol=4e-5)
    assert torch.isnan(out["dQp"][0, i]).all() and torch.isfinite(out["dQp"][0, :i]).all()
    assert torch.isnan(out["dKp"][0]).all() and torch.isnan(out["dv"]).all()
    want = out["P"][1].double().T @ dC[1, :, d].double()
    assert float(((out["dV"][1, :, d].double() - want) / want).abs().max()) <= 1e-5
    for n in ("dQp", "dKp"):
        assert torch.isfinite(out[n][1]).all()
    for n in ("dQp", "dKp", "dV"):
        assert torch.equal(out[n][2:], plain[n][2:]), n


NOT_FINITE = [
    ("50_keys", 64, 50, 50, 512, 512, "f32"),
    ("50_keys_bf16", 128, 50, 50, 1024, 1024, "bf16"),
    ("100_keys", 64, 64, 100, 512, 768, "f32"),
    ("300_keys", 32, 300, 300, 256, 1024, "f32"),
    ("300_keys_bf16", 32, 300, 300, 256, 1024, "bf16"),
]


@pytest.mark.parametrize("what", ["one_row", "all", "values"])
@pytest.mark.parametrize("case", NOT_FINITE, ids=[c[0] for c in NOT_FINITE])
def test_operands_that_do_not_split_cost_little(case, what):
    """Products formed again in fp32, as after a loss that overflowed.  They take about 1.8 times what split ones do (134 against 76 us for 300 keys
    of 1024 columns), in addition to these, on up to half of the backward here: up to 1.9 times the time.  With one trip to memory per two
    columns, as it was first done, 1.7 to 3 times."""
    import torch
    assert torch.cuda.is_available(), "needs the GPU"
    print("time with infinities", case, what, flush=True)
    run = _Backward(case)
    without = _best_time(run)
    if what == "all":
        run.dC.fill_(float("nan"))
    elif what == "one_row":
        run.dC[:, run.Tq // 2, 3] = float("inf")
    else:
        run.V[:, 0, 5] = float("inf")
    withal = _best_time(run)
    print(f"{1e3 * without:.1f} -> {1e3 * withal:.1f} us", flush=True)
    assert withal <= 2 * without, (without, withal)
