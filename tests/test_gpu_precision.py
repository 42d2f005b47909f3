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
