"""Attention scores beyond float32: an overflowed score leaves NaN behind, as inf - inf does in any softmax, and never
plausible values; one that overflowed to -inf weighs nothing.  Values beyond bf16: an infinite V reaches every query that
sees its key and no other.

The weights are steered so that token 0 is a key that every query of token 1 scores with 8 * a * b and nothing else is
scored at all; RoPE is the identity on the dimension used (its angle is below 1e-29)."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2404_08856_amd import synth
from tests.helpers import check_logits, oracle_cfg, to_device

pytestmark = pytest.mark.gpu

KEY, QUERY, PLAIN = 0, 1, 2                     # tokens


def steered(heads, a, key_b, query_b=0.0, layers=1, d=64):
    """Queries of QUERY: 8 a on one dimension; keys of KEY and QUERY: 8 key_b and 8 query_b on it, all others 0 (d = 128: 11.3 for 8)."""
    shape = synth.ModelShape(layers, d, heads, 64, 64, 64, rope_theta=1e30)
    w = synth.make_weights(shape, 3)
    w["embed"] = torch.zeros(64, d, dtype=torch.bfloat16)
    for t in range(64):
        w["embed"][t, min(t, 2)] = 1.0          # an RMS norm of 1 / 8: the normalised row is 8 on this dimension
    for lw in w["layers"]:
        lw["wq"].zero_()
        lw["wk"].zero_()
        for h in range(heads):
            lw["wq"][64 * h + 31, QUERY] = a
            lw["wk"][64 * h + 31, KEY] = key_b
            lw["wk"][64 * h + 31, QUERY] = query_b
    return shape, w


def prompt(n, at):
    ids = np.full(n, PLAIN, dtype=np.int32)
    ids[at] = KEY
    return ids


# one wave of keys; several units per wave; more pairs than slices; runs of keys (33 to 64 pairs, a long cache); two query groups
@pytest.mark.parametrize("n_seqs,heads,context,M", [(1, 1, 40, 1), (1, 2, 1500, 1), (2, 65, 200, 1), (5, 8, 900, 1), (1, 2, 1500, 6)])
@pytest.mark.parametrize("sign", [1, -1])
def test_cached_key_with_an_overflowed_score(n_seqs, heads, context, M, sign):
    from paper_2404_08856_amd import spd
    print(f"overflowed score: {n_seqs} x {heads} heads, context {context}, M {M}, sign {sign}", flush=True)
    shape, w = steered(heads, 1e19, sign * 1e19)            # 8e38: beyond float32's 3.4e38
    model = spd.Model(spd.make_config(shape, n_seqs, context + M), to_device(w))
    ids = prompt(context, context // 3)
    for s in range(n_seqs):
        model.spd_prefill_tokens(s, torch.from_numpy(ids).cuda())
    vt = torch.full((n_seqs, M), QUERY, dtype=torch.int32, device="cuda")
    out = torch.empty((n_seqs, M, shape.vocab), device="cuda")
    model.spd_verify_forward(vt, out)
    if sign > 0:
        assert torch.isnan(out).all()
        return
    cfg, wn = oracle_cfg(shape), synth.weights_to_numpy(w)
    cache = dec.KVCache(cfg, context + M)
    dec.forward_tokens(cfg, wn, cache, ids)
    want = dec.forward_tokens(cfg, wn, cache, np.full(M, QUERY, dtype=np.int32))
    for s in range(n_seqs):
        check_logits(out[s].cpu().numpy(), want, f"seq {s}")


@pytest.mark.parametrize("at,n", [(39, 40), (31, 48), (32, 33), (0, 40), (50, 150), (127, 200)])
def test_an_infinite_value_reaches_the_queries_that_see_it(at, n):
    """Two layers: keys and values of the second are finite before the row whose first-layer V overflows bf16, and not from there on."""
    from paper_2404_08856_amd import spd
    print(f"infinite value at {at} of {n}", flush=True)
    shape, w = steered(2, 0.0, 0.0, layers=2)
    w["layers"][0]["wv"][5, KEY] = 2.0 ** 127                   # times 8: one component of V is infinite
    model = spd.Model(spd.make_config(shape, 1, n), to_device(w))
    last = torch.empty(shape.vocab, device="cuda")
    model.spd_prefill_tokens(0, torch.from_numpy(prompt(n, at)).cuda(), last)
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(0, 0, 0, k, v)
    assert torch.isinf(v[at, 0, 5]) and torch.isinf(v).sum() == 1 and torch.isfinite(k).all()
    model.spd_kv_export(1, 0, 0, k, v)
    v = v.cpu().numpy()
    assert np.isfinite(v[:at]).all()
    assert (~np.isfinite(v[at:])).all()
    assert not torch.isfinite(last).any()


@pytest.mark.parametrize("n", [33, 40, 130])
@pytest.mark.parametrize("what", ["inf", "minus_inf", "all_very_low"])
def test_prompt_with_scores_of_any_size(n, what):
    """The last row's score of one key overflows, or every score of every row is near -1e31 (all values are equal then, so
    that the softmax of any such scores gives the value)."""
    from paper_2404_08856_amd import spd
    print(f"prompt of {n}, scores {what}", flush=True)
    if what == "all_very_low":
        shape, w = steered(2, 1.0, 0.0, query_b=-1.25e30)
        ids = np.full(n, QUERY, dtype=np.int32)
    else:
        shape, w = steered(2, 1e19, 1e19 if what == "inf" else -1e19)
        ids = prompt(n, n // 2)
        ids[-1] = QUERY
    model = spd.Model(spd.make_config(shape, 1, n), to_device(w))
    last = torch.empty(shape.vocab, device="cuda")
    model.spd_prefill_tokens(0, torch.from_numpy(ids).cuda(), last)
    if what == "inf":
        assert torch.isnan(last).all()
        return
    cfg, wn = oracle_cfg(shape), synth.weights_to_numpy(w)
    cache = dec.KVCache(cfg, n)
    check_logits(last.cpu().numpy(), dec.forward_tokens(cfg, wn, cache, ids)[-1], "last row")


@pytest.mark.parametrize("heads,n", [(1, 40), (2, 64), (2, 1500), (33, 130)])
def test_last_row_of_a_prompt_that_sees_an_infinite_key(heads, n):
    """A key that is infinite on a dimension where the queries are zero: the score is 0 * inf, and every row that sees the key is NaN, as in
    any softmax.  Values are finite everywhere, so nothing else makes it NaN."""
    from paper_2404_08856_amd import spd
    print(f"infinite key: {heads} heads, prompt of {n}", flush=True)
    shape, w = steered(heads, 1.0, 2.0 ** 126)              # times 8: beyond float32
    model = spd.Model(spd.make_config(shape, 1, n), to_device(w))
    last = torch.empty(shape.vocab, device="cuda")
    model.spd_prefill_tokens(0, torch.from_numpy(prompt(n, n // 3)).cuda(), last)
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(0, 0, 0, k, v)
    assert torch.isinf(k[n // 3]).any() and torch.isfinite(v).all()
    assert torch.isnan(last).all()


# d = 128: calls of up to 5 rows are one launch of all layers.  Slices of a head and runs of keys; one sequence among others
@pytest.mark.parametrize("n_seqs,heads,context,M", [(1, 1, 40, 1), (1, 2, 40, 5), (3, 2, 40, 1), (1, 2, 900, 1), (1, 2, 900, 5), (3, 2, 900, 1)])
@pytest.mark.parametrize("sign", [1, -1])
def test_overflowed_score_in_the_launch_of_all_layers(n_seqs, heads, context, M, sign):
    from paper_2404_08856_amd import spd
    print(f"overflowed score, one launch: {n_seqs} x {heads} heads, context {context}, M {M}, sign {sign}", flush=True)
    shape, w = steered(heads, 1e19, sign * 1e19, layers=2, d=128)
    model = spd.Model(spd.make_config(shape, n_seqs, context + M), to_device(w))
    asks = n_seqs // 2                                       # the sequence whose queries ask for the key
    for s in range(n_seqs):
        model.spd_prefill_tokens(s, torch.from_numpy(prompt(context, context // 3)).cuda())
    vt = torch.full((n_seqs, M), PLAIN, dtype=torch.int32, device="cuda")
    vt[asks] = QUERY
    outs = []
    for one_by_one in (0, 1):
        model.spd_model_set_tuning(separate_qkv_attention=one_by_one)
        model.spd_kv_set_len([context] * n_seqs)
        outs.append(torch.empty((n_seqs, M, shape.vocab), device="cuda"))
        model.spd_verify_forward(vt, outs[-1])
    model.spd_device_status()
    others = [s for s in range(n_seqs) if s != asks]
    for out in outs:
        assert torch.isfinite(out[others]).all()
        assert torch.isnan(out[asks]).all() if sign > 0 else torch.isfinite(out[asks]).all()
    if sign < 0:                                             # keys and values flip a rounding now and then
        assert float((outs[0] - outs[1]).norm()) <= 1e-4 * float(outs[1].norm())


@pytest.mark.parametrize("context", [40, 900])
@pytest.mark.parametrize("at", [0, 1, 4])
def test_infinite_value_in_the_launch_of_all_layers(context, at):
    """A new row whose first-layer V overflows bf16: finite and not finite where the separate kernels leave it so, and in every row from there on."""
    from paper_2404_08856_amd import spd
    print(f"infinite value, one launch: context {context}, row {at}", flush=True)
    shape, w = steered(2, 0.0, 0.0, layers=2, d=128)
    w["layers"][0]["wv"][5, KEY] = 2.0 ** 127
    model = spd.Model(spd.make_config(shape, 1, context + 5), to_device(w))
    model.spd_prefill_tokens(0, torch.full((context,), PLAIN, dtype=torch.int32, device="cuda"))
    vt = torch.full((1, 5), PLAIN, dtype=torch.int32, device="cuda")
    vt[0, at] = KEY
    seen = []
    for one_by_one in (0, 1):
        model.spd_model_set_tuning(separate_qkv_attention=one_by_one)
        model.spd_kv_set_len([context])
        out = torch.empty((1, 5, shape.vocab), device="cuda")
        model.spd_verify_forward(vt, out)
        k, v = (torch.empty((5, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
        model.spd_kv_export(0, 0, context, k, v)
        assert torch.isinf(v[at, 0, 5]) and torch.isinf(v).sum() == 1 and torch.isfinite(k).all()
        model.spd_kv_export(1, 0, context, k, v)
        assert not torch.isfinite(v[at:]).any() and not torch.isfinite(out[0, at:]).any()
        seen.append(torch.cat([torch.isfinite(x).flatten() for x in (k, v, out)]))
    assert torch.equal(*seen)
    model.spd_device_status()
