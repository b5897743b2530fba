"""GPU parity of long prompts of wide models (projections that contract over 2048 values or more, 385 rows and more, and fewer) against the
float64 oracle: both head sizes, K ranges that end inside a K-step, a second pass over a cached prefix, factors far from one; that no prompt
leaves anything behind for the next, and that every activation keeps its own 24 bits."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2404_08856_amd import synth
from tests.helpers import check_logits, oracle_cfg, randomize_gains, to_device
from tests.test_gpu_prefill import cached

pytestmark = pytest.mark.gpu

SHAPES = {
    "even": synth.ModelShape(2, 2048, 16, 128, 2048, 256),
    "ragged": synth.ModelShape(2, 2080, 33, 64, 2056, 256),               # 65, 66 and 64.25 K-steps; 257 gate|up tiles
    "ragged128": synth.ModelShape(2, 2144, 17, 128, 2120, 256),           # 67, 68 and 66.25
    "deep": synth.ModelShape(2, 2048, 16, 128, 4104, 128),                # down: 128.25 K-steps
}


def check_cache(model, cache, shape, n):
    """K and V are bf16 on both sides.  Layer 0: equal or one step apart, near zero float32 rounding.  Layer 1: a flipped step of one V
    component (2^-8 of up to 4 units) reaches early rows with a weight near 1, through Wo (0.02) and Wk (0.02, 2048 columns): 2^-8 * 4 *
    0.02 * 0.02 * sqrt(2048) = 2.8e-4 against values of 0.9; at 4 sigma and with room for a second flip 2e-3 of them."""
    for l in range(shape.n_layers):
        for got, want in zip(cached(model, l, n, shape), (cache.k[l][:n], cache.v[l][:n])):
            want = np.asarray(want, dtype=np.float64).reshape(got.shape)
            err = np.abs(got - want)
            floor = (1e-5 if l == 0 else 2e-3) * np.sqrt(np.mean(want * want))
            assert np.all(err <= np.maximum(2.0 ** -7 * np.abs(want), floor)), (l, err.max())
            assert np.mean(err > 0) < 0.02, (l, np.mean(err > 0))
            assert np.linalg.norm(err) <= 1e-3 * np.linalg.norm(want), (l, np.linalg.norm(err) / np.linalg.norm(want))


def run_prompt(shape, w, x, parts, capacity):
    """One sequence, the prompt in the given parts; checks the logits behind every part and the cache against the oracle."""
    from paper_2404_08856_amd import spd
    n = len(x)
    cfg, wn = oracle_cfg(shape), synth.weights_to_numpy(w)
    cache = dec.KVCache(cfg, n + 4)
    ref = dec.forward_rows(cfg, wn, cache, x)
    model = spd.Model(spd.make_config(shape, 1, capacity), to_device(w))
    rows = torch.from_numpy(x.astype(np.float32)).cuda()
    last = torch.empty(shape.vocab, device="cuda")
    at = 0
    for part in parts:
        model.spd_prefill(0, rows[at:at + part].contiguous(), last)
        at += part
        check_logits(last.cpu().numpy(), ref[at - 1], f"row {at}")
    assert at == n
    check_cache(model, cache, shape, n)


@pytest.mark.parametrize("name,parts", [
    ("even", (385,)), ("even", (384,)), ("even", (641, 400)), ("even", (1100,)),
    ("ragged", (385,)), ("ragged", (500, 40, 390)), ("ragged128", (449,)), ("ragged128", (1030,)), ("deep", (512,)),
])
def test_wide_prompts_against_oracle(name, parts):
    shape = SHAPES[name]
    print(f"wide {name} {parts}", flush=True)
    n = sum(parts)
    w = randomize_gains(synth.make_weights(shape, 5))
    run_prompt(shape, w, synth.image_rows(n, shape.d_model, 3).astype(np.float64), parts, n + 4)


def test_wide_prompt_with_factors_far_from_one():
    """Powers of two moved between gains and columns, query and key rows, up rows and down columns: the same function, but rows and blocks
    that differ by up to 2^80 in size, and columns inside one row by up to 2^16."""
    shape = SHAPES["even"]
    w = randomize_gains(synth.make_weights(shape, 6))
    g = torch.Generator().manual_seed(9)
    for lw in w["layers"]:
        for gain, mats in (("attn_norm", ("wq", "wk", "wv")), ("mlp_norm", ("w_gate", "w_up"))):
            p = 2.0 ** torch.randint(-8, 9, (shape.d_model,), generator=g)
            lw[gain] = (lw[gain].float() * p).to(lw[gain].dtype)
            for m in mats:
                lw[m] = (lw[m].float() / p).to(lw[m].dtype)
        lw["wq"] = (lw["wq"].float() * 2.0 ** 40).to(lw["wq"].dtype)
        lw["wk"] = (lw["wk"].float() * 2.0 ** -40).to(lw["wk"].dtype)
        p = 2.0 ** torch.randint(-8, 9, (shape.d_ffn,), generator=g)
        lw["w_up"] = (lw["w_up"].float() * p[:, None]).to(lw["w_up"].dtype)
        lw["w_down"] = (lw["w_down"].float() / p).to(lw["w_down"].dtype)
    run_prompt(shape, w, synth.image_rows(400, shape.d_model, 7).astype(np.float64), (400,), 404)


def test_wide_prompt_with_a_row_that_is_not_finite_and_a_zero_row():
    from paper_2404_08856_amd import spd
    shape = SHAPES["ragged"]
    w = to_device(synth.make_weights(shape, 11))
    rows = torch.from_numpy(synth.image_rows(400, shape.d_model, 12)).cuda()
    rows[20] = 0.0
    bad = rows.clone()
    bad[300, 5] = float("nan")
    bad[310, 7] = float("inf")
    kv = []
    for x in (rows, bad):
        m = spd.Model(spd.make_config(shape, 1, 400), w)
        last = torch.empty(shape.vocab, device="cuda")
        m.spd_prefill(0, x.contiguous(), last)
        kv.append((cached(m, 1, 400, shape), last.cpu()))
    (clean, last), (dirty, bad_last) = kv
    for a, b in zip(clean, dirty):
        assert np.isfinite(a).all() and np.array_equal(a[:300], b[:300]) and np.isnan(b[300:]).all()
    assert torch.isfinite(last).all() and torch.isnan(bad_last).all()


@pytest.mark.parametrize("first,second", [(40, 400), (400, 40), (384, 385), (640, 129)])
def test_a_prompt_behind_one_that_was_not_finite_has_the_bits_of_a_fresh_model(first, second):
    """d_ffn = 2056: the last K-step of the down projection is a quarter full.  Whatever a prompt of another length left in the buffers, the
    columns that pad that step count as zero: 0 * NaN would reach every later row."""
    from paper_2404_08856_amd import spd
    shape = SHAPES["ragged"]
    w = to_device(synth.make_weights(shape, 19))
    bad = torch.from_numpy(synth.image_rows(first, shape.d_model, 20)).cuda()
    bad[:, 3] = float("nan")
    rows = torch.from_numpy(synth.image_rows(second, shape.d_model, 21)).cuda()
    outs = []
    for dirty in (False, True):
        m = spd.Model(spd.make_config(shape, 1, 700), w)
        last = torch.empty(shape.vocab, device="cuda")
        if dirty:
            m.spd_prefill(0, bad.contiguous(), last)
            assert torch.isnan(last).all()
            m.spd_kv_set_len([0])
        m.spd_prefill(0, rows, last)
        outs.append([last.cpu().numpy()] + [x for l in range(shape.n_layers) for x in cached(m, l, second, shape)])
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("n", [100, 384, 385, 640])
def test_a_column_without_weights_takes_no_bits_from_its_neighbours(n):
    """Every activation keeps its own 24 bits, whatever stands next to it: a column whose weights are zero changes no bit of the result, also where
    its gain makes it 2^40 times as large as the others."""
    from paper_2404_08856_amd import spd
    shape = SHAPES["even"]
    w = randomize_gains(synth.make_weights(shape, 22))
    columns = torch.arange(5, shape.d_model, 64)                # two in every block of 128
    for lw in w["layers"]:
        for m in ("wq", "wk", "wv", "w_gate", "w_up"):
            lw[m][:, columns] = 0
    rows = torch.from_numpy(synth.image_rows(n, shape.d_model, 23)).cuda()
    outs = []
    for size in (1.0, 2.0 ** 40):
        for lw in w["layers"]:
            lw["attn_norm"][columns] = size
            lw["mlp_norm"][columns] = size
        m = spd.Model(spd.make_config(shape, 1, n), to_device(w))
        last = torch.empty(shape.vocab, device="cuda")
        m.spd_prefill(0, rows, last)
        outs.append([last.cpu().numpy()] + [x for l in range(shape.n_layers) for x in cached(m, l, n, shape)])
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_the_last_position_s_keys_and_values_do_not_depend_on_the_logits():
    """16 last rows of 4096 values per layer: about one in 10^4 lies so close to a rounding boundary of bf16 that another order of the sums takes
    it to the other side."""
    from paper_2404_08856_amd import spd
    shape = SHAPES["even"]
    m = spd.Model(spd.make_config(shape, 1, 64), to_device(randomize_gains(synth.make_weights(shape, 24))))
    rows = torch.from_numpy(synth.image_rows(64, shape.d_model, 25)).cuda()
    last = torch.empty(shape.vocab, device="cuda")
    for n in range(33, 49):
        kv = []
        for logits in (None, last):
            m.spd_kv_set_len([0])
            m.spd_prefill(0, rows[:n].contiguous(), logits)
            kv.append([x for l in range(shape.n_layers) for x in cached(m, l, n, shape)])
        for a, b in zip(*kv):
            assert np.array_equal(a, b), n


def o_model(layers):
    """The O projection alone: no queries (one token repeated: attention returns the cached value), no MLP, an LM head that hands the
    normalised row through.  Of two layers the second adds nothing: the prompt kernels' O.  One layer: the last row's."""
    from paper_2404_08856_amd import spd
    shape = synth.ModelShape(layers, 4096, 32, 128, 64, 4096)
    w = to_device(synth.make_weights(shape, 26))
    w["embed"] = (0.01 * w["embed"].float()).to(torch.bfloat16)
    w["lm_head"] = torch.eye(4096, device="cuda").to(torch.bfloat16)
    w["layers"][0]["wq"].zero_()
    w["layers"][-1]["wo"].mul_(0 if layers > 1 else 1)
    for lw in w["layers"]:
        lw["w_down"].zero_()
    return shape, w, spd.Model(spd.make_config(shape, 1, 384), w)


def o_error(shape, w, m, n):
    """Relative error of the O projection over prompts of n equal tokens, 16 tokens."""
    last = torch.empty(shape.vocab, device="cuda")
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    square = 0.0
    for token in range(16):
        m.spd_kv_set_len([0])
        m.spd_prefill_tokens(0, torch.full((n,), token, dtype=torch.int32, device="cuda"), last)
        m.spd_kv_export(0, 0, 0, k, v)
        assert (v == v[0]).all()
        x = w["embed"][token].double() + w["layers"][0]["wo"].double() @ v[0].reshape(-1).double()
        want = x / torch.sqrt(x.square().mean() + shape.rms_eps)
        got = last.double()
        got = got * ((got * want).sum() / got.square().sum())       # the row's common factor is not the sums' error
        square += ((got - want).square().sum() / want.square().sum()).item()
    return (square / 16) ** 0.5


def test_a_prompt_s_sums_are_as_exact_in_few_slices_as_in_many():
    """64 rows take 6 slices of K, 384 rows 2.  Chains of additions of independent roundings: the errors go with the square root of
    their lengths, 22 / 4 + 6 additions next to the products' own (about 4 additions' worth for each of 4) and 64 / 4 + 2 (11 %
    more) or, with sums of 16 steps in between, 4 + 4 + 2.  65536 errors tell the ratio to 0.4 %."""
    shape, w, m = o_model(2)
    many, few = o_error(shape, w, m, 64), o_error(shape, w, m, 384)
    print(f"O of a prompt: 64 rows {many:.3e}, 384 rows {few:.3e}", flush=True)
    assert few <= 1.05 * many


@pytest.mark.parametrize("n", [40, 384])
def test_the_last_row_s_sums_are_as_exact_as_the_other_rows(n):
    """The last row goes through its layer by the kernels of single rows: 8 waves of 16 K-steps, each with sums of 4, in the end 4 + 8
    additions next to the products' own, as many as a prompt of few rows has.  In chains of 16 the products' own errors alone
    would be half as large again."""
    others, last = (o_error(*o_model(layers), n) for layers in (2, 1))
    print(f"O at {n} rows: others {others:.3e}, last {last:.3e}", flush=True)
    assert last <= 1.1 * others
