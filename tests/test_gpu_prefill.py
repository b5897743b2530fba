"""GPU parity of the prefill passes (many rows of one sequence per pass) against the float64 oracle: row counts around
the edges of the row tiles, workgroup tiles, slices of K and key units, a second pass on top of a cached prefix, ragged d_ffn,
both head sizes, the KV cache it leaves and the decode step that follows."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2404_08856_amd import synth
from tests.helpers import check_logits, oracle_cfg, randomize_gains, to_device

pytestmark = pytest.mark.gpu

SHAPES = {
    "dh64_ragged_ffn": synth.ModelShape(2, 256, 4, 64, 688, 1024),        # 43 / 2 K-steps: the last one half empty
    "dh128": synth.ModelShape(2, 512, 4, 128, 1408, 512),
    "deep_k": synth.ModelShape(2, 128, 32, 64, 2728, 256),                # O and down: one feature tile, K cut into 8 slices
    "heads_wider_than_d": synth.ModelShape(1, 160, 3, 64, 424, 256),      # 10 feature tiles: a workgroup tile is partly empty
}


def cached(model, layer, n, shape):
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(layer, 0, 0, k, v)
    return k.cpu().numpy(), v.cpu().numpy()


@pytest.mark.parametrize("name,first,second", [
    ("dh64_ragged_ffn", 45, 0), ("dh64_ragged_ffn", 64, 65), ("dh64_ragged_ffn", 127, 128), ("dh64_ragged_ffn", 255, 47),
    ("dh128", 48, 0), ("dh128", 129, 63), ("dh128", 300, 45), ("heads_wider_than_d", 81, 79),
    ("deep_k", 25, 64), ("deep_k", 129, 47), ("deep_k", 700, 0),
])
def test_prefill_passes_against_oracle(name, first, second):
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    print(f"prefill {name} {first}+{second}", flush=True)
    w = randomize_gains(synth.make_weights(shape, 5))
    wn = synth.weights_to_numpy(w)
    n = first + second
    img = synth.image_rows(n // 2, shape.d_model, 3)
    toks = synth.text_tokens(n - n // 2, shape.vocab, 4)
    x = np.concatenate([img.astype(np.float64), dec.embed_tokens(wn, toks)])
    cfg = oracle_cfg(shape)
    cache = dec.KVCache(cfg, n + 4)
    ref = dec.forward_rows(cfg, wn, cache, x)
    model = spd.Model(spd.make_config(shape, 2, n + 4), to_device(w))
    rows = torch.from_numpy(x.astype(np.float32)).cuda()
    last = torch.empty(shape.vocab, device="cuda")
    model.spd_prefill(0, rows[:first].contiguous(), last)
    check_logits(last.cpu().numpy(), ref[first - 1], "first pass")
    if second:
        model.spd_prefill(0, rows[first:].contiguous(), last)
        check_logits(last.cpu().numpy(), ref[n - 1], "second pass")
    # K and V are bf16 values on both sides: equal, or one bf16 step apart where float32 and float64 fall on different
    # sides of a rounding boundary.  Near zero the error of the sums counts instead: float32 rounding in layer 0; behind
    # it, a flipped step of one V component (2^-8 of it) goes through Wo and Wk (0.02 per entry, width d <= 512:
    # 2^-8 * 0.02 * 0.02 * sqrt(512) = 4e-5 of a unit value), with room for a few of them at 4 sigma.
    for l in range(shape.n_layers):
        for got, want in zip(cached(model, l, n, shape), (cache.k[l][:n], cache.v[l][:n])):
            want = np.asarray(want, dtype=np.float64).reshape(got.shape)
            err = np.abs(got - want)
            floor = (1e-5 if l == 0 else 5e-4) * np.sqrt(np.mean(want * want))
            assert np.all(err <= np.maximum(2.0 ** -7 * np.abs(want), floor)), (l, err.max())
            assert np.mean(err > 0) < 0.02, (l, np.mean(err > 0))
    vt = synth.text_tokens(3, shape.vocab, 6)
    out = torch.empty((1, 3, shape.vocab), device="cuda")
    model.spd_verify_forward(torch.from_numpy(vt).cuda()[None].contiguous(), out)
    check_logits(out[0].cpu().numpy(), dec.forward_tokens(cfg, wn, cache, vt), "step after the prefill")


def test_prefill_with_the_length_on_the_device_and_another_sequence_untouched():
    from paper_2404_08856_amd import spd
    shape = SHAPES["dh128"]
    w = to_device(randomize_gains(synth.make_weights(shape, 7)))
    ids = torch.from_numpy(synth.text_tokens(150, shape.vocab, 8)).cuda()
    other = torch.from_numpy(synth.text_tokens(40, shape.vocab, 9)).cuda()
    outs = []
    for on_device in (False, True):
        m = spd.Model(spd.make_config(shape, 2, 200), w)
        m.spd_prefill_tokens(0, other)
        if on_device:
            m.spd_kv_lens_to_device()
        last = torch.empty(shape.vocab, device="cuda")
        m.spd_prefill_tokens(1, ids[:70].contiguous())
        m.spd_prefill_tokens(1, ids[70:].contiguous(), last)
        if on_device:
            m.spd_kv_lens_from_device()
        assert m.spd_kv_get_len(2) == [40, 150]
        step = torch.empty((2, 1, shape.vocab), device="cuda")
        m.spd_verify_forward(torch.tensor([[1], [2]], dtype=torch.int32, device="cuda"), step)
        outs.append((last.cpu(), step.cpu()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


def test_a_row_that_is_not_finite_does_not_reach_earlier_rows():
    """Causality also for 0 * NaN: keys hidden by the mask contribute nothing, whatever their values are."""
    from paper_2404_08856_amd import spd
    shape = SHAPES["dh128"]
    w = to_device(synth.make_weights(shape, 11))
    rows = torch.from_numpy(synth.image_rows(100, shape.d_model, 12)).cuda()
    bad = rows.clone()
    bad[60] = float("nan")
    kv = []
    for x in (rows, bad):
        m = spd.Model(spd.make_config(shape, 1, 128), w)
        last = torch.empty(shape.vocab, device="cuda")
        m.spd_prefill(0, x.contiguous(), last)
        kv.append((cached(m, 1, 100, shape), last.cpu()))
    (clean, _), (dirty, last) = kv
    for a, b in zip(clean, dirty):
        assert np.array_equal(a[:60], b[:60]) and np.isnan(b[60:]).all()
    assert torch.isnan(last).all()
