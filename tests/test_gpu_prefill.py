"""GPU parity of the prefill passes (many rows of one sequence per pass) against the float64 oracle: row counts around
the edges of the row tiles, workgroup tiles, slices of K and key units, a second pass on top of a cached prefix, prompts of
more than one pass with a long or a short rest, ragged d_ffn, both head sizes, the KV cache it leaves and the decode step that
follows; and the read-out of that cache."""
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
    "wide": synth.ModelShape(2, 4096, 2, 128, 264, 256),                  # above 1024 rows O and down take the large workgroup shape
    "small": synth.ModelShape(2, 128, 2, 64, 168, 256),
}


def cached(model, layer, n, shape):
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(layer, 0, 0, k, v)
    return k.cpu().numpy(), v.cpu().numpy()


@pytest.mark.parametrize("name,first,second", [
    ("dh64_ragged_ffn", 45, 0), ("dh64_ragged_ffn", 64, 65), ("dh64_ragged_ffn", 127, 128), ("dh64_ragged_ffn", 255, 47),
    ("dh128", 48, 0), ("dh128", 129, 63), ("dh128", 300, 45), ("heads_wider_than_d", 81, 79),
    ("deep_k", 25, 64), ("deep_k", 129, 47), ("deep_k", 700, 0),
    ("wide", 1025, 0), ("wide", 1100, 1037),
    ("small", 2048 + 10, 0), ("small", 2048 + 70, 40),                    # a rest below and above the shortest run these kernels take
])
def test_prefill_passes_against_oracle(name, first, second):
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    print(f"prefill {name} {first}+{second}", flush=True)
    w = randomize_gains(synth.make_weights(shape, 5))
    wn = synth.weights_to_numpy(w)
    n = first + second
    # (wide: unit rows only -- against text rows, 0.02 per entry, a flipped step of V weighs up to 50 times as much, which the
    # bound on K and V below leaves out and 4096 columns show: 2e-3 of a row on this path and on the batched verify path)
    n_img = n if name == "wide" else n // 2
    img = synth.image_rows(n_img, shape.d_model, 3)
    toks = synth.text_tokens(n - n_img, shape.vocab, 4)
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


# heads of 64 take two units of 32 keys per step: prompts that end, and second passes that start, at every place of a step
@pytest.mark.parametrize("first,second", [(32, 0), (33, 0), (63, 0), (65, 0), (95, 0), (96, 0), (97, 0), (128, 33), (31, 98), (47, 65), (64, 128), (79, 130)])
def test_steps_of_two_units_against_oracle(first, second):
    test_prefill_passes_against_oracle("small", first, second)


@pytest.mark.parametrize("n", [2048 + 10, 2048 + 70, 4096 + 25])
def test_a_prompt_of_several_passes_by_ids_has_the_bits_of_its_rows(n):
    from paper_2404_08856_amd import spd
    shape = SHAPES["small"]
    w = to_device(synth.make_weights(shape, 13))
    ids = torch.from_numpy(synth.text_tokens(n, shape.vocab, 14)).cuda()
    outs = []
    for by_ids in (True, False):
        m = spd.Model(spd.make_config(shape, 1, n), w)
        last = torch.empty(shape.vocab, device="cuda")
        if by_ids:
            m.spd_prefill_tokens(0, ids, last)
        else:
            m.spd_prefill(0, w["embed"][ids.long()].float().contiguous(), last)
        assert m.spd_kv_get_len(1) == [n]
        outs.append((last.cpu().numpy(), *cached(m, 0, n, shape), *cached(m, 1, n, shape)))
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("name,capacity", [("dh128", 150), ("dh64_ragged_ffn", 160)])
def test_cache_read_out_of_any_range(name, capacity):
    """Ranges that start and end inside a unit of 32 positions, into outputs aligned to 16 bytes and to single floats only."""
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    m = spd.Model(spd.make_config(shape, 2, capacity), to_device(synth.make_weights(shape, 15)))
    m.spd_prefill_tokens(1, torch.from_numpy(synth.text_tokens(capacity, shape.vocab, 16)).cuda())
    H, dh = shape.n_heads, shape.head_dim
    full = [torch.empty((capacity, H, dh), device="cuda") for _ in range(2)]
    m.spd_kv_export(1, 1, 0, *full)
    assert all(len(torch.unique(x)) > 1000 for x in full)
    for pos0, n in ((0, 1), (31, 2), (5, 20), (32, 32), (33, 64), (capacity - 1, 1), (7, capacity - 7)):
        for offset in (0, 1, 2):
            flat = [torch.full((n * H * dh + 8,), -9.0, device="cuda") for _ in range(2)]
            out = [f[offset:offset + n * H * dh].view(n, H, dh) for f in flat]
            m.spd_kv_export(1, 1, pos0, *out)
            for f, o, want in zip(flat, out, full):
                assert torch.equal(o, want[pos0:pos0 + n]), (pos0, n, offset)
                assert (f[:offset] == -9.0).all() and (f[offset + n * H * dh:] == -9.0).all()


@pytest.mark.parametrize("name,n", [("dh64_ragged_ffn", 25), ("dh128", 33), ("dh128", 130), ("wide", 70), ("wide", 1030), ("small", 2048 + 40)])
@pytest.mark.parametrize("on_device", [False, True])
def test_a_prompt_without_logits_leaves_the_cache_of_one_with_them(name, n, on_device):
    """Only the last row passes through the whole last layer, and only where its logits are asked for: no key and no value depends on that."""
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    w = to_device(randomize_gains(synth.make_weights(shape, 17)))
    rows = torch.from_numpy(synth.image_rows(n, shape.d_model, 18)).cuda()
    kv, steps = [], []
    for with_logits in (True, False):
        m = spd.Model(spd.make_config(shape, 1, n + 4), w)
        if on_device:
            m.spd_kv_lens_to_device()
        m.spd_prefill(0, rows, torch.empty(shape.vocab, device="cuda") if with_logits else None)
        if on_device:
            m.spd_kv_lens_from_device()
        assert m.spd_kv_get_len(1) == [n]
        kv.append([x for l in range(shape.n_layers) for x in cached(m, l, n, shape)])
        out = torch.empty((1, 2, shape.vocab), device="cuda")
        m.spd_verify_forward(torch.tensor([[1, 2]], dtype=torch.int32, device="cuda"), out)
        steps.append(out.cpu().numpy())
    for a, b in zip(*kv):
        assert np.array_equal(a, b)
    assert np.array_equal(steps[1], steps[0])
