"""GPU parity of the batched projection kernel's plans: 4, 6 and 8 multiplying waves, one and several K slices with ragged last
units, two row groups with a long K, two tiles per wave, matrices too wide for the kernel; and the wave counts of
the kernels for one row group over a short K -- over models whose matrices make the plan come out that way."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2404_08856_amd import synth
from tests.helpers import check_logits, oracle_cfg, randomize_gains, to_device

pytestmark = pytest.mark.gpu

SHAPES = {
    # K = 2048 everywhere: four waves with 16 resident K-steps each at one row group, eight waves at two
    "k2048": synth.ModelShape(1, 2048, 16, 128, 2048, 1024),
    # K = 768: waves of 6, 3 or 1.5 K-steps by the number of rows
    "k768": synth.ModelShape(1, 768, 12, 64, 768, 512),
    # QKV 96 tiles, gate|up 172 (4 waves: 24 and 43 groups), down K = 1376: 43 steps, the last unit ragged
    "d512": synth.ModelShape(1, 512, 4, 128, 1376, 1040),
    # LM head 258 tiles of 16: 65 groups of 4, the last one partly empty
    "wide_head": synth.ModelShape(1, 256, 4, 64, 688, 4128),
    # gate|up 68 groups of 8 in 3 slices; down: K = 4352 (136 steps) with 256 tiles -- two row groups through the batched kernel at 6..10 rows
    "long_down": synth.ModelShape(1, 4096, 2, 128, 4352, 512),
    # LM heads of 1030 and 1541 tiles: 172 groups of 6 and 193 of 8, the last ones partly empty
    "head_of_sixes": synth.ModelShape(1, 256, 4, 64, 688, 16480),
    "head_of_eights": synth.ModelShape(1, 256, 4, 64, 688, 24656),
    # LM heads of 8194 tiles (more than 1024 groups of 8: two tiles per wave) and of 16386 (more than 1024 groups of 16)
    "two_tiles": synth.ModelShape(1, 64, 1, 64, 64, 131104),
    "too_wide": synth.ModelShape(1, 64, 1, 64, 64, 262176),
}


@pytest.mark.parametrize("name,n_seqs,M", [("d512", 3, 5), ("d512", 8, 5), ("d512", 8, 8), ("d512", 4, 7), ("d512", 6, 8), ("wide_head", 2, 6), ("wide_head", 5, 7),
                                           ("k2048", 1, 3), ("k2048", 5, 1), ("k2048", 2, 4),
                                           ("k768", 1, 1), ("k768", 3, 1), ("k768", 4, 1), ("k768", 1, 5), ("k768", 6, 1),
                                           ("long_down", 1, 6), ("long_down", 2, 5), ("long_down", 7, 1), ("long_down", 3, 4)])
def test_batched_step_against_oracle(name, n_seqs, M):
    check(name, n_seqs, M)


# k2048: QKV 64 groups of 6 waves in 4 slices, the others 4 waves in 4 (more than 8 row groups) or 8 slices, the most there are
@pytest.mark.parametrize("name,n_seqs,M", [("k2048", 3, 4), ("k2048", 4, 4), ("k2048", 5, 4), ("k2048", 6, 5), ("k2048", 8, 5), ("k2048", 7, 7), ("k2048", 8, 8),
                                           ("k768", 3, 4), ("k768", 8, 8), ("long_down", 8, 8),
                                           ("head_of_sixes", 3, 4), ("head_of_sixes", 8, 8), ("head_of_eights", 3, 4), ("head_of_eights", 8, 5)])
def test_waves_and_slices_against_oracle(name, n_seqs, M):
    check(name, n_seqs, M)


# rows 6..10 take the batched kernel at a short K only when told to
@pytest.mark.parametrize("name,n_seqs,M,batch_kernel", [("two_tiles", 2, 4, 1), ("two_tiles", 3, 4, 0), ("two_tiles", 5, 8, 0), ("two_tiles", 6, 8, 0),
                                                        ("too_wide", 2, 4, 1), ("too_wide", 3, 4, 0), ("too_wide", 6, 8, 0)])
def test_very_wide_head_against_oracle(name, n_seqs, M, batch_kernel):
    check(name, n_seqs, M, batch_kernel)


def check(name, n_seqs, M, batch_kernel=0):
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    print(f"batch plan {name} {n_seqs}x{M}", flush=True)
    w = randomize_gains(synth.make_weights(shape, 21))
    wn = synth.weights_to_numpy(w)
    cfg = oracle_cfg(shape)
    model = spd.Model(spd.make_config(shape, n_seqs, 64), to_device(w))
    if batch_kernel:
        model.spd_model_set_tuning(batch_kernel=batch_kernel)
    caches = []
    for s in range(n_seqs):
        ids = synth.text_tokens(9 + 2 * s, shape.vocab, 30 + s)
        cache = dec.KVCache(cfg, 64)
        dec.forward_tokens(cfg, wn, cache, ids)
        model.spd_prefill_tokens(s, torch.from_numpy(ids).cuda())
        caches.append(cache)
    vt = np.stack([synth.text_tokens(M, shape.vocab, 60 + s) for s in range(n_seqs)])
    out = torch.empty((n_seqs, M, shape.vocab), device="cuda")
    for _ in range(2):                       # the arrival counters are zero again after a launch
        model.spd_kv_set_len([c.length for c in caches])
        model.spd_verify_forward(torch.from_numpy(vt).cuda(), out)
    got = out.cpu().numpy()
    for s in range(n_seqs):
        check_logits(got[s], dec.forward_tokens(cfg, wn, caches[s], vt[s]), f"{name} seq {s}")


# rows 6..10, matrices of 256 tiles or more: QKV in groups of 6 waves, gate|up of 4, both in 4 slices
@pytest.mark.parametrize("n_seqs,M", [(1, 6), (2, 5)])
def test_two_groups_in_four_slices_against_oracle(n_seqs, M):
    check("k2048", n_seqs, M, batch_kernel=1)


@pytest.mark.parametrize("d,heads,n_seqs", [(4096, 32, 12), (4096, 32, 40), (4096, 32, 64), (2048, 16, 64)])
def test_slices_in_halves_are_as_exact_as_the_kernel_that_splits_k_over_waves(d, heads, n_seqs):
    """The O projection alone: one row per sequence at position 0 (attention returns the cached value, which is read back), no MLP, an LM head that
    hands the normalised row through.  A chain of n additions has an error that grows with sqrt(n) (roundings are independent): with the
    chains of this kernel at most as long as the other kernel's (K / 8 waves) the ratio is at most 1, a chain twice as long makes it
    1.41; 1.15 lies between.  An estimate from 50000 errors or more is good to 1 %."""
    from paper_2404_08856_amd import spd
    shape = synth.ModelShape(1, d, heads, 128, 64, d)
    w = to_device(synth.make_weights(shape, 41))
    w["embed"] = (0.01 * w["embed"].float()).to(torch.bfloat16)
    w["lm_head"] = torch.eye(d, device="cuda").to(torch.bfloat16)
    w["layers"][0]["w_down"].zero_()
    ids = torch.from_numpy(synth.text_tokens(n_seqs, shape.vocab, 42)).cuda()
    errors = []
    for batch_kernel in (1, 2):
        m = spd.Model(spd.make_config(shape, n_seqs, 8), w)
        m.spd_model_set_tuning(batch_kernel=batch_kernel)
        out = torch.empty((n_seqs, 1, shape.vocab), device="cuda")
        m.spd_verify_forward(ids[:, None].contiguous(), out)
        values = []
        for s in range(n_seqs):
            k, v = (torch.empty((1, heads, 128), device="cuda") for _ in range(2))
            m.spd_kv_export(0, s, 0, k, v)
            values.append(v.reshape(-1).double())
        x = w["embed"][ids.long()].double() + torch.stack(values) @ w["layers"][0]["wo"].double().T
        want = x / torch.sqrt(x.square().mean(-1, keepdim=True) + shape.rms_eps)
        # the row's common factor (its own rounding of 1 / rms) is not the sums' error
        got = out[:, 0].double()
        got = got * ((got * want).sum(-1, keepdim=True) / got.square().sum(-1, keepdim=True))
        errors.append(((got - want).norm() / want.norm()).item())
    print(f"O at {n_seqs} rows: {errors[0]:.3e}, K over waves {errors[1]:.3e}", flush=True)
    assert errors[0] <= 1.15 * errors[1], errors


def test_activations_of_more_than_four_gib():
    """64 rows of 11.2 million columns: 13 row groups of 350000 K-steps of 1 KiB.  The last rows' activations lie beyond 2^32 bytes."""
    from paper_2404_08856_amd import spd
    shape = synth.ModelShape(1, 64, 1, 64, 11_200_000, 64)
    g = torch.Generator(device="cuda").manual_seed(51)
    mat = lambda *s: (0.02 * torch.randn(s, generator=g, device="cuda")).to(torch.bfloat16)
    w = to_device(synth.make_weights(synth.ModelShape(1, 64, 1, 64, 64, 64), 50))
    lw = w["layers"][0]
    lw["wo"].zero_()
    lw["w_gate"], lw["w_up"], lw["w_down"] = mat(shape.d_ffn, 64), mat(shape.d_ffn, 64), mat(64, shape.d_ffn)
    ids = torch.arange(64, dtype=torch.int32, device="cuda")
    m = spd.Model(spd.make_config(shape, 64, 1), w)
    out = torch.empty((64, 1, 64), device="cuda")
    m.spd_verify_forward(ids[:, None].contiguous(), out)
    x = w["embed"].double()
    b = x / torch.sqrt(x.square().mean(-1, keepdim=True) + shape.rms_eps)
    y = x.clone()
    for at in range(0, shape.d_ffn, 800_000):
        part = slice(at, at + 800_000)
        act = torch.nn.functional.silu(b @ lw["w_gate"][part].double().T) * (b @ lw["w_up"][part].double().T)
        y += act @ lw["w_down"][:, part].double().T
    want = y / torch.sqrt(y.square().mean(-1, keepdim=True) + shape.rms_eps) @ w["lm_head"].double().T
    check_logits(out[:, 0].cpu().numpy(), want.cpu().numpy(), "rows behind 4 GiB")
