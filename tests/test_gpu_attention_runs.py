"""GPU parity of attention over runs of keys (a long cache, 33 to 64 (sequence, head) pairs): lengths on both sides of the rule's
line, a sequence so short that later runs have no unit, both head sizes, one and five queries, launches repeated on the
same counters, lengths on the device; and of whole heads with 225 to 256 pairs, where the keys' loads depend on the length."""
import numpy as np
import pytest
import torch

from oracle import decoder as dec
from paper_2404_08856_amd import synth
from tests.helpers import check_logits, oracle_cfg, randomize_gains, to_device

pytestmark = pytest.mark.gpu

SHAPES = {"dh128": synth.ModelShape(1, 256, 16, 128, 688, 512), "dh64": synth.ModelShape(1, 256, 13, 64, 688, 512)}


@pytest.mark.parametrize("name,lens,M,device_lens", [
    ("dh128", [1100, 3, 40, 700], 5, False), ("dh128", [607, 1, 600], 1, False), ("dh128", [608, 0, 33], 1, True),
    ("dh64", [1024, 31, 32, 65], 4, False), ("dh64", [995, 500, 2], 5, True),
    ("dh128", [600] + 15 * [33], 1, False), ("dh128", [650] + 14 * [70], 4, True), ("dh128", [599] + 15 * [2], 3, False),
])
def test_runs_of_keys_against_oracle(name, lens, M, device_lens):
    from paper_2404_08856_amd import spd
    shape = SHAPES[name]
    print(f"attention runs {name} {lens} M {M} device lengths {device_lens}", flush=True)
    w = randomize_gains(synth.make_weights(shape, 31))
    wn = synth.weights_to_numpy(w)
    cfg = oracle_cfg(shape)
    n = len(lens)
    model = spd.Model(spd.make_config(shape, n, max(lens) + 3 * M), to_device(w))
    caches = []
    for s, length in enumerate(lens):
        cache = dec.KVCache(cfg, max(lens) + 3 * M)
        if length:
            ids = synth.text_tokens(length, shape.vocab, 40 + s)
            dec.forward_tokens(cfg, wn, cache, ids)
            model.spd_prefill_tokens(s, torch.from_numpy(ids).cuda())
        caches.append(cache)
    if device_lens:
        model.spd_kv_lens_to_device()
    out = torch.empty((n, M, shape.vocab), device="cuda")
    for step in range(2):                    # the second step reads what the first one appended
        vt = np.stack([synth.text_tokens(M, shape.vocab, 70 + 10 * step + s) for s in range(n)])
        model.spd_verify_forward(torch.from_numpy(vt).cuda(), out)
        got = out.cpu().numpy()
        for s in range(n):
            check_logits(got[s], dec.forward_tokens(cfg, wn, caches[s], vt[s]), f"{name} step {step} seq {s}")
    if device_lens:
        model.spd_kv_lens_from_device()
    assert model.spd_kv_get_len(n) == [c + 2 * M for c in lens]


def test_lengths_on_the_device_that_stay_short_do_not_take_the_runs():
    """Blocks that accept nothing: the host's upper bound passes the rule's line while the caches hold 124 positions.  The
    step then has the bits of the same step with the lengths on the host."""
    from paper_2404_08856_amd import spd
    shape, gamma, n = SHAPES["dh64"], 7, 3
    target = spd.Model(spd.make_config(shape, n, 700), to_device(synth.make_weights(shape, 31)))
    draft_shape = synth.ModelShape(1, 64, 1, 64, 64, shape.vocab)
    draft = spd.Model(spd.make_config(draft_shape, n, 700), to_device(synth.make_weights(draft_shape, 32)))
    for m in (target, draft):
        for s in range(n):
            m.spd_prefill_tokens(s, torch.from_numpy(synth.text_tokens(40, shape.vocab, 50 + s)).cuda())
        m.spd_kv_lens_to_device()
    vt = torch.ones((n, gamma + 1), dtype=torch.int32, device="cuda")
    logits = torch.empty((n, gamma + 1, shape.vocab), device="cuda")
    other = torch.empty_like(logits)
    D = torch.zeros((n, gamma, shape.vocab), device="cuda")
    u = torch.full((n, gamma + 1), 0.75, device="cuda")
    k, y, n_out = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3))
    draft_in = torch.zeros((n, 2), dtype=torch.int32, device="cuda")
    for _ in range(84):
        vt[:, 1:] = 1
        D.zero_()
        D[:, :, 1] = 1.0                     # 0.75 * 1 is not below T(1): rejected
        target.spd_verify_forward(vt, logits)
        draft.spd_verify_forward(vt, other)
        spd.spd_block_finish(target, draft, logits, D, vt, u, 1.0, k, y, draft_in)
    step = torch.full((n, 1), 5, dtype=torch.int32, device="cuda")
    outs = [torch.empty((n, 1, shape.vocab), device="cuda") for _ in range(2)]
    target.spd_verify_forward(step, outs[0])
    target.spd_kv_lens_from_device()
    assert target.spd_kv_get_len(n) == [125] * n
    target.spd_kv_set_len([124] * n)
    target.spd_verify_forward(step, outs[1])
    assert torch.equal(outs[0], outs[1])


@pytest.fixture
def kernel_by_kernel(monkeypatch):
    """Models whose calls of up to 5 rows run the separate kernels: by default these small ones take the launch of all layers, whose rule has its own line."""
    from paper_2404_08856_amd import spd

    class Separate(spd.Model):
        def __init__(self, *args):
            super().__init__(*args)
            self.spd_model_set_tuning(separate_qkv_attention=1)

    monkeypatch.setattr(spd, "Model", Separate)


@pytest.mark.parametrize("lens,device_lens", [([607, 1, 600], False), ([608, 0, 33], True)])
def test_one_query_on_both_sides_of_the_line(lens, device_lens, kernel_by_kernel):
    test_runs_of_keys_against_oracle("dh128", lens, 1, device_lens)


def test_short_lengths_on_the_device_kernel_by_kernel(kernel_by_kernel):
    test_lengths_on_the_device_that_stay_short_do_not_take_the_runs()
