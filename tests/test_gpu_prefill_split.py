"""Both forms of the prompt attention -- 64 queries a workgroup, or 32 with two waves for the same queries -- at the edges of the rule that
chooses between them, against the float64 oracle, and with values and scores that are not finite in the form that the small shapes of
the other tests never take."""
import numpy as np
import pytest
import torch

from paper_2404_08856_amd import synth
from tests import test_gpu_prefill as prefill
from tests.helpers import to_device
from tests.test_gpu_nonfinite import KEY, QUERY, prompt, steered

pytestmark = pytest.mark.gpu

SHAPES = {
    "heads64": synth.ModelShape(1, 128, 32, 64, 168, 256),      # 512 workgroups of 64 queries at 1024 rows
    "heads128": synth.ModelShape(1, 128, 16, 128, 168, 256),    # 128 at 512 rows, 16 blocks of queries from 961 rows, 256 workgroups at 1024
}


@pytest.mark.parametrize("name,rows", [("heads64", 1024), ("heads64", 1025), ("heads128", 512), ("heads128", 513), ("heads128", 960), ("heads128", 961), ("heads128", 1025)])
def test_rule_edges_against_oracle(name, rows, monkeypatch):
    monkeypatch.setitem(prefill.SHAPES, name, SHAPES[name])
    prefill.test_prefill_passes_against_oracle(name, rows, 0)


@pytest.mark.parametrize("at", [0, 299, 320, 599])
def test_infinite_value_without_the_split(at):
    """60 heads, 600 rows: 600 workgroups of 64 queries."""
    from paper_2404_08856_amd import spd
    print(f"infinite value at {at}, whole form", flush=True)
    n = 600
    shape, w = steered(60, 0.0, 0.0, layers=2)
    w["layers"][0]["wv"][5, KEY] = 2.0 ** 127                   # times 8: one component of V is infinite
    model = spd.Model(spd.make_config(shape, 1, n), to_device(w))
    model.spd_prefill_tokens(0, torch.from_numpy(prompt(n, at)).cuda())
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(1, 0, 0, k, v)
    v = v.cpu().numpy()
    assert np.isfinite(v[:at]).all() and (~np.isfinite(v[at:])).all()


@pytest.mark.parametrize("heads,n", [(2, 97), (60, 600)])
@pytest.mark.parametrize("at", [1, 33, 95])
def test_overflowed_score_of_a_row_in_the_middle(heads, n, at):
    """A query whose score of one key overflows is NaN, the rows that do not ask are not: keys and values of the layer behind say so."""
    from paper_2404_08856_amd import spd
    print(f"overflowed score at {at}, {heads} heads, {n} rows", flush=True)
    shape, w = steered(heads, 1e19, 1e19, layers=2)
    ids = prompt(n, at)
    ids[n - 1] = QUERY
    model = spd.Model(spd.make_config(shape, 1, n), to_device(w))
    model.spd_prefill_tokens(0, torch.from_numpy(ids).cuda())
    k, v = (torch.empty((n, shape.n_heads, shape.head_dim), device="cuda") for _ in range(2))
    model.spd_kv_export(1, 0, 0, k, v)
    assert torch.isfinite(v[:n - 1]).all() and torch.isnan(v[n - 1]).all()
