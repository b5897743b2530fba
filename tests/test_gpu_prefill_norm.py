"""The norm of a prompt's rows from its partial sums of squares, read 32 parts at a time: whole and ragged groups, one group and two,
against the float64 oracle."""
import pytest

from paper_2404_08856_amd import synth
from tests import test_gpu_prefill as prefill

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,parts", [(32, 1), (1984, 31), (2048, 32), (2080, 33), (2272, 36)])
@pytest.mark.parametrize("rows", [33, 130])
def test_groups_of_parts_against_oracle(d, parts, rows, monkeypatch):
    assert (d // 16 + 3) // 4 == parts
    monkeypatch.setitem(prefill.SHAPES, "norm", synth.ModelShape(2, d, 2, 64, 168, 256))
    prefill.test_prefill_passes_against_oracle("norm", rows, 0)
