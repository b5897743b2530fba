"""The accept step's sliced draw against the oracle where its dispatch changes: 1 or 4 slices by draft length, batch
size and alignment of the workspace, slices emptier than others (small and ragged vocabularies), each
mix of logit and probability inputs, rows that end in a part of a quad or are not 16-byte aligned, and the generic kernel
next to them (vocabularies beyond 32768)."""
import numpy as np
import pytest
import torch

from oracle import spec_sampling as ss
from paper_2404_08856_amd import synth
from tests.helpers import accept_margins, drawn_token_is_valid

pytestmark = pytest.mark.gpu


def check(V, gamma, n_seqs, target_probs, draft_probs, temp, misalign=False, repeat=1, ws_offset=0):
    from paper_2404_08856_amd import spd
    print(f"accept slices V={V} gamma={gamma} n={n_seqs} T {target_probs} D {draft_probs} temp {temp} misaligned {misalign}", flush=True)
    lt, ld = synth.accept_workload(n_seqs, gamma, V, 1.0, seed=V + 64 * gamma + n_seqs)
    T, D = ss.softmax_probs(lt, temp), ss.softmax_probs(ld, temp)
    d = np.array([[ss.sample_row(D[s, j], x) for j, x in enumerate(r)] for s, r in enumerate(synth.uniforms((n_seqs, gamma), 3))], dtype=np.int32)
    u = synth.uniforms((n_seqs, gamma + 1), 4)
    u[0, -1] = 0.0
    u[-1, -1] = np.float32(1 - 2.0 ** -24)

    def place(x, side):
        flat = torch.zeros(x.size + 4, device="cuda")
        out = flat[1 if misalign in (True, side) else 0:][:x.size].view(x.shape)
        out.copy_(torch.from_numpy(np.ascontiguousarray(x)))
        return out

    flags = (spd.SPD_TARGET_IS_PROBS if target_probs else 0) | (spd.SPD_DRAFT_IS_PROBS if draft_probs else 0)
    gt, gd = place(T if target_probs else lt, "target"), place(D if draft_probs else ld, "draft")
    ws = torch.full((spd.spd_accept_workspace_bytes(n_seqs, gamma, V) + ws_offset,), 0xAB, dtype=torch.uint8, device="cuda")[ws_offset:]
    for _ in range(repeat):                                # the workspace starts dirty and is used again as it is
        k, y = (torch.full((n_seqs,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        ap = torch.empty((n_seqs, gamma), device="cuda")
        spd.spd_speculative_accept(gt, gd, torch.from_numpy(d).cuda(), torch.from_numpy(u).cuda(), temp, flags, k, y, ap, ws)
        k, y, ap = k.cpu().numpy(), y.cpu().numpy(), ap.cpu().numpy()
        for s in range(n_seqs):
            if int(k[s]) != ss.speculative_accept(T[s], D[s], d[s], u[s])[0]:
                assert min(accept_margins(T[s], D[s], d[s], u[s])) < 1e-5, s
            # a float32 softmax is within 4e-6 of the float64 one (argument up to 20 units of 6e-8, the exponential, the sum), so
            # the running sums of T and D move by at most that, against the mass of the distribution drawn from
            row = ss.residual(T[s, k[s]], D[s, k[s]]) if k[s] < gamma else T[s, gamma]
            assert drawn_token_is_valid(T[s], D[s], int(k[s]), u[s, gamma], int(y[s]), tol=8e-6 / float(row.sum())), (s, int(k[s]), int(y[s]))
            for j in range(gamma):
                assert abs(ap[s, j] - ss.accept_probability(T[s, j, d[s, j]], D[s, j, d[s, j]])) < 1e-5


@pytest.mark.parametrize("gamma,n_seqs", [(1, 1), (1, 128), (1, 129), (2, 64), (3, 65), (4, 1), (4, 32), (4, 33), (7, 2), (8, 2), (63, 1), (5, 257)])
def test_slices_by_draft_length_and_batch(gamma, n_seqs):
    check(1024, gamma, n_seqs, False, False, 1.0, repeat=2)


@pytest.mark.parametrize("V", [1, 2, 3, 4, 5, 16, 36, 1000, 4096, 4097, 4098, 4099, 4100, 32000, 32003, 32764, 32767, 32768, 32769, 32772])
def test_slices_by_vocabulary(V):
    check(V, 4, 2, False, False, 1.0)


@pytest.mark.parametrize("target_probs,draft_probs", [(False, True), (True, False), (False, False)])
@pytest.mark.parametrize("temp", [0.7, 1.0])
def test_slices_by_kind_of_input(target_probs, draft_probs, temp):
    check(2048, 4, 3, target_probs, draft_probs, temp, repeat=2)


@pytest.mark.parametrize("V", [2048, 2047, 32765])
def test_rows_that_are_not_16_byte_aligned(V):
    check(V, 4, 3, False, False, 1.0, misalign=True)
    check(V, 1, 2, False, True, 1.0, misalign=True)


@pytest.mark.parametrize("offset", [4, 8, 12])
def test_workspace_not_aligned_to_its_rows(offset):
    """The slices' totals are 8-byte words: a workspace aligned to single floats only keeps one slice."""
    check(2048, 4, 3, False, False, 1.0, repeat=2, ws_offset=offset)


@pytest.mark.parametrize("V", [1000, 32003, 32768, 40000])
def test_greedy_draw(V):
    """Temperature 0: one-hot rows, so accept counts and tokens are exact."""
    check(V, 4, 5, False, False, 0.0, repeat=2)


@pytest.mark.parametrize("side", ["target", "draft"])
@pytest.mark.parametrize("V,temp", [(2048, 1.0), (8000, 1.0), (12284, 1.0), (12284, 0.0), (16384, 0.7)])
def test_one_side_s_rows_not_aligned(side, V, temp):
    """Statistics in registers for the aligned side and from memory for the other, from 8000 to 12287 entries."""
    check(V, 4, 3, False, False, temp, misalign=side, repeat=2)
