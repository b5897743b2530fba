"""The accept step in one launch (a workgroup per position, up to 256 of them) against the oracle: both sides of the edge to the
statistics-and-slices path, each kind of row and input, workspaces that hold anything, and draws whose residual is empty.  With
probabilities on both sides every answer is exact; with logits the tests of the sliced draw apply as they are."""
import numpy as np
import pytest
import torch

from oracle import spec_sampling as ss
from paper_2404_08856_amd import synth
from tests.test_gpu_accept_slices import check

pytestmark = pytest.mark.gpu


def exact(T, D, d, u, ws):
    from paper_2404_08856_amd import spd
    n, gamma = d.shape
    k, y = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    spd.spd_speculative_accept(torch.from_numpy(T).cuda(), torch.from_numpy(D).cuda(), torch.from_numpy(d).cuda(), torch.from_numpy(u).cuda(),
                               1.0, spd.SPD_TARGET_IS_PROBS | spd.SPD_DRAFT_IS_PROBS, k, y, None, ws)
    assert list(zip(k.tolist(), y.tolist())) == [ss.speculative_accept(T[s], D[s], d[s], u[s]) for s in range(n)]


def rows(n, gamma, V, seed):
    lt, ld = synth.accept_workload(n, gamma, V, 1.0, seed=seed)
    T, D = ss.softmax_probs(lt, 1.0), ss.softmax_probs(ld, 1.0)
    d = np.array([[ss.sample_row(D[s, j], x) for j, x in enumerate(r)] for s, r in enumerate(synth.uniforms((n, gamma), seed + 1))], dtype=np.int32)
    return T, D, d, synth.uniforms((n, gamma + 1), seed + 2)


@pytest.mark.parametrize("gamma,n", [(1, 1), (4, 1), (63, 1), (63, 4), (1, 128), (4, 51), (4, 52), (3, 64), (3, 65)])
@pytest.mark.parametrize("V", [4, 1024])
def test_positions_by_count(gamma, n, V):
    from paper_2404_08856_amd import spd
    print(f"accept positions gamma={gamma} n={n} V={V}", flush=True)
    ws = torch.full((spd.spd_accept_workspace_bytes(n, gamma, V),), 0xFF, dtype=torch.uint8, device="cuda")
    for seed in range(3):                                  # the same workspace again and again
        exact(*rows(n, gamma, V, 10 * seed + V), ws)


def test_one_workspace_through_both_paths():
    from paper_2404_08856_amd import spd
    print("accept positions: one workspace", flush=True)
    ws = torch.full((spd.spd_accept_workspace_bytes(65, 3, 1024),), 0x5A, dtype=torch.uint8, device="cuda")
    for n in (64, 65, 2, 65, 64):
        exact(*rows(n, 3, 1024, n), ws)


@pytest.mark.parametrize("V", [4, 12288, 12289, 32765, 32768])
@pytest.mark.parametrize("misalign", [False, True])
def test_positions_by_kind_of_row(V, misalign):
    check(V, 2, 2, False, True, 1.0, misalign=misalign, repeat=2)
    check(V, 2, 2, True, True, 1.0, misalign=misalign)


@pytest.mark.parametrize("n,gamma", [(1, 1), (1, 4), (51, 4), (4, 63)])
def test_answers_left_in_the_workspace(n, gamma):
    """Words that look like another call's answers for every position (calls that overlapped leave some): each sequence would stop at its first
    position with token 7."""
    from paper_2404_08856_amd import spd
    print(f"accept positions: leftovers n={n} gamma={gamma}", flush=True)
    T, D, d, u = rows(n, gamma, 1024, 21)
    T[:, :gamma] = D                                       # accepted wherever u < 1
    left = torch.tensor([7, 0xffc5a11c, ~7 & 0xffffffff, 0x9e3779b9], dtype=torch.int64).to(torch.uint32).view(torch.uint8)
    ws = torch.zeros(spd.spd_accept_workspace_bytes(n, gamma, 1024), dtype=torch.uint8, device="cuda")
    ws.view(-1, 16)[:n * (gamma + 1)] = left.cuda()
    exact(T, D, d, u, ws)


def test_residual_that_truncates_to_zero():
    """A reject whose residual has no mass draws from the target row."""
    from paper_2404_08856_amd import spd
    n, gamma, V = 2, 2, 1024
    print("accept positions: empty residual", flush=True)
    T, D, d, u = rows(n, gamma, V, 5)
    D[:] = T[:, :gamma]
    for s in range(n):
        T[s, 1, d[s, 1]] = 0.0                             # rejects at position 1; T <= D everywhere
    u[:, 1] = 0.5
    exact(T, D, d, u, torch.full((spd.spd_accept_workspace_bytes(n, gamma, V),), 0xAB, dtype=torch.uint8, device="cuda"))


def test_masked_logits():
    """Entries at -inf on both sides: weight 0, and the row's other entries as without them."""
    from paper_2404_08856_amd import spd
    n, gamma, V = 3, 4, 4096
    print("accept positions: masked logits", flush=True)
    lt, ld = synth.accept_workload(n, gamma, V, 1.0, seed=8)
    for x in (lt, ld):
        x[..., 100:] = -np.inf
    T, D = ss.softmax_probs(lt, 1.0), ss.softmax_probs(ld, 1.0)
    d = np.array([[ss.sample_row(D[s, j], x) for j, x in enumerate(r)] for s, r in enumerate(synth.uniforms((n, gamma), 3))], dtype=np.int32)
    u = synth.uniforms((n, gamma + 1), 4)
    k, y = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    ap = torch.empty((n, gamma), device="cuda")
    spd.spd_speculative_accept(torch.from_numpy(lt).cuda(), torch.from_numpy(ld).cuda(), torch.from_numpy(d).cuda(), torch.from_numpy(u).cuda(), 1.0, 0, k, y, ap)
    want = np.array([[ss.accept_probability(T[s, j, d[s, j]], D[s, j, d[s, j]]) for j in range(gamma)] for s in range(n)])
    assert np.max(np.abs(ap.cpu().numpy() - want)) < 1e-5
    assert int(y.min()) >= 0 and int(y.max()) < 100
