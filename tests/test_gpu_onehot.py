"""The sampling walk of one-hot draft distributions (csrc/onehot.h) at the sizes where it can go wrong: trees at the edge of what
it holds, shares of a row around whole batches and chunks, rejected tokens that hold most of a row's mass at every kind of place
in it, draws at both ends of the distribution, and a workspace without room for the sums of the chunks.  Against the oracle, to
the bar of the other parity tests.

Which walk a call takes depends on the number of requests, too (mars.hip: onehot_form): with the few that most tests here have, rows longer than a page are
gone over by several work-groups.  test_gpu_onehot_forms.py has each walk at sizes that are held to it."""
import numpy as np
import pytest
import torch

from mars_inputs import f32_to_bf16_bits, make_workload
from tests.gpu_util import compare, say, to_device

pytestmark = pytest.mark.gpu

BATCH = {"bf16": 8192, "f32": 4096}   # entries the row reduction takes at a time


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65])
@pytest.mark.parametrize("dtype,V", [("bf16", 32000), ("f32", 9001)])
def test_trees_at_the_edge_of_a_wave(N, dtype, V):
    tree = {"kind": "chain"} if N < 3 else {"kind": "tree", "depth": 5, "max_children": 4}
    compare(make_workload(f"onehot_N{N}_{dtype}", B=3, N=N, V=V, dtype=dtype, temperature=1.0, tree=tree, plant_frac=0.6, seed=N))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("batches,more", [(1, -8), (2, 1), (3, -8), (3, 0), (4, 5), (5, 0), (8, 3), (19, 8), (21, 0), (38, 1)])
def test_shares_around_whole_batches(dtype, batches, more):
    # 130 rows: one share each, or a few; B = 65 chains of two
    V = batches * BATCH[dtype] + more
    compare(make_workload(f"onehot_{dtype}_{batches}_{more}", B=43, N=3, V=V, dtype=dtype, temperature=0.9,
                          tree={"kind": "chain"}, plant_frac=0.5, seed=batches))


def heavy_workload(dtype, V, at, left, draws, seed):
    """A root with three children of which the first carries the row's largest entry, at `at`, with all but about `left` of
    the mass, and is rejected; the others are unlikely.  (left < 0.1: the normaliser is summed, not 1 - f.)"""
    rng = np.random.default_rng(seed)
    B, N = len(draws), 4
    z = rng.normal(0, 2, size=(B, N, V)).astype(np.float32)
    other = np.delete(np.arange(V), at)
    for b in range(B):
        rest = np.log(np.exp(z[b, 0, other].astype(np.float64)).sum())
        z[b, 0, at] = rest + np.log((1 - left) / left)
    tok = np.zeros((B, N), np.int32)
    tok[:, 1] = at
    tok[:, 2:] = np.stack([rng.permutation(other)[:2] for _ in range(B)])
    u = np.full((B, N + 1), 0.9995, np.float32)
    u[:, N] = draws
    from tests.test_gpu_parity import custom
    par = np.tile(np.array([-1, 0, 0, 0], np.int32), (B, 1))
    return custom(f"heavy_{dtype}_V{V}_at{at}_left{left}", f32_to_bf16_bits(z) if dtype == "bf16" else z, tok, par, 2.0, 1.0, u=u)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [3, 7, 8, 9, 511, 4096, 16367, 16368, 16369, 16376, 24001, 32751, 32752, 32753])
def test_vocabularies_of_one_page(dtype, V):
    # (16 368 and 32 752 entries are a page; trees where siblings wait for a sum, and chains)
    tree = {"kind": "chain"} if V < 10 else {"kind": "tree", "depth": 4, "max_children": 4}
    compare(make_workload(f"onehot_page_{dtype}_{V}", B=5, N=2 if V < 10 else 21, V=V, dtype=dtype, temperature=0.8, tree=tree,
                          plant_frac=0.7, seed=V), allow_small_norm=True)


@pytest.mark.parametrize("dtype,V", [("bf16", 65536), ("f32", 40003), ("bf16", 70001), ("bf16", 5003), ("f32", 16360), ("f32", 32752), ("bf16", 30011)])
@pytest.mark.parametrize("left", [0.04, 0.3])
def test_rejected_tokens_that_hold_most_of_the_row(dtype, V, left):
    batch = BATCH[dtype]
    for i, at in enumerate((0, 1, V - 1, V - 2, min(2 * batch, V) - 1, min(2 * batch, V - 9), V // 2)):
        compare(heavy_workload(dtype, V, at, left, [0.0, 0.31, 0.74, 0.9999], seed=i))


def test_workspace_without_room_for_the_sums_of_the_chunks():
    from paper_2601_15498_amd import binding as M
    w = make_workload("onehot_least", B=3, N=9, V=40000, dtype="f32", temperature=1.0, tree={"kind": "chain"}, plant_frac=0.5, seed=5)
    total = M.mars_workspace_bytes(3, 9, 40000)
    table = 27 * 4 * 1 * 8 * 8    # 27 rows, four shares of one chunk, eight waves
    d = to_device(w)

    def run(w, size=total - table):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        out = M.mars_verify(d["logits"], d["draft_tokens"], d["tree_parent"], d["theta"], w.temperature,
                            torch.from_numpy(w.uniforms).to("cuda:0"), None, workspace=ws)
        torch.cuda.synchronize()
        return out

    compare(w, run=run)
    compare(w, run=lambda w: run(w, total))
    with pytest.raises(M.MarsError):
        run(w, total - table - 1)
    say("[ok]   least workspace")
