"""The greedy kernel behind the row reduction (csrc/tail.h) at the sizes where it changes form: trees around the 64 nodes that a
wave holds, rows with few partial results and with more than a lane merges alone, chains as long as the pointer jumping has
to reach, malformed requests.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from mars_inputs import make_workload
from tests.gpu_util import compare, compare_ex

pytestmark = pytest.mark.gpu

TREE = {"kind": "tree", "depth": 6, "max_children": 4}
CHAIN = {"kind": "chain"}


@pytest.mark.parametrize("N", [1, 2, 3, 33, 63, 64, 65, 128])
@pytest.mark.parametrize("B,V", [(1, 100000), (2, 40001), (70, 9000)])   # up to twelve partial results per row; one
def test_trees_around_a_wave(N, B, V):
    tree = CHAIN if N < 10 else TREE
    compare(make_workload(f"greedy_B{B}_N{N}_V{V}", B=B, N=N, V=V, dtype="bf16", temperature=0.0, tree=tree, plant_frac=0.6, seed=N))


@pytest.mark.parametrize("N", [2, 64, 65])
@pytest.mark.parametrize("B", [1, 5])
def test_chains_with_every_draft_accepted(N, B):
    w = make_workload(f"greedy_chain_{B}_{N}", B=B, N=N, V=20000, dtype="f32", temperature=0.0, tree=CHAIN, plant_frac=0.5, seed=3)
    z = w.logits.reshape(B, N, -1)
    w.draft_tokens[:, 1:] = z.argmax(axis=2)[:, :-1]
    compare(w)
    compare_ex(w, label="greedy_chain_commit")


@pytest.mark.parametrize("N", [3, 64, 65])
@pytest.mark.parametrize("B", [2, 60])
def test_malformed_requests(N, B):
    w = make_workload(f"greedy_bad_{B}_{N}", B=B, N=N, V=9000, dtype="bf16", temperature=0.0, tree=CHAIN, plant_frac=0.5, seed=4)
    w.tree_parent[0, N - 1] = N - 1
    w.draft_tokens[1, N - 1] = 9000
    compare(w)
