"""The sampling walk with dense draft distributions (csrc/tail.h) around the 64 nodes that a wave holds, in every form a
slice takes: one, two and three groups per thread, streamed, rows at every alignment; siblings that wait for each other's
normaliser, more of them than a residual chain keeps in registers; rows with one, four and more partial results.  Against the
oracle, to the bar of the other parity tests."""
import numpy as np
import pytest

from mars_inputs import make_workload
from tests.gpu_util import compare, compare_ex

pytestmark = pytest.mark.gpu

# vocabularies whose slices take 1 | 2 and 3 groups of eight per thread, and streamed ones
FORMS = [("f32", 4001), ("bf16", 4096), ("f32", 11000), ("bf16", 11003), ("bf16", 30000)]


def tree_of(N, children):
    return {"kind": "chain"} if N < 12 else {"kind": "tree", "depth": 3 if children > 4 else 6, "max_children": children}


@pytest.mark.parametrize("N", [1, 2, 12, 63, 64, 65])
@pytest.mark.parametrize("dtype,V", FORMS)
def test_trees_around_a_wave(N, dtype, V):
    # (130 requests: one work-group each)
    B = 130 if V >= 30000 and N <= 12 else 3
    compare(make_workload(f"lanes_{dtype}_{V}_{N}", B=B, N=N, V=V, dtype=dtype, temperature=0.9, dense_q=True, tree=tree_of(N, 4),
                          plant_frac=0.6, seed=N), allow_small_norm=True)


@pytest.mark.parametrize("N", [40, 64])
def test_long_chains_of_rejections(N):
    w = make_workload(f"lanes_siblings_{N}", B=6, N=N, V=9000, dtype="f32", temperature=1.0, dense_q=True, tree=tree_of(N, 10),
                      plant_frac=0.2, seed=7)
    compare(w, allow_small_norm=True)


@pytest.mark.parametrize("N", [20, 64, 65])
def test_sweep_with_committed_tokens(N):
    w = make_workload(f"lanes_sweep_{N}", B=4, N=N, V=12000, dtype="bf16", temperature=0.7, dense_q=True, tree=tree_of(N, 4),
                      plant_frac=0.6, seed=N, sweep_thetas=(0.85, 0.95))
    compare_ex(w, thetas=np.tile(np.array([[0.85], [0.9], [0.95]], np.float32), (1, 4)), allow_small_norm=True)


@pytest.mark.parametrize("N", [5, 64, 65])
def test_malformed_requests(N):
    w = make_workload(f"lanes_bad_{N}", B=3, N=N, V=5000, dtype="bf16", temperature=1.0, dense_q=True, tree={"kind": "chain"},
                      plant_frac=0.5, seed=4)
    w.tree_parent[0, N - 1] = N - 1
    w.draft_tokens[1, N - 1] = 5000
    compare(w)
