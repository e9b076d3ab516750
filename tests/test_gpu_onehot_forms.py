"""The walks of one-hot draft distributions, each at the sizes at which mars_verify takes it: draws by sums of chunks with
rejected tokens that hold most of the row at every kind of place in it, the page of 1 024 threads up to its last entry, and the walk over the row in
every form that a slice takes there.  Which form a case runs is held on the CPU (test_device_code_on_cpu.py reads the lists here).
Against the oracle, to the bar of the other parity tests."""
import numpy as np
import pytest
import torch

from mars_inputs import f32_to_bf16_bits, make_workload
from tests.gpu_util import compare, compare_ex, to_device
from tests.test_gpu_parity import custom

pytestmark = pytest.mark.gpu

# B, N, V, type of the logits
HEAVY_BY_CHUNKS = [(128, 4, 100001, "bf16"), (128, 4, 98331, "f32"), (128, 4, 65536, "bf16"), (128, 4, 40003, "f32"), (128, 4, 70001, "bf16"),
                   (128, 4, 98304, "f32")]
SHARES_BY_CHUNKS = [(130, 2, V, dtype) for dtype, sizes in (("bf16", (40960, 65539, 155656, 172032, 311297)), ("f32", (32771, 77832, 86016, 155649)))
                    for V in sizes]
BEYOND_A_PAGE = [(100, 5, 32760, "f32"), (100, 5, 32760, "bf16"), (250, 3, 32753, "bf16"), (100, 5, 32753, "f32")]
SWEEPS_BY_CHUNKS = [(12, 20, 100001, "bf16"), (12, 20, 65536, "f32"), (12, 12, 69231, "bf16")]   # seven thresholds
WIDE_PAGES = [(100, 5, V, "f32") for V in (20000, 24577, 32749, 32751, 32752)] + [(100, 5, 16377, "f32"), (3, 20, 32751, "bf16"), (3, 20, 32752, "bf16")]
# with a workspace of the least size; the walk's kernel
OVER_THE_ROW = [(128, 3, 40008, "f32", "tail_sampling_streamed_kernel<float, float, true, true>"),
                (128, 3, 65544, "bf16", "tail_sampling_streamed_kernel<bf16, float, true, true>"),
                (128, 3, 147464, "f32", "tail_sampling_streamed_kernel<float, float, true, true>"),
                (128, 3, 65547, "bf16", "tail_sampling_streamed_kernel<bf16, float, false, true>"),
                (128, 3, 147467, "f32", "tail_sampling_streamed_kernel<float, float, false, true>"),
                (1, 4, 262144, "bf16", "tail_sampling_resident_kernel<bf16, float, 2, true, true>"),
                (1, 4, 262152, "bf16", "tail_sampling_resident_kernel<bf16, float, 3, true, true>"),
                (1, 4, 393216, "bf16", "tail_sampling_resident_kernel<bf16, float, 3, true, true>"),
                (1, 4, 393728, "bf16", "tail_sampling_streamed_kernel<bf16, float, true, true>"),
                (1, 4, 262147, "bf16", "tail_sampling_resident_kernel<bf16, float, 3, false, true>")]


def edges(V, dtype, rows, row):
    """Entries next to where chunks and shares of a row begin (splits, chunks.h), and its ends, loose ones among them."""
    epv = 8 if dtype == "bf16" else 4
    splits = max(1, min(-(-max(128, min(768, rows * V >> 16)) // rows), V // 8192))
    head = -row * V % epv
    vps = -(-(V // epv) // splits)
    nfull = vps // 1024
    end = (nfull - 1) & ~1 if nfull > 2 else 0
    k = 1
    while (end >> k) + 1 > 10 or (end >> k and splits * ((end >> k) + 1) > 64):
        k += 1
    starts = [head + epv * (s * vps + j * (1024 << k)) for s in range(splits) for j in range((end >> k) + 1)]
    near = [x + d for x in starts for d in (-1, 0, epv)] + [0, 1, head, V - 1, V - 2, V - epv, V // 2]
    return sorted({x for x in near if 0 <= x < V})


@pytest.mark.parametrize("B,N,V,dtype", HEAVY_BY_CHUNKS)
def test_rejected_tokens_that_hold_most_of_the_row(B, N, V, dtype):
    """Roots with three children of which the first carries the row's largest entry, all but 4 % or 30 % of the mass (the
    normaliser is summed, or 1 - f), and is rejected; the others are unlikely."""
    rng = np.random.default_rng(V)
    z = rng.standard_normal((B, N, V), dtype=np.float32) * 2
    tok = rng.integers(V, size=(B, N)).astype(np.int32)
    for b in range(B):
        places = edges(V, dtype, B * N, b * N)
        at, left = places[b % len(places)], (0.04, 0.3)[b // len(places) % 2] if b >= len(places) else (0.04, 0.3)[b % 2]
        rest = np.log(np.exp(z[b, 0].astype(np.float64)).sum() - np.exp(float(z[b, 0, at])))
        z[b, 0, at] = rest + np.log((1 - left) / left)
        tok[b, 1] = at
        for j in (2, 3):
            tok[b, j] = (at + 1 + rng.integers(V - 1)) % V
    u = np.full((B, N + 1), 0.9995, np.float32)
    u[:, N] = rng.choice([0.0, 0.31, 0.74, 0.9999], size=B)
    par = np.tile(np.array([-1, 0, 0, 0], np.int32), (B, 1))
    compare(custom(f"heavy_{dtype}_V{V}", f32_to_bf16_bits(z) if dtype == "bf16" else z, tok, par, 2.0, 1.0, u=u))


@pytest.mark.parametrize("B,N,V,dtype", SHARES_BY_CHUNKS + BEYOND_A_PAGE)
def test_shares_around_whole_batches(B, N, V, dtype):
    compare(make_workload(f"chunks_{dtype}_{V}", B=B, N=N, V=V, dtype=dtype, temperature=0.9, tree={"kind": "chain"}, plant_frac=0.5, seed=V))


@pytest.mark.parametrize("B,N,V,dtype", SWEEPS_BY_CHUNKS)
def test_sweep_by_chunks(B, N, V, dtype):
    thetas = (0.84, 0.86, 0.88, 0.90, 0.92, 0.94, 0.96)
    w = make_workload(f"sweep_{dtype}_{V}", B=B, N=N, V=V, dtype=dtype, temperature=0.9, tree={"kind": "tree", "depth": 4, "max_children": 3},
                      plant_frac=0.6, seed=V, sweep_thetas=thetas)
    compare_ex(w, thetas=np.tile(np.array(thetas, np.float32)[:, None], (1, B)), allow_small_norm=True)


@pytest.mark.parametrize("B,N,V,dtype", WIDE_PAGES)
def test_draws_at_the_end_of_a_wide_page(B, N, V, dtype):
    # every second request: half of each row's mass and more in its last entry, or in the last vector's first
    w = make_workload(f"wide_{dtype}_{V}", B=B, N=N, V=V, dtype=dtype, temperature=0.8, tree={"kind": "chain"}, plant_frac=0.3, seed=V)
    big = np.float32(24.0)
    for b in range(0, B, 2):
        w.logits[b, :, V - 1 if b % 4 else V - 8] = f32_to_bf16_bits(big[None])[0] if dtype == "bf16" else big
    compare(w, allow_small_norm=True)


@pytest.mark.parametrize("B,N,V,dtype,kernel", OVER_THE_ROW)
def test_over_the_row_with_the_least_workspace(B, N, V, dtype, kernel):
    from paper_2601_15498_amd import binding as M
    w = make_workload(f"least_{dtype}_{V}", B=B, N=N, V=V, dtype=dtype, temperature=0.9,
                      tree={"kind": "tree", "depth": 1 if B > 1 else 2, "max_children": 2}, plant_frac=0.5, seed=V)
    d = to_device(w)

    def run(w):   # (256 bytes less than what holds the sums of chunks)
        ws = torch.empty(M.mars_workspace_bytes(B, N, V) - 256, dtype=torch.uint8, device="cuda:0")
        out = M.mars_verify(d["logits"], d["draft_tokens"], d["tree_parent"], d["theta"], w.temperature,
                            torch.from_numpy(w.uniforms).to("cuda:0"), None, workspace=ws)
        torch.cuda.synchronize()
        return out

    compare(w, cdf_guard=5e-6, allow_small_norm=True, run=run)
