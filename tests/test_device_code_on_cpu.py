"""Parts of the device code that are plain arithmetic and loads, compiled for the host and run on the CPU under
sanitizers: no GPU needed, and an access out of range ends the test instead of the GPU's work."""
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def run_on_cpu(source, tmp_path, *sanitizers, options=(), args=()):
    exe = tmp_path / "main"
    # the host half alone (no kernel is launched); the symbol of the missing device half is any address
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-fuse-cuid=none", "-Wl,--defsym=__hip_fatbin=main", "-O1", "-g",
           "-std=c++17", "-w", *options]
    for s in sanitizers:
        cmd += ["-Xarch_host", "-fsanitize=" + s, "-Xarch_host", "-fno-sanitize-recover=" + s]
    build = subprocess.run(cmd + ["-o", str(exe), os.path.join(HERE, source)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    env = dict(os.environ)
    # (another library may already be preloaded into every process; leak checking needs ptrace)
    env["ASAN_OPTIONS"] = "verify_asan_link_order=0:detect_leaks=0:abort_on_error=0"
    env["UBSAN_OPTIONS"] = "print_stacktrace=1"
    run = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, env=env, timeout=600)
    assert run.returncode == 0, (run.stdout[-1000:], run.stderr[-3000:])
    assert "runtime error" not in run.stderr and "AddressSanitizer" not in run.stderr, run.stderr[-3000:]
    return run.stdout


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_walk_reads_rows_and_nothing_around_them(tmp_path):
    out = run_on_cpu("walk_loads_main.hip", tmp_path, "address", "alignment")
    assert " 0 failed" in out, out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_walk_orders_its_residual_chain(tmp_path):
    out = run_on_cpu("walk_order_main.hip", tmp_path)
    assert " 0 out of order, a missing barrier shows" in out, out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_chunks_cover_a_row_and_end_where_the_row_reduction_ends_them(tmp_path):
    out = run_on_cpu("chunks_main.hip", tmp_path, "undefined", options=["-no-hip-rt"])
    assert " 0 failed" in out, out


OVER_THE_ROW, BY_CHUNKS, BY_PAGE, BY_WIDE_PAGE = "tail_sampling", "chunks", "page", "wide page"


def dispatch_case(B, N, V, dtype, form, offset=0, K=1, workspace="full"):
    """Arguments of dispatch_main.hip: a call of one-hot draft distributions, logits from `offset` entries behind a 16-byte boundary on,
    that takes `form`, or, if that is the beginning of a kernel's name, that one."""
    even = "false" if offset == 0 and V % (8 if dtype == "bf16" else 4) == 0 else "true"
    T = "bf16" if dtype == "bf16" else "float"
    rows = f"row_reduce_kernel<{T}, {8 if dtype == 'bf16' else 4}, true, {even}, "
    kernels = {BY_CHUNKS: f"{rows}true>|tail_onehot_kernel<{T}, {even}, false, 512>", BY_PAGE: f"row_reduce_kernel<|tail_onehot_kernel<{T}, {even}, true, 512>",
               BY_WIDE_PAGE: f"{rows}false>|tail_onehot_kernel<{T}, {even}, true, 1024>"}.get(form, f"row_reduce_kernel<|{form}")
    return B, N, V, dtype, offset, K, "onehot", workspace, kernels


def check_dispatch(tmp_path, cases):
    out = run_on_cpu("dispatch_main.hip", tmp_path, options=["-no-hip-rt"], args=[x for c in cases for x in c])
    assert f"{len(cases)} cases, 0 failed" in out, out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_one_hot_draft_distributions_take_the_quicker_walk(tmp_path):
    # both sides of every line that mars.hip draws (onehot_form)
    cases = [dispatch_case(*c) for c in [
        (64, 6, 49152, "bf16", OVER_THE_ROW), (85, 6, 49152, "bf16", BY_CHUNKS), (25, 6, 120000, "bf16", OVER_THE_ROW), (32, 6, 120000, "f32", BY_CHUNKS),
        (1, 60, 151936, "bf16", OVER_THE_ROW), (256, 26, 151936, "f32", BY_CHUNKS), (16, 26, 128256, "bf16", OVER_THE_ROW), (32, 26, 128256, "bf16", BY_CHUNKS),
        (8, 26, 100001, "bf16", OVER_THE_ROW), (85, 6, 74001, "bf16", OVER_THE_ROW), (128, 6, 65537, "bf16", BY_CHUNKS), (42, 6, 100001, "f32", BY_CHUNKS),
        (1, 6, 151936, "bf16", BY_CHUNKS), (1, 6, 100001, "bf16", BY_CHUNKS), (3, 6, 151936, "bf16", OVER_THE_ROW), (256, 65, 40000, "bf16", OVER_THE_ROW),
        (33, 12, 32000, "bf16", BY_WIDE_PAGE), (1, 12, 16369, "bf16", BY_WIDE_PAGE), (1, 12, 16368, "f32", BY_PAGE), (1, 12, 7, "bf16", BY_PAGE),
        (4, 12, 28000, "f32", OVER_THE_ROW), (86, 12, 28000, "f32", BY_WIDE_PAGE), (85, 12, 28000, "f32", OVER_THE_ROW), (4, 12, 19999, "f32", BY_WIDE_PAGE)]]
    cases += [dispatch_case(256, 26, 151936, "f32", OVER_THE_ROW, workspace="least"), dispatch_case(7, 6, 49152, "bf16", OVER_THE_ROW, K=7),
              dispatch_case(16, 6, 49152, "bf16", BY_CHUNKS, K=7), dispatch_case(5, 26, 100001, "bf16", BY_CHUNKS, K=7),
              dispatch_case(12, 26, 100001, "bf16", BY_CHUNKS, K=4), dispatch_case(16, 26, 100001, "bf16", OVER_THE_ROW, K=3), dispatch_case(64, 6, 65536, "bf16", OVER_THE_ROW, offset=1)]
    check_dispatch(tmp_path, cases)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_gpu_tests_of_one_hot_draft_distributions_run_the_forms_they_name(tmp_path):
    from tests import test_gpu_draw as draw, test_gpu_onehot_forms as forms
    cases = [dispatch_case(*c, BY_CHUNKS) for c in forms.HEAVY_BY_CHUNKS + forms.SHARES_BY_CHUNKS + forms.BEYOND_A_PAGE]
    cases += [dispatch_case(*c, BY_CHUNKS, K=7) for c in forms.SWEEPS_BY_CHUNKS]
    cases += [dispatch_case(*c, BY_WIDE_PAGE) for c in forms.WIDE_PAGES]
    cases += [dispatch_case(*c, workspace="least") for c in forms.OVER_THE_ROW]
    for dtype, B, V, _, _, rejected in draw.BY_CHUNKS:
        call = B, 1 + rejected, V, "bf16" if dtype == draw.BF16 else "f32"
        cases += [dispatch_case(*call, BY_CHUNKS), dispatch_case(*call, OVER_THE_ROW, workspace="least")]
    check_dispatch(tmp_path, cases)


def check_plans(tmp_path, cases):
    out = run_on_cpu("lm_plan_main.hip", tmp_path, options=["-no-hip-rt"], args=[x for c in cases for x in c])
    assert f"{len(cases)} cases, 0 failed" in out, out


# B, N, V, H, sampling; then what the case stands for: bands of slabs, launches, cells shared by two work-groups
PLANS = [
    (1, 40, 5003, 128, 0, 1, 1, 0), (1, 100, 60001, 128, 0, 1, 1, 0), (1, 520, 33011, 128, 0, 1, 1, 0),
    (1, 1000, 32400, 128, 1, 1, 1, 1),        # shared cells in the last column of a single band
    (2, 1000, 12001, 128, 0, 2, 1, 1), (3, 1000, 12001, 128, 0, 2, 1, 1), (3, 800, 12000, 128, 1, 2, 1, 1),
    (8, 900, 9001, 128, 0, 3, 1, 0),
    (16, 60, 151936, 4096, 1, 1, 1, 0), (16, 60, 151936, 4096, 0, 1, 1, 0), (256, 26, 151936, 4096, 0, 2, 1, 1),
    (1, 1, 304, (1 << 22) + 128, 0, 1, 1, 0),   # beyond what a buffer spans
    (1, 2, (1 << 25) + 8, 128, 1, 1, 1, 0),
    (4096, 1024, (1 << 25) + 8, 128, 0, "-", 9, "-"),   # more units than a launch takes
    (4096, 1024, (1 << 24) + 256, 128, 0, "-", 2, "-"), (1000, 1024, (1 << 27) + 8, 128, 1, "-", 8, "-"),
]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_lm_head_work_is_dealt_out_exactly_once(tmp_path):
    rng = random.Random(7)
    cases = list(PLANS)
    for _ in range(300):
        rows = int(2 ** rng.uniform(0, 14))
        n = rng.randint(1, min(rows, 1024))
        sampling = rng.randint(0, 1)
        v = int(2 ** rng.uniform(3, 18.5)) // (8 if sampling else 1) * (8 if sampling else 1)
        cases.append((max(1, rows // n), n, max(8, v), 128 * rng.randint(1, 64), sampling, "-", "-", "-"))
    check_plans(tmp_path, [c + ("-",) for c in cases])


# Sizes at which another form was measured to be slower, with a weight that lies in the cache and with one that does not: B, N,
# V, H, sampling and the form.  Many rows under sampling with few hidden elements; tiles so narrow that the merging of
# their partial results costs more than they save; and sizes that keep the form they had.
FORMS = [
    (32, 62, 64000, 1024, 1, "192x256"), (32, 62, 100000, 1024, 1, "192x256"), (32, 62, 128256, 1024, 1, "192x256"),
    (32, 62, 151936, 1024, 1, "192x256"), (37, 55, 9496, 640, 1, "192x256"), (36, 45, 62816, 640, 1, "192x256"),
    (1, 60, 32000, 1024, 0, "64x256ring"), (1, 60, 32000, 1024, 1, "64x256ring"), (1, 40, 32000, 1024, 1, "64x256ring"),
    (1, 60, 12000, 4096, 0, "64x64ring"), (1, 60, 32000, 4096, 0, "64x128ring"), (2, 60, 32000, 4096, 1, "128x128ring"),
    (1, 60, 151936, 4096, 0, "64x256ring-once"), (16, 60, 151936, 4096, 0, "192x256"), (16, 60, 151936, 4096, 1, "192x256"),
    (256, 26, 151936, 4096, 0, "256x256"),
]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_lm_head_takes_the_form_that_was_measured_to_be_faster(tmp_path):
    check_plans(tmp_path, [c[:5] + ("-", "-", "-") + c[5:] for c in FORMS])


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_lm_head_cases_of_the_gpu_tests_run_the_forms_they_name(tmp_path):
    from tests.test_gpu_lmhead import RING_SHAPES
    from tests.test_gpu_lmhead_sampling import STORE_EDGE_FORMS, STORE_EDGES
    cases = [(1, rows, V, H, int(T > 0.0), form) for rows, V, H, T, form in RING_SHAPES]
    assert len(STORE_EDGES) == len(STORE_EDGE_FORMS)
    cases += [(c["B"], c["N"], c["V"], c["H"], 1, form) for c, form in zip(STORE_EDGES, STORE_EDGE_FORMS)]
    check_plans(tmp_path, [c[:5] + ("-", "-", "-") + c[5:] for c in cases])
