"""Which launch the GPU tests' problems get, without a GPU: a new rule of the dispatch shows here if it takes a test's problems to
another kernel, or leaves a kernel without a comparison with the oracle."""
import test_gpu_causal
import test_gpu_launches
import test_gpu_ragged
import test_gpu_short
import test_gpu_split
import test_gpu_stage
import test_gpu_wide
from paper_2312_11918_amd import workloads
from _routes import routes


def _params(test):
    """The argument lists of a parametrised test, those of its last (lowest) decorator first."""
    return [m.args[1] for m in test.pytestmark if m.name == "parametrize"]


def _with_and_without(problems):
    """Launch with the workspace that a call takes; where that is another than without one, both."""
    both = zip(routes([(*p, 1) for p in problems]), routes([(*p, 0) for p in problems]))
    return [a if a == b else f"{a} | {b}" for a, b in both]


def test_launches():
    cases = test_gpu_launches.CASES
    assert routes([(B, H, Nq, Nk, d, causal, 1) for _, B, H, Nq, Nk, d, _, causal, _ in cases]) == [c[0] for c in cases]
    masked = test_gpu_launches.MASKED
    problems = [(B, H, Nq, Nk, d, 0) for _, _, B, H, Nq, Nk, _, d in masked]
    assert _with_and_without(problems) == [a if a == b else f"{a} | {b}" for a, b, *_ in masked]


def test_cut_keys():
    got = _with_and_without([(B, H, Nq, Nk, d, causal) for B, H, Nq, Nk, d, _, causal, _, _ in test_gpu_split.CASES])
    assert got == ["short slices | short", "short", "short slices | short", "short slices | halves", "short slices | halves",
                   "short slices | stage", "short slices | stage", "halves", "short", "short", "short", "slices | halves",
                   "short slices | short", "short slices | single", "short", "halves", "single", "halves"]
    masked = _params(test_gpu_split.test_keys_masked_by_the_lowest_value)[1]
    got = _with_and_without([(1, 2, Nq, Nk, d, 0) for Nq, Nk, _, d, _ in masked])
    assert got == ["short", "short slices | short", "short slices | short", "short slices | halves", "short slices | stage"]
    edges = _params(test_gpu_split.test_workspace_one_byte_short_and_exact)[0]
    got = _with_and_without([(B, H, Nq, Nk, d, causal) for B, H, Nq, Nk, d, causal in edges])
    assert got == ["short slices | short", "slices | halves", "slices | halves", "short slices | stage", "decode",
                   "short slices | halves", "short slices | stage", "short slices | short", "short slices | short"]
    for test in (test_gpu_split.test_split_on_another_stream_and_in_a_graph,
                 test_gpu_split.test_capture_begun_without_torch_holds_no_pool_memory):
        got = _with_and_without([(1, 8, Nq, Nk, d, 0) for Nq, Nk, d in _params(test)[0]])
        assert got == ["short slices | halves", "decode", "slices | halves"]


def test_partial_tiles():
    (cases,) = _params(test_gpu_ragged.test_ragged_parity_elementwise)
    got = _with_and_without([(B, H, Nq, Nk, d, causal) for B, H, Nq, Nk, d, _, causal, _ in cases])
    assert got == ["decode", "decode"] + ["short"] * 9 + ["stage"] + ["short"] * 6
    (headline,) = _params(test_gpu_ragged.test_ragged_headline_shape_whole_output)
    assert _with_and_without([(8, 16, N, N, 128, causal) for N, causal in headline]) == ["wide", "partial tiles", "wide"]
    assert set(_with_and_without([(B, H, Nq, Nk, 128, causal) for B, H, Nq, Nk, _, causal in test_gpu_wide.CASES])) == {"wide"}


def test_causal():
    (cases,) = _params(test_gpu_causal.test_causal_parity_elementwise)
    got = _with_and_without([(B, H, N, N, d, 1) for B, H, N, d, _, _ in cases])
    assert got == ["short"] * 7 + ["short slices | short"] + ["short"] * 2 + ["tiles of 256 rows"] * 2
    full = [workloads.CONFIGS[i] for i in (2, 3, 4, 5)]
    assert _with_and_without([(w.B, w.H, w.N, w.N, w.d, 1) for w in full]) == ["tiles", "tiles of 256 rows", "tiles of 256 rows", "stage"]


def test_staged():
    got = _with_and_without([(B, H, Nq, Nk, 256, causal) for B, H, Nq, Nk, _, causal, _ in test_gpu_stage.CASES_256])
    assert got == ["short"] * 4 + ["stage", "short", "stage", "stage"]
    assert set(_with_and_without([(B, H, Nq, Nk, 64, causal) for B, H, Nq, Nk, _, causal, _ in test_gpu_stage.CASES])) == {"stage"}
    assert set(_with_and_without([(B, H, N, N, d, 0) for B, H, N, d, _ in test_gpu_stage.SAME_BITS])) == {"stage"}
    assert set(_with_and_without([(B, H, Nq, Nk, d, causal) for B, H, Nq, Nk, d, _, causal in test_gpu_stage.SINKING])) == {"stage"}
    assert _with_and_without([(*test_gpu_stage.COMPANY[d], d, 0) for d in (64, 256)]) == ["stage", "stage"]


def test_every_launch_is_compared_with_the_oracle():
    # launch x head dimension x mask, each with a problem that an oracle test runs with the workspace that the call takes
    problems = [(B, H, Nq, Nk, d, causal, 1) for _, B, H, Nq, Nk, d, _, causal, _ in test_gpu_launches.CASES]
    problems += [(B, H, Nq, Nk, d, causal, 1) for B, H, Nq, Nk, d, _, causal, *_ in test_gpu_short.CASES]
    problems += [(B, H, Nq, Nk, d, causal, 1) for B, H, Nq, Nk, d, _, causal, _, _ in test_gpu_split.CASES]
    problems += [(B, H, Nq, Nk, 128, causal, 1) for B, H, Nq, Nk, _, causal in test_gpu_wide.CASES]
    problems += [(B, H, Nq, Nk, d, causal, 1) for d, cases in ((64, test_gpu_stage.CASES), (256, test_gpu_stage.CASES_256))
                 for B, H, Nq, Nk, _, causal, _ in cases]
    problems += [(B, H, N, N, d, 1, 1) for B, H, N, d, _, _ in _params(test_gpu_causal.test_causal_parity_elementwise)[0]]
    problems += [(w.B, w.H, w.N, w.N, w.d, 0, 1) for w in (workloads.CONFIGS[i] for i in (2, 3, 4, 5))]
    problems += [(4, 64, 256, 256, 256, 0, 1)]   # test_parity_d256_chained_q_tiles
    covered = {(launch, p[4], bool(p[5])) for launch, p in zip(routes(problems), problems)}
    every = {(launch, d, causal) for launch in ("short", "short slices", "slices", "partial tiles", "tiles")
             for d in (64, 128, 256) for causal in (False, True)}
    every |= {("halves", d, causal) for d in (64, 128) for causal in (False, True)} | {("single", 256, True)}
    every |= {("stage", d, causal) for d in (64, 256) for causal in (False, True)}
    every |= {("wide", 128, causal) for causal in (False, True)}
    every |= {("tiles of 256 rows", 64, False), ("tiles of 256 rows", 128, False), ("tiles of 256 rows", 128, True)}
    assert covered == every, (every - covered, covered - every)
