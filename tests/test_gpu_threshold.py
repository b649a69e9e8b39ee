"""The speculative threshold over a long run.  Once the residual has built up
(about n/k steps) a component reaches the threshold as often as it is sent, so
a threshold at rank k would leave too few candidates every other step; the
rank follows the measured growth instead.  Results are the oracle's bit for
bit either way; the count of full-data selections is what this pins."""
import dataclasses

import pytest

import synth
from gpu_harness import Case, run_lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("comp,sizes,ratio", [
    ("topk", [30_001], 0.02),
    ("topk_seg", [9000, 6007, 4099, 12_000], 0.05),
    ("topk", [4097], 0.3),
])
def test_steady_state_resolves_from_candidates(comp, sizes, ratio):
    wl = dataclasses.replace(synth.workload("tiny"), name="steady", sizes=sizes, K=3, ratio=ratio, compressor=comp,
                             steps=500)
    batches = [wl.grads(t) for t in range(4)]
    wl.grads = lambda t: batches[t % 4]   # four batches in turn, as a small epoch
    st = run_lockstep(Case(wl, steps=500, iteration=True, sparse_w=True, label="steady"), check_every=125,
                      verbose=False)
    total = st["from_candidates"] + st["full_data"]
    # the first steps of unsampled segments and the odd fluctuation (the rank
    # leaves four standard deviations of a count): a threshold at rank k takes
    # the full-data path on a third of them.  Segments of a few components
    # (k = 1) have no steady rank and are not meant.
    assert st["full_data"] <= 0.03 * total + 4 * len(sizes) * wl.K, st
