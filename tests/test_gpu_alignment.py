"""The worker passes at every alignment of rows and segments: worker rows 4, 8
and 12 bytes off a 16-byte boundary, segments that start and end anywhere (so
the four marks of a float4 lie in two words, and last chunks hold 1 to 2047
components), RBGS blocks that a float4 straddles; each against the oracle, bit
for bit."""
import dataclasses

import pytest

import synth
from gpu_harness import Case, run_lockstep

pytestmark = pytest.mark.gpu

OPT_LIST = 7     # GMC_OPT_CHANGE_LIST
SIZES = [2051, 2047, 4, 1, 6149, 2048, 2049, 3, 8195, 30]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def wl(comp, sizes, ratio, **kw):
    return dataclasses.replace(synth.workload("tiny"), name="align", sizes=list(sizes), K=3, ratio=ratio,
                               compressor=comp, steps=4, **kw)


@pytest.mark.parametrize("pad", [0, 1, 2, 3])
@pytest.mark.parametrize("how", ["dense", "sparse", "inplace", "detach", "approx"])
def test_rows_and_segments_off_alignment(pad, how):
    kw = {"dense": dict(), "sparse": dict(iteration=True, sparse_w=True),
          "inplace": dict(inplace="iteration", sparse_w=True, options=((OPT_LIST, 3),)),
          "detach": dict(detach="fused", lam=0.5, sparse_w=True), "approx": dict(iteration=True, sparse_w=True)}[how]
    w = wl("approx", [sum(SIZES)], 0.02) if how == "approx" else wl("topk_seg", SIZES, 0.05)
    run_lockstep(Case(w, steps=4, row_pad=pad, label="pad %d %s" % (pad, how), **kw), verbose=False)


@pytest.mark.parametrize("pad", [0, 1, 2, 3])
@pytest.mark.parametrize("block", [1, 3, 333, 1000])
@pytest.mark.parametrize("detach", [False, True])
def test_rbgs_off_alignment(pad, block, detach):
    w = wl("rbgs", [10_007], 0.1, block=block)
    kw = dict(detach="fused", lam=0.5) if detach else dict(fused_apply=True)
    run_lockstep(Case(w, steps=4, row_pad=pad, sparse_w=True, label="pad %d B %d" % (pad, block), **kw),
                 verbose=False)
