"""The selection at the edges of its paths: segments at and around the size
selected whole (4096), pairs at and around the sizes one workgroup takes (k =
1024 and 15,000), ties, zeros and non-finite values in them, candidates
crowded into a few chunks; and the server pass at and around its batch sizes.
Everything against the oracle (or the sum in worker order), bit for bit."""
import dataclasses

import numpy as np
import pytest

import synth
from gpu_harness import Case, run_lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def wl(sizes, ratio, comp="topk_seg", K=2):
    return dataclasses.replace(synth.workload("tiny"), name="edges", sizes=list(sizes), K=K, ratio=ratio,
                               compressor=comp, steps=4)


HOOKS = {
    "plain": lambda t, g: g,
    "ties": lambda t, g: np.sign(g).astype(np.float32),
    "zeros": lambda t, g: np.where(np.arange(g.shape[1]) % 97 == 0, g, 0).astype(np.float32),
    "crowded": lambda t, g: (g * np.where(np.arange(g.shape[1]) % 16384 < 700, 1000, 1)).astype(np.float32),
    "non-finite": lambda t, g: np.where(np.arange(g.shape[1]) % 1999 == 0, [np.inf, np.nan][t % 2], g).astype(np.float32),
}


@pytest.mark.parametrize("hook", sorted(HOOKS))
@pytest.mark.parametrize("sizes,ratio", [
    ([4096, 4097, 1, 2, 255, 8192, 4095], 0.1),      # whole segments beside others
    ([1, 4096, 257], 1.0),                            # whole segments only, all kept
    ([102_400], 0.01),                                # k = 1024: the smaller workgroup's largest
    ([102_401], 0.01),                                # k = 1025
    ([50_000, 6000], 0.3),                            # k = 15,000 beside a small pair
    ([50_001, 6000], 0.3),                            # k = 15,001: the multi-workgroup passes
])
def test_selection_paths(sizes, ratio, hook):
    run_lockstep(Case(wl(sizes, ratio), steps=4, iteration=True, sparse_w=True, grad_hook=HOOKS[hook],
                      label="%s %g %s" % (sizes, ratio, hook)), verbose=False)


def test_segments_selected_whole_are_not_fallbacks():
    st = run_lockstep(Case(wl([4096, 1, 300], 0.1), steps=4, iteration=True, label="whole"), verbose=False)
    assert (st["from_candidates"], st["full_data"], st["whole_segments"]) == (0, 0, 3 * 2 * 4), st


def test_pair_stats_tell_the_paths_apart():
    import torch
    from paper_1905_12948_amd import Gmc
    K, seg = 2, [0, 4096, 4097, 104_097]
    g = Gmc(seg[-1], K, "topk_seg", 0.01, 0.9, 0.1, segments=seg)
    w, e = torch.zeros(seg[-1], device="cuda:0"), torch.zeros((K, seg[-1]), device="cuda:0")
    msg = g.alloc_messages("cuda:0")
    for _ in range(2):
        g.iteration(w, w.clone(), torch.randn((K, seg[-1]), device="cuda:0"), e, *msg)
    mode, cand = g.pair_stats()
    assert mode[:, :2].tolist() == [[2, 2]] * K and not cand[:, :2].any()
    assert (mode[:, 2] == 0).all() and (cand[:, 2] >= 1000).all()
    g.set_option(1, 1)  # GMC_OPT_FORCE_FULL_SELECT
    g.iteration(w, w.clone(), torch.randn((K, seg[-1]), device="cuda:0"), e, *msg)
    mode, _ = g.pair_stats()
    assert mode.tolist() == [[2, 2, 1]] * K


@pytest.mark.parametrize("K,per", [(1, 0), (1, 1024), (1, 1025), (3, 341), (3, 342), (4, 512), (4, 513), (16, 33),
                                   (16, 65), (16, 600), (2, 4096), (64, 1), (64, 40)])
def test_server_batches(K, per):
    """Ranges of K * per entries: one batch, several, a round per worker."""
    import torch
    from paper_1905_12948_amd.gmc import aggregate_static
    d = 3 * 4096 + 5
    rng = np.random.default_rng(100 * K + per)
    n = per + 2
    idx = np.zeros((K, n), np.int32)
    for k in range(K):  # the middle range gets `per` entries, the last components two
        idx[k] = np.concatenate([4096 + np.sort(rng.choice(4096, per, replace=False)), [d - 2, d - 1]])
    val = rng.standard_normal((K, n)).astype(np.float32)
    want = np.zeros(d, np.float32)
    for k in range(K):
        want[idx[k]] = want[idx[k]] + val[k]
    want = -(np.float32(0.1 / K) * want)
    upd = torch.empty(d, dtype=torch.float32, device="cuda:0")
    aggregate_static(d, K, 0.1, torch.from_numpy(idx).to("cuda:0"), torch.from_numpy(val).to("cuda:0"),
                     torch.full((K,), n, dtype=torch.int64, device="cuda:0"), upd)
    assert np.array_equal(upd.cpu().numpy().view(np.uint32), want.view(np.uint32))
