"""The selection at the edges of its paths: segments at and around the size
selected whole (4096), pairs at and around the sizes one workgroup takes (k =
1024 and 14,600, 512 and 2048 chunks of 2048), ties, zeros and non-finite
values in them, candidates crowded into a few chunks; and the server pass at and around its batch sizes.
Everything against the oracle (or the sum in worker order), bit for bit."""
import dataclasses

import numpy as np
import pytest

import synth
from paper_1905_12948_amd.gmc import count
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
@pytest.mark.parametrize("sizes,ratio,solo", [
    ([4096, 4097, 1, 2, 255, 8192, 4095], 0.1, True),  # whole segments beside others
    ([1, 4096, 257], 1.0, False),                       # whole segments only, all kept
    ([102_400], 0.01, True),                            # k = 1024: the smaller workgroup's largest
    ([102_401], 0.01, True),                            # k = 1025
    ([46_666, 6000], 0.3, True),                        # k = 14,000 beside a small pair, in one launch
    ([48_667, 6000], 0.3, False),                       # k = 14,601: the multi-workgroup passes
    ([50_000, 6000], 0.3, False),
])
def test_selection_paths(sizes, ratio, solo, hook):
    """solo: one workgroup takes the pairs once their candidates fit, within
    twelve steps of an undisturbed run."""
    st = run_lockstep(Case(wl(sizes, ratio), steps=12, iteration=True, sparse_w=True, grad_hook=HOOKS[hook],
                           label="%s %g %s" % (sizes, ratio, hook)), verbose=False)
    assert st["one_workgroup"] > 0 if solo and hook == "plain" else st["one_workgroup"] == 0 or solo, st


@pytest.mark.parametrize("n,ratio,solo", [(2 * 256 * 2048, 0.0009, True), (2 * 256 * 2048 + 1, 0.0009, False),
                                          (2 * 1024 * 2048, 0.0005, True), (2 * 1024 * 2048 + 1, 0.0005, False)])
def test_longest_segments_of_one_workgroup(n, ratio, solo):
    """Two chunks a thread, and one component more.  From step 3 on the
    gradients are small, so the residual stands still and the candidates fit."""
    st = run_lockstep(Case(wl([n], ratio, comp="topk"), steps=7, iteration=True, sparse_w=True,
                           grad_hook=lambda t, g: g if t < 3 else g * np.float32(1e-4), label="n %d" % n),
                      check_every=3, verbose=False)
    assert (st["one_workgroup"] > 0) == solo, st


@pytest.mark.parametrize("sizes,ratio", [([4097], 0.2), ([6000], 0.3)])
def test_candidates_far_above_the_threshold(sizes, ratio):
    """Half of the gradients a thousand times larger from one step to the next:
    more than k candidates lie over two octaves above the threshold that
    collected them, beyond the first histogram, in lists that fit."""
    def jump(t, g):
        return g if t < 2 else (g * np.where(np.arange(g.shape[1]) % 2, 1, 1000)).astype(np.float32)
    st = run_lockstep(Case(wl(sizes, ratio), steps=3, iteration=True, grad_hook=jump, label="jump"), verbose=False)
    assert st["one_workgroup"] == 2 * 2, st  # steps 1 and 2; step 0 has no threshold


def test_steps_with_and_without_the_one_workgroup_launch():
    """k = 10,000: the launch waits for ceil(0.4 n / (16,384 - k)) = 3 steps,
    and forced full-data steps do without it; neither it nor its marks of an
    earlier step change what a step sends."""
    import torch
    from paper_1905_12948_amd import Gmc
    d, K = 33_333, 2
    grads = torch.randn((4, K, d), device="cuda:0")

    def run(force):
        g = Gmc(d, K, "topk", 0.3, 0.9, 0.1)
        w, wp, e = (torch.zeros(s, device="cuda:0") for s in (d, d, (K, d)))
        msg, out, one = g.alloc_messages("cuda:0"), [], []
        for t in range(24):
            g.set_option(1, int(force(t)))  # GMC_OPT_FORCE_FULL_SELECT
            g.iteration(w, wp, grads[t % 4], e, *msg)
            w, wp = wp, w
            out.append([x.clone() for x in (w, e, *msg)])
            one.append(g.stats()["one_workgroup"])
        return out, np.diff([0] + one)
    want, none = run(lambda t: True)
    got, one = run(lambda t: t % 5 == 4)
    assert not none.any() and not one[:3].any() and not one[4::5].any() and one[10:].sum() > 0, one
    for t, (x, y) in enumerate(zip(got, want)):
        assert all(torch.equal(p, q) for p, q in zip(x, y)), t


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


# entries per worker in one range: one round of 256, one batch, several, a
# round per worker, with the larger batch (1024 entries) and, where most ranges
# are empty, the smaller one (512)
DENSE = [(1, 0), (1, 1024), (1, 1025), (3, 341), (3, 342), (4, 512), (4, 513), (16, 33), (16, 65), (16, 600), (2, 4096),
         (64, 1), (64, 40)]
SPARSE = [(1, 1), (1, 256), (1, 257), (1, 513), (2, 128), (2, 129), (3, 170), (3, 171), (4, 200), (4, 300), (16, 16),
          (16, 17), (16, 33), (16, 200), (64, 4), (64, 5), (64, 70)]


@pytest.mark.parametrize("K,per,empty", [(K, n, 1) for K, n in DENSE] + [(K, n, 100) for K, n in SPARSE])
def test_server_batches(K, per, empty):
    import torch
    from paper_1905_12948_amd.gmc import aggregate_static
    d = (2 + empty) * 4096 + 5
    rng = np.random.default_rng(100 * K + per)
    n = per + 2
    idx = np.zeros((K, n), np.int32)
    for k in range(K):  # the second range gets `per` entries, the last components two
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


@pytest.mark.parametrize("calls", ["iteration", "two calls", "momentum on the server"])
@pytest.mark.parametrize("K,per,empty", [(1, 1024, 1), (1, 1025, 1), (3, 341, 1), (3, 342, 1), (4, 600, 1), (16, 65, 1),
                                         (2, 128, 100), (2, 129, 100), (2, 256, 100), (2, 257, 100), (4, 129, 100),
                                         (4, 300, 100), (16, 16, 100), (16, 33, 100)])
def test_server_batches_applied(K, per, empty, calls):
    """The same with the update applied: every worker's whole message in one
    range, where its gradients are a thousand times larger."""
    d = (2 + empty) * 4096 + 5
    how = {"iteration": dict(iteration=True, sparse_w=True), "two calls": dict(fused_apply=True, write_update=False),
           "momentum on the server": dict(rule="server_momentum")}[calls]

    def crowd(t, g):
        g = g.copy()
        g[:, 4096:8192] *= np.float32(1000)
        return g
    w = wl([d], per / d, comp="topk", K=K)
    assert count(d, per / d) == per
    run_lockstep(Case(w, steps=4, grad_hook=crowd, label="K %d per %d" % (K, per), **how), verbose=False)
