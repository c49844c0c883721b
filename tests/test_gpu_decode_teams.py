"""Decoding instances at their edges: profile sizes on both sides of every change
of vectors per lane or waves per target, with random transitions at every node
(a value taken from the wrong neighbour at a lane's, or a wave's, edge changes
the posteriors) and with zero-probability transitions (the gated instances)."""
import numpy as np
import pytest

import paper_2111_06340_amd as hg
from conftest import random_profile
from synth import gen
from test_gpu_decode import _check_selection, compare_decode, gpu, run  # noqa: F401
from test_gpu_parity import _ragged_db, announce
from test_oracle_decode import _zero_transition_profile

pytestmark = pytest.mark.gpu

SIZES = [192, 193, 257, 320, 321, 384, 385, 512, 513, 640, 641, 768, 769, 1024, 1025, 1280, 1281, 1536, 1537, 1792, 1793,
         2048, 2049, 2560, 2561, 3072]


@pytest.mark.parametrize("M", SIZES)
def test_random_transitions(M):
    prof = random_profile(M, 3000 + M, alpha=0.3, talpha=0.6)
    res_, off = _ragged_db(prof, M, lengths=[M + M // 4, 2, 130, 1, 65], homolog_every=2)
    res, g = run(prof, res_, off, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), decode_all=True)
    st = compare_decode(prof, res_, off, g, _check_selection(res, g, True), f"teams M={M}")
    announce(f"decode teams M={M}: {st}")
    assert st["regions"] >= 1


@pytest.mark.parametrize("M", [128, 320, 512, 641, 1000, 1281, 2100])
def test_zero_transitions(M):
    prof = _zero_transition_profile(M, 70 + M)
    res_, off = _ragged_db(prof, M, lengths=[M + M // 4, 3, 129], homolog_every=1)
    res, g = run(prof, res_, off, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), decode_all=True)
    st = compare_decode(prof, res_, off, g, _check_selection(res, g, True), f"zero transitions M={M}")
    announce(f"decode teams, zero transitions M={M}: {st}")


def test_regions_at_both_ends():
    """A region that starts at residue 1 and one that ends at the last, in targets of one and of several windows."""
    prof = gen.make_profile(60, 5)
    res_, off = _ragged_db(prof, 9, lengths=[60, 63, 64, 65, 128, 129], homolog_every=1)
    res, g = run(prof, res_, off, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), decode_all=True)
    compare_decode(prof, res_, off, g, _check_selection(res, g, True), "ends")
    assert any(d["s"] == 1 for d in g["doms"])


@pytest.mark.parametrize("M,longest", [(256, 3900), (256, 7000), (384, 8200), (734, 5300), (734, 8000), (1500, 3000)])
def test_few_slots(M, longest):
    """Static scratch for 9 to 20 blocks: every target decoded once, as with as many slots as fit the chip."""
    import torch
    prof = gen.make_profile(M, 8000 + M)
    rng = np.random.default_rng(M)
    lengths = [longest] + [int(v) for v in rng.integers(20, 90, size=300)]
    res_, off = _ragged_db(prof, M, lengths=lengths, homolog_every=3)
    P, D = hg.Profile(prof, 0.0, 0.0, 0.0), hg.Database(res_, off)
    announce(f"few slots M={M} longest={longest} n={D.n}")
    a, b = (hg.decode(P, D, None, pp=True, aln=True, static=s) for s in (True, False))
    torch.cuda.synchronize()
    assert hg.domains_table(a) == hg.domains_table(b)
    for k in ("n_dom", "exp_dom", "pp", "aln"):
        assert torch.equal(a[k], b[k]), k
    assert bool(torch.isfinite(a["exp_dom"]).all())


@pytest.mark.parametrize("M", [60, 150, 600, 1100])
def test_transitions_below_the_float_range(M):
    """A transition that is 0 in the kernel's floats is closed like a 0, also across lanes and waves."""
    import torch
    prof = gen.make_profile(M, 8100 + M)
    rng = np.random.default_rng(M)
    seqs = []
    for gap in (3, 20, M // 3):   # homologs without a stretch of nodes: the alignment would delete them
        h = prof.match.argmax(axis=1).astype(np.uint8)
        at = int(rng.integers(5, M - gap - 5))
        seqs.append(np.concatenate([h[:at], h[at + gap:]]))
    off = np.concatenate([[0], np.cumsum([s.size for s in seqs])]).astype(np.int64)
    D = hg.Database(np.concatenate(seqs), off)
    announce(f"transitions below the float range M={M} n={D.n}")
    got = []
    for dd in (0.0, 1e-50):
        prof.trans[:, 5:7] = [1.0 - dd, dd]
        got.append(hg.decode(hg.Profile(prof, 0.0, 0.0, 0.0), D, None, pp=True, aln=True))
        torch.cuda.synchronize()
    assert hg.domains_table(got[0]) == hg.domains_table(got[1])
    for k in ("exp_dom", "pp", "aln"):
        assert torch.equal(got[0][k], got[1][k]), k
