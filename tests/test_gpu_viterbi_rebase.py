"""Viterbi scores past the int16 range, bit-exact against the oracle, for every
instance that re-bases its values and the first sizes that leave overflows to
the int32 rescore: targets that reach the limit once and many times, cut so
that they end on every row around it; inserts that grow the values; profiles
whose scores don't allow re-basing; all ways to run the stages."""
import numpy as np
import pytest

import oracle
import paper_2111_06340_amd as hg
import test_viterbi_rebase_model as model
from synth import gen

pytestmark = pytest.mark.gpu

F = (1.0, 1.0, 1.0)
TRANS = [0.9, 0.05, 0.05, 0.6, 0.4, 0.5, 0.5]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    hg.lib()


def _profile(M, kind):
    """A profile with one likely residue per node, and its consensus."""
    rng = np.random.default_rng(9000 + M)
    bg = gen.BACKGROUND.copy()
    c = rng.integers(1, 20, size=M)
    match = np.full((M, 20), 0.1 / 19)
    match[np.arange(M), c] = 0.9
    insert = np.tile(bg, (M - 1, 1))
    trans = np.tile(TRANS, (M - 1, 1))
    if kind == "inserts":        # residue 0 scores in an insert and keeps it open
        insert[:] = 0.2 / 19
        insert[:, 0] = 0.8
        trans[:, 3:5] = [0.05, 0.95]
    elif kind == "no_insert":    # one node can't open an insert: its score is minus infinity
        trans[M // 2] = [0.95, 0.0, 0.05, 0.6, 0.4, 0.5, 0.5]
    return gen.Profile(M, bg, match, insert, trans), c.astype(np.uint8)


def _targets(M, c, kind):
    rng = np.random.default_rng(M)
    rep = np.concatenate([c] * (2600 // M + 1))[:2600]
    seqs = [rep, np.concatenate([c, rep[::-1], rep]), gen.background_residues(rng, 700)]
    # a match scores about 2,100 units, so these cross the limit of 32,767
    seqs += [rep[:n] for n in range(8, 41)]
    for n in (63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025):
        seqs.append(rep[:n])
        mixed = gen.background_residues(rng, n)
        at = rng.random(n) < 0.7
        mixed[at] = rep[:n][at]
        seqs.append(mixed)
    if kind == "inserts":
        for n in (3, 40, 200, 1500):
            z = np.zeros(n, np.uint8)
            seqs += [z, np.concatenate([c[: M // 2 + 1], z, c[M // 2 + 1:], rep]), np.concatenate([rep, z, rep])]
    return seqs


@pytest.mark.parametrize("kind", ["plain", "inserts", "no_insert"])
@pytest.mark.parametrize("M", [3, 40, 64, 127, 128, 129, 256, 257, 384, 385, 512, 640, 768, 769, 1025])
def test_overflows(M, kind):
    import torch
    prof, c = _profile(M, kind)
    seqs = _targets(M, c, kind)
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([s.size for s in seqs])
    res = np.concatenate(seqs)
    o = oracle.search(oracle.OracleProfile(prof), res, off, (0.0, 0.0, 0.0), F, nthreads=8)
    n_ovf = int(np.sum((o["flags"] & oracle.F_VIT_OVF) != 0))
    assert n_ovf >= 2
    P, D = hg.Profile(prof, 0.0, 0.0, 0.0), hg.Database(res, off)
    E = D.share()
    for mode in (1, 2):
        print(f"[rebase] M={M} {kind} mode={mode} n={D.n} overflows={n_ovf}", flush=True)
        for h in (D, E):
            hg.hmm_db_fused_tail(h.handle, mode)
        outs = [hg.search(P, D, F)] + hg.search_group([P, P], [D, E], [F, F])
        torch.cuda.synchronize()
        for out in outs:
            g = {k: v.cpu().numpy() for k, v in out.items()}
            for k in ("vit", "flags"):
                bad = np.nonzero(g[k] != o[k])[0]
                assert bad.size == 0, f"M={M} {kind}: {k} differs at {bad[:5]}: {g[k][bad[:5]]} {o[k][bad[:5]]}"
            assert g["counts"][1] == n_ovf


def _compare(prof, seqs, what):
    """Scores, flags and the overflow count of both ways to run the stages; returns the overflows."""
    import torch
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([s.size for s in seqs])
    res = np.concatenate(seqs)
    o = oracle.search(oracle.OracleProfile(prof), res, off, (0.0, 0.0, 0.0), F, nthreads=8)
    n_ovf = int(np.sum((o["flags"] & oracle.F_VIT_OVF) != 0))
    P, D = hg.Profile(prof, 0.0, 0.0, 0.0), hg.Database(res, off)
    for mode in (1, 2):
        print(f"[rebase] {what} M={prof.M} mode={mode} n={D.n} overflows={n_ovf}", flush=True)
        hg.hmm_db_fused_tail(D.handle, mode)
        out = hg.search(P, D, F)
        torch.cuda.synchronize()
        g = {k: v.cpu().numpy() for k, v in out.items()}
        for k in ("vit", "flags"):
            bad = np.nonzero(g[k] != o[k])[0]
            assert bad.size == 0, f"{what} M={prof.M}: {k} differs at {bad[:5]}: {g[k][bad[:5]]} {o[k][bad[:5]]}"
        assert g["counts"][1] == n_ovf
    return n_ovf


@pytest.mark.parametrize("M,ins,ii", model.SWEEP)
def test_insert_before_the_first_match(M, ins, ii):
    for mi in model.MI:
        prof, c = model.peaked(M, 0.7, ins, mi, ii)
        assert _compare(prof, model.insert_first(prof, c), f"M->I {mi:.1e}") > 0


def test_insert_at_a_lone_node():
    for prof, seqs in model.lone_node():
        _compare(prof, seqs, "lone node")


@pytest.mark.parametrize("M", [3, 64, 128, 256, 384, 385, 768])
def test_insert_short_of_the_limit(M):
    prof, seqs = model.insert_to_the_limit(M)
    assert 0 < _compare(prof, seqs, "insert to the limit") < len(seqs)
