"""The re-based int16 Viterbi against the oracle, on the CPU: a cell-by-cell
model of the kernel's stored values (true values less an offset, clipped at
the int16 floor), over profiles and targets for which the floor matters.

The model takes its tables from the library's own quantisation.  Where a score
passes the int16 range the model must give the exact int32 score, and it must
say so for exactly the targets of which the oracle says it."""
import numpy as np
import pytest

import oracle
import paper_2111_06340_amd as hg
from synth import gen

NEG, TOP, REBASE_TO = -32768, 32767, 8000


def rebase_room(t, M):
    """W: how far above the stored floor xBe has to stay."""
    msc_min = min(0, int(t["msc16"].min()))
    mi_min = min([0] + [int(v) for v in t["t16"][:, 1]])
    isc_max = max([0] + [int(v) for v in t["isc16"].reshape(-1)])
    return -msc_min - mi_min + isc_max


def vit16_model(t, M, mv, x, W, carry_on=True):
    """(score, overflow, left to the rescore) of the re-based kernel."""
    sat = lambda v: np.clip(v, NEG, TOP)  # noqa: E731
    z = np.full((1,), NEG)
    into = lambda k: np.concatenate([z, t["t16"][:, k].astype(int)]) if M > 1 else z  # noqa: E731
    out = lambda k: np.concatenate([t["t16"][:, k].astype(int), z]) if M > 1 else z  # noqa: E731
    mm, im, dm, md, dd, mi, ii = into(0), into(3), into(5), into(2), into(6), out(1), out(4)
    msc = t["msc16"].astype(int)
    isc = np.concatenate([t["isc16"].astype(int).reshape(-1, 20), np.full((1, 20), NEG)])
    chain = np.concatenate([[0], np.cumsum(dd[1:])])   # sum of D->D into the cells up to k
    s_max = max(0, int(msc.max()), int(isc.max()))
    entry, ej = t["entry16"], t["ej16"]
    dm_max = int(dm[1:].max()) if M > 1 else NEG
    reb = s_max <= 12000 and mv + entry >= NEG + W
    RL = TOP - 1 - s_max if reb else TOP - 1
    Mv, Iv, Dv = (np.full(M, NEG) for _ in range(3))
    accM, accI, xJt, off, top, redo = NEG, NEG, NEG, 0, 0, False
    xbt = mv + entry

    def derived():
        xbe = int(sat(xbt - off))
        return xbe, min(xbe - dm_max, TOP)
    xbe, tau = derived()
    for a in x:
        up = lambda v: np.concatenate([[0], v[:-1]])  # noqa: E731
        m = np.maximum(np.maximum(xbe, sat(up(Mv) + mm)), np.maximum(sat(up(Iv) + im), sat(up(Dv) + dm)))
        Iv = sat(np.maximum(sat(Mv + mi), sat(Iv + ii)) + isc[:, a])
        Mv = sat(m + msc[:, a])
        # max over j <= k of md_j + (sum of D->D from j to k), and the floor
        md_ = np.maximum(sat(up(Mv) + md), tau)
        Dv = np.maximum(np.maximum.accumulate(md_ - chain) + chain, tau)
        accM, accI = max(accM, int(Mv.max())), max(accI, int(Iv.max()))
        if not reb and (accM >= TOP or accI >= TOP):
            redo = True
            break
        if reb and max(accM, accI) > RL:
            hi = max(accM, accI)
            sh = hi - REBASE_TO
            if xbt - off - sh < NEG + W:
                if carry_on and off == 0:   # nothing has passed the range yet: go on without re-basing
                    reb, RL = False, TOP - 1
                else:
                    redo = True
                    break
            else:
                top = max(top, hi + off)
                off += sh
                Mv, Iv, Dv = sat(Mv - sh), sat(Iv - sh), sat(Dv - sh)
                accM, accI = int(sat(accM - sh)), int(sat(accI - sh))
        xJt = max(xJt, accM + off + ej)
        xbt = max(mv, xJt + mv) + entry
        xbe, tau = derived()
    if redo:
        return 0, True, True
    m = accM + off
    if off > 0:
        top = max(top, m, accI + off)
    ovf = top >= TOP
    return (m + ej + mv if ovf else int(sat(sat(m + ej) + mv))), ovf, False


def agrees(prof, seqs, **mutant):
    """Targets on which the model and the oracle differ, and how the targets were scored."""
    t = hg.hmm_debug_tables(prof)
    op = oracle.OracleProfile(prof)
    W = mutant.pop("W", rebase_room)(t, prof.M)
    bad, n = [], dict(rebased=0, overflow=0, redo=0)
    for j, x in enumerate(seqs):
        mv = oracle.length_params(len(x))["move16"]
        raw, ovf, redo = vit16_model(t, prof.M, mv, x, W, **mutant)
        want, o = oracle.vit16(op, x)
        if o:
            want = oracle.vit32(op, x)
        n["overflow"] += bool(o)
        n["redo"] += redo
        n["rebased"] += ovf and not redo
        if ovf != bool(o) or (not redo and raw != want):
            bad.append(j)
    return bad, n


# ---------------------------------------------------------------- profiles and targets

def peaked(M, match, insert, mi, ii):
    """One likely residue (never 0) per node, inserts that prefer residue 0; and the consensus."""
    rng = np.random.default_rng(4200 + M)
    c = rng.integers(1, 20, size=M)
    m = np.full((M, 20), (1 - match) / 19)
    m[np.arange(M), c] = match
    i = np.full((M - 1, 20), (1 - insert) / 19)
    i[:, 0] = insert
    trans = np.tile([0.95 - mi, mi, 0.05, 1 - ii, ii, 0.5, 0.5], (M - 1, 1))
    return gen.Profile(M, gen.BACKGROUND.copy(), m, i, trans), c.astype(np.uint8)


def insert_first(prof, c):
    """Targets that open with a run of residue 0 and go on with the consensus, some past the int16 range."""
    need = int(np.ceil(60 / len(c)))
    return [np.concatenate([np.zeros(n, np.uint8), np.tile(c, r)]) for n in (1, 2, 5, 30, 60) for r in (1, need, 4 * need)]


def lone_node():
    """A node whose match is all but impossible for a residue that its insert is almost sure of."""
    out = []
    for e in (22, 24, 25):
        for M in (3, 20):
            prof, c = peaked(M, 0.9, 0.5, 0.05, 0.5)
            k, r = M // 2, 7
            prof.match[k - 1] = (1 - 2.0 ** -e) / 19
            prof.match[k - 1, r] = 2.0 ** -e
            prof.insert[k - 1] = (1 - 0.9995) / 19
            prof.insert[k - 1, r] = 0.9995
            prof.trans[k - 1] = [0.95, 2.0 ** -30, 0.05 - 2.0 ** -30, 0.01, 0.99, 0.5, 0.5]
            tail = [np.zeros(0, np.uint8), c[-1:], np.tile(c, 30 // M + 1)]
            out.append((prof, [np.concatenate([np.full(n, r, np.uint8), s]) for n in (2, 20, 50, 200) for s in tail]))
    return out


def insert_to_the_limit(M):
    """An insert that is all but never left: its value alone nears the limit while xBe stays low."""
    prof, c = peaked(M, 0.9, 0.8, 0.05, 0.5)
    prof.trans[:, 3:5] = [1e-15, 1.0 - 1e-15]
    return prof, [np.concatenate([c[: k], np.zeros(n, np.uint8)]) for k in (1, 2) for n in range(8, 61)]


MI = [1e-3, 1e-5, 10 ** -8.7, 1e-12, 1e-14, 1e-16, 1e-17, 1e-19]
SWEEP = [(M, ins, ii) for M in (3, 20, 128) for ins, ii in ((0.3, 0.9), (0.8, 0.95))]


@pytest.mark.parametrize("M,ins,ii", SWEEP)
def test_insert_before_the_first_match(M, ins, ii):
    for mi in MI:
        prof, c = peaked(M, 0.7, ins, mi, ii)
        bad, n = agrees(prof, insert_first(prof, c))
        assert not bad and n["overflow"] > 0, (mi, bad, n)


def test_insert_at_a_lone_node():
    for prof, seqs in lone_node():
        bad, n = agrees(prof, seqs)
        assert not bad, (prof.M, bad, n)


@pytest.mark.parametrize("M", [3, 64, 128, 256])
def test_insert_short_of_the_limit(M):
    prof, seqs = insert_to_the_limit(M)
    bad, n = agrees(prof, seqs)
    assert not bad, (bad, n)
    assert 0 < n["overflow"] < len(seqs)


@pytest.mark.parametrize("seed", range(4))
def test_random_profiles(seed):
    rng = np.random.default_rng(seed)
    hits = 0
    for _ in range(40):
        M = int(rng.integers(1, 13))
        prof, c = peaked(M, 1 - 10 ** rng.uniform(-3, -0.3), rng.uniform(0.05, 0.99), 10 ** rng.uniform(-14, -1.5),
                         rng.uniform(0.05, 0.999))
        rnd = lambda *s: np.maximum(rng.dirichlet(np.full(20, 10 ** rng.uniform(-1.5, 0)), size=s), 1e-9)  # noqa: E731
        if rng.random() < 0.5:
            prof.match[:] = rnd(M)
            prof.match /= prof.match.sum(1, keepdims=True)
            if M > 1:
                prof.insert[:] = rnd(M - 1)
                prof.insert /= prof.insert.sum(1, keepdims=True)
        seqs = insert_first(prof, c) + [rng.integers(0, 20, size=int(rng.integers(1, 200))).astype(np.uint8)
                                        for _ in range(4)]
        bad, n = agrees(prof, seqs)
        assert not bad, (M, bad, n)
        hits += n["rebased"]
    assert hits > 20


def test_the_sweeps_reach_the_rules_edges():
    """Without the insert score in W, or with a value that only nears the limit
    taken for an overflow, the model and the oracle disagree on these inputs."""
    def narrow(t, M):
        return rebase_room(t, M) - max([0] + [int(v) for v in t["isc16"].reshape(-1)])
    prof, c = peaked(3, 0.7, 0.8, 1e-16, 0.95)
    assert any(agrees(p, s, W=narrow)[0] for p, s in lone_node() + [(prof, insert_first(prof, c))])
    prof, seqs = insert_to_the_limit(128)
    assert agrees(prof, seqs, carry_on=False)[0]
