"""MSV kernel instances at their edges, bit-exact against the oracle: profile
sizes on both sides of every change of layout or vector count, target lengths
on both sides of a residue dword, a residue chunk and a phase, targets that need
the exact pass (homologs, targets without a positive cell), and groups with and
without absent profiles."""
import numpy as np
import pytest

import oracle
import paper_2111_06340_amd as hg
from synth import gen

pytestmark = pytest.mark.gpu

F = (1e-3, 1e-6, 1.0)
LENGTHS = [1, 2, 3, 4, 5, 7, 8, 9, 60, 63, 64, 65, 66, 127, 128, 129, 191, 193, 252, 255, 256, 257, 258, 259, 260,
           383, 384, 385, 388, 511, 512, 513, 515, 639, 641, 767, 769, 900, 1023, 1025, 1030, 1300]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    hg.lib()


def _db(prof, seed):
    """Background and, for every length, a homolog cut to it; and targets of the profile's least likely residue."""
    rng = np.random.default_rng(seed)
    homs = gen.sample_homologs(rng, prof, len(LENGTHS))
    rare = int(np.argmax((prof.bg / prof.match).min(axis=0)))
    seqs = []
    for L, h in zip(LENGTHS, homs):
        seqs.append(gen.background_residues(rng, L))
        s = gen.background_residues(rng, L)
        o = int(rng.integers(0, max(L - h.size, 0) + 1))
        s[o:o + h.size] = h[:L]
        seqs.append(s)
        seqs.append(np.full(L, rare, np.uint8))
    off = np.zeros(len(seqs) + 1, np.int64)
    off[1:] = np.cumsum([s.size for s in seqs])
    return np.concatenate(seqs), off


def _check(g, prof, res, off, what):
    o = oracle.search(oracle.OracleProfile(prof), res, off, (0.0, 0.0, 0.0), F, nthreads=8)
    for k in ("msv", "flags"):
        bad = np.nonzero(g[k] != o[k])[0]
        assert bad.size == 0, f"{what}: {k} differs at {bad[:5]} lengths {np.diff(off)[bad[:5]]}"
    return int(np.sum((o["flags"] & oracle.F_MSV_OVF) != 0))


@pytest.mark.parametrize("M", [1, 2, 5, 126, 127, 128, 255, 383, 511, 512, 639, 640, 767, 768, 895, 896, 1022, 1023, 1024,
                               1025, 1152, 1153, 1281, 1409, 1537, 1793, 2049, 2305, 2561, 2817, 3072])
def test_instance_edges(M):
    import torch
    prof = gen.make_profile(M, 7000 + M)
    res, off = _db(prof, M)
    P, D = hg.Profile(prof, 0.0, 0.0, 0.0), hg.Database(res, off)
    print(f"[msv] M={M} n={D.n}", flush=True)
    out = hg.search(P, D, F)
    torch.cuda.synchronize()
    ovf = _check({k: v.cpu().numpy() for k, v in out.items()}, prof, res, off, f"M={M}")
    assert ovf > 0 or M < 77


@pytest.mark.parametrize("M,count", [(60, 2), (100, 3), (127, 4), (128, 2), (200, 3), (255, 4), (300, 2), (383, 3),
                                     (384, 2), (511, 3), (600, 2)])
def test_groups(M, count):
    import torch
    profs = [gen.make_profile(M - 3 * i, 7100 + M + i) for i in range(count)]
    res, off = _db(profs[0], M)
    Ps = [hg.Profile(p, 0.0, 0.0, 0.0) for p in profs]
    D = hg.Database(res, off)
    handles = [D] + [D.share() for _ in profs[1:]]
    print(f"[msv] group of {count}, M={M}, n={D.n}", flush=True)
    outs = hg.search_group(Ps, handles, F)
    torch.cuda.synchronize()
    for p, o in zip(profs, outs):
        _check({k: v.cpu().numpy() for k, v in o.items()}, p, res, off, f"group of {count}, M={p.M}")
