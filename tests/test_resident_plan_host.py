"""Plan of the resident CG (csrc/resident_plan.cpp) on the CPU: shares cover every
problem's octs once, every face between two shares has one unit on each side and the two
name each other, the place of each of a face's four cells is the same seen from both
sides, and no order of execution of the blocks' lists can make two blocks wait for each
other.  Plain build and with AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

from synth.hierarchy import random_balanced_hierarchy

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_1112_amd", "csrc")
OFF = [(-1, 0, 0), (1, 0, 0), (0, -1, 0), (0, 1, 0), (0, 0, -1), (0, 0, 1)]
SANITIZE = ["-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module", params=["plain", "asan_ubsan"])
def harness(request, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / f"plan_dump_{request.param}")
    extra = SANITIZE if request.param == "asan_ubsan" else []
    subprocess.run(["g++", "-O1", "-std=c++17"] + extra + ["-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "resident_plan_dump.cpp"),
                    os.path.join(CSRC, "resident_plan.cpp"), "-o", exe], check=True)
    return exe


def _morton(o):
    k = np.zeros(len(o), dtype=np.int64)
    for b in range(10):
        for a in range(3):
            k |= ((o[:, a].astype(np.int64) >> b) & 1) << (3 * b + a)
    return k


def _table(octs):
    """Neighbour octs of Morton-sorted octs, -1 where absent."""
    octs = np.asarray(octs, dtype=np.int64)
    octs = octs[np.argsort(_morton(octs))]
    at = {tuple(o): i for i, o in enumerate(octs.tolist())}
    return np.array([[at.get((o[0] + d[0], o[1] + d[1], o[2] + d[2]), -1) for d in OFF] for o in octs.tolist()],
                    dtype=np.int32)


def _box(m):
    return np.array([[i, j, k] for i in range(m) for j in range(m) for k in range(m)])


def _plan(harness, tmp_path, tables, n_blocks, target):
    """Problems one after another, with a gap of unused rows between them."""
    rows, probs, at = [], [], 0
    for t in tables:
        probs.append((at, len(t)))
        rows.append(np.where(t >= 0, t + at, -1))
        rows.append(np.full((3, 6), -1))
        at += len(t) + 3
    nbr = np.concatenate(rows).astype(np.int32)
    path = tmp_path / "p.bin"
    with open(path, "wb") as f:
        f.write(struct.pack("<iii", len(probs), n_blocks, target))
        for p in probs:
            f.write(struct.pack("<qq", *p))
        f.write(struct.pack("<q", len(nbr)))
        f.write(nbr.tobytes())
    run = subprocess.run([harness, str(path)], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-3000:]
    arr = [np.array(x.split(), dtype=np.int64) for x in run.stdout.splitlines()]
    _check_peers(arr[0].reshape(-1, 7), arr[2], arr[-1])
    return probs, nbr, arr[0].reshape(-1, 7), arr[1].reshape(-1, 6), arr[2], arr[3], arr[4], arr[5], arr[6]


def _check_peers(parts, partner, peers):
    """The second numbering of the units: every unit its own number, a share's contiguous
    and from a multiple of two on, so that no line of two units belongs to two shares."""
    n_near, peers = peers[-1], peers[:-1].reshape(-1, 2)
    share = np.concatenate([np.full(p[3], k) for k, p in enumerate(parts)] + [np.zeros(0, dtype=int)])
    near = np.full(len(partner), -1)
    near[partner] = peers[:, 0]
    assert len(np.unique(near)) == len(near) and (near >= 0).all() and (near < n_near).all()
    for k, (s0, ns, u0, nu, q, p0, g) in enumerate(parts):
        if nu:
            base = (u0 + k + 1) & ~1
            assert np.array_equal(near[u0:u0 + nu], base + np.arange(nu))
    owner = {}
    for n, k in zip(near, share):
        assert owner.setdefault(n // 2, k) == k
    for u, v in enumerate(partner):
        assert peers[u, 1] == share[v] - parts[share[v], 5]


CASES = {
    "one_oct": lambda: ([_box(1)], 256, 64),
    "one_share": lambda: ([_box(4)], 256, 2048),
    "many_shares": lambda: ([_box(8)], 24, 64),
    "every_oct_a_share": lambda: ([_box(3)], 256, 8),
    "irregular": lambda: ([random_balanced_hierarchy(3, 3, 5, 0.5).octs[5]], 16, 128),
    "batch": lambda: ([_box(m) for m in (6, 5, 4, 4, 3, 2, 1, 1)], 8, 256),
    "batch_whole_chip": lambda: ([_box(m) for m in (7, 7, 6, 2, 1)], 5, 100),
}


@pytest.mark.parametrize("case", list(CASES))
def test_plan(harness, tmp_path, case):
    octs, n_blocks, target = CASES[case]()
    probs, nbr, parts, unit_of, partner, task0, task, most, places = _plan(
        harness, tmp_path, [_table(o) for o in octs], n_blocks, target)
    part_of = np.full(len(nbr), -1)
    for k, (s0, ns, u0, nu, q, p0, g) in enumerate(parts):
        assert s0 % 8 == 0 and ns % 8 == 0 and ns > 0
        assert np.all(part_of[s0 // 8:(s0 + ns) // 8] == -1)
        part_of[s0 // 8:(s0 + ns) // 8] = k
        assert p0 <= k < p0 + g and g <= n_blocks
        assert np.all(parts[p0:p0 + g, 4] == q)
    for o0, m in probs:
        assert np.all(part_of[o0:o0 + m] >= 0)
    assert int((part_of >= 0).sum()) == sum(m for _, m in probs)
    assert most[0] == parts[:, 1].max() and most[1] == parts[:, 3].max()

    seen = set()
    for o in range(len(nbr)):
        for d in range(6):
            u, nb = unit_of[o, d], nbr[o, d]
            cross = part_of[o] >= 0 and nb >= 0 and part_of[nb] != part_of[o]
            assert (u >= 0) == cross
            if not cross:
                continue
            seen.add(int(u))
            k = part_of[o]
            assert parts[k, 2] <= u < parts[k, 2] + parts[k, 3]
            assert partner[u] == unit_of[nb, d ^ 1] and partner[partner[u]] == u
    assert seen == set(range(len(partner)))

    # every share once; a problem's shares on different blocks; lists in the problems'
    # order, so that the first unfinished problem always has all its blocks
    assert sorted(task) == list(range(len(parts))) and len(task0) == n_blocks + 1
    for b in range(n_blocks):
        mine = parts[task[task0[b]:task0[b + 1]], 4]
        assert np.all(np.diff(mine) > 0)

    # what a thread reads for the out-of-oct neighbours of its pairs: the slots of its own
    # share directly; halo cells through the export list of the neighbour share, whose
    # entry 4 u + c is filled with the cell whose own place is that entry
    places = (places & 0xffffffff).reshape(-1, 2)
    filled = {}

    def entries(o, k):
        p0, p1 = (int(v) for v in places[4 * o + k])
        s = 8 * o + 2 * k
        out = [(s, 0, k, p0 & 0xffff, 1), (s + 1, 1, k, p0 >> 16, 1)]
        return out + [(s, 2 + (k & 1), k, p1 & 0xffff, 2), (s, 4 + (k >> 1), k, p1 >> 16, 2)]

    rows = [o for o in range(len(nbr)) if part_of[o] >= 0]
    for o in rows:
        for k in range(4):
            for s, d, _, place, w in entries(o, k):
                if place & 0x8000:
                    for j in range(w):
                        key = (int(part_of[o]), (place & 0x7fff) + j)
                        assert key not in filled
                        filled[key] = s + j
    assert len(filled) == 4 * len(partner)
    for o in rows:
        me = parts[part_of[o]]
        for k in range(4):
            for s, d, _, place, w in entries(o, k):
                nb = nbr[o, d]
                for j in range(w):
                    pos = (s + j) & 7
                    want = 8 * nb + (pos ^ (1 << (d >> 1))) if nb >= 0 else s + j
                    if place & 0x8000:
                        cell = (place & 0x7fff) + j
                        other = partner[me[2] + cell // 4]
                        owner = part_of[nb]
                        got = filled[(int(owner), int(4 * (other - parts[owner, 2]) + cell % 4))]
                    else:
                        got = me[0] + place + j
                    assert got == want, (case, o, k, d)


def _composite_tables(h):
    """Neighbour octs, coarser leaves and refining octs of all levels one after another,
    each level padded to whole tiles of 256 slots."""
    octs, base = {}, {}
    n = 0
    for l in h.levels:
        o = np.asarray(h.octs[l], dtype=np.int64)
        octs[l] = o[np.argsort(_morton(o))]
        base[l] = n
        n += (len(o) + 31) // 32 * 32
    at = {l: {tuple(o): base[l] + i for i, o in enumerate(octs[l].tolist())} for l in h.levels}
    nbr, cnb, child = np.full((n, 6), -1), np.full((n, 6), -1), np.full(8 * n, -2)
    for l in h.levels:
        for (x, y, z), o in at[l].items():
            for d, (i, j, k) in enumerate(OFF):
                cell = (x + i, y + j, z + k)  # an oct of level l is a cell of level l - 1
                nbr[o, d] = at[l].get(cell, -1)
                up = at[l - 1].get(tuple(c >> 1 for c in cell), -1) if l > h.base_level else -1
                if nbr[o, d] < 0 and up >= 0 and min(cell) >= 0:
                    cnb[o, d] = 8 * up + (cell[0] & 1) + 2 * (cell[1] & 1) + 4 * (cell[2] & 1)
            for pos in range(8):
                cell = (2 * x + (pos & 1), 2 * y + ((pos >> 1) & 1), 2 * z + (pos >> 2))
                child[8 * o + pos] = at[l + 1].get(cell, -1) if l < h.max_level else -1
    return nbr.astype(np.int32), cnb.astype(np.int32), child.astype(np.int32)


@pytest.mark.parametrize("n_blocks,target", [(2, 4096), (7, 512), (64, 64)])
def test_couplings_between_levels(harness, tmp_path, n_blocks, target):
    nbr, cnb, child = _composite_tables(random_balanced_hierarchy(7, 2, 5, 0.5))
    assert (cnb >= 0).any()
    path = tmp_path / "c.bin"
    with open(path, "wb") as f:
        f.write(struct.pack("<iiiqqq", 1, n_blocks, target, 0, len(nbr), len(nbr)))
        f.write(nbr.tobytes() + cnb.tobytes() + child.tobytes())
    run = subprocess.run([harness, str(path)], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-3000:]
    arr = [np.array(x.split(), dtype=np.int64) for x in run.stdout.splitlines()]
    parts, unit_of, partner, places = arr[0].reshape(-1, 7), arr[1].reshape(-1, 6), arr[2], arr[6] & 0xffffffff
    n_coarse, coarse, couplings = arr[7], arr[8].reshape(-1, 2), arr[9] & 0xffffffff
    _check_peers(parts, partner, arr[-1])
    part_of = np.concatenate([np.full(p[1], k) for k, p in enumerate(parts)])
    assert np.array_equal(partner[partner], np.arange(len(partner)))

    # the slots whose values a unit sends, in its order: a finer face's four cells by the
    # places that name the unit, a coarse unit's leaf four times
    sends = np.full((len(partner), 4), -1)
    reads = []  # (slot, direction, unit, cell)
    for s in range(8 * len(nbr)):
        k, pos, o = s >> 1, s & 7, s >> 3
        p0, p1 = int(places[2 * k]), int(places[2 * k + 1])
        place = [p0 >> 16 if pos & 1 else p0 & 0xffff, (p1 & 0xffff) + (pos & 1), (p1 >> 16) + (pos & 1)]
        for a in range(3):
            d = 2 * a + ((pos >> a) & 1)
            assert bool(place[a] & 0x8000) == (unit_of[o, d] >= 0)
            if place[a] & 0x8000:
                u, c = parts[part_of[s], 2] + (place[a] & 0x7fff) // 4, place[a] & 3
                assert u == unit_of[o, d] and sends[u, c] == -1
                sends[u, c] = s
                reads.append((s, d, u, c))
    want = set()
    for k, (p, nc) in enumerate(zip(parts, n_coarse)):
        first = p[2] + p[3] - nc
        for s in range(p[0], p[0] + p[1], 2):
            w = int(couplings[s >> 1])
            u = first + (w & 0xffff)
            for e, m in ((s, (w >> 16) & 0xff), (s + 1, w >> 24)):
                for v in range(u, u + m):
                    assert coarse[v, 0] == e - p[0]
                    sends[v] = e
                    want.add(v)
                u += m
        assert want >= set(range(first, p[2] + p[3]))
    assert len(want) == n_coarse.sum() and (sends >= 0).all()
    for s, d, u, c in reads:
        a = d >> 1
        other = 8 * nbr[s >> 3, d] + ((s & 7) ^ (1 << a)) if nbr[s >> 3, d] >= 0 else cnb[s >> 3, d]
        assert sends[partner[u], c] == other
    # a coarse unit receives the cells on the near face of the oct that refines the leaf's
    # neighbour, and every such face of every leaf has one
    faces = set()
    for v in want:
        f, d = coarse[v, 1] >> 3, coarse[v, 1] & 7
        a, leaf = d >> 1, sends[v, 0]
        t = [b for b in range(3) if b != a]
        cells = [8 * f + ((d & 1) << a) + ((c & 1) << t[0]) + ((c >> 1) << t[1]) for c in range(4)]
        assert list(sends[partner[v]]) == cells and cnb[f, d] == leaf
        faces.add((f, d))
    assert len(faces) == len(want) == int((cnb >= 0).sum())
