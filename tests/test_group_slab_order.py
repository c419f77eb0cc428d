"""The order of the workgroups of a GroupNorm in slices: the index map of the kernel, compiled for the host, and a device of eight dies on
which two launches whose slices wait for one another share the places.  Nothing runs on a GPU."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2307_04995_amd import build

DIES = 8


class _Place(ctypes.Structure):
    _fields_ = [(n, ctypes.c_uint32) for n in ("at", "sample", "slab", "slice")]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("order")
    src, out = d / "order.cpp", d / "order.so"
    src.write_text('#include "pf_common.h"\n'
                   'namespace pf { struct Div { uint32_t d; }; constexpr uint32_t quotient(uint32_t n, Div f) { return n / f.d; } }\n'
                   'extern "C" pf::GroupSlabPlace place(uint32_t b, uint32_t per_die, uint32_t runs, uint32_t run_slabs, uint32_t slices) {\n'
                   '    return pf::group_slab_place<true>(b, per_die, pf::Div{run_slabs * slices}, pf::Div{runs}, pf::Div{run_slabs});\n}\n'
                   'extern "C" int shares(uint32_t run_blocks, uint32_t per_die, uint32_t places) { return pf::group_slab_shares(run_blocks, per_die, places); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + os.path.abspath(build.CSRC), str(src), "-o", str(out)], check=True)
    lib = ctypes.CDLL(str(out))
    lib.place.restype = _Place
    lib.place.argtypes = [ctypes.c_uint32] * 5
    lib.shares.argtypes = [ctypes.c_uint32] * 3
    return lib


def _launch(host, samples, slabs, slices, run):
    """Per die, what its workgroups belong to, in the order they are dispatched: (sample, slab), or None for one with nothing to do."""
    blocks = samples * slabs * slices
    per_die = -(-blocks // DIES)
    dies, seen = [[] for _ in range(DIES)], set()
    for b in range(per_die * DIES):
        p = host.place(b, per_die, slabs // run, run, slices)
        if p.at < blocks:
            assert p.sample < samples and p.slab < slabs and p.slice < slices
            seen.add((p.sample, p.slab, p.slice))
        dies[b % DIES].append((p.sample, p.slab) if p.at < blocks else None)
    assert len(seen) == blocks
    return dies


def _ends(launches, slices, places, rng):
    """Dispatch in order on every die, launches and dies taking turns at random, until nothing moves; a slab whose slices are all
    dispatched ends and frees its places.  True when everything was dispatched."""
    todo = [[list(reversed(die)) for die in dies] for dies in launches]
    used, waiting = [0] * DIES, {}
    weight = {(k, d): rng.random() ** 3 + 1e-3 for k in range(len(launches)) for d in range(DIES)}  # (dies and launches progress unevenly)
    while True:
        ready = [(k, d) for k in range(len(launches)) for d in range(DIES) if todo[k][d] and used[d] < places]
        if not ready:
            return not any(todo[k][d] for k in range(len(launches)) for d in range(DIES))
        k, d = rng.choices(ready, [weight[r] for r in ready])[0]
        unit = todo[k][d].pop()
        if unit is None:
            continue
        used[d] += 1
        held = waiting.setdefault((k, unit), [])
        held.append(d)
        if len(held) == slices[k]:
            for x in waiting.pop((k, unit)):
                used[x] -= 1


def _run(host, samples, slabs, slices, places):
    """The most slabs to a run with which two launches share the device; 0 where not even one does."""
    per_die = -(-samples * slabs * slices // DIES)
    return max([r for r in range(1, slabs + 1) if slabs % r == 0 and host.shares(r * slices, per_die, places)], default=0)


# (samples, slabs to a sample, slices): as many workgroups as units, nearly as many, few; slabs that end inside a die's range, one slab
SHAPES = [(7, 4, 9), (21, 2, 6), (32, 1, 8), (1, 16, 16), (2, 8, 16), (13, 2, 9), (1, 28, 9), (17, 1, 15), (1, 1, 16), (5, 3, 2), (10, 8, 3), (1, 8, 31)]


@pytest.mark.parametrize("places", [32, 64])
def test_two_launches_on_one_device_end(host, places):
    rng = random.Random(5)
    runs = {s: _run(host, *s, places) for s in SHAPES}
    assert sum(r == 0 for r in runs.values()) == (places == 32)  # (31 slices)
    assert places == 64 or (runs[7, 4, 9], runs[21, 2, 6], runs[10, 8, 3]) == (1, 2, 4)
    for a in SHAPES:
        for b in SHAPES:
            if runs[a] and runs[b]:
                launches = [_launch(host, *a, runs[a]), _launch(host, *b, runs[b])]
                for _ in range(6):
                    assert _ends(launches, (a[2], b[2]), places, rng), f"{a} beside {b} on {places} places to a die"


def test_runs_follow_each_other(host):
    for samples, slabs, slices in SHAPES:
        for run in (r for r in range(1, slabs + 1) if slabs % r == 0):
            for die in _launch(host, samples, slabs, slices, run):
                runs = [(u[0], u[1] // run) for u in die if u is not None]
                starts = [r for k, r in enumerate(runs) if k == 0 or runs[k - 1] != r]
                assert len(starts) == len(set(starts))


def test_slices_far_apart_get_stuck(host):
    # (a sample to a run: 36 workgroups, more than a die has places)
    rng = random.Random(5)
    assert not all(_ends([_launch(host, 7, 4, 9, 4)] * 2, (9, 9), 32, rng) for _ in range(20))


def test_where_two_launches_do_not_share(host):
    assert host.shares(16, 32, 32) and not host.shares(17, 32, 32)  # 2 * 16 workgroups that wait fill a die of 32 units
    assert host.shares(64, 16, 32) and host.shares(64, 32, 64)      # both launches fit whole
