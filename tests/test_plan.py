"""Host tests of the launch plans (no GPU): a probe linked against libqgbe.so
prints the plans that the library makes for given descriptors and LDS budgets.
"""
import json
import os
import subprocess

import numpy as np
import pytest

from paper_1912_04457_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"
LDS = 160 * 1024
# dynamic LDS beside the kernels' own: plain and learned [long, short items],
# roots, replay, the queues [ring, tight][long, short items]
BUDGETS = {0: (LDS, LDS - 6168, LDS, LDS - 30840, LDS - 61464, LDS, 0, LDS - 110616, 0, LDS - 49176),
           1: (LDS - 24, LDS - 6168, LDS - 6216, LDS - 12360, LDS - 61464, LDS, LDS - 80280, LDS - 86040, LDS - 31128,
               LDS - 36888)}


@pytest.fixture(scope="session")
def probe(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("no clang with the HIP headers here")
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.PKG, "csrc"),
                    os.path.join(HERE, "plan_probe.cpp"), build.LIB, "-Wl,-rpath," + build.PKG,
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)

    def run(cases):
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases) + "\n"
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [json.loads(line) for line in out.splitlines()]
    return run


def _case(mask, n_x, n_p, precision, symmetric, long_form=0, n_samples=64, capacity=1 << 23):
    return (mask, *n_x, *n_p, precision, symmetric, long_form, *BUDGETS[precision], n_samples, capacity)


GRIDS = [(2, 2, 2), (5, 6, 7), (16, 16, 16), (20, 20, 20), (22, 22, 22), (24, 24, 23), (30, 30, 30), (64, 64, 64),
         (128, 100, 90)]


@pytest.mark.parametrize("mask", [0x40, 0x49, 0x7F])
def test_device_lists_depend_on_the_masks_alone(probe, mask):
    """The channel and match lists that calls without a context share on a GPU,
    and that a captured call reads again at each replay, are the same for every
    grid and precision; the channels that take several launches are the last of
    their order; and every deposit of a channel has its match."""
    cases = [_case(mask, (1, 1, 1), n_p, precision, sym) for n_p in GRIDS for precision in (0, 1) for sym in (0, 1)]
    plans = probe(cases)
    first = plans[0]
    nch = first["nch"]
    sp = np.array(first["species"]).reshape(nch, 4)
    order = first["lists"][:nch]
    assert sorted(order) == list(range(nch))
    assert [first["nslot"][c] for c in order] == sorted(first["nslot"])
    per = (len(first["lists"]) - 70) // 7
    for y in range(7):
        want = [4 * i + p for i, c in enumerate(order) for p in (1, 2, 3) if sp[c, p] == y]
        assert first["lists"][70 + y * per: 70 + y * per + len(want)] == want
    for plan in plans:
        assert plan["lists"] == first["lists"]
        for start, count in zip(plan["replay_start"], plan["replay_count"]):
            assert count == 0 or start + count == nch
    assert any(p["replay_count"][0] for p in plans) and any(not p["replay_count"][0] for p in plans)


def _boundary_grids():
    """Grids around every node count at which one, two or three accumulators or
    tiles, alone or together, stop fitting in a budget."""
    rng = np.random.default_rng(3)
    want = sorted({b // (8 * a + 4 * t) for b in BUDGETS[1] for a in range(4) for t in range(4) if a + t})
    grids = set()
    for n in want:
        for _ in range(8):
            x = int(np.clip(round(n ** (1 / 3) * np.exp(rng.normal(0, 0.2))), 2, n))
            y = int(np.clip(round((n / x) ** 0.5 * np.exp(rng.normal(0, 0.2))), 2, n))
            z = max(2, n // (x * y) + int(rng.integers(-1, 3)))
            grids.add((x, y, z))
    return sorted(grids)


@pytest.mark.parametrize("symmetric", [0, 1])
@pytest.mark.parametrize("mask", [0x40, 0x49, 0x7F])
def test_long_form_where_the_short_one_lacks_lds(probe, mask, symmetric):
    """FP32, uniform and learned sampler: a group takes several launches only
    where the accumulators do not fit beside the long form's own LDS either, its
    plan fits in the LDS of the form it runs in, and the plan that the call
    without allocation falls back to needs node quads exactly where a tile does
    not fit beside the long form or its ring of samples fits."""
    grids = _boundary_grids()
    plans = probe([_case(mask, (1, 1, 1), n_p, 1, symmetric) for n_p in grids])
    long_plans = probe([_case(mask, (1, 1, 1), n_p, 1, symmetric, 1) for n_p in grids])
    b = BUDGETS[1]
    seen = {"long": 0, "several": 0}
    for n_p, plan, long_plan in zip(grids, plans, long_plans):
        nodes = int(np.prod(n_p))
        quads = False
        for g, h in zip(plan["groups"], long_plan["groups"]):
            k = g["nslot"]
            for l in (0, 1):
                p, (long_b, short_b) = g[str(l)], b[2 * l:2 * l + 2]
                assert p["several"] == (symmetric and 8 * nodes * k > long_b), (n_p, k, l)
                assert p["long"] == (symmetric and not p["several"] and 8 * nodes * k > short_b)
                if p["win"] == nodes:
                    used = nodes * (8 * p["acc"] + 4 * p["tiles"])
                else:
                    used = 8 * p["win"] * p["acc"]
                    assert p["acc"] == k and p["tiles"] == 0
                assert used <= (long_b if p["long"] else short_b)
                seen["long"] += p["long"]
                seen["several"] += p["several"]
            tiles = b[0] >= nodes * k * (12 if symmetric else 4)
            ring = symmetric and 8 * nodes * k <= b[6]
            quads = quads or not tiles or ring
            assert h["0"]["long"] and h["queue"] == [int(ring), 0]
        assert long_plan["quads"] == quads, n_p
    assert not symmetric or min(seen.values()) > 0


AGAIN, RECORD, GLOBAL = 0, 1, 2


def test_deposit_routes(probe):
    """The route of the channels that take several launches, over grids, samples
    and record buffers: never records without buffers, without room for a node's
    samples, or with the scale output; global atomics in FP64 only; and the side
    that was the faster one on the GPU where they were timed."""
    ns = (16, 20, 24, 30, 40, 48, 64, 80, 96, 128)
    cases = [(n, precision, mask, samples, cap) for n in ns for precision in (0, 1) for mask in (0x40, 0x7F)
             for samples in (1, 64, 2048, 100000) for cap in (0, 1 << 16, 1 << 23) if not (mask == 0x7F and n > 96)]
    plans = probe([_case(m, (1, 1, 1), (n, n, n), p, 1, 0, samples, cap) for n, p, m, samples, cap in cases])
    for (n, precision, mask, samples, cap), plan in zip(cases, plans):
        for l in range(3):
            plain, scale = plan["route"][2 * l:2 * l + 2]
            several = any(g[str(l)]["several"] for g in plan["groups"])
            assert several or plain == scale == AGAIN
            assert scale != RECORD and (plain != RECORD or samples <= cap)
            if precision == 1 and l < 2:
                assert GLOBAL not in (plain, scale)
    faster = {  # (cube, samples, precision, sampler, buffers): the faster route of one gluon cell
        (30, 128, 1, 0, 1): RECORD, (30, 2048, 1, 0, 1): RECORD, (48, 64, 0, 0, 1): RECORD, (64, 64, 0, 0, 1): RECORD,
        (80, 64, 0, 0, 1): RECORD, (96, 512, 0, 0, 1): GLOBAL, (128, 64, 0, 0, 1): GLOBAL, (80, 64, 0, 2, 1): RECORD,
        (96, 64, 0, 2, 1): GLOBAL, (128, 64, 0, 2, 1): GLOBAL, (80, 64, 0, 1, 1): RECORD, (96, 64, 0, 1, 1): GLOBAL,
        (48, 64, 0, 0, 0): AGAIN, (80, 64, 0, 0, 0): GLOBAL, (128, 64, 0, 0, 0): GLOBAL, (40, 64, 0, 2, 0): AGAIN,
        (64, 64, 0, 2, 0): GLOBAL, (64, 64, 0, 1, 0): GLOBAL, (128, 64, 1, 0, 1): RECORD, (96, 512, 1, 0, 1): RECORD,
        (96, 64, 1, 0, 0): AGAIN}
    plans = probe([_case(0x40, (1, 1, 1), (n, n, n), p, 1, 0, samples, buffers << 23)
                   for n, samples, p, _, buffers in faster])
    for (case, want), plan in zip(faster.items(), plans):
        assert plan["route"][2 * case[3]] == want, case


@pytest.mark.parametrize("mask,n_x,n_p,precision,samples,capacity",
                         [(0x40, (1, 1, 1), (30, 30, 30), 1, 128, 1 << 23), (0x7F, (1, 1, 1), (20, 20, 20), 1, 4096, 1 << 23),
                          (0x7F, (3, 5, 7), (28, 27, 29), 0, 77, 1 << 20), (0x40, (1, 1, 1), (128, 128, 64), 1, 9, 1 << 23),
                          (0x7F, (35, 13, 10), (30, 30, 30), 1, 8192, 1 << 23), (0x7F, (35, 13, 10), (30, 30, 30), 1, 1 << 23, 1 << 23)],
                         ids=["gluons", "seven", "cells", "large", "beyond_32_bits", "a_node_per_batch"])
def test_recording_batches(probe, mask, n_x, n_p, precision, samples, capacity):
    """The batches of recorded deposits: their workgroups lie in the (cell,
    channel, chunk) order that replay reads, in range also where all of them are
    more than 32 bits count, and their records fit in the buffers."""
    plan = probe([_case(mask, n_x, n_p, precision, 1, 0, samples, capacity)])[0]
    cells, nodes = int(np.prod(n_x)), int(np.prod(n_p))
    total = 0
    for l in range(3):
        if not plan["batches"][str(l)]:
            continue
        (chunk, n_chunks, n_group, cap, region, wgs, per), *batches = plan["batches"][str(l)]
        total = max(total, wgs)
        assert n_group == plan["replay_count"][l] and cap == capacity * (2 if l == 2 else 1)
        assert region == chunk * samples * (2 if l == 2 else 1) and (n_chunks - 1) * chunk < nodes <= n_chunks * chunk
        assert wgs == cells * n_group * n_chunks and 0 < per * region <= cap
        per_cell = n_group * n_chunks
        assert batches[0][0] == 0 and batches[-1][0] + batches[-1][1] == wgs
        for wg, n, cell_lo, base, n_cells, gi_lo, gi_hi in batches:
            assert 0 < n <= per and n == min(per, wgs - wg)
            assert cell_lo * per_cell + base == wg and 0 <= base < per_cell
            assert (cell_lo + n_cells - 1) == (wg + n - 1) // per_cell < cells
            assert base + n < 1 << 31
            first, last = wg % per_cell // n_chunks, (wg + n - 1) % per_cell // n_chunks
            assert (gi_lo, gi_hi) == ((first, last) if n_cells == 1 else (0, n_group - 1))
    assert total > 0
    if cells == 4550:
        assert total > 1 << 31


@pytest.mark.parametrize("mask,n_x,n_p", [(0x40, (1, 1, 1), (2, 2, 2)), (0x40, (16, 16, 1), (20, 20, 20)),
                                          (0x7F, (4, 1, 1), (20, 20, 20)), (0x7F, (1, 1, 1), (30, 30, 30))])
def test_chunks_of_many_samples(probe, mask, n_x, n_p):
    """A wave of the short-item form counts its nodes' accepted samples in 32
    bits, two of them per sample with the root samplers: a workgroup of several
    nodes has less than 2^30 samples.  (Beyond that a run takes minutes to hours.)"""
    samples = (1, 100, 1023, 1024, 10 ** 5, 7 * 10 ** 6, 2 ** 29, 2 ** 30, 2 ** 31 - 1)
    cells, nodes = int(np.prod(n_x)), int(np.prod(n_p))
    for precision in (0, 1):
        plans = probe([_case(mask, n_x, n_p, precision, 1, 0, n, 0) for n in samples])
        for n, plan in zip(samples, plans):
            for i, chunk in enumerate(plan["chunks"]):
                assert 1 <= chunk and cells * plan["nch"] * -(-nodes // chunk) < 1 << 31
                if precision == 0 or i >= 2:  # always in the short form
                    assert chunk == 1 or chunk * n < 1 << 30


@pytest.mark.parametrize("n_p", [(6, 6, 6), (9, 10, 11), (20, 20, 20)])
def test_direct_sums_fill_the_compute_units(probe, n_p):
    """Without accumulators a workgroup costs little, so the rounds of workgroups
    over the 256 compute units are nearly full also where one for each (cell,
    channel) pair would leave the last round nearly empty."""
    cells = list(range(20, 120, 3))
    nodes = int(np.prod(n_p))
    for mask in (0x49, 0x7F):
        for samples in (300, 2048):
            plans = probe([_case(mask, (n, 1, 1), n_p, 0, 0, 0, samples, 0) for n in cells])
            for n, plan in zip(cells, plans):
                chunk, split, block = plan["direct"]
                wgs = n * plan["nch"] * -(-nodes // chunk)
                assert wgs / (256 * -(-wgs // 256)) >= 0.85, (mask, samples, n)
