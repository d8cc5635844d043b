"""Launches as the library would make them, seen through a fake HIP runtime (no GPU needed)."""
import random

import pytest

import launch_probe
import tri_rules as R


def test_lds_limits_do_not_depend_on_the_call():
    """The limit on a kernel's dynamic LDS is an attribute of the process: were it each call's own size, a second thread with a
    smaller call could lower it between another's setting and launch."""
    calls = [dict(entry="select", n=n) for n in (1000, 13000, 20000, 32768, 40000)]
    for n in (1000, 4096, 13000, 32768, 40000):
        for offsets in (1, 16, 40, 64):
            calls.append(dict(entry="step", n=n, offsets=offsets, seqs=1 + n % 40, group=4, kv_heads=2, fill=n == 4096, budget=900))
    calls += [dict(entry="step", n=20000, fill=1, budget=b) for b in (1000, 6500, 9000, 16384)]
    calls += [dict(entry="score", group=g, dtype=0, n=600) for g in (1, 8)]
    limits = {}
    for status, launches, set_ in launch_probe.run(calls):
        assert status == 0 and launches
        for name, value in set_:
            limits.setdefault(name, set()).add(value)
        for name, _, _, lds in launches:
            if lds > 48 * 1024:
                assert max(v for k, v in set_ if k == name) >= lds, name
    assert len(limits) > 4
    for name, values in limits.items():
        assert len(values) == 1, "%s: %s" % (name, sorted(values))
        assert max(values) <= 160 * 1024


@pytest.mark.parametrize("layers,heads", [(1, 1), (36, 32), (1, 1 << 23), (65536, 256), (40000, 1024)])
def test_calibration_launches_fit_the_grid(layers, heads):
    """Every (layer, head) has its workgroups, and no launch 2^32 threads along x (the runtime refuses those)."""
    [(status, launches, _)] = launch_probe.run([dict(entry="centers", layers=layers, kv_heads=heads, group=1, tokens=3)])
    assert status == 0
    covered = 0
    for name, (x, y, z), threads, _ in launches:
        assert "centers_kernel" in name and x * threads < 2 ** 32 and y == z == 1
        covered += x
    assert covered >= layers * heads


@pytest.mark.parametrize("layers,heads,rotated,dtype", [(1, 1, 0, 1), (1, 8, 0, 1), (13, 2, 0, 1), (36, 8, 0, 1), (36, 8, 1, 1), (61, 8, 0, 0)])
def test_every_workgroup_of_the_fold_has_work(layers, heads, rotated, dtype):
    """A workgroup per (layer, KV head) -- or per part of its bands, where there are few -- and those that list the batch, write the frequencies
    and fill the phasor table (13 at most) once, not once per layer: less than one per layer leaves without work."""
    [(status, launches, _)] = launch_probe.run([dict(entry="score", layers=layers, kv_heads=heads, group=2, n=500, rotated=rotated, dtype=dtype)])
    assert status == 0
    [(name, (x, y, z))] = [(name, grid) for name, grid, _, _ in launches if "fold_kernel" in name]
    assert y == layers and z == 1
    [parts] = [p for p in (1, 2, 4) if layers * heads * p <= x * y < layers * heads * p + 13 + layers]
    assert ("ILb1E" in name) == (parts > 1), name   # the bands of a workgroup are a variable only where they have to be


def test_the_score_kernel_that_the_rules_name():
    """What R.score_path says, by which the GPU tests know the path that they take, against the kernels that the library launches."""
    rng = random.Random(9)
    calls, paths = [], []
    while len(calls) < 300:
        layers, seqs, heads, group = rng.randint(1, 40), rng.choice([rng.randint(1, 60), 1023, 1024, 1025]), rng.choice([1, 2, 4, 8]), rng.randint(1, 8)
        n, block = int(2 ** rng.uniform(0, 17)), rng.choice([0, 0, 16, 32])
        if layers * seqs * heads * -(-n // 256) >= 2 ** 31 or group * n * 4 >= 2 ** 31:
            continue
        pairs, rotated = int(rng.random() < 0.4), int(rng.random() < 0.3)
        calls.append(dict(entry="score", layers=layers, seqs=seqs, kv_heads=heads, group=group, n=n, block=block, pairs=pairs, rotated=rotated))
        paths.append((group, R.score_path(group, layers * seqs * heads, n, 256, seqs, bool(pairs), bool(block), bool(rotated)), pairs, block, rotated))
    for c, (group, path, pairs, block, rotated), (status, launches, _) in zip(calls, paths, launch_probe.run(calls)):
        assert status == 0, c
        [name] = [name for name, _, _, _ in launches if "score_" in name]
        if path == "sixteen":
            assert "score_mfma_kernel" in name, (c, name)
        else:
            flags = "".join("Lb%dE" % bool(x) for x in (block, rotated, pairs, path == "stretches"))
            assert "score_lane_kernelILi%dE%s" % (group, flags) in name, (c, name)
    assert {p[1] for p in paths} == {"sixteen", "stretches", "items"}
