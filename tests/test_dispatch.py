"""Which kernel a call ends in, without a GPU: a call that the entry points accept is one kernel launch or an error, and
none may return success without having launched anything."""
import json
import os
import re
import subprocess
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUBS = os.path.join(ROOT, "tests", "host_stubs")


def test_a_combination_that_is_not_compiled_is_an_error(tmp_path):
    from paper_2002_11082_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    program = str(tmp_path / "team_without_kernel")
    flags = [f for f in build.HIPCC_FLAGS if f != "-O3"]
    subprocess.run([hipcc, *flags, "-O0", os.path.join(STUBS, "team_without_kernel.hip"), "-o", program], check=True, timeout=300)
    res = subprocess.run([program], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    """The launches of every_call.py on the built library."""
    from paper_2002_11082_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    stub = str(tmp_path_factory.mktemp("record") / "record_launches.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", os.path.join(STUBS, "record_launches.cpp"), "-o", stub], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = ":".join(x for x in (stub, env.get("LD_PRELOAD")) if x)
    env["PYTHONPATH"] = ROOT + os.pathsep + env.get("PYTHONPATH", "")
    res = subprocess.run([sys.executable, os.path.join(STUBS, "every_call.py"), stub], cwd=ROOT, env=env, capture_output=True,
                         text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    return json.loads(res.stdout)


def test_every_accepted_call_is_one_launch(recorded):
    assert recorded["calls"] > 1_000_000
    assert recorded["wrong"] == [] and recorded["unknown"] == 0


def test_every_kernel_of_the_library_is_reached(recorded):
    assert len(recorded["launches"]) > 400
    assert [name for name, launches in recorded["launches"].items() if launches == 0] == []


def test_the_benchmark_names_the_kernels_that_run(recorded):
    assert len(recorded["named"]) > 200
    for what, stated, launched, wavefronts, wavefronts_launched in recorded["named"]:
        assert re.search(rf"ogq\d+{stated}I", launched), (what, stated, launched)
        if wavefronts and what.endswith("at 400000000"):  # (few buckets: whole workgroups, whole groups of buckets)
            assert abs(wavefronts_launched / wavefronts - 1) < 0.01, (what, wavefronts, wavefronts_launched)


def test_the_benchmark_repeats_the_dispatch(recorded):
    """bench.py names the kernel of a call from limits of its own: the same as the library's, on both sides of each."""
    assert recorded["misnamed"] == []


def test_the_listed_limits_are_those_of_the_dispatch():
    """limits.py against the limits that bench.py repeats (which the test above holds against the library): every number of buckets up to
    40000 where the kernel changes, whatever the form of the rule, but for ranges of fewer than 16."""
    import bench
    import paper_2002_11082_amd as ogq
    from paper_2002_11082_amd import synth
    from tests import limits

    def changes(kernel, low, high):
        if kernel(low) == kernel(high):
            return []
        middle = (low + high) // 2
        return [low] if middle == low else changes(kernel, low, middle) + changes(kernel, middle, high)

    for d, stated in limits.CHANGES.items():
        found = {}
        for name, (scheme, bits, sweeps) in limits.RULES.items():
            wl = types.SimpleNamespace(bucket_size=d, scheme=scheme, clip_factor=0.0, level_iters=sweeps)
            levels = ogq.ogq_levels_per_bucket(ogq.make_params(d, bits, scheme))
            for low in range(0, 40000, 16):
                for nb in changes(lambda nb: bench.quantize_kernel(synth, wl, nb * d, levels), max(low, 1), low + 16):
                    found.setdefault(nb, []).append(name)
        assert found == {limit: limits.rules(names) for limit, names in stated.items()}, d


def test_the_pool_is_taken_where_the_record_shows_a_gain(recorded):
    """profiles/pool_scan.txt and pool_clip_scan.txt: the calls that end in orq_pool_kernel against the same calls in the kernel it
    stands in for, on the mean of the recorded kinds of values and last buckets, and for each kind; and the calls that do not.  0.035: single
    sizes of ranges that gain, and what two scans of the same kernels differ by; 0.13: one kind in few buckets, where the slowest bucket is
    the call's time, and numbers of buckets below a limit that several sizes share."""
    points = {}
    for d, rule, sweeps, nb, clip, launched, other, pool in recorded["scanned"]:
        taken, kinds = points.setdefault((d, rule, sweeps, nb, clip), (set(), [[] for _ in other]))
        taken.add("orq_pool_kernel" in launched)
        for kind, a, b in zip(kinds, other, pool):  # (rows of a section: one per kind, in the same order)
            kind.append(b / a)
    assert len(points) > 8000
    assert all(len(taken) == 1 and len(kinds) == 4 for taken, kinds in points.values())
    mean = {point: sum(map(sum, kinds)) / sum(map(len, kinds)) - 1.0 for point, (_, kinds) in points.items()}
    worst = {point: max(sum(kind) / len(kind) for kind in kinds) - 1.0 for point, (_, kinds) in points.items()}
    pool = [point for point, (taken, _) in points.items() if taken == {True}]
    assert len(pool) > 6000 and sum(mean[point] for point in pool) / len(pool) < -0.15
    assert {point: round(mean[point], 3) for point in pool if mean[point] > 0.035} == {}
    assert {point: round(worst[point], 3) for point in pool if worst[point] > 0.13} == {}
    assert {point: round(mean[point], 3) for point in points if points[point][0] == {False} and mean[point] < -0.13} == {}


def test_buckets_share_a_wavefront_where_the_record_shows_a_gain(recorded):
    """profiles/bingrad_scan.txt: one bucket per wavefront or several; without updates on the mean of BinGrad-b and Scaled SignSGD.  0.05:
    ranges that gain with a number in them that does not; 0.25: numbers below a limit that gain, with others between that lose."""
    points = {}
    for d, clip, updates, nb, launched, one, several in recorded["shared"]:
        taken, ratios = points.setdefault((d, clip, updates, nb), (set(), []))
        taken.add("bingrad_chunk_kernel" in launched)
        ratios.append(several / one)
    assert len(points) > 1600 and all(len(taken) == 1 for taken, _ in points.values())
    change = {point: (taken == {True}, sum(ratios) / len(ratios) - 1.0) for point, (taken, ratios) in points.items()}
    assert {point: loss for point, (taken, loss) in change.items() if taken and loss > 0.05} == {}
    assert {point: gain for point, (taken, gain) in change.items() if not taken and gain < -0.25} == {}


def _buckets_of_a_span(d):
    """The most buckets that any 1024 consecutive elements touch which begin at a multiple of 1024."""
    return max((start % d + 1023) // d + 1 for start in range(0, 1024 * d, 1024))


def test_joint_decoder_holds_the_buckets_of_a_span(recorded):
    """dequantize_joint_kernel<BITS, S, BUCKETS, ...> keeps BUCKETS tables in LDS per wavefront: as many as a span of one of
    its bucket sizes touches, neither fewer (a write out of its range) nor more (wavefronts that do not fit)."""
    tables = {}
    for name, sizes in recorded["decoded_sizes"].items():
        form = re.search(r"dequantize_joint_kernelILi(\d+)ELi(\d+)ELj(\d+)E", name)
        if form:
            for d in sizes:
                tables.setdefault(d, set()).add(int(form.group(3)))
    assert len(tables) > 500
    for d, held in tables.items():
        assert len(held) == 1 and min(held) >= _buckets_of_a_span(d), (d, held)
        if d < 512:
            assert held == {_buckets_of_a_span(d)}, (d, held)
