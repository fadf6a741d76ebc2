"""Test infrastructure: makes the calls below on the built library, with record_launches.cpp preloaded in place of the HIP
runtime, and prints what they launched.  Run as a child process by test_dispatch.py; argument: the stand-in's path.

Every scheme and width, every bucket size, clipping on and off, every power of two and every number of the dispatch in
rounding_part.hip and bingrad.hip as number of buckets, with its neighbours, whole and ragged last buckets, sweeps where the dispatch looks at them,
each with the kernel that the benchmark names for it, and every 64th number of buckets up to 40000 at the sizes of limits.py; the decoder with every number of workers at which it changes its form.
Also the benchmark's workloads at several lengths, with the kernels that the benchmark says they take, and the calls that
profiles/pool_scan.txt, pool_clip_scan.txt and bingrad_scan.txt hold times of."""
import ctypes
import json
import os
import re
import sys
import types

import bench
import paper_2002_11082_amd as ogq
from paper_2002_11082_amd import synth
from tests import limits

SCHEMES = ((ogq.BINGRAD_B, (1,)), (ogq.ORQ, (1, 2, 3)), (ogq.BINGRAD_PB, (1,)), (ogq.ORQ_PAPER, (2, 3, 4)), (ogq.SCALED_SIGN, (1,)),
           (ogq.EVEN, (2, 3, 4)), (ogq.LINEAR, (2, 3, 4)))
SIZES = range(64, 32768 + 1, 64)
ROOT = os.path.dirname(os.path.abspath(bench.__file__))
CSRC = os.path.join(ROOT, "paper_2002_11082_amd", "csrc")
DISPATCH = re.sub("//.*", "", open(os.path.join(CSRC, "rounding_part.hip")).read() +
                  open(os.path.join(CSRC, "bingrad.hip")).read().partition("uint32_t several_buckets_from")[2])
LIMITS = {int(x) for x in re.findall(r"\b(\d+)u\b", DISPATCH)} | {1 << k for k in range(17)}
BUCKETS = sorted({max(1, limit + step) for limit in LIMITS for step in (-1, 0, 1)})
WORKERS = (1, 2, 3, 4, 5, 8, 9, 64)
ADDRESS = 0x10000  # aligned; never looked at
SCANS = (("pool_scan.txt", 0.0), ("pool_clip_scan.txt", 2.5))
SCANNED = {"ORQ 2-bit": (ogq.ORQ, 2), "ORQ 3-bit": (ogq.ORQ, 3), "ORQ-5": (ogq.ORQ_PAPER, 3), "ORQ-9": (ogq.ORQ_PAPER, 4)}


def pool_scan(name):
    """(bucket size, rule, sweeps, buckets, elements cut off) -> times without the pool, times with it."""
    times, d, cut, numbers = {}, 0, 0, []
    for line in open(os.path.join(ROOT, "profiles", name)):
        head = re.match(r"(\d+) elements per bucket, last bucket (whole|cut)$", line)
        if head:
            d, cut = int(head.group(1)), 29 if head.group(2) == "cut" else 0
        elif line.startswith("buckets") and d:
            numbers = [int(x) for x in line.split()[1:]]
        elif d and line.strip():
            rule, sweeps, rest = line.split(",")
            values = [float(x) for x in rest.replace("/", " ").split()[1:]]
            assert len(values) == 2 * len(numbers), line
            for k, nb in enumerate(numbers):
                other, pool = times.setdefault((d, rule, int(sweeps), nb, cut), ([], []))
                other.append(values[2 * k])
                pool.append(values[2 * k + 1])
    return times


def bingrad_scan():
    """(bucket size, rule, threshold updates, clipping factor, buckets), times with one bucket per wavefront and with several."""
    d, numbers = 0, []
    for line in open(os.path.join(ROOT, "profiles", "bingrad_scan.txt")):
        head = re.match(r"(\d+) elements per bucket$", line)
        if head:
            d = int(head.group(1))
        elif line.startswith("buckets") and d:
            numbers = [int(x) for x in line.split()[1:]]
        elif d and line.strip():
            rule, updates, rest = line.split(",")
            clip, *values = [float(x) for x in rest.replace("/", " ").split()]
            assert len(values) == 2 * len(numbers), line
            for k, nb in enumerate(numbers):
                yield (d, rule, int(updates), clip, nb), values[2 * k], values[2 * k + 1]


def main():
    stub = ctypes.CDLL(sys.argv[1])
    for name in ("recorded_launches", "recorded_unknown", "recorded_launches_of"):
        getattr(stub, name).restype = ctypes.c_uint64
    for name in ("recorded_kernels", "recorded_last"):
        getattr(stub, name).restype = ctypes.c_size_t
    stub.recorded_name.restype = ctypes.c_char_p
    stub.recorded_name.argtypes = stub.recorded_launches_of.argtypes = [ctypes.c_size_t]
    lib = ogq.lib()
    quantize, average = lib.ogq_quantize, lib.ogq_dequantize_average
    wrong, decoders = [], {}
    seen = stub.recorded_launches()

    def once(what, status):
        nonlocal seen
        now = stub.recorded_launches()
        if status != 0 or now != seen + 1:
            wrong.append([what, status, now - seen])
        seen = now

    bases = [re.search(r"3ogq\d+([a-z_]+)", stub.recorded_name(i).decode()).group(1) for i in range(stub.recorded_kernels())]
    calls, misnamed = 0, []
    for scheme, widths in SCHEMES:
        for bits in widths:
            for d in SIZES:
                for clip, sweeps in ((0.0, 0), (2.5, 0), (0.0, 1), (0.0, 2)):
                    if sweeps and scheme not in (ogq.BINGRAD_B, ogq.ORQ, ogq.ORQ_PAPER):
                        continue
                    p = ogq.make_params(d, bits, scheme, sweeps, 0, 0, clip)
                    by = ctypes.byref(p)
                    levels = ogq.ogq_levels_per_bucket(p)
                    wl = types.SimpleNamespace(bucket_size=d, scheme=scheme, clip_factor=clip, level_iters=sweeps)
                    for nb in BUCKETS:
                        for n in (nb * d, nb * d - 1):
                            what = f"quantize scheme {scheme} bits {bits} d {d} n {n} clip {clip} sweeps {sweeps}"
                            once(what, quantize(ADDRESS, n, by, ADDRESS, ADDRESS, None))
                            named = bench.quantize_kernel(synth, wl, n, levels)[0]
                            if named != bases[stub.recorded_last()]:
                                misnamed.append([what, named, bases[stub.recorded_last()]])
                            calls += 1
    for d in limits.CHANGES:
        for scheme, bits, sweeps in limits.RULES.values():
            for clip in (0.0, 2.5):
                p = ogq.make_params(d, bits, scheme, sweeps, 0, 0, clip)
                by, levels = ctypes.byref(p), ogq.ogq_levels_per_bucket(p)
                wl = types.SimpleNamespace(bucket_size=d, scheme=scheme, clip_factor=clip, level_iters=sweeps)
                for nb in range(32, 40000, 64):
                    what = f"quantize scheme {scheme} bits {bits} d {d} n {nb * d} clip {clip} sweeps {sweeps}"
                    once(what, quantize(ADDRESS, nb * d, by, ADDRESS, ADDRESS, None))
                    named = bench.quantize_kernel(synth, wl, nb * d, levels)[0]
                    if named != bases[stub.recorded_last()]:
                        misnamed.append([what, named, bases[stub.recorded_last()]])
                    calls += 1
    pointers = (ctypes.c_void_p * 64)(*[ADDRESS] * 64)
    at = ctypes.addressof(pointers)
    for scheme, bits in ((ogq.ORQ, 1), (ogq.ORQ, 2), (ogq.ORQ, 3), (ogq.ORQ_PAPER, 2), (ogq.ORQ_PAPER, 3), (ogq.ORQ_PAPER, 4)):
        for d in SIZES:
            by = ctypes.byref(ogq.make_params(d, bits, scheme))
            for workers in WORKERS:
                once(f"decode scheme {scheme} bits {bits} d {d} workers {workers}",
                     average(at, at, workers, 100 * d + 1, by, ADDRESS, None))
                decoders.setdefault(stub.recorded_last(), set()).add(d)
                calls += 1
    named = []
    for name in bench.WORKLOAD_NAMES:
        wl = synth.WORKLOADS[name]
        for n in (1000, 100_000, 1_000_000, 10_000_000, 25_600_000, wl.n, 400_000_000):
            p = ogq.make_params(wl.bucket_size, wl.bits, wl.scheme, wl.level_iters, 0, 0, wl.clip_factor)
            once(f"quantize {name} at {n}", quantize(ADDRESS, n, ctypes.byref(p), ADDRESS, ADDRESS, None))
            kernel, wavefronts = bench.quantize_kernel(synth, wl, n, ogq.ogq_levels_per_bucket(p))
            here = stub.recorded_last_blocks() * stub.recorded_last_threads() / 64 * wl.bucket_size / n
            named.append([f"quantize {name} at {n}", kernel, stub.recorded_last(), wavefronts, here])
            once(f"decode {name} at {n}", average(at, at, wl.workers, n, ctypes.byref(p), ADDRESS, None))
            named.append([f"decode {name} at {n}", bench.decode_kernel_name(wl.bucket_size, wl.workers), stub.recorded_last(), 0, 0])
    scanned = []
    for name, clip in SCANS:
        for (d, rule, sweeps, nb, cut), (other, pool) in pool_scan(name).items():
            scheme, bits = SCANNED[rule]
            p = ogq.make_params(d, bits, scheme, sweeps, 0, 0, clip)
            once(f"quantize {rule} {sweeps} sweeps d {d} n {nb * d - cut} clip {clip}",
                 quantize(ADDRESS, nb * d - cut, ctypes.byref(p), ADDRESS, ADDRESS, None))
            scanned.append([d, rule, sweeps, nb, clip, stub.recorded_last(), other, pool])
    shared = []
    for (d, rule, updates, clip, nb), one, several in bingrad_scan():
        scheme = ogq.BINGRAD_B if rule == "BinGrad-b" else ogq.SCALED_SIGN
        p = ogq.make_params(d, 1, scheme, updates, 0, 0, clip)
        once(f"quantize {rule} {updates} updates d {d} n {nb * d - 29} clip {clip}",
             quantize(ADDRESS, nb * d - 29, ctypes.byref(p), ADDRESS, ADDRESS, None))
        shared.append([d, clip, updates, nb, stub.recorded_last(), one, several])
    once("probe_read", lib.ogq_probe_read(ADDRESS, 64, ADDRESS, None))
    once("probe_copy", lib.ogq_probe_copy(ADDRESS, ADDRESS, 64, None))
    names = [stub.recorded_name(i).decode() for i in range(stub.recorded_kernels())]
    print(json.dumps({"calls": calls, "wrong": wrong[:20], "misnamed": misnamed[:20], "unknown": stub.recorded_unknown(),
                      "launches": {name: stub.recorded_launches_of(i) for i, name in enumerate(names)},
                      "named": [[what, kernel, names[i], stated, here] for what, kernel, i, stated, here in named],
                      "scanned": [[d, rule, sweeps, nb, clip, names[i], other, pool] for d, rule, sweeps, nb, clip, i, other, pool in scanned],
                      "shared": [[d, clip, updates, nb, names[i], one, several] for d, clip, updates, nb, i, one, several in shared],
                      "decoded_sizes": {names[i]: sorted(sizes) for i, sizes in decoders.items()}}))


if __name__ == "__main__":
    main()
