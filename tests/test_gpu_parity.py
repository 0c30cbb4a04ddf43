"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same seeded inputs.

Bucketing is integer work: perm, inv_perm, offsets, scan_bucket_start and the per-round placement
counts must match bit for bit. Attention is compared element by element within max-abs 1e-2
(bf16 inputs and outputs, fp32 accumulation on the GPU; binary64 in the oracle); at the full
benchmark sizes the comparison runs on sampled query rows, each computed in full by the oracle.
"""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2412_16481_amd as f3d
from paper_2412_16481_amd import workloads as wl

pytestmark = pytest.mark.gpu

ATOL = 1e-2   # max-abs bound on attention outputs
HASHES = ["xor_mod", "xor_div", "zorder_mod", "zorder_div"]
DEV = "cuda:0"


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.view(dtype)
    return t.to(DEV)


def run_bucketize(coords, bo, voxel, cap, m=4, hash="zorder_div", n_probes=6, max_scan_points=0, div=0, probe_step=0,
                  schedule="auto", order="index", probe_mode="axes", probe_seed=0, probe_table=None):
    p = f3d.make_params(voxel, cap, m, hash, n_probes, div, probe_step, max_scan_points, schedule, order, probe_mode,
                        probe_seed, probe_table)
    bk = f3d.psh_bucketize(dev(coords), None if bo is None else dev(bo.astype(np.int32)), p)
    torch.cuda.synchronize()
    return bk


def check_bucketize(coords, bo, voxel, cap, m=4, hash="zorder_div", n_probes=6, **kw):
    S = cap // m
    bo_arr = np.array([0, coords.shape[0]], dtype=np.int32) if bo is None else bo
    ref = oracle.bucketize(coords, bo_arr, voxel, S, hash, n_probes, kw.get("div", 0), kw.get("probe_step", 0),
                           kw.get("order", "index"), kw.get("probe_mode", "axes"), kw.get("probe_seed", 0),
                           kw.get("probe_table"))
    bk = run_bucketize(coords, bo, voxel, cap, m, hash, n_probes, **kw)
    K = len(ref["offsets"]) - 1
    assert bk.scan_bucket_start.cpu().numpy().tolist() == ref["scan_bucket_start"].tolist()
    assert np.array_equal(bk.offsets.cpu().numpy()[:K + 1], ref["offsets"])
    assert (bk.offsets.cpu().numpy()[K:] == coords.shape[0]).all()
    assert np.array_equal(bk.perm.cpu().numpy(), ref["perm"])
    assert np.array_equal(bk.inv_perm.cpu().numpy(), ref["inv_perm"])
    rc = np.bincount(ref["round_of"], minlength=8)[:8] if coords.shape[0] else np.zeros(8, dtype=np.int64)
    assert bk.placed_per_round.cpu().numpy().tolist() == rc.tolist()
    return bk, ref


# ----------------------------------------------------------------------------- bucketize


@pytest.mark.parametrize("name", wl.CONFIG_NAMES)
@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_matches_oracle_on_workloads(name, hash):
    w = wl.make_workload(name)
    check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, w.scope_buckets, hash)


@pytest.mark.parametrize("n", [1, 1023, 1024, 2049, 9000, 70001, 262145])
def test_bucketize_one_scan_with_a_launch_per_step(n):
    # one scan's chunks (of 1024 and of 2048 points) follow from the launch; offsets that say otherwise are flagged and nothing is written
    rng = np.random.default_rng(17)
    pts = (rng.random((n, 3)) * [9.0, 7.0, 2.0]).astype(np.float32)
    cap = 1024 if n < 200_000 else 2048
    for bo, most in ((None, 0), (np.array([0, n], dtype=np.int32), 0), (None, 2 * n)):
        check_bucketize(pts, bo, 0.05, cap, schedule="steps", max_scan_points=most)
    for bo, most in (([0, n - 1], 0), ([1, n], 0), ([0, n + 1], 0), ([0, n], n - 1)):
        if n == 1 and most == 0 and bo == [0, n]:
            continue   # no bound at all
        p = f3d.make_params(0.05, cap, 4, schedule="steps", max_scan_points=most)
        bk = f3d.psh_bucketize(dev(pts), dev(np.array(bo, dtype=np.int32)), p)
        bk.perm.fill_(-7)
        bk.inv_perm.fill_(-7)
        f3d.psh_bucketize(dev(pts), dev(np.array(bo, dtype=np.int32)), p, out=bk)
        torch.cuda.synchronize()
        assert int(bk.scan_bucket_start[-1]) == -1
        assert bool((bk.perm == -7).all()) and bool((bk.inv_perm == -7).all())


@pytest.mark.parametrize("order", ["index", "canonical"])
@pytest.mark.parametrize("n_scans", [64, 65, 200])
def test_bucketize_many_scans_with_a_launch_per_step_flags_bad_offsets(n_scans, order):
    # the steps load what the chunk table names before they look at the status: the set-up (one kernel up to 64 scans, another for more)
    # names no chunk in a flagged call. A row of the table is 32 bytes and begins with its scan, -1 for none.
    n = 9001
    pts = (np.random.default_rng(18).random((n, 3)) * [9.0, 7.0, 2.0]).astype(np.float32)
    good = np.linspace(0, n, n_scans + 1).astype(np.int32)
    check_bucketize(pts, good, 0.05, 64, schedule="steps", order=order)
    back, early, late, above = good.copy(), good.copy(), good + 1, good.copy()
    back[[n_scans // 2, n_scans // 2 + 1]] = back[[n_scans // 2 + 1, n_scans // 2]]
    early[-1] = n - 1
    most = int(np.diff(good).max())
    for bo, bound in ((back, 0), (early, 0), (late, 0), (above, most - 1)):
        p = f3d.make_params(0.05, 64, 4, schedule="steps", order=order, max_scan_points=bound)
        ws = torch.zeros(f3d.workspace_bytes(n, n_scans, p), dtype=torch.uint8, device=DEV)
        bk = f3d.psh_bucketize(dev(pts), dev(good), f3d.make_params(0.05, 64, 4, schedule="steps"))
        for t in (bk.perm, bk.inv_perm):
            t.fill_(-7)
        f3d.psh_bucketize(dev(pts), dev(bo), p, ws, out=bk)
        torch.cuda.synchronize()
        assert int(bk.scan_bucket_start[-1]) == -1
        assert bool((bk.perm == -7).all()) and bool((bk.inv_perm == -7).all())
        none = (ws[:ws.numel() // 32 * 32].view(torch.int32).reshape(-1, 8)[:, 0] == -1).cpu().numpy()
        ends = np.flatnonzero(np.diff(np.concatenate([[0], none.astype(np.int8), [0]])))
        # longer than the run of empty bounding boxes, one per scan, which look the same
        assert int(np.diff(ends)[::2].max()) >= n // 2048 + n_scans


@pytest.mark.parametrize("n", [1, 2, 2047, 2048, 2049, 4096, 4097, 6145, 8193, 12289])
def test_bucketize_canonical_order_at_sort_tile_edges(n):
    # sizes around the sort's tiles and runs (an odd run without a partner among them), a lattice with many equal points
    # (ties by index), signed coordinates, and one voxel for everything (the coordinates decide)
    rng = np.random.default_rng(32)
    lattice = rng.integers(-3, 4, (n, 3)).astype(np.float32) * np.float32(0.25)
    check_bucketize(lattice, None, 0.5, 128, 4, "zorder_div", order="canonical")
    check_bucketize((rng.random((n, 3)) - 0.5).astype(np.float32), None, 16.0, 256, 4, "xor_mod", order="canonical")
    bo = np.array([0, n // 3, n // 3, n], dtype=np.int32)
    check_bucketize(clustered_cloud(rng, n), bo, 0.05, 128, 4, "zorder_mod", order="canonical")


@pytest.mark.parametrize("schedule", ["general", "steps", "scans"])
@pytest.mark.parametrize("name,hash", [("tiny", "xor_mod"), ("indoor", "zorder_div"), ("indoor", "xor_div"), ("lidar4", "zorder_mod")])
def test_bucketize_every_schedule_gives_the_oracle_result(name, hash, schedule):
    # the two ways of putting the steps on the GPU (two launches per step, one per step) are the same function
    w = wl.make_workload(name)
    largest = int(np.diff(w.batch_offsets).max()) if w.batch_offsets is not None else w.n   # sizes the count matrix per scan
    check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, w.scope_buckets, hash, schedule=schedule,
                    max_scan_points=largest)


@pytest.mark.parametrize("schedule", ["general", "steps", "scans"])
def test_bucketize_schedules_on_ragged_scans(schedule):
    rng = np.random.default_rng(27)
    sizes = [1, 2047, 2048, 2049, 0, 5000, 77, 0, 12000]
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = np.concatenate([wl.uniform_cube(rng, s, 1.0 + i) + 10.0 * i for i, s in enumerate(sizes)]).astype(np.float32)
    for n_probes in (0, 3, 6):
        check_bucketize(c, bo, 0.05, 256, 4, "zorder_div", n_probes, schedule=schedule)


@pytest.mark.parametrize("n", [1, 5, 64, 65, 2047, 2048, 2049, 4097, 20000])
def test_bucketize_one_workgroup_per_scan_small_and_ragged_sizes(n):
    rng = np.random.default_rng(300 + n)
    c = clustered_cloud(rng, n)
    for hash in HASHES:
        check_bucketize(c, None, 0.05, 128, 4, hash, schedule="scans")
    check_bucketize(c, None, 0.05, 1 << 17, 4, "zorder_div", n_probes=0, schedule="scans")   # one bucket, no probes
    check_bucketize(c, None, 0.05, 256, 2, "xor_div", n_probes=3, schedule="scans", order="canonical")


def test_bucketize_batches_of_many_scans_take_the_scan_path_by_themselves():
    """100 uneven scans (some empty), none above 1/24 of the points: the automatic choice is one workgroup per scan
    (its workspace holds the two lists of unplaced points); the result is the oracle's whatever the schedule."""
    rng = np.random.default_rng(310)
    sizes = rng.integers(0, 3000, 100)
    sizes[[3, 50, 99]] = 0
    sizes[7] = 1
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(bo[-1])
    c = np.concatenate([clustered_cloud(rng, int(sz), 2.0 * i) for i, sz in enumerate(sizes)]).astype(np.float32).reshape(n, 3)
    largest = int(sizes.max())
    p_auto = f3d.make_params(0.05, 256, 4, "zorder_div", max_scan_points=largest)
    p_steps = f3d.make_params(0.05, 256, 4, "zorder_div", max_scan_points=largest, schedule="steps")
    assert f3d.workspace_bytes(n, 100, p_auto) >= f3d.workspace_bytes(n, 100, p_steps) + 24 * n
    for hash in ("zorder_div", "xor_mod"):
        for schedule in ("auto", "scans", "steps"):
            check_bucketize(c, bo, 0.05, 256, 4, hash, max_scan_points=largest, schedule=schedule)
    check_bucketize(c, bo, 0.05, 256, 4, "zorder_mod", max_scan_points=largest, probe_mode="seeded", probe_seed=5)
    check_bucketize(c, bo, 0.05, 256, 4, "xor_div", max_scan_points=largest, order="canonical")


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_more_scans_than_compute_units(hash):
    """300 uneven scans: more workgroups than the GPU has compute units, which takes the form of the one-workgroup-
    per-scan kernel that is compiled for two workgroups per compute unit."""
    rng = np.random.default_rng(311 + HASHES.index(hash))
    sizes = rng.integers(0, 2500, 300)
    sizes[[0, 17, 299]] = 0
    sizes[5] = 9000
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(bo[-1])
    c = np.concatenate([clustered_cloud(rng, int(sz), 1.5 * i) for i, sz in enumerate(sizes)]).astype(np.float32).reshape(n, 3)
    largest = int(sizes.max())
    check_bucketize(c, bo, 0.05, 256, 4, hash, max_scan_points=largest, schedule="scans")
    check_bucketize(c, bo, 0.05, 128, 2, hash, n_probes=3, max_scan_points=largest, schedule="scans")


def test_bucketize_one_workgroup_per_scan_is_refused_above_1024_buckets_per_scan():
    p = f3d.make_params(0.05, 64, 4, "zorder_div", schedule="scans")      # S = 16: 20000 points are 1250 buckets
    with pytest.raises(f3d.Flash3DError) as e:
        f3d.psh_bucketize(dev(np.zeros((20000, 3), np.float32)), None, p)
    assert e.value.code == f3d.ERR_UNSUPPORTED


@pytest.mark.parametrize("hash", ["zorder_div", "zorder_mod"])
def test_bucketize_scan_path_axis_probes_with_wide_voxels(hash):
    # voxel coordinates below and above 2^11 and up to the saturation at 2^21 - 1, an axis on which the scan is flat, probe
    # steps from one voxel to beyond the box: the workgroup that walks a scan moves the Z-order code itself
    rng = np.random.default_rng(33)
    c = np.concatenate([clustered_cloud(rng, 3000), (rng.random((3000, 3)) * 6.0).astype(np.float32)])
    flat = c.copy()
    flat[:, 1] = 2.5
    bo = np.array([0, 2900, 2900, 6000], dtype=np.int32)
    for cloud in (c, flat):
        for voxel in (0.02, 0.0015, 1e-6):
            for step in (0, 1, 700, 1 << 22):
                check_bucketize(cloud, bo, voxel, 128, 4, hash, schedule="scans", probe_step=step)


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_small_scans_eight_points_per_thread(hash):
    # more than four points per thread: around the last of them and one past it (another path), few and many survivors, most
    # buckets the path takes, every number of probes, a batch whose scans end inside and at the end of a wave's run
    rng = np.random.default_rng(36)
    for n in (4097, 5000, 8191, 8192, 8193):
        check_bucketize(clustered_cloud(rng, n), None, 0.05, 64 if n <= 8192 else 128, 4, hash, n_probes=(n % 7))
        for probe_mode in ("seeded", "axes"):     # codes of more than 30 bits
            check_bucketize((rng.random((n, 3)) * 4.0).astype(np.float32), None, 0.0005, 256, 4, hash, probe_mode=probe_mode, probe_seed=3)
    check_bucketize((rng.random((8192, 3)) * 4.0).astype(np.float32), None, 0.05, 32, 2, hash)    # buckets of 16 rows, 512 of them
    bo = np.array([0, 8192, 8192, 8193, 12289, 20000, 25121], dtype=np.int32)
    c = np.concatenate([clustered_cloud(rng, int(k), float(i)) for i, k in enumerate(np.diff(bo)) if k])
    check_bucketize(c, bo, 0.05, 128, 4, hash, max_scan_points=8192)


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_small_scans_every_width_and_number_of_probes(hash):
    # one to eight groups of 64 per wave, at both ends of each and on both sides of the line to the other path (4096 points and 682
    # more per probe); few points left (they change waves) and most of them
    rng = np.random.default_rng(39)
    for n in (1024, 1025, 2048, 2049, 3072, 3073, 4096, 5120, 5121, 6144, 6145, 7168, 7169, 8192):
        for c in (clustered_cloud(rng, n), (rng.random((n, 3)) * 4.0).astype(np.float32)):
            check_bucketize(c, None, 0.05, 128, 4, hash)
    for n_probes in range(6):
        for n in (4096 + n_probes * 2048 // 3, 4097 + n_probes * 2048 // 3):
            check_bucketize(clustered_cloud(rng, n), None, 0.05, 128, 4, hash, n_probes)
            check_bucketize((rng.random((n, 3)) * 4.0).astype(np.float32), None, 0.05, 512, 4, hash, n_probes)


@pytest.mark.parametrize("per_bucket,edge", [(1600, 4096 // 6), (3200, 6144 // 6), (5120, 8192 // 6)])
def test_bucketize_small_scans_at_the_edge_of_few_points_left(per_bucket, edge):
    # all but three points in one voxel: its bucket takes `per_bucket`, `edge` are left and change waves, one more and they stay.
    # Probes over the whole box reach the other bucket and place some of them
    table = [[0, 0, 0], [9, 0, 0], [0, 9, 0], [9, 9, 9], [3, 0, 7], [-1, -1, -1]]
    for left in (edge - 1, edge, edge + 1):
        c = np.full((per_bucket + left, 3), 0.5, dtype=np.float32)
        c[[7, 1000, 1500]] = [[9.5, 9.5, 9.5], [9.5, 0.5, 0.5], [0.5, 9.5, 0.5]]
        for hash in HASHES:
            check_bucketize(c, None, 1.0, 4 * per_bucket, 4, hash, probe_mode="table", probe_table=table)
            check_bucketize(c, None, 1.0, 4 * per_bucket, 4, hash)


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_scan_path_block_edges_in_unequal_scans(hash):
    # the walk of a scan in blocks (8192 points, 4096 with more scans than compute units), its lists beside those of the other
    # scans: sizes around a block, most points left over or hardly any, codes of up to and of more than 30 bits
    rng = np.random.default_rng(34)
    sizes = np.array([8191, 0, 8193, 4096, 16385, 1, 8192, 24577])
    many = np.concatenate([sizes, rng.integers(0, 130, 292)])
    for sz, voxels in ((sizes, (0.05, 0.0005)), (many, (0.05,))):
        bo = np.concatenate([[0], np.cumsum(sz)]).astype(np.int32)
        for voxel in voxels:
            for cloud in (lambda k: clustered_cloud(rng, k), lambda k: rng.random((k, 3)) * 4.0):
                c = np.concatenate([cloud(int(k)) for k in sz if k]).astype(np.float32)
                check_bucketize(c, bo, voxel, 256, 4, hash, max_scan_points=int(sz.max()), schedule="scans")


@pytest.mark.parametrize("schedule", ["auto", "general", "steps", "scans"])
def test_bucketize_quotients_at_bucket_boundaries(schedule):
    # every voxel of a 16^3, 32^3 and 64 x 64 x 16 lattice once, in mixed order: with the Z-order-div hash the codes run through
    # all multiples of the divisor, where a quotient estimate must be settled by the exact remainder
    rng = np.random.default_rng(35)
    for shape, cap in (((16, 16, 16), 64), ((32, 32, 32), 128), ((32, 32, 32), 192), ((64, 64, 16), 256)):
        g = np.stack(np.meshgrid(*(np.arange(k) for k in shape), indexing="ij"), axis=-1).reshape(-1, 3)
        c = (rng.permutation(g) * 0.25 + 0.0625).astype(np.float32)     # exact in binary32, a quarter voxel from the faces
        check_bucketize(c, None, 0.25, cap, 4, "zorder_div", schedule=schedule)


def compact3(code):
    """Every third bit of the codes: one axis of a Z-order code of up to 60 bits."""
    return sum(((code >> np.uint64(3 * k)) & np.uint64(1)) << np.uint64(k) for k in range(20)).astype(np.int64)


@pytest.mark.parametrize("bits", [10, 12, 20])
@pytest.mark.parametrize("schedule,n", [("auto", 4000), ("auto", 8000), ("scans", 16000), ("steps", 32000), ("general", 130000)])
def test_bucketize_quotients_beside_multiples_of_other_divisors(schedule, n, bits):
    # Z-order-div over a voxel box of 2^bits per axis with 250 to 8125 buckets: the divisor is no power of two, so its reciprocal is
    # rounded. Codes one below, at and one above its multiples, up to 30 bits (the 32-bit form), 36 and 60 (the conversion to
    # binary32 rounds too), and random ones; buckets of 16 rows, so that a point in the wrong one moves others
    rng = np.random.default_rng(40)
    K = n // 16
    D = (2 ** (3 * bits) - 1) // K + 1
    assert D & (D - 1)
    near = np.array([k * D + d for k in range(1, K) for d in (-1, 0, 1)], dtype=np.uint64)
    ends = np.array([0, 2 ** (3 * bits) - 1], dtype=np.uint64)          # the corners of the box
    code = rng.permutation(np.concatenate([near, near, ends, rng.integers(0, 2 ** (3 * bits), n - 2 * len(near) - 2, dtype=np.uint64)]))
    c = np.stack([compact3(code >> np.uint64(a)) for a in range(3)], axis=1) + 0.5      # exact in binary32
    for n_probes in (0, 6):
        check_bucketize(c.astype(np.float32), None, 1.0, 64, 4, "zorder_div", n_probes, schedule=schedule)


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_small_scans_in_registers(hash):
    # scans that fit one workgroup's registers: around a wave, a workgroup, and one past the last (another path); clustered
    # points (most are left over) and uniform ones (closed up early); single scans (one launch) and batches with empty
    # and one-point scans
    rng = np.random.default_rng(31)
    for n in (1, 63, 64, 65, 1023, 1024, 1025, 2049, 4095, 4096, 4097):
        c = clustered_cloud(rng, n)
        check_bucketize(c, None, 0.05, 64 if n != 4095 else 192, 4, hash, n_probes=(n % 7))
        check_bucketize((rng.random((n, 3)) * 4.0).astype(np.float32), None, 0.02, 128, 4, hash)
    bo = np.array([0, 0, 1, 4097, 4097, 7000, 9049, 9050, 9050], dtype=np.int32)
    c = np.concatenate([clustered_cloud(rng, int(k), float(i)) for i, k in enumerate(np.diff(bo)) if k])
    for order, probe_mode in (("index", "axes"), ("canonical", "seeded")):
        check_bucketize(c, bo, 0.05, 128, 4, hash, max_scan_points=4096, order=order, probe_mode=probe_mode, probe_seed=5)


@pytest.mark.parametrize("schedule", ["general", "steps", "scans"])
def test_bucketize_probe_offsets_at_the_limits_of_int32(schedule):
    """A probe step or a table offset of any size is legal: the moved voxel is clamped to the scan's voxel box."""
    rng = np.random.default_rng(320)
    c = clustered_cloud(rng, 9000)
    big = 2 ** 31 - 1
    check_bucketize(c, None, 0.01, 256, 4, "zorder_div", probe_step=big, schedule=schedule)
    check_bucketize(c, None, 0.01, 256, 4, "xor_mod", probe_step=1 << 22, schedule=schedule)
    table = [[big, 0, 0], [-big - 1, 3, 0], [0, -big, big], [1 << 21, -(1 << 21), 0], [5, 5, -5], [-(1 << 22) - 1, (1 << 22) + 1, 7]]
    check_bucketize(c, None, 0.01, 256, 4, "zorder_mod", probe_mode="table", probe_table=table, schedule=schedule)
    check_bucketize(c, None, 1e-6, 256, 4, "xor_div", probe_mode="table", probe_table=table, schedule=schedule)   # saturated voxels


def test_bucketize_one_launch_per_step_is_refused_for_a_large_count_matrix():
    w = wl.make_workload("lidar8")   # taken as ONE scan of 9e5 points: 447 chunks x 3573 buckets
    p = f3d.make_params(w.voxel_size, w.bucket_cap, w.scope_buckets, "zorder_div", schedule="steps")
    with pytest.raises(f3d.Flash3DError) as e:
        f3d.psh_bucketize(dev(w.coords), None, p)
    assert e.value.code == f3d.ERR_UNSUPPORTED


@pytest.mark.parametrize("n", [1, 5, 63, 64, 65, 1023, 1024, 1025, 4097, 20000])
def test_bucketize_small_and_ragged_sizes(n):
    rng = np.random.default_rng(n)
    c = wl.uniform_cube(rng, n, 1.5)
    for hash in ("zorder_div", "xor_mod"):
        check_bucketize(c, None, 0.05, 64, 4, hash)


@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_half_chunks_on_the_one_launch_per_step_path(hash):
    # batches small enough for chunks of 1024 points: scans around a chunk, empty ones, the most chunks (256 with 262143 points, the
    # largest count matrix as well) and the first size past them, most points left over (their rank runs on over chunks and
    # buckets of odd capacity) or hardly any
    rng = np.random.default_rng(37)
    for sizes in ([1023, 0, 1025, 1024, 2049, 1, 9000, 0], [65536], [261119], [262143], [262144], [65537, 3]):
        bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        cap = 128 if max(sizes) < 10000 else 2048 if max(sizes) > 70000 else 128      # 65536 points in 2048 buckets
        for cloud in (lambda k: clustered_cloud(rng, k), lambda k: rng.random((k, 3)) * 4.0):
            c = np.concatenate([cloud(int(k)) for k in sizes if k]).astype(np.float32)
            for n_probes in (6, 0):
                check_bucketize(c, bo, 0.05, cap, 4, hash, n_probes, max_scan_points=max(sizes), schedule="steps" if max(sizes) < 65537 or cap > 128 else "auto")


@pytest.mark.parametrize("sizes,cap,small", [([9000], 1024, 77312), ([185344], 1024, 2028544), ([262143], 2048, 2640384),
                                             ([30000, 0, 40000, 40000, 40000], 256, 1615104)])
def test_bucketize_takes_a_workspace_without_room_for_half_chunks(sizes, cap, small):
    """The workspace asked for has rows for chunks of 1024 points; a buffer with room for those of 2048 (`small` bytes: 64 bytes
    of tables and two count rows per chunk) is taken all the same, and one of 256 bytes less refused."""
    rng = np.random.default_rng(38)
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = np.concatenate([clustered_cloud(rng, k) for k in sizes if k]).astype(np.float32)
    _, ref = check_bucketize(c, bo, 0.05, cap, 4, max_scan_points=max(sizes), schedule="steps")
    p = f3d.make_params(0.05, cap, 4, max_scan_points=max(sizes), schedule="steps")
    assert f3d.workspace_bytes(len(c), len(sizes), p) > small
    ws = torch.empty(small, dtype=torch.uint8, device=DEV)
    got = f3d.psh_bucketize(dev(c), dev(bo), p, workspace=ws)
    assert np.array_equal(got.perm.cpu().numpy(), ref["perm"]) and np.array_equal(got.inv_perm.cpu().numpy(), ref["inv_perm"])
    with pytest.raises(f3d.Flash3DError) as e:
        f3d.psh_bucketize(dev(c), dev(bo), p, workspace=ws[:-256])
    assert e.value.code == f3d.ERR_WORKSPACE_TOO_SMALL


def test_bucketize_widest_count_rows_on_the_one_launch_per_step_path():
    # 2048 buckets in one scan of 64 chunks: the largest LDS footprint of the step kernel (above the 64 KB default)
    rng = np.random.default_rng(28)
    c = wl.uniform_cube(rng, 2048 * 64, 3.0)
    check_bucketize(c, None, 0.02, 256, 4, "zorder_mod", schedule="steps")
    check_bucketize(c[:2048 * 64 - 100], None, 0.02, 256, 4, "xor_div", n_probes=2, schedule="steps")


def test_bucketize_empty_input_and_empty_scans():
    c = np.zeros((0, 3), dtype=np.float32)
    bk = run_bucketize(c, np.array([0, 0, 0]), 0.05, 64)
    assert bk.scan_bucket_start.cpu().numpy().tolist() == [0, 0, 0]
    assert (bk.offsets.cpu().numpy() == 0).all()
    rng = np.random.default_rng(20)
    c = wl.uniform_cube(rng, 3000, 2.0)
    check_bucketize(c, np.array([0, 0, 1000, 1000, 2500, 3000, 3000]), 0.05, 128)


def test_bucketize_many_uneven_scans():
    rng = np.random.default_rng(21)
    sizes = rng.integers(1, 5000, 70)
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = np.concatenate([wl.uniform_cube(rng, int(s), 3.0) + np.float32(10 * i) for i, s in enumerate(sizes)])
    for hash in HASHES:
        check_bucketize(c, bo, 0.04, 256, 4, hash, max_scan_points=5000)


@pytest.mark.parametrize("n_probes", [0, 1, 3])
def test_bucketize_fewer_probes(n_probes):
    rng = np.random.default_rng(22)
    c = wl.indoor_room(rng, 30000)
    check_bucketize(c, None, 0.02, 512, 4, "zorder_div", n_probes)
    check_bucketize(c, None, 0.02, 512, 4, "xor_div", n_probes)


def test_bucketize_coincident_points_and_overrides():
    c = np.full((5000, 3), 0.25, dtype=np.float32)          # everything overflows into recycle
    check_bucketize(c, None, 1.0, 64, 4, "xor_mod")
    rng = np.random.default_rng(23)
    c = wl.uniform_cube(rng, 50000, 4.0)
    check_bucketize(c, None, 0.02, 1024, 4, "zorder_div", div=777, probe_step=3)
    check_bucketize(c, None, 0.02, 1024, 2, "xor_div", div=5)
    check_bucketize(c, None, 0.02, 1024, 8, "zorder_mod")
    check_bucketize(c, None, 0.02, 16, 1, "zorder_div")      # 3125 buckets of 16 in one scan


def test_bucketize_at_the_bucket_limit():
    rng = np.random.default_rng(24)
    n = 8192 * 16 - 5
    c = wl.uniform_cube(rng, n, 4.0)
    check_bucketize(c, None, 0.02, 64, 4, "zorder_mod")      # K = 8192 buckets of 16


def test_bucketize_is_deterministic_and_reuses_workspace():
    w = wl.make_workload("indoor")
    p = f3d.make_params(w.voxel_size, w.bucket_cap)
    ws = torch.empty(f3d.workspace_bytes(w.n, 1, p), dtype=torch.uint8, device=DEV)
    cd = dev(w.coords)
    a = f3d.psh_bucketize(cd, None, p, ws)
    pa = a.perm.clone()
    ws.fill_(0xAB)                                            # stale workspace contents must not matter
    b = f3d.psh_bucketize(cd, None, p, ws)
    torch.cuda.synchronize()
    assert torch.equal(pa, b.perm)


def test_inconsistent_batch_offsets_are_flagged_not_faulted():
    rng = np.random.default_rng(25)
    c = wl.uniform_cube(rng, 1000, 2.0)
    for bo in ([0, 600, 400, 1000], [0, 500, 900], [5, 500, 1000]):
        bk = run_bucketize(c, np.array(bo), 0.05, 64)
        assert int(bk.scan_bucket_start[-1]) == -1
    bk = run_bucketize(c, np.array([0, 900, 1000]), 0.05, 64, max_scan_points=800)   # a scan above the stated bound
    assert int(bk.scan_bucket_start[-1]) == -1



# ----------------------------------------------------------------------------- rebalancing variants


def clustered_cloud(rng, n, offset=0.0):
    centres = rng.random((12, 3)) * 6.0
    return (centres[rng.integers(0, 12, n)] + rng.normal(0, 0.08, (n, 3)) + offset).astype(np.float32)


@pytest.mark.parametrize("schedule", ["general", "steps", "scans"])
@pytest.mark.parametrize("name,hash", [("tiny", "xor_mod"), ("indoor", "zorder_div"), ("lidar4", "xor_div"), ("lidar4", "zorder_mod")])
def test_bucketize_canonical_order_matches_oracle(name, hash, schedule):
    w = wl.make_workload(name)
    msp = int(np.diff(w.batch_offsets).max())
    check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, w.scope_buckets, hash, order="canonical",
                    schedule=schedule, max_scan_points=msp)


@pytest.mark.parametrize("n", [1, 2, 63, 255, 256, 257, 2047, 2048, 2049, 6145, 30011])
def test_bucketize_canonical_order_small_and_ragged_sizes(n):
    rng = np.random.default_rng(300 + n)
    c = clustered_cloud(rng, n)
    if n > 300:
        c[100:180] = c[100]                      # identical points: ties fall to the input index
        c[200:260, 1:] = c[200, 1:]              # equal y and z, different x
        c[5] = -c[5]                             # negative coordinates and a negative zero
        c[6, 0] = -0.0
    check_bucketize(c, None, 0.05, 128, 4, "zorder_div", order="canonical")


def test_bucketize_canonical_order_many_scans_with_empty_ones():
    rng = np.random.default_rng(31)
    sizes = [0, 700, 1, 0, 5000, 2048, 333, 0]
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = np.concatenate([clustered_cloud(rng, s, 3.0 * i) for i, s in enumerate(sizes)])
    for hash in HASHES:
        check_bucketize(c, bo, 0.05, 128, 4, hash, order="canonical")
    sizes = [37] * 300                           # more than 256 scans: the scan index takes two digits of the sort key
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = clustered_cloud(rng, int(bo[-1]))
    check_bucketize(c, bo, 0.05, 64, 4, "zorder_div", order="canonical")


@pytest.mark.parametrize("n,scans,cap", [(9000, 1, 4096), (9000, 1, 128), (30_000, 1, 512), (60_000, 1, 256), (120_000, 1, 1024), (150_000, 1, 512),
                                         (200_000, 1, 1024), (206_000, 1, 1024), (215_000, 1, 1024), (224_000, 1, 1024), (300_000, 1, 2048), (800_000, 8, 1024),
                                         (400_000, 20, 2048)])
def test_bucketize_steps_with_few_and_many_count_rows_per_thread(n, scans, cap):
    """One launch per step: a thread sums up to 4, 7, 10 or 12 count rows at a time, in one or several goes, and threads without a row do
    not join. From 1 to 13 rows a thread, more threads than rows and column groups from 2 to 147."""
    rng = np.random.default_rng(n + cap)
    bo = np.round(np.linspace(0, n, scans + 1)).astype(np.int32)
    c = (rng.random((n, 3)) * 12).astype(np.float32)
    c[::2] = (c[::2] * 0.1).astype(np.float32)
    check_bucketize(c, bo, 0.05, cap, 4, "zorder_div", max_scan_points=int(np.diff(bo).max()), schedule="steps")


@pytest.mark.parametrize("hash", ["zorder_div", "xor_div"])
@pytest.mark.parametrize("n_scans,points,cap", [(60, 20_000, 1024), (60, 40_000, 256), (300, 16_300, 64), (300, 5000, 64), (49, 1025, 128)])
def test_bucketize_scans_with_more_contenders_than_a_queue_holds(n_scans, points, cap, hash):
    """One workgroup per scan: the contenders of a probe step are queued in what LDS the counters of the buckets leave. Room for all
    of them, for 50 per wave (1019 buckets, two workgroups per compute unit) and sizes between; Z-order-div uses its table of codes
    with one workgroup per compute unit and not with two."""
    rng = np.random.default_rng(70 + n_scans)
    sizes = rng.integers(points * 9 // 10, points + 1, n_scans)
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = (rng.random((int(bo[-1]), 3)) * 20).astype(np.float32)
    c[::3] = (c[::3] * 0.05 + 3.0).astype(np.float32)      # a dense corner that overflows into its neighbours
    check_bucketize(c, bo, 0.05, cap, 4, hash, max_scan_points=int(sizes.max()), schedule="scans")


@pytest.mark.parametrize("n_scans", [2, 63, 64, 65, 511, 512, 513])
def test_bucketize_canonical_order_sorts_every_scan_by_itself(n_scans):
    """Tiles of the sort never reach over the end of a scan: scans of no, one and two tiles and one point around that, scans of more
    merges than the others, up to the number of scans that are still sorted one by one and beyond it; with the largest scan known
    and not. Codes of 3 bits to 63, and one of them beside coordinates that are no numbers (whose order itself is looked at below)."""
    rng = np.random.default_rng(60 + n_scans)
    sizes = rng.choice([0, 1, 7, 60], n_scans)
    for at, size in zip(rng.permutation(n_scans), (2048, 2049, 4096, 4097, 6145, 0)):
        sizes[at] = size
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = clustered_cloud(rng, int(bo[-1]))
    for voxel in (0.05, 1e-6, 1e3):
        check_bucketize(c, bo, voxel, 256, 4, "zorder_div", order="canonical", max_scan_points=int(sizes.max()))
    check_bucketize(c, bo, 0.05, 256, 4, "xor_mod", order="canonical")
    c[bo[np.argmax(sizes)] + 5] = np.nan
    got = run_bucketize(c, bo, 0.05, 256, order="canonical")
    assert np.array_equal(np.sort(got.perm.cpu().numpy()), np.arange(len(c)))


def canonical_order_of(c, voxel):
    """Places of a scan's points by (Z-order code, x, y, z, place), floats as ordered integers, a voxel that is no number as 0; and the codes."""
    u = c.view(np.uint32)
    o = np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint32)
    low = o.min(axis=0)
    mn = np.where(low >> 31, low ^ np.uint32(0x80000000), ~low).astype(np.uint32).view(np.float32)
    with np.errstate(invalid="ignore"):
        f = np.floor((c - mn) * (np.float32(1) / np.float32(voxel)))
    v = np.clip(np.nan_to_num(f, nan=0.0, posinf=2.0 ** 21, neginf=0.0), 0, 2 ** 21 - 1).astype(np.uint64)
    code = np.zeros(len(c), np.uint64)
    for axis in range(3):
        for bit in range(21):
            code |= ((v[:, axis] >> np.uint64(bit)) & np.uint64(1)) << np.uint64(3 * bit + axis)
    return np.lexsort((np.arange(len(c)), o[:, 2], o[:, 1], o[:, 0], code)), code


@pytest.mark.parametrize("more", [0, 510])
def test_bucketize_canonical_order_beside_coordinates_that_are_no_numbers(more):
    """The key holds as many bits of the code as the scan's largest needs, by the far corner of its box. A NaN there says nothing of the other
    points, one with its sign set is the box's minimum, infinities make a box of codes at the limit. One bucket holds the scan, so that its
    rows are the order itself. With 513 scans (`more`) the code has all its bits."""
    rng = np.random.default_rng(95)
    nan, minus_nan, inf = np.float32(np.nan), np.copysign(np.float32(np.nan), np.float32(-1)), np.float32(np.inf)
    special = [[(nan, 1, 1)], [(1, minus_nan, 1)], [(1, 1, inf)], [(-inf, 1, 1), (1, 1, nan)], [(nan, minus_nan, inf), (inf, nan, -inf)], []]
    if more:
        special = special[:3]
    scans = []
    for points in special:
        c = clustered_cloud(rng, 2500) * np.array([16, 1, 1], np.float32)
        for at, point in zip((5, 2100), points):
            c[at] = point
        scans.append(c)
    scans += [np.full((3, 3), nan, np.float32)] * 2 + [clustered_cloud(rng, 9)] * more
    bo = np.concatenate([[0], np.cumsum([len(c) for c in scans])]).astype(np.int32)
    assert len(scans) == (515 if more else 8)
    got = run_bucketize(np.concatenate(scans), bo, 0.05, 4 * 4096, hash="xor_mod", order="canonical").perm.cpu().numpy()
    for b, c in enumerate(scans):
        order, code = canonical_order_of(c, 0.05)
        assert np.array_equal(got[bo[b]:bo[b + 1]], bo[b] + order), b
    # without a word for the NaN, the first scan's code would have the bits of y and z only, and its order would be another
    order, code = canonical_order_of(scans[0], 0.05)
    y, z = (int((scans[0][:, axis].max() - scans[0][:, axis].min()) / 0.05).bit_length() for axis in (1, 2))
    bits = max(3 * y - 1, 3 * z)
    assert int(code.max()).bit_length() > bits
    assert not np.array_equal(np.argsort(code & np.uint64(2 ** bits - 1), kind="stable"), np.argsort(code, kind="stable"))


@pytest.mark.parametrize("sizes", [[768 * 2048], [768 * 2048 + 1], [3000, 768 * 2048 + 1, 1, 0, 50_000]])
def test_bucketize_canonical_order_of_scans_around_the_length_whose_boxes_are_joined_once(sizes):
    rng = np.random.default_rng(sizes[0])
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    c = (rng.random((int(bo[-1]), 3)) * 30 - 15).astype(np.float32)
    for b, size in enumerate(sizes):
        if size > 3000:      # the corners of the box in tiles far apart
            c[bo[b] + size - 2] = (-20 - b, 14, 3)
            c[bo[b] + 2500] = (3, -18 - b, 22)
    check_bucketize(c, bo, 0.05, 2048, 4, "zorder_div", order="canonical", max_scan_points=max(sizes))


@pytest.mark.parametrize("n_scans", [2, 64, 65])
def test_bucketize_canonical_order_in_a_workspace_of_another_batch(n_scans):
    """Every tile of the sort writes its place and its bounding box, or that there is no such tile, before either is read: in one workspace
    a batch of many tiles far away, one of bad offsets, one of few tiles, and bytes that are no boxes."""
    rng = np.random.default_rng(80 + n_scans)
    far = np.linspace(0, 40_000, n_scans + 1).astype(np.int32)
    near = np.zeros(n_scans + 1, np.int32)
    near[n_scans // 2 + 1:] = 3000
    near[-1] = 7001
    p = f3d.make_params(0.05, 256, order="canonical")
    ws = torch.empty(f3d.workspace_bytes(40_000, n_scans, p), dtype=torch.uint8, device="cuda")
    c = clustered_cloud(rng, 7001)
    ref = oracle.bucketize(c, near, 0.05, 64, "zorder_div", order="canonical")
    for before in ("far", "bad", 0, 255):
        if before == "far":
            f3d.psh_bucketize(dev(clustered_cloud(rng, 40_000, -90.0)), dev(far), p, workspace=ws)
        elif before == "bad":
            bad = f3d.psh_bucketize(dev(c), dev(near + 1), p, workspace=ws)
            assert int(bad.scan_bucket_start[-1]) == -1
        else:
            ws.fill_(before)
        got = f3d.psh_bucketize(dev(c), dev(near), p, workspace=ws)
        assert np.array_equal(got.perm.cpu().numpy(), ref["perm"]), before


@pytest.mark.parametrize("probe_mode", ["axes", "seeded"])
def test_bucketize_canonical_order_is_equivariant_to_input_order_on_the_gpu(probe_mode):
    rng = np.random.default_rng(32)
    n0, n1 = 30001, 17777
    c = np.concatenate([clustered_cloud(rng, n0), clustered_cloud(rng, n1, 3.0)])
    bo = np.array([0, n0, n0 + n1], dtype=np.int32)
    shuffle = np.concatenate([rng.permutation(n0), n0 + rng.permutation(n1)])
    c2 = c[shuffle]
    kw = dict(order="canonical", probe_mode=probe_mode, probe_seed=9)
    a = run_bucketize(c, bo, 0.05, 256, **kw)
    b = run_bucketize(c2, bo, 0.05, 256, **kw)
    pa, pb = a.perm.cpu().numpy(), b.perm.cpu().numpy()
    assert np.array_equal(c[pa], c2[pb])                                   # the same point in every row
    assert torch.equal(a.offsets, b.offsets)
    assert a.placed_per_round.cpu().numpy()[1:].sum() > 0.05 * (n0 + n1)    # overflow is common here
    a0 = run_bucketize(c, bo, 0.05, 256, probe_mode=probe_mode, probe_seed=9)
    b0 = run_bucketize(c2, bo, 0.05, 256, probe_mode=probe_mode, probe_seed=9)
    assert not np.array_equal(c[a0.perm.cpu().numpy()], c2[b0.perm.cpu().numpy()])


def test_bucketize_canonical_order_flags_bad_offsets_without_faulting():
    rng = np.random.default_rng(33)
    c = wl.uniform_cube(rng, 1000, 2.0)
    for bo in ([0, 600, 400, 1000], [0, 500, 900], [5, 500, 1000], [0, 5000, 1000]):
        bk = run_bucketize(c, np.array(bo), 0.05, 64, order="canonical")
        assert int(bk.scan_bucket_start[-1]) == -1


@pytest.mark.parametrize("schedule", ["general", "steps", "scans"])
@pytest.mark.parametrize("hash", HASHES)
def test_bucketize_probe_table_and_seeded_probes_match_oracle(hash, schedule):
    rng = np.random.default_rng(34)
    n0, n1 = 20000, 9001
    c = np.concatenate([clustered_cloud(rng, n0), clustered_cloud(rng, n1, 2.0)])
    bo = np.array([0, n0, n0 + n1], dtype=np.int32)
    table = rng.integers(-12, 13, (6, 3))
    kw = dict(schedule=schedule, max_scan_points=n0)
    _, ref = check_bucketize(c, bo, 0.05, 256, 4, hash, probe_mode="table", probe_table=table, **kw)
    assert ((ref["round_of"] > 0) & (ref["round_of"] < 7)).sum() > 100
    for seed in (0, 1, 0xFFFFFFFF):
        _, ref = check_bucketize(c, bo, 0.05, 256, 4, hash, probe_mode="seeded", probe_seed=seed, **kw)
        assert ((ref["round_of"] > 0) & (ref["round_of"] < 7)).sum() > 100
    check_bucketize(c, bo, 0.05, 256, 4, hash, n_probes=3, probe_mode="table", probe_table=table[:3], order="canonical", **kw)


def test_bucketize_variants_on_the_indoor_workload():
    w = wl.make_workload("indoor")
    check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, w.scope_buckets, "zorder_div",
                    order="canonical", probe_mode="seeded", probe_seed=2024)


# ----------------------------------------------------------------------------- attention


def attn_case(q, k, v, bk, ref_layout, heads, d, mode, use_perm, rows=None, shift=2, stride=2, scale=0.0, atol=ATOL):
    """Run the GPU attention and the oracle on the same layout; compare all rows or the sampled ones."""
    n = q.shape[0]
    # the output starts as NaN everywhere: a row that no workgroup wrote fails the finiteness check below
    out = torch.full((n, heads * d), float("nan"), dtype=torch.bfloat16, device=DEV)
    f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, heads, d, mode,
                         shift, stride, use_perm, scale, out)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    sel = None
    if rows is not None:
        sel = np.zeros(n, dtype=np.uint8)
        sel[rows] = 1
    ref = oracle.attn(q, k, v, ref_layout["perm"] if use_perm else None, ref_layout["offsets"],
                      ref_layout["scan_bucket_start"], bk.scope_buckets, mode, heads, d, shift, stride,
                      None if scale == 0.0 else scale, sel)
    mask = slice(None) if rows is None else rows
    err = np.abs(got[mask] - ref[mask])
    assert np.isfinite(got).all()
    assert err.max() <= atol, f"max-abs {err.max():.4g} (mean {err.mean():.3g})"
    return got, err.max()


def sample_rows(rng, ref_layout, n, count):
    """Random rows plus the first and last rows of every scan (edge scopes, ragged tails)."""
    rows = set(rng.integers(0, n, count).tolist())
    off, sbs = ref_layout["offsets"], ref_layout["scan_bucket_start"]
    for b in range(len(sbs) - 1):
        if sbs[b + 1] > sbs[b]:
            lo, hi = off[sbs[b]], off[sbs[b + 1]]
            rows.update(range(lo, min(lo + 3, hi)))
            rows.update(range(max(hi - 40, lo), hi))
    return np.array(sorted(rows))


def test_attention_tiny_workload_all_rows():
    w = wl.make_workload("tiny")
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    for mode in ("plain", "shift", "stride"):
        attn_case(q, k, v, bk, ref, w.heads, w.head_dim, mode, True)
    perm = ref["perm"]
    attn_case(q[perm], k[perm], v[perm], bk, ref, w.heads, w.head_dim, "shift", False)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name", ["lidar4", "wide", "lidar8"])
def test_attention_full_size_every_row(name):
    """Configurations 3, 4 and 5 in the launch configuration bench.py times: EVERY row of every distinct pass against the
    oracle (the oracle needs about 10-40 s per pass on the machine's host cores)."""
    w = wl.make_workload(name)
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    bucket_major = name == "lidar8"                      # that workload runs its layers on bucket-major features
    if bucket_major:
        q, k, v = q[ref["perm"]], k[ref["perm"]], v[ref["perm"]]
    for mode in dict.fromkeys(w.modes):
        print(f"{name} {mode}: all {w.n} rows", flush=True)
        attn_case(q, k, v, bk, ref, w.heads, w.head_dim, mode, not bucket_major)


def big_ragged_layout():
    """Four scans, 266 buckets of capacity 256 (scope 1024): full buckets mixed with short and one-row ones, scopes that
    end inside a 32-row tile, a scan of a single short bucket. Large enough (67 scopes and more per pass) for the launch
    to take two query tiles per wave with 8 heads."""
    pat = [256, 256, 37, 256, 1, 256, 256, 256, 50, 256, 200, 256, 131, 256, 256, 7]
    sizes = [(pat * 8)[:121], [17], [256] * 40 + [255, 256, 3, 256] * 11 + [90], [256, 129] * 30]
    return hand_layout(sizes, 1024, 4)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("d", [16, 32])
def test_attention_ragged_buckets_two_query_tiles_per_wave(d):
    # all rows, all three patterns, with and without the permutation, on a launch of several thousand workgroups
    heads = 8
    bk, ref, n = big_ragged_layout()
    assert f3d.attn_block_rows(bk, heads, d) == 256
    rng = np.random.default_rng(34 + d)
    q, k, v = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(3))
    for mode, kw in (("plain", {}), ("shift", {"shift": 1}), ("shift", {"shift": 2}), ("stride", {"stride": 2}),
                     ("stride", {"stride": 3})):
        attn_case(q, k, v, bk, ref, heads, d, mode, True, **kw)
        attn_case(q, k, v, bk, ref, heads, d, mode, False, **kw)


@pytest.mark.parametrize("name", ["indoor", "scope8k"])
def test_attention_full_size_sampled_rows(name):
    # the launch configuration bench.py times, on sampled query rows (each needs its whole scope in the oracle)
    w = wl.make_workload(name)
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    rng = np.random.default_rng(30)
    count = 1500 if w.channels <= 128 and w.bucket_cap <= 1024 else 400
    bucket_major = name == "lidar8"                      # that workload runs its layers on bucket-major features
    if bucket_major:
        q, k, v = q[ref["perm"]], k[ref["perm"]], v[ref["perm"]]
    for mode in dict.fromkeys(w.modes):
        rows = sample_rows(rng, ref, w.n, count)
        attn_case(q, k, v, bk, ref, w.heads, w.head_dim, mode, not bucket_major, rows)


def test_attention_indoor_plain_every_row():
    w = wl.make_workload("indoor")
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    attn_case(q, k, v, bk, ref, w.heads, w.head_dim, "plain", True)


def hand_layout(sizes_per_scan, cap, m):
    """A Buckets object over hand-made (ragged) bucket sizes, to exercise general offsets."""
    sizes = [s for scan in sizes_per_scan for s in scan]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    sbs = np.concatenate([[0], np.cumsum([len(s) for s in sizes_per_scan])]).astype(np.int32)
    n = int(off[-1])
    kmax = n // (cap // m) + len(sizes_per_scan)
    off_pad = np.full(max(kmax, len(sizes)) + 1, n, dtype=np.int32)
    off_pad[:len(off)] = off
    perm = np.random.default_rng(31).permutation(n).astype(np.int32)
    bk = f3d.Buckets(dev(perm), None, dev(off_pad), dev(sbs), None, n, len(sizes_per_scan), cap, m, len(sizes))
    return bk, {"perm": perm, "offsets": off, "scan_bucket_start": sbs}, n


@pytest.mark.parametrize("d,heads", [(16, 2), (32, 2), (16, 5), (32, 3)])
def test_attention_ragged_buckets_all_modes(d, heads):
    # buckets of uneven size (all <= S = 64), scopes that end inside a 32-row tile, three scans
    sizes = [[64, 64, 37, 64, 1, 64, 64, 64, 50], [17], [64, 64, 64, 64, 64, 3]]
    bk, ref, n = hand_layout(sizes, 256, 4)
    rng = np.random.default_rng(32)
    q, k, v = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(3))
    for mode, kw in (("plain", {}), ("shift", {"shift": 1}), ("shift", {"shift": 3}), ("stride", {"stride": 2}),
                     ("stride", {"stride": 3})):
        attn_case(q, k, v, bk, ref, heads, d, mode, True, **kw)
        attn_case(q, k, v, bk, ref, heads, d, mode, False, **kw)


def test_attention_other_scope_shapes_and_scale():
    rng = np.random.default_rng(33)
    for cap, m, sizes in ((32, 2, [[16] * 9 + [5]]), (512, 8, [[64] * 21 + [9]]), (2048, 1, [[2048, 2048, 700]]),
                          (1024, 16, [[64] * 40])):
        bk, ref, n = hand_layout(sizes, cap, m)
        q, k, v = (wl.f32_to_bf16_bits(rng.standard_normal((n, 32)).astype(np.float32)) for _ in range(3))
        modes = ["plain", "stride"] + (["shift"] if m > 1 else [])
        for mode in modes:
            attn_case(q, k, v, bk, ref, 2, 16, mode, True, shift=max(1, m // 2), scale=0.31)


def scope_search_layouts():
    """What the search for a workgroup's scope tells apart: scans up to 63 (a lane each), more (halving), one (no search), with scans
    that have no buckets; and runs without rows, as the first, the last and between others, in up to four runs and in more."""
    rng = np.random.default_rng(34)
    for n_scans in (63, 64, 65, 300):
        sizes = [list(rng.integers(1, 17, rng.choice([0, 0, 1, 3, 4, 7, 9]))) for _ in range(n_scans)]
        sizes[n_scans // 2] = [16] * 25
        if n_scans != 64:
            sizes[0], sizes[-1] = [], [5, 16]
        yield f"{n_scans} scans", sizes, 64, 4
    for m in (2, 3, 4, 8, 16):
        full = [[16 if (i + j) % 3 else 9 for i in range(m)] for j in range(5)]
        holes = ({0}, {m - 1}, set(range(1, m - 1)) or {0}, set(range(m - 1)), set(range(m)))
        one = [0 if i in hole else rows for scope, hole in zip(full, holes) for i, rows in enumerate(scope)]
        turned = [one[j * m + i] for i in range(m) for j in range(5)]      # the same holes for a stride of five
        yield f"runs of {m} without rows", [one + [0, 3]], 16 * m, m
        yield f"strided runs of {m} without rows", [turned, [0] * m, [4, 0] + turned + [0]], 16 * m, m


def short_scope_atol(v):
    """Scopes of a few rows give results as large as the values. A weight p_i is rounded to bfloat16 (relative 2^-9) above and below the
    fraction, which moves the result by at most 2^-9 sum p_i |v_i - o| <= 2^-8 max |v|; the result is rounded by 2^-9 max |v|."""
    return 3 * 2.0 ** -9 * float(np.abs(wl.bf16_bits_to_f32(v)).max())


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("case", range(14))
def test_attention_forward_and_backward_find_every_scope(case, d):
    name, sizes, cap, m = list(scope_search_layouts())[case]
    bk, ref, n = hand_layout(sizes, cap, m)
    rng = np.random.default_rng(35 + case)
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, 2 * d)).astype(np.float32)) for _ in range(4))
    for mode, kw in (("plain", {}), ("shift", {"shift": 1}), ("stride", {"stride": 2}), ("stride", {"stride": 5})):
        attn_case(q, k, v, bk, ref, 2, d, mode, True, atol=short_scope_atol(v), **kw)
        bwd_case(q, k, v, g, bk, ref, 2, d, mode, True, **kw)


@pytest.mark.parametrize("n_scans", [1, 3, 63, 64, 200])
def test_attention_on_a_flagged_layout_writes_nothing(n_scans):
    sizes = [[16, 16, 9]] * n_scans
    bk, ref, n = hand_layout(sizes, 64, 4)
    bk.scan_bucket_start[-1] = -1
    q = torch.ones(n, 32, dtype=torch.bfloat16, device=DEV)
    lse = torch.ones(n, 2, device=DEV)
    for mode in ("plain", "shift", "stride"):
        out = torch.full_like(q, 7.0)
        f3d.bucket_swin_attn(q, q, q, bk, 2, 16, mode, out=out, lse=lse)
        assert (out == 7.0).all() and (lse == 1.0).all(), mode


@pytest.mark.parametrize("sizes,cap,m,heads,max_buckets,mode,kw", [
    ([[1] * 69_000, [1] * 900], 256, 16, 1, 70_000, "stride", {"stride": 4095}),        # buckets by 16 x 4095: 65 520 x 70 000
    ([[1] * 40_000, [1] * 900], 64, 4, 1, 1_100_000, "stride", {"stride": 4095}),    # scopes by the stride: 4095 x 1 100 001
    ([[900, 70] * 5, [333]], 256_064, 4, 2, 10_000, "shift", {"shift": 3}),             # 5 or 10 million workgroups by 1001 or 2001 a scope
    ([[16, 3, 16] * 3, [8]], 64, 4, 4095, 1200, "plain", {}),                           # scopes by 4095 heads
])
def test_attention_where_dividends_are_too_large_for_a_product(sizes, cap, m, heads, max_buckets, mode, kw):
    """Quotients in the search for a scope are the upper half of a product where largest dividend times divisor is below 2^32; in each of
    these calls one of them is not. (The bound on the number of buckets is the caller's and may be far above what there is.)"""
    bk, ref, n = hand_layout(sizes, cap, m)
    offsets = torch.full((max_buckets + 1,), n, dtype=torch.int32, device=DEV)
    offsets[:len(ref["offsets"])] = dev(ref["offsets"])
    bk.offsets, bk.max_buckets = offsets, max_buckets
    rng = np.random.default_rng(36)
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, 16 * heads), dtype=np.float32)) for _ in range(4))
    attn_case(q, k, v, bk, ref, heads, 16, mode, True, atol=short_scope_atol(v), **kw)
    if n < 1000 and heads < 4095:
        bwd_case(q, k, v, g, bk, ref, heads, 16, mode, True, **kw)


def test_attention_large_logits_stay_finite():
    # peaked softmax: scores of order +-60 exercise the running-max rescaling
    bk, ref, n = hand_layout([[64] * 8], 256, 4)
    rng = np.random.default_rng(34)
    q, k, v = (wl.f32_to_bf16_bits((rng.standard_normal((n, 32)) * s).astype(np.float32)) for s in (8.0, 8.0, 1.0))
    attn_case(q, k, v, bk, ref, 2, 16, "plain", True)


@pytest.mark.parametrize("d", [16, 32])
def test_attention_every_score_far_below_zero(d):
    """All scores of a scope near -370 in log2 units (q = +8, k = -8 and a little noise): the sweep against the fixed
    reference underflows, the running-maximum sweep takes over, and its first tile meets a maximum below -128. The
    softmax is that of the small differences between the scores."""
    bk, ref, n = hand_layout([[2], [40], [64, 64, 3], [1]], 256, 4)
    rng = np.random.default_rng(37)
    heads = 2
    q = wl.f32_to_bf16_bits(np.full((n, heads * d), 8.0, np.float32))
    k = wl.f32_to_bf16_bits((-8.0 + 0.25 * rng.standard_normal((n, heads * d))).astype(np.float32))
    v = wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32))
    for mode in ("plain", "shift"):
        attn_case(q, k, v, bk, ref, heads, d, mode, True, scale=0.25)
    attn_case_f16(wl.bf16_bits_to_f32(q).astype(np.float16), wl.bf16_bits_to_f32(k).astype(np.float16),
                  wl.bf16_bits_to_f32(v).astype(np.float16), bk, ref, heads, d, "plain", True, scale=0.25)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("d", [16, 32])
def test_attention_running_maximum_sweep_on_two_query_tiles_per_wave(d):
    """The checked fallback (scores outside the window of the sweep against the fixed reference) on the large ragged
    layout, i.e. on the kernels that keep two query tiles per wave: q and k of standard deviation 4 give scores of
    +-100 and more in log2 units for some rows of nearly every scope; a second case has every score far below zero
    (first tile of the running-maximum sweep meets a maximum below -128). bf16 and binary16."""
    heads = 8
    bk, ref, n = big_ragged_layout()
    assert f3d.attn_block_rows(bk, heads, d) == 256
    rng = np.random.default_rng(44 + d)
    q, k = (wl.f32_to_bf16_bits((4.0 * rng.standard_normal((n, heads * d))).astype(np.float32)) for _ in range(2))
    v = wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32))
    # a softmax this peaked returns single V rows: the bound is the relative one of the large-values test below
    # (rounding of the output and of a dominating probability), 1.25 * 2^-8 * max|v|
    vmax = float(np.abs(wl.bf16_bits_to_f32(v)).max())
    peaked = 1.25 * 2.0 ** -8 * vmax
    attn_case(q, k, v, bk, ref, heads, d, "shift", True, atol=peaked)
    attn_case(q, k, v, bk, ref, heads, d, "stride", False, stride=3, atol=peaked)
    ql = wl.f32_to_bf16_bits(np.full((n, heads * d), 8.0, np.float32))
    kl = wl.f32_to_bf16_bits((-8.0 + 0.25 * rng.standard_normal((n, heads * d))).astype(np.float32))
    attn_case(ql, kl, v, bk, ref, heads, d, "plain", True, scale=0.25)
    attn_case_f16(wl.bf16_bits_to_f32(q).astype(np.float16), wl.bf16_bits_to_f32(k).astype(np.float16),
                  wl.bf16_bits_to_f32(v).astype(np.float16), bk, ref, heads, d, "shift", True,
                  atol=max(ATOL_F16, 1.25 * 2.0 ** -11 * vmax))


@pytest.mark.parametrize("d", [16, 32])
def test_attention_two_term_query_at_very_large_norms(d):
    """At head_dim 16 the scale is folded into q as two bf16 terms, so a scaled score is exact to about 2^-16 of
    sum_c |q_c k_c| scale (not of the score). The header states the size of the effect: with |q||k| scale near 10^4 single outputs move by a
    few 10^-2 where two top scores lie within a unit of each other, and the log-sum-exp by up to about 0.1. This pins
    that statement: outputs finite, within 0.06 of the oracle everywhere, within 1e-2 for all but a small share of the
    elements, lse within 2^-15 of sum_c |q_c||k_c| scale maximised over the scope, plus the 4e-3 of the probabilities'
    rounding; and the lse does leave the 4e-3, so the case shows the effect. At head_dim 32 the scale is a binary32
    multiply on the score: what is left is the binary32 accumulation of 32 products and that multiply, each rounding at
    most 2^-24 of the norm, 33 * 2^-24 norm < 2^-18.9 norm in lse in the worst case, and outputs are as close as
    everywhere (1e-2) up to a tenth for scores wrong by what such roundings add up to, about 2^-22 of the norm."""
    bk, ref, n = hand_layout([[64, 64, 64, 64, 64, 64, 64, 40]], 256, 4)
    rng = np.random.default_rng(45)
    heads = 2
    # common offsets make |q||k| large while the score differences stay moderate: q = 40 + N(0,1), k = 8 + N(0, 0.02)
    q = wl.f32_to_bf16_bits((40.0 + rng.standard_normal((n, heads * d))).astype(np.float32))
    k = wl.f32_to_bf16_bits((8.0 + 0.02 * rng.standard_normal((n, heads * d))).astype(np.float32))
    v = wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32))
    scale = 1.0
    qf, kf = wl.bf16_bits_to_f32(q).astype(np.float64), wl.bf16_bits_to_f32(k).astype(np.float64)
    norm = float((np.abs(qf[:, :d]).sum(axis=1).max()) * np.abs(kf[:, :d]).max() * scale)
    assert 5e3 < norm < 5e4                                   # the regime the header talks about
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, heads, d, "plain",
                               2, 2, True, scale, lse=lse)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    want = oracle.attn(q, k, v, ref["perm"], ref["offsets"], ref["scan_bucket_start"], 4, "plain", heads, d, 2, 2, scale)
    ref_b = oracle.attn_bwd(q, k, v, v, ref["perm"], ref["offsets"], ref["scan_bucket_start"], 4, "plain", heads, d, 2, 2, scale)
    err = np.abs(got - want)
    assert np.isfinite(got).all()
    lerr = np.abs(lse.cpu().numpy().astype(np.float64) - ref_b["lse"]).max()
    print(f"d {d} norm {norm:.5g}: max-abs {err.max():.4g}, lse error {lerr:.4g} = 2^{np.log2(lerr / norm):.1f} of the norm")
    if d == 16:
        assert err.max() <= 0.06, f"max-abs {err.max():.4g}"
        assert (err > 1e-2).mean() <= 0.02, f"share above 1e-2: {(err > 1e-2).mean():.4g}"
        assert 4e-3 < lerr <= 4e-3 + 2.0 ** -15 * norm, f"lse error {lerr:.4g} at norm {norm:.4g}"
    else:
        assert err.max() <= 1.1e-2, f"max-abs {err.max():.4g}"
        assert lerr <= 4e-3 + 2.0 ** -18.9 * norm, f"lse error {lerr:.4g} at norm {norm:.4g}"


@pytest.mark.parametrize("d", [16, 32])
def test_attention_products_beyond_binary32_with_finite_scores(d):
    """Only the scaled scores have to be finite. q and k times 2^63 and the scale times 2^-126 leave every score as it is,
    while most products q k^T pass the largest binary32. All factors are powers of two: output, log-sum-exp and
    gradients are those of the unscaled inputs, bit for bit up to the same powers of two."""
    heads = 4
    rng = np.random.default_rng(46)
    # short scopes, long ones with one and with two tiles per wave
    for sizes, rows in (([[64, 64, 64, 50, 64, 64, 9], [64, 3]], 128), ([[128] * 8 + [33]], 128), ([[128] * 32 + [17]] * 10, 256)):
        bk, ref, n = hand_layout(sizes, 4 * max(max(s) for s in sizes), 4)
        assert f3d.attn_block_rows(bk, heads, d) == rows
        q, k, v, g = (dev(wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)), torch.bfloat16) for _ in range(4))
        assert float((q[:64].float() @ k[:64].float().t()).abs().max()) * 2.0 ** 126 > 2.0 ** 128
        for mode in ("plain", "stride"):
            got = []
            for up, scale in ((1.0, 1.0), (2.0 ** 63, 2.0 ** -126)):
                lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
                out = f3d.bucket_swin_attn(q * up, k * up, v, bk, heads, d, mode, softmax_scale=scale, lse=lse)
                dq, dk, dv = f3d.bucket_swin_attn_bwd(q * up, k * up, v, out, g, lse, bk, heads, d, mode, softmax_scale=scale)
                got.append((out, lse, dq * up, dk * up, dv))
            for a, b in zip(*got):
                assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("d", [16, 32])
def test_attention_f16_finite_for_every_scale(d):
    # a softmax that has long saturated: the value of the key with the largest score, whatever finite scale comes on top
    bk, ref, n = hand_layout([[64, 64, 64, 50, 64, 64, 9], [64, 3]], 256, 4)
    rng = np.random.default_rng(47)
    q, k, v = (dev(rng.standard_normal((n, 2 * d)).astype(np.float16)) for _ in range(3))
    for size in (1.0, 2000.0):
        for mode in ("plain", "stride"):
            out = [f3d.bucket_swin_attn(q * size, k * size, v, bk, 2, d, mode, softmax_scale=s) for s in (1e20, 1e30, 3e38)]
            assert all(torch.isfinite(o).all() for o in out)
            if d == 32:
                assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


def test_attention_large_values_meet_the_relative_bound():
    """Values of magnitude up to about 12 and a peaked softmax (scale 1): outputs are then near single V rows and the
    absolute 1e-2 no longer covers the bf16 rounding of the output itself (2^-9 |o|), nor that of the probabilities
    (2^-9 relative each, worth up to 2^-9 max|v| when one key dominates). Bound: 1.25 * 2^-8 * max|v| element by element."""
    bk, ref, n = hand_layout([[64, 64, 64, 50, 64, 64, 9], [64, 3]], 256, 4)
    rng = np.random.default_rng(36)
    for d, heads in ((16, 3), (32, 2)):
        q, k, v = (wl.f32_to_bf16_bits((rng.standard_normal((n, heads * d)) * 3.0).astype(np.float32)) for _ in range(3))
        bound = 1.25 * 2.0 ** -8 * float(np.abs(wl.bf16_bits_to_f32(v)).max())
        for mode in ("plain", "shift", "stride"):
            out = f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, heads, d, mode,
                                       2, 2, True, 1.0)
            torch.cuda.synchronize()
            want = oracle.attn(q, k, v, ref["perm"], ref["offsets"], ref["scan_bucket_start"], 4, mode, heads, d, 2, 2, 1.0)
            got = out.float().cpu().numpy().astype(np.float64)
            assert np.isfinite(got).all()
            assert np.abs(got - want).max() <= bound
            assert np.abs(want).max() > 4.0   # the case is what it claims to be


def test_attention_closed_forms_on_gpu():
    bk, ref, n = hand_layout([[64] * 7 + [30]], 256, 4)
    rng = np.random.default_rng(35)
    q, k, v = (wl.f32_to_bf16_bits(rng.standard_normal((n, 64)).astype(np.float32)) for _ in range(3))
    const = np.tile(v[:1], (n, 1))
    out = f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(const, torch.bfloat16), bk, 4, 16, "shift")
    torch.cuda.synchronize()
    want = wl.bf16_bits_to_f32(const)
    assert np.abs(out.float().cpu().numpy() - want).max() <= 2.0 ** -7 * np.abs(want).max()


def test_attention_log_sum_exp_output():
    # natural-log sum of exponentials per row and head, bucket-major; also on scores large enough for the second sweep
    for d, heads, scale_in in ((16, 2, 1.0), (32, 2, 1.0), (16, 2, 8.0)):
        bk, ref, n = hand_layout([[64, 64, 37, 64, 1, 64, 64, 64, 50], [17]], 256, 4)
        rng = np.random.default_rng(36)
        q, k, v = (wl.f32_to_bf16_bits((rng.standard_normal((n, heads * d)) * s).astype(np.float32)) for s in (scale_in, scale_in, 1.0))
        for mode in ("plain", "shift", "stride"):
            lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
            f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, heads, d, mode, lse=lse)
            torch.cuda.synchronize()
            want = oracle.attn_bwd(q, k, v, v, ref["perm"], ref["offsets"], ref["scan_bucket_start"], 4, mode, heads, d)["lse"]
            # the denominator is a sum of probabilities rounded to bf16 (relative 2^-9 each): 4e-3 bounds the logarithm's error
            assert np.abs(lse.cpu().numpy() - want).max() <= 4e-3


# ----------------------------------------------------------------------------- attention on binary16 tensors

ATOL_F16 = 3e-3   # output rounding 2^-12*|o| (|o| < 4: 1e-3), probabilities rounded to binary16 (2^-12 each), fp32 sums


def attn_case_f16(q, k, v, bk, ref_layout, heads, d, mode, use_perm, rows=None, shift=2, stride=2, scale=0.0, atol=ATOL_F16,
                  original_order=False):
    """q, k, v: numpy float16 arrays. The binary16 entry point against the oracle fed with the same bit patterns."""
    n = q.shape[0]
    out = torch.full((n, heads * d), float("nan"), dtype=torch.float16, device=DEV)   # an unwritten row stays NaN
    f3d.bucket_swin_attn(dev(q), dev(k), dev(v), bk, heads, d, mode, shift, stride, use_perm, scale, out,
                         original_order=original_order)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    if original_order:
        got = got[ref_layout["perm"]]
    sel = None
    if rows is not None:
        sel = np.zeros(n, dtype=np.uint8)
        sel[rows] = 1
    ref = oracle.attn(q.view(np.uint16), k.view(np.uint16), v.view(np.uint16), ref_layout["perm"] if use_perm else None,
                      ref_layout["offsets"], ref_layout["scan_bucket_start"], bk.scope_buckets, mode, heads, d, shift, stride,
                      None if scale == 0.0 else scale, sel, fmt="f16")
    mask = slice(None) if rows is None else rows
    err = np.abs(got[mask] - ref[mask])
    assert np.isfinite(got).all()
    assert err.max() <= atol, f"max-abs {err.max():.4g} (mean {err.mean():.3g})"
    return err.max()


@pytest.mark.parametrize("d,heads", [(16, 2), (32, 2), (16, 5)])
def test_attention_f16_ragged_buckets_all_modes(d, heads):
    sizes = [[64, 64, 37, 64, 1, 64, 64, 64, 50], [17], [64, 64, 64, 64, 64, 3]]
    bk, ref, n = hand_layout(sizes, 256, 4)
    rng = np.random.default_rng(61)
    q, k, v = (rng.standard_normal((n, heads * d)).astype(np.float16) for _ in range(3))
    for mode, kw in (("plain", {}), ("shift", {"shift": 1}), ("shift", {"shift": 3}), ("stride", {"stride": 2}),
                     ("stride", {"stride": 3})):
        attn_case_f16(q, k, v, bk, ref, heads, d, mode, True, **kw)
        attn_case_f16(q, k, v, bk, ref, heads, d, mode, False, **kw)
    attn_case_f16(q, k, v, bk, ref, heads, d, "shift", True, original_order=True)   # the store in input order


@pytest.mark.timeout(600)
@pytest.mark.parametrize("d", [16, 32])
def test_attention_f16_ragged_buckets_two_query_tiles_per_wave(d):
    heads = 8
    bk, ref, n = big_ragged_layout()
    assert f3d.attn_block_rows(bk, heads, d) == 256
    rng = np.random.default_rng(64 + d)
    q, k, v = (rng.standard_normal((n, heads * d)).astype(np.float16) for _ in range(3))
    # (the oracle's binary16 decoder makes a pass cost 10-20 s here: one pass per pattern)
    attn_case_f16(q, k, v, bk, ref, heads, d, "plain", True)
    attn_case_f16(q, k, v, bk, ref, heads, d, "shift", False, shift=3)
    attn_case_f16(q, k, v, bk, ref, heads, d, "stride", True, original_order=True)


@pytest.mark.parametrize("name", ["tiny", "indoor", "lidar8"])
def test_attention_f16_on_workloads(name):
    w = wl.make_workload(name)
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    rng = np.random.default_rng(62)
    q, k, v = (rng.standard_normal((w.n, w.channels)).astype(np.float16) for _ in range(3))
    rows = None if name == "tiny" else sample_rows(rng, ref, w.n, 600 if w.channels <= 128 else 300)
    for mode in dict.fromkeys(w.modes):
        attn_case_f16(q, k, v, bk, ref, w.heads, w.head_dim, mode, True, rows)


def test_attention_f16_scores_outside_the_optimistic_window():
    """binary16 probabilities overflow at 2^16 and vanish below 2^-24: large positive scores, uniformly very negative
    scores and a mix of both must all end in the running-maximum sweep and stay within tolerance."""
    bk, ref, n = hand_layout([[64] * 8 + [20]], 256, 4)
    rng = np.random.default_rng(63)
    base = rng.standard_normal((n, 32))
    # peaked: scores of order +-60
    attn_case_f16((base * 8).astype(np.float16), (rng.standard_normal((n, 32)) * 8).astype(np.float16),
                  rng.standard_normal((n, 32)).astype(np.float16), bk, ref, 2, 16, "plain", True)
    # every score about -40 (natural-log units): all probabilities vanish against the fixed reference
    qn = np.full((n, 32), 2.0) + 0.05 * base
    kn = np.full((n, 32), -5.0) + 0.05 * rng.standard_normal((n, 32))
    attn_case_f16(qn.astype(np.float16), kn.astype(np.float16), rng.standard_normal((n, 32)).astype(np.float16), bk, ref, 2, 16,
                  "shift", True)
    # every score about +40: every probability overflows against the fixed reference
    attn_case_f16(qn.astype(np.float16), (-kn).astype(np.float16), rng.standard_normal((n, 32)).astype(np.float16), bk, ref, 2, 16,
                  "stride", True)
    # head_dim 32, where the denominator is summed on the vector unit
    q32 = (rng.standard_normal((n, 64)) * 6).astype(np.float16)
    k32 = (rng.standard_normal((n, 64)) * 6).astype(np.float16)
    attn_case_f16(q32, k32, rng.standard_normal((n, 64)).astype(np.float16), bk, ref, 2, 32, "plain", True)


def test_attention_f16_log_sum_exp_and_largest_finite_inputs():
    bk, ref, n = hand_layout([[64, 64, 37, 64, 1, 64, 64, 64, 50], [17]], 256, 4)
    rng = np.random.default_rng(64)
    q, k, v = (rng.standard_normal((n, 32)).astype(np.float16) for _ in range(3))
    lse = torch.empty(n, 2, dtype=torch.float32, device=DEV)
    f3d.bucket_swin_attn(dev(q), dev(k), dev(v), bk, 2, 16, "shift", lse=lse)
    torch.cuda.synchronize()
    # the oracle's log-sum-exp comes with its bf16 gradient routine; for binary16 it is written out here in numpy
    from test_oracle_attn import row_groups
    qf, kf = q.astype(np.float64), k.astype(np.float64)
    gid = row_groups(ref["offsets"], ref["scan_bucket_start"], 4, "shift")
    want = np.zeros((n, 2))
    for h in range(2):
        sl = slice(16 * h, 16 * h + 16)
        qs, ks = qf[ref["perm"]][:, sl], kf[ref["perm"]][:, sl]                  # bucket-major rows
        s = qs @ ks.T * 0.25
        s = np.where(gid[:, None] == gid[None, :], s, -np.inf)
        mx = s.max(axis=1)
        want[:, h] = mx + np.log(np.exp(s - mx[:, None]).sum(axis=1))
    assert np.abs(lse.cpu().numpy() - want).max() <= 2e-3
    # the largest finite values as values (the output is a convex combination: it must stay finite and close)
    vbig = np.where(rng.random((n, 32)) < 0.5, 65504.0, -65504.0).astype(np.float16)
    out = f3d.bucket_swin_attn(dev(q), dev(k), dev(vbig), bk, 2, 16, "plain")
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    want_o = oracle.attn(q.view(np.uint16), k.view(np.uint16), vbig.view(np.uint16), ref["perm"], ref["offsets"],
                         ref["scan_bucket_start"], 4, "plain", 2, 16, fmt="f16")
    assert np.isfinite(got).all()
    assert np.abs(got - want_o).max() <= 2.0 ** -9 * 65504.0


def test_whole_step_replays_from_a_hip_graph():
    """The calls launch kernels only (no memset nodes, no allocation, no host synchronisation), so a caller can capture
    bucketize + attention passes in a HIP graph. Every replay, with eager work and synchronisations in between, must
    reproduce the eager result bit for bit."""
    w = wl.make_workload("indoor")
    n, C = w.n, w.channels
    coords, bo = dev(w.coords), dev(w.batch_offsets)
    q, k, v = (dev(a, torch.bfloat16) for a in w.qkv())
    p = f3d.make_params(w.voxel_size, w.bucket_cap, order="canonical", probe_mode="seeded", probe_seed=3)
    ws = torch.empty(f3d.workspace_bytes(n, 1, p), dtype=torch.uint8, device=DEV)
    bk = f3d.psh_bucketize(coords, bo, p, ws)
    out, back = torch.empty_like(q), torch.empty_like(q)
    lse = torch.empty(n, w.heads, dtype=torch.float32, device=DEV)

    def step():
        f3d.psh_bucketize(coords, bo, p, ws, bk)
        f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, "plain", out=out, lse=lse)
        f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, "shift", out=back, original_order=True)

    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in (bk.perm, bk.inv_perm, bk.offsets, out, back, lse)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                      # warm-up on the capture stream's side
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    torch.cuda.synchronize()
    for it in range(4):
        for t in (bk.perm, bk.inv_perm, out, back, lse):
            t.zero_()                               # eager work between the replays; also proves the replay rewrites all
        ws.fill_(0x5A + it)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = (bk.perm, bk.inv_perm, bk.offsets, out, back, lse)
        for a, b in zip(got, want):
            assert torch.equal(a, b), f"replay {it} differs"


# ----------------------------------------------------------------------------- attention backward


def bwd_bounds(ref, q, k, v, g, out, lse, perm, heads, d, scale):
    """Worst-case bound on |GPU gradient - oracle.attn_bwd_saved| per element, from the kernel's designed roundings (u = 2^-8,
    the unit roundoff of bfloat16) and the magnitudes of the terms, first order in u:
      - the stored gradient is rounded once:                                   u |g|
      - P is recomputed as 2^(score - lse) with the scale folded into q (or k) as two bf16 terms (residual 2^-16 per
        component), lse*log2(e) and D carried as two bf16 terms each (residual 2^-16), everything else in fp32:
        relative error of P at most rho_ij = 1.25 * 2^-16 * scale * sum_c |q_ic||k_jc| + 2^-16 |lse_i| + 2^-19
      - dS = P (dP - D) is rounded to bf16 before dS K and dS^T Q, P before P^T dO:  u |dS_ij|,  u P_ij
      - D enters dS as P_ij * (2^-16 sum_c |dO_ic O_ic|); dP carries fp32 summation error 2^-21 sum_c |dO_ic||v_jc|
      - the products are accumulated in fp32 over the n_g rows of the scope:      n_g 2^-23 of the magnitudes.
    Sums of magnitudes, no cancellation assumed: holds for every input whose intermediate values stay finite in fp32."""
    u = 2.0 ** -8
    qf, kf, vf, gf = (wl.bf16_bits_to_f32(x).astype(np.float64) for x in (q, k, v, g))
    if perm is not None:
        qf, kf, vf = qf[perm], kf[perm], vf[perm]
    bound = {name: np.full(qf.shape, np.nan) for name in ("dq", "dk", "dv")}
    for rows, per_head in ref["scopes"]:
        ng = len(rows)
        acc = ng * 2.0 ** -23
        for h, im in enumerate(per_head):
            sl = slice(h * d, (h + 1) * d)
            Qa, Ka, Va, Ga = (np.abs(x[rows, sl]) for x in (qf, kf, vf, gf))
            P, dS = im["P"], np.abs(im["dS"])
            aD = (Ga * np.abs(out[rows, sl])).sum(axis=1)
            rho = 1.25 * 2.0 ** -16 * scale * (Qa @ Ka.T) + (2.0 ** -16 * np.abs(lse[rows, h]))[:, None] + 2.0 ** -19
            EdS = (u + rho + acc) * dS + P * (1.07 * 2.0 ** -16 * aD)[:, None] + P * (2.0 ** -21 * (Ga @ Va.T))
            EP = (u + rho + acc) * P
            bound["dq"][rows, sl] = u * np.abs(ref["dq"][rows, sl]) + (1 + u) * scale * (EdS @ Ka)
            bound["dk"][rows, sl] = u * np.abs(ref["dk"][rows, sl]) + (1 + u) * scale * (EdS.T @ Qa)
            bound["dv"][rows, sl] = u * np.abs(ref["dv"][rows, sl]) + (1 + u) * (EP.T @ Ga)
    return {name: 1.02 * b + 1e-30 for name, b in bound.items()}   # second-order terms


def bwd_case(q, k, v, g, bk, ref_layout, heads, d, mode, use_perm, scope_sel=None, shift=2, stride=2):
    """Forward (with log-sum-exp) and backward on the GPU. The backward call is a function of what the forward stored
    (D = rowsum(dO o O) from the stored bf16 output, P = exp(S - lse) from the stored log-sum-exp), so it is compared
    with oracle.attn_bwd_saved on those very arrays, element by element, within the worst-case bound of bwd_bounds.
    (tests/test_oracle_attn_bwd.py ties attn_bwd_saved to the plain gradient; the forward's out and lse are compared
    with the oracle by the forward tests.)"""
    n = q.shape[0]
    tq, tk, tv, tg = (dev(x, torch.bfloat16) for x in (q, k, v, g))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(tq, tk, tv, bk, heads, d, mode, shift, stride, use_perm, lse=lse)
    grads = f3d.bucket_swin_attn_bwd(tq, tk, tv, out, tg, lse, bk, heads, d, mode, shift, stride, use_perm)
    torch.cuda.synchronize()
    out64 = out.float().cpu().numpy().astype(np.float64)
    lse64 = lse.cpu().numpy().astype(np.float64)
    perm = ref_layout["perm"] if use_perm else None
    scale = 1.0 / np.sqrt(d)
    want = oracle.attn_bwd_saved(q, k, v, g, out64, lse64, perm, ref_layout["offsets"], ref_layout["scan_bucket_start"],
                                 bk.scope_buckets, mode, heads, d, shift, stride, scope_sel=scope_sel)
    bound = bwd_bounds(want, q, k, v, g, out64, lse64, perm, heads, d, scale)
    rows = want["done"].astype(bool)
    assert rows.any()
    worst = 0.0
    for name, got in zip(("dq", "dk", "dv"), grads):
        gg = got.float().cpu().numpy().astype(np.float64)
        assert np.isfinite(gg).all()
        err = np.abs(gg[rows] - want[name][rows])
        ratio = err / bound[name][rows]
        worst = max(worst, float(ratio.max()))
        assert (ratio <= 1.0).all(), (f"{name}: error up to {ratio.max():.3g} of the bound (max-abs {err.max():.4g}, "
                                      f"largest gradient {np.abs(want[name][rows]).max():.4g})")
    return grads


@pytest.mark.parametrize("d,heads", [(16, 2), (32, 2), (16, 5)])
def test_attention_backward_ragged_buckets_all_modes(d, heads):
    sizes = [[64, 64, 37, 64, 1, 64, 64, 64, 50], [17], [64, 64, 64, 64, 64, 3]]
    bk, ref, n = hand_layout(sizes, 256, 4)
    rng = np.random.default_rng(60)
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(4))
    for mode, kw in (("plain", {}), ("shift", {"shift": 1}), ("shift", {"shift": 3}), ("stride", {"stride": 2}), ("stride", {"stride": 3})):
        bwd_case(q, k, v, g, bk, ref, heads, d, mode, True, **kw)
        bwd_case(q, k, v, g, bk, ref, heads, d, mode, False, **kw)


def test_attention_backward_other_scope_shapes():
    rng = np.random.default_rng(61)
    for cap, m, sizes in ((32, 2, [[16] * 9 + [5]]), (512, 8, [[64] * 21 + [9]]), (2048, 1, [[2048, 700]]), (1024, 16, [[64] * 40])):
        bk, ref, n = hand_layout(sizes, cap, m)
        q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, 32)).astype(np.float32)) for _ in range(4))
        modes = ["plain", "stride"] + (["shift"] if m > 1 else [])
        for mode in modes:
            bwd_case(q, k, v, g, bk, ref, 2, 16, mode, True, shift=max(1, m // 2))


@pytest.mark.parametrize("name", ["indoor", "lidar8"])
def test_attention_backward_full_size_sampled_scopes(name):
    # the launch configuration the benchmark times; the oracle computes the scopes of a few sampled rows in full
    w = wl.make_workload(name)
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    rng = np.random.default_rng(62)
    g = wl.f32_to_bf16_bits(rng.standard_normal(q.shape).astype(np.float32))
    bucket_major = name == "lidar8"
    if bucket_major:
        q, k, v = q[ref["perm"]], k[ref["perm"]], v[ref["perm"]]
    for mode in dict.fromkeys(w.modes):
        sel = np.zeros(w.n, dtype=np.uint8)
        sel[[0, w.n // 2, w.n - 1]] = 1          # first, middle and last (ragged) scope
        bwd_case(q, k, v, g, bk, ref, w.heads, w.head_dim, mode, not bucket_major, scope_sel=sel)


@pytest.mark.parametrize("d,heads", [(16, 4), (32, 3)])
def test_attention_backward_two_tiles_per_wave_ragged(d, heads):
    # enough workgroups for two row tiles per wave, last buckets around the 32-row tile, 128-row stage and 256-row block:
    # scans of many scopes take two tiles, scans of one or two the form for short scopes
    tails = [1, 31, 32, 33, 64, 95, 96, 97, 127, 128]
    for scan, scans in ((32, 10), (2, 40)):
        sizes = [[128] * (scan + i % 4) + [tails[i % len(tails)]] for i in range(scans)]
        bk, ref, n = hand_layout(sizes, 512, 4)
        rng = np.random.default_rng(64)
        q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(4))
        sel = np.zeros(n, dtype=np.uint8)
        ends = np.cumsum([sum(x) for x in sizes])
        sel[ends[:10] - 1] = 1                       # the last scope of ten scans, and a whole one
        sel[0] = 1
        for mode in ("plain", "shift", "stride"):
            assert f3d.attn_block_rows(bk, heads, d, mode) == 256
            bwd_case(q, k, v, g, bk, ref, heads, d, mode, mode != "shift", scope_sel=sel)


def one_kernel_share(n, heads, run, size):
    """Share of the rows and heads whose gradients one kernel computes in run(workspace): only the two kernels keep D, the workspace's
    first n x heads words."""
    ws = torch.full((size,), 255, dtype=torch.uint8, device=DEV)
    run(ws)
    return float((ws[:n * heads * 4].view(torch.int32) == -1).float().mean())


def bwd_workspace_bytes(n, heads):
    size = ctypes.c_size_t(0)
    assert f3d.lib().f3d_attn_bwd_workspace_bytes(n, heads, ctypes.byref(size)) == 0
    return size.value


@pytest.mark.parametrize("d,heads,cap,m,scopes,tail,share", [
    (32, 4, 512, 4, 36, 33, 1),       # one pass of 512 keys, a last scope of two tiles
    (16, 5, 928, 1, 29, 545, 1),      # 29 tiles: the second pass begins in the middle of a stage; a last scope of 33 keys in its second pass
    (32, 3, 1024, 8, 50, 31, 1),      # strided scopes of eight runs, a last scope of one tile
    (16, 4, 1024, 4, 68, 700, 0.9),   # a round of tasks and a rest for the two kernels
    (32, 5, 2048, 4, 37, 1030, 1),    # the longest scopes: four passes, all of the LDS
])
def test_attention_backward_one_kernel(d, heads, cap, m, scopes, tail, share):
    # launches whose scopes are computed once for all gradients, and the same call with a workspace that has no room for that
    s = cap // m
    bk, ref, n = hand_layout([[s] * (m * scopes + tail // s) + ([tail % s] if tail % s else [])], cap, m)
    rng = np.random.default_rng(68)
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(4))
    sel = np.zeros(n, dtype=np.uint8)
    sel[[0, n // 2, n - 1]] = 1
    ws = torch.empty((n * heads * 4 + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    for mode in ("plain", "stride") if m == 1 else ("plain", "shift", "stride"):
        perm = mode != "shift"
        one = bwd_case(q, k, v, g, bk, ref, heads, d, mode, perm, scope_sel=sel)
        tq, tk, tv, tg = (dev(x, torch.bfloat16) for x in (q, k, v, g))
        lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
        out = f3d.bucket_swin_attn(tq, tk, tv, bk, heads, d, mode, use_perm=perm, lse=lse)

        def again(w):
            for a, b in zip(one, f3d.bucket_swin_attn_bwd(tq, tk, tv, out, tg, lse, bk, heads, d, mode, use_perm=perm, workspace=w)):
                assert torch.equal(a, b)

        assert abs(one_kernel_share(n, heads, again, bwd_workspace_bytes(n, heads)) - share) <= 0.03
        two = f3d.bucket_swin_attn_bwd(tq, tk, tv, out, tg, lse, bk, heads, d, mode, use_perm=perm, workspace=ws)
        for a, b in zip(one, two):
            # every row of both: P and dS are rounded to bf16 alike, so what differs is the order of binary32 sums and, at the edge of a
            # rounding, single terms by 2^-8 of themselves: a few times 2^-9 of the result's scale, and the stored rounding
            assert float((a.float() - b.float()).abs().max()) <= 2.0 ** -6 * float(b.float().abs().max())
            assert float((a.float() - b.float()).norm()) <= 2.0 ** -9 * float(b.float().norm())


@pytest.mark.parametrize("d,heads,cap,scopes,share", [
    (16, 4, 512, 100, 1),       # one pass
    (16, 4, 1024, 69, 0.9),     # two, and a rest for the two kernels
    (32, 3, 1024, 60, 1),
    (32, 5, 2048, 38, 1),       # four
])
def test_attention_backward_one_kernel_stores_elsewhere(d, heads, cap, scopes, share):
    # gradients in the input order of the points are the same rows, moved; one that takes the forward output's place is the same too (D is read
    # before anything is stored, and of a rest the two kernels read rows of other scopes or heads); at rows of another order the two kernels do all
    bk, _, n = hand_layout([[cap // 4] * (4 * scopes - 2) + [cap // 8 + 1]], cap, 4)
    rng = np.random.default_rng(69)
    q, k, v, g = (dev(wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)), torch.bfloat16) for _ in range(4))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    perm, size = bk.perm.data_ptr(), bwd_workspace_bytes(n, heads)
    for mode in ("plain", "stride"):
        out = f3d.bucket_swin_attn(q, k, v, bk, heads, d, mode, lse=lse)
        want = f3d.bucket_swin_attn_bwd(q, k, v, out, g, lse, bk, heads, d, mode)

        def moved(ws):
            for a, b in zip(want, f3d.bucket_swin_attn_bwd(q, k, v, out, g, lse, bk, heads, d, mode, original_order=True, workspace=ws)):
                assert torch.equal(f3d.unpermute(a, bk.perm), b)

        assert abs(one_kernel_share(n, heads, moved, size) - share) <= 0.03
        for which in range(3):
            for original_order in (False, True):
                def in_place(ws):
                    o = out.clone()
                    grads = [o if i == which else torch.empty_like(q) for i in range(3)]
                    rc = f3d.lib().f3d_bucket_swin_attn_bwd(
                        q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), g.data_ptr(), lse.data_ptr(), perm, bk.offsets.data_ptr(),
                        bk.scan_bucket_start.data_ptr(), n, bk.n_scans, bk.max_buckets, bk.bucket_cap, bk.scope_buckets, f3d.MODES[mode], 2, 2,
                        heads, d, 0.0, *(t.data_ptr() for t in grads), perm if original_order else None, ws.data_ptr(), ws.numel(),
                        torch.cuda.current_stream().cuda_stream)
                    assert rc == 0
                    for a, b in zip(grads, want):
                        if original_order:
                            b = f3d.unpermute(b, bk.perm)
                            assert float((a.float() - b.float()).abs().max()) <= 2.0 ** -6 * float(b.float().abs().max())
                            assert float((a.float() - b.float()).norm()) <= 2.0 ** -9 * float(b.float().norm())
                        else:
                            assert torch.equal(a, b)

                assert abs(one_kernel_share(n, heads, in_place, size) - (0 if original_order else share)) <= 0.03


@pytest.mark.parametrize("d,heads,share", [(16, 4, 0.86), (32, 3, 1)])
def test_attention_backward_one_kernel_batches(d, heads, share):
    # several scans of different length whose last scopes are short: sharp softmaxes, and q and k whose products pass the largest binary32
    # (see test_attention_products_beyond_binary32_with_finite_scores)
    sizes = [[256] * 260 + [1], [256] * 187 + [33], [256] * 110 + [188]]
    bk, ref, n = hand_layout(sizes, 1024, 4)
    rng = np.random.default_rng(70)
    q, k, v, g = (wl.f32_to_bf16_bits((rng.standard_normal((n, heads * d)) * s).astype(np.float32)) for s in (3.0, 3.0, 1.0, 1.0))
    sel = np.zeros(n, dtype=np.uint8)
    ends = np.cumsum([sum(x) for x in sizes])
    sel[ends - 1] = 1
    sel[ends[0]] = sel[ends[1] + 5000] = 1
    t = [dev(x, torch.bfloat16) for x in (q, k, v, g)]
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    for mode in ("plain", "shift", "stride"):
        grads = bwd_case(q, k, v, g, bk, ref, heads, d, mode, True, scope_sel=sel)
        out = f3d.bucket_swin_attn(*t[:3], bk, heads, d, mode, lse=lse)

        def again(ws):
            for a, b in zip(grads, f3d.bucket_swin_attn_bwd(*t[:3], out, t[3], lse, bk, heads, d, mode, workspace=ws)):
                assert torch.equal(a, b)

        assert abs(one_kernel_share(n, heads, again, bwd_workspace_bytes(n, heads)) - share) <= 0.03
        got = []
        for up, scale in ((0.25, 1.0), (2.0 ** 61, 2.0 ** -126)):   # no gradient so small that it would be flushed
            out = f3d.bucket_swin_attn(t[0] * up, t[1] * up, t[2], bk, heads, d, mode, softmax_scale=scale, lse=lse)
            dq, dk, dv = f3d.bucket_swin_attn_bwd(t[0] * up, t[1] * up, t[2], out, t[3], lse, bk, heads, d, mode, softmax_scale=scale)
            got.append((dq * up, dk * up, dv))
        for a, b in zip(*got):
            assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("d,heads,cap,tasks,share", [
    # tasks: scopes and spare scope slots times heads; faster, and taken, by
    (32, 8, 640, 408, 0),      # the two kernels: a second pass of 128 keys
    (16, 8, 1280, 408, 0),     # ... a third pass of 256 keys
    (16, 4, 2048, 192, 0),     # ... a round of four passes that is three quarters full
    (32, 4, 1536, 152, 0),
    (32, 8, 1024, 328, 0),     # ... at head_dim 32, a round and a rest of 72
    (32, 4, 1024, 928, 0),     # ... at head_dim 32, three rounds and a rest of 160
    (32, 8, 512, 600, 0),      # ... at head_dim 32, one pass, more than two rounds
    (32, 8, 512, 288, 0),      # ... one pass, a round and a rest
    (16, 8, 512, 264, 0),      # ... at head_dim 16 of less than 16
    (16, 8, 512, 328, 0),      # ... and of more than 64
    (16, 8, 512, 1720, 0),     # ... at head_dim 16, one pass, more than six rounds
    (16, 16, 512, 6128, 0),    # ... and up to 24
    (32, 8, 512, 480, 1),      # the one kernel: two rounds of one pass
    (16, 8, 512, 1000, 1),     # ... four rounds at head_dim 16
    (16, 8, 512, 272, 0.94),   # ... a round, the rest of 16 by the two
    (16, 8, 512, 320, 0.8),    # ... of 64
    (16, 16, 512, 6144, 1),    # ... 24 rounds
    (16, 8, 832, 216, 1),      # ... a second pass of 320 keys
    (16, 4, 2048, 200, 1),     # ... a round of four passes
    (32, 4, 1024, 936, 1),     # ... the fourth round with 168 tasks
    (32, 8, 1024, 320, 0.8),   # a round of them, the rest of 64 by the two
])
def test_attention_backward_kernels_by_size(d, heads, cap, tasks, share):
    bk, _, n = hand_layout([[cap // 4] * (4 * (tasks // heads - 3) - 1) + [5]], cap, 4)
    q, k, v, g = (torch.randn(n, heads * d, device=DEV).to(torch.bfloat16) for _ in range(4))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(q, k, v, bk, heads, d, "plain", lse=lse)
    got = one_kernel_share(n, heads, lambda ws: f3d.bucket_swin_attn_bwd(q, k, v, out, g, lse, bk, heads, d, "plain", workspace=ws),
                           n * heads * 4 + 512 + (64 << 20))
    assert abs(got - share) <= 0.03, got


@pytest.mark.parametrize("n,heads,cap,share", [(14700, 8, 1024, 1), (25000, 8, 1024, 1), (32500, 8, 1024, 0.94), (50000, 4, 1024, 1), (100000, 4, 2048, 1)])
def test_attention_backward_one_kernel_has_room_in_the_workspace_the_library_asks_for(n, heads, cap, share):
    # a round of tasks or less, head_dim 32: there are more workgroups, each with a strip of sums between its passes, than scopes
    bk, _, n = hand_layout([[cap // 4] * (4 * n // cap) + [n % (cap // 4)]], cap, 4)
    q, k, v, g = (torch.randn(n, heads * 32, device=DEV).to(torch.bfloat16) for _ in range(4))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(q, k, v, bk, heads, 32, "plain", lse=lse)
    got = one_kernel_share(n, heads, lambda ws: f3d.bucket_swin_attn_bwd(q, k, v, out, g, lse, bk, heads, 32, "plain", workspace=ws),
                           bwd_workspace_bytes(n, heads))
    assert abs(got - share) <= 0.03, got


@pytest.mark.parametrize("d,heads", [(16, 3), (32, 2)])
def test_attention_backward_short_and_long_scopes_one_tile_per_wave(d, heads):
    # the form for short scopes (an average below 448 rows) over one to four stages with last tiles of every kind, and
    # scopes of 512 rows in a launch too small for two tiles
    rng = np.random.default_rng(67)
    rows = [1, 31, 32, 33, 127, 128, 129, 160, 255, 257, 384, 385, 440, 512]
    scans = [[128] * (r // 128) + ([r % 128] if r % 128 else []) for r in rows]
    for sizes in (scans, [[128] * 8 + [97]]):
        bk, ref, n = hand_layout(sizes, 512, 4)
        q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(4))
        for mode in ("plain", "shift", "stride"):
            assert f3d.attn_block_rows(bk, heads, d, mode) == 128
            bwd_case(q, k, v, g, bk, ref, heads, d, mode, mode != "shift")


@pytest.mark.parametrize("d", [16, 32])
def test_attention_backward_gradient_in_place_of_the_output(d):
    # any of the three gradients may take the forward output's place, bucket-major or at permuted rows
    heads, rng = 3, np.random.default_rng(66)
    bk, ref, n = hand_layout([[64] * 9 + [40], [64] * 30 + [1]], 256, 4)
    q, k, v, g = (dev(wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)), torch.bfloat16) for _ in range(4))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(q, k, v, bk, heads, d, "plain", lse=lse)
    ws = torch.empty(n * heads * 4 + 256, dtype=torch.uint8, device=DEV)
    for original_order in (False, True):
        want = f3d.bucket_swin_attn_bwd(q, k, v, out, g, lse, bk, heads, d, "plain", original_order=original_order)
        for which in range(3):
            o = out.clone()
            grads = [o if i == which else torch.empty_like(q) for i in range(3)]
            perm = bk.perm.data_ptr()
            rc = f3d.lib().f3d_bucket_swin_attn_bwd(
                q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), g.data_ptr(), lse.data_ptr(), perm, bk.offsets.data_ptr(),
                bk.scan_bucket_start.data_ptr(), n, bk.n_scans, bk.max_buckets, bk.bucket_cap, bk.scope_buckets, 0, 2, 2, heads, d, 0.0,
                *(t.data_ptr() for t in grads), perm if original_order else None, ws.data_ptr(), ws.numel(),
                torch.cuda.current_stream().cuda_stream)
            assert rc == 0
            for a, b in zip(grads, want):
                # D may be summed in another order: binary32, far below the rounding of the gradients to bf16
                assert float((a.float() - b.float()).abs().max()) <= 2.0 ** -6 * float(b.float().abs().max())
                assert float((a != b).float().mean()) <= 0.01


def test_attention_backward_short_scopes_with_peaked_softmax():
    """Where a flat bound on the gradient error fails: scopes of a few dozen rows with a peaked softmax, in which the
    rounding of the stored output moves D by an amount common to all keys of a row. (a) 27218 points in four uneven
    scans, scopes of 128 rows, five heads of 16, every second bucket; (b) a single scope of 28 rows, large scores."""
    rng = np.random.default_rng(154)
    bo = np.array([0, 6622, 6696, 24799, 27218], dtype=np.int32)
    pts = np.concatenate([clustered_cloud(rng, int(bo[i + 1] - bo[i]), 3.0 * i) for i in range(4)]).astype(np.float32)
    bk, ref = check_bucketize(pts, bo, 0.02, 128, 4, "zorder_mod", 3, probe_mode="seeded", probe_seed=667689232)
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((27218, 80)).astype(np.float32)) for _ in range(4))
    bwd_case(q, k, v, g, bk, ref, 5, 16, "stride", True)
    bk, ref, n = hand_layout([[28]], 128, 4)
    q, k, v, g = (wl.f32_to_bf16_bits((rng.standard_normal((n, 32)) * s).astype(np.float32)) for s in (3.0, 3.0, 1.0, 1.0))
    for mode in ("plain", "stride"):
        bwd_case(q, k, v, g, bk, ref, 2, 16, mode, True)


def test_attention_backward_peaked_softmax_and_input_order():
    bk, ref, n = hand_layout([[64] * 8], 256, 4)
    rng = np.random.default_rng(63)
    q, k, v, g = (wl.f32_to_bf16_bits((rng.standard_normal((n, 32)) * s).astype(np.float32)) for s in (6.0, 6.0, 1.0, 1.0))
    dq, dk, dv = bwd_case(q, k, v, g, bk, ref, 2, 16, "plain", True)
    # gradients stored in the input order of the points: the same rows, moved by perm
    tq, tk, tv, tg = (dev(x, torch.bfloat16) for x in (q, k, v, g))
    lse = torch.empty(n, 2, dtype=torch.float32, device=DEV)
    out = f3d.bucket_swin_attn(tq, tk, tv, bk, 2, 16, "plain", lse=lse)
    eq, ek, ev = f3d.bucket_swin_attn_bwd(tq, tk, tv, out, tg, lse, bk, 2, 16, "plain", original_order=True)
    torch.cuda.synchronize()
    for a_, b_ in ((dq, eq), (dk, ek), (dv, ev)):
        assert torch.equal(f3d.unpermute(a_, bk.perm), b_)


# ----------------------------------------------------------------------------- unpermute, end to end


@pytest.mark.parametrize("cols,dtype", [(64, torch.bfloat16), (256, torch.bfloat16), (3, torch.float32), (10, torch.bfloat16)])
def test_unpermute_is_exact(cols, dtype):
    rng = np.random.default_rng(36)
    n = 10007
    perm = rng.permutation(n).astype(np.int32)
    src = torch.randn(n, cols, device=DEV).to(dtype)
    got = f3d.unpermute(src, dev(perm))
    torch.cuda.synchronize()
    want = torch.empty_like(src)
    want[dev(perm).long()] = src
    assert torch.equal(got, want)
    raw = src.cpu().view(torch.uint8).numpy().reshape(n, -1)
    assert np.array_equal(got.cpu().view(torch.uint8).numpy().reshape(n, -1), oracle.unpermute(raw, perm))


def test_end_to_end_original_order():
    # bucketize -> attention through perm -> unpermute equals the oracle's result in input order
    w = wl.make_workload("tiny")
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, hash="zorder_mod")
    q, k, v = w.qkv()
    out = f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, w.heads,
                               w.head_dim, "shift")
    back = f3d.unpermute(out, bk.perm)
    torch.cuda.synchronize()
    want = oracle.unpermute(oracle.attn(q, k, v, ref["perm"], ref["offsets"], ref["scan_bucket_start"], 4, "shift",
                                        w.heads, w.head_dim), ref["perm"])
    assert np.abs(back.float().cpu().numpy() - want).max() <= ATOL


@pytest.mark.parametrize("name,bucket_major", [("tiny", False), ("indoor", False), ("lidar8", True)])
def test_attention_stores_in_input_order_on_request(name, bucket_major):
    # the unpermute folded into the attention kernel's store is the same function as the separate kernel: bit for bit
    w = wl.make_workload(name)
    largest = int(np.diff(w.batch_offsets).max())
    bk = run_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, w.scope_buckets, max_scan_points=largest)
    q, k, v = (dev(x, torch.bfloat16) for x in w.qkv())
    if bucket_major:
        q, k, v = (x[bk.perm.long()].contiguous() for x in (q, k, v))
    for mode in dict.fromkeys(w.modes):
        two_step = f3d.unpermute(f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, mode, 2, 2, not bucket_major), bk.perm)
        fused = f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, mode, 2, 2, not bucket_major, original_order=True)
        torch.cuda.synchronize()
        assert torch.equal(fused, two_step)


# ----------------------------------------------------------------------------- in-bucket pooling


def bf16_ulp(x):
    """Spacing of bf16 at |x| (8 significant bits), with a floor for values near zero."""
    e = np.floor(np.log2(np.maximum(np.abs(x), 2.0 ** -20)))
    return 2.0 ** (e - 7)


def check_pool(coords_in, perm, feat_bm_bits, bo, tile, rho, voxel, hash="zorder_div", op="mean"):
    """GPU pooling against the oracle: the row -> pooled row map and the offsets bit for bit; min/max rows bit for
    bit; sum/mean rows within one bf16 spacing of the binary64 result (fp32 accumulation of at most rho terms can
    move a value across a rounding boundary, never further); positions to 1e-5 of the coordinate range."""
    n = feat_bm_bits.shape[0]
    coords_bm = coords_in if perm is None else coords_in[perm]
    ro = np.array([0, n], dtype=np.int32) if bo is None else bo.astype(np.int32)
    ref = oracle.pool_assign(coords_bm, ro, tile, rho, voxel, hash)
    want = oracle.pool_reduce(feat_bm_bits, ref["sub_of"], ref["n_out"], op, coords_bm)
    got = f3d.inbucket_pool(dev(coords_in), None if perm is None else dev(perm), dev(feat_bm_bits, torch.bfloat16),
                            None if bo is None else dev(bo.astype(np.int32)), tile, rho, voxel, hash, op)
    torch.cuda.synchronize()
    n_out = ref["n_out"]
    assert got.pooled_offsets.cpu().numpy().tolist() == ref["pooled_offsets"].tolist()
    assert np.array_equal(got.sub_of.cpu().numpy(), ref["sub_of"])
    g = got.feat[:n_out].float().cpu().numpy().astype(np.float64)
    w = wl.bf16_bits_to_f32(want["feat"]).astype(np.float64)
    if op in ("min", "max"):
        assert np.array_equal(got.feat[:n_out].view(torch.int16).cpu().numpy().view(np.uint16), want["feat"])
    else:
        assert (np.abs(g - w) <= bf16_ulp(w)).all(), f"max deviation {np.abs(g - w).max()}"
        assert (np.abs(g - w) > 0).mean() < 0.02           # and almost every value is the correctly rounded one
    span = float(np.abs(coords_bm).max()) if n else 1.0
    assert np.abs(got.coords[:n_out].cpu().numpy() - want["coords"]).max(initial=0.0) <= 1e-5 * span
    return ref


@pytest.mark.parametrize("hash", HASHES)
@pytest.mark.parametrize("rho,op", [(2, "mean"), (4, "max"), (3, "sum"), (8, "min")])
def test_pool_matches_oracle_on_the_indoor_layout(hash, rho, op):
    w = wl.make_workload("indoor")
    bk = run_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    perm = bk.perm.cpu().numpy()
    rng = np.random.default_rng(40)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((w.n, 64)).astype(np.float32))
    check_pool(w.coords, perm, feat, w.batch_offsets, 1024, rho, 0.1, hash, op)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("rho,op", [(2, "mean"), (5, "max")])
def test_pool_matches_oracle_on_the_largest_lidar_layout(rho, op):
    """893 tiles of 1024 rows: more tiles than resident workgroups, so every workgroup takes several tiles in turn and
    reuses its LDS and its list area; tiles of this layout leave about 480 rows to the rounds and need up to 400 of
    them, one row joining per round (the long walk along the sorted lists, chunk after chunk through the ring)."""
    w = wl.make_workload("lidar8")
    bk = run_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap, max_scan_points=int(np.diff(w.batch_offsets).max()))
    perm = bk.perm.cpu().numpy()
    rng = np.random.default_rng(47)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((w.n, 16)).astype(np.float32))
    ref = check_pool(w.coords, perm, feat, w.batch_offsets, 1024, rho, 0.1, "zorder_div", op)
    if rho == 2:
        assert ref["step_of"].max() >= 300


@pytest.mark.timeout(600)
def test_pool_more_tiles_than_compute_units_other_shapes():
    """More tiles than the GPU has compute units: the form of the kernel with two workgroups per compute unit, on
    tiles of 512 and 1000 rows, other capacities, hashes and reductions than the LiDAR test above, clustered input."""
    rng = np.random.default_rng(48)
    n = 330_000
    c = (rng.normal(size=(n, 3)) * 0.02 + rng.integers(0, 40, (n, 1)) * 1.5).astype(np.float32)   # 40 tight clusters on a line
    c[::5] = (rng.random((len(c[::5]), 3)) * 60).astype(np.float32)
    bo = np.array([0, 100_000, 100_000, 215_321, n], dtype=np.int32)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 8)).astype(np.float32))
    check_pool(c, None, feat, bo, 512, 3, 0.25, "xor_mod", "sum")
    check_pool(c, None, feat, bo, 1000, 2, 0.1, "zorder_mod", "min")
    check_pool(c, None, feat, bo, 1024, 16, 0.5, "xor_div", "mean")


def test_pool_on_scans_with_ragged_tiles_and_bucket_major_coordinates():
    rng = np.random.default_rng(41)
    sizes = [1, 1023, 1024, 1025, 0, 3000, 77, 0, 5]
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(bo[-1])
    c = np.concatenate([wl.uniform_cube(rng, s, 1.0 + i) + 10.0 * i for i, s in enumerate(sizes)]).astype(np.float32)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 32)).astype(np.float32))
    for tile, rho in ((1024, 2), (512, 4), (100, 3), (64, 1), (1000, 64)):
        check_pool(c, None, feat, bo, tile, rho, 0.05, "zorder_div", "mean")
        check_pool(c, None, feat, bo, tile, rho, 0.3, "xor_mod", "max")


def test_pool_dense_clusters_need_many_rounds():
    # almost all points in two tight clusters: most rows overflow their hash value and take several rounds
    rng = np.random.default_rng(42)
    n = 4096
    c = (rng.normal(size=(n, 3)) * 0.01).astype(np.float32)
    c[::2] += 5.0
    c[:50] = rng.random((50, 3)).astype(np.float32) * 10
    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 16)).astype(np.float32))
    ref = check_pool(c, None, feat, None, 1024, 2, 0.5, "zorder_div", "mean")
    assert ref["step_of"].max() >= 6
    check_pool(c, None, feat, None, 1024, 4, 0.5, "xor_div", "sum")


def test_pool_near_ties_on_a_lattice():
    """Points on a lattice of pitch 0.1 (not a binary fraction): very many candidate sub-buckets lie at distances that
    are equal in exact arithmetic and differ, if at all, in the last bit of the binary32 evaluation. The choice then
    depends on every product and sum being rounded on its own, in the stated order (a fused multiply-add rounds
    differently), and on the tie rule."""
    rng = np.random.default_rng(45)
    n = 6000
    ijk = rng.integers(0, 14, (n, 3))
    c = (ijk * 0.1).astype(np.float32) + np.float32(0.37)
    c[::7] += (rng.integers(-1, 2, (len(c[::7]), 3)) * np.float32(1e-7)).astype(np.float32)   # and a few one-ulp shifts
    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 16)).astype(np.float32))
    for rho, hash in ((2, "zorder_div"), (3, "xor_mod"), (4, "zorder_mod")):
        ref = check_pool(c, None, feat, None, 1024, rho, 0.25, hash, "max")
        assert ref["step_of"].max() >= 3


@pytest.mark.parametrize("spread", [0.0, 1e-7, 3e-6, 1e-4, 3e-3])
def test_pool_candidates_at_nearly_equal_distances(spread):
    """Many rows at one point, the centre of a shell of points: when these rows run out of sub-buckets of
    their own, every sub-bucket on the shell is a candidate at almost the same distance (relative differences of
    `spread`: exactly equal, in the last bits of binary32, in the bits a shortened sort key drops, and well apart).
    The order of a row's choices, and with it every later round, hangs on the full (distance, id) comparison."""
    rng = np.random.default_rng(46)
    for tile_rows, rho in ((1024, 2), (1024, 3), (600, 2)):
        n = 3 * tile_rows + 17
        c = np.zeros((n, 3), np.float32)
        for t0 in range(0, n, tile_rows):
            m = min(tile_rows, n - t0)
            shell = (3 * m) // 5   # the shell's rows come first and found the sub-buckets; the cluster's rows are left over
            u = rng.normal(size=(shell, 3))
            u /= np.linalg.norm(u, axis=1, keepdims=True)
            radius = 3.0 * (1.0 + spread * rng.random((shell, 1)))
            pts = np.concatenate([u * radius, np.zeros((m - shell, 3))])   # the cluster: one point, many times
            c[t0:t0 + m] = (pts + np.array([7.0, -2.0, 1.5])).astype(np.float32)
        feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 16)).astype(np.float32))
        ref = check_pool(c, None, feat, None, tile_rows, rho, 0.2, "zorder_div", "mean")
        assert ref["step_of"].max() >= 100   # the cluster's rows take the shell's sub-buckets one round at a time


@pytest.mark.parametrize("octaves", [10, 30, 60])
def test_pool_candidates_over_many_octaves_of_distance(octaves):
    """As above with the shell's radii spread over a range of 2^octaves around the cluster: the shortened sort keys hold sixteen
    octaves of squared distance, everything nearer is one value to them. Scans of one to many tiles."""
    rng = np.random.default_rng(47)
    sizes = [1024, 5000, 1, 0, 700, 2048]
    parts = []
    for n in sizes:
        for t0 in range(0, n, 1024):
            m = min(1024, n - t0)
            shell = (3 * m) // 5
            u = rng.normal(size=(shell, 3))
            u /= np.linalg.norm(u, axis=1, keepdims=True) if shell else 1.0
            parts.append(np.concatenate([u * 1000.0 * 2.0 ** (-0.5 * octaves * rng.random((shell, 1))), np.zeros((m - shell, 3))]))
    c = np.concatenate(parts).astype(np.float32)
    bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((len(c), 16)).astype(np.float32))
    for rho, voxel in ((2, 50.0), (3, 0.01)):
        check_pool(c, None, feat, bo, 1024, rho, voxel, "zorder_div", "max")


@pytest.mark.parametrize("at", [0, 1023, 1024, 2500])
def test_pool_many_short_scans_around_a_long_one(at):
    """The tile table is written 1024 scans at a time: those of short scans (at most four tiles) by the scan's own thread, those
    beside a longer one by all threads. 2600 scans, some empty, one of 5 or 9 tiles at the ends and edges of the 1024."""
    rng = np.random.default_rng(48)
    for long in (5 * 64, 4 * 64 + 1, 4 * 64, 9 * 64 - 1):
        sizes = rng.integers(0, 9, 2600)
        sizes[at] = long
        bo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
        c = rng.random((int(bo[-1]), 3)).astype(np.float32)
        feat = wl.f32_to_bf16_bits(rng.standard_normal((len(c), 8)).astype(np.float32))
        check_pool(c, None, feat, bo, 64, 2, 0.1, "zorder_div", "max")


@pytest.mark.parametrize("tiles", [3, 300])
@pytest.mark.parametrize("tile", [66, 130, 134, 262, 518, 1022, 1024])
def test_pool_pairs_where_most_rows_are_left_to_the_rounds(tile, tiles):
    """Capacity 2, half of every tile one point, the rest spread out: about half of the tile's rows are left to the rounds and a few
    join in each. Around 64 rows left one wave goes on alone, around 130 (few tiles: one workgroup per compute unit, more LDS) or
    more the lists that remain move to LDS."""
    rng = np.random.default_rng(50 + tile)
    n = tiles * tile - 3
    c = (rng.random((n, 3)) * 8).astype(np.float32)
    c[(np.arange(n) % tile) % 2 == 1] = 4.0
    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, 8)).astype(np.float32))
    ref = check_pool(c, None, feat, None, tile, 2, 0.01, "zorder_div", "max")
    assert ref["step_of"].max() >= 10


def test_pool_empty_input_and_bad_offsets():
    z = np.zeros((0, 3), np.float32)
    got = f3d.inbucket_pool(dev(z), None, dev(np.zeros((0, 8), np.uint16), torch.bfloat16), None, 1024, 2, 0.1)
    torch.cuda.synchronize()
    assert got.pooled_offsets.cpu().numpy().tolist() == [0, 0]
    rng = np.random.default_rng(43)
    c = rng.random((1000, 3)).astype(np.float32)
    feat = wl.f32_to_bf16_bits(rng.standard_normal((1000, 8)).astype(np.float32))
    for bo in ([0, 600, 400, 1000], [0, 500, 900], [5, 500, 1000]):
        got = f3d.inbucket_pool(dev(c), None, dev(feat, torch.bfloat16), dev(np.array(bo, dtype=np.int32)), 256, 2, 0.1)
        torch.cuda.synchronize()
        assert int(got.pooled_offsets[-1]) == -1


def test_pool_after_attention_end_to_end():
    # bucketize -> attention (bucket-major output) -> pooling of that output: the stage's three operators in a row
    w = wl.make_workload("tiny")
    bk, ref = check_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = w.qkv()
    out = f3d.bucket_swin_attn(dev(q, torch.bfloat16), dev(k, torch.bfloat16), dev(v, torch.bfloat16), bk, w.heads, w.head_dim, "plain")
    torch.cuda.synchronize()
    feat_bits = out.view(torch.int16).cpu().numpy().view(np.uint16)
    check_pool(w.coords, ref["perm"], feat_bits, w.batch_offsets, 128, 2, 0.1, "zorder_div", "mean")


# ----------------------------------------------------------------------------- LayerNorm + linear (block glue)


def check_ln_linear(n, c_in, c_out, n_outs, rng, ln=True, with_bias=True, with_res=False, gather=False, scatter=False,
                    statistical=True):
    """GPU against the binary64 oracle, which is the plain definition with no intermediate rounding. Bound per element:
    2^-8 |y| for the final bf16 rounding, plus what the kernel's own arithmetic adds before it.
    With LayerNorm the kernel rounds the normalised row to bf16 (the matrix core's operand): c_in terms of size
    |ln_c w_c| with independent relative errors of up to 2^-9 give a standard deviation of about 2^-9 |ln| |w| / sqrt(3)
    ~ 1.4e-3 for rows of norm 1.2 sqrt(c_in) and weight rows of norm 1 as generated here; 0.012 allows eight of those
    (a statistical allowance, left out with statistical=False where tens of millions of elements would hold rows of larger
    norm; the worst case, 2^-8 sum |ln_c w_c| ~ 0.04, is always asserted).
    Without LayerNorm the operands are the stored bf16 values themselves, so only the binary32 accumulation is left:
    c_in 2^-24 sum |x_c w_c| in the worst case."""
    x = wl.f32_to_bf16_bits((rng.standard_normal((n, c_in)) * 2 + 0.5).astype(np.float32))
    w = wl.f32_to_bf16_bits((rng.standard_normal((c_out, c_in)) / np.sqrt(c_in)).astype(np.float32))
    gamma = (1 + 0.2 * rng.standard_normal(c_in)).astype(np.float32) if ln else None
    beta = (0.1 * rng.standard_normal(c_in)).astype(np.float32) if ln else None
    bias = rng.standard_normal(c_out).astype(np.float32) if with_bias else None
    res = wl.f32_to_bf16_bits(rng.standard_normal((n, c_out)).astype(np.float32)) if with_res else None
    row_in = rng.permutation(n).astype(np.int32) if gather else None
    row_out = rng.permutation(n).astype(np.int32) if scatter else None
    want = oracle.ln_linear(x, w, bias, gamma, beta, 1e-5, row_in, res, row_out)
    t = lambda a, dt=None: None if a is None else dev(a, dt)
    outs = f3d.ln_linear(t(x, torch.bfloat16), t(w, torch.bfloat16), t(bias), t(gamma), t(beta), 1e-5, t(row_in),
                         t(res, torch.bfloat16), t(row_out), n_outs)
    torch.cuda.synchronize()
    got = np.concatenate([o.float().cpu().numpy() for o in outs], axis=1).astype(np.float64)
    assert np.isfinite(got).all()
    xs = wl.bf16_bits_to_f32(x).astype(np.float64)
    xs = xs if row_in is None else xs[row_in]
    if ln:
        xs = (xs - xs.mean(1, keepdims=True)) / np.sqrt(xs.var(1, keepdims=True) + 1e-5) * gamma + beta
    mag = np.abs(xs) @ np.abs(wl.bf16_bits_to_f32(w).astype(np.float64)).T        # sum_c |operand_c w_c| per output element
    if row_out is not None:
        full = np.zeros_like(mag); full[row_out] = mag; mag = full
    err = np.abs(got - want)
    if ln:
        assert not statistical or (err <= 2.0 ** -8 * np.abs(want) + 0.012).all(), f"max excess {(err - 2.0 ** -8 * np.abs(want) - 0.012).max():.4g}"
        worst = 2.0 ** -8 * np.abs(want) * 1.01 + (2.0 ** -8 + c_in * 2.0 ** -23) * mag + 1e-6
    else:
        worst = 2.0 ** -8 * np.abs(want) * 1.01 + c_in * 2.0 ** -23 * mag + 1e-6
    assert (err <= worst).all(), f"worst-case bound exceeded by {(err - worst).max():.4g}"
    assert np.abs(got - want).mean() <= 4e-3


@pytest.mark.parametrize("c_in,c_out,n_outs", [(64, 192, 3), (128, 384, 3), (256, 768, 3), (64, 64, 1), (256, 256, 1), (128, 512, 1)])
def test_ln_linear_matches_oracle(c_in, c_out, n_outs):
    rng = np.random.default_rng(80 + c_in)
    check_ln_linear(1000, c_in, c_out, n_outs, rng, ln=True, gather=True)                                  # q, k, v in bucket-major order
    check_ln_linear(777, c_in, c_out, n_outs, rng, ln=False, with_res=True, scatter=True)                   # output projection + residual, back in input order
    check_ln_linear(129, c_in, c_out, n_outs, rng, ln=True, with_bias=False, with_res=True, gather=True, scatter=True)


@pytest.mark.parametrize("c_in,c_out,n_outs", [(64, 64, 4), (64, 192, 4), (128, 64, 1), (128, 384, 3), (256, 768, 3), (256, 320, 4)])
def test_ln_linear_row_and_column_splits(c_in, c_out, n_outs):
    # rows: last waves with 1, 24, 25 and 32 rows (stores left out or not), waves without rows; columns split over the
    # grid (few rows) and not (512 workgroups and more); output tensors of 16, 48, 64 and 80 columns
    rng = np.random.default_rng(82)
    for n in (1, 24, 25, 33, 97, 121, 152, 2049):
        check_ln_linear(n, c_in, c_out, n_outs, rng, ln=True, gather=True)
        check_ln_linear(n, c_in, c_out, n_outs, rng, ln=False, with_res=True, scatter=True)
    check_ln_linear(65536 + 25, c_in, c_out, n_outs, rng, ln=False, with_res=True, gather=True, scatter=True)
    check_ln_linear(65536 + 25, c_in, c_out, n_outs, rng, ln=True, gather=True, statistical=False)


@pytest.mark.parametrize("c", [64, 128, 256])
def test_ln_linear_stored_through_and_past_the_caches(c):
    # results of 4 MB (and more) are stored past the caches: the last size below and the first one at it, both forms of the store
    rng = np.random.default_rng(600 + c)
    for c_out, n_outs, ln in ((3 * c, 3, True), (c, 1, False)):
        edge = -(-(4 << 20) // (2 * c_out))
        for n in (edge - 1, edge):
            check_ln_linear(n, c, c_out, n_outs, rng, ln=ln, with_res=not ln, gather=ln, scatter=not ln)


@pytest.mark.parametrize("c_out,n_outs", [(3648, 3), (4096, 1), (4096, 4)])
@pytest.mark.parametrize("c_in", [64, 128, 256])
def test_ln_linear_most_output_columns(c_in, c_out, n_outs):
    # the bias and the column table take the workgroup's LDS past 64 KB at 128 and 256 inputs from 3648 columns on
    rng = np.random.default_rng(84)
    check_ln_linear(200, c_in, c_out, n_outs, rng, ln=True, gather=True)
    check_ln_linear(33, c_in, c_out, n_outs, rng, ln=False, with_res=True, scatter=True)


@pytest.mark.parametrize("c", [64, 128, 256])
def test_ln_linear_in_place(c):
    # x as output, with the residual too and through one row map: a row's whole input is read before any of it is
    # overwritten, also at the sizes whose columns several workgroups would share
    rng = np.random.default_rng(83)
    w = dev(wl.f32_to_bf16_bits(rng.standard_normal((c, c)).astype(np.float32) / c ** 0.5), torch.bfloat16)
    gamma = dev(1 + 0.1 * rng.standard_normal(c).astype(np.float32))
    for n in (1, 129, 1500, 9000, 32768, 66000):
        x = dev(wl.f32_to_bf16_bits(rng.standard_normal((n, c)).astype(np.float32)), torch.bfloat16)
        rows = dev(rng.permutation(n).astype(np.int32))
        for rmap in (None, rows):
            for res in (None, x):
                for g in (None, gamma):
                    (want,) = f3d.ln_linear(x, w, None, g, None, 1e-5, rmap, res, rmap)
                    y = x.clone()
                    at, ptr = y.data_ptr(), lambda t: None if t is None else t.data_ptr()
                    rc = f3d.lib().f3d_ln_linear(at, ptr(rmap), ptr(g), None, 1e-5, w.data_ptr(), None, None if res is None else at, n, c, c,
                                                 (f3d.ctypes.c_void_p * 1)(at), 1, ptr(rmap), torch.cuda.current_stream().cuda_stream)
                    assert rc == 0
                    assert torch.equal(y, want), (n, rmap is None, res is None, g is None)


def test_ln_linear_edge_sizes_and_block_composition():
    rng = np.random.default_rng(81)
    for n in (1, 127, 128, 129, 4096):
        check_ln_linear(n, 64, 192, 3, rng, gather=True)
    # empty input
    outs = f3d.ln_linear(torch.empty(0, 64, dtype=torch.bfloat16, device=DEV), dev(np.zeros((64, 64), np.uint16), torch.bfloat16))
    assert outs[0].shape == (0, 64)
    # the first half of a block on the tiny workload: q, k, v written bucket-major feed the attention without a gather
    w_ = wl.make_workload("tiny")
    bk, ref = check_bucketize(w_.coords, w_.batch_offsets, w_.voxel_size, w_.bucket_cap)
    C = w_.channels
    feat = wl.f32_to_bf16_bits(rng.standard_normal((w_.n, C)).astype(np.float32))
    wq = wl.f32_to_bf16_bits((rng.standard_normal((3 * C, C)) / np.sqrt(C)).astype(np.float32))
    gamma, beta = np.ones(C, np.float32), np.zeros(C, np.float32)
    q, k, v = f3d.ln_linear(dev(feat, torch.bfloat16), dev(wq, torch.bfloat16), None, dev(gamma), dev(beta), 1e-5, bk.perm, n_outs=3)
    out = f3d.bucket_swin_attn(q, k, v, bk, w_.heads, w_.head_dim, "shift", use_perm=False)
    torch.cuda.synchronize()
    bits = lambda t_: t_.view(torch.int16).cpu().numpy().view(np.uint16)
    want = oracle.attn(bits(q), bits(k), bits(v), None, ref["offsets"], ref["scan_bucket_start"], 4, "shift", w_.heads, w_.head_dim)
    assert np.abs(out.float().cpu().numpy() - want).max() <= ATOL


# ----------------------------------------------------------------------------- random configurations


def random_cloud(rng, n, kind):
    if kind == 0:
        return (rng.random((n, 3)) * rng.uniform(0.5, 30)).astype(np.float32)
    if kind == 1:
        return clustered_cloud(rng, n)
    if kind == 2:   # a lattice: many coincident points
        return (rng.integers(0, rng.integers(2, 40), (n, 3)) * 0.1).astype(np.float32)
    if kind == 3:   # far from the origin: the spacing of binary32 exceeds small voxels
        return (rng.random((n, 3)) * 20 + rng.choice([-1e6, 1e5, 3e4])).astype(np.float32)
    if kind == 4:   # a line along one axis, negative coordinates
        c = np.zeros((n, 3), np.float32)
        c[:, int(rng.integers(0, 3))] = -rng.random(n) * 50
        return c
    return np.tile(rng.random((1, 3)).astype(np.float32) * 5, (n, 1))   # every point the same


@pytest.mark.parametrize("seed", range(24))
def test_random_configurations_of_every_entry_point(seed):
    """A configuration drawn from the whole parameter space of the calls (sizes, ragged and empty scans, cloud shape,
    hash, probes, order, schedule, scope shape, pass mode, heads, element type, pooling and glue shapes), every entry
    point against the oracle under the bounds of the tests above."""
    rng = np.random.default_rng(7000 + seed)
    n_scans = int(rng.choice([1, 2, 5, 60]))
    n = int(rng.integers(n_scans, 200 * n_scans if n_scans == 60 else 7000))
    bo = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n_scans - 1)), [n]]).astype(np.int32)
    kind = int(rng.integers(0, 6))
    coords = np.concatenate([random_cloud(rng, int(bo[i + 1] - bo[i]), kind) + 3.0 * i for i in range(n_scans)]).reshape(n, 3)
    m = int(rng.choice([1, 2, 3, 4, 8, 16]))
    cap = 16 * m * int(rng.choice([1, 2, 4, 8, 16]))
    kw = {"order": str(rng.choice(["index", "index", "canonical"])), "schedule": str(rng.choice(["auto", "general", "scans"])),
          "probe_mode": str(rng.choice(["axes", "axes", "seeded", "table"])), "probe_seed": int(rng.integers(0, 2 ** 31)),
          "probe_table": rng.integers(-5, 6, (6, 3)).tolist(), "max_scan_points": int(np.diff(bo).max())}
    if rng.random() < 0.2:
        kw["div"] = int(rng.integers(1, 5000))
    bk, ref = check_bucketize(coords, bo, float(rng.choice([1e-6, 0.01, 0.05, 0.5, 7.0])), cap, m, str(rng.choice(HASHES)),
                              int(rng.choice([0, 1, 3, 6, 6])), **kw)

    heads, d = int(rng.choice([1, 2, 3, 8])), int(rng.choice([16, 32]))
    mode = str(rng.choice(["plain", "shift", "stride"])) if m > 1 else str(rng.choice(["plain", "stride"]))
    shift, stride = (int(rng.integers(1, m)) if m > 1 else 1), int(rng.integers(1, 6))
    use_perm, scale = bool(rng.random() < 0.5), float(rng.choice([0.0, 0.1]))
    q, k, v, g = (wl.f32_to_bf16_bits(rng.standard_normal((n, heads * d)).astype(np.float32)) for _ in range(4))
    attn_case(q, k, v, bk, ref, heads, d, mode, use_perm, None, shift, stride, scale)
    qh, kh, vh = (wl.bf16_bits_to_f32(x).astype(np.float16) for x in (q, k, v))
    attn_case_f16(qh, kh, vh, bk, ref, heads, d, mode, use_perm, None, shift, stride, scale)
    grads = bwd_case(q, k, v, g, bk, ref, heads, d, mode, use_perm, None, shift, stride)
    # the same results in input order, from the kernels' own stores
    tq, tk, tv, tg = (dev(x, torch.bfloat16) for x in (q, k, v, g))
    lse = torch.empty(n, heads, dtype=torch.float32, device=DEV)
    out_bm = f3d.bucket_swin_attn(tq, tk, tv, bk, heads, d, mode, shift, stride, use_perm, lse=lse)
    out_in = f3d.bucket_swin_attn(tq, tk, tv, bk, heads, d, mode, shift, stride, use_perm, original_order=True)
    g_in = f3d.bucket_swin_attn_bwd(tq, tk, tv, out_bm, tg, lse, bk, heads, d, mode, shift, stride, use_perm, original_order=True)
    torch.cuda.synchronize()
    assert torch.equal(f3d.unpermute(out_bm, bk.perm).view(torch.int16), out_in.view(torch.int16))
    for a_, b_ in zip(grads, g_in):
        assert torch.equal(f3d.unpermute(a_, bk.perm).view(torch.int16), b_.view(torch.int16))

    feat = wl.f32_to_bf16_bits(rng.standard_normal((n, int(rng.choice([8, 16, 64, 128])))).astype(np.float32))
    check_pool(coords, ref["perm"], feat, bo, int(rng.choice([1, 7, 64, 100, 512, 1000, 1024])), int(rng.choice([1, 2, 3, 4, 8, 33, 64])),
               float(rng.choice([0.02, 0.1, 0.5])), str(rng.choice(HASHES)), str(rng.choice(["sum", "mean", "min", "max"])))

    c_in, n_outs = int(rng.choice([64, 128, 256])), int(rng.choice([1, 2, 3]))
    c_out = 64 * n_outs * int(rng.choice([1, 2, 4]))
    check_ln_linear(n, c_in, c_out, n_outs, rng, ln=bool(rng.random() < 0.6), with_bias=bool(rng.random() < 0.7),
                    with_res=bool(rng.random() < 0.5), gather=bool(rng.random() < 0.5), scatter=bool(rng.random() < 0.5))


def test_calls_on_two_streams_do_not_share_state():
    """The library keeps no state between calls: two different jobs enqueued alternately on two streams, each with
    its own buffers, give exactly what each gives alone."""
    wa, wb = wl.make_workload("tiny"), wl.make_workload("indoor")
    jobs = []
    for w, hash_ in ((wa, "xor_mod"), (wb, "zorder_div")):
        p = f3d.make_params(w.voxel_size, w.bucket_cap, w.scope_buckets, hash_)
        coords, bo = dev(w.coords), dev(w.batch_offsets.astype(np.int32))
        q, k, v = (dev(x, torch.bfloat16) for x in w.qkv())
        alone = f3d.psh_bucketize(coords, bo, p)
        out_alone = f3d.bucket_swin_attn(q, k, v, alone, w.heads, w.head_dim, "shift")
        torch.cuda.synchronize()
        ws = torch.empty(f3d.workspace_bytes(w.n, w.n_scans, p), dtype=torch.uint8, device=DEV)
        jobs.append((w, p, coords, bo, q, k, v, alone, out_alone, ws, torch.cuda.Stream()))
    results = [[], []]
    for rep in range(3):
        for j, (w, p, coords, bo, q, k, v, alone, out_alone, ws, stream) in enumerate(jobs):
            with torch.cuda.stream(stream):
                bk = f3d.psh_bucketize(coords, bo, p, ws)
                results[j].append((bk, f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, "shift")))
    torch.cuda.synchronize()
    for j, (w, p, coords, bo, q, k, v, alone, out_alone, ws, stream) in enumerate(jobs):
        for bk, out in results[j]:
            assert torch.equal(bk.perm, alone.perm) and torch.equal(bk.offsets, alone.offsets)
            assert torch.equal(out.view(torch.int16), out_alone.view(torch.int16))


def test_calls_of_two_threads_with_different_sizes():
    """Two threads, each on a stream of its own, call the kernels that take as much LDS as a call's sizes need, with different sizes: each
    gets what it gets alone."""
    rng = np.random.default_rng(90)
    jobs = []
    for tile, sizes in ((1024, [30_000] * 60), (256, [3000] * 49)):
        n = sum(sizes)
        coords, bo = dev(clustered_cloud(rng, n)), dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
        feat = torch.randn(n, 8, device=DEV).bfloat16()
        p = f3d.make_params(0.05, 256, max_scan_points=max(sizes), schedule="scans")

        def call(coords=coords, bo=bo, feat=feat, p=p, tile=tile):
            bk = f3d.psh_bucketize(coords, bo, p)
            return bk.perm, f3d.inbucket_pool(coords, bk.perm, feat, bo, tile, 2, 0.1)
        jobs.append((call, call(), [], torch.cuda.Stream()))
    torch.cuda.synchronize()

    def work(call, alone, got, stream):
        with torch.cuda.stream(stream):
            for _ in range(8):
                got.append(call())
            stream.synchronize()
    threads = [threading.Thread(target=work, args=job) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for call, (perm, pooled), got, stream in jobs:
        rows = int(pooled.pooled_offsets[-1])
        assert len(got) == 8
        for perm2, pooled2 in got:
            assert torch.equal(perm2, perm) and torch.equal(pooled2.sub_of, pooled.sub_of)
            assert torch.equal(pooled2.feat[:rows].view(torch.int16), pooled.feat[:rows].view(torch.int16))


def test_binding_refuses_wrong_shapes_and_types_on_the_device():
    """Optional arguments reach the library as bare addresses: a gamma of the wrong length, a float64 bias, a short
    log-sum-exp buffer or a permutation of another size must be refused before anything is launched."""
    w = wl.make_workload("tiny")
    bk = run_bucketize(w.coords, w.batch_offsets, w.voxel_size, w.bucket_cap)
    q, k, v = (dev(x, torch.bfloat16) for x in w.qkv())
    n, C = q.shape
    with pytest.raises(ValueError, match="lse"):
        f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, lse=torch.empty(n, device=DEV))
    with pytest.raises(ValueError, match="out"):
        f3d.bucket_swin_attn(q, k, v, bk, w.heads, w.head_dim, out=torch.empty(n - 1, C, dtype=torch.bfloat16, device=DEV))
    with pytest.raises(ValueError, match="k must have shape"):
        f3d.bucket_swin_attn(q, k[:, :C // 2].contiguous(), v, bk, w.heads, w.head_dim)
    wq = torch.zeros(3 * C, C, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(ValueError, match="gamma"):
        f3d.ln_linear(q, wq, None, torch.ones(C + 1, device=DEV), torch.zeros(C + 1, device=DEV), n_outs=3)
    with pytest.raises(TypeError, match="bias"):
        f3d.ln_linear(q, wq, torch.zeros(3 * C, dtype=torch.float64, device=DEV), n_outs=3)
    with pytest.raises(ValueError, match="row_in"):
        f3d.ln_linear(q, wq, row_in=bk.perm[:-1].contiguous(), n_outs=3)
    with pytest.raises(ValueError, match="perm"):
        f3d.unpermute(q, bk.perm[:-1].contiguous())
    with pytest.raises(ValueError, match="perm"):
        f3d.inbucket_pool(dev(w.coords), bk.perm[:-1].contiguous(), q, None, 128, 2, 0.1)
    torch.cuda.synchronize()
