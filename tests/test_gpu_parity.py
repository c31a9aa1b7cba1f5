"""GPU parity: libcvlc's HIP path against the CPU oracle, element by element,
through the C ABI (paper_2402_03770_amd.cvlc is argument marshalling only).

Bars: streams, group assignments (which records land in which group) and CIDs
are compared bit for bit; min/max exactly; sums of squares to 1e-6 relative;
the aggregate to 1e-5 * sum_i |w_i xhat_ij| per element (fp summation order is
free), single-client decode bit for bit.
"""
import ctypes as C
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import cvlc_synth as syn
import paper_2402_03770_amd.cvlc as cv
from oracle import cvlc_oracle as orc

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def to_lib_plan(po: orc.Plan) -> cv.Plan:
    """The same plan in the library's struct (plans are inputs to both sides)."""
    return cv.plan_manual(po.d, po.code_len(), po.counts(), B=float(po.B), quant=int(po.quant))


def gpu_encode(host_updates, oracle_plans, seed, client_ids, want_stats=True, error_stats=False):
    n = len(host_updates)
    d = host_updates[0].size
    plans = [to_lib_plan(p) for p in oracle_plans]
    updates = [torch.from_numpy(u).to(DEV) for u in host_updates]
    streams = [cv.new_stream_buffer(p, DEV) for p in plans]
    for s in streams:
        s.fill_(-1)  # the encoder must overwrite every word
    ws = cv.new_workspace(cv.encode_workspace_bytes(d, n), DEV)
    stats = torch.zeros(n * cv.STATS_STRIDE * C.sizeof(cv.SegStats), dtype=torch.uint8, device=DEV) if want_stats else None
    cv.encode_batch(plans, updates, seed, client_ids, streams, ws, stats, error_stats=error_stats)
    status = cv.device_status(ws)
    words = [s.cpu().numpy().view(np.uint32)[: p.stream_bytes // 4] for s, p in zip(streams, plans)]
    st = [cv.read_stats(stats, c, plans[c].n_coded) for c in range(n)] if want_stats else None
    return words, st, status, streams


def assert_stream_equal(got, ref, what=""):
    assert got.size == ref.size, what
    if not np.array_equal(got, ref):
        bad = np.flatnonzero(got != ref)
        raise AssertionError(f"{what}: {bad.size} of {ref.size} words differ, first at word {bad[0]}: "
                             f"{got[bad[0]]:#x} != {ref[bad[0]]:#x}")


def assert_stats_close(got, ref, R, error_stats=False):
    for r in range(R + 1):
        assert got[r].count == ref[r].count, r
        assert np.float32(got[r].min).view(np.uint32) == np.float32(ref[r].min).view(np.uint32), r
        assert np.float32(got[r].max).view(np.uint32) == np.float32(ref[r].max).view(np.uint32), r
        assert got[r].sumsq == pytest.approx(ref[r].sumsq, rel=1e-6, abs=1e-300), r
        if error_stats or r == R:   # every term is computed alike on both sides; only the order of the fp64 sum differs
            assert got[r].errsq == pytest.approx(ref[r].errsq, rel=1e-6, abs=1e-300), r
        else:
            assert got[r].errsq == 0.0, r


def check_encode(host_updates, oracle_plans, seed, client_ids):
    words, stats, status, streams = gpu_encode(host_updates, oracle_plans, seed, client_ids)
    assert status == 0
    refs = []
    for c, (u, p) in enumerate(zip(host_updates, oracle_plans)):
        ref = orc.encode(u, p, seed, client_ids[c])
        assert_stream_equal(words[c], ref.words, f"client {c}")
        assert_stats_close(stats[c], ref.stats, p.R)
        refs.append(ref.words)
    return refs, streams


def gpu_decode(streams_dev, d, weights=None, accumulate_into=None, quant=cv.QUANT_PQ):
    out = torch.full((d,), float("nan"), dtype=torch.float32, device=DEV) if accumulate_into is None else accumulate_into
    ws = cv.new_workspace(cv.decode_workspace_bytes(d, len(streams_dev)), DEV)
    cv.decode_aggregate(streams_dev, out, ws, weights=weights, accumulate=accumulate_into is not None, quant=quant)
    return out.cpu().numpy(), cv.device_status(ws)


def abs_terms(ref_streams, d, weights=None):
    """sum_i |w_i xhat_ij| from the oracle's single-client decodes."""
    n = len(ref_streams)
    tot = np.zeros(d)
    for i, s in enumerate(ref_streams):
        w = weights[i] if weights is not None else None
        single = orc.decode_aggregate([s], d, weights=[1.0]).astype(np.float64)
        B = float(s[5:6].view(np.float32)[0])
        tot += np.abs(single) * (abs(float(np.float32(w))) if w is not None else 1.0 / (n * B))
    return tot


def check_decode(ref_streams, d, weights=None):
    dev_streams = [torch.from_numpy(s.view(np.int32)).to(DEV) for s in ref_streams]
    got, status = gpu_decode(dev_streams, d, weights)
    assert status == 0
    ref = orc.decode_aggregate(ref_streams, d, weights=weights)
    tol = 1e-5 * abs_terms(ref_streams, d, weights)
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    assert np.all(err <= tol), f"max excess {np.max(err - tol)}"
    return got, ref


# --------------------------------------------------------------------------- configuration 1, full size
def test_cfg1_roundtrip_bit_exact():
    w = syn.WORKLOADS[1]
    U = syn.update_vector(1, 0)
    p = orc.plan_for(w)
    refs, dev_streams = check_encode([U], [p], w.quant_seed, [0])
    got, status = gpu_decode(dev_streams, w.d, weights=[1.0])
    assert status == 0
    ref = orc.decode_aggregate(refs, w.d, weights=[1.0])
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))      # one client: bit exact
    kept = orc.segments(U, p) > 0
    assert np.all(got[~kept] == 0) and kept.sum() == p.k


@pytest.mark.parametrize("cfg,clients,kernel", [(1, 1, "short_select_kernel"), (2, 2, "filter_kernel")])
def test_benchmark_reports_the_kernel_that_ran(cfg, clients, kernel, monkeypatch, capsys):
    """Short vectors have no filter launch, whose bracket the benchmark's roofline was read off."""
    import json
    import sys

    import bench

    monkeypatch.setattr(sys, "argv", ["bench.py", "--cfg", str(cfg), "--clients", str(clients), "--steps", "2", "--warmup", "1",
                                      "--no-cpu-baseline", "--stages"])
    assert bench.main() == 0
    line = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    assert line["roofline"]["kernel"] == kernel and line["roofline"]["launch_ms"] > 0.0 and line["value"] > 0.0


def test_encode_is_deterministic_and_seed_sensitive():
    U = syn.update_vector(1, 5, d=50_000)
    p = orc.plan_fractions(U.size, [6, 3, 1], [0.05, 0.1, 0.2])
    a, _, sa, _ = gpu_encode([U], [p], 11, [4], want_stats=False)
    b, _, sb, _ = gpu_encode([U], [p], 11, [4], want_stats=False)
    c, _, _, _ = gpu_encode([U], [p], 12, [4], want_stats=False)
    e, _, _, _ = gpu_encode([U], [p], 11, [5], want_stats=False)
    assert sa == 0 and sb == 0
    assert np.array_equal(a[0], b[0])
    assert not np.array_equal(a[0], c[0]) and not np.array_equal(a[0], e[0])


# --------------------------------------------------------------------------- shapes: ragged tails, tiny inputs, odd plans
@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 63, 64, 65, 1000, 4095, 4096, 4097, 8191, 12_289, 100_003])
def test_ragged_sizes(d):
    rng = np.random.default_rng(d)
    U = syn.update_vector(1, d % 7, d=d)
    R = int(min(4, d))
    cuts = np.sort(rng.integers(0, d + 1, size=R))
    counts = np.diff(np.concatenate([[0], cuts])).tolist()
    y = sorted(rng.choice([1, 2, 5, 8, 16, 32], size=R).tolist(), reverse=True)
    p = orc.plan_manual(d, y, counts)
    refs, _ = check_encode([U], [p], 1000 + d, [d % 5])
    check_decode(refs, d)


@pytest.mark.parametrize("d", [20_000, 70_001])
def test_degenerate_plans(d):
    U = syn.update_vector(2, 1, d=d)
    cases = [
        ([], []),                                  # nothing coded: header-only stream
        ([8], [d]),                                # everything coded: plain quantisation
        ([32], [d]),                               # everything raw
        ([16, 8, 4], [0, 0, 0]),                   # empty groups only
        ([16, 8, 8, 2], [0, 7, 0, 1]),             # empty groups between tiny ones
        ([4, 4, 4], [1, 1, 1]),                    # single-member groups: one centroid each
        ([1] * 31, [100] * 31),                    # the maximum number of groups
        ([16] + [3] * 30, [1] + [600] * 30),
    ]
    for y, counts in cases:
        p = orc.plan_manual(d, y, counts)
        refs, _ = check_encode([U], [p], 5, [9])
        check_decode(refs, d)


TIE_KINDS = ["all_equal", "all_equal_mixed_sign", "two_valued", "few_levels", "zeros_and_denormals", "all_zero"]


@pytest.mark.parametrize("kind", TIE_KINDS)
def test_tie_heavy_vectors(kind):
    for d in (777, 65_536, 70_001):
        U = syn.tie_heavy_vector(kind, d, seed=d)
        p = orc.plan_manual(d, [8, 4, 4, 1], [d // 50, 0, d // 3, d // 4])
        refs, _ = check_encode([U], [p], 3, [1])
        check_decode(refs, d)


@pytest.mark.parametrize("kind", ["all_equal_mixed_sign", "two_valued", "few_levels", "zeros_and_denormals"])
def test_tie_heavy_vectors_with_more_than_fifteen_groups(kind):
    """Plans of more than 15 groups select all their boundaries in one round of wider kernels: the same
    colliding magnitudes through those, with many boundaries inside one class of equal keys."""
    for d, R in ((65_536, 31), (70_001, 20)):
        U = syn.tie_heavy_vector(kind, d, seed=d + R)
        code_len = [max(1, 16 - r // 2) for r in range(R)]
        counts = [d // (3 * R) + 7 * r for r in range(R)]
        counts[R // 2] = 0
        p = orc.plan_manual(d, code_len, counts)
        refs, _ = check_encode([U], [p], 5, [4])
        check_decode(refs, d)


SAMPLE_PIECE, SAMPLE_PIECES = 64, 4096  # the encoder's sample: evenly spread pieces of 64 coordinates


def plant_on_the_sampled_pieces(U, rng):
    """Large values on exactly the coordinates the encoder samples (262 144 of them), in place."""
    n_src, n_s = U.size // SAMPLE_PIECE, SAMPLE_PIECES
    pieces = (np.arange(n_s, dtype=np.int64) * n_src) // n_s
    for off in range(SAMPLE_PIECE):
        U[pieces * SAMPLE_PIECE + off] = (rng.standard_normal(n_s) * 10.0).astype(np.float32)


def test_misjudged_sample_in_a_workspace_sized_to_the_plan():
    """When the sampled threshold keeps fewer than k coordinates every coordinate becomes a candidate, which a
    workspace sized to the plan has no room for: that client is refused, not encoded wrongly."""
    d = 2_000_000
    rng = np.random.default_rng(5)
    U = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    plant_on_the_sampled_pieces(U, rng)
    po = orc.plan_manual(d, [8, 4, 2], [50_000, 100_000, 150_000])
    p = to_lib_plan(po)
    stream = cv.new_stream_buffer(p, DEV)
    stream.fill_(-1)
    ws = cv.new_workspace(cv.encode_workspace_bytes_for(d, 1, cv.plan_candidates_hint(p)), DEV)
    cv.encode_batch([p], [torch.from_numpy(U).to(DEV)], 21, [3], [stream], ws)
    assert cv.device_status(ws) == cv.DEV_WORKSPACE
    assert int(stream[0].item()) == 0


def test_boundary_ties_inside_smooth_data():
    """A smooth vector into which runs of equal magnitudes (mixed signs) are planted
    right at the group boundaries."""
    d = 300_000
    U = syn.update_vector(1, 8, d=d)
    order = np.argsort(-np.abs(U), kind="stable")
    counts = [3000, 7000, 20_000]
    for Z in np.cumsum(counts):
        members = order[Z - 40: Z + 40]
        U[members] = np.abs(U[order[Z]]) * np.where(np.arange(80) % 3 == 0, -1.0, 1.0).astype(np.float32)
    p = orc.plan_manual(d, [8, 4, 2], counts)
    refs, _ = check_encode([U], [p], 8, [2])
    check_decode(refs, d)


@pytest.mark.parametrize("n,d", [(1, 1024), (1, 1025), (2, 3 * 1024 - 1), (6, 1024 * 1024), (6, 1024 * 1024 + 1),
                                 (7, 2048 * 877 + 2047), (12, 1024 * 1024 + 8191),
                                 (1, 65 * 1024), (1, 65 * 1024 + 1), (2, 66 * 1024 - 1),   # lengths that have a filter
                                 (1, 2048 * 1024), (1, 2048 * 1024 + 1), (1, 4096 * 8192 + 1)])
def test_region_lengths(n, d):
    """The filter's regions have 1024 to 8192 coordinates, by the size of the batch: sizes at the steps of that rule
    and with a last region of one coordinate, one missing, or one too many; and one region more than the threads of the
    region scan take at one, two and four each."""
    host = [syn.update_vector(2 + c % 2, 300 + c, d=d) for c in range(n)]
    plans = [orc.plan_fractions(d, [9, 6, 3], [0.004, 0.01, 0.03 + 0.01 * (c % 3)]) for c in range(n)]
    check_encode(host, plans, 14, list(range(n)))


def _keep_all_plan(d, quant=cv.QUANT_PQ):
    counts = [d // 50, d // 7, d // 3]
    return orc.plan_manual(d, [11, 6, 4, 2], counts + [d - sum(counts)], quant=quant)


def check_some_streams(host, plans, which, seed=21):
    """A batch without a layout kernel whose streams are compared for the clients in `which` only."""
    cv.profile_start(["enc_layout"])
    words, stats, status, _ = gpu_encode(host, plans, seed, list(range(len(host))), error_stats=True)
    assert not cv.profile_stop()
    assert status == 0
    for c in which:
        ref = orc.encode(host[c], plans[c], seed, c)
        assert_stream_equal(words[c], ref.words, f"client {c}")
        assert_stats_close(stats[c], ref.stats, plans[c].R, error_stats=True)


@pytest.mark.parametrize("quant", [cv.QUANT_PQ, cv.QUANT_QSGD])
@pytest.mark.parametrize("chunks,more", [(16, 1), (128, 0), (128, 1), (256, 1)])
def test_packing_at_the_steps_of_the_chunk_prefix(chunks, more, quant):
    """Sixteen blocks of eight chunks of 4096 candidates, of sixteen from the 129th chunk on, of 32 from the 257th on."""
    d = chunks * 4096 + more
    check_some_streams([syn.update_vector(2, 60 + chunks, d=d)], [_keep_all_plan(d, quant)], [0])


def test_packing_by_workgroups_of_more_chunks_than_their_counters_hold():
    """1024 clients: one counting workgroup each, with counters for sixteen chunks at a time; two clients have 21."""
    n, d = 1024, 20 * 4096 + 1
    vectors = [syn.update_vector(2, 70 + c, d=d) for c in range(4)]
    plans = [_keep_all_plan(d) if c in (3, 1022) else orc.plan_manual(d, [9, 4], [100, 200 + c % 5]) for c in range(n)]
    check_some_streams([vectors[c % 4] for c in range(n)], plans, [0, 3, 517, 1022, 1023])


@pytest.mark.parametrize("quant", [cv.QUANT_PQ, cv.QUANT_QSGD])
def test_packing_by_the_layout(quant):
    """Many clients that keep all of vectors just too short for a layout kernel to number their chunks."""
    n, d = 48, 128 * 4096 + 1537
    vectors = [syn.update_vector(2, 80 + c, d=d) for c in range(3)]
    check_some_streams([vectors[c % 3] for c in range(n)], [_keep_all_plan(d, quant)] * n, [0, 25, 47])


@pytest.mark.parametrize("quant", [cv.QUANT_PQ, cv.QUANT_QSGD])
def test_packing_by_the_layout_of_plans_that_differ(quant):
    """So many clients that keep so much that a layout kernel numbers the chunks: plans of 4 and of 31 groups, some of them
    empty, and a client of equal magnitudes, for all of which the workspace has no room."""
    n, d, seed, flat = 128, 128 * 4096 + 1537, 21, 77
    rng = np.random.default_rng(8)
    vectors = [syn.update_vector(2, 80 + c, d=d) for c in range(3)]
    vectors.append(np.where(rng.random(d) < 0.4, -0.25, 0.25).astype(np.float32))
    few, half = [d // 50, d // 7, d // 5], d // 2
    oplans = [orc.plan_manual(d, [11, 6, 4, 2], few + [half - sum(few)], quant=quant),
              orc.plan_manual(d, [11, 6, 6, 4, 3, 2], [0] + few[:2] + [0, half - sum(few[:2]), 0], quant=quant),
              orc.plan_manual(d, [14] * 9 + [11] * 9 + [7] * 13, [half // 31 - 15 + c for c in range(31)], quant=quant)]
    plans = [to_lib_plan(p) for p in oplans]
    room = max(cv.plan_candidates_hint(p) for p in plans)
    assert room < d
    updates = [torch.from_numpy(v).to(DEV) for v in vectors]
    streams = [cv.new_stream_buffer(plans[c % 3], DEV).fill_(-1) for c in range(n)]
    stats = torch.full((n * cv.STATS_STRIDE * C.sizeof(cv.SegStats),), 255, dtype=torch.uint8, device=DEV)
    ws = cv.new_workspace(cv.encode_workspace_bytes_for(d, n, room), DEV)
    cv.profile_start(["enc_layout"])
    cv.encode_batch([plans[c % 3] for c in range(n)], [updates[3 if c == flat else c // 3 % 3] for c in range(n)], seed,
                    list(range(n)), streams, ws, stats, error_stats=True)
    assert "enc_layout" in cv.profile_stop()
    assert cv.device_status(ws) == cv.DEV_WORKSPACE
    assert int(streams[flat][0].item()) == 0 and bool((streams[flat][1:] == -1).all())
    assert bool((stats.view(n, -1)[flat] == 255).all())
    for c in (0, 4, 8, flat - 1, flat + 1, n - 3, n - 2, n - 1):
        ref = orc.encode(vectors[c // 3 % 3], oplans[c % 3], seed, c)
        assert_stream_equal(streams[c].cpu().numpy().view(np.uint32)[: plans[c % 3].stream_bytes // 4], ref.words, f"client {c}")
        assert_stats_close(cv.read_stats(stats, c, plans[c % 3].n_coded), ref.stats, plans[c % 3].n_coded, error_stats=True)


@pytest.mark.parametrize("n,share,layout", [(1, 1.0, False), (8, 0.03, False), (8, 1.0, True)])
def test_which_kernel_numbers_the_chunks(n, share, layout):
    """Several clients that keep all of 11.2 M coordinates were 8 % slower without the layout kernel than with it."""
    d = 11_200_000
    plan = cv.plan_manual(d, [6, 4], [int(d * share) // 2] * 2)
    update = torch.randn(d, device=DEV)
    streams = [cv.new_stream_buffer(plan, DEV) for _ in range(n)]
    ws = cv.new_workspace(cv.encode_workspace_bytes_for(d, n, cv.plan_candidates_hint(plan)), DEV)
    cv.profile_start(["enc_layout"])
    cv.encode_batch([plan] * n, [update] * n, 3, [5] * n, streams, ws)
    assert ("enc_layout" in cv.profile_stop()) == layout
    assert cv.device_status(ws) == 0
    assert all(torch.equal(s, streams[0]) for s in streams[1:])


def _selection_vectors(kind, d, rng):
    """Magnitudes that the selection bins (a thousandth of the sampled candidates each, 16 octaves of them) fit badly."""
    sign = np.where(rng.random(d) < 0.5, -1.0, 1.0)
    if kind == "octaves":          # far more octaves than the fine bins reach
        return (sign * 10.0 ** rng.uniform(-36.0, 36.0, d)).astype(np.float32)
    if kind == "few values":       # thousands of equal keys in every boundary's bin
        return (sign * 2.0 ** rng.integers(-3, 4, d)).astype(np.float32)
    if kind == "bfloat16":         # seven mantissa bits: every bin one key, some of them full
        return (torch.from_numpy((rng.standard_normal(d) * 1e-2).astype(np.float32)).to(torch.bfloat16).float().numpy().copy())
    if kind == "zeros":            # nothing above zero below the first tenth
        return np.where(rng.random(d) < 0.1, sign * rng.random(d), 0.0).astype(np.float32)
    if kind == "ramp":             # neighbours in one bin, a few of the bins in each part of the vector
        return np.linspace(1e-6, 1.0, d).astype(np.float32)
    U = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    if kind == "sorted":
        return np.sort(U)
    if kind == "one outlier":
        U[rng.integers(d)] = 1e30
    return U


@pytest.mark.parametrize("share", [0.02, 0.45, 1.0])
@pytest.mark.parametrize("kind", ["octaves", "few values", "bfloat16", "zeros", "one outlier", "plain"])
@pytest.mark.parametrize("d", [50, 5000, 600_000])
def test_selection_bins(d, kind, share):
    """Boundaries in bins that hold next to nothing, everything, or more than their list has room for; with `share` 1
    every coordinate is coded and no threshold is sampled."""
    U = _selection_vectors(kind, d, np.random.default_rng(d))
    counts = [max(1, int(d * share * f)) for f in (0.001, 0.009, 0.09, 0.2, 0.3, 0.2)]
    counts.append(max(int(d * share) - sum(counts), 0))
    p = orc.plan_manual(d, [12, 10, 8, 6, 4, 2, 1], counts)
    check_encode([U], [p], 17, [4])


# A bin's members fit LDS up to 2048 of them, and the pool of its first boundary (6735 entries here) up to half of that.
@pytest.mark.parametrize("members", [2047, 2048, 2049, 2700, 3367, 3368])
def test_boundaries_that_share_a_bin_on_both_sides_of_its_lists_limits(members):
    """32 classes of equal keys, each a selection bin of its own, most of them with two boundaries."""
    d = 600_001
    rng = np.random.default_rng(members)
    U = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    U[rng.permutation(d)[: 32 * members]] = np.repeat(1.0 + np.arange(32) / 1024.0, members).astype(np.float32)
    U *= np.where(rng.random(d) < 0.5, -1.0, 1.0).astype(np.float32)
    p = orc.plan_manual(d, [max(1, 12 - r // 3) for r in range(31)], [300 + 17 * (r % 7) if r % 2 else 3300 for r in range(31)])
    check_encode([U], [p], 33, [6])


SHORT_MAX = 65_536  # vectors up to here are selected by one workgroup


@pytest.mark.parametrize("R", [1, 7, 31])
@pytest.mark.parametrize("kind", ["plain", "bfloat16", "few values", "zeros", "one outlier"])
@pytest.mark.parametrize("d", [4097, 40_003, SHORT_MAX - 1, SHORT_MAX, SHORT_MAX + 1])
def test_short_vectors(d, kind, R):
    """Half of the coordinates kept: boundaries among distinct keys, pairs of equal ones, and classes larger than what is
    set aside, which are counted by parts of the vector."""
    U = _selection_vectors(kind, d, np.random.default_rng(d + R))
    counts = [max(1, d * (r + 1) // (R * (R + 1))) for r in range(R)]
    p = orc.plan_manual(d, [max(1, 14 - r // 2) for r in range(R)], counts)
    check_encode([U], [p], 19, [6])
    q = orc.plan_manual(d, [max(2, 14 - r // 2) for r in range(R)], counts, quant=orc.QSGD)
    words, _, status, _ = gpu_encode([U], [q], 20, [7], error_stats=True)
    assert status == 0
    assert_stream_equal(words[0], orc.encode(U, q, 20, 7).words)


@pytest.mark.parametrize("n,d,share,filtered", [(144, SHORT_MAX, 0.03, False), (145, SHORT_MAX, 0.03, True), (145, SHORT_MAX, 0.007, False),
                                                (145, SHORT_MAX, 0.301, False), (231, 40_961, 0.03, True), (300, 40_960, 0.03, False)])
def test_many_short_vectors(n, d, share, filtered):
    """Many long ones of the short vectors, of which some but not much is kept, are encoded like long vectors."""
    rng = np.random.default_rng(n)
    U = [rng.standard_normal(d).astype(np.float32) for _ in range(3)]
    p = orc.plan_manual(d, [9, 5], [d // 1000, int(d * share) - d // 1000])
    cv.profile_start(["enc_filter"])
    words, _, status, _ = gpu_encode([U[c % 3] for c in range(n)], [p] * n, 31, list(range(n)), want_stats=False)
    assert ("enc_filter" in cv.profile_stop()) == filtered
    assert status == 0
    for c in (0, 1, 2, n // 2, n - 1):
        assert_stream_equal(words[c], orc.encode(U[c % 3], p, 31, c).words, f"client {c}")


def test_short_vectors_of_many_plans():
    """More different plans than one launch's arguments hold, groups of no coordinates among them."""
    d, n = 3001, 45
    rng = np.random.default_rng(9)
    host = [_selection_vectors("plain", d, rng) for _ in range(n)]
    plans = [orc.plan_manual(d, [9, 6, 3], [0 if c % 5 == 0 else c, 40 + c, 0 if c % 7 == 0 else 300]) for c in range(n)]
    check_encode(host, plans, 23, list(range(n)))


@pytest.mark.parametrize("error_stats", [False, True])
@pytest.mark.parametrize("d", [50_047, SHORT_MAX + 47])
def test_short_vectors_are_refused_by_the_same_rule(d, error_stats):
    """A vector has as many candidates as it has keys at or above the lower edge of the 13-bit bin that holds the sample's
    rank-th largest, the sample being all but the last d mod 64 coordinates; a workspace with less room refuses it."""
    k = 9_000
    rng = np.random.default_rng(31)
    U = rng.standard_normal(d).astype(np.float32)
    key = U.view(np.uint32) & np.uint32(0x7FFFFFFF)
    sampled = d // 64 * 64
    E = k * sampled / d
    rank = int(np.ceil(E + 6.0 * np.sqrt(E) + 16.0))
    edge = (np.sort(key[:sampled])[::-1][rank - 1] >> 18) << 18
    c = int(np.count_nonzero(key >= edge))
    p = to_lib_plan(orc.plan_manual(d, [8, 4], [k // 3, k - k // 3]))
    slack = 512  # a workspace of so many bytes has room for a few hundred candidates more than it was asked for
    for room, expected in ((c, 0), (c - slack, cv.DEV_WORKSPACE)):
        stream = cv.new_stream_buffer(p, DEV)
        stream.fill_(-1)
        stats = torch.full((cv.STATS_STRIDE * C.sizeof(cv.SegStats),), 0xA5, dtype=torch.uint8, device=DEV)
        ws = cv.new_workspace(cv.encode_workspace_bytes_for(d, 1, room), DEV)
        ws.fill_(255)
        cv.encode_batch([p], [torch.from_numpy(U).to(DEV)], 21, [3], [stream], ws, stats, error_stats=error_stats)
        assert cv.device_status(ws) == expected
        assert (int(stream[0].item()) == 0) == (expected != 0)
        # a refused client's entries are not written, not even in part; an encoded one's all are
        entries = stats.view(cv.STATS_STRIDE, -1)
        assert bool((entries[p.n_coded + 1:] == 0xA5).all())
        assert bool((entries[: p.n_coded + 1] == 0xA5).all(dim=1).any()) == (expected != 0)
        if expected:
            assert bool((stats == 0xA5).all())


def _equal_keys(kind, d, rng):
    """Short vectors whose boundaries' bins (14 bits of the key) hold more than is set aside, or large classes of equal keys."""
    sign = np.where(rng.random(d) < 0.5, -1.0, 1.0)
    if kind == "one magnitude":
        return (sign * 1e-3).astype(np.float32)
    if kind == "two magnitudes":
        return (sign * np.where(rng.random(d) < 0.4, 3e-3, 1e-3)).astype(np.float32)
    if kind == "seven magnitudes":
        return (sign * rng.integers(1, 8, d) * 1e-3).astype(np.float32)
    if kind == "int8":
        x = rng.standard_normal(d)
        return (np.round(x * 127 / np.abs(x).max()) * 1e-5).astype(np.float32)
    if kind == "two a bin":        # as many keys as bfloat16 has in a bin, most of the vector in three bins
        return (sign * (1.0 + rng.integers(0, 6, d) / 128.0)).astype(np.float32)
    if kind == "five in one bin":  # no key of a bin is most of it
        return (sign * (1.0 + rng.integers(0, 5, d) / 1024.0)).astype(np.float32)
    if kind == "one bin":          # nothing but different keys
        return (sign * (1.0 + rng.permutation(d) * 2.0 ** -23)).astype(np.float32)
    if kind == "sorted":           # a bin's keys side by side: few wavefronts come across them
        return np.sort(rng.standard_normal(d)).astype(np.float32)
    assert kind == "at the ends"   # a class whose members are the first and the last coordinates
    x = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    x[:70] = x[-150:] = 2e-3
    return x


@pytest.mark.parametrize("R", [1, 6, 31])
@pytest.mark.parametrize("kind", ["one magnitude", "two magnitudes", "seven magnitudes", "int8", "two a bin", "five in one bin", "one bin",
                                  "sorted", "at the ends"])
@pytest.mark.parametrize("d", [479, 9001, 12_591, 40_003, SHORT_MAX - 1, SHORT_MAX])   # 479, 12 591: the last three in a part of their own
def test_short_vectors_with_full_bins(d, kind, R):
    """All three ways that the members of the boundaries' bins are counted in, and the ties of each."""
    U = _equal_keys(kind, d, np.random.default_rng(d + R))
    counts = [max(1, d * 9 // 10 * (r + 1) // (R * (R + 1) // 2)) for r in range(R)]
    if kind == "at the ends":      # a boundary inside the class, in each of its halves
        k = int(np.count_nonzero(np.abs(U) > 2e-3))
        counts = [k + 60, 50, 100][: min(R, 3)] + [7] * max(R - 3, 0)
    p = orc.plan_manual(d, [max(1, 14 - r // 2) for r in range(R)], counts)
    check_encode([U], [p], 29, [5])


def encode_stage_us(update, plan, stage, repeats=5):
    """Shortest time of a stage of an encode call, on a workspace full of ones: what the call before left there must not matter."""
    ws = cv.new_workspace(cv.encode_workspace_bytes(plan.d, 1), DEV)
    stream = cv.new_stream_buffer(plan, DEV)
    best = float("inf")
    for _ in range(repeats):
        ws.fill_(255)
        cv.profile_start([stage])
        cv.encode_batch([plan], [update], 3, [1], [stream], ws)
        best = min(best, cv.profile_stop()[stage][0] * 1e3)
        assert cv.device_status(ws) == 0
    return best


def test_boundaries_that_share_a_tied_bin_cost_what_one_does():
    """Seven magnitudes: the boundaries cut one class of a million equal keys, and every boundary's workgroup starts from
    a member of the class.  (From anything else the search takes twice as long.)"""
    d = 8_000_000
    U = torch.from_numpy((2.0 ** np.random.default_rng(1).integers(-3, 4, d)).astype(np.float32)).to(DEV)
    one = encode_stage_us(U, cv.plan_manual(d, [8], [80_000]), "enc_select")
    three = encode_stage_us(U, cv.plan_manual(d, [8, 6, 4], [20_000, 20_000, 40_000]), "enc_select")
    assert three < 1.25 * one, (one, three)


@pytest.mark.parametrize("kind", ["laplace", "fp16", "sorted"])
def test_half_of_a_large_vector_kept(kind):
    """Bins grow with the candidates, and so do the lists of the boundaries' bins: with six million candidates and keys
    that are not all equal no boundary's search goes through all of them (which took a hundred times as long)."""
    rng = np.random.default_rng(6)

    def vector(d):
        U = (rng.laplace(size=d) * 1e-3).astype(np.float32)
        if kind == "fp16":      # a handful of equal keys to a bin
            U = U.astype(np.float16).astype(np.float32)
        return np.sort(np.abs(U)) if kind == "sorted" else U

    fractions, y = (0.10, 0.15, 0.25), [8, 4, 2]
    U = vector(12_000_037)
    po = orc.plan_manual(U.size, y, [int(f * U.size) for f in fractions])
    check_encode([U], [po], 9, [5])
    small = vector(3_000_000)
    t = [encode_stage_us(torch.from_numpy(u).to(DEV), cv.plan_manual(u.size, y, [int(f * u.size) for f in fractions]), "enc_select")
         for u in (small, U)]
    assert t[1] < 10 * t[0], t      # four times the candidates


@pytest.mark.parametrize("kind", ["neighbours", "low octave", "signs", "late class"])
def test_bins_that_hold_a_large_part_of_all_candidates(kind):
    """Such a bin has no list, its boundaries are looked for in the dense list: two classes of equal keys one apart among
    close ones (the key counted by itself may be the wrong one), half a million different keys of one octave far below the
    window of fine bins, one magnitude for all, and a class that begins late in the vector."""
    rng = np.random.default_rng(8)
    d = 700_001
    bits = np.full(d, 0x3F800000, np.uint32)
    if kind == "neighbours":
        u = rng.random(d)
        bits = np.where(u < 0.3, 0x3F800040, np.where(u < 0.6, 0x3F800041, 0x3F800000 + rng.integers(0, 400, d))).astype(np.uint32)
    if kind == "low octave":
        bits = np.where(rng.random(d) < 0.05, 0x3F800000 + rng.integers(0, 1 << 23, d), 0x20000000 + rng.integers(0, 1 << 23, d)).astype(np.uint32)
    if kind == "late class":
        bits = np.where(np.arange(d) < 9 * d // 10, 0x3F800000 + rng.integers(0, 3, d), 0x3F900000).astype(np.uint32)
    U = (bits | np.where(rng.random(d) < 0.5, 0x80000000, 0).astype(np.uint32)).view(np.float32)
    for share in (0.03, 0.4, 1.0):
        counts = [1, int(0.1 * share * d), int(0.2 * share * d), 0, int(0.3 * share * d), 2]
        counts.append(int(share * d) - sum(counts))
        check_encode([U], [orc.plan_manual(d, [12, 10, 8, 6, 6, 4, 1], counts)], 17, [4])


def test_a_misjudged_sample_costs_one_pass_of_one_workgroup():
    """Every coordinate is then a candidate and one workgroup counts them all, once; the vector's other pass, by
    the whole device, is the measure (a factor of 50 here; 330 with two passes and an LDS atomic for every key)."""
    d = 8_000_000
    rng = np.random.default_rng(3)
    U = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    plant_on_the_sampled_pieces(U, rng)
    p = cv.plan_manual(d, [8, 4], [100_000, 140_000])
    update = torch.from_numpy(U).to(DEV)
    t = [encode_stage_us(update, p, stage) for stage in ("enc_filter", "enc_refilter")]
    assert t[1] < 120 * t[0], t


def test_a_class_of_equal_keys_is_cut_in_few_passes():
    """(A hundred times the time of the smooth vector before the passes were made to use the CU's bandwidth.)"""
    d = 8_000_000
    rng = np.random.default_rng(2)
    p = cv.plan_manual(d, [8, 6, 4], [800_000, 800_000, 2_000_000])
    smooth, tied = (torch.from_numpy(u.astype(np.float32)).to(DEV) for u in (rng.laplace(size=d), 2.0 ** rng.integers(-3, 4, d)))
    t = [encode_stage_us(u, p, "enc_select") for u in (smooth, tied)]
    assert t[1] < 40 * t[0], t


@pytest.mark.parametrize("n,R", [(1, 1), (9, 7), (16, 4), (13, 5), (16, 31), (17, 3), (17, 4), (25, 31), (133, 31)])
def test_decode_at_the_steps_of_the_list_search(n, R):
    """1, 63, 64, 65, 496, 51, 68, 775 and 4123 lists with records, nearly all of one item: numbered and gone through in one launch
    up to 112 streams, in three beyond."""
    d = 6000
    rng = np.random.default_rng(n)
    host = [(rng.standard_normal(d) * 1e-3).astype(np.float32) for _ in range(min(n, 8))]
    p = orc.plan_manual(d, [8] * R, [600 if r == R // 2 and R < 8 else 20 for r in range(R)])
    refs = [orc.encode(host[c % 8], p, 3, c).words for c in range(n)]
    check_decode(refs, d, weights=rng.uniform(0.5, 1.5, n).tolist())


@pytest.mark.parametrize("n,lists", [(113, 0), (113, 1), (113, 63), (113, 64), (113, 65), (113, 68), (113, 496), (113, 3503), (133, 4096), (133, 4097),
                                     (133, 4123)])
def test_decode_at_the_steps_of_the_list_search_of_many_streams(n, lists):
    """The search for an item's list, in calls of more streams than one launch parses and numbers, takes 64 lists a round: up to
    64, up to 4096 and more of the streams' 31 groups each have records, a few of them several items."""
    d = 6000
    rng = np.random.default_rng(lists)
    host = [(rng.standard_normal(d) * 1e-3).astype(np.float32) for _ in range(8)]
    filled = np.zeros(n * 31, dtype=int)
    filled[rng.permutation(n * 31)[:lists]] = 20
    filled[np.flatnonzero(filled)[::29]] = 1100
    refs = [orc.encode(host[c % 8], orc.plan_manual(d, [8] * 31, filled[c * 31: c * 31 + 31].tolist()), 3, c).words for c in range(n)]
    check_decode(refs, d, weights=rng.uniform(0.5, 1.5, n).tolist())


# Lists are dealt out to 1, 2, 4 or 8 groups of wavefronts, 60 to each, and to several sweeps beyond 480: both sides of
# every step, empty lists among them, with few records and with every coordinate kept (a wavefront's share is many turns).
@pytest.mark.parametrize("quant", [cv.QUANT_PQ, cv.QUANT_QSGD])
@pytest.mark.parametrize("n,R", [(1, 1), (1, 31), (8, 31), (9, 31), (12, 5), (61, 1), (15, 8), (11, 11), (16, 15), (241, 1), (32, 15), (37, 13), (70, 14)])
def test_decode_at_the_steps_of_the_lists_share(n, R, quant):
    rng = np.random.default_rng(n * 100 + R)
    d = 9001                                       # two tiles and a part of a third
    refs = []
    for c in range(n):
        full = c % 7 == 0
        cnt = [d // R] * R if full else [int(v) for v in rng.integers(0, 1 + d // (8 * R), R)]
        cnt[-1] = max(cnt[-1], 1)
        ys = sorted((int(v) for v in rng.integers(2, 17, R)), reverse=True)
        u = rng.standard_t(3, d).astype(np.float32)
        refs.append(orc.encode(u, orc.plan_manual(d, ys, cnt, quant=quant), 5, c).words)
    dev = [torch.from_numpy(s.view(np.int32)).to(DEV) for s in refs]
    got, status = gpu_decode(dev, d, quant=quant)
    assert status == 0
    ref = orc.decode_aggregate(refs, d).astype(np.float64)
    # fp64 sums in free order, rounded to fp32 once: half a unit of the last place on either side
    assert np.all(np.abs(got - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12 * abs_terms(refs, d))


@pytest.mark.parametrize("n", [8, 9, 64, 65, 112, 113])
def test_decode_of_streams_of_unequal_lengths(n):
    """Few and many streams' arguments, the last number that one launch parses and the first that it does not; the workgroups
    go by the streams' lengths: one stream has nearly all records, some have empty groups, some none at all."""
    d = 200_003
    refs = []
    for c in range(n):
        U = syn.update_vector(2 + c % 2, 2500 + c, d=d)
        counts = [40_000, 90_000, 30_000] if c == n // 2 else [[0, 0, 0], [5, 0, 40], [0, 700, 0], [300, 513, 1024]][c % 4]
        refs.append(orc.encode(U, orc.plan_manual(d, [9, 6, 2], counts), 9, c).words)
    check_decode(refs, d)
    order = list(range(n))[::-1]
    check_decode([refs[c] for c in order], d, weights=np.random.default_rng(n).uniform(-1.0, 1.0, n).astype(np.float32).tolist())


@pytest.mark.parametrize("n,R,filled", [(1, 31, 1), (3, 31, 0), (8, 31, 2), (9, 31, 30), (70, 7, 6), (100, 31, 8), (112, 31, 1), (112, 31, 20)])
def test_decode_of_streams_of_many_empty_groups(n, R, filled):
    """Lists with records are numbered, and swept over, without the empty ones (one to six sweeps here); a stream whose header is
    wrong, first, last or in the middle, is left out and reported."""
    rng = np.random.default_rng(n * 40 + filled)
    d = 9001
    refs = []
    for c in range(n):
        counts = np.zeros(R, dtype=int)
        counts[rng.permutation(R)[:filled]] = rng.integers(1, d // (4 * R), filled)
        ys = sorted((int(v) for v in rng.integers(2, 17, R)), reverse=True)
        refs.append(orc.encode(rng.standard_t(3, d).astype(np.float32), orc.plan_manual(d, ys, counts.tolist()), 5, c).words)
    weights = rng.uniform(0.5, 1.5, n).astype(np.float32).tolist()
    check_decode(refs, d, weights=weights)
    for wrong in sorted({0, n // 2, n - 1}):
        bad = refs[wrong].copy()
        bad[2] += 1
        dev = [torch.from_numpy((bad if c == wrong else w).view(np.int32)).to(DEV) for c, w in enumerate(refs)]
        got, status = gpu_decode(dev, d, weights=weights)
        assert status == cv.DEV_STREAM
        rest = [c for c in range(n) if c != wrong]
        left = [refs[c] for c in rest], d, [weights[c] for c in rest]
        expected = orc.decode_aggregate(left[0], d, weights=left[2]).astype(np.float64) if rest else np.zeros(d)
        tol = 1e-5 * abs_terms(*left) if rest else 0.0
        assert np.all(np.abs(got - expected) <= tol)


# Tiles of 4096 coordinates below 2^23, of 8192 from there on.
@pytest.mark.parametrize("d", [(1 << 23) - 1, 1 << 23, (1 << 23) + 4097])
def test_decode_on_both_sides_of_the_large_tiles(d):
    rng = np.random.default_rng(d)
    refs = []
    for c in range(3):
        u = np.zeros(d, dtype=np.float32)
        at = np.concatenate([rng.choice(d, 50_000, replace=False), np.arange(8192 * 3, 8192 * 4), np.arange(d - 5000, d)])
        u[at] = rng.standard_t(3, at.size).astype(np.float32)
        refs.append(orc.encode(u, orc.plan_manual(d, [32, 16, 3][: c + 1], [20_000, 10_000, 5_000][: c + 1]), 9, c).words)
    check_decode(refs, d)
    dev = [torch.from_numpy(s.view(np.int32)).to(DEV) for s in refs]
    start = rng.standard_normal(d).astype(np.float32)
    got, status = gpu_decode(dev, d, accumulate_into=torch.from_numpy(start.copy()).to(DEV))
    assert status == 0
    exact = start.astype(np.float64)
    for s in refs:
        exact += orc.decode_aggregate([s], d, weights=[1.0]).astype(np.float64) / 3.0
    assert np.all(np.abs(got - exact) <= 2.0 ** -23 * np.abs(exact) + 1e-12)


# --------------------------------------------------------------------------- batches of clients with different plans
def test_batch_with_mixed_plans():
    d = 150_000
    host, plans = [], []
    for c in range(6):
        host.append(syn.update_vector(2 if c % 2 else 3, c, d=d))
        R = [3, 7, 15, 16, 31, 1][c]
        plans.append(orc.plan_alg1(d, int(d * (0.4 + 0.3 * c)), R, -0.6, B=[1.0, 2.0, 1.0, 1.5, 1.0, 3.0][c]))
    ids = [10, 11, 12, 13, 14, 15]
    refs, _ = check_encode(host, plans, 99, ids)
    check_decode(refs, d)
    check_decode(refs, d, weights=[0.5, -1.0, 2.0, 0.25, 1.0, 1e-3])


def test_more_clients_than_the_chip_holds_workgroups_for():
    """96 clients: the per-(slot, client) launches are then larger than one resident set of workgroups, so
    workgroups that start late run after others of the same launch have finished."""
    d, n = 40_000, 96
    host, plans = [], []
    for c in range(n):
        host.append(syn.update_vector(3 if c % 3 else 2, 1000 + c, d=d))
        plans.append(orc.plan_alg1(d, int(d * (0.5 + 0.02 * (c % 11))), [15, 31, 4][c % 3], -0.6))
    refs, _ = check_encode(host, plans, 5, list(range(n)))
    check_decode(refs, d)


def test_more_clients_of_long_vectors_than_the_chip_holds_workgroups_for():
    """The same for vectors that pass the filter, whose gather and layout have a workgroup or more per client."""
    d, n = 66_001, 96
    host = [syn.update_vector(3 if c % 3 else 2, 1100 + c, d=d) for c in range(n)]
    plans = [orc.plan_manual(d, [max(1, 12 - r) for r in range(R)], [(d // 60 + 13 * (c % 5)) // R + r for r in range(R)])
             for c, R in ((c, (15, 31, 4)[c % 3]) for c in range(n))]
    refs, _ = check_encode(host, plans, 5, list(range(n)))
    check_decode(refs, d)


def test_more_streams_than_one_header_launch_takes():
    """130 streams: their pointers travel as kernel arguments, 112 a launch, so the headers are parsed by two
    launches and the lists numbered by a third (up to 112 streams one launch does both)."""
    d, n = 30_000, 130
    refs = []
    for c in range(n):
        U = syn.update_vector(2 + c % 2, 2000 + c, d=d)
        refs.append(orc.encode(U, orc.plan_fractions(d, [8, 4, 1], [0.01, 0.03, 0.05 + 0.001 * (c % 7)]), 9, c).words)
    check_decode(refs, d)
    rng = np.random.default_rng(3)
    check_decode(refs, d, weights=rng.uniform(-1.0, 1.0, n).astype(np.float32).tolist())


@pytest.mark.parametrize("cfg,d,n", [(2, 1_200_000, 8), (3, 700_001, 4), (4, 1_000_000, 4), (5, 800_000, 3)])
def test_workloads_at_oracle_friendly_sizes(cfg, d, n):
    w = syn.WORKLOADS[cfg]
    host = [syn.update_vector(cfg, c, d=d) for c in range(n)]
    plans = [orc.plan_for(w, client=c, alpha=orc.fit_alpha(host[c]), d=d) for c in range(n)]
    refs, _ = check_encode(host, plans, w.quant_seed, list(range(n)))
    check_decode(refs, d)


# --------------------------------------------------------------------------- the encoder's internal fallbacks
def test_sample_that_misjudges_the_threshold():
    """The encoder places its candidate threshold from a strided sample of 256-byte pieces.
    Here exactly the sampled pieces hold large values and everything else small ones, so the
    sampled threshold keeps far fewer than k coordinates and the keep-all pass has to run."""
    d = 2_000_000
    rng = np.random.default_rng(5)
    U = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    plant_on_the_sampled_pieces(U, rng)
    p = orc.plan_manual(d, [8, 4, 2], [50_000, 100_000, 150_000])   # k = 300 000 > the 262 144 large values
    refs, _ = check_encode([U], [p], 21, [3])
    check_decode(refs, d)


def test_workspace_sized_to_the_candidates():
    """A workspace with room for cvlc_plan_candidates_hint candidates (a fraction of the worst case)
    gives the very streams the worst-case workspace gives; a vector whose magnitudes are all equal has
    d candidates, so in that workspace it is refused (status bit, cleared first word) while the other
    clients of the batch are encoded as usual."""
    cfg, d, n = 3, 1_500_000, 3
    w = syn.WORKLOADS[cfg]
    host = [syn.update_vector(cfg, c, d=d) for c in range(n)]
    oplans = [orc.plan_for(w, client=c, alpha=orc.fit_alpha(host[c]), d=d) for c in range(n)]
    plans = [to_lib_plan(p) for p in oplans]
    cap = max(cv.plan_candidates_hint(p) for p in plans)
    k_max = max(sum(p.counts()) for p in oplans)
    assert k_max <= cap < d // 4
    small = cv.encode_workspace_bytes_for(d, n, cap)
    assert small < 0.6 * cv.encode_workspace_bytes(d, n)

    def run(updates_host, ws_bytes):
        updates = [torch.from_numpy(u).to(DEV) for u in updates_host]
        streams = [cv.new_stream_buffer(p, DEV) for p in plans]
        for s in streams:
            s.fill_(-1)
        ws = cv.new_workspace(ws_bytes, DEV)
        cv.encode_batch(plans, updates, w.quant_seed, list(range(n)), streams, ws)
        status = cv.device_status(ws)
        return [s.cpu().numpy().view(np.uint32)[: p.stream_bytes // 4] for s, p in zip(streams, plans)], status

    words, status = run(host, small)
    assert status == 0
    for c in range(n):
        assert_stream_equal(words[c], orc.encode(host[c], oplans[c], w.quant_seed, c).words, f"client {c}")

    flat = host[1].copy()
    flat[:] = np.where(np.arange(d) % 3 == 0, -0.25, 0.25).astype(np.float32)
    words, status = run([host[0], flat, host[2]], small)
    assert status == cv.DEV_WORKSPACE
    assert words[1][0] == 0
    for c in (0, 2):
        assert_stream_equal(words[c], orc.encode(host[c], oplans[c], w.quant_seed, c).words, f"client {c}")
    # the same batch in the worst-case workspace: every client encoded
    words, status = run([host[0], flat, host[2]], cv.encode_workspace_bytes(d, n))
    assert status == 0
    assert_stream_equal(words[1], orc.encode(flat, oplans[1], w.quant_seed, 1).words, "flat client")

    # less room than the largest k of the batch can never work: refused before anything is launched
    with pytest.raises(cv.CvlcError):
        run(host, cv.encode_workspace_bytes_for(d, n, k_max // 2))


def test_candidates_spread_thinly_over_many_regions():
    """Stretches where the encoder's 8192-coordinate regions keep one or two coordinates each: a span of 512
    candidates then crosses hundreds of runs (several windows of 64 run offsets), next to a dense stretch
    where it crosses one."""
    d = 6_000_000
    rng = np.random.default_rng(17)
    U = (rng.standard_normal(d) * 1e-5).astype(np.float32)
    thin = np.arange(0, 3_600_000, 8192) + rng.integers(0, 8192, size=440)       # one large value per region
    U[thin] = (rng.standard_normal(thin.size) * 3.0 + np.sign(rng.standard_normal(thin.size)) * 5.0).astype(np.float32)
    twice = np.arange(100, 1_600_000, 8192 * 2) + 4096                           # and a second one in every other
    U[twice] = (rng.standard_normal(twice.size) * 2.0 + 6.0).astype(np.float32)
    U[4_000_000:4_030_000] = (rng.standard_normal(30_000) * 4.0).astype(np.float32)   # the dense stretch
    U[5_999_000:] = (rng.standard_normal(1000) * 4.0).astype(np.float32)
    p = orc.plan_manual(d, [10, 6, 3, 1], [300, 700, 9_000, 20_000])
    refs, _ = check_encode([U, U[::-1].copy()], [p, p], 31, [0, 1])
    check_decode(refs, d)


def test_values_rounded_to_few_mantissa_bits():
    """Updates that were computed in a very short format: thousands of coordinates share each
    magnitude, so every boundary cuts through a large class of equal keys."""
    d = 400_000
    U = syn.update_vector(2, 3, d=d)
    U = (U.view(np.uint32) & np.uint32(0xFFF00000)).view(np.float32).copy()   # keep 3 mantissa bits
    p = orc.plan_manual(d, [8, 6, 4, 2], [4_000, 12_000, 30_000, 50_000])
    refs, _ = check_encode([U], [p], 77, [6])
    check_decode(refs, d)


def test_repeatable_and_without_statistics():
    d = 120_000
    host = [syn.update_vector(3, c, d=d) for c in range(3)]
    plans = [orc.plan_alg1(d, d, 5, -0.6)] * 3
    a, _, sa, streams = gpu_encode(host, plans, 4, [0, 1, 2], want_stats=False)
    b, _, sb, _ = gpu_encode(host, plans, 4, [0, 1, 2], want_stats=True)
    assert sa == 0 and sb == 0
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    out1, st1 = gpu_decode(streams, d)
    out2, st2 = gpu_decode(streams, d)
    assert st1 == 0 and st2 == 0
    # the order of the fp64 additions may differ between runs: the rounded sum of a coordinate that three or
    # more lists meet in may then differ by one unit in the last place (about once in 2^29 such coordinates)
    gap = np.abs(out1.view(np.int32).astype(np.int64) - out2.view(np.int32).astype(np.int64))
    assert gap.max() <= 1 and np.count_nonzero(gap) <= 2


# --------------------------------------------------------------------------- decode / aggregate specifics
def test_decode_accumulate_mode_and_empty_batch():
    d = 90_000
    refs = []
    for c in range(5):
        U = syn.update_vector(2, c, d=d)
        refs.append(orc.encode(U, orc.plan_fractions(d, [8, 3], [0.02, 0.1]), 7, c).words)
    wts = [1.0, 0.5, 0.25, 2.0, 4.0]
    dev = [torch.from_numpy(s.view(np.int32)).to(DEV) for s in refs]
    first, st = gpu_decode(dev[:2], d, weights=wts[:2])
    assert st == 0
    acc = torch.from_numpy(first.copy()).to(DEV)
    both, st = gpu_decode(dev[2:], d, weights=wts[2:], accumulate_into=acc)
    assert st == 0
    ref_first = orc.decode_aggregate(refs[:2], d, weights=wts[:2])
    ref = orc.decode_aggregate(refs[2:], d, weights=wts[2:], out=ref_first.copy())
    tol = 1e-5 * abs_terms(refs, d, wts) + 1e-30
    assert np.all(np.abs(both.astype(np.float64) - ref) <= tol)
    none, st = gpu_decode([], d)
    assert st == 0 and np.all(none == 0)


def test_malformed_streams_set_status_and_stay_in_bounds():
    d = 40_000
    U = syn.update_vector(1, 0, d=d)
    good = orc.encode(U, orc.plan_fractions(d, [8, 2], [0.05, 0.2]), 1, 0).words
    cases = []
    w = good.copy(); w[0] ^= 1; cases.append(w)                           # magic
    w = good.copy(); w[2] = d + 1; cases.append(w)                        # other model size
    w = good.copy(); w[8] = 17; cases.append(w)                           # unsupported code length
    w = good.copy(); w[9] += 1; cases.append(w)                           # count does not match the length
    w = good.copy(); w[16] |= (1 << 16) - 1; cases.append(w)              # first PID = 65535 >= d
    w = good.copy(); w[16:20] = good[40:44]; cases.append(w)              # positions out of order
    for w in cases:
        with pytest.raises(orc.OracleError):
            orc.decode_aggregate([w], d)
        out, status = gpu_decode([torch.from_numpy(w.view(np.int32)).to(DEV)], d)
        assert status & cv.DEV_STREAM
        assert np.all(np.isfinite(out))
    out, status = gpu_decode([torch.from_numpy(good.view(np.int32)).to(DEV)], d)   # the untouched stream still decodes
    assert status == 0


def build_stream(d, groups, quant=cv.QUANT_PQ, client=0):
    """A stream written by hand: groups of (code length, ascending positions, codes, first and second header value)."""
    s = max(1, (d - 1).bit_length())
    words = [np.array([0x434C5643, 1 | quant << 16, d, len(groups), s, np.float32(1.0).view(np.uint32), client, 0], dtype=np.uint64)]
    payloads = []
    for y, pos, codes, a, b in groups:
        words.append(np.array([y, len(pos), np.float32(a).view(np.uint32), np.float32(b).view(np.uint32)], dtype=np.uint64))
        W, n = s + y, len(pos)
        rec = np.asarray(pos, np.uint64) | np.asarray(codes, np.uint64) << np.uint64(s)
        bit = np.arange(n, dtype=np.uint64) * np.uint64(W)
        bits = np.zeros(((n * W + 31) // 32 + 3) * 32, dtype=np.uint8)
        for i in range(W):
            bits[bit + np.uint64(i)] = (rec >> np.uint64(i)) & np.uint64(1)
        payloads.append(np.packbits(bits, bitorder="little").view(np.uint32)[: (n * W + 31) // 32].astype(np.uint64))
    out = np.concatenate(words + payloads).astype(np.uint32)
    out[7] = out.size
    return out


def check_decode_ulp(refs, d, quant=cv.QUANT_PQ):
    got, status = gpu_decode([torch.from_numpy(s.view(np.int32)).to(DEV) for s in refs], d, quant=quant)
    assert status == 0
    ref = orc.decode_aggregate(refs, d).astype(np.float64)
    # fp64 sums in free order, rounded to fp32 once: half a unit of the last place on either side
    assert np.all(np.abs(got - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12 * abs_terms(refs, d))


# Positions of more than 25 bits are read by eight bytes and, where a raw code follows, a ninth: 1 .. 8 streams (headers, numbers and
# table in one launch), 9 and 26 of them (two and three launches).
@pytest.mark.parametrize("quant", [cv.QUANT_PQ, cv.QUANT_QSGD])
@pytest.mark.parametrize("n", [1, 3, 8, 9, 26])
def test_decode_positions_of_26_bits(n, quant):
    d = (1 << 25) + 12_345
    rng = np.random.default_rng(n)
    refs = []
    for c in range(n):
        groups = [(32, [d - 1 - c], [np.float32(0.5 + c).view(np.uint32)], 1.0, 0.0)]     # one record, in the last tile
        for y, count in ((32, 500), (16, 3000), (7, 1), (2, 2000)):
            pos = np.sort(np.unique(np.concatenate([rng.integers(0, d, count), [c, d - 1]]))) if count > 1 else [d // 2 + c]
            codes = rng.standard_normal(len(pos)).astype(np.float32).view(np.uint32) if y == 32 else rng.integers(0, 1 << y, len(pos))
            groups.append((y, pos, codes, *((2.0, 0.0) if quant else (-1.0, 1.5))))
        groups.append((3, np.arange(8192 * 7 - 1, 8192 * 8 + 1), rng.integers(0, 8, 8194), *((2.0, 0.0) if quant else (-1.0, 1.5))))   # a whole tile
        refs.append(build_stream(d, groups, quant, c))
    check_decode_ulp(refs, d, quant)


# Tiles of 8192 coordinates with lists dealt out to 1, 2, 4 and 8 groups of wavefronts and to two sweeps.
@pytest.mark.parametrize("n,R", [(1, 31), (8, 8), (5, 25), (9, 28), (17, 31)])
def test_decode_large_tiles_of_many_lists(n, R):
    d = (1 << 23) + 77
    rng = np.random.default_rng(n * 100 + R)
    refs = []
    for c in range(n):
        groups = []
        for r in range(R):
            pos = np.unique(rng.integers(0, d, int(rng.integers(0, 3000))))
            if (c + r) % 9 == 0:                                   # every coordinate of a tile and of the last one
                pos = np.unique(np.concatenate([pos, np.arange(8192 * (5 + r) - 1, 8192 * (6 + r) + 1), np.arange(d - 700, d)]))
            y = max(1, 16 - r // 2)
            groups.append((y, pos, rng.integers(0, 1 << y, len(pos)), -0.5 - r, 2.0 + r))
        refs.append(build_stream(d, groups, client=c))
    check_decode_ulp(refs, d)


# One malformed stream among good ones: 1 + 1 (headers, numbers and table in one launch), 1 + 8 (numbered by the launch that parses)
# and 1 + 27 (by a launch of its own), tiles of 4096 and of 8192 coordinates.
@pytest.mark.parametrize("n_good", [1, 8, 27])
@pytest.mark.parametrize("d", [40_000, (1 << 23) + 77])
def test_a_malformed_stream_among_good_ones(d, n_good):
    rng = np.random.default_rng(d + n_good)
    s = (d - 1).bit_length()

    def one(client):
        groups = []
        for y in (9, 4):
            pos = np.unique(np.concatenate([rng.integers(0, d, 3000), np.arange(9000, 9500)]))
            groups.append((y, pos, rng.integers(0, 1 << y, len(pos)), -1.0, 1.5))
        return build_stream(d, groups, client=client)

    good = [one(c) for c in range(n_good)]
    base = one(99)
    weights = rng.uniform(0.5, 1.5, n_good + 1).tolist()
    expected = orc.decode_aggregate(good, d, weights=weights[:n_good]).astype(np.float64)
    tol = 2.0 ** -22 * np.abs(expected) + 1e-12
    headers, records = [], []
    for at, value in ((0, 1), (1, 2 << 16), (2, 1), (3, 64), (4, 1), (5, 0x80000000), (7, 1), (8, 16), (9, 1), (10, 0x40000000)):
        w = base.copy()
        w[at] ^= np.uint32(value)
        headers.append(w)
    w = base.copy(); w[16] |= np.uint32((1 << s) - 1); records.append(w)      # first position >= d
    w = base.copy(); w[16:40] = base[40:64]; records.append(w)                 # positions out of order
    for w in headers + records:
        with pytest.raises(orc.OracleError):
            orc.decode_aggregate([w], d)
        streams = [torch.from_numpy(x.view(np.int32)).to(DEV) for x in good + [w]]
        got, status = gpu_decode(streams, d, weights=weights)
        assert status & cv.DEV_STREAM
        assert np.all(np.isfinite(got))
        if any(w is h for h in headers):                          # contributes nothing; the others add up
            assert np.all(np.abs(got - expected) <= tol)
    got, status = gpu_decode([torch.from_numpy(x.view(np.int32)).to(DEV) for x in good + [base]], d, weights=weights)
    assert status == 0                                            # the untouched stream decodes


@pytest.mark.parametrize("d,n", [(1_200_007, 1), (5_000_000, 1), (5_000_000, 3), (9_000_001, 1), (9_000_001, 5)])
def test_a_position_twice_anywhere_in_a_long_stream(d, n):
    """Two equal positions in a row are seen by the table's pass only, in one of up to 2048 workgroups; what those find lies in the
    place of the list descriptors or where the table ends.  Records of 32 bits, a word each."""
    s = (d - 1).bit_length()
    plan = cv.plan_manual(d, [32 - s], [d // 2])
    streams = [cv.new_stream_buffer(plan, DEV) for _ in range(n)]
    ws = cv.new_workspace(cv.encode_workspace_bytes(d, n), DEV)
    cv.encode_batch([plan] * n, [torch.randn(d, device=DEV, generator=torch.Generator(DEV).manual_seed(c)) for c in range(n)], 3,
                    list(range(n)), streams, ws)
    clean, status = gpu_decode(streams, d)
    assert status == 0
    words = streams[-1]
    for e in (1, 511, 512, 513, d // 6, d // 4 + 1, d // 2 - 513, d // 2 - 1):
        kept = words[12 + e].item()
        words[12 + e] = words[11 + e]
        got, status = gpu_decode(streams, d)
        assert status == cv.DEV_STREAM, e
        # fp64 sums in free order, each rounded to fp32 once: a unit of the last place, but for the coordinate hit twice and the one left
        # out (several streams' values may cancel: the terms are below 4, fp64 keeps 2^-50 of them)
        assert np.count_nonzero(np.abs(got - clean) > 2.0 ** -23 * np.abs(clean) + 2.0 ** -48) <= 2
        words[12 + e] = kept


@pytest.mark.parametrize("d", [30_000, 70_001])
def test_non_finite_update_sets_status(d):
    p = orc.plan_fractions(d, [8], [0.1])
    for bad in (np.nan, np.inf, -np.inf):
        U = syn.update_vector(1, 0, d=d)
        U[12_345] = bad
        _, _, status, _ = gpu_encode([U], [p], 1, [0], want_stats=False)
        assert status & cv.DEV_NONFINITE
        with pytest.raises(orc.OracleError):
            orc.encode(U, p, 1, 0)


@pytest.mark.parametrize("d", [9001, 40_003, SHORT_MAX - 1, 70_001])
def test_nan_of_the_largest_patterns(d):
    """The largest keys there are, at a boundary, in vectors whose last visit has lanes to spare: reported, and the groups
    have their sizes all the same (the selection goes by bit patterns)."""
    rng = np.random.default_rng(d)
    U = rng.standard_normal(d).astype(np.float32)
    at = rng.choice(d, 230, replace=False)
    U.view(np.uint32)[at[:30]] = 0x7FFFFFFF
    U.view(np.uint32)[at[30:]] = 0xFFFE1234
    p = to_lib_plan(orc.plan_manual(d, [8, 4], [100, 500]))
    stream = cv.new_stream_buffer(p, DEV)
    ws = cv.new_workspace(cv.encode_workspace_bytes(d, 1), DEV)
    ws.fill_(255)
    cv.encode_batch([p], [torch.from_numpy(U).to(DEV)], 3, [1], [stream], ws)
    assert cv.device_status(ws) == cv.DEV_NONFINITE


# --------------------------------------------------------------------------- seeded random sweep
def test_random_plans_sizes_and_quantisers():
    """150 seeded combinations of length, group count, code lengths (raw, empty and 1-bit groups
    included), group sizes from a handful to everything, scale factor, quantiser, client ids and
    vector family: streams, statistics and error energy, aggregate, packets and their reassembly,
    the exponent fit."""
    rng = np.random.default_rng(int(os.environ.get("CVLC_SWEEP_SEED", "20240203")))   # another seed: another 150 cases
    for case in range(150):
        d = int(rng.choice([1, 2, 7, 63, 64, 65, 511, 4097, 8192, 8193, 20_000, 70_001, 131_072]))
        quant = int(rng.integers(0, 2))
        R = int(rng.integers(1, 9)) if rng.random() < 0.7 else int(rng.integers(9, 32))   # beyond 15: several selection rounds
        pool = [2, 3, 4, 6, 8, 11, 16, 32] if quant else [1, 2, 3, 4, 6, 8, 11, 16, 32]
        ys = sorted(rng.choice(pool, size=R).tolist(), reverse=True)
        k = int(rng.integers(0, d + 1)) if rng.random() < 0.3 else int(rng.integers(0, max(1, d // 8) + 1))
        cuts = np.sort(rng.integers(0, k + 1, size=R - 1)) if R > 1 else np.array([], dtype=np.int64)
        counts = np.diff(np.concatenate([[0], cuts, [k]])).astype(int).tolist()
        B = float(rng.choice([1.0, 1.0, 2.5, 40.0]))
        po = orc.plan_manual(d, ys, counts, B=B, quant=quant)
        n = int(rng.integers(1, 4))
        kind = rng.choice(["cfg1", "cfg3", "few_levels", "zeros_and_denormals"])
        host = []
        for c in range(n):
            if kind.startswith("cfg"):
                host.append(syn.update_vector(int(kind[3]), 100 * case + c, d=d))
            else:
                host.append(syn.tie_heavy_vector(str(kind), d, seed=100 * case + c))
        ids = [int(v) for v in rng.integers(0, 2**32, size=n)]
        seed = int(rng.integers(0, 2**63))
        what = f"case {case}: d={d} quant={quant} y={ys} P={counts} B={B} {kind} n={n}"
        words, stats, status, streams = gpu_encode(host, [po] * n, seed, ids, error_stats=True)
        assert status == 0, what
        refs = []
        for c in range(n):
            ref = orc.encode(host[c], po, seed, ids[c])
            assert_stream_equal(words[c], ref.words, what + f" client {c}")
            assert_stats_close(stats[c], ref.stats, po.R, error_stats=True)
            refs.append(ref.words)
        got, status = gpu_decode(streams, d, quant=quant)
        assert status == 0, what
        ref = orc.decode_aggregate(refs, d)
        assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= 1e-5 * abs_terms(refs, d)), what
        # caller's weights (either sign), added to what the output holds
        wts = [float(np.float32(v)) for v in rng.uniform(-2.0, 2.0, size=n)]
        start = rng.standard_normal(d).astype(np.float32)
        acc, status = gpu_decode(streams, d, weights=wts, accumulate_into=torch.from_numpy(start.copy()).to(DEV), quant=quant)
        assert status == 0, what
        ref = orc.decode_aggregate(refs, d, weights=wts, out=start.copy())
        tol = 1e-5 * (abs_terms(refs, d, weights=wts) + np.abs(start.astype(np.float64)))
        assert np.all(np.abs(acc.astype(np.float64) - ref.astype(np.float64)) <= tol), what
        mtu = int(rng.choice([64, 1500]))
        pl = to_lib_plan(po)
        buf, npk = gpu_packetize(pl, streams[0], mtu)
        ref_pk, _ = orc.packetize(refs[0], d, mtu)
        assert np.array_equal(buf.cpu().numpy().view(np.uint32)[: npk * mtu // 4].reshape(npk, mtu // 4), ref_pk), what
        out, status = gpu_depacketize(buf.view(-1, mtu // 4)[:npk].flip(0).contiguous(), npk, d, mtu, refs[0].size)
        assert status == 0 and np.array_equal(out.cpu().numpy().view(np.uint32), refs[0]), what
        check_fit(host)


# --------------------------------------------------------------------------- the caller's stream
@pytest.mark.parametrize("d", [150_001, 40_001])
def test_every_call_runs_on_the_callers_stream(d):
    """All work is enqueued on the stream handed in: on a side stream, behind a long-running
    kernel that produces the input, results are right without any device-wide synchronisation."""
    n = 2
    host = [syn.update_vector(2, c, d=d) for c in range(n)]
    po = orc.plan_alg1(d, d, 5, -0.6)
    pl = to_lib_plan(po)
    side = torch.cuda.Stream()
    staged = [torch.from_numpy(u).to(DEV) for u in host]
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        filler = torch.empty(1 << 28, dtype=torch.float32, device=DEV)
        for _ in range(4):
            filler.normal_()                                       # keeps the side stream busy for a while
        updates = [u * 1.0 for u in staged]                        # the inputs exist only once the side stream gets here
        streams = [cv.new_stream_buffer(pl, DEV) for _ in range(n)]
        ws = cv.new_workspace(cv.encode_workspace_bytes(d, n), DEV)
        cv.encode_batch([pl] * n, updates, 8, [0, 1], streams, ws)
        out = torch.empty(d, dtype=torch.float32, device=DEV)
        dws = cv.new_workspace(cv.decode_workspace_bytes(d, n), DEV)
        cv.decode_aggregate(streams, out, dws)
        alpha = torch.empty(n, dtype=torch.float64, device=DEV)
        fws = cv.new_workspace(cv.fit_workspace_bytes(n), DEV)
        cv.fit_alpha(updates, alpha, fws)
        npk = cv.packet_count(pl, 1500)
        pk = torch.empty(npk * 375, dtype=torch.int32, device=DEV)
        cv.packetize(pl, streams[1], pk)
        back = torch.empty_like(streams[1])
        pws = cv.new_workspace(cv.depacketize_workspace_bytes(npk), DEV)
        cv.depacketize(pk, npk, d, back, pws)
        assert cv.device_status(ws) == 0 and cv.device_status(dws) == 0 and cv.device_status(pws) == 0
        assert cv.device_status(fws) == 0                          # each waits for the side stream only
        refs = [orc.encode(u, po, 8, c).words for c, u in enumerate(host)]
        for c in range(n):
            assert_stream_equal(streams[c].cpu().numpy().view(np.uint32)[: refs[c].size], refs[c], f"client {c}")
        assert np.array_equal(back.cpu().numpy().view(np.uint32)[: refs[1].size], refs[1])
        ref = orc.decode_aggregate(refs, d)
        assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * abs_terms(refs, d))
        assert alpha.cpu().numpy().tolist() == pytest.approx([orc.fit_alpha(u) for u in host], rel=1e-11)
    torch.cuda.synchronize()
    del filler


@pytest.mark.parametrize("d", [90_001, 30_001])
def test_calls_can_be_captured_in_a_graph_and_replayed(d):
    """The calls only launch kernels on the caller's stream (clears included), so a step can be
    recorded once and replayed: three replays on fresh inputs, with eager work and
    synchronisation in between, each checked against the oracle."""
    n = 3
    po = orc.plan_manual(d, [10, 5, 2], [900, 4000, 9000])
    pl = to_lib_plan(po)
    updates = [torch.zeros(d, dtype=torch.float32, device=DEV) for _ in range(n)]
    streams = [cv.new_stream_buffer(pl, DEV) for _ in range(n)]
    ws = cv.new_workspace(cv.encode_workspace_bytes(d, n), DEV)
    dws = cv.new_workspace(cv.decode_workspace_bytes(d, n), DEV)
    fws = cv.new_workspace(cv.fit_workspace_bytes(n), DEV)
    out = torch.empty(d, dtype=torch.float32, device=DEV)
    alpha = torch.empty(n, dtype=torch.float64, device=DEV)

    def step():
        cv.encode_batch([pl] * n, updates, 21, [0, 1, 2], streams, ws)
        cv.decode_aggregate(streams, out, dws)
        cv.fit_alpha(updates, alpha, fws)

    for c in range(n):
        updates[c].copy_(torch.from_numpy(syn.update_vector(1, c, d=d)))
    step()                                                         # first use outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        host = [syn.update_vector(2 + rep % 2, 10 * rep + c, d=d) for c in range(n)]
        for c in range(n):
            updates[c].copy_(torch.from_numpy(host[c]))
        out.fill_(float("nan"))
        for s_ in streams:
            s_.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert cv.device_status(ws) == 0 and cv.device_status(dws) == 0 and cv.device_status(fws) == 0
        refs = [orc.encode(u, po, 21, c).words for c, u in enumerate(host)]
        for c in range(n):
            assert_stream_equal(streams[c].cpu().numpy().view(np.uint32)[: refs[c].size], refs[c], f"replay {rep} client {c}")
        ref = orc.decode_aggregate(refs, d)
        assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * abs_terms(refs, d)), rep
        assert alpha.cpu().numpy().tolist() == pytest.approx([orc.fit_alpha(u) for u in host], rel=1e-11)


# --------------------------------------------------------------------------- error energy, scale factor across rounds
def test_error_statistics_and_the_scale_factor_carried_across_rounds():
    """Round t uses B from round t-1's plan (footnote to Proposition 1); the encoder reports the
    error energy of quantisation + scaling per group (Lemma 1's left side), from which the
    empirical gamma follows; the parameter server divides by B."""
    d, n, seed = 300_007, 3, 99
    host = [syn.update_vector(3, c, d=d) for c in range(n)]
    host[2] = syn.tie_heavy_vector("few_levels", d, seed=2)
    B = 1.0
    for rnd in range(2):
        plans = [orc.plan_manual(d, [32, 10, 4, 2, 1], [500, 3000, 6000, 9000, 12000], B=B),
                 orc.plan_alg1(d, d, 6, -0.6, B=B),
                 orc.plan_manual(d, [5, 1], [10_000, 20_001], B=B)]
        words, stats, status, streams = gpu_encode(host, plans, seed + rnd, [4, 5, 6], error_stats=True)
        assert status == 0
        plain, plain_stats, _, _ = gpu_encode(host, plans, seed + rnd, [4, 5, 6])
        for c in range(n):
            ref = orc.encode(host[c], plans[c], seed + rnd, 4 + c)
            assert_stream_equal(words[c], ref.words, f"round {rnd} client {c}")
            assert_stream_equal(plain[c], ref.words, f"round {rnd} client {c}, no error statistics")
            assert_stats_close(stats[c], ref.stats, plans[c].R, error_stats=True)
            assert_stats_close(plain_stats[c], ref.stats, plans[c].R)
            assert cv.stats_gamma(stats[c], plans[c].R) == pytest.approx(orc.empirical_gamma(ref.stats, plans[c].R), rel=1e-6)
        got, status = gpu_decode(streams, d)
        assert status == 0
        ref_words = [orc.encode(host[c], plans[c], seed + rnd, 4 + c).words for c in range(n)]
        ref = orc.decode_aggregate(ref_words, d)
        assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= 1e-5 * abs_terms(ref_words, d))
        nxt = [cv.plan_next_scale(to_lib_plan(p)) for p in plans]
        assert nxt == [orc.next_scale(p) for p in plans]
        B = float(np.float32(max(nxt)))   # one factor for the round, as the paper's constant B
    assert B > 1.0


# --------------------------------------------------------------------------- QSGD, the second quantiser
def check_qsgd(host, plans, seed, ids, weights=None):
    """Streams bit for bit (header norms included), statistics, error energy, aggregate."""
    d = host[0].size
    words, stats, status, streams = gpu_encode(host, plans, seed, ids, error_stats=True)
    assert status == 0
    refs = []
    for c, (u, p) in enumerate(zip(host, plans)):
        ref = orc.encode(u, p, seed, ids[c])
        assert_stream_equal(words[c], ref.words, f"client {c}")
        assert_stats_close(stats[c], ref.stats, p.R, error_stats=True)
        refs.append(ref.words)
    got, status = gpu_decode(streams, d, weights=weights, quant=cv.QUANT_QSGD)
    assert status == 0
    ref = orc.decode_aggregate(refs, d, weights=weights)
    n = len(host)
    tol = np.zeros(d)
    for i, s in enumerate(refs):
        w = abs(float(np.float32(weights[i]))) if weights is not None else 1.0 / (n * float(s[5:6].view(np.float32)[0]))
        tol += np.abs(orc.decode_aggregate([s], d, weights=[1.0]).astype(np.float64)) * w
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= 1e-5 * tol)
    if n == 1 and weights is None:
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    return streams


def test_qsgd_on_the_workload_distributions():
    d = 200_003
    host = [syn.update_vector(3, c, d=d) for c in range(4)]
    plans = [orc.plan_manual(d, [32, 12, 7, 4, 2], [300, 2000, 5000, 9000, 14000], quant=orc.QSGD),
             orc.plan_manual(d, [16, 8, 5, 3, 2], [1000, 3000, 7000, 11000, 20001], B=1.5, quant=orc.QSGD),
             orc.plan_manual(d, [2], [50_000], quant=orc.QSGD),
             orc.plan_manual(d, [9, 9, 9], [1, 0, 4097], quant=orc.QSGD)]
    check_qsgd(host, plans, 31, [9, 8, 7, 6])
    check_qsgd(host[:1], plans[:1], 32, [0])
    check_qsgd(host[:2], plans[:2], 33, [1, 2], weights=[0.25, -2.0])
    check_qsgd([syn.update_vector(1, 0)], [orc.plan_manual(65_536, [8, 4, 2], [6553, 9831, 16384], quant=orc.QSGD)], 34, [3])


@pytest.mark.parametrize("kind", ["all_equal_mixed_sign", "few_levels", "zeros_and_denormals", "all_zero"])
def test_qsgd_on_colliding_magnitudes_and_extreme_exponents(kind):
    """Ties, signed zeros, denormals (squares down at 2^-298) and, in one vector, magnitudes from
    1e-38 to 1e18: every limb of the exact sum of squares is exercised."""
    d = 30_011
    U = syn.tie_heavy_vector(kind, d, seed=5)
    plans = [orc.plan_manual(d, [10, 4, 2], [2000, 6000, 12_000], quant=orc.QSGD)]
    check_qsgd([U], plans, 41, [2])
    rng = np.random.default_rng(43)
    wide = (rng.standard_normal(d) * 10.0 ** rng.uniform(-38, 18, d)).astype(np.float32)
    check_qsgd([wide, -wide[::-1].copy()], plans * 2, 42, [0, 1])


@pytest.mark.parametrize("d", [10_000, 70_001])
def test_qsgd_norm_overflow_and_mismatched_quantiser_are_reported(d):
    U = np.full(d, 3.0e38, dtype=np.float32)                       # every square is finite in the limbs, the norm is not
    p = orc.plan_manual(d, [8], [100], quant=orc.QSGD)
    _, _, status, _ = gpu_encode([U], [p], 1, [0], want_stats=False)
    assert status & cv.DEV_NONFINITE
    with pytest.raises(orc.OracleError):
        orc.encode(U, p, 1, 0)
    V = syn.update_vector(1, 0, d=d)
    _, _, status, streams = gpu_encode([V], [p], 1, [0], want_stats=False)
    assert status == 0
    _, status = gpu_decode(streams, d)                             # the server expects PQ streams
    assert status & cv.DEV_STREAM
    pq = orc.plan_manual(d, [8], [100])
    _, _, _, streams = gpu_encode([V], [pq], 1, [0], want_stats=False)
    out, status = gpu_decode(streams, d, quant=cv.QUANT_QSGD)      # and the other way round
    assert status & cv.DEV_STREAM and not out.any()
    with pytest.raises(cv.CvlcError):                              # one quantiser per batch
        gpu_encode([V, V], [p, pq], 1, [0, 1], want_stats=False)
    with pytest.raises(cv.CvlcError):
        cv.plan_manual(d, [4, 1], [10, 10], quant=cv.QUANT_QSGD)


# --------------------------------------------------------------------------- packets
def gpu_packetize(plan_lib, stream_dev, mtu):
    n = cv.packet_count(plan_lib, mtu)
    buf = torch.full((max(n, 1) * mtu // 4,), -1, dtype=torch.int32, device=DEV)   # every word of every slot is written
    cv.packetize(plan_lib, stream_dev, buf, mtu)
    torch.cuda.synchronize()
    return buf, n


def gpu_depacketize(packets_dev, n, d, mtu, cap_words):
    out = torch.full((cap_words,), -1, dtype=torch.int32, device=DEV)
    ws = cv.new_workspace(cv.depacketize_workspace_bytes(n), DEV)
    ws.fill_(0x5A)
    cv.depacketize(packets_dev, n, d, out, ws, mtu)
    return out, cv.device_status(ws)


@pytest.mark.parametrize("mtu", [1500, 64, 9000])
def test_packets_match_the_oracle_and_reassemble(mtu):
    """Sender: the packets of a GPU-encoded stream are the oracle's, byte for byte.  Receiver: from
    the packets in shuffled order the stream comes back bit for bit and decodes as before."""
    d = 120_011
    host = [syn.update_vector(3, 0, d=d), syn.tie_heavy_vector("few_levels", d, seed=1)]
    plans = [orc.plan_manual(d, [32, 11, 5, 2, 1], [200, 3000, 0, 9000, 17_001], B=2.0),
             orc.plan_manual(d, [7, 3], [1, 40_000], quant=orc.QSGD)]
    for U, po in zip(host, plans):
        words, _, status, streams = gpu_encode([U], [po], 17, [12], want_stats=False)
        assert status == 0
        ref_pk, ref_sizes = orc.packetize(words[0], d, mtu)
        pl = to_lib_plan(po)
        buf, n = gpu_packetize(pl, streams[0], mtu)
        assert n == ref_pk.shape[0]
        got = buf.cpu().numpy().view(np.uint32).reshape(n, mtu // 4)
        assert np.array_equal(got, ref_pk)
        assert [cv.packet_size(pl, i, mtu) for i in range(n)] == ref_sizes.tolist()
        g = torch.Generator(device="cpu")
        g.manual_seed(5)
        shuffled = buf.view(n, mtu // 4)[torch.randperm(n, generator=g).to(DEV)].contiguous()
        out, status = gpu_depacketize(shuffled, n, d, mtu, words[0].size + 7)
        assert status == 0
        back = out.cpu().numpy().view(np.uint32)
        assert np.array_equal(back[: words[0].size], words[0])
        assert np.array_equal(back[: words[0].size], orc.depacketize(ref_pk, d, mtu))
        assert np.all(back[words[0].size:] == 0xFFFFFFFF)                      # nothing written behind the stream
        dec, status = gpu_decode([out], d, quant=int(po.quant))
        assert status == 0
        assert np.array_equal(dec.view(np.uint32), orc.decode_aggregate([words[0]], d).view(np.uint32))


def test_reassembly_refuses_loss_duplicates_tampering_and_short_buffers():
    d, mtu = 50_000, 1500
    U = syn.update_vector(1, 1, d=d)
    po = orc.plan_manual(d, [12, 6, 3], [700, 0, 9000])
    words, _, _, streams = gpu_encode([U], [po], 3, [1], want_stats=False)
    buf, n = gpu_packetize(to_lib_plan(po), streams[0], mtu)
    pk = buf.view(n, mtu // 4)
    cap = words[0].size
    out, status = gpu_depacketize(pk.contiguous(), n, d, mtu, cap)
    assert status == 0 and np.array_equal(out.cpu().numpy().view(np.uint32), words[0])

    def refused(packets, count, cap_words=cap):
        out, status = gpu_depacketize(packets.contiguous(), count, d, mtu, cap_words)
        got = out.cpu().numpy().view(np.uint32)
        with pytest.raises(orc.OracleError):
            orc.depacketize(packets.cpu().numpy().view(np.uint32)[:count], d, mtu, cap_words=cap_words)
        return bool(status & cv.DEV_STREAM) and got[0] == 0

    assert refused(pk[:-1], n - 1)                                             # a packet is missing
    assert refused(torch.cat([pk, pk[3:4]]), n + 1)                            # one arrives twice
    assert refused(torch.cat([pk[:5], pk[4:5], pk[6:]]), n)                    # one replaced by a copy of another
    for word, value in ((0, 1), (2, d - 1), (4, 0), (6, int(pk[4, 6]) + 1), (7, 1), (8, 0)):
        bad = pk.clone()
        bad[4, word] = value
        assert refused(bad, n), word
    bad = pk.clone()
    bad[4, 5] = int(pk[4, 5]) ^ (1 << 16)                                      # another code length
    assert refused(bad, n)
    assert refused(pk, n, cap_words=cap - 1)                                   # the stream does not fit
    # the tail of a packet's payload is not trusted: junk behind the records does not reach the stream
    junk = pk.clone()
    last = n - 1                                                               # last packet of the last group
    size = cv.packet_size(to_lib_plan(po), last, mtu) // 4
    junk[last, size:] = -1
    out, status = gpu_depacketize(junk.contiguous(), n, d, mtu, cap)
    assert status == 0 and np.array_equal(out.cpu().numpy().view(np.uint32), words[0])


def test_packets_at_the_benchmark_size():
    """One client of cfg 3 at d = 11.2 M: 1.4 MB stream, 15 groups, about 950 packets of 1500 bytes."""
    w = syn.WORKLOADS[3]
    d = w.d
    U = syn.update_vector(3, 5)
    po = orc.plan_for(w, client=0, alpha=-0.5)
    words, _, status, streams = gpu_encode([U], [po], w.quant_seed, [5], want_stats=False)
    assert status == 0
    ref_pk, _ = orc.packetize(words[0], d, 1500)
    buf, n = gpu_packetize(to_lib_plan(po), streams[0], 1500)
    assert np.array_equal(buf.cpu().numpy().view(np.uint32).reshape(n, 375), ref_pk)
    out, status = gpu_depacketize(buf.view(n, 375).flip(0).contiguous(), n, d, 1500, words[0].size)
    assert status == 0 and np.array_equal(out.cpu().numpy().view(np.uint32), words[0])


@pytest.mark.parametrize("mtu,packets", [(552, 300), (556, 300), (1576, 2047), (1576, 2049), (1580, 2049)])
def test_packets_at_the_steps_of_their_kernels(mtu, packets):
    """A packet is moved by one wavefront up to 128 words behind its header, up to 384 where there are more than 2048 of them, and
    by four else."""
    s = 21
    d = (1 << s) - 3
    cap = (8 * mtu - 320) // (s + 9)
    po = orc.plan_manual(d, [9, 9, 9], [cap * (packets - 7) - 1, 2 * cap, 4 * cap + 1])
    words, _, status, streams = gpu_encode([syn.update_vector(2, 3, d=d)], [po], 4, [2], want_stats=False)
    assert status == 0
    pl = to_lib_plan(po)
    buf, n = gpu_packetize(pl, streams[0], mtu)
    ref, _ = orc.packetize(words[0], d, mtu)
    assert n == packets and np.array_equal(buf.cpu().numpy().view(np.uint32)[: ref.size], ref.ravel())
    out, status = gpu_depacketize(buf.view(-1, mtu // 4)[:n].flip(0).contiguous(), n, d, mtu, words[0].size)
    assert status == 0
    assert np.array_equal(out.cpu().numpy().view(np.uint32)[: words[0].size], words[0])


@pytest.mark.parametrize("bits", [23, 24, 26])
def test_more_packets_than_a_grid_holds_threads_for(bits):
    """A grid has less than 2^32 threads, and the launch of one of more starts the rest of that division without an error: four
    wavefronts to 2^24 packets left all but five of them out, one to 2^26 too.  The stream's records are any bits: neither
    side looks at them."""
    d, mtu, n = (1 << 30) + 1, 64, (1 << bits) + 5
    plan = cv.plan_manual(d, [13], [4 * n - 1])                # 44 bits a record, four to a packet
    assert cv.packet_count(plan, mtu) == n
    stream = torch.randint(-2 ** 31, 2 ** 31 - 1, (plan.stream_bytes // 4,), dtype=torch.int32, device=DEV)
    header = [0x434C5643, 1, d, 1, 31, np.float32(1.0).view(np.uint32), 7, plan.stream_bytes // 4, 13, 4 * n - 1, 0, 0]
    stream[:12] = torch.from_numpy(np.array(header, dtype=np.uint32).view(np.int32)).to(DEV)
    stream[-1] &= (1 << ((4 * n - 1) * 44 % 32)) - 1           # the bits behind the last record are zero
    packets, count = gpu_packetize(plan, stream, mtu)
    assert count == n
    out, status = gpu_depacketize(packets, n, d, mtu, stream.numel())
    assert status == 0
    assert torch.equal(out[: stream.numel()], stream)


@pytest.mark.parametrize("k,mtu", [(6 * 1024, 64), (6 * 1024 + 1, 64), (40_000, 64), (1_700_000, 64)])
def test_packets_more_than_threads_and_more_than_bits_in_lds(k, mtu):
    """The receiver keeps the headers of its first 1024 packets in registers and ticks off up to 262 144 in LDS: counts
    at and beyond both, in reverse order; one packet replaced by a copy of another is refused."""
    d = 1 << 22
    U = np.random.default_rng(k).standard_normal(d).astype(np.float32)
    po = orc.plan_manual(d, [10], [k])            # 32-bit records, six to a packet of 64 bytes
    words, _, status, streams = gpu_encode([U], [po], 3, [1], want_stats=False)
    assert status == 0
    buf, n = gpu_packetize(to_lib_plan(po), streams[0], mtu)
    assert n == -(-k // 6)
    packets = buf.view(n, mtu // 4).flip(0).contiguous()
    out, status = gpu_depacketize(packets, n, d, mtu, words[0].size)
    assert status == 0 and np.array_equal(out.cpu().numpy().view(np.uint32), words[0])
    packets[n // 2] = packets[n // 2 - 1]
    _, status = gpu_depacketize(packets, n, d, mtu, words[0].size)
    assert status & cv.DEV_STREAM


# --------------------------------------------------------------------------- power-law exponent (Algorithm 1, first step)
def gpu_fit_alpha(host_updates, two_passes=True):
    """two_passes: in the workspace that has room for the keys set aside by the second pass; else in the
    least workspace (three passes)."""
    n = len(host_updates)
    d = host_updates[0].size
    updates = [torch.from_numpy(u).to(DEV) for u in host_updates]
    alpha = torch.full((n,), float("nan"), dtype=torch.float64, device=DEV)
    keys = torch.full((n * cv.FIT_RANKS_MAX,), -1, dtype=torch.int32, device=DEV)
    small, large = cv.fit_workspace_bytes(n), cv.fit_workspace_bytes_for(n, d)
    assert large > small
    ws = cv.new_workspace(large if two_passes else large - 256, DEV)
    ws.fill_(0xA5)  # the call must clear what it counts in
    cv.fit_alpha(updates, alpha, ws, keys)
    status = cv.device_status(ws)
    return alpha.cpu().numpy(), keys.cpu().numpy().view(np.uint32).reshape(n, cv.FIT_RANKS_MAX), status


def check_fit(host_updates):
    """Magnitudes at the fitted ranks bit for bit; the slope to 1e-11 (fp64 on both
    sides, but two implementations of log)."""
    of = {id(u): u for u in host_updates}       # some clients may share a vector
    of = {i: (orc.fit_points(u), orc.fit_alpha(u)) for i, u in of.items()}
    refs = [of[id(u)] for u in host_updates]
    for two_passes in (True, False):
        alpha, keys, status = gpu_fit_alpha(host_updates, two_passes)
        assert status == 0
        for c, u in enumerate(host_updates):
            (ranks, ref_keys), ref_alpha = refs[c]
            assert ranks.tolist() == cv.fit_ranks(u.size)
            assert keys[c, : ranks.size].tolist() == ref_keys.tolist(), f"client {c}, two passes: {two_passes}"
            assert not keys[c, ranks.size:].any()
            assert alpha[c] == pytest.approx(ref_alpha, rel=1e-11, abs=1e-11), f"client {c}"
    return alpha


def test_fit_alpha_on_the_workload_distributions():
    check_fit([syn.update_vector(1, 0)])
    check_fit([syn.update_vector(2, c, d=300_001) for c in range(8)])
    check_fit([syn.update_vector(3, c, d=1_000_003) for c in range(5)])
    check_fit([syn.update_vector(4, c, d=250_000) for c in range(3)])


@pytest.mark.parametrize("kind", ["all_equal", "all_equal_mixed_sign", "two_valued", "few_levels",
                                  "zeros_and_denormals", "all_zero"])
def test_fit_alpha_on_colliding_magnitudes(kind):
    """Ranks that fall into one class at every radix level, zeros and denormals at the low ranks."""
    check_fit([syn.tie_heavy_vector(kind, 70_001, seed=1)])
    check_fit([syn.tie_heavy_vector(kind, 81_920, seed=3), syn.tie_heavy_vector(kind, 81_920, seed=4)])
    check_fit([syn.tie_heavy_vector(kind, 16_384, seed=3), syn.tie_heavy_vector(kind, 16_384, seed=4)])


def test_fit_alpha_tiny_and_ragged_lengths():
    rng = np.random.default_rng(11)
    for d in (1, 2, 3, 4, 5, 7, 8, 63, 4095, 4096, 4097, 16_385, 65_539):
        check_fit([(rng.standard_normal(d) * 10.0 ** rng.uniform(-6, 2, d)).astype(np.float32)])


def test_fit_alpha_recovers_a_power_law_and_feeds_the_planner():
    """Definition 1 in closed form: magnitudes l^alpha in shuffled order give alpha back;
    Algorithm 1 run with the fitted exponent yields the plan the oracle's planner makes from it."""
    d = 1 << 20
    rng = np.random.default_rng(5)
    vecs = []
    for a in (-0.3, -0.6, -0.9):
        mags = (np.arange(1, d + 1, dtype=np.float64) ** a).astype(np.float32)
        vecs.append((mags * rng.choice([-1.0, 1.0], d)).astype(np.float32)[rng.permutation(d)])
    alpha = check_fit(vecs)
    assert np.allclose(alpha, [-0.3, -0.6, -0.9], atol=1e-3)
    for a in alpha:
        pg = cv.plan(d, d, n_coded=6, alpha=float(a))
        po = orc.plan_alg1(d, d, 6, float(a))
        assert pg.counts() == po.counts() and pg.code_lens() == po.code_len() and pg.total_bits == po.total_bits


def test_fit_alpha_more_clients_than_one_upload_holds():
    """600 short vectors: the pointers are the arguments of two launches, one workgroup per client."""
    rng = np.random.default_rng(13)
    check_fit([(rng.standard_t(3, 5000) * 1e-3).astype(np.float32) for _ in range(600)])


def test_fit_alpha_more_long_vectors_than_one_upload_holds():
    """449 vectors of more than 65 536 coordinates, five different ones: the pointer table travels in two launches."""
    rng = np.random.default_rng(13)
    host = [(rng.standard_t(3, SHORT_MAX + 3) * 1e-3).astype(np.float32) for _ in range(5)]
    check_fit([host[c * c % 5] for c in range(449)])


@pytest.mark.parametrize("kind", ["plain", "bfloat16", "few values", "zeros", "octaves", "sorted", "ramp"])
@pytest.mark.parametrize("n,d", [(1, 3), (1, 1023), (2, 4099), (1, SHORT_MAX - 1), (1, SHORT_MAX), (2, SHORT_MAX), (1, SHORT_MAX + 1), (449, 130)])
def test_fit_alpha_of_short_vectors(n, d, kind):
    """One workgroup per client, up to 448 clients a launch; a single one writes the status word itself."""
    rng = np.random.default_rng(d)
    host = [_selection_vectors(kind, d, rng) for _ in range(n)]
    check_fit(host)
    for value in (np.inf, np.nan, np.uint32(0xFFFFFFFF).view(np.float32)):
        if n <= 2:
            host[-1][d // 2] = value
            assert gpu_fit_alpha(host)[-1] == 1


@pytest.mark.parametrize("bins,waves", [(160, 16), (160, 4), (80, 2), (80, 1)])
@pytest.mark.parametrize("d", [SHORT_MAX, SHORT_MAX - 253])
def test_fit_alpha_of_short_vectors_whose_members_a_few_wavefronts_come_across(d, bins, waves):
    """The keys that share a bin with a rank lie in every sixteenth 256 coordinates: lists of their own for all wavefronts, the
    common part of the lists in use, and overrun."""
    rng = np.random.default_rng(bins + waves)
    keys = np.sort((np.uint32(0x3C000000 >> 17) + rng.integers(0, bins, d, dtype=np.uint32) << 17) | rng.integers(0, 1 << 17, d, dtype=np.uint32))[::-1]
    member = np.isin(keys >> 17, np.unique(keys[np.array(cv.fit_ranks(d)) - 1] >> 17))
    order = np.argsort(np.arange(d) // 256 % 16 >= waves, kind="stable")         # the few wavefronts' places first
    placed = np.empty(d, dtype=np.uint32)
    placed[order] = np.concatenate([rng.permutation(keys[member]), rng.permutation(keys[~member])])
    check_fit([np.where(rng.random(d) < 0.5, -1, 1).astype(np.float32) * placed.view(np.float32)])


# The collecting pass has a workgroup for every CU, two where a client's share of them is not a whole number, or those of the
# other passes where short lists would need more room; the lists' passes 16 a client or, up to eight clients, one for every CU.
@pytest.mark.parametrize("n,d", [(1, 16_385), (1, 4_200_001), (2, 2_104_225), (8, 150_003), (9, 150_003), (12, 70_001), (100, 40_000), (129, 20_000),
                                 (1, SHORT_MAX + 1), (100, 70_001), (129, 66_003)])
def test_fit_alpha_at_the_steps_of_the_workgroups(n, d):
    rng = np.random.default_rng(n + d)
    host = [(rng.standard_t(3, d) * 1e-3).astype(np.float32) for _ in range(min(n, 5))]
    check_fit([host[c % len(host)] for c in range(n)])


@pytest.mark.parametrize("bins", [(0, 8159), (127, 128, 129), tuple(range(0, 8160, 128)), tuple(range(127, 8160, 128)), (8159,), (4095, 4096)])
def test_fit_alpha_at_the_borders_of_the_walks_blocks(bins):
    """The level-1 walk searches blocks of 128 bins (key >> 18), then a block's bins: keys in the bins next to the borders, in the
    lowest and in the highest bin of finite numbers."""
    d = SHORT_MAX + 4097
    rng = np.random.default_rng(len(bins) + bins[0])
    keys = (rng.choice(np.array(bins, dtype=np.uint32), d) << 18) | rng.integers(0, 1 << 18, d, dtype=np.uint32)
    check_fit([keys.view(np.float32), -np.sort(keys).view(np.float32)])


@pytest.mark.parametrize("d", [2_100_003, 2_097_152])
def test_fit_alpha_in_one_pass(d):
    """From 7 x 2^24 coordinates on the level-1 bins of the ranks are guessed from a sample: ordinary vectors, tied ones, and
    one whose sampled pieces hold what the rest does not, so that the guess is wrong and the vector is read again."""
    rng = np.random.default_rng(d)
    planted = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    plant_on_the_sampled_pieces(planted, rng)
    tied = (2.0 ** rng.integers(-3, 4, d)).astype(np.float32)
    host = [planted, syn.update_vector(3, 1, d=d), tied, (rng.standard_normal(d) * 1e-3).astype(np.float32)]
    n = 56
    assert n * d >= 7 << 24
    refs = [(orc.fit_points(u)[1], orc.fit_alpha(u)) for u in host]
    dev = [torch.from_numpy(u).to(DEV) for u in host]
    ws = cv.new_workspace(cv.fit_workspace_bytes_for(n, d), DEV)
    alpha_dev = torch.zeros(n, dtype=torch.float64, device=DEV)
    keys_dev = torch.zeros((n, cv.FIT_RANKS_MAX), dtype=torch.int32, device=DEV)
    cv.fit_alpha([dev[c % 4] for c in range(n)], alpha_dev, ws, keys_dev)
    assert cv.device_status(ws) == 0
    alpha, keys = alpha_dev.cpu().numpy(), keys_dev.cpu().numpy().view(np.uint32)
    # A client's state lies behind the status word's 256 bytes and ends in {missed, 8 bytes, 1024 bytes of guessed bins}.
    size = (cv.fit_workspace_bytes(512) - cv.fit_workspace_bytes(256)) // 256 - 8
    state = ws[256:256 + n * size].view(n, size).cpu().numpy()
    guessed, missed = state[:, -1024:].any(axis=1), state[:, -1036:-1032].any(axis=1)
    assert guessed.all() and missed[0::4].all() and not missed[1::2].any()
    for c in range(n):
        ref_keys, ref_alpha = refs[c % 4]
        assert keys[c, : ref_keys.size].tolist() == ref_keys.tolist(), c
        assert not keys[c, ref_keys.size:].any()
        assert alpha[c] == pytest.approx(ref_alpha, rel=1e-11, abs=1e-11), c


def test_fit_alpha_of_vectors_of_rows():
    """Rows of 64 with a scale of their own: the sample's pieces are as alike as rows are, the margins of the guess take
    that in, and the call costs a little more than for coordinates drawn one by one (twice as much when rows were
    missed as a rule and their vectors read twice more by few workgroups)."""
    n, d = 12, 11_200_000
    gen = torch.Generator(device=DEV).manual_seed(9)
    plain = [torch.randn(d, device=DEV, generator=gen) for _ in range(n)]
    rows = [(u.view(-1, 64) * torch.exp(torch.randn(d // 64, 1, device=DEV, generator=gen))).view(-1) for u in plain]
    ws = cv.new_workspace(cv.fit_workspace_bytes_for(n, d), DEV)
    alpha = torch.zeros(n, dtype=torch.float64, device=DEV)
    best = []
    for updates in (plain, rows):
        times = []
        for _ in range(7):
            cv.profile_start(["fit_alpha"])
            cv.fit_alpha(updates, alpha, ws)
            times.append(cv.profile_stop()["fit_alpha"][0])
        best.append(min(times))
    assert best[1] < 1.35 * best[0], best
    assert alpha[3].item() == pytest.approx(orc.fit_alpha(rows[3].cpu().numpy()), rel=1e-11, abs=1e-11)


def test_fit_alpha_flags_non_finite_input():
    U = syn.update_vector(1, 0).copy()
    U[777] = np.float32("inf")
    _, _, status = gpu_fit_alpha([U])
    assert status & cv.DEV_NONFINITE
    with pytest.raises(orc.OracleError):
        orc.fit_points(U)


# --------------------------------------------------------------------------- full benchmark size
def _parallel(fn, items, workers=12):
    with ThreadPoolExecutor(max_workers=workers) as ex:
        return list(ex.map(fn, items))


@pytest.mark.parametrize("cfg", [3, 4])
def test_full_size_32_clients(cfg):
    """The benchmark's launch configuration: 32 clients, d = 11.2M, one batched encode
    and one decode-aggregate.  Every client's stream is compared with the oracle's, and
    the aggregate is compared element by element."""
    w = syn.WORKLOADS[cfg]
    n, d = w.n_clients, w.d
    host = _parallel(lambda c: syn.update_vector(cfg, c), range(n), workers=8)
    alpha = -0.5
    plans = [orc.plan_for(w, client=c, alpha=alpha) for c in range(1)] * n
    words, stats, status, dev_streams = gpu_encode(host, plans, w.quant_seed, list(range(n)))
    assert status == 0
    refs = _parallel(lambda c: orc.encode(host[c], plans[c], w.quant_seed, c), range(n))
    for c in range(n):
        assert_stream_equal(words[c], refs[c].words, f"cfg {cfg} client {c}")
        assert_stats_close(stats[c], refs[c].stats, plans[c].R)
    got, status = gpu_decode(dev_streams, d)
    assert status == 0
    ref_streams = [r.words for r in refs]
    ref = orc.decode_aggregate(ref_streams, d)
    tol = 1e-5 * abs_terms(ref_streams, d)
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= tol)


def _progress(msg):
    """A line in the file CVLC_TEST_PROGRESS names (when set), so that a long test is seen to be alive."""
    path = os.environ.get("CVLC_TEST_PROGRESS")
    if path:
        with open(path, "a") as f:
            f.write(msg + "\n")


def _stored_cfg5_plans():
    """The 100 plans of configuration 5 as the oracle's Algorithm 1 made them from the oracle's exponent fit
    (tests/golden/cfg5_plans.txt, written by tests/golden/make_cfg5_plans.py: minutes of CPU time).  Each is
    rebuilt through the oracle's validation and must fit the client's budget."""
    w = syn.WORKLOADS[5]
    plans = []
    with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "cfg5_plans.txt")) as f:
        for line in f:
            if line.startswith("#") or not line.strip():
                continue
            head, ys, Ps = line.split("|")
            client, _alpha, budget, total = head.split()
            assert int(client) == len(plans) and int(budget) == w.budget_bits(int(client))
            p = orc.plan_manual(w.d, [int(v) for v in ys.split()], [int(v) for v in Ps.split()])
            assert p.total_bits == int(total) <= int(budget)
            plans.append(p)
    assert len(plans) == w.n_clients
    return plans


def test_full_size_100_clients_31_groups_streamed_aggregate():
    """Configuration 5 at full size: 100 clients, d = 25.6M, Laplace or Gaussian per client, a budget of its
    own per client (0.25 .. 2 bit/coordinate), 31 coded groups planned by Algorithm 1 from each vector's
    fitted exponent; one batched encode, every stream compared word for word with the oracle's; then the
    100 streams are aggregated in four calls of 25 in accumulate mode with the caller's weights 1/100 and
    compared element by element with the oracle doing the same.  n * d passes 2^31 (workspace offsets),
    the plans differ (several parameter uploads), the selection takes three rounds of 15 boundaries and a
    decode call sees 775 record lists."""
    w = syn.WORKLOADS[5]
    n, d = w.n_clients, w.d
    _progress("cfg5: vectors")
    host = _parallel(lambda c: syn.update_vector(5, c), range(n), workers=16)
    plans = _stored_cfg5_plans()
    assert len({tuple(p.counts()) for p in plans}) > 50 and all(p.R == 31 for p in plans)
    _progress("cfg5: gpu encode")
    words, stats, status, dev_streams = gpu_encode(host, plans, w.quant_seed, list(range(n)))
    assert status == 0
    _progress("cfg5: oracle encode")
    refs = _parallel(lambda c: orc.encode(host[c], plans[c], w.quant_seed, c), range(n), workers=16)
    for c in range(n):
        assert_stream_equal(words[c], refs[c].words, f"cfg 5 client {c}")
        assert_stats_close(stats[c], refs[c].stats, plans[c].R)
    del host, words
    _progress("cfg5: decode")
    ref_streams = [r.words for r in refs]
    wts = [float(np.float32(1.0 / n))] * n
    acc = torch.zeros(d, dtype=torch.float32, device=DEV)
    ref = np.zeros(d, dtype=np.float32)
    for b in range(0, n, 25):
        got, status = gpu_decode(dev_streams[b:b + 25], d, weights=wts[b:b + 25], accumulate_into=acc)
        assert status == 0
        ref = orc.decode_aggregate(ref_streams[b:b + 25], d, weights=wts[b:b + 25], out=ref)
        _progress(f"cfg5: batch {b}")
    # sum_i |w_i xhat_ij|: the oracle's aggregate of the same streams with the signs of the values removed,
    # i.e. of |xhat|; computed from single-client decodes, a few at a time
    tot = np.zeros(d)
    for part in _parallel(lambda c: np.abs(orc.decode_aggregate([ref_streams[c]], d, weights=[1.0]).astype(np.float64)),
                          range(n), workers=8):
        tot += part * wts[0]
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= 1e-5 * tot)
    assert int(np.count_nonzero(ref)) > d // 2


def test_full_size_qsgd_8_clients():
    """cfg 3's vectors at full length with the second quantiser: 8 clients, 1 bit/coordinate spread
    over eight code lengths; streams (norms included) word for word, aggregate element by element."""
    w = syn.WORKLOADS[3]
    n, d = 8, w.d
    host = _parallel(lambda c: syn.update_vector(3, c), range(n), workers=8)
    pq = orc.plan_budget(d, w.budget_bits(0), [12, 10, 8, 6, 5, 4, 3, 2])
    plan = orc.plan_manual(d, pq.code_len(), pq.counts(), quant=orc.QSGD)
    words, stats, status, dev_streams = gpu_encode(host, [plan] * n, w.quant_seed, list(range(n)), error_stats=True)
    assert status == 0
    refs = _parallel(lambda c: orc.encode(host[c], plan, w.quant_seed, c), range(n))
    for c in range(n):
        assert_stream_equal(words[c], refs[c].words, f"client {c}")
        assert_stats_close(stats[c], refs[c].stats, plan.R, error_stats=True)
    got, status = gpu_decode(dev_streams, d, quant=cv.QUANT_QSGD)
    assert status == 0
    ref_streams = [r.words for r in refs]
    ref = orc.decode_aggregate(ref_streams, d)
    tol = 1e-5 * abs_terms(ref_streams, d)
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= tol)


def test_fit_alpha_full_size_32_clients():
    """The benchmark's launch configuration of the exponent fit: 32 clients, d = 11.2M."""
    w = syn.WORKLOADS[3]
    host = _parallel(lambda c: syn.update_vector(3, c), range(w.n_clients), workers=8)
    alpha, keys, status = gpu_fit_alpha(host)
    assert status == 0
    refs = _parallel(lambda c: (orc.fit_points(host[c]), orc.fit_alpha(host[c])), range(w.n_clients))
    for c, ((ranks, ref_keys), ref_alpha) in enumerate(refs):
        assert keys[c, : ranks.size].tolist() == ref_keys.tolist(), f"client {c}"
        assert alpha[c] == pytest.approx(ref_alpha, rel=1e-11, abs=1e-11)


# --------------------------------------------------------------------------- vectors the oracle cannot sort in test time
@pytest.mark.parametrize("d,ys,counts", [
    (300_000_007, [12, 8, 2], [2_000_003, 3_000_000, 5_000_001]),      # 29 position bits, records of 41, 37, 31 bits
    (2**31 - 1, [32, 12, 1], [1_000_001, 4_000_000, 7_000_003]),        # the largest d the ABI takes: 63, 43, 32 bits
])
def test_properties_at_sizes_beyond_the_oracle(d, ys, counts):
    """The oracle's sort would take minutes at these sizes, so the encoder is checked through what must
    hold at any size: the records the oracle's parser reads back are the top-k coordinates, in position
    order inside magnitude-ordered groups; the headers hold the groups' exact min and max; every
    reconstruction lies within one centroid spacing of its value (exactly on it for 32-bit codes); and
    the library's decode of the stream equals the oracle's decode of the same stream bit for bit.
    Records wider than 33 bits span three stream words."""
    k = sum(counts)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2402_03770)
    U = torch.randn(d, dtype=torch.float32, device=DEV, generator=gen)
    # 1000 "layers" of different scale, as in the benchmark workload
    scale = 10.0 ** (torch.rand(1000, device=DEV, generator=gen) * 3.0 - 5.0)
    U *= scale.repeat_interleave((d + 999) // 1000)[:d]
    del scale
    plan = cv.plan_manual(d, ys, counts)
    stream = cv.new_stream_buffer(plan, DEV)
    stream.fill_(-1)
    ws = cv.new_workspace(cv.encode_workspace_bytes(d, 1), DEV)
    cv.encode_batch([plan], [U], 77, [5], [stream], ws)
    assert cv.device_status(ws) == 0
    del ws
    words = stream.cpu().numpy().view(np.uint32)[: plan.stream_bytes // 4]

    pid, cid, seg = orc.unpack(words, d)
    assert pid.size == k
    bounds = np.concatenate([[0], np.cumsum(counts)])
    pid_dev = torch.from_numpy(pid.astype(np.int64)).to(DEV)
    kept = U[pid_dev]
    mag = kept.abs()
    lowest_above = None
    headers = []
    for r in range(len(ys)):
        a, b = int(bounds[r]), int(bounds[r + 1])
        assert np.all(seg[a:b] == r + 1)
        assert np.all(np.diff(pid[a:b].astype(np.int64)) > 0), f"group {r}: positions must ascend"
        assert int(pid[a:b].max()) < d
        g = mag[a:b]
        if lowest_above is not None:
            assert float(g.max()) <= lowest_above, "groups must be ordered by magnitude"
        lowest_above = float(g.min())
        # header: exact min and max of the group's values
        h = words[8 + 4 * r: 12 + 4 * r]
        assert int(h[0]) == ys[r] and int(h[1]) == counts[r]
        m, M = h[2:3].view(np.float32)[0], h[3:4].view(np.float32)[0]
        assert m == float(kept[a:b].min()) and M == float(kept[a:b].max())
        headers.append((float(m), float(M)))
    # the kept set is the top k: nothing outside it is larger than its smallest member
    tau = float(mag.min())
    n_gt = int((U.abs() > tau).sum())
    n_ge = int((U.abs() >= tau).sum())
    assert n_gt == int((mag > tau).sum()) and n_gt < k <= n_ge

    out = torch.full((d,), float("nan"), dtype=torch.float32, device=DEV)
    dws = cv.new_workspace(cv.decode_workspace_bytes(d, 1), DEV)
    cv.decode_aggregate([stream], out, dws)
    assert cv.device_status(dws) == 0
    xhat = out[pid_dev]
    for r in range(len(ys)):
        a, b = int(bounds[r]), int(bounds[r + 1])
        m, M = headers[r]
        err = float((xhat[a:b].double() - kept[a:b].double()).abs().max())
        if ys[r] == 32:
            assert err == 0.0
        else:
            assert err <= (M - m) / (2 ** ys[r] - 1) * (1 + 1e-5)
    assert int((out != 0).sum()) <= k
    del kept, mag, xhat, pid_dev
    ref = orc.decode_aggregate([words], d)
    got = out.cpu().numpy()
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), "single-client decode is bit exact"
    del out, dws, ref, got

    # the exponent fit at the same length: its order statistics against a library sort on the device
    alpha = torch.empty(1, dtype=torch.float64, device=DEV)
    keys = torch.empty(cv.FIT_RANKS_MAX, dtype=torch.int32, device=DEV)
    fws = cv.new_workspace(cv.fit_workspace_bytes(1), DEV)
    cv.fit_alpha([U], alpha, fws, keys)
    assert cv.device_status(fws) == 0
    ranks = cv.fit_ranks(d)
    desc = torch.sort(U.abs_(), descending=True).values            # U is not needed any more
    want = desc[torch.tensor([l - 1 for l in ranks], device=DEV)].view(torch.int32).cpu().numpy()
    del desc
    got_keys = keys.cpu().numpy()
    assert np.array_equal(got_keys[: len(ranks)], want) and not got_keys[len(ranks):].any()
    mags = want.view(np.float32).astype(np.float64)
    use = mags > 0.0                                               # a zero magnitude has no logarithm
    x, y, m = np.log(np.array(ranks, dtype=np.float64)[use]), np.log(mags[use]), int(use.sum())
    slope = (m * (x * y).sum() - x.sum() * y.sum()) / (m * (x * x).sum() - x.sum() ** 2)
    assert float(alpha[0]) == pytest.approx(slope, rel=1e-9)
