"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs -- indices, level codes, packed bytes, bit counts and the error memory bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_1906_02367_amd import workloads as W  # noqa: E402

f32 = np.float32


@pytest.fixture(scope="module")
def P():
    import parity_util
    return parity_util


def custom(d, seg_offset, seg_k, s, sparsifier, quantizer, R, name="custom", cfg=2, seed=12345):
    return W.Workload(cfg, name, R, d, np.asarray(seg_offset, dtype=np.uint64), np.asarray(seg_k, dtype=np.uint32), s,
                      sparsifier, quantizer, 1, seed)


# ---------------------------------------------------------------------------------------------
# small shapes: the general (multi-pass) path; several tiles and a ragged tail
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
def test_configs_reduced_size(P, cfg):
    d = {1: 65_536, 2: 70_001, 3: 70_001, 4: 150_000, 5: 99_991}[cfg]
    wl = W.config(cfg, d=d, R=2 if cfg != 1 else None, rounds=4)
    print(f"\n[{wl.name}] d={wl.d} K={wl.K} L={wl.L}", flush=True)
    P.run_parity(wl, 4 if cfg != 1 else 10)


@pytest.mark.parametrize("sparsifier", [W.TOPK, W.RANDK])
@pytest.mark.parametrize("quantizer,s", [(W.QSGD, 15), (W.QSGD, 1), (W.QSGD, 32768), (W.SIGN_L1, 1), (W.SIGN_L2, 1),
                                         (W.FP32, 1), (W.QSGD_SCALED, 4), (W.QSGD_SCALED, 15), (W.SIGN_L3, 1), (W.SIGN_L4, 1)])
def test_operator_grid_small(P, sparsifier, quantizer, s):
    wl = custom(40_003, [0, 40_003], [777], s, sparsifier, quantizer, R=3)
    P.run_parity(wl, 2, worker0=5)


@pytest.mark.parametrize("quantizer,s", [(W.SIGN_L2, 1), (W.FP32, 1), (W.QSGD_SCALED, 2), (W.SIGN_L3, 1), (W.SIGN_L4, 1)])
def test_operator_variants_on_the_fast_path_and_layerwise(P, quantizer, s):
    # the variants next to the hot path: sign scaled by the l2, l3, l4 norm (Lemma 3, m = 2, 3, 4), no quantiser
    # (TopK-SGD), scaled QSGD (Lemma 2)
    wl = custom(1_000_003, [0, 1_000_003], [1000], s, W.TOPK, quantizer, R=2)
    run, op, m_host, _ = P.run_parity(wl, 2, expect_path=0)
    out = torch.zeros(wl.d, dtype=torch.float32, device=run.q.device)
    run.q.aggregate(run.msg, out, 0.5)
    torch.cuda.synchronize()
    want = op.aggregate(run.msg.cpu().numpy(), 0.5)
    assert np.allclose(out.cpu().numpy(), want, rtol=1e-6, atol=1e-30)
    off = [0, 64, 1_000, 40_000, 70_001]
    wl = custom(70_001, off, [3, 10, 400, 30], s, W.RANDK, quantizer, R=2)
    P.run_parity(wl, 2)


def test_not_in_place(P):
    wl = W.config(2, d=50_000, R=2)
    P.run_parity(wl, 3, in_place=False)


# ---------------------------------------------------------------------------------------------
# the single-pass fast path (guess + candidate pool) at sizes that enable it
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("cfg,d", [(2, 1_000_003), (3, 600_011), (5, 4_000_037)])
def test_fast_path_mid_size(P, cfg, d):
    wl = W.config(cfg, d=d, R=3, rounds=3)
    print(f"\n[{wl.name}] d={wl.d} K={wl.K}", flush=True)
    P.run_parity(wl, 3, expect_path=0)


def test_fast_and_general_paths_agree_layerwise(P):
    # segments from 64 coordinates to ~1.9 M: a mix of fast and general units in one call
    wl = W.config(4, d=20_000_000, R=2)
    run, op, m_host, paths = P.run_parity(wl, 2)
    assert (paths[0] == 0).any() and (paths[0] == 3).any()
    run, op, m_host, paths = P.run_parity(wl, 1, flags=3)          # every unit through the multi-pass kernels
    assert (paths[0] == 1).all()


def test_failed_guess_falls_back(P):
    # large values exactly where the sample looks -> the guess is far too high -> too few candidates
    d, k, R = 1_000_003, 1000, 2
    wl = custom(d, [0, d], [k], 16, W.TOPK, W.QSGD, R)
    rng = np.random.default_rng(3)
    delta = rng.standard_normal((R, d)).astype(f32)
    n_s = 42.25 * 3.0 / (4.0 * (k / d))                    # the library's sampling plan at alpha = 3
    n_runs = int(np.ceil(n_s / 64.0))
    starts = np.arange(n_runs, dtype=np.int64) * (d // n_runs)          # the library samples runs of 64 at this stride
    pos = (starts[:, None] + np.arange(64)[None, :]).ravel()
    delta[:, pos] *= 1000.0
    run, op, m_host, paths = P.run_parity(wl, 1, deltas=[delta])
    assert np.all(paths[0] == 2), paths
    # ... and the opposite failure: tiny values where the sample looks -> far too many candidates
    delta = rng.standard_normal((R, d)).astype(f32)
    delta[:, pos] *= 1e-6
    run, op, m_host, paths = P.run_parity(wl, 1, deltas=[delta])
    print("paths after a low guess:", paths)


def test_clustered_candidates_use_the_overflow_pool(P):
    # most of the large values sit in a few chunks of 1024 coordinates: their slots cannot hold them,
    # they spill to the overflow pool, and the unit still runs on the single-pass path
    d, k, R = 1_000_003, 1000, 2
    rng = np.random.default_rng(23)
    for sp, qz, s in [(W.TOPK, W.QSGD, 16), (W.TOPK, W.SIGN_L1, 1)]:
        wl = custom(d, [0, d], [k], s, sp, qz, R)
        deltas = []
        for t in range(2):
            delta = rng.standard_normal((R, d)).astype(f32)
            for r in range(R):
                delta[r, 5_000:5_700] *= 50.0                  # 700 coordinates of one chunk-and-a-bit
                delta[r, 777_000:777_040] *= 80.0
                hot = rng.choice(d, 300, replace=False)
                delta[r, hot] *= 30.0
            deltas.append(delta)
        P.run_parity(wl, 2, deltas=deltas, expect_path=0)


# ---------------------------------------------------------------------------------------------
# degenerate inputs
# ---------------------------------------------------------------------------------------------
def _adversarial(d, rng):
    yield "all_equal", np.full(d, 1.5, dtype=f32)
    yield "all_zero", np.zeros(d, dtype=f32)
    yield "signed_zeros", np.where(np.arange(d) % 2 == 0, 0.0, -0.0).astype(f32)
    one = np.full(d, 1e-3, dtype=f32); one[d // 3] = -1e6
    yield "one_dominant", one
    yield "denormals", (rng.integers(-200, 200, d) * 1e-45).astype(f32)
    yield "few_values", rng.integers(-2, 3, d).astype(f32)
    yield "wide_range", (rng.standard_normal(d) * np.exp(8 * rng.standard_normal(d))).astype(f32)


@pytest.mark.parametrize("flags,path", [(0, 3), (2, 1)])      # one launch for the whole call / multi-pass kernels
@pytest.mark.parametrize("quantizer,s", [(W.QSGD, 16), (W.SIGN_L1, 1)])
@pytest.mark.parametrize("k", [1, 37, 4_001])
def test_degenerate_inputs(P, quantizer, s, k, flags, path):
    d = 4_001
    rng = np.random.default_rng(17)
    wl = custom(d, [0, d], [k], s, W.TOPK, quantizer, R=1)
    if k == d and flags == 2:
        path = 4                                     # nothing to select: not a case for the multi-pass kernels
    for name, v in _adversarial(d, rng):
        P.run_parity(wl, 1, deltas=[v[None, :].copy()], flags=flags, expect_path=path)


# the one-block selection of a segment of a larger operator (4,001: inside the streaming kernel) and of one of more than 16,384 coordinates
@pytest.mark.parametrize("quantizer,s", [(W.QSGD, 16), (W.SIGN_L1, 1)])
@pytest.mark.parametrize("off,k", [([0, 4_001, 4_100], [1, 9]), ([0, 4_001, 4_100], [37, 9]), ([0, 20_011], [2_500]), ([0, 16_385], [9_000])])
def test_degenerate_inputs_one_block(P, quantizer, s, off, k):
    rng = np.random.default_rng(17)
    wl = custom(off[-1], off, k, s, W.TOPK, quantizer, R=1)
    for name, v in _adversarial(off[-1], rng):
        P.run_parity(wl, 1, deltas=[v[None, :].copy()], expect_path=3)


@pytest.mark.parametrize("d,k", [(40_009, 1), (40_009, 37), (40_009, 200), (16_411, 1), (20_011, 37), (18_003, 60), (12_011, 1), (12_011, 37), (12_011, 60)])
def test_degenerate_inputs_whole_unit_guess(P, k, d):
    # 17 .. 255 chunks: the guess comes from a histogram of the whole unit; inputs with few distinct
    # magnitudes put everything into one bin, overflow the candidate list and must fall back.  12,011: the whole call is one
    # launch (path 2: its lower bound leaves more than 4096 coordinates)
    rng = np.random.default_rng(23)
    wl = custom(d, [0, d], [k], 16, W.TOPK, W.QSGD, R=1)
    seen = set()
    for name, v in _adversarial(d, rng):
        run, op, m_host, paths = P.run_parity(wl, 1, deltas=[v[None, :].copy()])
        seen.update(paths[0].tolist())
    assert seen == {0, 2}, seen


# sizes around the limit of the one-block selection (4096 coordinates) and of its 16-per-thread layout: by itself (up to 16,384 coordinates one
# launch for the whole call), and as a segment beside another
@pytest.mark.parametrize("sparsifier", [W.TOPK, W.RANDK])
@pytest.mark.parametrize("d,k", [(4_096, 100), (4_096, 4_096), (4_097, 4_097), (4_097, 3), (4_095, 4_095), (2_063, 1_000),
                                 (16_385, 16_385), (8_209, 4_000), (32_769, 1), (65_537, 655), (17, 16), (15, 15),
                                 (1_025, 1_024), (262_143, 250)])
def test_small_units_one_block_boundaries(P, sparsifier, d, k):
    small = d <= 4_096
    wl = custom(d, [0, d], [k], 7, sparsifier, W.QSGD, R=2)
    P.run_parity(wl, 2, expect_path=3 if small else None)
    wl = custom(d, [0, d], [k], 1, sparsifier, W.SIGN_L1, R=2)
    P.run_parity(wl, 1, flags=3, expect_path=1)                   # the same through the multi-pass kernels
    ties = np.round(np.random.default_rng(d).standard_normal((1, 2, d)) * 2).astype(f32)     # many equal magnitudes
    P.run_parity(wl, 1, deltas=ties, expect_path=3 if small else None)
    if small:
        wl = custom(d + 70, [0, d, d + 70], [k, 9], 7, sparsifier, W.QSGD, R=2)
        P.run_parity(wl, 2, expect_path=3)
        ties = np.round(np.random.default_rng(d).standard_normal((1, 2, d + 70)) * 2).astype(f32)
        P.run_parity(wl, 1, deltas=ties, expect_path=3)


def test_small_and_large_units_mixed(P):
    # one call with one-block units, multi-pass units and guessed units side by side
    off = [0, 100, 70_000, 70_001, 400_000, 410_000, 1_100_000]
    k = [100, 70, 1, 30_000, 650, 600]
    for sp, qz, s in [(W.TOPK, W.QSGD, 16), (W.RANDK, W.SIGN_L1, 1)]:
        wl = custom(1_100_000, off, k, s, sp, qz, R=3)
        run, op, m_host, paths = P.run_parity(wl, 2)
        assert sorted(set(paths[0].tolist())) == [0, 1, 3], paths[0]


# multi-pass units, one-block units and guessing units of a single block in one call: the one-block units beside the multi-pass kernels (few
# workers), or in one launch with the guessing units (more than 300 blocks of those)
@pytest.mark.parametrize("sparsifier,quantizer,s", [(W.TOPK, W.QSGD, 15), (W.TOPK, W.SIGN_L1, 1), (W.RANDK, W.SIGN_L2, 1)])
@pytest.mark.parametrize("R", [2, 40])
def test_one_block_units_with_multi_pass_units(P, sparsifier, quantizer, s, R):
    sizes = [20_011] + [5_003] * 8 + [46_815, 300]
    k = [2_500] + [10] * 8 + [4_000, 40]
    off = np.concatenate([[0], np.cumsum(sizes)])
    wl = custom(int(off[-1]), off, k, s, sparsifier, quantizer, R=R)
    run, op, m_host, paths = P.run_parity(wl, 2)
    assert paths[0][:11].tolist() == [3] + [0] * 8 + [1, 3], paths[0][:11]


def test_degenerate_inputs_on_fast_sizes(P):
    d, k = 600_000, 500
    rng = np.random.default_rng(19)
    wl = custom(d, [0, d], [k], 4, W.TOPK, W.QSGD, R=1)
    for name, v in _adversarial(d, rng):
        print(name, flush=True)
        P.run_parity(wl, 1, deltas=[v[None, :].copy()])


def test_tiny_segments_and_unaligned_offsets(P):
    off = [0, 64, 65, 130, 1_031, 5_000, 5_003, 40_000, 70_001]
    k = [1, 1, 65, 9, 100, 3, 35, 30_001]
    for sp, qz, s in [(W.TOPK, W.SIGN_L1, 1), (W.TOPK, W.QSGD, 4), (W.RANDK, W.QSGD, 2)]:
        wl = custom(70_001, off, k, s, sp, qz, R=3)
        P.run_parity(wl, 2)


def test_d_equals_one_and_k_equals_d(P):
    wl = custom(1, [0, 1], [1], 16, W.TOPK, W.QSGD, R=2)
    P.run_parity(wl, 2)
    wl = custom(5_000, [0, 5_000], [5_000], 16, W.TOPK, W.QSGD, R=1)      # QSGD on the whole vector
    P.run_parity(wl, 2)
    # the sign of the whole vector (every message lists every coordinate), and the master line on such messages
    wl = custom(20_003, [0, 20_003], [20_003], 1, W.TOPK, W.SIGN_L1, R=3)
    run, op, m_host, _ = P.run_parity(wl, 2)
    x0 = np.random.default_rng(8).standard_normal(wl.d).astype(f32)
    out = torch.from_numpy(x0).to(run.q.device)
    run.q.aggregate(run.msg, out, -1.0 / 3, worker_list=[2, 0], accumulate=True)
    torch.cuda.synchronize()
    msgs = run.msg.cpu().numpy()
    want = op.aggregate(msgs, -1.0 / 3, worker_list=[2, 0], out=x0)
    mag = sum(np.abs(op.decode(msgs[r])[1].astype(np.float64)) for r in (2, 0))
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - want) <= 1e-6 * (mag / 3 + np.abs(want)) + 1e-38)


# k = size of the segment (the error-feedback schemes without sparsification that Section 5 compares with, as
# this operator): no selection at all; ragged sizes around the 4096-coordinate tiles and the 512-block limit
@pytest.mark.parametrize("sparsifier", [W.TOPK, W.RANDK])
@pytest.mark.parametrize("quantizer,s", [(W.QSGD, 15), (W.SIGN_L1, 1), (W.SIGN_L2, 1), (W.FP32, 1), (W.QSGD_SCALED, 3),
                                         (W.SIGN_L3, 1), (W.SIGN_L4, 1)])
def test_every_coordinate_kept(P, sparsifier, quantizer, s):
    for d in (4_097, 300_001, 2_200_003):                        # 2, 74 and 538 tiles (more than the blocks of a unit)
        wl = custom(d, [0, d], [d], s, sparsifier, quantizer, R=2)
        run, op, m_host, _ = P.run_parity(wl, 2, expect_path=4)
        if d == 300_001:
            # the master line on messages that list every coordinate; the third listed row is an empty (all-zero) message
            msgs = torch.cat([run.msg, torch.zeros_like(run.msg[:1])])
            msgs_host = msgs.cpu().numpy()
            x0 = np.random.default_rng(d).standard_normal(d).astype(f32)
            for lst, accumulate in (([1, 0], False), ([0, 2, 1], True)):
                out = torch.from_numpy(x0).to(run.q.device)
                run.q.aggregate(msgs, out, -0.5, worker_list=lst, accumulate=accumulate)
                torch.cuda.synchronize()
                want = op.aggregate(msgs_host, -0.5, worker_list=lst, out=x0.copy() if accumulate else None)
                mag = np.zeros(d)
                for r in lst:
                    i, vv = op.decode(msgs_host[r])
                    mag[i] += np.abs(vv.astype(np.float64))
                got = out.cpu().numpy().astype(np.float64)
                assert np.all(np.abs(got - want) <= 1e-6 * (mag * 0.5 + np.abs(want)) + 1e-38)
            from paper_1906_02367_amd import binding as B
            assert run.q.device_status() == B.OK
    # segments that keep everything beside segments that select, in one call; degenerate values
    off = [0, 5_000, 70_000, 70_001, 400_000, 410_001, 1_100_000]
    k = [5_000, 65_000, 1, 30_000, 10_001, 600]
    wl = custom(1_100_000, off, k, s, sparsifier, quantizer, R=3)
    run, op, m_host, paths = P.run_parity(wl, 2)
    assert paths[0].reshape(3, 6)[0].tolist() == [4, 4, 3, 1, 4, 0], paths[0]
    rng = np.random.default_rng(31)
    d = 50_000
    wl = custom(d, [0, d], [d], s, sparsifier, quantizer, R=1)
    for name, v in _adversarial(d, rng):
        P.run_parity(wl, 1, deltas=[v[None, :].copy()], expect_path=4)
    P.run_parity(wl, 1, flags=1, expect_path=1)                   # the same through the multi-pass kernels


def test_plan_query_agrees_with_what_the_kernels_report(P):
    # the host-only plan (qsl_plan_paths) and the path each unit reports after a call (no guess fails on these inputs)
    from paper_1906_02367_amd import binding as B
    off = [0, 100, 70_000, 70_001, 400_000, 410_001, 1_100_000]
    k = [100, 70, 1, 30_000, 10_001, 600]
    for sp, qz, s, flags in [(W.TOPK, W.QSGD, 16, 0), (W.RANDK, W.SIGN_L1, 1, 0), (W.TOPK, W.SIGN_L1, 1, 2), (W.TOPK, W.FP32, 1, 3)]:
        wl = custom(1_100_000, off, k, s, sp, qz, R=2)
        run, op, m_host, paths = P.run_parity(wl, 1, flags=flags)
        plan = B.plan_paths(wl.d, wl.seg_offset, wl.seg_k, wl.s, wl.sparsifier, wl.quantizer, flags)
        assert paths[0].reshape(2, len(k)).tolist() == [plan.tolist()] * 2, (paths[0], plan)


# ---------------------------------------------------------------------------------------------
# the other entry points
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("cfg", [1, 2, 4])
def test_aggregate_error_update_bits(P, cfg):
    from paper_1906_02367_amd import binding as B
    wl = W.config(cfg, d=80_000, R=4)
    run, op, m_host, _ = P.run_parity(wl, 2)
    q = run.q
    msgs_host = run.msg.cpu().numpy()
    # payload bits
    assert q.bits_sent(run.msg) == [op.bits_sent(msgs_host[r]) for r in range(wl.R)]
    # master line: all workers, then a subset accumulated onto x with scale -1/R
    out = torch.full((wl.d,), 7.0, dtype=torch.float32, device=q.device)
    q.aggregate(run.msg, out, 1.0 / wl.R)
    torch.cuda.synchronize()
    want = op.aggregate(msgs_host, 1.0 / wl.R)
    dense_abs = np.zeros(wl.d)
    for r in range(wl.R):
        i, v = op.decode(msgs_host[r])
        dense_abs[i] += np.abs(v.astype(np.float64))
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - want) <= 1e-6 * dense_abs / wl.R + 1e-38)
    x0 = np.random.default_rng(5).standard_normal(wl.d).astype(f32)
    out = torch.from_numpy(x0).to(q.device)
    q.aggregate(run.msg, out, -1.0 / wl.R, worker_list=[1, 3], accumulate=True)
    torch.cuda.synchronize()
    want = op.aggregate(msgs_host, -1.0 / wl.R, worker_list=[1, 3], out=x0)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - want) <= 1e-6 * (dense_abs / wl.R + np.abs(want)) + 1e-38)
    # stand-alone error update reproduces the fused one bit for bit
    rng = np.random.default_rng(9)
    m0 = rng.standard_normal((wl.R, wl.d)).astype(f32)
    d0 = W.delta_all(wl, 7)
    m_dev, d_dev = torch.from_numpy(m0).to(q.device), torch.from_numpy(d0).to(q.device)
    m_fused = torch.empty_like(m_dev)
    q.compress(m_dev, d_dev, m_fused, 0, 7, run.msg)
    q.error_update(m_dev, d_dev, run.msg)
    torch.cuda.synchronize()
    assert torch.equal(m_dev.view(torch.int32), m_fused.view(torch.int32))
    assert q.device_status() == B.OK


def test_nonfinite_input_is_reported(P):
    from paper_1906_02367_amd import binding as B
    wl = W.config(2, d=100_000, R=2)
    q = B.from_workload(wl)
    m = torch.zeros(2, wl.d, device=q.device)
    delta = torch.randn(2, wl.d, device=q.device)
    delta[1, 77_777] = float("inf")
    q.compress(m, delta, m, 0, 0, q.new_msg(2))
    assert q.device_status() == B.ERR_NONFINITE_INPUT
    assert q.device_status() == B.OK                     # the word is cleared by the query


def test_argument_errors_are_synchronous(P):
    from paper_1906_02367_amd import binding as B
    wl = W.config(2, d=10_000, R=2)
    q = B.from_workload(wl)
    m = torch.zeros(2, wl.d, device=q.device)
    with pytest.raises(B.QslError):
        q.compress(m, m, m, 0, 1 << 62, q.new_msg(2))                   # round out of range
    big = torch.zeros(3, wl.d, device=q.device)
    with pytest.raises(B.QslError):
        q.compress(big, big, big, 0, 0, q.new_msg(3))                   # R > max_workers
    with pytest.raises(B.QslError):
        B.Qsl(100, [0, 100], [101], 16, B.TOPK, B.QSGD, 1, 1)          # k > d
    with pytest.raises(B.QslError):
        q.aggregate(q.new_msg(2), torch.zeros(wl.d, device=q.device), 1.0, worker_list=[0, 0])


def test_results_do_not_depend_on_launch_history(P):
    # same inputs three times, with unrelated calls in between: identical bytes (no stale scratch)
    wl = W.config(2, d=1_000_003, R=2)
    from paper_1906_02367_amd import binding as B
    q = B.from_workload(wl)
    d0 = torch.from_numpy(W.delta_all(wl, 0)).to(q.device)
    d1 = torch.from_numpy(W.delta_all(wl, 1)).to(q.device)
    outs = []
    for rep in range(3):
        m = torch.zeros(2, wl.d, device=q.device)
        msg = q.new_msg(2)
        q.compress(m, d0, m, 0, 0, msg)
        outs.append((m.clone(), msg.clone()))
        junk = torch.zeros(2, wl.d, device=q.device)
        q.compress(junk, d1 * (rep + 1), junk, 0, 5, q.new_msg(2))
    torch.cuda.synchronize()
    for m, msg in outs[1:]:
        assert torch.equal(m.view(torch.int32), outs[0][0].view(torch.int32)) and torch.equal(msg, outs[0][1])


# ---------------------------------------------------------------------------------------------
# Delta = x_t - xhat_{t+1/2} formed on the fly (the synchronisation line of Algorithm 1 as written)
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("cfg,d,R", [(2, 1_000_003, 3), (3, 600_011, 2), (1, 65_536, 2), (4, 2_000_000, 5), (2, 70_001, 9)])
def test_compress_diff_matches_oracle_and_plain_entry(P, cfg, d, R):
    from paper_1906_02367_amd import binding as B
    wl = W.config(cfg, d=d, R=R)
    op = P.oracle_for(wl)
    q = B.from_workload(wl)
    rng = np.random.default_rng(cfg * 100 + R)
    x = rng.standard_normal(wl.d).astype(f32)
    m_host = (0.3 * W.delta_all(wl, 11)).astype(f32)
    for t in range(2):
        xhat = (x[None, :] - W.delta_all(wl, t)).astype(f32)            # so that x - xhat has the workload's shape
        m_dev, x_dev, xh_dev = (torch.from_numpy(a).to(q.device) for a in (m_host, x, xhat))
        msg, msg2 = q.new_msg(R).fill_(0xCD), q.new_msg(R)
        m_out, m_out2 = torch.empty_like(m_dev), torch.empty_like(m_dev)
        q.compress_diff(m_dev, x_dev, xh_dev, m_out, 3, t, msg)
        q.compress(m_dev, x_dev.unsqueeze(0) - xh_dev, m_out2, 3, t, msg2)
        torch.cuda.synchronize()
        assert q.device_status() == B.OK
        assert torch.equal(msg, msg2) and torch.equal(m_out.view(torch.int32), m_out2.view(torch.int32))
        want = [op.compress_diff(m_host[r], x, xhat[r], 3 + r, t) for r in range(R)]
        got_msg, got_m = msg.cpu().numpy(), m_out.cpu().numpy()
        for r in range(R):
            assert np.array_equal(got_msg[r], want[r]["msg"]), f"round {t} worker {r}: message differs"
            assert np.array_equal(P.bits(got_m[r]), P.bits(want[r]["m_out"])), f"round {t} worker {r}: memory differs"
        m_host = got_m


# ---------------------------------------------------------------------------------------------
# the counter of the random words at the far ends of its fields: round near 2^62, worker ids near
# 2^32, a 64-bit seed with the high bits set (Rand_k uses stream 0, the QSGD rounding stream 1)
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("d,k", [(9_001, 90), (300_007, 3_000)])
def test_random_word_counter_extremes(P, d, k):
    from paper_1906_02367_amd import binding as B
    seed = (1 << 64) - 59
    wl = custom(d, [0, d], [k], 5, W.RANDK, W.QSGD, R=2, seed=seed)
    op = P.oracle_for(wl)
    q = B.from_workload(wl)
    rng = np.random.default_rng(d)
    m_host = rng.standard_normal((2, d)).astype(f32)
    delta = rng.standard_normal((2, d)).astype(f32)
    for rnd, worker0 in [((1 << 62) - 1, (1 << 32) - 2), ((1 << 32) + 7, 0), ((1 << 61) + (1 << 31), 1 << 31)]:
        m_dev, d_dev = torch.from_numpy(m_host).to(q.device), torch.from_numpy(delta).to(q.device)
        msg = q.new_msg(2)
        q.compress(m_dev, d_dev, m_dev, worker0, rnd, msg)
        torch.cuda.synchronize()
        assert q.device_status() == B.OK
        got_msg, got_m = msg.cpu().numpy(), m_dev.cpu().numpy()
        for r in range(2):
            o = op.compress(m_host[r], delta[r], worker0 + r, rnd)
            assert np.array_equal(got_msg[r], o["msg"]), f"round {rnd} worker {worker0 + r}: message differs"
            assert np.array_equal(P.bits(got_m[r]), P.bits(o["m_out"])), f"round {rnd} worker {worker0 + r}: memory differs"
    with pytest.raises(B.QslError):
        q.compress(m_dev, d_dev, m_dev, 0, 1 << 62, msg)                  # round out of range
    with pytest.raises(B.QslError):
        q.compress(m_dev, d_dev, m_dev, (1 << 32) - 1, 0, msg)            # worker0 + R > 2^32


# ---------------------------------------------------------------------------------------------
# the paper's own per-tensor rule (Section 5.1.1): k_t = min(d_t, 1000) for every tensor -- whole small
# tensors, dense selections in the mid-sized ones, sparse ones in the large
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("quantizer,s", [(W.SIGN_L1, 1), (W.QSGD, 15), (W.SIGN_L3, 1), (W.SIGN_L4, 1)])
def test_per_tensor_rule_k_min_d_1000(P, quantizer, s):
    base = W.config(4, d=6_000_000, R=2)
    sizes = np.diff(base.seg_offset.astype(np.int64))
    k = np.minimum(sizes, 1000).astype(np.uint32)
    wl = W.Workload(4, "cfg4_k_min_d_1000", 2, base.d, base.seg_offset, k, s, W.TOPK, quantizer, 2, base.seed)
    run, op, m_host, paths = P.run_parity(wl, 2)
    assert set(paths[0].tolist()) == {0, 1, 3}, np.bincount(paths[0])


# ---------------------------------------------------------------------------------------------
# dense selections in many mid-sized segments: more multi-pass selection blocks than the GPU holds at once,
# so the blocks of one launch start at different times (a field of the unit state that one launch both read
# and rewrote once showed late blocks the new value here)
# ---------------------------------------------------------------------------------------------
def test_dense_k_in_many_segments_more_blocks_than_fit(P):
    rng = np.random.default_rng(5282)
    d, L, R = 3_328_894, 17, 3
    cuts = np.sort(rng.choice(np.arange(1, d), size=L - 1, replace=False))
    off = np.concatenate([[0], cuts, [d]]).astype(np.uint64)
    sizes = np.diff(off.astype(np.int64))
    k = np.maximum(1, (sizes * rng.uniform(0.05, 1.0, size=L)).astype(np.int64)).astype(np.uint32)
    wl = custom(d, off, k, 1, W.TOPK, W.SIGN_L1, R=R)
    deltas = [(rng.standard_normal((R, d)) * np.exp(2 * rng.standard_normal(d))).astype(f32) for _ in range(3)]
    run, op, m_host, paths = P.run_parity(wl, 3, deltas=deltas, worker0=55)
    assert (paths[0] == 1).sum() >= 30, np.bincount(paths[0])          # most of the 51 units take the multi-pass kernels


def test_side_stream_gives_the_same_bytes(P):
    # the library launches on whatever stream the caller hands it; two contexts on two streams at once
    from paper_1906_02367_amd import binding as B
    wl = W.config(2, d=1_000_003, R=2)
    d0 = torch.from_numpy(W.delta_all(wl, 0)).to("cuda")
    d1 = torch.from_numpy(W.delta_all(wl, 1)).to("cuda")
    qa, qb = B.from_workload(wl), B.from_workload(wl)
    ma, mb = torch.zeros(2, wl.d, device="cuda"), torch.zeros(2, wl.d, device="cuda")
    msga, msgb = qa.new_msg(2), qb.new_msg(2)
    xa, xb = torch.zeros(wl.d, device="cuda"), torch.zeros(wl.d, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for t, dl in enumerate((d0, d1)):
        qa.compress(ma, dl, ma, 0, t, msga)
        qa.aggregate(msga, xa, -0.5, accumulate=True)
        with torch.cuda.stream(side):
            qb.compress(mb, dl, mb, 0, t, msgb)
            qb.aggregate(msgb, xb, -0.5, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(msga, msgb) and torch.equal(ma.view(torch.int32), mb.view(torch.int32))
    assert torch.equal(xa.view(torch.int32), xb.view(torch.int32))
    assert qa.device_status() == B.OK and qb.device_status() == B.OK


# ---------------------------------------------------------------------------------------------
# the guess carried from call to call: what happens when the next call's values do not look like the last one's
# ---------------------------------------------------------------------------------------------
def test_guess_from_the_previous_call_survives_a_change_of_the_inputs(P):
    """From the second call on a guessing unit takes its threshold guess from the previous call's candidates.  Inputs
    that collapse (v a thousandth of what it was: too few candidates), then grow a millionfold (too many), then
    settle: every round bit for bit the oracle's; the round of a jump runs through the failure path (reported as
    path 2), the round after it is back on the short one."""
    d, k, R = 1_000_003, 1000, 2
    rng = np.random.default_rng(77)
    for qz, s, flags in [(W.QSGD, 16, 0), (W.SIGN_L1, 1, 0), (W.QSGD, 16, 8)]:       # 8: a fresh sample every call
        wl = custom(d, [0, d], [k], s, W.TOPK, qz, R)
        op = P.oracle_for(wl)
        deltas = [rng.standard_normal((R, d)).astype(f32) for _ in range(2)]
        m = np.zeros((R, d), dtype=f32)
        for t in range(2):                                   # the memory after two rounds, from the oracle
            m = np.stack([o["m_out"] for o in P.oracle_round(op, m, deltas[t], t)])
        deltas.append((-m + 1e-3 * rng.standard_normal((R, d))).astype(f32))          # v collapses
        deltas += [(rng.standard_normal((R, d)) * sc).astype(f32) for sc in (1e-3, 1e3, 1e3, 1.0, 1.0)]
        run, op, m_host, paths = P.run_parity(wl, len(deltas), deltas=deltas, flags=flags)
        seen = [sorted(set(p.tolist())) for p in paths]
        print("paths per round:", seen)
        assert seen[0] == [0] and seen[1] == [0]
        if flags == 0:
            assert 2 in seen[2] and 2 in seen[4], seen            # the rounds of the two jumps take the failure path ...
            assert seen[3] == [0] and seen[5] == [0] and seen[7] == [0], seen     # ... and the next ones do not
        else:
            assert all(sset == [0] for sset in seen), seen        # a fresh sample never fails on these inputs


# a failed guess made good by all blocks of a unit: values spread over many bins (the waves' parts hold them), and values of
# nearly one magnitude (one bin holds them all, the parts overflow and one block walks through v)
@pytest.mark.parametrize("d,k", [(300_007, 300), (1_000_003, 1000), (2_000_001, 20_000)])
@pytest.mark.parametrize("cluster", [False, True])
def test_failed_guess_made_good_by_many_blocks(P, d, k, cluster):
    rng = np.random.default_rng(d + cluster)
    R = 2
    deltas = [rng.standard_normal((R, d)).astype(f32) for _ in range(2)]
    x = 1e6 * (1.0 + 0.1 * rng.random((R, d))) * np.sign(rng.standard_normal((R, d))) if cluster else 1e4 * rng.standard_normal((R, d))
    deltas.append(x.astype(f32))
    wl = custom(d, [0, d], [k], 16, W.TOPK, W.QSGD, R)
    run, op, m_host, paths = P.run_parity(wl, 3, deltas=deltas)
    assert (paths[2] == 2).all(), paths[2]


def test_ties_at_the_threshold_beyond_the_short_list(P):
    """Thousands of equal magnitudes exactly at the threshold: the threshold's histogram bin holds more candidates
    than the short list takes, so one block selects the unit from its dense candidate list (ties to the lower
    coordinate)."""
    d, k, R = 1_000_003, 4000, 2
    rng = np.random.default_rng(78)
    wl = custom(d, [0, d], [k], 16, W.TOPK, W.QSGD, R)
    deltas = []
    for t in range(3):
        x = (rng.standard_normal((R, d)) * 0.01).astype(f32)
        for r in range(R):
            big = rng.choice(d, 6000, replace=False)
            x[r, big[:3000]] = (10.0 + rng.random(3000)).astype(f32) * np.sign(rng.standard_normal(3000)).astype(f32)
            x[r, big[3000:]] = f32(5.0) * np.sign(rng.standard_normal(3000)).astype(f32)     # 3000 ties; 1000 of them are kept
        deltas.append(x)
    run, op, m_host, paths = P.run_parity(wl, 3, deltas=deltas)
    print("paths:", [p.tolist() for p in paths])


def test_guess_carried_over_layerwise_and_rand_k(P):
    # several rounds on the segmented and the Rand_k shapes: guesses of many units carried along
    wl = W.config(4, d=6_000_000, R=3)
    P.run_parity(wl, 5)
    wl = W.config(3, d=2_000_003, R=2)
    P.run_parity(wl, 4, expect_path=0)
    wl = W.config(5, d=8_000_003, R=2)
    P.run_parity(wl, 4, expect_path=0)


# ---------------------------------------------------------------------------------------------
# every coordinate kept, index-free messages (the error-feedback schemes without sparsification that Section 5
# compares with, as this operator): two streaming passes
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("sparsifier", [W.TOPK, W.RANDK])
@pytest.mark.parametrize("quantizer,s", [(W.QSGD, 15), (W.QSGD, 1), (W.QSGD, 256), (W.QSGD, 32768), (W.SIGN_L1, 1),
                                         (W.SIGN_L2, 1), (W.FP32, 1), (W.QSGD_SCALED, 3), (W.SIGN_L3, 1), (W.SIGN_L4, 1)])
def test_index_free_format(P, sparsifier, quantizer, s):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(900 + s + quantizer)
    # one segment, ragged sizes around the 4096-coordinate tiles; many segments, tiny ones inside one tile included
    for d, off in [(1, [0, 1]), (4_095, [0, 4_095]), (300_001, [0, 300_001]),
                   (1_100_003, [0, 5, 70, 4_000, 4_097, 70_001, 400_000, 400_064, 1_100_003])]:
        k = np.diff(np.array(off, dtype=np.int64))
        wl = custom(d, off, k, s, sparsifier, quantizer, R=2)
        run, op, m_host, paths = P.run_parity(wl, 2, dense=True, expect_path=4, worker0=3)
        q = run.q
        msgs = run.msg.cpu().numpy()
        assert q.bits_sent(run.msg) == [op.bits_sent(msgs[r]) for r in range(wl.R)]
        w_code = 32 if quantizer == W.FP32 else 1 + (int(s).bit_length() if quantizer in (W.QSGD, W.QSGD_SCALED) else 0)
        assert q.bits_sent(run.msg)[0] == 32 + 32 * len(k) + d * w_code                    # the closed form
        # the master line and the stand-alone error update on such messages
        x0 = rng.standard_normal(d).astype(f32)
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(run.msg, out, -0.5, worker_list=[1, 0], accumulate=True)
        torch.cuda.synchronize()
        want = op.aggregate(msgs, -0.5, worker_list=[1, 0], out=x0)
        mag = sum(np.abs(op.decode(msgs[r])[1].astype(np.float64)) for r in (0, 1))
        assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - want) <= 1e-6 * (mag * 0.5 + np.abs(want)) + 1e-38)
        m0 = rng.standard_normal((2, d)).astype(f32)
        dl = rng.standard_normal((2, d)).astype(f32)
        m_dev, d_dev = torch.from_numpy(m0).to(q.device), torch.from_numpy(dl).to(q.device)
        m_fused, m_diff = torch.empty_like(m_dev), torch.empty_like(m_dev)
        msg2 = q.new_msg(2)
        q.compress(m_dev, d_dev, m_fused, 0, 7, run.msg)
        xx = torch.from_numpy(x0).to(q.device)
        q.compress_diff(m_dev, xx, xx.unsqueeze(0) - d_dev, m_diff, 0, 7, msg2)
        q.compress(m_dev, xx.unsqueeze(0) - (xx.unsqueeze(0) - d_dev), m_fused, 0, 7, run.msg)
        q.error_update(m_dev, xx.unsqueeze(0) - (xx.unsqueeze(0) - d_dev), run.msg)
        torch.cuda.synchronize()
        assert torch.equal(m_dev.view(torch.int32), m_fused.view(torch.int32))
        assert torch.equal(msg2, run.msg) and torch.equal(m_diff.view(torch.int32), m_fused.view(torch.int32))
        assert q.device_status() == B.OK
    # degenerate values
    d = 50_000
    wl = custom(d, [0, d], [d], s, sparsifier, quantizer, R=1)
    for name, v in _adversarial(d, rng):
        P.run_parity(wl, 1, deltas=[v[None, :].copy()], dense=True, expect_path=4)
    with pytest.raises(B.QslError):
        B.Qsl(100, [0, 100], [99], 16, B.TOPK, B.QSGD, 1, 1, flags=B.FLAG_DENSE_FORMAT)      # not every coordinate kept


# ---------------------------------------------------------------------------------------------
# the master line with many messages (from 12 on a kernel whose work is linear in the entries takes over)
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("case", ["long_sign_layerwise", "short_qsgd", "rand_fp32"])
def test_aggregate_many_messages(P, case):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(len(case))
    if case == "long_sign_layerwise":      # long messages, segments kept whole beside sparse ones (dense runs of entries)
        off = [0, 700, 1_724, 300_000, 301_000, 1_000_003]
        wl = custom(1_000_003, off, [700, 1_024, 9_000, 1_000, 3_000], 1, W.TOPK, W.SIGN_L1, R=8)
    elif case == "short_qsgd":
        wl = custom(300_007, [0, 300_007], [900], 16, W.TOPK, W.QSGD, R=8)
    else:
        wl = custom(70_001, [0, 64, 70_001], [64, 5_000], 1, W.RANDK, W.FP32, R=8)
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    msg = q.new_msg(64)
    m = torch.zeros(8, wl.d, device=q.device)
    for b in range(8):                                       # 64 messages, eight workers at a time
        delta = torch.from_numpy((rng.standard_normal((8, wl.d)) * np.exp(rng.standard_normal(wl.d))).astype(f32)).to(q.device)
        m.zero_()
        q.compress(m, delta, m, 8 * b, b, msg[8 * b: 8 * b + 8])
    torch.cuda.synchronize()
    msgs = msg.cpu().numpy()
    decoded = [op.decode(msgs[r]) for r in range(64)]
    x0 = rng.standard_normal(wl.d).astype(f32)
    for lst, accumulate in [(list(range(12)), True), ([int(x) for x in rng.permutation(64)[:33]], False), (list(range(63, -1, -1)), True)]:
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(msg, out, -1.0 / 64, worker_list=lst, accumulate=accumulate)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        # the library's own definition, written out: fp32 additions in list order, one rounding for the scale, one for the accumulate
        acc = np.zeros(wl.d, f32)
        has = np.zeros(wl.d, bool)
        for r in lst:
            i, v = decoded[r]
            acc[i] = np.where(has[i], acc[i] + v, v).astype(f32)
            has[i] = True
        term = (f32(-1.0 / 64) * acc).astype(f32)
        want = x0.copy() if accumulate else np.zeros(wl.d, f32)
        want[has] = (want[has] + term[has]).astype(f32) if accumulate else term[has]
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), (case, len(lst))
        # and the oracle's double sum within the tolerance of the aggregate
        ref = op.aggregate(msgs, -1.0 / 64, worker_list=lst, out=x0 if accumulate else None)
        mag = np.zeros(wl.d)
        for r in lst:
            i, v = decoded[r]
            mag[i] += np.abs(v.astype(np.float64))
        assert np.all(np.abs(got.astype(np.float64) - ref) <= 1e-6 * (mag / 64 + np.abs(ref)) + 1e-38)
    assert q.device_status() == B.OK


# ---------------------------------------------------------------------------------------------
# the master line on long messages whose coordinates are shared by all, by about half or by hardly any of the listed
# messages, call after call on one context, with lists that change
# ---------------------------------------------------------------------------------------------
def _aggregate_by_definition(decoded, lst, scale, x0, accumulate, d):
    acc = np.zeros(d, f32)
    has = np.zeros(d, bool)
    for r in lst:
        i, v = decoded[r]
        acc[i] = np.where(has[i], acc[i] + v, v).astype(f32)
        has[i] = True
    term = (f32(scale) * acc).astype(f32)
    want = x0.copy() if accumulate else np.zeros(d, f32)
    want[has] = (want[has] + term[has]).astype(f32) if accumulate else term[has]
    return want


@pytest.mark.parametrize("case", ["sign_layerwise", "qsgd_layerwise", "sign_one_segment"])
def test_aggregate_long_messages_shared_coordinates(P, case):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(77 + len(case))
    if case == "sign_layerwise":           # segments kept whole (at the same places in every message) beside sparse ones
        off = [0, 700, 1_724, 300_000, 301_000, 1_000_003]
        wl = custom(1_000_003, off, [700, 1_024, 9_000, 1_000, 3_000], 1, W.TOPK, W.SIGN_L1, R=8)
    elif case == "qsgd_layerwise":         # entries drop out: no two messages alike, whole segments included
        off = [0, 700, 1_724, 300_000, 301_000, 1_000_003]
        wl = custom(1_000_003, off, [700, 1_024, 9_000, 1_000, 3_000], 4, W.TOPK, W.QSGD, R=8)
    else:
        wl = custom(2_000_003, [0, 2_000_003], [20_000], 1, W.TOPK, W.SIGN_L1, R=8)
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    msg = q.new_msg(8)
    # what the workers share decides how many coordinates several messages hold: all, about half, hardly any
    common = (rng.standard_normal(wl.d) * np.exp(rng.standard_normal(wl.d))).astype(f32)
    for share in (1.0, 0.5, 0.0):
        own = (rng.standard_normal((8, wl.d)) * np.exp(rng.standard_normal(wl.d))).astype(f32)
        delta = torch.from_numpy((f32(share) * common[None, :] + f32(1.0 - share) * own).astype(f32)).to(q.device)
        m = torch.zeros(8, wl.d, device=q.device)
        q.compress(m, delta, m, 0, int(share * 10), msg)
        torch.cuda.synchronize()
        msgs = msg.cpu().numpy()
        decoded = [op.decode(msgs[r]) for r in range(8)]
        if share == 0.5:
            both = len(np.intersect1d(decoded[0][0], decoded[1][0]))
            assert 0 < both < len(decoded[0][0])
        x0 = rng.standard_normal(wl.d).astype(f32)
        for lst, accumulate in [(list(range(8)), True), ([5, 2], False), ([7, 0, 3, 6, 1], True), ([4], True),
                                (list(range(7, -1, -1)), False), ([1, 2, 3], True)]:
            out = torch.from_numpy(x0).to(q.device)
            q.aggregate(msg, out, -0.125, worker_list=lst, accumulate=accumulate)
            torch.cuda.synchronize()
            want = _aggregate_by_definition(decoded, lst, -0.125, x0, accumulate, wl.d)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, share, lst)
    # a message cut short (here: empty) among full ones: its coordinates are not at the places the others have them
    cut = msg.clone()
    cut[3].zero_()
    torch.cuda.synchronize()
    msgs = cut.cpu().numpy()
    decoded = [op.decode(msgs[r]) if r != 3 else (np.zeros(0, np.int64), np.zeros(0, f32)) for r in range(8)]
    for lst in ([3, 0, 1], [0, 1, 3, 2], list(range(8))):
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(cut, out, 0.5, worker_list=lst, accumulate=True)
        torch.cuda.synchronize()
        want = _aggregate_by_definition(decoded, lst, 0.5, x0, True, wl.d)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, "cut", lst)
    # ... and full lists again afterwards
    msgs = msg.cpu().numpy()
    decoded = [op.decode(msgs[r]) for r in range(8)]
    out = torch.from_numpy(x0).to(q.device)
    q.aggregate(msg, out, 1.0, accumulate=False)
    torch.cuda.synchronize()
    want = _aggregate_by_definition(decoded, list(range(8)), 1.0, x0, False, wl.d)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert q.device_status() == B.OK


# k_aggregate_cells at the edges of its dispatch: more segments in a cell than a wave's table holds, a vector of a few cells
# in many parts, a last cell of one coordinate, a message per lane, lists out of order
@pytest.mark.parametrize("case", ["tiny_segments", "few_cells", "one_coordinate_in_the_last_cell", "kept_whole_and_sparse"])
def test_aggregate_by_cells_edges(P, case):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(len(case))
    if case == "tiny_segments":            # 34 segments in every cell, 40 messages: scales read one by one
        off = list(range(0, 3_001, 30)) + [3_001]
        wl = custom(3_001, off, [min(7, b - a) for a, b in zip(off, off[1:])], 3, W.TOPK, W.QSGD, R=8)
        lists = [list(range(40)), [int(x) for x in rng.permutation(64)[:63]]]
    elif case == "few_cells":              # 69 cells with up to 4,600 entries: 16 waves per cell
        wl = custom(70_001, [0, 70_001], [5_000], 1, W.TOPK, W.SIGN_L1, R=8)
        lists = [list(range(64)), [9, 2, 40, 3], [int(x) for x in rng.permutation(64)[:31]]]
    elif case == "one_coordinate_in_the_last_cell":
        wl = custom(20_481, [0, 20_481], [6_000], 1, W.RANDK, W.FP32, R=8)
        lists = [list(range(17)), [63, 1], list(range(33))]
    else:
        off = [0, 900, 2_948, 200_000, 200_064, 260_000]
        wl = custom(260_000, off, [900, 2_048, 3_000, 64, 900], 1, W.TOPK, W.SIGN_L2, R=8)
        lists = [list(range(64)), [5, 3, 60, 2, 1, 8, 7], list(range(12))]
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    msg = q.new_msg(64)
    common = rng.standard_normal(wl.d).astype(f32)
    for b in range(8):
        own = rng.standard_normal((8, wl.d)).astype(f32)
        delta = torch.from_numpy(((common[None, :] + f32(b % 3) * own) * np.exp(rng.standard_normal(wl.d))).astype(f32)).to(q.device)
        m = torch.zeros(8, wl.d, device=q.device)
        q.compress(m, delta, m, 8 * b, b, msg[8 * b: 8 * b + 8])
    torch.cuda.synchronize()
    decoded = [op.decode(x) for x in msg.cpu().numpy()]
    x0 = rng.standard_normal(wl.d).astype(f32)
    for lst in lists:
        for accumulate in (True, False):
            out = torch.from_numpy(x0).to(q.device)
            q.aggregate(msg, out, -1.0 / 64, worker_list=lst, accumulate=accumulate)
            torch.cuda.synchronize()
            want = _aggregate_by_definition(decoded, lst, -1.0 / 64, x0, accumulate, wl.d)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, len(lst), accumulate)
    assert q.device_status() == B.OK


# a dense k on a large vector (the way of the window): inputs on which the window holds, and ones -- ties, zeros, one
# magnitude, scales in stretches -- on which the multi-pass kernels have to take over; against those kernels (NO_FAST_PATH),
# which the tests above compare with the oracle, and against the oracle itself.  What the kernels report shows which way a call
# went: 1 with candidates, the window held; 2, it was tried and failed; 1 without, it was left out (the two calls after a failure)
@pytest.mark.parametrize("kind,expect_held", [("normal", True), ("heavy", True), ("stretches", None), ("sorted", None), ("zeros", False),
                                              ("ties", False), ("constant", False)])
def test_window_of_a_dense_k(P, kind, expect_held):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(len(kind))
    # (the second to last: QSGD with two workers, below the size from which the window pays there -- it is left out)
    shapes = [(3_145_729, 50_001, W.TOPK, W.QSGD, 15, 3), (3_145_728, 2_900_000, W.TOPK, W.SIGN_L1, 1, 2), (3_200_003, 400_000, W.RANDK, W.FP32, 1, 1),
              (4_194_307, 314_573, W.TOPK, W.QSGD_SCALED, 3, 1), (4_194_303, 314_573, W.TOPK, W.QSGD, 3, 2), (3_145_733, 1_000_000, W.TOPK, W.SIGN_L4, 1, 1)]
    for d, k, sp, qz, s, R in shapes:
        left_out = qz == W.QSGD and R == 2
        wl = custom(d, [0, d], [k], s, sp, qz, R=R)
        qa, qb = B.from_workload(wl), B.from_workload(wl, flags=B.FLAG_NO_FAST_PATH)
        ma = torch.zeros(R, d, device=qa.device)
        mb = torch.zeros(R, d, device=qa.device)
        for t in range(4):
            ma.zero_(); mb.zero_()
            v = rng.standard_normal((R, d), dtype=f32)
            if kind == "heavy":
                v *= np.exp(2 * rng.standard_normal(d)).astype(f32)
            elif kind == "stretches":
                v *= np.repeat(np.exp(3 * rng.standard_normal(d // 700 + 1)), 700)[:d].astype(f32)
            elif kind == "sorted":
                v = np.sort(np.abs(v), axis=1)
            elif kind == "zeros":
                v[rng.random((R, d), dtype=f32) < 0.99] = 0
            elif kind == "ties":
                v = np.round(v * 4) / f32(4)
            elif kind == "constant":
                v[:] = 0.5
            delta = torch.from_numpy(v).to(qa.device)
            outs = []
            for q, m in ((qa, ma), (qb, mb)):
                msg, bits = q.new_msg(R).fill_(0xCD), torch.zeros(R, dtype=torch.int64, device=q.device)
                idx, lev = torch.zeros(R, k, dtype=torch.int32, device=q.device), torch.zeros(R, k, dtype=torch.int16, device=q.device)
                if t < 2:
                    q.compress(m, delta, m, 3, t, msg, bits, idx, lev)
                else:                                             # Delta formed on the fly: x = 0, xhat = -Delta
                    q.compress_diff(m, torch.zeros(d, device=q.device), -delta, m, 3, t, msg, bits, idx, lev)
                outs.append((m.view(torch.int32), msg, bits, idx, lev))
            torch.cuda.synchronize()
            assert qa.device_status() == B.OK and qb.device_status() == B.OK
            for a, b in zip(*outs):
                assert torch.equal(a, b), (kind, d, k, t)
            if t == 0:
                op = P.oracle_for(wl)
                o = op.compress(np.zeros(d, f32), v[0], 3, 0)
                assert np.array_equal(outs[0][1][0].cpu().numpy(), o["msg"]) and np.array_equal(P.bits(ma[0].cpu().numpy()), P.bits(o["m_out"]))
            units = qa.debug_units()
            if left_out:
                assert np.all((units[:, 0] == 1) & (units[:, 1] == 0)), (kind, d, k, t, units)
            elif expect_held or sp == W.RANDK:                    # (the keys of Rand_k do not depend on the values)
                assert np.all((units[:, 0] == 1) & (units[:, 1] > 0) & (units[:, 1] < d // 8)), (kind, d, k, t, units)
            elif expect_held is False:
                assert np.all(units[:, 0] == (2 if t in (0, 3) else 1)), (kind, d, k, t, units)
                # closed by the sample, or left out: nothing was listed; ties: listed, and too many in the threshold's bin
                assert np.all((units[:, 1] > 0) == (kind == "ties" and t in (0, 3))), (kind, d, k, t, units)
            assert np.all(qb.debug_units()[:, 0] == 1)


# index-free messages where the second pass and the master line change their way: norms outside the range of the short
# division, coordinates far below the norm, codes of 1, 8, 9 and 17 bits, the last chunk of one coordinate, the largest
# vector whose sums one block adds up (1024 rows of 4096 coordinates) and the one after it, tables that just fit or do not
@pytest.mark.parametrize("d,quantizer,s,factor", [
    (5_003, W.QSGD, 15, 1e-30), (5_003, W.QSGD, 15, 1e25), (5_003, W.QSGD_SCALED, 3, "mixed"), (1_025, W.QSGD, 127, 1.0), (1_024, W.QSGD, 128, 1.0),
    (1_023, W.QSGD, 32768, "mixed"), (2_049, W.QSGD, 1, 1e-13), (4_097, W.SIGN_L1, 1, 1.0), (3_001, W.FP32, 1, "mixed"), (4_194_304, W.QSGD, 4, 1.0),
    (4_194_305, W.QSGD, 4, 1.0), (4_194_305, W.SIGN_L2, 1, 1.0)])
def test_index_free_edges(P, d, quantizer, s, factor):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d + s)
    R = 2 if d > 100_000 else 34
    wl = custom(d, [0, d], [d], s, W.TOPK, quantizer, R=R)
    v = rng.standard_normal((1, R, d)).astype(f32)
    if factor == "mixed":                                # the norm comes from a few; the others lie up to 10^30 below it, some are zero
        v *= (10.0 ** rng.uniform(-30, 0, size=(1, R, d))).astype(f32)
        v[0, :, ::7] = 0
    else:
        v = (v * f32(factor)).astype(f32)
    run, op, m_host, _ = P.run_parity(wl, 1, deltas=v, dense=True, expect_path=4, worker0=7)
    decoded = [op.decode(x) for x in run.msg.cpu().numpy()]
    x0 = (rng.standard_normal(d) * np.abs(v).max()).astype(f32)
    for lst, accumulate in [(list(range(R)), True), ([1], False), ([1, 0] + list(range(2, min(R, 9))), True)]:
        out = torch.from_numpy(x0).to(run.q.device)
        run.q.aggregate(run.msg, out, -0.25, worker_list=lst, accumulate=accumulate)
        torch.cuda.synchronize()
        want = _aggregate_by_definition(decoded, lst, -0.25, x0, accumulate, d)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (d, quantizer, s, lst)
    assert run.q.device_status() == B.OK


# guessing units of a single block with more candidates than the list in LDS takes (13,500 of 8192), with more slot rows than a wave
# keeps in registers, with chunks that spill to the overflow pool, with ties beyond the short list; beside them units that one block
# selects from v, in the same launch; against the multi-pass kernels, and one worker against the oracle
@pytest.mark.parametrize("sparsifier,quantizer,s,dense_unit", [(W.TOPK, W.SIGN_L1, 1, True), (W.TOPK, W.QSGD, 15, False), (W.TOPK, W.FP32, 1, True),
                                                               (W.RANDK, W.QSGD, 4, True), (W.RANDK, W.SIGN_L2, 1, False)])
def test_single_block_units_with_long_lists(P, sparsifier, quantizer, s, dense_unit):
    from paper_1906_02367_amd import binding as B
    R, sizes, ks = 32, [600_011, 90_001, 20_003, 70_000] * 2, [9_000, 90, 20, 1_000] * 2
    if dense_unit:
        sizes.append(36_864); ks.append(3_000)
    off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    d = off[-1]
    wl = custom(d, off, ks, s, sparsifier, quantizer, R=R)
    assert set(B.plan_paths(d, wl.seg_offset, wl.seg_k, s, sparsifier, quantizer).tolist()) == ({0, 3} if dense_unit else {0})
    qa, qb, op = B.from_workload(wl), B.from_workload(wl, flags=B.FLAG_NO_FAST_PATH), P.oracle_for(wl)
    g = torch.Generator(device=qa.device); g.manual_seed(11)
    m = torch.zeros(R, d, device=qa.device)
    for t in range(3):
        delta = torch.randn(R, d, generator=g, device=qa.device)
        delta[:, 5_000:5_700] *= 50                              # one chunk and a half of large values
        if t == 2:
            delta = torch.round(delta)
        outs = []
        for q in (qa, qb):
            msg, m_out = q.new_msg(R).fill_(0xCD), torch.empty_like(m)
            q.compress(m, delta, m_out, 0, t, msg)
            outs.append((msg, m_out))
        torch.cuda.synchronize()
        assert qa.device_status() == B.OK and qb.device_status() == B.OK
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1].view(torch.int32), outs[1][1].view(torch.int32)), t
        units = qa.debug_units()
        if t == 0:
            assert not np.any(units[:, 0] == 2) and units[:, 1].max() > 8_192
            o = op.compress(np.zeros(d, f32), delta[R - 1].cpu().numpy(), R - 1, 0)
            assert np.array_equal(outs[0][0][R - 1].cpu().numpy(), o["msg"]) and np.array_equal(P.bits(outs[0][1][R - 1].cpu().numpy()), P.bits(o["m_out"]))
        m = outs[0][1]


# directories of messages with many entries per 1024 coordinates, by search (the large lists, see directory_by_search) or by reading every entry:
# entries that lie evenly, that all lie far from where an even message would have them, a last cell of one coordinate; messages of QSGD
# that are shorter than expected, and empty
@pytest.mark.parametrize("d,k,quantizer,s,where,R", [
    (300_033, 30_000, W.SIGN_L1, 1, "even", 5), (300_033, 30_000, W.FP32, 1, "front", 5), (409_601, 40_000, W.SIGN_L1, 1, "back", 5),
    (409_600, 40_000, W.QSGD, 1_000, "back", 5), (5_000, 4_500, W.SIGN_L2, 1, "front", 5),
    (300_033, 60_000, W.SIGN_L1, 1, "even", 50), (300_033, 60_000, W.FP32, 1, "front", 50), (409_601, 82_000, W.SIGN_L1, 1, "back", 40),
    (409_600, 90_000, W.QSGD, 1_000, "back", 64), (51_000, 50_000, W.SIGN_L2, 1, "front", 60)])
def test_aggregate_directory_by_search(P, d, k, quantizer, s, where, R):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d)
    wl = custom(d, [0, d], [k], s, W.TOPK, quantizer, R=R)
    q, op = B.from_workload(wl), P.oracle_for(wl)
    v = rng.standard_normal((R, d)).astype(f32)
    if where != "even":
        v[:, slice(0, k + 999) if where == "front" else slice(d - k - 999, d)] *= 1e3
    v[3] = 0
    msg, m = q.new_msg(R), torch.zeros(R, d, device=q.device)
    q.compress(m, torch.from_numpy(v).to(q.device), m, 0, 0, msg)
    torch.cuda.synchronize()
    decoded = [op.decode(x) for x in msg.cpu().numpy()]
    x0 = rng.standard_normal(d).astype(f32)
    for lst, accumulate in ((list(range(R)), True), ([4, 3, 1, 0], False)):
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(msg, out, -1.0 / R, worker_list=lst, accumulate=accumulate)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), _aggregate_by_definition(decoded, lst, -1.0 / R, x0, accumulate, d).view(np.uint32)), lst
    assert q.device_status() == B.OK


# the stand-alone error update, in one launch up to 2^23 coordinates of all rows and in two beyond: m + delta - g in single operations,
# messages that hold nothing, everything or the ends of chunks only, segments (more than 64 to a chunk, ends on the ends of chunks), a last
# chunk of one coordinate; an index >= d is reported
@pytest.mark.parametrize("d,off,k,quantizer,s,R", [(1, [0, 1], [1], W.FP32, 1, 2), (1_025, [0, 1_025], [1_025], W.SIGN_L1, 1, 2), (5_121, [0, 1_000, 5_121], [1_000, 9], W.QSGD, 3, 3),
                                                   (70_001, [0, 70_001], [40], W.SIGN_L2, 1, 2), (3_000, list(range(0, 3_001, 5)), [2, 5] * 300, W.SIGN_L1, 1, 2),
                                                   (5_121, [0, 1, 1_024, 2_048, 2_049, 3_071, 5_121], [1, 1_000, 1_024, 1, 1_022, 3], W.SIGN_L2, 1, 2), (1_048_577, [0, 1_048_577], [30_000], W.FP32, 1, 8), (1_048_576, [0, 1_048_576], [30_000], W.QSGD, 15, 8)])
def test_error_update_launches(P, d, off, k, quantizer, s, R):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d)
    wl = custom(d, off, k, s, W.TOPK, quantizer, R=R)
    q, op = B.from_workload(wl), P.oracle_for(wl)
    m0, delta = rng.standard_normal((R, d)).astype(f32), rng.standard_normal((R, d)).astype(f32)
    edge = np.arange(d) % 1_024
    delta[0, (edge == 0) | (edge == 1_023)] *= 100
    m0[R - 1], delta[R - 1] = 0, 0                               # QSGD sends nothing
    m, dl = torch.from_numpy(m0).to(q.device), torch.from_numpy(delta).to(q.device)
    msg, v = q.new_msg(R), torch.empty_like(m)
    q.compress(m, dl, v, 0, 0, msg)
    q.error_update(m, dl, msg)
    torch.cuda.synchronize()
    assert q.device_status() == B.OK
    host = msg.cpu().numpy()
    for r in (0, R - 1):
        want = m0[r] + delta[r]
        i, g = op.decode(host[r])
        want[i] = want[i] - g.astype(f32)
        assert np.array_equal(P.bits(m[r].cpu().numpy()), P.bits(want)), r
    if d == 70_001:                                              # the last index beyond the vector
        bits = np.unpackbits(host[0], bitorder="little")
        bits[64 + 39 * 17: 64 + 40 * 17] = (d + 1 >> np.arange(17)) & 1
        bad = torch.from_numpy(np.stack([np.packbits(bits, bitorder="little"), host[1]])).to(q.device)
        q.error_update(m, dl, bad)
        torch.cuda.synchronize()
        assert q.device_status() != B.OK


# messages with indices >= d in the stand-alone error update: each such entry is reported and skipped, wherever it stands and however many
# there are; every other entry is subtracted
@pytest.mark.parametrize("d,off,k,quantizer,s", [(70_001, [0, 70_001], [3_000], W.SIGN_L1, 1), (70_001, [0, 30_000, 70_001], [1_000, 2_000], W.QSGD, 15),
                                                 (5_000, [0, 5_000], [5_000], W.FP32, 1), (1_500_001, [0, 1_500_001], [20_000], W.SIGN_L2, 1)])
def test_error_update_malformed_indices(P, d, off, k, quantizer, s):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d + s)
    wl = custom(d, off, k, s, W.TOPK, quantizer, R=2)
    q, op = B.from_workload(wl), P.oracle_for(wl)
    m0, delta = rng.standard_normal((2, d)).astype(f32), rng.standard_normal((2, d)).astype(f32)
    dl = torch.from_numpy(delta).to(q.device)
    msg, v = q.new_msg(2), torch.empty(2, d, device=q.device)
    q.compress(torch.from_numpy(m0).to(q.device), dl, v, 0, 0, msg)
    torch.cuda.synchronize()
    good = msg.cpu().numpy()
    i0, g0 = op.decode(good[0])
    i1, g1 = op.decode(good[1])
    n, w_idx, L = i0.size, (d - 1).bit_length(), len(k)
    bit0 = 32 * (1 + L + (L if quantizer == W.QSGD and L > 1 else 0))
    other = m0[1] + delta[1]
    other[i1] = other[i1] - g1.astype(f32)
    for where in ([0], [n // 2], [n - 1], [16 * n // 33], [32 * n // 33], range(n // 3, n // 2), range(0, n, 2), range(1, n), range(n)):
        where = np.array(where)
        bad = good.copy()
        bits = np.unpackbits(bad[0], bitorder="little")
        for j in where:
            bits[bit0 + j * w_idx: bit0 + (j + 1) * w_idx] = ((d if j % 3 else (1 << w_idx) - 1) >> np.arange(w_idx)) & 1
        bad[0] = np.packbits(bits, bitorder="little")
        m = torch.from_numpy(m0).to(q.device)
        q.error_update(m, dl, torch.from_numpy(bad).to(q.device))
        assert q.device_status() == B.ERR_DEVICE and q.device_status() == B.OK, where[:3]
        keep = np.ones(n, bool)
        keep[where] = False
        want = m0[0] + delta[0]
        want[i0[keep]] = want[i0[keep]] - g0[keep].astype(f32)
        got = m.cpu().numpy()
        assert np.array_equal(P.bits(got[0]), P.bits(want)) and np.array_equal(P.bits(got[1]), P.bits(other)), where[:3]


# short vectors, one launch per call: both sides of the limits (4096, 8192, 16,384 coordinates, 4096 selected ones, guesses from 1024 groups
# and from groups of four), ties that the guess lets through or not, ties at the threshold in several waves, an update formed from models
@pytest.mark.parametrize("d,k", [(1, 1), (63, 40), (4_095, 513), (4_097, 1), (4_097, 4_096), (8_192, 512), (8_192, 1_024), (8_193, 1_025), (8_193, 2_049),
                                 (16_383, 4_096), (16_384, 512), (16_384, 2_048), (16_384, 4_097), (16_385, 300)])
@pytest.mark.parametrize("sparsifier,quantizer,s", [(W.TOPK, W.QSGD, 15), (W.TOPK, W.FP32, 1), (W.TOPK, W.SIGN_L4, 1), (W.RANDK, W.QSGD_SCALED, 4), (W.RANDK, W.SIGN_L1, 1)])
def test_short_vectors(P, d, k, sparsifier, quantizer, s):
    rng = np.random.default_rng(d + k)
    R = 3
    wl = custom(d, [0, d], [k], s, sparsifier, quantizer, R=R)
    v = rng.standard_normal((4, R, d)).astype(f32)
    v[1] = np.round(v[1] * 2)                                # few magnitudes
    v[2, :, rng.random(d) < 0.99] = 0                        # fewer values than places
    v[3, 0] = 1.5
    run, op, m_host, _ = P.run_parity(wl, 4, deltas=v, worker0=5)
    x, xhat = rng.standard_normal(d).astype(f32), rng.standard_normal((R, d)).astype(f32)
    dev = run.q.device
    m = torch.from_numpy(m_host).to(dev)
    msg = run.q.new_msg(R).fill_(0xCD)
    run.q.compress_diff(m, torch.from_numpy(x).to(dev), torch.from_numpy(xhat).to(dev), m, 5, 4, msg)
    torch.cuda.synchronize()
    for r in range(R):
        o = op.compress(m_host[r], x - xhat[r], 5 + r, 4)
        assert np.array_equal(msg[r].cpu().numpy(), o["msg"]) and np.array_equal(P.bits(m[r].cpu().numpy()), P.bits(o["m_out"]))


# the master line in one launch (up to 35 messages; lists of 64 go by cells): ranges of 512 coordinates, segments, entries shared by all
# messages; few messages with many entries (64 of them are looked at first, one in 2 .. 128), all of them in one range or everywhere
@pytest.mark.parametrize("d,off,k,quantizer,s,R", [(1, [0, 1], [1], W.SIGN_L1, 1, 2), (511, [0, 511], [100], W.FP32, 1, 33), (513, [0, 200, 513], [40, 60], W.QSGD, 3, 64),
                                                   (100_001, [0, 100_001], [128], W.SIGN_L1, 1, 64), (5_000, [0, 100, 5_000], [100, 400], W.SIGN_L2, 1, 9),
                                                   (70_001, [0, 70_001], [234], W.FP32, 1, 35), (1_025, [0, 1_025], [64], W.FP32, 1, 24), (1_025, [0, 1_025], [65], W.SIGN_L1, 1, 24),
                                                   (262_144, [0, 262_144], [8_192], W.SIGN_L1, 1, 1), (20_001, [0, 3_000, 20_001], [2_990, 1_000], W.FP32, 1, 2),
                                                   (9_001, [0, 9_001], [4_095], W.QSGD, 32, 2), (60_000, [0, 59_000, 60_000], [10, 999], W.SIGN_L2, 1, 3)])
def test_aggregate_small(P, d, off, k, quantizer, s, R):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d + R)
    wl = custom(d, off, k, s, W.TOPK, quantizer, R=R)
    q, op = B.from_workload(wl), P.oracle_for(wl)
    v = (rng.standard_normal((R, d)) * np.exp(2 * rng.standard_normal(d))).astype(f32)
    v[1 % R] = 0                                             # zeros kept, of both signs (a QSGD message of none)
    v[1 % R, ::2] = -0.0
    msg, m = q.new_msg(R), torch.zeros(R, d, device=q.device)
    q.compress(m, torch.from_numpy(v).to(q.device), m, 0, 0, msg)
    torch.cuda.synchronize()
    decoded = [op.decode(x) for x in msg.cpu().numpy()]
    x0 = rng.standard_normal(d).astype(f32)
    x0[::3] = -0.0
    for lst in (list(range(R)), [R - 1, 0] if R > 1 else [0], list(rng.permutation(R))):
        for accumulate in (False, True):
            out = torch.from_numpy(x0).to(q.device)
            q.aggregate(msg, out, -1.0 / R, worker_list=[int(r) for r in lst], accumulate=accumulate)
            torch.cuda.synchronize()
            want = _aggregate_by_definition(decoded, lst, -1.0 / R, x0, accumulate, d)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (lst, accumulate)
    assert q.device_status() == B.OK


# ... and with malformed messages: every index >= d is reported and skipped, wherever it stands (the last block is a ragged one), and no
# other entry is lost; a length above K is K
@pytest.mark.parametrize("d,off,k,quantizer,s,R,accumulate", [(50_001, [0, 50_001], [200], W.SIGN_L1, 1, 32, True), (50_001, [0, 50_001], [1_500], W.FP32, 1, 4, False),
                                                              (3_001, [0, 700, 3_001], [30, 25], W.QSGD, 15, 4, False), (200_001, [0, 200_001], [8_000], W.SIGN_L2, 1, 1, False),
                                                              (9_000, [0, 4_000, 9_000], [1_000, 3_000], W.SIGN_L1, 1, 2, False), (20_001, [0, 20_001], [100], W.FP32, 1, 8, False)])
def test_aggregate_small_malformed(P, d, off, k, quantizer, s, R, accumulate):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(d + R)
    wl = custom(d, off, k, s, W.TOPK, quantizer, R=R)
    q, op = B.from_workload(wl), P.oracle_for(wl)
    msg, m = q.new_msg(R), torch.zeros(R, d, device=q.device)
    q.compress(m, torch.from_numpy(rng.standard_normal((R, d)).astype(f32)).to(q.device), m, 0, 0, msg)
    torch.cuda.synchronize()
    good = msg.cpu().numpy()
    decoded = [op.decode(x) for x in good]
    n, w_idx, L, r = decoded[R - 1][0].size, (d - 1).bit_length(), len(k), R - 1
    bit0 = 32 * (1 + L + (L if quantizer == W.QSGD and L > 1 else 0))
    x0 = rng.standard_normal(d).astype(f32)

    def check(bad, entries, status):
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(torch.from_numpy(bad).to(q.device), out, -0.5, accumulate=accumulate)
        assert q.device_status() == status and q.device_status() == B.OK
        want = _aggregate_by_definition(decoded[:r] + [entries], list(range(R)), -0.5, x0, accumulate, d)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))

    for where in ([0], [1], [n // 2], [n - 1], [n * 40 // 64], range(n // 3, n // 2), range(0, n, 2), range(1, n), range(n)):
        where = np.array(where)
        bad, keep = good.copy(), np.ones(n, bool)
        bits = np.unpackbits(bad[r], bitorder="little")
        for j in where:
            bits[bit0 + j * w_idx: bit0 + (j + 1) * w_idx] = ((d if j % 3 else (1 << w_idx) - 1) >> np.arange(w_idx)) & 1
        bad[r] = np.packbits(bits, bitorder="little")
        keep[where] = False
        check(bad, tuple(x[keep] for x in decoded[r]), B.ERR_DEVICE)
    if quantizer != W.QSGD:
        bad = good.copy()
        bad[r, :4].view(np.uint32)[0] = sum(k) + 7
        check(bad, decoded[r], B.OK)


# ... and with a message that holds more entries than one of its operator is expected to (QSGD; written by hand: all of level 1)
@pytest.mark.parametrize("n", [128, 129, 300, 5_000])
def test_aggregate_small_longer_than_expected(P, n):
    from paper_1906_02367_amd import binding as B
    d, rng = 200_001, np.random.default_rng(n)
    wl = custom(d, [0, d], [10_000], 1, W.TOPK, W.QSGD, R=2)                    # expected: 125 entries at most
    q, op = B.from_workload(wl), P.oracle_for(wl)
    w_idx, x0 = (d - 1).bit_length(), rng.standard_normal(d).astype(f32)
    for at in (None, 3, 70, n - 1):                                            # an entry with an index >= d
        msgs = np.zeros((2, q.capacity), np.uint8)
        decoded = []
        for r in range(2):
            idx = np.sort(rng.choice(d, n, replace=False))
            neg = rng.integers(0, 2, n)
            if at is not None and r == 1:
                idx[at] = d
            fields = ((idx[:, None] >> np.arange(w_idx)) & 1).astype(np.uint8).ravel()
            words = 2 + (n * w_idx + 31) // 32
            bits = np.zeros(msgs.shape[1] * 8, np.uint8)
            bits[64: 64 + fields.size] = fields
            bits[32 * words: 32 * words + n] = neg                            # s = 1: a code is the sign
            msgs[r] = np.packbits(bits, bitorder="little")
            msgs[r, :8].view(np.uint32)[:] = [n, np.float32(1.5 + r).view(np.uint32)]
            i, v = (idx, np.where(neg, -1.0, 1.0) * (1.5 + r))
            keep = idx < d
            decoded.append((i[keep], v[keep].astype(f32)))
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(torch.from_numpy(msgs).to(q.device), out, -0.5)
        assert q.device_status() == (B.OK if at is None else B.ERR_DEVICE)
        if at is None:
            for r in range(2):
                i, v = op.decode(msgs[r])
                assert np.array_equal(i, decoded[r][0]) and np.array_equal(v.astype(f32), decoded[r][1])
        want = _aggregate_by_definition(decoded, [0, 1], -0.5, x0, False, d)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), at


# ... whose time goes with the entries, not with how many of the messages there are: one message of 8192 takes what eight of 1024 take
# (30.5 against 8.4 us when a wave went through the whole of each of its messages)
def test_aggregate_small_time_of_few_messages(P):
    def us(R):
        wl = custom(130_003, [0, 130_003], [8_192 // R], 1, W.TOPK, W.SIGN_L1, R=R)
        from paper_1906_02367_amd import binding as B
        q = B.from_workload(wl)
        msg, m, out = q.new_msg(R), torch.zeros(R, wl.d, device=q.device), torch.zeros(wl.d, device=q.device)
        q.compress(m, torch.randn(R, wl.d, device=q.device), m, 0, 0, msg)
        best = 1e9
        for _ in range(10):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(50):
                q.aggregate(msg, out, 0.5)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) * 20)
        return best
    one, eight = us(1), us(8)
    assert one < 2 * eight, (one, eight)


# index-free messages of one segment: the norm of values from the smallest subnormal to 1e36, side by side in one wave (several windows
# of exponents), alone in a chunk, and only subnormal ones; chunks of zeros; a last chunk of one coordinate.  Bit for bit (exact sums).
@pytest.mark.parametrize("quantizer,s", [(W.SIGN_L1, 1), (W.SIGN_L2, 1), (W.QSGD, 15)])
@pytest.mark.parametrize("d,kind", [(6_145, "all"), (6_145, "subnormal"), (1_024, "zeros"), (66_561, "windows"), (1, "all")])
def test_index_free_norms_over_the_whole_range(P, quantizer, s, d, kind):
    rng = np.random.default_rng(d + s)
    v = rng.standard_normal((2, 2, d)).astype(f32)
    if kind == "all":
        v = np.ldexp(v, rng.integers(-148, 119, v.shape)).astype(f32)
    elif kind == "subnormal":
        v = (v * f32(1e-40)).astype(f32)
        v[:, :, 1_024:2_048] = 0
    elif kind == "zeros":
        v[:] = 0
    else:                                                # chunk c: magnitudes around 2^(4 c - 140), a few others 2^30 and 2^64 below them
        e = np.repeat(np.arange(66) * 4 - 140, 1_024)[:d]
        e = np.concatenate([e, np.full(d - e.size, 0)])
        v = np.ldexp(v, np.maximum(e - rng.choice([0, 0, 0, 29, 30, 31, 32, 64], v.shape), -149)).astype(f32)
    P.run_parity(custom(d, [0, d], [d], s, W.TOPK, quantizer, R=2), 2, deltas=v, dense=True, expect_path=4)


# a message with an index >= d: reported by the status word (once), the entry skipped, everything else added up
# as ever -- whichever kernel meets it: one wave per cell, a cell in parts (where the entry lies behind d, in a part that has
# no coordinates), a last cell that the plan calls crowded, short messages, look-ups
@pytest.mark.parametrize("case", ["cells", "parts", "crowded_last_cell", "short", "lookups", "qsgd_segments"])
def test_aggregate_reports_malformed_indices(P, case):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(len(case))
    d, off, k, s, qz, R = {"cells": (300_001, [0, 300_001], [5_000], 1, W.SIGN_L1, 8),
                           "parts": (70_001, [0, 70_001], [5_000], 1, W.SIGN_L1, 64),          # 16 parts of 64; 369 coordinates in the last cell
                           "crowded_last_cell": (260_100, [0, 259_700, 260_100], [6_000, 400], 1, W.SIGN_L2, 24),
                           "short": (50_001, [0, 50_001], [500], 1, W.FP32, 40),
                           "lookups": (9_000_001, [0, 9_000_001], [5_000], 1, W.SIGN_L1, 2),
                           "qsgd_segments": (300_001, [0, 900, 300_001], [900, 9_000], 15, W.QSGD, 12)}[case]
    wl = custom(d, off, k, s, W.TOPK, qz, R=R)
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    msg = q.new_msg(R)
    delta = torch.from_numpy(rng.standard_normal((R, d)).astype(f32)).to(q.device)
    m = torch.zeros(R, d, device=q.device)
    q.compress(m, delta, m, 0, 0, msg)
    torch.cuda.synchronize()
    good = msg.cpu().numpy()
    decoded = [op.decode(x) for x in good]
    w_idx, L = (d - 1).bit_length(), len(k)
    bit0 = 32 * (1 + L + (L if qz == W.QSGD and L > 1 else 0))
    x0 = rng.standard_normal(d).astype(f32)

    def patched(r, j, value):
        bad = good.copy()
        bits = np.unpackbits(bad[r], bitorder="little")
        at = bit0 + j * w_idx
        bits[at: at + w_idx] = (value >> np.arange(w_idx)) & 1
        bad[r] = np.packbits(bits, bitorder="little")
        return torch.from_numpy(bad).to(q.device)

    for r in (0, R - 1):
        n = int(good[r].view(np.uint32)[0])
        for value in (d, (1 << w_idx) - 1):              # the message's last entry: its order stays right
            out = torch.from_numpy(x0).to(q.device)
            q.aggregate(patched(r, n - 1, value), out, -0.5, accumulate=True)
            assert q.device_status() == B.ERR_DEVICE and q.device_status() == B.OK, (case, r, value)
            rest = [(i[:-1], v[:-1]) if p == r else (i, v) for p, (i, v) in enumerate(decoded)]
            want = _aggregate_by_definition(rest, list(range(R)), -0.5, x0, True, d)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, r, value)
        out = torch.from_numpy(x0).to(q.device)          # in the middle: what else happens to that message is open
        q.aggregate(patched(r, n // 2, d), out, -0.5, accumulate=True)
        assert q.device_status() == B.ERR_DEVICE and q.device_status() == B.OK, (case, r, "middle")
    out = torch.from_numpy(x0).to(q.device)
    q.aggregate(msg, out, -0.5, accumulate=True)
    assert q.device_status() == B.OK
    assert np.array_equal(out.cpu().numpy().view(np.uint32), _aggregate_by_definition(decoded, list(range(R)), -0.5, x0, True, d).view(np.uint32))


# NaNs of every kind in a message reach the model, through each way of the master line: none of them stands for "no entry"
@pytest.mark.parametrize("R,d,k", [(8, 300_001, 5_000), (64, 70_001, 5_000), (40, 50_001, 500), (2, 50_001, 500)])
@pytest.mark.parametrize("quantizer", [W.FP32, W.SIGN_L1])
def test_aggregate_keeps_nans(P, R, d, k, quantizer):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(R)
    wl = custom(d, [0, d], [k], 1, W.TOPK, quantizer, R=R)
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    msg = q.new_msg(R)
    base = rng.standard_normal(d).astype(f32)
    base[100:104] = 50.0                                  # four coordinates that every message holds
    v = (base[None, :] + rng.standard_normal((R, d))).astype(f32)
    m = torch.zeros(R, d, device=q.device)
    q.compress(m, torch.from_numpy(v).to(q.device), m, 0, 0, msg)
    torch.cuda.synchronize()
    good = msg.cpu().numpy()
    decoded = [op.decode(x) for x in good]
    bad = good.copy()
    if quantizer == W.FP32:                               # the codes are the values
        n_idx = (k * (d - 1).bit_length() + 31) // 32
        for r, coord, code in ((0, 100, 0xFFFFFFFF), (R - 1, 101, 0xFFFFFFFF), (R // 2, 102, 0xFFBFFFFF), (0, 103, 0x7FC00000), (R - 1, 103, 0xFFFFFFFF)):
            bad[r].view(np.uint32)[2 + n_idx + int(np.searchsorted(decoded[r][0], coord))] = code
        nan_at = np.arange(100, 104)
    else:                                                 # the scale: its negative is the NaN with all bits set
        bad[R - 1].view(np.uint32)[1] = 0x7FFFFFFF
        nan_at = decoded[R - 1][0].astype(np.int64)
    x0 = rng.standard_normal(d).astype(f32)
    for accumulate in (True, False):
        out = torch.from_numpy(x0).to(q.device)
        q.aggregate(torch.from_numpy(bad).to(q.device), out, -1.0 / R, accumulate=accumulate)
        torch.cuda.synchronize()
        want = _aggregate_by_definition(decoded, list(range(R)), -1.0 / R, x0, accumulate, d)
        got = out.cpu().numpy()
        assert np.all(np.isnan(got[nan_at]))
        got[nan_at] = want[nan_at] = 0
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


# guessing units of a single block (segments x workers >= 256 blocks), small ones and ones that the host is to hear about as
# walked through by one block: thresholds that jump down and up, too few non-zero values, ties; two jumps in a row
def test_failed_guesses_of_single_block_units(P):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(31)
    sizes = [140_001, 20_003] * 8
    off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    R = 16
    wl = custom(off[-1], off, [max(1, n // 400) for n in sizes], 1, W.TOPK, W.SIGN_L1, R=R)
    assert set(B.plan_paths(wl.d, wl.seg_offset, wl.seg_k, wl.s, wl.sparsifier, wl.quantizer).tolist()) == {0}
    qa, qb = B.from_workload(wl), B.from_workload(wl, flags=B.FLAG_NO_FAST_PATH)
    op = P.oracle_for(wl)
    ma, mb = torch.zeros(R, wl.d, device=qa.device), torch.zeros(R, wl.d, device=qa.device)
    failed = []
    for t, kind in enumerate(["plain", "plain", "down", "up", "plain", "zeros", "zeros", "zeros", "plain", "ties", "plain"]):
        v = rng.standard_normal((R, wl.d), dtype=f32)
        if kind == "down":
            v *= f32(0.01)
        elif kind == "up":
            v *= f32(100)
        elif kind == "zeros":
            v[rng.random((R, wl.d), dtype=f32) < 0.999] = 0
        elif kind == "ties":
            v = np.round(v)
        delta = torch.from_numpy(v).to(qa.device)
        if t % 3 == 2 or kind == "zeros":                       # the error memory starts anew, so that thresholds do jump
            ma.zero_(); mb.zero_()
        m_before = ma[3].cpu().numpy()
        outs = []
        for q, m in ((qa, ma), (qb, mb)):
            msg = q.new_msg(R).fill_(0xCD)
            q.compress(m, delta, m, 0, t, msg)
            outs.append((m.view(torch.int32), msg))
        torch.cuda.synchronize()
        assert qa.device_status() == B.OK and qb.device_status() == B.OK
        for a, b in zip(*outs):
            assert torch.equal(a, b), (t, kind)
        o = op.compress(m_before, v[3], 3, t)
        assert np.array_equal(outs[0][1][3].cpu().numpy(), o["msg"]) and np.array_equal(P.bits(ma[3].cpu().numpy()), P.bits(o["m_out"]))
        failed.append(int((qa.debug_units()[:, 0] == 2).sum()))
    assert failed[0] == 0 and failed[2] > 0 and max(failed[5:8]) > 0, failed


# entries that pile up in a few cells which no plan foresees: worked through as they are by the first call, listed and given to many
# waves by the calls after it (and by the call without a context), beside calls with entries all over the vector; cells at the
# start, across a segment's end, in a last cell of few coordinates; cells that the plan calls crowded beside them
@pytest.mark.parametrize("case", ["start", "last_cell", "few_messages", "segments", "short", "fp32", "split"])
def test_aggregate_piled_up_cells(P, case):
    from paper_1906_02367_amd import binding as B
    rng = np.random.default_rng(len(case))
    d, off, k, s, sp, qz, spot, lists = {
        "start": (1_000_003, [0, 1_000_003], [10_000], 1, W.TOPK, W.SIGN_L1, (0, 11_000), [range(64), range(40), [63, 5, 9, 8, 7, 1, 0, 33, 21, 40]]),
        "last_cell": (300_033, [0, 300_033], [4_500], 1, W.TOPK, W.SIGN_L2, (295_000, 300_033), [range(64), range(16)]),
        "few_messages": (2_000_001, [0, 2_000_001], [60_000], 1_000, W.TOPK, W.QSGD, (700_000, 762_000), [range(3), [5, 4, 3, 2, 1, 0, 7, 6]]),
        "segments": (600_000, [0, 900, 2_000, 250_500, 600_000], [900, 1_100, 4_000, 6_000], 1, W.TOPK, W.SIGN_L1, (248_000, 254_000), [range(64), range(24)]),
        "short": (200_000, [0, 200_000], [2_000], 1, W.TOPK, W.SIGN_L1, (1_000, 4_000), [range(40), range(64)]),
        "fp32": (1_000_003, [0, 1_000_003], [10_000], 1, W.TOPK, W.FP32, (500_000, 511_000), [range(33)]),
        "split": (70_001, [0, 70_001], [2_000], 1, W.TOPK, W.SIGN_L1, (20_000, 22_100), [range(64)])}[case]
    wl = custom(d, off, k, s, sp, qz, R=8)
    q = B.from_workload(wl)
    op = P.oracle_for(wl)
    both = []
    for piled in (True, False):
        msg = q.new_msg(64)
        for b in range(8):
            v = rng.standard_normal((8, d)).astype(f32)
            if piled:
                v[:, spot[0]:spot[1]] *= f32(100)
            m = torch.zeros(8, d, device=q.device)
            q.compress(m, torch.from_numpy(v).to(q.device), m, 8 * b, b, msg[8 * b: 8 * b + 8])
        torch.cuda.synchronize()
        both.append((msg, [op.decode(x) for x in msg.cpu().numpy()]))
    in_spot = np.bincount((both[0][1][0][0] >> 10).astype(np.int64)).max()
    assert in_spot >= 128                                     # two whole waves of entries of one message in a cell
    x0 = rng.standard_normal(d).astype(f32)
    for call in range(6):                                     # piled up, again, all over, piled up ...
        msg, decoded = both[1 if call in (2, 4) else 0]
        for lst in lists:
            lst = [int(x) for x in lst]
            accumulate = call % 2 == 0
            want = _aggregate_by_definition(decoded, lst, -1.0 / 64, x0, accumulate, d)
            out = torch.from_numpy(x0).to(q.device)
            q.aggregate(msg, out, -1.0 / 64, worker_list=lst, accumulate=accumulate)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, call, len(lst))
            if len(off) == 2 and call < 3:
                out = torch.from_numpy(x0).to(q.device)
                B.aggregate_static(d, k[0], s, sp, qz, msg, out, -1.0 / 64, worker_list=lst, accumulate=accumulate)
                torch.cuda.synchronize()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (case, call, len(lst), "static")
    assert q.device_status() == B.OK
