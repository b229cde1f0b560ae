"""Tuning knobs and the autotuner (GPU tier): results do not depend on the
persistent-grid size; both engines of the FP16-multiply mode meet the parity
bar; the autotuner stores and reuses its choice."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_28451_amd import api, autotune, scenes
from paper_2605_28451_amd.metrics import sqnr_db
from tests.gpu_util import announce, download, need_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,n", [("fp16", 4096), ("fp16_mul_fp32_acc", 4096), ("fp32", 1024)])
def test_grid_size_does_not_change_results(mode, n):
    need_gpu()
    announce(f"tuning grid mode={mode} n={n}")
    fmt = api.storage_format(mode)
    rows = 300
    sc = scenes.range_scene(seed=2, n_pulses=rows, n=n, length=n // 4)
    x = upload(scenes.quantize(sc.echo, fmt), fmt)
    H = api.filter_tensor(sc.replica, n, mode)
    plan = api.FFTPlan(n, rows, mode)
    ref_f = plan.forward(x).clone()
    ref_c = plan.range_compress(x, H).clone()
    engine, bpc0 = plan.get_tuning()
    # a new plan: vector ALU, grid chosen per operation (-1)
    assert (engine, bpc0) == (1, -1)
    for bpc in (0, 1, 2, 8):
        plan.set_tuning(engine, bpc)
        assert plan.get_tuning() == (engine, bpc)
        assert torch.equal(plan.forward(x), ref_f)
        assert torch.equal(plan.range_compress(x, H), ref_c)


@pytest.mark.parametrize("n,rows", [(256, 333), (512, 101), (1024, 257), (2048, 130), (4096, 1029)])
def test_pipelined_kernel_bitwise_equal(n, rows):
    # pure FP16 up to n = 4096: a persistent grid runs the pipelined kernel
    # (register twiddles, next group's data in flight); every operation must
    # give the bits of the one-workgroup-per-group kernel, including ragged
    # last groups (several transforms per workgroup below n = 4096) and grids
    # smaller and larger than the group count
    need_gpu()
    announce(f"pipelined kernel fp16 n={n} rows={rows}")
    sc = scenes.range_scene(seed=2, n_pulses=rows, n=n, length=n // 4)
    x = upload(scenes.quantize(sc.echo, "fp16"), "fp16")
    H = api.filter_tensor(sc.replica, n, "fp16")
    plan = api.FFTPlan(n, rows, "fp16")
    plan.set_tuning(1, 0)
    ref = [plan.forward(x).clone(), plan.inverse_bfp(x, H).clone(), plan.range_compress(x, H).clone()]
    for bpc in (1, 3, 64):
        plan.set_tuning(1, bpc)
        got = [plan.forward(x), plan.inverse_bfp(x, H), plan.range_compress(x, H)]
        for name, a, b in zip(("forward", "inverse", "compress"), got, ref):
            assert torch.equal(a, b), f"{name} blocks_per_cu={bpc}"


@pytest.mark.parametrize("mode", ["fp32", "fp16", "fp16_fp32", "fp16_mul_fp32_acc", "e4m3", "e5m2"])
@pytest.mark.parametrize("n,rows", [(64, 301), (512, 33), (2048, 9), (4096, 7), (8192, 5), (16384, 3)])
def test_rows_per_thread_bitwise_equal(mode, n, rows):
    # two rows per thread (shared twiddles and barriers) must give the bits
    # of one row per thread, for odd batches (a group's second row absent),
    # several transforms per workgroup, and persistent grids
    need_gpu()
    announce(f"rows per thread mode={mode} n={n} rows={rows}")
    fmt = api.storage_format(mode)
    sc = 0.125 if mode in ("e4m3", "e5m2") else 1.0
    x = upload(scenes.quantize(sc * scenes.gaussian_rows(80 + n, rows, n), fmt), fmt)
    z = upload(scenes.quantize(sc * np.sqrt(n) * scenes.gaussian_rows(81 + n, rows, n), fmt), fmt)
    H = api.filter_tensor(scenes.range_replica_padded(n, max(n // 4, 1)), n, mode)
    ph = torch.tensor(np.random.default_rng(n).uniform(-3, 3, n).astype(np.float32), device="cuda")
    plan = api.FFTPlan(n, rows, mode)
    ops = {
        "forward": lambda: plan.forward(x),
        "inverse": lambda: plan.inverse_bfp(z),
        "inverse_filter": lambda: plan.inverse_bfp(z, H),
        "inverse_conj": lambda: plan.inverse_bfp(z, H, conj_filter=True),
        "compress": lambda: plan.range_compress(x, H),
        "compress_fp32": lambda: plan.range_compress(x, H, out_fp32=True),
        "compress_adjoint": lambda: plan.azimuth_compress(x, H, adjoint=True),
        "compress_phase": lambda: plan.azimuth_compress(x, H, phase=ph),
    }
    plan.set_tuning_ex(1, 0, 1)
    ref = {k: f().clone() for k, f in ops.items()}
    for bpc in (0, 1, 3):
        plan.set_tuning_ex(1, bpc, 2)
        assert plan.get_tuning_ex() == (1, bpc, 2, 0)
        for k, f in ops.items():
            same = torch.equal(f(), ref[k])
            assert same, f"{k} blocks_per_cu={bpc}: two rows per thread differ from one"


@pytest.mark.parametrize("mode", ["fp32", "fp16", "fp16_fp32", "fp16_mul_fp32_acc", "e4m3", "e5m2"])
@pytest.mark.parametrize("n", [32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384])
def test_second_radix_plan_matches_oracle(mode, n):
    # the autotuner's second radix plan (radix-8 passes with 8 values per
    # thread, or another radix-16 order): every covered variant against the
    # oracle with the same bars as the first plan, one and two rows per
    # thread, several transforms per workgroup and a ragged batch; the
    # variants it does not cover (here the naive schedule) run the first plan
    need_gpu()
    from tests.test_paths_gpu import PATH_SQNR_MIN, SMALL_FWD_MIN
    from tests.gpu_util import FWD_SQNR_MIN
    rows = 37 if n <= 1024 else 5
    announce(f"second radix plan mode={mode} n={n}")
    fmt = api.storage_format(mode)
    sc = 0.125 if mode in ("e4m3", "e5m2") else 1.0
    x = scenes.quantize(sc * scenes.gaussian_rows(90 + n, rows, n), fmt)
    z = scenes.quantize(sc * np.sqrt(n) * scenes.gaussian_rows(91 + n, rows, n), fmt)
    h = scenes.range_replica_padded(n, max(n // 4, 1))
    Hq = scenes.quantize(oracle.matched_filter(h, n), api.filter_format(mode))
    H = api.filter_tensor(h, n, mode)
    phi = np.random.default_rng(n).uniform(-3, 3, n).astype(np.float32)
    ph = torch.tensor(phi, device="cuda")
    plan = api.FFTPlan(n, rows, mode)
    xd, zd = upload(x, fmt), upload(z, fmt)
    bar_f = SMALL_FWD_MIN[mode] if n <= 128 else FWD_SQNR_MIN[mode] - (1.5 if n > 4096 else 0.0)
    for rr in (1, 2):
        plan.set_tuning_ex(1, 0, rr, 1)
        assert plan.get_tuning_ex() == (1, 0, rr, 1)
        got = {
            "forward": (sqnr_db(oracle.fft(x), download(plan.forward(xd), fmt)), bar_f),
            "inverse": (sqnr_db(oracle.fft(z, inverse=True), download(plan.inverse_bfp(zd), fmt)), bar_f),
            "inverse_conj": (sqnr_db(oracle.fft(z * np.conj(Hq), inverse=True),
                                     download(plan.inverse_bfp(zd, H, conj_filter=True), fmt)), PATH_SQNR_MIN[mode]),
            "compress": (sqnr_db(oracle.compress(x, Hq), download(plan.range_compress(xd, H), fmt)),
                         PATH_SQNR_MIN[mode]),
            "compress_phase": (sqnr_db(oracle.compress(oracle.apply_phase(x, phi.astype(np.float64)), Hq),
                                       download(plan.azimuth_compress(xd, H, phase=ph), fmt)), PATH_SQNR_MIN[mode]),
            "compress_phase_fp32_out": (sqnr_db(oracle.compress(oracle.apply_phase(x, phi.astype(np.float64)), Hq),
                                                download(plan.azimuth_compress(xd, H, phase=ph, out_fp32=True),
                                                         "fp32")), PATH_SQNR_MIN[mode]),
        }
        for k, (s, bar) in got.items():
            print(f"[measure] plan1.{mode}.n{n}.rr{rr}.{k} {s:.3f}")
            assert s >= bar, (k, rr, s, bar)
    # one and two rows per thread give the same bits within the plan
    plan.set_tuning_ex(1, 0, 1, 1)
    a = plan.range_compress(xd, H).clone()
    plan.set_tuning_ex(1, 3, 2, 1)
    assert torch.equal(plan.range_compress(xd, H), a)


def test_second_plan_rejected_where_absent():
    need_gpu()
    for n in (8, 16):
        with pytest.raises(api._lib.BfpError):
            api.FFTPlan(n, 4, "fp16").set_tuning_ex(1, 0, 1, 1)
    with pytest.raises(api._lib.BfpError):
        api.UnevenPlan([10], [0], "fp16").set_tuning_ex(0, 0, 1, 1)


def test_default_rows_per_thread():
    need_gpu()
    for mode, rr in (("fp32", 2), ("fp16", 1), ("fp16_fp32", 2), ("fp16_mul_fp32_acc", 1),
                     ("e4m3", 2), ("e5m2", 2)):
        assert api.FFTPlan(1024, 4, mode).get_tuning_ex() == (1, -1, rr, 0)
    # autofocus plans: the second radix plan (the faster phase gradient)
    from paper_2605_28451_amd.autofocus import AutofocusPlan
    for mode in ("fp32", "fp16_fp32"):
        assert AutofocusPlan(4096, 8, mode).get_tuning_ex() == (1, -1, 2, 1)
    with pytest.raises(api._lib.BfpError):
        api.FFTPlan(1024, 4, "fp16").set_tuning_ex(1, 0, 3)


def test_both_engines_meet_parity():
    need_gpu()
    x = scenes.quantize(scenes.gaussian_rows(1, 64, 4096), "fp16")
    plan = api.FFTPlan(4096, 64, "fp16_mul_fp32_acc")
    for engine in (0, 1):
        plan.set_tuning(engine, 0)
        X = download(plan.forward(upload(x, "fp16")), "fp16")
        s = sqnr_db(oracle.fft(x), X)
        print(f"[measure] engine{engine}.forward {s:.3f}")
        assert s >= (62.4 if engine == 0 else 64.5)  # measured 65.4 / 67.5


def test_autotune_and_cache(tmp_path, monkeypatch):
    need_gpu()
    monkeypatch.setenv("BFP_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    x = upload(scenes.quantize(scenes.gaussian_rows(1, 512, 4096), "fp16"), "fp16")
    out = torch.empty_like(x)
    plan = api.FFTPlan(4096, 512, "fp16_mul_fp32_acc")
    e = autotune.tune(plan, "forward", x, out, reps=5)
    assert e["ms"] > 0 and e["engine"] in (0, 1) and e["blocks_per_cu"] in (-1, 0, 1, 2, 3, 4, 5, 6, 8)
    assert e["rows_per_thread"] in (1, 2) and e["radix_plan"] in (0, 1)
    plan2 = api.FFTPlan(4096, 512, "fp16_mul_fp32_acc")
    assert autotune.apply_cached(plan2, "forward")
    assert plan2.get_tuning_ex() == (e["engine"], e["blocks_per_cu"], e["rows_per_thread"], e["radix_plan"])
    # tuned plan still correct
    X = download(plan2.forward(x), "fp16")
    xq = scenes.decode(x.cpu().numpy(), "fp16")
    assert sqnr_db(oracle.fft(xq), X) >= 60.0


def test_autotune_over_rotating_sets():
    # the candidates timed over several buffer pairs; the pick is a valid
    # tuning and the tuned compression still meets the parity bar
    need_gpu()
    from tests.test_paths_gpu import PATH_SQNR_MIN
    n, rows = 4096, 64
    sc = scenes.range_scene(seed=2, n_pulses=rows, n=n)
    echo = scenes.quantize(sc.echo, "fp16")
    ins = [upload(echo, "fp16") for _ in range(3)]
    outs = [torch.empty_like(ins[0]) for _ in range(3)]
    plan = api.FFTPlan(n, rows, "fp16_fp32")
    H = api.filter_tensor(sc.replica, n, "fp16_fp32")
    ms = plan.autotune_on(2, ins, outs, H, reps=3)
    e, b, rr, pl = plan.get_tuning_ex()
    assert ms > 0 and e == 1 and b in (-1, 0, 1, 2, 3, 4, 5, 6, 8) and rr in (1, 2) and pl in (0, 1)
    got = download(plan.range_compress(ins[1], H), "fp16")
    Hq = scenes.quantize(oracle.matched_filter(sc.replica, n), "fp16")
    assert sqnr_db(oracle.compress(echo, Hq), got) >= PATH_SQNR_MIN["fp16_fp32"]
    with pytest.raises(ValueError):
        plan.autotune_on(2, ins, outs[:2], H)


def test_uneven_grid_size_does_not_change_results():
    need_gpu()
    ub = scenes.uneven_batch(seed=4, count=500)
    x = upload(scenes.quantize(ub.x, "fp16"), "fp16")
    plan = api.UnevenPlan(ub.log2n, ub.inverse, "fp16")
    ref = plan.execute(x).clone()
    for bpc in (1, 2):
        plan.set_tuning(0, bpc)
        assert torch.equal(plan.execute(x), ref)
    ms = plan.autotune_on(0, x, torch.empty_like(x), reps=3)
    assert ms > 0
    assert torch.equal(plan.execute(x), ref)


@pytest.mark.parametrize("mode", ["fp32", "fp16_fp32", "e4m3"])
@pytest.mark.parametrize("n", [64, 256, 512, 2048])
def test_automatic_rows_per_thread_bits(mode, n):
    # automatic tuning takes one or two rows per thread by operation, size and
    # one-row workgroups per CU; on both sides of each line the results are
    # the bits of either explicit setting
    need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    per_wg = {64: 64, 256: 16, 512: 4, 2048: 2}[n]
    fmt = api.storage_format(mode)
    top = 8 * cus * per_wg + 1
    x = upload(0.25 * scenes.gaussian_rows(n, 97, n), fmt).repeat(top // 97 + 1, 1, 1)
    rng = np.random.default_rng(n)
    H = api.filter_tensor(rng.standard_normal(n) + 1j * rng.standard_normal(n), n, mode)
    for rows in (1, 2 * cus * per_wg, 2 * cus * per_wg + 1, 4 * cus * per_wg, 4 * cus * per_wg + 1, top - 2, top):
        announce(f"automatic rows per thread {mode} {rows}x{n}")
        auto, plan = api.FFTPlan(n, rows, mode), api.FFTPlan(n, rows, mode)
        xr = x[:rows].contiguous()
        for op in ("forward", "inverse", "inverse_filter", "compress"):
            run = {"forward": lambda p: p.forward(xr), "inverse": lambda p: p.inverse_bfp(xr),
                   "inverse_filter": lambda p: p.inverse_bfp(xr, H), "compress": lambda p: p.range_compress(xr, H)}[op]
            want = run(auto)
            for rr in (1, 2):
                plan.set_tuning_ex(1, 0, rr, 0)
                assert torch.equal(run(plan), want), (op, rows, rr)


def kernels_of(call):
    """Names of the kernels that `call` launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "row_kernel" in e.name or "uneven" in e.name]
    assert names, "no kernel recorded"
    return names


def test_explicit_rows_per_thread_is_kept():
    # a rows_per_thread that was set, also one beside automatic blocks_per_cu
    # (as a stored tuning may hold), is what runs, on both sides of the line
    # that the default draws (2 one-row workgroups per CU)
    need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for rows, default in ((cus, 1), (4 * cus, 2)):
        announce(f"explicit rows per thread fp32 {rows}x4096")
        x = torch.zeros((rows, 4096, 2), device="cuda")
        plan = api.FFTPlan(4096, rows, "fp32")
        two_rows = [any("row_kernel_rr" in k for k in kernels_of(lambda: plan.forward(x)))]
        for rr in (1, 2):
            plan.set_tuning_ex(1, -1, rr, 0)
            assert plan.get_tuning_ex() == (1, -1, rr, 0)
            two_rows.append(any("row_kernel_rr" in k for k in kernels_of(lambda: plan.forward(x))))
        assert two_rows == [default == 2, False, True], (rows, two_rows)


@pytest.mark.parametrize("mode", ["e4m3", "e5m2"])
def test_automatic_rows_per_thread_short_fp8(mode):
    # 16-point FP8 rows: two rows per thread from 8 one-row workgroups per CU
    # on, with the bits of either setting on both sides
    need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    line = 8 * cus * 256 - 255  # the first row count of 8 workgroups per CU
    x = upload(0.125 * scenes.gaussian_rows(5, 97, 16), mode).repeat(line // 97 + 1, 1, 1)
    for rows, two in ((line - 1, False), (line, True)):
        announce(f"automatic rows per thread {mode} {rows}x16")
        auto, plan, xr = api.FFTPlan(16, rows, mode), api.FFTPlan(16, rows, mode), x[:rows].contiguous()
        want = auto.forward(xr)
        assert any("row_kernel_rr" in k for k in kernels_of(lambda: auto.forward(xr))) == two
        for rr in (1, 2):
            plan.set_tuning_ex(1, 0, rr, 0)
            assert torch.equal(plan.forward(xr), want)


def test_uneven_autotune_keeps_the_default_where_it_is_the_same_launch():
    # a batch of no more tiles than CUs has one launch, the default's; one
    # beyond 64 tiles per CU (the largest explicit grid) has the default, one
    # workgroup per tile, among its candidates, and any pick gives the same bits
    need_gpu()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    announce("uneven autotune small and beyond 64 tiles per CU")
    small = api.UnevenPlan(np.full(20, 10, np.int32), np.zeros(20, np.uint8), "fp16")
    x = torch.zeros((small.total, 2), dtype=torch.float16, device="cuda")
    small.set_tuning(0, 2)
    assert small.autotune_on(0, x, torch.empty_like(x), reps=2) > 0 and small.get_tuning()[1] == 0
    log2n = np.full(64 * cus + 16, 14, np.int32)
    plan = api.UnevenPlan(log2n, np.zeros(log2n.size, np.uint8), "fp16")
    x = torch.randn((plan.total, 2), device="cuda").half()
    y, out = plan.execute(x), torch.empty_like(x)
    assert plan.autotune_on(0, x, out, reps=2) > 0
    assert plan.get_tuning()[1] in (0, 1, 2, 4, 8, 16, 32, 64)
    assert torch.equal(plan.execute(x), y)
