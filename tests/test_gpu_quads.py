"""GPU parity of the row-quad kernel (the kernel of default plans) at the edges of its tiles,
programs and ring, against the CPU oracle with the parity bar, and bit for bit against the
panel kernel (a plan of 4-row panels): both sum each row's entries in ascending column order
with fused multiply-adds."""
import os

import numpy as np
import pytest

import oracle
import paper_2101_07948_amd as sd
from conftest import tol_fp32
from paper_2101_07948_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def force():
    """Sets the kernel's launch overrides for one test."""
    keys = ("SDNN_FORCE_QUAD_CAP", "SDNN_FORCE_QUAD_WAVES")
    old = {k: os.environ.get(k) for k in keys}

    def set_(cap, waves):
        os.environ.update({keys[0]: str(cap), keys[1]: str(waves)})
    yield set_
    for k, v in old.items():
        if v is None:
            os.environ.pop(k, None)
        else:
            os.environ[k] = v


def run(plan, Bt, bias, epi):
    bt = None if bias is None else torch.from_numpy(np.ascontiguousarray(bias)).to(DEV)
    C = torch.full((plan.M, Bt.shape[1]), float("nan"), device=DEV)
    plan.spmm(Bt, C, bt, epi)
    torch.cuda.synchronize()
    return C.cpu().numpy()


def check(W, N, label, epi="none", bias=True, offset=0, **kw):
    print(f"quads: {label} N={N}", flush=True)
    B = inputs.dense_B(W.K, N, inputs.CFG_TEST, 7000 + N)
    b = inputs.bias_normal(W.M, inputs.CFG_TEST, 7001, 0.02) if bias else None
    flat = torch.empty(W.K * N + 4, device=DEV)
    Bt = flat[offset:offset + W.K * N].view(W.K, N)
    Bt.copy_(torch.from_numpy(B))
    with sd.Plan.from_csr(W, **kw) as plan:
        got, perm = run(plan, Bt, b, epi), plan.perm
    with sd.Plan.from_csr(W, panel_rows=4, **kw) as plan:
        panel = run(plan, Bt, b, epi)
    ref, bound = oracle.spmm_f64(W.row_ptr, W.col_idx, W.values, W.K, B, b, epi)
    if kw.get("out_permuted"):
        ref, bound = ref[perm], bound[perm]
    err = np.abs(got.astype(np.float64) - ref)
    assert (err <= tol_fp32(bound, epi)).all(), label
    assert np.array_equal(got, panel), label


@pytest.mark.parametrize("cap", [1, 2, 4, 8])
@pytest.mark.parametrize("M,K,N", [
    (1, 1, 1), (3, 63, 4), (4, 64, 64), (33, 65, 68), (50, 300, 63),   # tile and chunk remainders
    (130, 512, 132), (130, 513, 130), (200, 1100, 65),                  # the ring's 512 rows, and past
])
def test_program_heights(force, cap, M, K, N):
    """Programs of up to 4, 8, 16 and 32 rows over one and several tiles, 16- and 4-byte
    staging, rows past M, K inside one chunk, exactly the ring and wrapping it."""
    force(cap, 3)
    W = inputs.pattern_uniform(M, K, 0.2, inputs.CFG_TEST, 7100 + M + K, 0.05)
    check(W, N, f"cap {cap} M {M} K {K}", "relu")


@pytest.mark.parametrize("cap,waves", [(1, 1), (2, 12), (4, 5), (8, 12)])
def test_row_length_mix(force, cap, waves):
    """Lognormal rows with a few full and many empty ones: programs of every height in one
    launch, programs without entries, GELU, permuted output."""
    force(cap, waves)
    rng = np.random.default_rng(7200)
    M, K = 500, 900
    lens = np.minimum(K, (30 * np.exp(rng.normal(0, 1.2, M))).astype(int))
    lens[:3], lens[100:220] = K, 0
    cols = [np.sort(rng.choice(K, n, replace=False)) for n in lens]
    row_ptr = np.zeros(M + 1, dtype=np.int32)
    np.cumsum(lens, out=row_ptr[1:])
    ci = np.concatenate(cols).astype(np.int32)
    W = inputs.CSR(row_ptr, ci, rng.standard_normal(len(ci)).astype(np.float32) * np.float32(0.05), M, K)
    check(W, 196, f"mix cap {cap}", "gelu")
    check(W, 196, f"mix cap {cap} permuted", "none", out_permuted=True)


@pytest.mark.parametrize("cap", [1, 8])
def test_scattered_columns_and_many_descriptors(force, cap):
    """K = 9000 (141 chunks: more than 64 descriptors a program, loaded 64 at a time) with rows
    whose entries lie at opposite ends of K, so that programs fill in and wait for one another."""
    force(cap, 2)
    rng = np.random.default_rng(7300)
    M, K = 40, 9000
    mask = rng.random((M, K)) < 0.02
    mask[::3, : K - 700] = False
    mask[1::3, 600:] = False
    mask[5] = rng.random(K) < 0.5
    rows, ci = np.nonzero(mask)
    row_ptr = np.zeros(M + 1, dtype=np.int32)
    np.cumsum(mask.sum(1), out=row_ptr[1:])
    W = inputs.CSR(row_ptr, ci.astype(np.int32), rng.standard_normal(len(ci)).astype(np.float32), M, K)
    check(W, 72, f"scattered cap {cap}", bias=False)


@pytest.mark.parametrize("cap,N,K", [(1, 4160, 200), (4, 8256, 600), (8, 16384, 520)])
def test_persistent_items(force, cap, N, K):
    """More items than workgroups: a workgroup takes several row-blocks and tiles in turn, the
    chunk numbers of an item rounded up to the ring."""
    force(cap, 2)
    W = inputs.pattern_uniform(300, K, 0.05, inputs.CFG_TEST, 7400 + K, 0.05)
    check(W, N, f"persistent cap {cap}", "relu")


@pytest.mark.parametrize("offset", [1, 2])
def test_misaligned_input(offset):
    """B not 16-byte aligned runs the 4-byte staging."""
    W = inputs.pattern_uniform(100, 200, 0.1, inputs.CFG_TEST, 7500, 0.05)
    check(W, 256, f"offset {offset}", offset=offset)


def test_rows_are_independent_of_other_rows_inputs():
    """A row's result does not read B rows it has no entry for: infinities there leave it
    finite, as in the panel kernel."""
    W = inputs.pattern_uniform(64, 128, 0.1, inputs.CFG_TEST, 7600, 0.05)
    B = torch.ones(128, 64, device=DEV)
    B[5] = float("inf")
    hit = np.zeros(64, bool)
    for i in range(64):
        hit[i] = 5 in W.col_idx[W.row_ptr[i]:W.row_ptr[i + 1]]
    with sd.Plan.from_csr(W) as plan:
        got = run(plan, B, None, "none")
    assert np.isfinite(got[~hit]).all() and not np.isfinite(got[hit]).any() and hit.any()


@pytest.mark.parametrize("cap", [1, 4, 8])
@pytest.mark.parametrize("OC,IC,H,W,NB", [(5, 1, 1, 1, 4), (9, 3, 5, 7, 4), (33, 8, 3, 11, 12),
                                          (40, 64, 9, 9, 8)])
def test_convolution(force, cap, OC, IC, H, W, NB):
    """The virtual operand of a 3x3 convolution: a single pixel, ragged tiles, K = 9 to 576
    (past the ring), every border, against the oracle and the panel kernel."""
    force(cap, 3)
    L = inputs.conv_layer(OC, IC, H, W, NB, 0.6, layer=700 + OC + IC, epi="relu")
    X = torch.from_numpy(L.X).to(DEV)
    bt = torch.from_numpy(L.bias).to(DEV)
    out = []
    for kw in ({}, {"panel_rows": 4}):
        with sd.Plan.from_csr(L.F, **kw) as plan:
            C = torch.full((OC, H, W, NB), float("nan"), device=DEV)
            plan.conv3x3(X, C, bt, "relu")
            torch.cuda.synchronize()
            out.append(C.cpu().numpy())
    ref, bound = oracle.conv3x3_f64(L.F.row_ptr, L.F.col_idx, L.F.values, L.X, L.bias, "relu")
    assert (np.abs(out[0].astype(np.float64) - ref) <= tol_fp32(bound, "relu")).all()
    assert np.array_equal(out[0], out[1])


def test_gelu_accuracy_and_special_values():
    """GELU within 0.5 |x| * 6.4e-7 of the exact one (over every float of 1e-7 <= |x| <= 14 the largest
    error was 6.31e-7, that of the two-sided form with the published coefficients 6.43e-7); at
    infinities and NaN what 0.5 x (1 + erf(x / sqrt 2)) gives."""
    from math import erf
    one = inputs.CSR(np.array([0, 1], np.int32), np.zeros(1, np.int32), np.ones(1, np.float32), 1, 1)
    with sd.Plan.from_csr(one) as plan:
        for sigma in (0.005, 0.02, 0.05, 0.1, 0.35, 1.0, 3.0):
            x = np.random.default_rng(int(sigma * 1000)).standard_normal(2000000).astype(np.float32) * np.float32(sigma)
            got = run(plan, torch.from_numpy(x[None]).to(DEV), None, "gelu")[0].astype(np.float64)
            t = torch.from_numpy(x).double()
            err = np.abs(got - (0.5 * t * torch.special.erfc(-t / 2 ** 0.5)).numpy())
            assert (err <= 6.4e-7 * 0.5 * np.abs(x) + 1e-14).all(), f"sigma {sigma}"
        x = np.array([np.inf, -np.inf, np.nan, 3e38, -3e38, 1e20, -1e20, 40, -40, 0, -0.0, 1e-40], np.float32)
        got = run(plan, torch.from_numpy(x[None]).to(DEV), None, "gelu")[0]
        with np.errstate(invalid="ignore"):
            want = np.array([0.5 * v * (1 + erf(v / 2 ** 0.5)) for v in x.astype(np.float64)])
        assert np.array_equal(np.isnan(got), np.isnan(want))
        ok = ~np.isnan(want)
        assert np.allclose(got[ok], want[ok], rtol=1e-6, atol=1e-30)


def spent(call, ref, tol, budget):
    """A call with every wait's budget forced to a few polls: within the bar or NaN, and NaN
    everywhere without any."""
    old = os.environ.get("SDNN_POLL_BUDGET")
    os.environ["SDNN_POLL_BUDGET"] = str(budget)
    try:
        got = call()
    finally:
        if old is None:
            os.environ.pop("SDNN_POLL_BUDGET")
        else:
            os.environ["SDNN_POLL_BUDGET"] = old
    ok = (np.abs(got.astype(np.float64) - ref) <= tol) | np.isnan(got)
    assert ok.all(), f"{int((~ok).sum())} finite outputs out of tolerance"
    assert budget > 0 or np.isnan(got).all()


@pytest.mark.parametrize("budget", [0, 3])
@pytest.mark.parametrize("epi", ["none", "relu", "gelu"])
@pytest.mark.parametrize("cap", [1, 2, 4, 8])
def test_spent_budget_is_nan_after_any_activation(force, cap, epi, budget):
    """A wave that stops waiting stores NaN whatever the activation: 16- and 4-byte staging (N of
    1024 and 1023), several items per workgroup, and a convolution."""
    force(cap, 4)
    print(f"spent budget {budget} cap {cap} {epi}", flush=True)
    W = inputs.pattern_uniform(300, 700, 0.1, inputs.CFG_TEST, 7700, 0.05)
    bias = inputs.bias_normal(300, inputs.CFG_TEST, 7701, 0.02)
    for N in (1024, 1023, 8192):
        B = inputs.dense_B(700, N, inputs.CFG_TEST, 7702)
        ref, bound = oracle.spmm_f64(W.row_ptr, W.col_idx, W.values, 700, B, bias, epi)
        with sd.Plan.from_csr(W) as plan:
            spent(lambda: run(plan, torch.from_numpy(B).to(DEV), bias, epi), ref, tol_fp32(bound, epi), budget)
    L = inputs.conv_layer(40, 64, 9, 9, 8, 0.6, layer=770, epi=epi)
    ref, bound = oracle.conv3x3_f64(L.F.row_ptr, L.F.col_idx, L.F.values, L.X, L.bias, epi)
    with sd.Plan.from_csr(L.F) as plan:
        def conv():
            C = torch.full((40, 9, 9, 8), float("nan"), device=DEV)
            plan.conv3x3(torch.from_numpy(L.X).to(DEV), C, torch.from_numpy(L.bias).to(DEV), epi)
            torch.cuda.synchronize()
            return C.cpu().numpy()
        spent(conv, ref, tol_fp32(bound, epi), budget)


@pytest.mark.parametrize("N", [1024, 1023])
@pytest.mark.parametrize("tile_cols", [128, 256])
def test_spent_budget_is_nan_after_relu_on_the_panel_kernel(N, tile_cols):
    """The same of the panel kernel, unsplit and on runs of K, whose reduction applies the ReLU."""
    W = inputs.pattern_uniform(300, 700, 0.1, inputs.CFG_TEST, 7710, 0.05)
    B = inputs.dense_B(700, N, inputs.CFG_TEST, 7711)
    ref, bound = oracle.spmm_f64(W.row_ptr, W.col_idx, W.values, 700, B, None, "relu")
    Bt = torch.from_numpy(B).to(DEV)
    with sd.Plan.from_csr(W, tile_cols=tile_cols, split_chunks=4) as plan:
        def split():
            C = torch.zeros(300, N, device=DEV)
            plan.spmm_split(Bt, C, None, "relu", splits=3)
            torch.cuda.synchronize()
            return C.cpu().numpy()
        for budget in (0, 3):
            spent(lambda: run(plan, Bt, None, "relu"), ref, tol_fp32(bound, "relu"), budget)
            spent(split, ref, tol_fp32(bound, "relu"), budget)


@pytest.mark.parametrize("kw,M,tile", [({}, 32, 64), ({"panel_rows": 16, "tile_cols": 256}, 16, 256)])
def test_budget_is_the_waves_in_total(force, kw, M, tile):
    """A wave that has spent its budget waits for nothing in its later items either: with one
    program (panel) and a tile per item, workgroup w takes the tiles w, w + 256, ..., and once
    one of them is NaN the later ones are."""
    force(8, 1)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N = tile * 4 * cus
    W = inputs.pattern_uniform(M, 512, 0.2, inputs.CFG_TEST, 7720, 0.05)
    B = torch.ones(512, N, device=DEV)
    old = os.environ.get("SDNN_POLL_BUDGET")
    try:
        with sd.Plan.from_csr(W, **kw) as plan:
            for budget in (5, 20, 60):
                os.environ["SDNN_POLL_BUDGET"] = str(budget)
                nan = np.isnan(run(plan, B, None, "none")[:, ::tile]).reshape(M, 4, cus)
                assert (nan[:, 1:] >= nan[:, :-1]).all(), f"budget {budget}"
    finally:
        os.environ.pop("SDNN_POLL_BUDGET")
        if old is not None:
            os.environ["SDNN_POLL_BUDGET"] = old


@pytest.mark.parametrize("cap", [2, 4, 8])
@pytest.mark.parametrize("M,K,N,density", [
    (700, 40, 3092, 0.2), (700, 40, 3001, 0.2),   # rows of C off 64 bytes, past 8 MB
    (160, 70, 1003, 0.3),                         # the same, below it
    (800, 32, 16384, 0.2), (800, 33, 16384, 0.2),  # aligned rows past 48 MB, K of 32 and above
])
def test_output_stores(force, cap, M, K, N, density):
    """Both sides of the rule that stores C through the caches or streams it, with 16-byte
    stores to rows that are 16- and 4-byte aligned."""
    force(cap, 12)
    W = inputs.pattern_uniform(M, K, density, inputs.CFG_TEST, 7300 + M + K, 0.05)
    check(W, N, f"stores cap {cap} M {M} K {K}")


def test_reported_launch(force):
    """sdnn_plan_launch_quads reports the launch of products: programs and waves of a default plan
    (forced ones, clipped to the programs there are), none for a plan that fixes an option of the
    panel kernel or for rows of B too long for the staging; and the info's packings."""
    W = inputs.pattern_grouped8(96, 200, 0.16, inputs.CFG_TEST, 7800, 0.05)
    with sd.Plan.from_csr(W) as plan:
        got = plan.launch_quads(64)
        assert got["program_rows"] in (4, 8, 16, 32) and 1 <= got["waves"] <= 12
        assert plan.launch_quads(1 << 25) is None
        assert plan.info["quad_packings"] == 4 and plan.info["quad_kib"] > 0
        host = sd.plan_check_host(W.row_ptr, W.col_idx, W.values, W.M, W.K)
        assert all(host[k] == plan.info[k] for k in ("quad_packings", "quad_kib", "packed_bytes"))
        for cap, waves, want in ((1, 12, 12), (4, 5, 5), (8, 12, 3)):
            force(cap, waves)
            assert plan.launch_quads(64) == {"program_rows": 4 * cap, "waves": want}
        for bad in (0, -1):
            with pytest.raises(sd.SdnnError) as ei:
                plan.launch_quads(bad)
            assert ei.value.code == 2
    for kw in ({"panel_rows": 8}, {"grouping": "order"}, {"grouping": "balanced"}, {"tile_cols": 128}):
        with sd.Plan.from_csr(W, **kw) as plan:
            assert plan.launch_quads(64) is None


def test_tuned_launch_is_the_one_calls_run_on():
    """After sdnn_plan_tune the reported launch is one that was timed, and calls agree with the panel
    kernel bit for bit."""
    W = inputs.pattern_uniform(512, 512, 0.2, inputs.CFG_TEST, 7810, 0.05)
    B = torch.from_numpy(inputs.dense_B(512, 784, inputs.CFG_TEST, 7811)).to(DEV)
    with sd.Plan.from_csr(W) as plan, sd.Plan.from_csr(W, panel_rows=4) as panel:
        rule = plan.launch_quads(784)
        plan.tune(784, B, torch.empty(512, 784, device=DEV))
        got = plan.launch_quads(784)
        assert got is None or got == rule or got["waves"] in (3, 6, 9, 12)
        assert np.array_equal(run(plan, B, None, "none"), run(panel, B, None, "none"))


def test_tuned_launch_is_kept_for_its_alignment():
    """A launch timed on a B off 16 bytes (4-byte staging, C through the caches) is not taken for
    aligned calls, whose rule picks 16-row programs and 7 waves here where that of the timed calls
    picks 32-row ones; both kinds of calls stay right."""
    M, K, N = 1000, 300, 3136
    W = inputs.pattern_uniform(M, K, 0.1, inputs.CFG_TEST, 7820, 0.05)
    flat = torch.empty(K * N + 1, device=DEV)
    B = flat[1:].view(K, N)
    B.copy_(torch.from_numpy(inputs.dense_B(K, N, inputs.CFG_TEST, 7821)))
    with sd.Plan.from_csr(W) as plan, sd.Plan.from_csr(W, panel_rows=4) as panel:
        rule = plan.launch_quads(N)
        plan.tune(N, B, torch.empty(M, N, device=DEV))
        assert plan.launch_quads(N) == rule
        want = run(panel, B, None, "none")
        assert np.array_equal(run(plan, B, None, "none"), want)
        assert np.array_equal(run(plan, B.clone(), None, "none"), want)
        plan.tune(N, B.clone(), torch.empty(M, N, device=DEV))  # the same N, aligned
        assert np.array_equal(run(plan, B, None, "none"), want)
        assert np.array_equal(run(plan, B.clone(), None, "none"), want)


def uneven_rows(kind, M, K, n, seed):
    """M rows of n entries that lie together: along the diagonal, at random places, or in random
    blocks of 64 columns."""
    rng = np.random.default_rng(seed)
    if kind == "blocks":
        cols = np.stack([np.sort(rng.choice(K // 64, n // 64, replace=False)) for _ in range(M)])
        cols = (64 * cols[:, :, None] + np.arange(64)).reshape(M, -1)
    else:
        start = np.arange(M) * (K - n) // (M - 1)
        cols = (start if kind == "band" else rng.permutation(start))[:, None] + np.arange(n)
    n = cols.shape[1]
    values = rng.standard_normal(M * n).astype(np.float32)
    return inputs.CSR(np.arange(0, M * n + 1, n, dtype=np.int32), cols.astype(np.int32).ravel(), values, M, K)


@pytest.mark.parametrize("kind", ["band", "runs", "blocks"])
def test_uneven_rows_run_on_the_panel_kernel(kind):
    """Rows whose entries lie in different parts of K leave the row-quad kernel filler and waves that
    wait for one another: where there are many of them (4096 x 4096, 2 %, N = 2048: 2.6 to 3 times
    slower there) products run on the panel kernel, uniform rows stay.  Small and ragged shapes of
    the same patterns agree with the oracle on whichever kernel the rule takes."""
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        with sd.Plan.from_csr(uneven_rows(kind, 4096, 4096, 82 if kind != "blocks" else 64, 7900)) as plan:
            assert plan.launch_quads(2048) is None
        with sd.Plan.from_csr(inputs.pattern_uniform(4096, 4096, 0.02, inputs.CFG_TEST, 7901, 0.05)) as plan:
            assert plan.launch_quads(2048) is not None
    for M, K, n, N in ((300, 2048, 64, 516), (1000, 1024, 128, 1023), (65, 4096, 64, 4096)):
        check(uneven_rows(kind, M, K, n, 7910 + M), N, f"{kind} M {M}", "relu")
        check(uneven_rows(kind, M, K, n, 7910 + M), N, f"{kind} M {M} permuted", out_permuted=True)


def test_uneven_filters_convolve(force):
    """The same rule of convolutions: block-structured filters, on both kernels."""
    F = uneven_rows("blocks", 128, 576, 64, 7950)
    X = torch.from_numpy(np.random.default_rng(7951).standard_normal((64, 28, 28, 8)).astype(np.float32)).to(DEV)
    out = []
    for forced in (False, True):
        if forced:
            force(4, 6)
        with sd.Plan.from_csr(F) as plan:
            C = torch.full((128, 28, 28, 8), float("nan"), device=DEV)
            plan.conv3x3(X, C, None, "relu")
            torch.cuda.synchronize()
            out.append(C.cpu().numpy())
    ref, bound = oracle.conv3x3_f64(F.row_ptr, F.col_idx, F.values, X.cpu().numpy(), None, "relu")
    assert (np.abs(out[0].astype(np.float64) - ref) <= tol_fp32(bound, "relu")).all()
    assert np.array_equal(out[0], out[1])
