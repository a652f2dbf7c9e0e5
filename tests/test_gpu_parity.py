"""GPU parity: every stage of the HIP path against the CPU oracle, element by element, through the
C ABI.  Integer results must match bit for bit; the dequantised fp32 output must be within 1e-6
relative of the oracle's fp64 value."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2403_07339_amd import workloads

pytestmark = pytest.mark.gpu

ROW, COL, BOTH = 0, 1, 2
STRATS = (ROW, COL, BOTH)
REL_TOL = 1e-6  # relative error allowed on the dequantised fp32 output


@pytest.fixture(scope="module")
def imu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_07339_amd import binding
    return binding


def dev(x):
    return x.to("cuda")


def oracle_quant(x: torch.Tensor, scale):
    q, st = oracle.rtn_quantize(x.contiguous().numpy(), scale)
    assert st == 0
    return q


def np_stats(q, s):
    a = np.abs(q.astype(np.int64))
    ob = a >= s
    return ob.sum(1), ob.sum(0), a.max(1), a.max(0)


# ------------------------------------------------------------------ quantize + scan
@pytest.mark.parametrize("shape", [(64, 256), (200, 1000), (77, 130), (1, 5), (513, 260), (300, 64)])
@pytest.mark.parametrize("b", [8, 4])
def test_quantize_and_scan(imu, shape, b):
    g = torch.Generator().manual_seed(shape[0] * 1000 + shape[1] + b)
    x = torch.randn(shape, generator=g) * 3
    x[torch.rand(shape, generator=g) < 0.01] *= 100
    # exact ties in units of the step
    scale = float(np.float32(0.0371))
    x.view(-1)[: min(64, x.numel())] = (torch.arange(min(64, x.numel())) - 20 + 0.5) * np.float32(scale)
    s = 1 << (b - 1)
    want = oracle_quant(x, scale)
    Q, st, status = imu.imunpack_quantize(dev(x), scale, b)
    assert int(status.item()) == 0
    assert np.array_equal(Q.cpu().numpy(), want)
    rc, cc, rm, cm = np_stats(want, s)
    assert np.array_equal(st.rowcnt.cpu().numpy(), rc) and np.array_equal(st.colcnt.cpu().numpy(), cc)
    assert np.array_equal(st.rowmax.cpu().numpy(), rm) and np.array_equal(st.colmax.cpu().numpy(), cm)
    st2 = imu.imunpack_scan(Q, b)
    for f in ("rowcnt", "colcnt", "rowmax", "colmax"):
        assert torch.equal(getattr(st, f), getattr(st2, f))
    # transposed view (unit stride down the rows) and a general strided view
    xt = dev(x.t().contiguous()).t()
    Qt, stt, _ = imu.imunpack_quantize(xt, scale, b)
    assert np.array_equal(Qt.cpu().numpy(), want)
    assert np.array_equal(stt.colmax.cpu().numpy(), cm) and np.array_equal(stt.rowcnt.cpu().numpy(), rc)
    wide = dev(torch.zeros(shape[0], 2 * shape[1]))
    wide[:, ::2] = dev(x)
    Qs, sts, _ = imu.imunpack_quantize(wide[:, ::2], scale, b)
    assert np.array_equal(Qs.cpu().numpy(), want)
    assert np.array_equal(sts.colcnt.cpu().numpy(), cc) and np.array_equal(sts.rowmax.cpu().numpy(), rm)


@pytest.mark.parametrize("n,h,d,b", [(200, 333, 520, 8), (70, 64, 256, 4), (1, 129, 4, 8), (130, 131, 130, 8), (64, 1, 256, 8)])
def test_quantize_pair_matches_the_oracle_for_both_operands(imu, n, h, d, b):
    """Both operands of a product in one call (one clearing launch, one launch over the rows of both when
    both take the fast path; d = 130 takes the general path): integers, all four statistics, the OB lists
    and the two status flags against the oracle's RTN (Sec. 2, Eq. quantized_A) and the IB/OB definition
    (Sec. 4); a NaN in B raises only B's flag."""
    g = torch.Generator().manual_seed(n + 31 * h + d + b)
    xa, xb = torch.randn((n, d), generator=g) * 2, torch.randn((h, d), generator=g)
    xa[torch.rand((n, d), generator=g) < 0.02] *= 150.0
    xb[torch.rand((h, d), generator=g) < 0.01] *= 90.0
    sa, sb = float(np.float32(0.0371)), float(np.float32(0.0113))
    s = 1 << (b - 1)
    sta = imu.Stats.empty(n, d, "cuda", ob_cap=max(1, n * d))
    stb = imu.Stats.empty(h, d, "cuda", ob_cap=max(1, h * d))
    Qa, Qb, sta, stb, status = imu.imunpack_quantize_pair(dev(xa), dev(xb), sa, sb, b, stats_a=sta, stats_b=stb)
    assert status.cpu().tolist() == [0, 0]
    for x, scale, Q, st in ((xa, sa, Qa, sta), (xb, sb, Qb, stb)):
        if x.shape[0] == 0:
            continue
        want = oracle_quant(x, scale)
        assert np.array_equal(Q.cpu().numpy(), want)
        rc, cc, rm, cm = np_stats(want, s)
        assert np.array_equal(st.rowcnt.cpu().numpy(), rc) and np.array_equal(st.colcnt.cpu().numpy(), cc)
        assert np.array_equal(st.rowmax.cpu().numpy(), rm) and np.array_equal(st.colmax.cpu().numpy(), cm)
        ii, jj = np.nonzero(np.abs(want.astype(np.int64)) >= s)
        n_ob = int(st.ob_count.item())
        assert n_ob == len(ii)
        ob = st.ob[:, :n_ob].cpu().numpy()
        assert sorted(zip(ob[0].tolist(), ob[1].tolist(), ob[2].tolist())) == sorted(zip(ii.tolist(), jj.tolist(), want[ii, jj].tolist()))
    if h > 0:
        xb[h // 2, d // 3] = float("nan")
        *_, status = imu.imunpack_quantize_pair(dev(xa), dev(xb), sa, sb, b)
        assert status.cpu().tolist() == [0, 1]


def test_quantize_pair_with_operands_of_different_layouts(imu):
    """One operand row-major, the other a transposed view (as in a backward GEMM): the pair call runs them
    through their own kernels, one after the other, with the same results."""
    g = torch.Generator().manual_seed(5)
    xa, xb = torch.randn((256, 384), generator=g) * 4, torch.randn((128, 384), generator=g) * 4
    xa[torch.rand((256, 384), generator=g) < 0.01] *= 80.0
    sa, sb, b = float(np.float32(0.05)), float(np.float32(0.03)), 8
    A_d, B_t = dev(xa), dev(xb.t().contiguous()).t()          # B: unit stride down its rows
    Qa, Qb, sta, stb, status = imu.imunpack_quantize_pair(A_d, B_t, sa, sb, b, want_ob_list=(True, True))
    assert status.cpu().tolist() == [0, 0]
    for x, scale, Q, st in ((xa, sa, Qa, sta), (xb, sb, Qb, stb)):
        want = oracle_quant(x, scale)
        assert np.array_equal(Q.cpu().numpy(), want)
        rc, cc, rm, cm = np_stats(want, 1 << (b - 1))
        assert np.array_equal(st.rowcnt.cpu().numpy(), rc) and np.array_equal(st.colcnt.cpu().numpy(), cc)
        assert np.array_equal(st.rowmax.cpu().numpy(), rm) and np.array_equal(st.colmax.cpu().numpy(), cm)
        assert int(st.ob_count.item()) == int(rc.sum())


@pytest.mark.parametrize("shape,b,frac", [((300, 520), 8, 0.01), ((132, 260), 4, 0.2), ((1024, 384), 8, 0.0005),
                                          ((256, 256), 2, 0.9)])
def test_ob_entry_list_for_every_input_layout(imu, shape, b, frac):
    """The OB entry list (row, column, value of every entry with |q| >= s, in any order) that UnpackBoth
    plans from, for a row-major operand, a transposed view (the tiled transposing kernel) and a view with
    neither stride 1: the same set as the definition gives, each entry once."""
    g = torch.Generator().manual_seed(shape[0] + 7 * shape[1] + b)
    x = torch.randn(shape, generator=g)
    x[torch.rand(shape, generator=g) < frac] *= 300.0
    scale = float(np.float32(0.021))
    s = 1 << (b - 1)
    want = oracle_quant(x, scale)
    ii, jj = np.nonzero(np.abs(want.astype(np.int64)) >= s)
    want_set = sorted(zip(ii.tolist(), jj.tolist(), want[ii, jj].tolist()))
    wide = dev(torch.zeros(shape[0], 3 * shape[1]))
    wide[:, 1::3] = dev(x)
    for view in (dev(x), dev(x.t().contiguous()).t(), wide[:, 1::3]):
        st = imu.Stats.empty(shape[0], shape[1], view.device, ob_cap=shape[0] * shape[1])  # room for every entry
        Q, st, status = imu.imunpack_quantize(view, scale, b, stats=st)
        assert int(status.item()) == 0 and np.array_equal(Q.cpu().numpy(), want)
        n_ob = int(st.ob_count.item())
        assert n_ob == len(want_set) <= st.ob.shape[1]
        ob = st.ob[:, :n_ob].cpu().numpy()
        assert sorted(zip(ob[0].tolist(), ob[1].tolist(), ob[2].tolist())) == want_set


@pytest.mark.parametrize("shape,pitch", [((37, 1031), 1031), ((700, 261), 263), ((5, 3), 7), ((1100, 1), 5), ((64, 514), 514), ((2100, 258), 259)])
def test_quantize_rows_that_start_anywhere(imu, shape, pitch):
    """Rows of a length and a pitch that are no multiples of four, from an odd address, in blocks of 16 and of 64 rows, into
    rows of integers like that: integers, statistics, the list, and nothing beside them."""
    rows, cols = shape
    g = torch.Generator().manual_seed(rows + cols)
    x = torch.randn(shape, generator=g)
    x[torch.rand(shape, generator=g) < 0.02] *= 300.0
    buf = torch.full((rows * pitch + 9,), float("nan"), device="cuda")
    view = buf[3:3 + rows * pitch].view(rows, pitch)[:, :cols]
    view.copy_(dev(x))
    want = oracle_quant(x, np.float32(0.021))
    around = torch.full((rows * cols + 10,), 77, dtype=torch.int32, device="cuda")
    Q = around[5:5 + rows * cols].view(rows, cols)
    st = imu.Stats.empty(rows, cols, view.device, ob_cap=rows * cols)
    _, st, status = imu.imunpack_quantize(view, 0.021, 8, Q, st)
    assert int(status.item()) == 0 and np.array_equal(Q.cpu().numpy(), want)
    assert bool((around[:5] == 77).all()) and bool((around[-5:] == 77).all())
    rc, cc, rm, cm = np_stats(want, 128)
    assert np.array_equal(st.rowcnt.cpu().numpy(), rc) and np.array_equal(st.colcnt.cpu().numpy(), cc)
    assert np.array_equal(st.rowmax.cpu().numpy(), rm) and np.array_equal(st.colmax.cpu().numpy(), cm)
    n_ob = int(st.ob_count.item())
    ii, jj = np.nonzero(np.abs(want.astype(np.int64)) >= 128)
    ob = st.ob[:, :n_ob].cpu().numpy()
    assert sorted(zip(ob[0].tolist(), ob[1].tolist(), ob[2].tolist())) == sorted(zip(ii.tolist(), jj.tolist(), want[ii, jj].tolist()))


@pytest.mark.parametrize("cap", [1, 1000, 70000, 229632, 229633, 400000])
@pytest.mark.parametrize("layout", ["rows", "columns", "neither"])
def test_list_of_an_operand_of_nothing_but_heavy_hitters(imu, layout, cap):
    """Far more entries than a workgroup stages, with no room, some, just enough and plenty: all are counted, the list holds as
    many as it has room for, each once."""
    rows, cols = 897, 256
    x = torch.arange(rows * cols, dtype=torch.float32).view(rows, cols) + 200.0  # every entry is one, all different
    view = dev(x) if layout == "rows" else dev(x.t().contiguous()).t()
    if layout == "neither":
        view = torch.zeros(rows, 2 * cols, device="cuda")
        view[:, ::2] = dev(x)
        view = view[:, ::2]
    st = imu.Stats.empty(rows, cols, view.device, ob_cap=cap)
    st.ob.fill_(-1)
    Q, st, _ = imu.imunpack_quantize(view, 1.0, 8, stats=st)
    assert int(st.ob_count.item()) == rows * cols
    ob = st.ob[:, :min(cap, rows * cols)].cpu().numpy()
    assert len(set(ob[2].tolist())) == ob.shape[1] and np.array_equal(ob[2], ob[0] * cols + ob[1] + 200)


@pytest.mark.parametrize("scale,lo_exp,negate", [(1.0, 21, False), (0.75, 21, True), (0.0371, -3, False)])
def test_quantize_every_float_of_two_binades(imu, scale, lo_exp, negate):
    """Every binary32 value of two adjacent binades (2 x 2^23 bit patterns) through the quantizer: the
    division must be the correctly rounded one and the rounding half-to-even for each of them.  With
    step 1 the binades [2^21, 2^23) hold every tie k + 0.5 up to 2^22; steps 0.75 and 0.0371 make
    nearly every quotient inexact, so a reciprocal-multiply or a fused form would show."""
    scale = float(np.float32(scale))
    lo = np.float32(2.0 ** lo_exp).view(np.uint32)
    bits = np.arange(int(lo), int(lo) + (1 << 24), dtype=np.uint32)
    if negate:
        bits = bits | np.uint32(0x80000000)
    x = bits.view(np.float32).reshape(4096, 4096)
    assert np.isfinite(x).all() and np.abs(x).min() == np.float32(2.0 ** lo_exp)
    want, st = oracle.rtn_quantize(x, scale)
    assert st == 0
    Q, _, status = imu.imunpack_quantize(dev(torch.from_numpy(x)), scale, 8, want_stats=False)
    assert int(status.item()) == 0
    assert np.array_equal(Q.cpu().numpy(), want)
    # the transposing path runs the same arithmetic on the same values
    Qt, _, status = imu.imunpack_quantize(dev(torch.from_numpy(x)).t(), scale, 8, want_stats=False)
    assert int(status.item()) == 0
    assert np.array_equal(Qt.cpu().numpy(), want.T)


def test_quantize_flags_bad_input(imu):
    x = torch.ones(8, 8)
    x[3, 4] = float("nan")
    _, _, status = imu.imunpack_quantize(dev(x), 1.0, 8)
    assert int(status.item()) == 1
    x[3, 4] = 3.0e9
    Q, _, status = imu.imunpack_quantize(dev(x), 1.0, 8)
    assert int(status.item()) == 1 and int(Q[3, 4].item()) == 0
    x[3, 4] = 2.0e9
    Q, _, status = imu.imunpack_quantize(dev(x), 1.0, 8)
    assert int(status.item()) == 0 and int(Q[3, 4].item()) == 2000000000
    with pytest.raises(imu.ImunpackError):
        imu.imunpack_quantize(dev(x), 0.0, 8)
    with pytest.raises(imu.ImunpackError):
        imu.imunpack_quantize(dev(x), 1.0, 9)


# ------------------------------------------------------------------ plan + operands + product
def check_against_oracle(imu, Aq, Bq, b, sa, sb, scale_a=0.013, scale_b=0.0021, full_product=True, fp6=False, lists=None):
    """Aq, Bq: int32 numpy.  Compares plan, unpacked operands, int64 product (fused and un-fused)
    and the fp32 output with the oracle.  fp6: the digits are stored as 6-bit floating-point codes.  lists: the plan is made from
    the caller's statistics and lists of heavy hitters, with so many places each, and not from scans of its own."""
    n, h = Aq.shape[0], Bq.shape[0]
    s = 1 << (b - 1)
    hnd = oracle.unpack_pair_handle(Aq, Bq, b, sa, sb)
    S, pas, paw, pbs, pbw = hnd.meta()
    assert hnd.max_abs() <= s - 1
    if lists is None:
        A_d, B_d = dev(torch.from_numpy(Aq)), dev(torch.from_numpy(Bq))
        plan = imu.imunpack_plan(A_d, B_d, b, sa, sb)
    else:
        (A_d, stats_a), (B_d, stats_b) = _listed(imu, Aq, b, lists[0]), _listed(imu, Bq, b, lists[1])
        plan = imu.imunpack_plan(A_d, B_d, b, sa, sb, stats_a, stats_b)
    n_u, d_u, h_u, ng = plan.dims()
    assert (n_u, d_u, h_u) == (hnd.n_u, hnd.d_u, hnd.h_u)
    ra_s, ra_e, rb_s, rb_e, c_s, c_e, c_par, ops = [t.numpy().astype(np.int64) for t in plan.export_all()]
    want_parent, want_ops = hnd.trace()
    assert np.array_equal(c_s, hnd.col_src()) and np.array_equal(c_par, want_parent)
    assert np.array_equal(ops, want_ops)          # every split, in the order Alg. 1 / 2 / 4 make them
    assert np.array_equal(ra_s, pas) and np.array_equal(s ** ra_e.astype(object), paw.astype(object))
    assert np.array_equal(rb_s, pbs) and np.array_equal(s ** rb_e.astype(object), pbw.astype(object))
    assert np.array_equal(s ** c_e.astype(object), S.astype(object))
    assert ng == len(np.unique(S))
    if fp6:
        plan.set_digits(imu.DIGITS_FP6)
    assert plan.digits() == (imu.DIGITS_FP6 if fp6 else imu.DIGITS_INT8)
    A_ue, B_eu = imu.imunpack_unpack(plan, A_d, B_d)
    Ac, Bc = imu.imunpack_unpack_canonical(plan, A_ue, B_eu)
    oa, ob = hnd.operands_i8()
    assert np.array_equal(Ac.cpu().numpy(), oa)
    assert np.array_equal(Bc.cpu().numpy(), ob)
    # B_eu is stored in full and its padding (and the zero columns beside columns of A it has no copy
    # for) must be zero: total magnitude is preserved.  Of A_ue every column of A_u is stored once (the
    # repeated columns are read from there), plus a few gathered copies: never more than A_ue holds.
    (ra, wa, pa), (rb, wb, pb) = plan.layout()
    assert A_ue.numel() == ra * pa == plan.unpacked_bytes()[0] and B_eu.numel() == rb * pb == plan.unpacked_bytes()[1]
    if fp6:  # 96 bytes per 128 columns; a zero digit is the code 0, so the number of non-zero bits bounds the padding
        assert pa >= wa * 3 // 4 and pb >= wb * 3 // 4
        nz_b = int((B_eu.view(rb, pb)[:, :wb * 3 // 4] != 0).sum().item())
        assert nz_b <= int((ob != 0).sum())  # every stored non-zero byte holds bits of a non-zero digit...
        assert nz_b * 2 >= int((ob != 0).sum())  # ... and a byte holds bits of at most two digits
    else:
        stored_b = B_eu.view(rb, pb)[:, :wb].to(torch.int64)
        assert int(stored_b.abs().sum().item()) == int(np.abs(ob.astype(np.int64)).sum())
        stored_a = A_ue.view(ra, pa)[:, :wa].to(torch.int64)
        assert int(stored_a.abs().sum().item()) <= int(np.abs(oa.astype(np.int64)).sum())
    assert wa <= wb and wa % 128 == 0 and wb % 128 == 0
    check_bounds(plan, oa, ob, S, s, fp6)
    want = oracle.int_gemm(Aq, Bq)
    want_fp = oracle.dequantize(want, scale_a, scale_b)
    ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
    results = []
    # un-fused: GEMM into the int64 workspace, then recombine
    C_int = torch.full((n, h), -7, dtype=torch.int64, device="cuda")
    C_fp = torch.full((n, h), -7.0, dtype=torch.float32, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, scale_a, scale_b, None, None, ws, fuse=False)
    imu.imunpack_recombine(plan, ws, scale_a, scale_b, C_int, C_fp)
    results.append(("unfused", C_int, C_fp))
    # fused (falls back to the un-fused kernels by itself when the int32 bound does not hold)
    C_int2 = torch.full((n, h), -7, dtype=torch.int64, device="cuda")
    C_fp2 = torch.full((n, h), -7.0, dtype=torch.float32, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, scale_a, scale_b, C_int2, C_fp2, ws, fuse=True)
    results.append(("fused" if plan.fusable() else "fused->fallback", C_int2, C_fp2))
    # fp32 output alone: the fused epilogue may then add the digit levels up in binary64 instead of
    # int64, which must not change a single bit of the result
    C_fp3 = torch.full((n, h), -7.0, dtype=torch.float32, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, scale_a, scale_b, None, C_fp3, ws, fuse=True)
    assert torch.equal(C_fp3, C_fp2), "fp32-only output differs from the fp32 + int64 call"
    for name, ci, cf in results:
        assert np.array_equal(ci.cpu().numpy(), want), name
        got = cf.cpu().numpy().astype(np.float64)
        err = np.abs(got - want_fp)
        assert (err <= REL_TOL * np.abs(want_fp)).all(), name
    hnd.close()
    return plan


def check_bounds(plan, oa, ob, S, s, fp6=False):
    """The accumulator bounds the scatter measured against their definition, evaluated on the
    oracle's unpacked operands: max over rows of sum_c S[c] |digit|; and the path they select."""
    w = np.array([int(x) for x in S], dtype=object)
    want = []
    for m in (oa, ob):
        if m.size == 0:
            want.append(0)
            continue
        rows = (np.abs(m.astype(np.int64)).astype(object) * w[None, :]).sum(1)
        want.append(int(max(rows)))
    got = plan.bounds()
    for g, t in zip(got, want):
        assert g == t if t < (1 << 44) else g >= (1 << 44), (got, want)
    m = min(want)
    assert plan.fusable() == (m < (1 << 40) and m * (s - 1) < (1 << (24 if fp6 else 31)))


def rand_ints(rng, rows, cols, s, p_ob, depth):
    M = rng.integers(-(s - 1), s, size=(rows, cols))
    mask = rng.random((rows, cols)) < p_ob
    big = rng.integers(-(s ** depth), s ** depth + 1, size=(rows, cols))
    return np.where(mask, big, M).astype(np.int32)


@pytest.mark.parametrize("n,d,h,share_a,share_b,longer,digits", [
    (900, 1200, 80, 0.04, 0.01, 0.0, 3),      # more heavy hitters than LDS holds, none of three digits
    (900, 1200, 80, 0.04, 0.01, 0.00002, 3),  # ... a few of three digits
    (900, 1200, 80, 0.04, 0.01, 0.004, 4),    # ... several of up to four in one row and column
    (60, 1500, 1100, 0.01, 0.03, 0.001, 3),   # the second operand, with repeated columns
    (2500, 700, 40, 0.02, 0.02, 0.0005, 3),
    (400, 300, 200, 0.05, 0.05, 0.002, 3),    # all of them in LDS
])
def test_greedy_with_entries_of_three_digits_and_many_heavy_hitters(imu, n, d, h, share_a, share_b, longer, digits):
    """UnpackBoth takes many slots in one batch also where some entries keep heavy hitters in the slots that a split appends:
    every split, in order, against Alg. 4 step by step.  Uneven rows and columns, so that both sides are split in turn."""
    s = 128
    rng = np.random.default_rng(n + d + digits)

    def draw(rows, share):
        M = rng.integers(-(s - 1), s, size=(rows, d))
        uneven = (rng.random(d) ** 3 * 3)[None, :] * (rng.random(rows) ** 2 * 2)[:, None]
        M = np.where(rng.random((rows, d)) < share * uneven, rng.integers(s, s * s, size=(rows, d)), M)
        return np.where(rng.random((rows, d)) < longer, rng.integers(s * s, s ** digits, size=(rows, d)), M).astype(np.int32)

    check_against_oracle(imu, draw(n, share_a), draw(h, share_b), 8, BOTH, BOTH)


@pytest.mark.parametrize("d", [1, 120, 128, 250, 380, 512, 640, 1000, 1030])
@pytest.mark.parametrize("sa,sb", [(ROW, ROW), (COL, ROW), (BOTH, ROW)])
def test_stores_of_every_width(imu, d, sa, sb):
    """Stores of one to eight blocks of 128 columns, where a wave of the scatter takes eight bands to half a band, and operands
    of different widths in one launch: digits, padding, norms and the product."""
    rng = np.random.default_rng(d)
    check_against_oracle(imu, rand_ints(rng, 150, d, 128, 0.004, 2), rand_ints(rng, 90, d, 128, 0.004, 3), 8, sa, sb)


@pytest.mark.parametrize("h", [6000, 6001])
@pytest.mark.parametrize("split_rows", [0, 40])
def test_large_products_without_levels_leave_by_rows(imu, h, split_rows):
    """Products whose operands outgrow the last-level cache: results go out row by row, ragged ends and some rows of two
    levels on either side among them.  The integer product is exact in binary64 (below 2^31), so the result is too but for its
    one rounding."""
    n, d = 4140, 4100
    g = torch.Generator(device="cuda").manual_seed(h + split_rows)
    A = torch.randint(-127, 128, (n, d), generator=g, device="cuda", dtype=torch.int32)
    B = torch.randint(-127, 128, (h, d), generator=g, device="cuda", dtype=torch.int32)
    for X in (A, B):
        at = torch.randperm(X.shape[0], generator=g, device="cuda")[:split_rows]
        X[at, at % d] = 700
    plan = imu.imunpack_plan(A, B, 8, ROW, ROW)
    A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
    C = torch.full((n + 1, h), 3.5, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C[:n], None)
    scale = float(np.float32(0.013)) * float(np.float32(0.0021))
    assert torch.equal(C[:n], ((A.double() @ B.double().t()) * scale).float())
    assert (C[n] == 3.5).all()


@pytest.mark.parametrize("n,d,h", [(1, 1, 1), (40, 8191, 24), (24, 8192, 24), (40, 8193, 24), (8192, 40, 16), (16, 40, 8193)])
@pytest.mark.parametrize("sa,sb", list(itertools.product([ROW, COL], [ROW, COL])))
def test_rows_and_columns_planned_in_one_launch(imu, n, d, h, sa, sb):
    """On either side of the 8192 rows and columns up to which one launch unpacks both operands; the second one splits the
    columns that the first one left, which are more than 8192 where the first one split some."""
    rng = np.random.default_rng(n + d + h)
    check_against_oracle(imu, rand_ints(rng, n, d, 128, 0.0005, 2), rand_ints(rng, h, d, 128, 0.0005, 3), 8, sa, sb)


@pytest.mark.parametrize("sa,sb", list(itertools.product(STRATS, STRATS)))
@pytest.mark.parametrize("b", [8, 4, 2])
def test_small_random_all_strategies(imu, sa, sb, b):
    rng = np.random.default_rng(100 * b + 10 * sa + sb)
    s = 1 << (b - 1)
    depth = 3 if b > 2 else 5
    Aq = rand_ints(rng, 70, 90, s, 0.03, depth)
    Bq = rand_ints(rng, 50, 90, s, 0.03, depth)
    check_against_oracle(imu, Aq, Bq, b, sa, sb)


@pytest.mark.parametrize("kind", ["scattered", "channels", "rows", "heavy", "clean", "deep"])
@pytest.mark.parametrize("sa,sb", [(BOTH, BOTH), (ROW, COL), (COL, ROW), (COL, COL)])
def test_structured_multi_tile(imu, kind, sa, sb):
    """Shapes that span several GEMM tiles with ragged tails, heavy hitters laid out as in the
    paper's workloads (a few channels, scattered entries, heavy tails)."""
    w = workloads.small(7, 300, 330, 270, kind=kind, b=8)
    Aq = oracle_quant(w.A, w.scale_a)
    Bq = oracle_quant(w.B, w.scale_b)
    check_against_oracle(imu, Aq, Bq, 8, sa, sb, w.scale_a, w.scale_b)


@pytest.mark.parametrize("sa,sb", [(ROW, COL), (BOTH, BOTH), (COL, COL), (COL, ROW), (BOTH, ROW)])
@pytest.mark.parametrize("b", [4, 3, 2])
def test_six_bit_floating_point_digits(imu, sa, sb, b):
    """b <= 4 (Sec. 4.2, low bit widths): the digits stored as e2m3 codes and multiplied by the
    f8f6f4 matrix instruction give the same unpacked operands (decoded) and the same product, bit for bit."""
    rng = np.random.default_rng(1000 * b + 10 * sa + sb)
    s = 1 << (b - 1)
    Aq = rand_ints(rng, 150, 300, s, 0.05, 3 if b > 2 else 5)
    Bq = rand_ints(rng, 270, 300, s, 0.05, 3 if b > 2 else 5)
    check_against_oracle(imu, Aq, Bq, b, sa, sb, fp6=True)


@pytest.mark.parametrize("sa,sb", [(COL, COL), (ROW, BOTH)])
@pytest.mark.parametrize("d", [890, 1025, 4100, 9000])
def test_columns_laid_out_by_several_workgroups(imu, d, sa, sb):
    """Stored columns from just one step of 1024 to more steps than workgroups that take them in turn."""
    rng = np.random.default_rng(d)
    check_against_oracle(imu, rand_ints(rng, 33, d, 16, 0.01, 2), rand_ints(rng, 20, d, 16, 0.002, 2), 5, sa, sb)


@pytest.mark.parametrize("sa,sb", [(ROW, COL), (BOTH, BOTH)])
@pytest.mark.parametrize("n,h,d", [(70, 40, 100), (70, 300, 257), (300, 520, 300), (290, 330, 2810)])
def test_six_bit_rows_that_share_their_bytes(imu, n, h, d, sa, sb):
    """One, two, an odd number of k-tiles, and rows wide enough to be padded: the last k-tile of an odd number has no partner, and its
    place in the odd row holds zeros.  The buffers hold other bytes before."""
    rng = np.random.default_rng(d)
    Aq, Bq = rand_ints(rng, n, d, 8, 0.01, 2), rand_ints(rng, h, d, 8, 0.01, 2)
    A_d, B_d = dev(torch.from_numpy(Aq)), dev(torch.from_numpy(Bq))
    plan = imu.imunpack_plan(A_d, B_d, 4, sa, sb)
    plan.set_digits(imu.DIGITS_FP6)
    ba, bb, _ = plan.unpacked_bytes()
    A6, B6 = torch.full((ba,), 0x55, dtype=torch.int8, device="cuda"), torch.full((bb,), 0x55, dtype=torch.int8, device="cuda")
    imu.imunpack_unpack(plan, A_d, B_d, A6, B6)
    for got, want in zip(imu.imunpack_unpack_canonical(plan, A6, B6), oracle.unpack_pair_handle(Aq, Bq, 4, sa, sb).operands_i8()):
        assert np.array_equal(got.cpu().numpy(), want)
    for buf, (rows, width, pitch) in zip((A6, B6), plan.layout()):
        if width // 128 % 2 and width > 128:
            assert not buf.view(rows, pitch)[1::2, width * 3 // 4 - 96:width * 3 // 4 + 96].any()
    C = torch.empty((n, h), dtype=torch.float32, device="cuda")
    imu.imunpack_gemm(plan, A6, B6, 1.0, 1.0, None, C, torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda"))
    want = oracle.dequantize(oracle.int_gemm(Aq, Bq), 1.0, 1.0)
    assert (np.abs(C.cpu().numpy() - want) <= 1e-6 * np.abs(want)).all()


def test_six_bit_digits_fused_path_and_format_rules(imu):
    """A case whose accumulator bound stays below 2^24 runs the fused 6-bit kernel (Horner step as a
    multiplication by a power of two in binary32); the format is refused for b > 4, and a plan object
    that asked for it goes back to int8 when it is re-planned with b > 4."""
    rng = np.random.default_rng(77)
    b, s = 4, 8
    Aq = rand_ints(rng, 300, 700, s, 0.02, 2)
    Bq = rand_ints(rng, 520, 700, s, 0.02, 2)
    plan = check_against_oracle(imu, Aq, Bq, b, COL, COL, fp6=True)
    assert plan.fusable() and plan.digits() == imu.DIGITS_FP6 and plan.dims()[3] >= 2
    # a second unpack of the same plan into fresh buffers (the row norms are cleared and measured again)
    A_d, B_d = dev(torch.from_numpy(Aq)), dev(torch.from_numpy(Bq))
    bounds = plan.bounds()
    A6, B6 = imu.imunpack_unpack(plan, A_d, B_d)
    assert plan.bounds() == bounds
    C = torch.empty((Aq.shape[0], Bq.shape[0]), dtype=torch.int64, device="cuda")
    imu.imunpack_gemm(plan, A6, B6, 1.0, 1.0, C, None, None, fuse=True)
    assert np.array_equal(C.cpu().numpy(), oracle.int_gemm(Aq, Bq))
    A8 = rand_ints(rng, 64, 128, 128, 0.02, 2)
    B8 = rand_ints(rng, 64, 128, 128, 0.02, 2)
    imu.imunpack_plan(dev(torch.from_numpy(A8)), dev(torch.from_numpy(B8)), 8, ROW, ROW, plan=plan)
    assert plan.digits() == imu.DIGITS_INT8
    with pytest.raises(imu.ImunpackError):
        plan.set_digits(imu.DIGITS_FP6)
    with pytest.raises(imu.ImunpackError):
        plan.set_digits(7)
    imu.imunpack_plan(dev(torch.from_numpy(Aq)), dev(torch.from_numpy(Bq)), b, COL, COL, plan=plan)
    assert plan.digits() == imu.DIGITS_FP6          # the request stayed with the plan object
    plan.set_digits(imu.DIGITS_INT8)
    assert plan.digits() == imu.DIGITS_INT8


@pytest.mark.parametrize("sa,sb", [(BOTH, BOTH), (ROW, BOTH), (COL, BOTH), (BOTH, COL), (ROW, COL), (COL, ROW), (BOTH, ROW)])
def test_keep_weights_takes_the_second_operand_over_only_when_it_may(imu, sa, sb):
    """Keep-weights mode (Sec. 4.2: weights unpacked once): with B fixed, a plan call reuses B's unpacking
    exactly when the column slots of A's unpacking are those of the call before.  Every call's plan (every
    split in order), unpacked operands and product are compared with the oracle's, reused or not."""
    rng = np.random.default_rng(4242 + 3 * sa + sb)
    b, s = 8, 128
    n, d, h = 150, 300, 270
    Bq = rand_ints(rng, h, d, s, 0.02, 2)
    def make_A(cols, seed):
        r = np.random.default_rng(seed)
        A = r.integers(-(s - 1), s, size=(n, d)).astype(np.int32)
        for c in cols:                                  # heavy columns: the column splits of A's unpacking
            A[:, c] = r.integers(s, s * s, size=n).astype(np.int32) * r.choice([-1, 1], size=n)
        if sa == ROW:
            A[r.integers(0, n, 5), :] = r.integers(-(s * s - 1), s * s, size=(5, d)).astype(np.int32)
        return A
    B_d = dev(torch.from_numpy(Bq))
    plan = imu.Plan()
    buf_a = torch.empty(8 << 20, dtype=torch.int8, device="cuda")
    buf_b = torch.empty(8 << 20, dtype=torch.int8, device="cuda")
    seq = [((3, 77, 200), 1, False),     # first call in this mode: B is unpacked
           ((3, 77, 200), 2, True),      # other values, same heavy columns: the same column slots
           ((3, 77, 200), 3, True),
           ((5, 77, 201), 4, False),     # other columns split: B is unpacked again
           ((5, 77, 201), 5, True),
           ((3, 77, 200), 6, False)]
    if sa == ROW:                        # no column of A is ever split: always the same column slots
        seq = [(c, k, i > 0) for i, (c, k, _) in enumerate(seq)]
    for i, (cols, seed, want_reuse) in enumerate(seq):
        Aq = make_A(cols, seed)
        A_d = dev(torch.from_numpy(Aq))
        imu.imunpack_plan(A_d, B_d, b, sa, sb, plan=plan)
        if i == 0:
            assert not plan.weights_reused()
            plan.keep_weights(True)      # from the next call on
            imu.imunpack_plan(A_d, B_d, b, sa, sb, plan=plan)
            assert not plan.weights_reused()
        else:
            assert plan.weights_reused() == want_reuse, (i, cols)
        hnd = oracle.unpack_pair_handle(Aq, Bq, b, sa, sb)
        assert plan.dims()[:3] == (hnd.n_u, hnd.d_u, hnd.h_u)
        got = [t.numpy().astype(np.int64) for t in plan.export_all()]
        S, pas, paw, pbs, pbw = hnd.meta()
        want_parent, want_ops = hnd.trace()
        assert np.array_equal(got[0], pas) and np.array_equal(got[2], pbs) and np.array_equal(got[4], hnd.col_src())
        assert np.array_equal(got[6], want_parent) and np.array_equal(got[7], want_ops)
        assert np.array_equal(s ** got[5].astype(object), S.astype(object))
        # the same two buffers in every call: with B's unpacking taken over, B_eu is left as the unpack before wrote it
        ba, bb, bw = plan.unpacked_bytes()
        assert ba <= buf_a.numel() and bb <= buf_b.numel()
        A_ue, B_eu = imu.imunpack_unpack(plan, A_d, B_d, buf_a, buf_b)
        Ac, Bc = imu.imunpack_unpack_canonical(plan, A_ue, B_eu)
        oa, ob = hnd.operands_i8()
        assert np.array_equal(Ac.cpu().numpy(), oa) and np.array_equal(Bc.cpu().numpy(), ob)
        check_bounds(plan, oa, ob, S, s)
        C = torch.empty((n, h), dtype=torch.int64, device="cuda")
        ws = torch.empty(bw // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C, None, ws, fuse=True)
        assert np.array_equal(C.cpu().numpy(), oracle.int_gemm(Aq, Bq)), i
        if i == 2:  # a second unpack of the same plan measures the row norms again: nothing may be left out then
            imu.imunpack_unpack(plan, A_d, B_d, buf_a, buf_b)
            check_bounds(plan, oa, ob, S, s)
        hnd.close()
    plan.keep_weights(False)
    imu.imunpack_plan(A_d, B_d, b, sa, sb, plan=plan)
    assert not plan.weights_reused()


def test_keep_weights_with_other_buffers(imu):
    """A plan that took B's unpacking over, unpacked into another B_eu buffer than before: B is written again and its row
    norms are measured afresh, not on top of the old ones."""
    rng = np.random.default_rng(77)
    Aq, Bq = (rand_ints(rng, r, 400, 128, 0.004, 2) for r in (60, 150))
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    want = oracle.int_gemm(Aq, Bq)
    plan, bounds, held = imu.Plan(), None, []
    for i in range(4):
        imu.imunpack_plan(Qa, Qb, 8, ROW, BOTH, plan=plan)
        plan.keep_weights(True)
        assert plan.weights_reused() == (i > 1)
        held.append(imu.imunpack_unpack(plan, Qa, Qb))
        bounds = bounds or plan.bounds()
        assert plan.bounds() == bounds, i
        C_int = torch.full(want.shape, -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, *held[-1], 1.0, 1.0, C_int, None, None, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), want)


@pytest.mark.parametrize("b", [3, 5, 6, 7])
def test_other_bit_widths(imu, b):
    w = workloads.small(11, 130, 200, 140, kind="scattered", b=b)
    Aq = oracle_quant(w.A, w.scale_a)
    Bq = oracle_quant(w.B, w.scale_b)
    check_against_oracle(imu, Aq, Bq, b, BOTH, COL, w.scale_a, w.scale_b)
    check_against_oracle(imu, Aq, Bq, b, ROW, BOTH, w.scale_a, w.scale_b)


def test_degenerate_shapes(imu):
    rng = np.random.default_rng(5)
    for (n, d, h) in [(1, 1, 1), (1, 300, 1), (257, 1, 3), (2, 65, 600)]:
        Aq = rand_ints(rng, n, d, 128, 0.1, 3)
        Bq = rand_ints(rng, h, d, 128, 0.1, 3)
        for sa, sb in [(ROW, ROW), (COL, COL), (BOTH, BOTH)]:
            check_against_oracle(imu, Aq, Bq, 8, sa, sb)
    # the scalar example of Sec. 4: five base-128 digits each, 25 low-bit multiplications
    Aq = np.array([[2 ** 31 - 1]], dtype=np.int32)
    Bq = np.array([[-(128 ** 4) - 77]], dtype=np.int32)
    for sa, sb in itertools.product(STRATS, STRATS):
        plan = check_against_oracle(imu, Aq, Bq, 8, sa, sb)
        n_u, d_u, h_u, _ = plan.dims()
        assert n_u * d_u * h_u == 25


def test_plan_object_is_reusable(imu):
    rng = np.random.default_rng(9)
    plan = None
    for (n, d, h, sa, sb) in [(40, 50, 30, BOTH, BOTH), (300, 100, 80, ROW, COL), (40, 50, 30, COL, BOTH)]:
        Aq = rand_ints(rng, n, d, 128, 0.05, 3)
        Bq = rand_ints(rng, h, d, 128, 0.05, 3)
        A_d, B_d = dev(torch.from_numpy(Aq)), dev(torch.from_numpy(Bq))
        plan = imu.imunpack_plan(A_d, B_d, 8, sa, sb, plan=plan)
        hnd = oracle.unpack_pair_handle(Aq, Bq, 8, sa, sb)
        assert plan.dims()[:3] == (hnd.n_u, hnd.d_u, hnd.h_u)
        A_ue, B_eu = imu.imunpack_unpack(plan, A_d, B_d)
        C_int = torch.empty((n, h), dtype=torch.int64, device="cuda")
        ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, ws, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), oracle.int_gemm(Aq, Bq))


def test_end_to_end_config1(imu):
    """Workload 1 (256 x 256 x 256, scattered heavy hitters, UnpackBoth on both operands) through the
    whole path, full comparison of every stage."""
    w = workloads.make(1)
    Aq = oracle_quant(w.A, w.scale_a)
    Bq = oracle_quant(w.B, w.scale_b)
    Qa, _, _ = imu.imunpack_quantize(dev(w.A), w.scale_a, w.b)
    Qb, _, _ = imu.imunpack_quantize(dev(w.B), w.scale_b, w.b)
    assert np.array_equal(Qa.cpu().numpy(), Aq) and np.array_equal(Qb.cpu().numpy(), Bq)
    check_against_oracle(imu, Aq, Bq, w.b, w.strategy_a, w.strategy_b, w.scale_a, w.scale_b)
    C_int, C_fp, plan = imu.exact_int_gemm(dev(w.A), dev(w.B), w.scale_a, w.scale_b, w.b, w.strategy_a,
                                           w.strategy_b)
    want = oracle.int_gemm(Aq, Bq)
    assert np.array_equal(C_int.cpu().numpy(), want)
    ref = oracle.dequantize(want, w.scale_a, w.scale_b)
    assert (np.abs(C_fp.cpu().numpy().astype(np.float64) - ref) <= REL_TOL * np.abs(ref)).all()


def test_run_to_run_determinism(imu):
    """All outputs are integers (the fp32 one is a function of an integer), atomics only add
    integers, so every stage must reproduce itself bit for bit, whatever the thread timing."""
    g = torch.Generator().manual_seed(3)
    A = torch.randn(600, 1100, generator=g) * 2
    B = torch.randn(520, 1100, generator=g)
    B[torch.randperm(520, generator=g)[:6], :] *= 60          # heavy-hitter rows: one big row batch
    A[torch.rand(A.shape, generator=g) < 0.004] *= 90         # scattered heavy hitters
    sa, sb = workloads.rtn_scale(A), workloads.rtn_scale(B)
    A_d, B_d = dev(A), dev(B)
    plan = imu.Plan()
    first = None
    for _ in range(12):
        Qa, st_a, _ = imu.imunpack_quantize(A_d, sa, 8, want_ob_list=True)
        Qb, st_b, _ = imu.imunpack_quantize(B_d, sb, 8, want_ob_list=True)
        imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH, st_a, st_b, plan)
        A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
        C_int = torch.empty((600, 520), dtype=torch.int64, device="cuda")
        ws = None if plan.fusable() else torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, sa, sb, C_int, None, ws, fuse=True)
        cur = [Qa, Qb, torch.tensor(plan.dims()), torch.cat(plan.export()), A_ue.clone(), B_eu.clone(), C_int]
        if first is None:
            first = [t.clone() for t in cur]
            want = oracle.int_gemm(oracle_quant(A, sa), oracle_quant(B, sb))
            assert np.array_equal(C_int.cpu().numpy(), want)
        else:
            for a, b in zip(first, cur):
                assert a.shape == b.shape and torch.equal(a, b)


def test_fused_launch_before_the_bounds_are_known(imu):
    """imunpack_unpack leaves the accumulator bounds in flight and a fused imunpack_gemm goes out
    guarded before the host has them.  On data whose shifted group sum does not fit int32 the guarded
    launch must write nothing: without a workspace the call reports ERANGE, with one it falls back to
    the un-fused path and the result is exact."""
    rng = np.random.default_rng(5)
    Aq = rng.integers(-(1 << 22), 1 << 22, size=(96, 320)).astype(np.int32)
    Bq = rng.integers(-(1 << 22), 1 << 22, size=(80, 320)).astype(np.int32)
    want = oracle.int_gemm(Aq, Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, ROW, COL)   # a new plan object guesses "fused"
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C_int = torch.full(want.shape, -7, dtype=torch.int64, device="cuda")
    with pytest.raises(imu.ImunpackError) as err:
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
    assert err.value.code == imu.ERANGE
    assert not plan.fusable()
    assert bool((C_int == -7).all()), "the guarded launch must not have written anything"
    plan2 = imu.imunpack_plan(Qa, Qb, 8, ROW, COL)
    A2, B2 = imu.imunpack_unpack(plan2, Qa, Qb)
    ws = torch.empty(plan2.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
    imu.imunpack_gemm(plan2, A2, B2, 1.0, 1.0, C_int, None, ws, fuse=True)   # guarded launch, then the fallback
    assert np.array_equal(C_int.cpu().numpy(), want)


def test_streaming_copy_copies(imu):
    """The copy kernel behind the benchmark's measured HBM rate moves every byte (3 MiB: three bands)."""
    g = torch.Generator().manual_seed(3)
    src = torch.randint(-2 ** 31, 2 ** 31 - 1, (3 << 18,), dtype=torch.int32, generator=g).to("cuda")
    dst = torch.zeros_like(src)
    assert imu.imunpack_diag_copy(src, dst) == 2 * (3 << 20)
    assert torch.equal(src, dst)
    with pytest.raises(imu.ImunpackError):
        imu.imunpack_diag_copy(src[:1000], dst[:1000])


def test_clock_probe_reports_a_plausible_clock_and_leaves_the_result_alone(imu):
    """While the probe is set a fused GEMM writes {shader cycles, 100 MHz ticks} of its first workgroup's
    loop over K; the product is the same with and without it, and nothing is written once it is off."""
    rng = np.random.default_rng(11)
    Aq = rng.integers(-300, 300, size=(300, 4096)).astype(np.int32)
    Bq = rng.integers(-300, 300, size=(260, 4096)).astype(np.int32)
    want = oracle.int_gemm(Aq, Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, ROW, COL)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    assert plan.fusable()
    C_int = torch.empty(want.shape, dtype=torch.int64, device="cuda")
    ticks = torch.zeros(2, dtype=torch.int64, device="cuda")
    imu.imunpack_diag_clock_probe(ticks)
    try:
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
        torch.cuda.synchronize()
    finally:
        imu.imunpack_diag_clock_probe(None)
    assert np.array_equal(C_int.cpu().numpy(), want)
    cyc, wall = ticks.tolist()
    assert cyc > 0 and wall > 0
    assert 300.0 < 100.0 * cyc / wall < 3000.0, (cyc, wall)
    ticks.zero_()
    imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
    torch.cuda.synchronize()
    assert ticks.tolist() == [0, 0]
    assert np.array_equal(C_int.cpu().numpy(), want)


@pytest.mark.parametrize("kind,b", [("scattered", 8), ("channels", 8), ("heavy", 4), ("deep", 8), ("clean", 8), ("rows", 3)])
def test_price_matches_unpacked_sizes(imu, kind, b):
    """Sec. 4.2: the sizes n', d', h' (and so the unpack ratio r) that imunpack_price reads off the scan
    statistics equal those of the oracle's literal UnpackRow / UnpackColumn for all four pairs, and
    the pair it picks has the smallest r."""
    w = workloads.small(seed=21, n=150, d=260, h=90, kind=kind, b=b)
    Aq, _ = oracle.rtn_quantize(w.A.numpy(), w.scale_a)
    Bq, _ = oracle.rtn_quantize(w.B.numpy(), w.scale_b)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    st_a, st_b = imu.imunpack_scan(Qa, b), imu.imunpack_scan(Qb, b)
    dims, ratios, best = imu.imunpack_price(st_a, w.n, st_b, w.h, w.d, b)
    want_r = {}
    for pair in dims:
        hnd = oracle.unpack_pair_handle(Aq, Bq, b, pair[0], pair[1])
        assert dims[pair] == (hnd.n_u, hnd.d_u, hnd.h_u), pair
        want_r[pair] = hnd.n_u * hnd.d_u * hnd.h_u / (w.n * w.d * w.h)
        assert abs(ratios[pair] - want_r[pair]) <= 1e-12 * want_r[pair]
        hnd.close()
    assert want_r[best] == min(want_r.values())
    # and the planner agrees with the price of the chosen pair
    plan = imu.imunpack_plan(Qa, Qb, b, best[0], best[1], st_a, st_b)
    assert plan.dims()[:3] == (dims[best][0], dims[best][1], dims[best][2])


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (64, 256), (200, 1000), (77, 130), (513, 260), (2048, 2048)])
@pytest.mark.parametrize("p", [0.5, 50.0, 95.0, 99.9, 100.0])
def test_percentile_matches_the_order_statistic(imu, shape, p):
    """alpha_p on the device is the oracle's order statistic, bit for bit (it is an entry of the
    matrix): heavy-tailed values with ties, infinities and zeros, row-major and transposed views."""
    g = torch.Generator().manual_seed(shape[0] * 7919 + shape[1] + int(p * 10))
    x = torch.randn(shape, generator=g) * 0.02
    x[torch.rand(shape, generator=g) < 0.01] *= 50.0
    flat = x.view(-1)
    n = flat.numel()
    if n > 8:
        flat[torch.randint(0, n, (max(1, n // 7),), generator=g)] = float(flat[0])      # ties
        flat[torch.randint(0, n, (max(1, n // 50),), generator=g)] = 0.0
        flat[1] = float("inf")
        flat[2] = -float("inf")
    want = oracle.percentile_alpha(x.numpy(), p)
    for view in (x.to("cuda"), x.t().contiguous().to("cuda").t()):           # unit column stride / unit row stride
        alpha, status = imu.imunpack_percentile(view, p)
        assert int(status.item()) == 0
        got = alpha.cpu().numpy()[0]
        assert got == want or (np.isinf(got) and np.isinf(want)), (got, want)
    # a view with neither stride 1 and an odd row pitch (scalar path)
    wide = torch.zeros((shape[0], 2 * shape[1] + 1), device="cuda")
    wide[:, 0:2 * shape[1]:2] = x.to("cuda")
    alpha, status = imu.imunpack_percentile(wide[:, 0:2 * shape[1]:2], p)
    assert alpha.cpu().numpy()[0] == want or np.isinf(want)


def test_percentile_flags_nan_and_rejects_bad_arguments(imu):
    x = torch.randn(33, 70, device="cuda")
    alpha, status = imu.imunpack_percentile(x, 95.0)
    assert int(status.item()) == 0
    x[5, 6] = float("nan")
    alpha, status = imu.imunpack_percentile(x, 95.0)
    assert int(status.item()) == 1
    for bad in (0.0, -1.0, 100.5, float("nan")):
        with pytest.raises(imu.ImunpackError) as err:
            imu.imunpack_percentile(x, bad)
        assert err.value.code == imu.EINVAL


def test_percentile_step_feeds_the_quantizer(imu):
    """Eq. (quantized_A) end to end: alpha_95 on the device, the step alpha / (0.5 beta), RTN on the
    device; equal to the oracle's chain on the same matrix."""
    g = torch.Generator().manual_seed(11)
    x = torch.randn((300, 520), generator=g) * 0.05
    x[:, 17] *= 40.0
    for beta in (15, 255):
        alpha, _ = imu.imunpack_percentile(x.to("cuda"), 95.0)
        a = alpha.cpu().numpy()[0]
        assert a == oracle.percentile_alpha(x.numpy(), 95.0)
        step = oracle.rtn_step(a, beta)
        Q, _, flag = imu.imunpack_quantize(x.to("cuda"), float(step), 8)
        want, st = oracle.rtn_quantize(x.numpy(), step)
        assert st == 0 and int(flag.item()) == 0
        assert np.array_equal(Q.cpu().numpy(), want)


def _oracle_matmul(A, B, p, beta_a, beta_b):
    """A B^T through the oracle: alpha_p, RTN step, RTN, exact int64 GEMM, fp64 dequantisation."""
    sa = oracle.rtn_step(oracle.percentile_alpha(A, p), beta_a)
    sb = oracle.rtn_step(oracle.percentile_alpha(B, p), beta_b)
    Aq, fa = oracle.rtn_quantize(np.ascontiguousarray(A), sa)
    Bq, fb = oracle.rtn_quantize(np.ascontiguousarray(B), sb)
    assert fa == 0 and fb == 0
    return oracle.dequantize(oracle.int_gemm(Aq, Bq), sa, sb)


@pytest.mark.parametrize("b,strategies", [(8, (BOTH, BOTH)), (5, (ROW, COL)), (4, (COL, ROW))])
def test_linear_layer_forward_and_backward(imu, b, strategies):
    """The three GEMMs of a linear layer (Sec. 3) against the oracle chain on the same operands:
    Y = X W^T, grad_X = grad_Y W, grad_W = grad_Y^T X, each within 1e-6 relative of the exactly
    dequantised integer product (the transposed operands go through the strided quantize path)."""
    from paper_2403_07339_amd import linear
    g = torch.Generator().manual_seed(100 + b)
    n, d, h = 200, 320, 136
    x = torch.randn((n, d), generator=g)
    x[:, 7] *= 30.0                                     # an outlier channel
    cfg = linear.QuantConfig(beta_x=31.0, beta_w=31.0, beta_g=255.0, p=95.0, b=b,
                             strategy_a=strategies[0], strategy_b=strategies[1])
    layer = linear.IMUnpackLinear(d, h, bias=True, cfg=cfg, device="cuda")
    with torch.no_grad():
        w = torch.randn((h, d), generator=g) * 0.05
        w[torch.rand((h, d), generator=g) < 0.002] *= 25.0
        layer.weight.copy_(w)
        layer.bias.copy_(torch.randn(h, generator=g))
    xg = x.to("cuda").requires_grad_(True)
    y = layer(xg)
    gy = torch.randn((n, h), generator=g) * 1e-3
    gy[torch.rand((n, h), generator=g) < 0.01] *= 40.0   # heavy-tailed gradient
    y.backward(gy.to("cuda"))
    xn, wn, gn = x.numpy(), w.numpy(), gy.numpy()
    bias = layer.bias.detach().cpu().numpy().astype(np.float64)
    want_c = _oracle_matmul(xn, wn, 95.0, 31.0, 31.0)
    want_gx = _oracle_matmul(gn, wn.T, 95.0, 255.0, 31.0)
    want_gw = _oracle_matmul(gn.T, xn.T, 95.0, 255.0, 31.0)
    # the product is rounded to fp32 once, the bias addition once more: both relative to their own operands
    got_y = y.detach().cpu().numpy().astype(np.float64)
    assert (np.abs(got_y - (want_c + bias)) <= 2 * REL_TOL * (np.abs(want_c) + np.abs(bias)[None, :])).all()
    for got, want in ((xg.grad, want_gx), (layer.weight.grad, want_gw)):
        got = got.detach().cpu().numpy().astype(np.float64)
        assert (np.abs(got - want) <= REL_TOL * np.abs(want)).all()
    assert np.allclose(layer.bias.grad.cpu().numpy(), gn.sum(0), rtol=1e-5, atol=1e-6)
    # and the quantised layer tracks the fp32 one to within the RTN error of beta = 31 / 255
    ref = torch.nn.functional.linear(x, w, layer.bias.detach().cpu())
    rel = (y.detach().cpu() - ref).norm() / ref.norm()
    assert float(rel) < 0.15


@pytest.mark.parametrize("b,strategies", [(8, (BOTH, BOTH)), (4, (ROW, COL))])
def test_attention_gemms_forward_and_backward(imu, b, strategies):
    """The six GEMMs of self-attention (Sec. 3), two sequences x three heads, each against the oracle
    chain on the very operands the module fed it (the softmax between them is fp32 arithmetic outside
    the GEMMs, so the intermediates are taken from the module's trace):
    P = Q K^T, O = M V, grad_M = grad_O V^T, grad_V = M^T grad_O, grad_Q = grad_P K, grad_K = grad_P^T Q."""
    from paper_2403_07339_amd import attention, linear
    g = torch.Generator().manual_seed(300 + b)
    lead, T, dh = (2, 3), 72, 40
    q = torch.randn((*lead, T, dh), generator=g)
    k = torch.randn((*lead, T, dh), generator=g)
    v = torch.randn((*lead, T, dh), generator=g)
    k[..., 5] *= 12.0                                     # an outlier channel in the keys
    cfg = linear.QuantConfig(beta_x=31.0, beta_w=31.0, beta_g=255.0, p=95.0, b=b,
                             strategy_a=strategies[0], strategy_b=strategies[1])
    trace = {}
    attn = attention.IMUnpackAttention(cfg, trace)
    qd, kd, vd = (t.to("cuda").requires_grad_(True) for t in (q, k, v))
    out = attn(qd, kd, vd)
    go = torch.randn((*lead, T, dh), generator=g) * 1e-2
    go[torch.rand(go.shape, generator=g) < 0.01] *= 30.0
    out.backward(go.to("cuda"))
    assert out.shape == (*lead, T, dh) and set(trace) == {"P", "M", "O", "grad_M", "grad_P"}
    t = {name: val.detach().cpu().numpy() for name, val in trace.items()}
    gq, gk, gv = (x.grad.detach().cpu().numpy() for x in (qd, kd, vd))
    qn, kn, vn, gon = q.numpy(), k.numpy(), v.numpy(), go.numpy()
    bx, bg = 31.0, 255.0

    def close(got, want):
        return (np.abs(got.astype(np.float64) - want) <= REL_TOL * np.abs(want)).all()

    assert np.array_equal(t["O"], out.detach().cpu().numpy())
    for i in range(lead[0]):
        for j in range(lead[1]):
            M, gP = t["M"][i, j], t["grad_P"][i, j]
            assert close(t["P"][i, j], _oracle_matmul(qn[i, j], kn[i, j], 95.0, bx, bx))
            assert close(t["O"][i, j], _oracle_matmul(M, vn[i, j].T, 95.0, bx, bx))
            assert close(t["grad_M"][i, j], _oracle_matmul(gon[i, j], vn[i, j], 95.0, bg, bx))
            assert close(gv[i, j], _oracle_matmul(M.T, gon[i, j].T, 95.0, bx, bg))
            assert close(gq[i, j], _oracle_matmul(gP, kn[i, j].T, 95.0, bg, bx))
            assert close(gk[i, j], _oracle_matmul(gP.T, qn[i, j].T, 95.0, bg, bx))
    # the fp32 steps between the GEMMs, and the whole against fp32 attention
    scale = 1.0 / np.sqrt(dh)
    Mref = torch.softmax(trace["P"].cpu() * scale, -1).numpy()
    assert np.allclose(t["M"], Mref, rtol=1e-5, atol=1e-7)
    gPref = (t["grad_M"] - (t["grad_M"] * t["M"]).sum(-1, keepdims=True)) * t["M"] * scale
    assert np.allclose(t["grad_P"], gPref, rtol=1e-4, atol=1e-8)
    ref = torch.nn.functional.scaled_dot_product_attention(q, k, v)
    rel = (out.detach().cpu() - ref).norm() / ref.norm()
    assert float(rel) < 0.2


@pytest.mark.parametrize("seed", list(range(24)))
def test_random_shapes_strategies_and_densities(imu, seed):
    """Seeded sweep over what the other cases fix: ragged shapes from one row to a few tiles, every
    bit width, every strategy pair, OB densities from none to most entries, up to five digits, heavy
    rows / heavy columns / scattered entries mixed."""
    rng = np.random.default_rng(9000 + seed)
    b = int(rng.integers(2, 9))
    s = 1 << (b - 1)
    n, d, h = (int(rng.integers(1, 520)) for _ in range(3))
    sa, sb = int(rng.integers(0, 3)), int(rng.integers(0, 3))
    depth = int(rng.integers(1, 6 if b <= 4 else 4))
    p_ob = float(rng.choice([0.0, 0.001, 0.02, 0.3, 0.9]))
    Aq = rand_ints(rng, n, d, s, p_ob, depth)
    Bq = rand_ints(rng, h, d, s, float(rng.choice([0.0, 0.005, 0.1])), depth)
    if rng.random() < 0.5 and d > 2:      # heavy columns of A (outlier channels)
        Aq[:, rng.integers(0, d, 2)] = rng.integers(-(s ** depth), s ** depth + 1, size=(n, 2)).astype(np.int32)
    if rng.random() < 0.5 and h > 2:      # heavy rows of B
        Bq[rng.integers(0, h, 2), :] = rng.integers(-(s ** depth), s ** depth + 1, size=(2, d)).astype(np.int32)
    check_against_oracle(imu, Aq, Bq, b, sa, sb)


def test_rtn_step_on_the_device(imu):
    """alpha_p / (0.5 beta) formed on the device against the oracle's order statistic and binary32 division;
    the fall-backs for a mostly-zero and an all-zero matrix (largest magnitude, then 1)."""
    g = torch.Generator().manual_seed(11)
    x = torch.randn((300, 260), generator=g) * 0.7
    x[torch.rand(x.shape, generator=g) < 0.01] *= 90.0
    xd = dev(x)
    for p, beta, view, view_d in ((95.0, 31.0, x, xd), (99.0, 255.0, x.t(), xd.t()), (50.0, 15.0, x[:, ::2], xd[:, ::2])):
        step, status = imu.imunpack_rtn_step(view_d, p, beta)
        want = oracle.rtn_step(oracle.percentile_alpha(view.contiguous().numpy(), p), beta)
        assert int(status.item()) == 0
        assert step.cpu().numpy().view(np.uint32)[0] == np.float32(want).view(np.uint32)
    sparse = torch.zeros((64, 64))
    sparse[3, 5] = -7.5                                    # the 95th percentile of the magnitudes is 0
    step, _ = imu.imunpack_rtn_step(dev(sparse), 95.0, 31.0)
    assert step.item() == float(np.float32(7.5) / np.float32(15.5))
    step, _ = imu.imunpack_rtn_step(dev(torch.zeros((64, 64))), 95.0, 31.0)
    assert step.item() == 1.0


@pytest.mark.parametrize("b,strategies", [(8, (BOTH, BOTH)), (4, (ROW, COL)), (6, (COL, BOTH))])
def test_gemm_batched_matches_the_oracle_chain_per_item(imu, b, strategies):
    """imunpack_gemm_batched: five products of one shape in one call, operands passed as strided views (one
    of them transposed), each against the oracle chain percentile -> step -> RTN -> exact int64 GEMM -> fp64
    dequantisation on that item's own operands; a second call on the same context with a smaller shape."""
    g = torch.Generator().manual_seed(500 + b)
    ctx = imu.BatchContext()
    for batch, n, d, h in ((5, 48, 72, 56), (2, 17, 40, 9)):
        a = torch.randn((batch, n, d), generator=g)
        a[:, :, 3] *= 25.0
        bt = torch.randn((batch, d, h), generator=g) * 0.03          # stored d x h: B_i is its transpose
        bt[torch.rand(bt.shape, generator=g) < 0.004] *= 30.0
        A_d, B_d = dev(a), dev(bt).transpose(-1, -2)
        out = imu.imunpack_gemm_batched(A_d, B_d, 95.0, 31.0, 63.0, b, strategies[0], strategies[1], ctx=ctx)
        assert out.shape == (batch, n, h)
        got = out.cpu().numpy().astype(np.float64)
        for i in range(batch):
            want = _oracle_matmul(a[i].numpy(), bt[i].t().contiguous().numpy(), 95.0, 31.0, 63.0)
            assert (np.abs(got[i] - want) <= REL_TOL * np.abs(want)).all(), i
    with pytest.raises(imu.ImunpackError):                           # a NaN in one item is reported
        bad = a.clone()
        bad[1, 2, 3] = float("nan")
        imu.imunpack_gemm_batched(dev(bad), B_d, 95.0, 31.0, 63.0, b, strategies[0], strategies[1], ctx=ctx)
    ctx.destroy()


@pytest.mark.parametrize("b,strategies", [(8, (BOTH, BOTH)), (4, (ROW, COL)), (8, (COL, ROW))])
def test_batched_items_that_differ(imu, b, strategies):
    """The items of one batch share their launches but not their plans: items without heavy hitters beside items
    with many (an OB list that overflows its first capacity), with three and more digits, and with an accumulator
    bound that only the un-fused path can take; operands at odd offsets; each item against the oracle chain."""
    g = torch.Generator().manual_seed(900 + b)
    batch, n, d, h = 6, 70, 129, 65
    a = torch.randn((batch, n, d), generator=g)
    bt = torch.randn((batch, h, d), generator=g)
    a[1][torch.rand((n, d), generator=g) < 0.04] *= 200.0          # many heavy hitters
    a[2, :, 7] *= 3.0e4                                            # deep columns in both operands: large bounds
    bt[2, :, 7] *= 3.0e4
    a[3, 5, :] *= 500.0                                            # one heavy row
    bt[4][torch.rand((h, d), generator=g) < 0.002] *= 1.0e5        # a few entries of many digits
    ctx = imu.BatchContext()
    for _ in range(2):                                             # the second call on the grown buffers
        out = imu.imunpack_gemm_batched(dev(a), dev(bt), 95.0, 63.0, 63.0, b, strategies[0], strategies[1], ctx=ctx)
        got = out.cpu().numpy().astype(np.float64)
        for i in range(batch):
            want = _oracle_matmul(a[i].numpy(), bt[i].numpy(), 95.0, 63.0, 63.0)
            assert (np.abs(got[i] - want) <= REL_TOL * np.abs(want)).all(), i
    ctx.destroy()


@pytest.mark.parametrize("b,beta", [(8, 31.0), (4, 5.0)])
@pytest.mark.parametrize("n,d,h,kinds", [
    # levels of most rows and how many rows have one (of one level: two), of A and of B
    (1030, 70, 1027, [((1, 0), (1, 12)), ((2, 4), (2, 0)), ((4, 0), (1, 0)), ((2, 500), (1, 0)), ((1, 0), (4, 3)), ((3, 0), (2, 300))]),
    # rows so few that three levels take four physical rows as well
    (16, 40, 21, [((la, 0), (lb, 0)) for la in (1, 2, 3, 4) for lb in (1, 2, 3, 4)] * 9),
])
def test_batched_items_of_large_tiles_that_differ(imu, n, d, h, kinds, b, beta):
    """Batches of more than 128 tiles of 256 x 256 (up to which the small ones run): rows of one to four levels, evenly laid out
    or not, of several kinds, a few split rows of B and many, from item to item, int8 and six-bit digits.  Items against
    the oracle chain, and bit for bit what they give in a batch of their own."""
    s = 1 << (b - 1)
    g = torch.Generator().manual_seed(n + b)
    assert -(-n // 256) * -(-h // 256) * len(kinds) > 128
    a, bt = (torch.randn((len(kinds), rows, d), generator=g).clamp_(-2.5, 2.5) for rows in (n, h))
    for i, sides in enumerate(kinds):
        for x, (levels, few) in zip((a[i], bt[i]), sides):
            others = torch.randperm(x.shape[0], generator=g)
            deep, digits = (others[few:], levels) if levels > 1 else (others[:few], 2)
            if deep.numel():
                x[deep, torch.randint(0, d, (deep.numel(),), generator=g)] = 2.0 * 1.96 / (beta / 2) * s ** (digits - 1)
            q = oracle_quant(x, oracle.rtn_step(oracle.percentile_alpha(x.numpy(), 95.0), beta))
            top = np.abs(q.astype(np.int64)).max(1)
            own = 1 + sum((top >= s ** l).astype(int) for l in range(1, 6))
            assert (own[deep.numpy()] == digits).all() and (own == 1).sum() == x.shape[0] - deep.numel()
    out = imu.imunpack_gemm_batched(dev(a), dev(bt), 95.0, beta, beta, b, ROW, ROW, ctx=imu.BatchContext())
    for i in range(min(len(kinds), 32)):
        alone = imu.imunpack_gemm_batched(dev(a[i:i + 1]), dev(bt[i:i + 1]), 95.0, beta, beta, b, ROW, ROW, ctx=imu.BatchContext())
        assert torch.equal(out[i], alone[0]), i
        want = _oracle_matmul(a[i].numpy(), bt[i].numpy(), 95.0, beta, beta)
        assert (np.abs(out[i].cpu().numpy().astype(np.float64) - want) <= REL_TOL * np.abs(want)).all(), i


def test_batched_more_items_than_one_group(imu):
    """A batch of more items than share one set of launches, of the smallest shapes."""
    g = torch.Generator().manual_seed(31)
    batch, n, d, h = 1030, 3, 8, 2
    a, bt = torch.randn((batch, n, d), generator=g), torch.randn((batch, h, d), generator=g)
    out = imu.imunpack_gemm_batched(dev(a), dev(bt), 95.0, 31.0, 31.0, 8, ROW, COL, ctx=imu.BatchContext()).cpu().numpy()
    for i in (0, 1, 511, 1023, 1024, 1029):
        want = _oracle_matmul(a[i].numpy(), bt[i].numpy(), 95.0, 31.0, 31.0)
        assert (np.abs(out[i] - want) <= REL_TOL * np.abs(want)).all(), i


def test_batched_memory_follows_what_an_item_takes(imu):
    """Items whose plans and unpacked operands are many times their operands (one row each, padded to a tile): they go
    through in groups that stay small, whatever their number."""
    g = torch.Generator().manual_seed(32)
    batch, n, d, h = 300, 1, 65536, 1
    a, bt = torch.randn((batch, n, d), generator=g), torch.randn((batch, h, d), generator=g)
    a[7, 0, 11] = 300.0
    a_d, bt_d, ctx = dev(a), dev(bt), imu.BatchContext()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    out = imu.imunpack_gemm_batched(a_d, bt_d, 95.0, 31.0, 31.0, 8, ROW, COL, ctx=ctx).cpu().numpy()
    # 2 GiB by the estimate, a quarter on top where a buffer grows, and the pinned and pooled rest
    assert before - torch.cuda.mem_get_info()[0] < 3 << 30
    for i in (0, 7, 150, 299):
        want = _oracle_matmul(a[i].numpy(), bt[i].numpy(), 95.0, 31.0, 31.0)
        assert (np.abs(out[i] - want) <= REL_TOL * np.abs(want)).all(), i


def test_batched_items_that_write_over_one_another(imu):
    """A chain (C_i is A_(i+1)), outputs all in one place, and outputs in the place of their own operands: as the items
    one by one, in order."""
    g = torch.Generator().manual_seed(33)
    batch, n, d = 3, 40, 64
    w = torch.randn((batch, d, d), generator=g).to("cuda")
    x = torch.randn((batch + 1, n, d), generator=g).to("cuda")

    def call(a, sa_b, c, sc_b, first, items, ctx):
        step = 4 * first
        code = imu._lib.imunpack_gemm_batched(a.data_ptr() + sa_b * step, sa_b, d, 1, w.data_ptr() + d * d * step, d * d, d, 1, items, n,
                                              d, d, 95.0, 31.0, 31.0, 8, ROW, COL, c + sc_b * step, sc_b, d, imu.C.byref(ctx._h),
                                              torch.cuda.current_stream().cuda_stream)
        assert code == imu.OK

    for where in ("chain", "one place", "own place"):
        got = []
        for one_by_one in (True, False):
            buf = x.clone()
            out = torch.zeros((n, d), device="cuda")
            c, sc_b = {"chain": (buf.data_ptr() + 4 * n * d, n * d), "one place": (out.data_ptr(), 0),
                       "own place": (buf.data_ptr(), n * d)}[where]
            ctx = imu.BatchContext()
            for i in range(batch) if one_by_one else (0,):
                call(buf, n * d, c, sc_b, i, 1 if one_by_one else batch, ctx)
            got.append((buf.cpu(), out.cpu()))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), where
        assert not torch.equal(got[0][0], x.cpu()) or where == "one place"


def _sampled_entries(total, count=4096):
    """The entries of a matrix that the percentile's sample looks at (a hash of the sample number)."""
    x = np.arange(count, dtype=np.uint64)
    m = np.uint64(0xffffffff)
    x = (x * np.uint64(0x9e3779b1) + np.uint64(0x7f4a7c15)) & m
    x = ((x ^ (x >> np.uint64(15))) * np.uint64(0x85ebca77)) & m
    x = ((x ^ (x >> np.uint64(13))) * np.uint64(0xc2b2ae3d)) & m
    x = x ^ (x >> np.uint64(16))
    return (x * np.uint64(total)) >> np.uint64(32)


@pytest.mark.parametrize("rows,cols", [(256, 192), (1, 49153), (257, 1031), (1024, 768)])
@pytest.mark.parametrize("kind", ["normal", "ties", "gap", "sparse", "misled", "wide"])
def test_percentile_windows(imu, rows, cols, kind):
    """Around the size where the selection leaves one workgroup, and what its window can meet: ties (values of eight
    significant bits), two far modes with the rank at the edge between them (the third pass), mostly zeros, a
    sample that shows something else than the matrix (the window misses), and magnitudes of every exponent, zero and
    infinity among them (windows of up to 2^31 values).  Contiguous, transposed and strided."""
    rng = np.random.default_rng(rows * 31 + cols)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    flat = x.reshape(-1)
    if kind == "ties":
        flat[:] = (flat.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    elif kind == "gap":
        flat[rng.random(flat.size) < 0.05] *= np.float32(1e12)
    elif kind == "sparse":
        flat[rng.random(flat.size) < 0.9995] = 0.0
    elif kind == "misled":
        flat[_sampled_entries(flat.size).astype(np.int64)] = np.float32(1e6)
    elif kind == "wide":
        flat[:] = (rng.integers(0, 1 << 32, flat.size, dtype=np.uint64).astype(np.uint32) & np.uint32(0xff7fffff)).view(np.float32)
        flat[rng.random(flat.size) < 0.4] = 0.0
        flat[rng.random(flat.size) < 0.001] = np.float32("inf")
    xt = torch.from_numpy(x)
    wide = torch.zeros((rows, cols + 4), device="cuda")
    wide[:, :cols] = xt.to("cuda")
    apart = torch.zeros((rows, 2 * cols + 1), device="cuda")
    apart[:, 0:2 * cols:2] = xt.to("cuda")
    for p in (0.01, 50.0, 95.0, 99.99, 100.0):
        want = oracle.percentile_alpha(x, p)
        for view in (xt.to("cuda"), xt.t().contiguous().to("cuda").t(), wide[:, :cols], apart[:, 0:2 * cols:2]):
            alpha, status = imu.imunpack_percentile(view, p)
            assert int(status.item()) == 0
            assert alpha.cpu().numpy()[0] == want, (p, tuple(view.stride()))
    x[rows // 2, cols // 3] = np.float32("nan")
    _, status = imu.imunpack_percentile(torch.from_numpy(x).to("cuda"), 95.0)
    assert int(status.item()) == 1


def test_percentile_of_nearly_four_billion_entries(imu):
    """Just below the 2^32 entries that the call takes, read one by one: three rows that overlap but for an entry."""
    cols = (2 ** 32 - 1) // 3 - 3
    x = torch.arange(cols + 2, dtype=torch.int32, device="cuda").remainder_(1000).to(torch.float32)
    view = torch.as_strided(x, (3, cols), (1, 1))
    alpha, status = imu.imunpack_percentile(view, 95.0)
    k = int(np.ceil(95.0 * 3 * cols / 100.0))
    upto = lambda i: i // 1000 * np.arange(1, 1001) + np.minimum(np.arange(1, 1001), i % 1000)   # entries <= 0 .. 999 of the first i
    counts = sum(upto(r + cols) - upto(r) for r in range(3))
    assert int(status.item()) == 0 and int(alpha.item()) == int(np.searchsorted(counts, k))


@pytest.mark.parametrize("b,strategies", [(8, (ROW, ROW)), (8, (COL, BOTH)), (4, (ROW, COL)), (3, (COL, ROW)), (8, (BOTH, BOTH))])
@pytest.mark.parametrize("n,d,h", [(1, 1, 1), (33, 127, 65), (64, 513, 64), (257, 640, 31), (300, 1500, 250), (2050, 130, 1990)])
def test_gemm_tiles_of_either_size(imu, n, d, h, b, strategies):
    """Around the edges of a 64 x 64 tile, with contractions of one k-tile to more than the waves of a workgroup share,
    several exponent groups inside one wave's share, and a product that the 256 x 256 tiles take although rows of B are
    laid out in chunks of 64 (some of its tiles unsplit but with gaps): both outputs, both digit formats."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n * 7 + d * 3 + h + b)

    def draw(rows, few):
        q = rng.integers(-(s - 1), s, size=(rows, d))
        if few:  # a few heavy hitters (UnpackBoth), all in the first rows
            for _ in range(min(40, rows * d // 3)):
                q[rng.integers(0, min(rows, 300)), rng.integers(0, d)] = rng.integers(-s * s * s, s * s * s)
        else:
            q[:, rng.integers(0, d, size=max(1, d // 40))] *= s
            q[: min(rows, 150)] *= rng.choice([1, 1, 1, s], size=(min(rows, 150), 1))
        return q.astype(np.int32)

    Aq, Bq = draw(n, strategies[0] == BOTH), draw(h, strategies[1] == BOTH)
    want = oracle.int_gemm(Aq, Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    for fp6 in ([False, True] if b <= 4 else [False]):
        plan = imu.imunpack_plan(Qa, Qb, b, *strategies)
        if fp6:
            plan.set_digits(imu.DIGITS_FP6)
        A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
        bw = plan.unpacked_bytes()[2]
        C_int = torch.full(want.shape, -1, dtype=torch.int64, device="cuda")
        C_fp = torch.full(want.shape, -1.0, device="cuda")
        ws = torch.empty(bw // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 0.5, 0.25, C_int, C_fp, ws, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), want)
        ref = want.astype(np.float64) * 0.125
        assert (np.abs(C_fp.cpu().numpy() - ref) <= REL_TOL * np.abs(ref)).all()


@pytest.mark.parametrize("b,levels,few,splits,blev,fp6", [
    (8, 1, 0, 0, 1, False),       # no row split, columns in place
    (8, 1, 0, 30, 2, False),      # ... a few split rows of B in every tile
    (8, 1, 40, 300, 2, False),    # rows of one and of two levels; more split columns in a tile than have strips
    (8, 2, 5, 30, 2, False),      # nearly every row has two levels: two physical rows each
    (8, 2, 900, 0, 1, False),     # too many have one: rows one behind the other, chunks of both kinds
    (8, 3, 10, 0, 1, False),      # three levels: four physical rows each would take more chunks
    (8, 4, 100, 30, 2, False),    # four levels, with split columns too high for binary64
    (8, 1, 0, 2885, 2, False), (8, 2, 2, 2890, 2, False), (8, 2, 1000, 2880, 2, False),  # the rows of B evenly laid out too
    (8, 4, 9, 2890, 2, False), (8, 1, 0, 2890, 3, False), (6, 2, 0, 2800, 4, False),
    (4, 4, 100, 30, 2, True), (4, 2, 3, 0, 1, True), (4, 3, 2900, 7, 2, True), (4, 6, 0, 3, 2, False),
    (4, 4, 0, 2890, 4, True), (4, 2, 1, 2888, 3, True), (4, 1, 0, 2890, 2, True), (4, 3, 1500, 2890, 5, True),
])
def test_results_of_the_large_tiles_for_every_number_of_levels(imu, b, levels, few, splits, blev, fp6):
    """The 256 x 256 tiles store from their registers where the source rows of a chunk have one, two or four levels each (and
    those of B few splits, or two or four each), and through LDS elsewhere.  Odd sizes: the last tile has chunks without rows,
    its columns end inside a quad.  The fp32 output has to be that of the call that also writes int64, bit for bit, and
    nothing around C may be touched."""
    n, d, h = 3003, 70, 2890
    s = 1 << (b - 1)
    rng = np.random.default_rng(b * 100 + levels * 10 + few)
    Aq = rng.integers(-(s - 1), s, size=(n, d)).astype(np.int32)
    Bq = rng.integers(-(s - 1), s, size=(h, d)).astype(np.int32)
    deep = np.setdiff1d(np.arange(n), rng.choice(n, few, replace=False)) if levels > 1 else rng.choice(n, few, replace=False)
    top = (s if levels > 1 else 1) if levels < 3 else s ** (levels - 1)
    Aq[deep, rng.integers(0, d, deep.size)] = max(top, s) + rng.integers(0, s, deep.size)
    if levels > 2:  # the few have a level less
        rest = np.setdiff1d(np.arange(n), deep)
        Aq[rest, 3] = s ** (levels - 2) + 1
    if splits:
        Bq[rng.choice(h, splits, replace=False), 5] = -3 * s ** (blev - 1) if blev > 1 else 0
    want = oracle.int_gemm(Aq, Bq)
    plan = imu.imunpack_plan(torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda(), b, ROW, ROW)
    if fp6:
        plan.set_digits(imu.DIGITS_FP6)
    A_ue, B_eu = imu.imunpack_unpack(plan, torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda())
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    C_both = torch.full((n, h), -1.0, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, C_int, C_both, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == 1 and np.array_equal(C_int.cpu().numpy(), want)
    around = torch.full((n * h + 2 * 4096,), -1.0, device="cuda")
    C = around[4096:-4096].view(n, h)
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None, fuse=True)
    assert torch.equal(C, C_both)
    assert bool((around[:4096] == -1).all()) and bool((around[-4096:] == -1).all())
    ref = oracle.dequantize(want, 0.013, 0.0021)
    assert (np.abs(C.cpu().numpy() - ref) <= REL_TOL * np.abs(ref)).all()


@pytest.mark.parametrize("n,d,h,b,sa,sb,kind", [
    (5, 8200, 7, 8, COL, COL, "every"),     # more column slots than one workgroup lays out
    (5, 6140, 7, 8, COL, COL, "every"),     # just as many as it does
    (9, 8192, 6, 4, COL, COL, "deep"),      # many pairs of levels
    (40, 600, 33, 2, COL, COL, "deep"),
    (20, 9000, 30, 2, COL, COL, "pairs"),   # few column slots, but more pairs of levels than LDS holds masks for
    (20, 4096, 30, 2, COL, COL, "pairs"),   # ... and just not too many
    (30, 4100, 20, 8, BOTH, BOTH, "deep"),
    (4097, 40, 9000, 8, ROW, ROW, "every"),  # rows shared by two and three workgroups
    (16385, 8, 18000, 4, ROW, COL, "deep"),  # more rows than registers and LDS hold
    (12300, 16, 4096, 3, BOTH, ROW, "few"),
])
def test_layouts_around_the_sizes_where_they_change(imu, n, d, h, b, sa, sb, kind):
    rng = np.random.default_rng(n + d + h)
    s = 1 << (b - 1)
    if kind == "every":
        Aq, Bq = (rng.integers(-(s * s - 1), s * s, size=(r, d)).astype(np.int32) for r in (n, h))
    elif kind == "deep":
        Aq, Bq = (rand_ints(rng, r, d, s, 0.3 if b != 8 else 0.002, 4 if b > 2 else 9) for r in (n, h))
    elif kind == "pairs":
        Aq, Bq = (rng.integers(-(s - 1), s, size=(r, d)).astype(np.int32) for r in (n, h))
        for M in (Aq, Bq):  # columns of one to eight levels
            cols = rng.permutation(d)[:24]
            M[3, cols] = s ** (np.arange(24) % 8)
    else:
        Aq, Bq = (rand_ints(rng, r, d, s, 0.001, 2) for r in (n, h))
    check_against_oracle(imu, Aq, Bq, b, sa, sb)


@pytest.mark.parametrize("n,d,h", [(1, 1, 1), (64, 65, 63), (197, 64, 197), (256, 256, 256), (257, 250, 130), (512, 400, 511), (300, 513, 200)])
@pytest.mark.parametrize("b,digits,share", [(8, 2, 0.02), (8, 3, 0.01), (5, 4, 0.004), (4, 3, 0.2), (2, 2, 0.5)])
def test_unpack_both_of_few_rows_and_columns(imu, n, d, h, b, digits, share):
    """Up to 256 and 512 rows and columns, and just beyond, in-bound but for a share of the entries, of up to three digits or more (four are
    left to the general greedy), spread evenly or crowded in a few rows and columns; columns of A that are split often enough for B_e to
    have more than 256, or 512.  One operand alone, and both in one launch."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + 3 * d + h + b + digits)

    def draw(rows):
        q = rng.integers(-(s - 1), s, size=(rows, d))
        crowd = np.outer(rng.random(rows) ** 4, rng.random(d) ** 4) * 12
        big = rng.random((rows, d)) < share * (crowd if rows % 2 else 1.0)
        q[big] = rng.choice([-1, 1], int(big.sum())) * (s ** (rng.integers(1, digits, int(big.sum()))) + rng.integers(0, s, int(big.sum())))
        return q.astype(np.int32)

    Aq, Bq = draw(n), draw(h)
    for sa, sb in ((BOTH, BOTH), (BOTH, COL), (COL, BOTH)):
        check_against_oracle(imu, Aq, Bq, b, sa, sb)
    # both in one launch, from lists of the caller: room for every entry; too little for A's, for B's (planned from scans then)
    for lists in ((n * d, h * d), (7, h * d), (n * d, 7)):
        check_against_oracle(imu, Aq, Bq, b, BOTH, BOTH, lists=lists)


@pytest.mark.parametrize("deep_a,deep_b", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("b,digits,share", [(2, 9, 0.3), (8, 3, 0.3), (4, 5, 0.12)])
def test_sets_that_outgrow_their_room_in_one_launch(imu, b, digits, share, deep_a, deep_b):
    """UnpackBoth on both operands of at most 256 rows and columns, from lists: rows, columns and edges of the first operand, of the second
    or of both are more than a plan has room for at first."""
    rng = np.random.default_rng(b + 2 * deep_a + deep_b)
    s = 1 << (b - 1)
    n, d, h = 256, 255, 250
    Aq, Bq = (_wide_ints(rng, rows, d, s, digits, share) if deep else rng.integers(-(s - 1), s, size=(rows, d)).astype(np.int32)
              for rows, deep in ((n, deep_a), (h, deep_b)))
    check_against_oracle(imu, Aq, Bq, b, BOTH, BOTH, lists=(n * d, h * d))


def _wide_ints(rng, rows, d, s, digits, share):
    """In-Bound integers but for a share of 2 to `digits` digits."""
    q = rng.integers(-(s - 1), s, size=(rows, d))
    big = rng.random((rows, d)) < share
    q[big] = rng.choice([-1, 1], int(big.sum())) * (s ** (rng.integers(1, digits, int(big.sum()))) + rng.integers(0, s, int(big.sum())))
    return q.astype(np.int32)


@pytest.mark.parametrize("n,d,h", [(256, 256, 255), (197, 64, 256), (255, 197, 64)])
@pytest.mark.parametrize("b", [8, 5])
def test_batched_unpack_both_whose_items_differ_in_digits(imu, n, d, h, b):
    """A batch whose items hold no heavy hitters, some of two and of three digits (in B_e of up to 256 columns and of more) and of four or
    more, in either operand or in both: each against the oracle chain, and bit for bit what it gives alone."""
    g = torch.Generator().manual_seed(n + d + b)
    s = float(1 << (b - 1))
    # digits of the longest entries of A, of B (at b = 8 no weight may exceed 62 bits: eight digits above the first in all)
    kinds = [(0, 0), (2, 2), (3, 0), (0, 3), (3, 3), (4, 0), (2, 4), (0, 5)]
    a, bt = (torch.randn((len(kinds), rows, d), generator=g).clamp_(-2.5, 2.5) for rows in (n, h))
    for i, digits in enumerate(kinds):
        for x, k in zip((a[i], bt[i]), digits):
            if k:
                big = torch.rand(x.shape, generator=g) < 0.01
                x[big] = 6.0 * 1.96 / s * s ** torch.randint(1, k, (int(big.sum()),), generator=g).float()   # 1.5 s^1 to 1.5 s^(k - 1)
    out = imu.imunpack_gemm_batched(dev(a), dev(bt), 95.0, s / 2, s / 2, b, BOTH, BOTH, ctx=imu.BatchContext())
    for i, digits in enumerate(kinds):
        for x, k in zip((a[i], bt[i]), digits):
            top = np.abs(oracle_quant(x, oracle.rtn_step(oracle.percentile_alpha(x.numpy(), 95.0), s / 2)).astype(np.int64)).max()
            assert s ** max(k - 1, 0) <= top < s ** max(k, 1)
        alone = imu.imunpack_gemm_batched(dev(a[i:i + 1]), dev(bt[i:i + 1]), 95.0, s / 2, s / 2, b, BOTH, BOTH, ctx=imu.BatchContext())
        assert torch.equal(out[i], alone[0]), i
        want = _oracle_matmul(a[i].numpy(), bt[i].numpy(), 95.0, s / 2, s / 2)
        assert (np.abs(out[i].cpu().numpy().astype(np.float64) - want) <= REL_TOL * np.abs(want)).all(), i


def _listed(imu, M, b, cap=None):
    """Integers on the device with their statistics and list of heavy hitters, as the quantizer hands them over."""
    X = dev(torch.from_numpy(M)).float()
    stats = imu.Stats.empty(*M.shape, X.device, cap or imu.Stats.default_ob_cap(*M.shape))
    Q, _, status = imu.imunpack_quantize(X, 1.0, b, stats=stats)
    assert int(status.item()) == 0 and np.array_equal(Q.cpu().numpy(), M)
    return Q, stats


@pytest.mark.parametrize("large", [(17000, 700, 32), (32, 700, 17000), (40, 17000, 24)])
def test_small_products_on_a_plan_that_has_held_a_large_one(imu, large):
    """UnpackBoth on both operands, a plan object whose rows of A, rows of B or columns once were so many that the greedy's counts of
    as many do not fit LDS (capacities only grow): small products are planned as by a plan of their own."""
    rng = np.random.default_rng(large[0])
    plan = imu.Plan()
    for n, d, h in (large, (256, 256, 256), (197, 64, 197), large, (1, 3, 2), (300, 280, 310)):
        Aq, Bq = (rand_ints(rng, r, d, 128, 0.001 if n * d > 1 << 20 or h * d > 1 << 20 else 0.01, 2) for r in (n, h))
        (Qa, st_a), (Qb, st_b) = _listed(imu, Aq, 8), _listed(imu, Bq, 8)
        imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH, st_a, st_b, plan)
        hnd = oracle.unpack_pair_handle(Aq, Bq, 8, BOTH, BOTH)
        assert plan.dims()[:3] == (hnd.n_u, hnd.d_u, hnd.h_u)
        A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
        if max(n, d, h) <= 310:
            Ac, Bc = imu.imunpack_unpack_canonical(plan, A_ue, B_eu)
            oa, ob = hnd.operands_i8()
            assert np.array_equal(Ac.cpu().numpy(), oa) and np.array_equal(Bc.cpu().numpy(), ob)
        hnd.close()
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, ws, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), oracle.int_gemm(Aq, Bq))


def test_attention_on_a_context_that_has_served_a_large_layer(imu):
    """The three products of a layer's training step over many tokens, then an attention's, UnpackBoth throughout: one context, the
    outputs of the small products bit for bit those of a context of their own and within tolerance of the oracle chain."""
    g = torch.Generator().manual_seed(61)
    tokens, d, h = 17000, 700, 32
    x, w, gy = (torch.randn(shape, generator=g) for shape in ((tokens, d), (h, d), (tokens, h)))
    x[:, 5] *= 30.0
    w[torch.rand(w.shape, generator=g) < 0.001] *= 20.0
    q, k = (torch.randn((6, 197, 64), generator=g) for _ in range(2))
    k[..., 5] *= 12.0
    p = torch.softmax(torch.randn((6, 197, 197), generator=g) * 3, -1)
    v = torch.randn((6, 64, 197), generator=g)
    ctx = imu.BatchContext()
    for A, B in ((x, w), (gy, w.t()), (gy.t(), x.t()), (q, k), (p, v), (x, w), (q, k)):
        got = imu.imunpack_gemm_batched(dev(A), dev(B), 95.0, 31.0, 31.0, 8, BOTH, BOTH, ctx=ctx)
        assert torch.equal(got, imu.imunpack_gemm_batched(dev(A), dev(B), 95.0, 31.0, 31.0, 8, BOTH, BOTH, ctx=imu.BatchContext()))
        for a_i, b_i, got_i in ((A, B, got),) if A.dim() == 2 else ((A[i], B[i], got[i]) for i in (0, 5)):
            want = _oracle_matmul(a_i.contiguous().numpy(), b_i.contiguous().numpy(), 95.0, 31.0, 31.0)
            assert (np.abs(got_i.cpu().numpy().astype(np.float64) - want) <= REL_TOL * np.abs(want)).all()
    ctx.destroy()


@pytest.mark.parametrize("b,depth", [(6, 3), (8, 2), (2, 5)])
def test_columns_that_outgrow_their_room_before_an_unpack_both(imu, b, depth):
    """UnpackColumn on A appends more columns than the plan has room for at first, UnpackBoth on B follows the links from a
    column to its copies before the plan is made again; in an arena that other plans have written all over."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(b)
    plan = imu.Plan()
    for n, d, h in ((900, 300, 800), (40, 460, 39)):
        Aq, Bq = (rand_ints(rng, r, d, s, 0.01, 2) for r in (n, h))
        big = d == 460
        if big:
            Aq[3] = s ** depth * rng.choice([-1, 1], d)         # every column has depth + 1 levels
        Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
        sa = COL if big else BOTH
        imu.imunpack_plan(Qa, Qb, b, sa, BOTH, plan=plan)
        hnd = oracle.unpack_pair_handle(Aq, Bq, b, sa, BOTH)
        assert plan.dims()[:3] == (hnd.n_u, hnd.d_u, hnd.h_u)
        if big:
            assert plan.dims()[1] > 2 * d + 256                 # more than the first guess
        hnd.close()
        A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, ws, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), oracle.int_gemm(Aq, Bq))


@pytest.mark.parametrize("n,d,h,tiles_b,parts", [(2000, 600, 2000, 24, 1), (300, 600, 300, 4, 0)])
def test_rows_of_b_are_laid_out_for_the_tiles_that_run(imu, n, d, h, tiles_b, parts):
    """Three digit levels in every row of both operands: 6000 unpacked rows of B fill 24 tiles of 256 (25 if no row may
    straddle 64), which the large tiles take; 900 rows go to the small ones."""
    rng = np.random.default_rng(n)
    Aq, Bq = (rng.integers(-127, 128, size=(r, d)).astype(np.int32) for r in (n, h))
    Aq[np.arange(n), rng.integers(0, d, n)] = 128 * 128 + 5
    Bq[np.arange(h), rng.integers(0, d, h)] = -128 * 128 - 7
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, ROW, ROW)
    assert plan.layout()[1][0] == tiles_b * 256
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == parts
    assert np.array_equal(C_int.cpu().numpy(), oracle.int_gemm(Aq, Bq))


def _product_in_parts(n, d, h, b, strategies, every):
    """Operands of a product with a long contraction: `every` splits each column of A (two exponent groups of the same
    width), else a few columns and, under UnpackRow, most rows."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + d + h)
    Aq = rng.integers(-(s - 1), s, size=(n, d)).astype(np.int32)
    Bq = rng.integers(-(s - 1), s, size=(h, d)).astype(np.int32)
    if every:
        Aq[n // 2] = s
    else:
        Aq[:, rng.integers(0, d, 9)] *= s
        if strategies[0] == ROW:
            Aq[rng.random(n) < 0.7] *= s
        if strategies[1] == COL:
            Bq[:, rng.integers(0, d, d // 40)] *= s
    return Aq, Bq


@pytest.mark.parametrize("n,d,h,b,strategies,every,parts", [
    (1000, 6100, 2500, 8, (ROW, COL), False, 2),    # fewer tiles than CUs; groups that end inside a part
    (2560, 3072, 2560, 8, (COL, COL), True, 2),     # a group that ends where a part does
    (2200, 3072, 2000, 8, (COL, ROW), True, 3),     # ... and inside a part
    (2048, 6400, 2048, 4, (COL, COL), False, 4),    # six-bit digits, groups inside parts
    (2048, 3072, 2048, 4, (COL, COL), True, 4),     # six-bit digits, a group that ends where a part does
    (4352, 6144, 4352, 8, (BOTH, COL), False, 4),   # a round of whole tiles before
    (2560, 5900, 2560, 8, (ROW, ROW), False, 1),    # a contraction that is too short for it
    (300, 8200, 600, 8, (COL, COL), False, 0),      # few tiles
])
def test_gemm_whose_last_round_is_cut_along_the_contraction(imu, n, d, h, b, strategies, every, parts):
    """Products whose last round of tiles would leave CUs idle: tiles in two to four parts, exponent groups that end
    inside a part and at its end, launches in a row on two streams.  Rows from every band of tiles against the oracle."""
    Aq, Bq = _product_in_parts(n, d, h, b, strategies, every)
    rows = np.unique(np.concatenate([np.arange(0, n, 61), np.arange(0, n, 256), [n // 2, n - 1]]))
    want = oracle.int_gemm(Aq[rows], Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, b, *strategies)
    if b <= 4:
        plan.set_digits(imu.DIGITS_FP6)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    assert plan.fusable()
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    outs = [torch.full((n, h), -1, dtype=torch.int64, device="cuda") for _ in range(4)]
    streams[1].wait_stream(streams[0])
    for i, C_int in enumerate(outs):
        with torch.cuda.stream(streams[i % 2]):
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
            assert imu.imunpack_diag_gemm_parts(plan) == parts
    torch.cuda.synchronize()
    for C_int in outs:
        assert np.array_equal(C_int[torch.from_numpy(rows).cuda()].cpu().numpy(), want)
        assert torch.equal(C_int, outs[0])


def _rows_of_levels(rng, rows, d, s, levels, few):
    """In-Bound integers, one entry of `levels` digits in every row but in `few`, which have a digit less (levels == 1: more)."""
    M = rng.integers(-(s - 1), s, size=(rows, d)).astype(np.int32)
    others = rng.choice(rows, few, replace=False)
    own = np.full(rows, levels)
    own[others] = levels - 1 if levels > 1 else 2
    deep = np.flatnonzero(own > 1)
    M[deep, rng.integers(0, d, deep.size)] = s ** (own[deep] - 1) + rng.integers(0, s, deep.size)
    return M


@pytest.mark.parametrize("n,d,h,b,lev_a,few_a,lev_b,few_b,every", [
    (2001, 7000, 2000, 8, 1, 0, 1, 0, False),     # nothing split
    (2001, 7000, 2000, 8, 1, 0, 1, 30, False),    # a few split rows of B in every tile
    (1001, 7000, 2003, 8, 2, 3, 1, 0, False),     # rows of A of two levels, evenly laid out
    (501, 7000, 2003, 8, 4, 9, 1, 0, False),      # ... of four and a few of three
    (1500, 7000, 2003, 8, 1, 500, 1, 0, False),   # chunks of rows of one and of two levels
    (2003, 7000, 1001, 8, 1, 0, 2, 0, False),     # rows of B of two levels, evenly laid out
    (2003, 7000, 1001, 8, 1, 0, 4, 2, False),     # ... of four
    (1003, 7000, 1001, 8, 2, 0, 2, 1, False),     # ... on either side
    (2001, 3500, 2000, 8, 1, 0, 1, 0, True),      # two exponent groups of one width: a part ends before the last group
    (2001, 3500, 1001, 8, 1, 0, 2, 0, True),
    (2001, 12000, 2000, 4, 1, 0, 1, 0, False),    # six-bit digits
    (2001, 12000, 2000, 4, 1, 0, 1, 30, False),
    (501, 12000, 2003, 4, 4, 9, 1, 0, False),
    (1003, 12000, 1001, 4, 2, 0, 2, 1, False),
    (2003, 12000, 1001, 4, 1, 0, 4, 2, False),
    (2001, 6000, 1001, 4, 1, 0, 2, 0, True),
])
def test_fp32_results_of_tiles_in_parts(imu, n, d, h, b, lev_a, few_a, lev_b, few_b, every):
    """The last part of a tile adds the sums of the others and stores fp32 results from its registers where the levels of the
    tile's rows allow it: rows of one, two and four levels on either side, split columns, both digit formats, parts that end
    before the last exponent group.  Bit for bit what the call gives that also writes int64 (through LDS); nothing
    around C is touched."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + d + h + b + few_b)
    Aq, Bq = _rows_of_levels(rng, n, d, s, lev_a, few_a), _rows_of_levels(rng, h, d, s, lev_b, few_b)
    if every:
        Aq[n // 2] = s
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, b, COL if every else ROW, ROW)
    if b <= 4:
        plan.set_digits(imu.DIGITS_FP6)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    assert plan.fusable()
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    C_both = torch.full((n, h), -1.0, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, C_int, C_both, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) > 1
    around = torch.full((n * h + 2 * 4096,), -1.0, device="cuda")
    C = around[4096:-4096].view(n, h)
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) > 1
    assert torch.equal(C, C_both)
    assert bool((around[:4096] == -1).all()) and bool((around[-4096:] == -1).all())
    rows = np.unique(np.concatenate([np.arange(0, n, 61), [n // 2, n - 1]]))
    want = oracle.int_gemm(Aq[rows], Bq)
    assert np.array_equal(C_int[torch.from_numpy(rows).cuda()].cpu().numpy(), want)
    ref = oracle.dequantize(want, 0.013, 0.0021)
    assert (np.abs(C[torch.from_numpy(rows).cuda()].cpu().numpy() - ref) <= REL_TOL * np.abs(ref)).all()


def test_products_in_parts_from_two_threads(imu):
    """A plan handed from one thread to another, each with its own per-thread default stream (one handle for both): the
    launches share the buffer that the parts meet in and must not overlap."""
    import threading
    n, d, h = 2560, 3072, 2560
    Aq, Bq = _product_in_parts(n, d, h, 8, (COL, COL), True)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, COL, COL)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    assert plan.fusable()
    outs = [torch.full((n, h), -1, dtype=torch.int64, device="cuda") for _ in range(6)]
    torch.cuda.synchronize()
    per_thread = 2  # hipStreamPerThread
    turn, done, codes = [threading.Event() for _ in range(7)], threading.Event(), []

    def work(me):
        torch.cuda.set_device(0)
        for i in range(me, 6, 2):
            turn[i].wait()
            codes.append(imu._lib.imunpack_gemm(plan.handle, A_ue.data_ptr(), B_eu.data_ptr(), None, outs[i].data_ptr(), None, h,
                                                1.0, 1.0, 1, per_thread))
            turn[i + 1].set()
        done.wait()  # neither stream ends before the other thread has launched

    threads = [threading.Thread(target=work, args=(me,)) for me in (0, 1)]
    for t in threads:
        t.start()
    turn[0].set()
    turn[6].wait()
    done.set()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert codes == [0] * 6 and imu.imunpack_diag_gemm_parts(plan) == 2
    rows = np.arange(0, n, 97)
    want = oracle.int_gemm(Aq[rows], Bq)
    for C_int in outs:
        assert np.array_equal(C_int[torch.from_numpy(rows).cuda()].cpu().numpy(), want)
        assert torch.equal(C_int, outs[0])


def _long_work(ms=20):
    """Queues some milliseconds of library work on the current stream."""
    x = torch.ones((4096, 4096), device="cuda")
    for _ in range(ms):
        x = torch.mm(x, x)


def _deep_in_both(rng, n, d, h, s, deep):
    """Integers for UnpackColumn on both sides; `deep`: a column of four-digit entries in both operands, whose shifted
    sum leaves int32."""
    Aq, Bq = (rng.integers(-(s - 1), s, size=(r, d)).astype(np.int32) for r in (n, h))
    if deep:
        Aq[:, 7] = Bq[:, 7] = (s - 1) * s ** 3
    return Aq, Bq


def test_gemm_on_another_stream_than_the_unpack(imu):
    """Plan and unpack on one stream, other work and then the GEMM on a second one that waits for an event of the
    first, nothing asked in between: the accumulator bounds arrive whatever the second stream is busy with.  First
    operands that the fused launch takes, then (on the same plan object, which expects the same again) operands that it
    must refuse: without a workspace on every try, with one exactly."""
    b, s = 8, 128
    n, d, h = 300, 520, 260
    rng = np.random.default_rng(5)
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    plan = imu.Plan()
    for deep in (False, True, False):
        Aq, Bq = _deep_in_both(rng, n, d, h, s, deep)
        want = oracle.int_gemm(Aq, Bq)
        Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(first):
            imu.imunpack_plan(Qa, Qb, b, COL, COL, plan=plan)
            A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
            unpacked = torch.cuda.Event()
            unpacked.record()
        with torch.cuda.stream(second):
            second.wait_event(unpacked)
            _long_work()
            if deep:
                for _ in range(2):
                    with pytest.raises(imu.ImunpackError) as e:
                        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
                    assert e.value.code == imu.ERANGE
                second.synchronize()
                assert int((C_int != -1).sum().item()) == 0
                assert not plan.fusable() and min(plan.bounds()) * (s - 1) >= 2 ** 31
            ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda") if deep else None
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, ws, fuse=True)
        second.synchronize()
        assert np.array_equal(C_int.cpu().numpy(), want)
        assert plan.fusable() == (not deep)


def test_bounds_do_not_need_the_stream_of_the_unpack(imu):
    """The bounds of an unpack on a stream that the caller has destroyed since, and of an unpack that ran in a graph."""
    import ctypes
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    rng = np.random.default_rng(6)
    Aq, Bq = (rand_ints(rng, r, 400, 128, 0.003, 2) for r in (130, 200))
    want = oracle.int_gemm(Aq, Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    bounds = plan.bounds()
    torch.cuda.synchronize()
    handle = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0
    with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
        imu.imunpack_unpack(plan, Qa, Qb, A_ue, B_eu)
    assert hip.hipStreamSynchronize(handle) == 0 and hip.hipStreamDestroy(handle) == 0
    assert plan.bounds() == bounds
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        imu.imunpack_unpack(plan, Qa, Qb, A_ue, B_eu)
    for _ in range(3):
        A_ue.zero_()
        graph.replay()
        C_int = torch.full(want.shape, -1, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        assert plan.bounds() == bounds
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None, fuse=True)
        assert np.array_equal(C_int.cpu().numpy(), want)


@pytest.mark.parametrize("n,d,h,sa,longer,parts", [
    (20, 1700, 8200, ROW, 0.0, 0),         # 64 x 64 tiles, one half of a row block; the full columns are stored beside the lists
    (150, 1670, 8265, COL, 0.00002, 0),    # ... columns of exponents 1 and 2 beside them, entries of three digits
    (2000, 1660, 8200, ROW, 0.0, 1),       # 256 x 256 tiles
    (3300, 1700, 8000, COL, 0.00002, 1),
    (400, 5800, 8000, COL, 0.0, 2),        # ... cut along the contraction (2: in two parts or more), the lists in one of them
])
def test_appended_columns_of_few_digits(imu, n, d, h, sa, longer, parts):
    """UnpackBoth appends a column for nearly every original one, each for a few heavy hitters: the fused GEMM takes their digits from
    lists, the un-fused one from B_eu.  Some columns are full of heavy hitters and are multiplied as columns."""
    g = torch.Generator(device="cuda").manual_seed(n + d)
    A = torch.randint(-127, 128, (n, d), generator=g, device="cuda", dtype=torch.int32)
    B = torch.randint(-127, 128, (h, d), generator=g, device="cuda", dtype=torch.int32)
    A[:, ::97] += 3000
    sign = torch.randint(0, 2, (h, d), generator=g, device="cuda", dtype=torch.int32) * 2 - 1
    for share, lo, hi in (((4 if d > 5000 else 8) / h, 128, 128 ** 2), (longer, 128 ** 2, 128 ** 3)):
        at = torch.rand((h, d), generator=g, device="cuda") < share
        B = torch.where(at, sign * torch.randint(lo, hi, (h, d), generator=g, device="cuda", dtype=torch.int32), B)
    B[:, 5::211] += 200
    want = A.double() @ B.double().t()      # exact: below 2^53
    plan = imu.imunpack_plan(A, B, 8, sa, BOTH)
    plan.keep_weights()                     # (products of this size have lists where the weights stay resident)
    for rows in (n, max(1, n - 3)):         # the plan object again, its buffers reused
        imu.imunpack_plan(A[:rows], B, 8, sa, BOTH, plan=plan)
        assert imu.imunpack_diag_list_columns(plan) > d // 2
        A_ue, B_eu = imu.imunpack_unpack(plan, A[:rows], B)
        for again in range(2):              # a second unpack of the plan leaves the lists as they are
            C = torch.full((rows, h), 3.5, device="cuda")
            C_int = torch.full((rows, h), -1, dtype=torch.int64, device="cuda")
            imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None)
            assert min(imu.imunpack_diag_gemm_parts(plan), 2) == parts
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
            scale = float(np.float32(0.013)) * float(np.float32(0.0021))
            assert torch.equal(C_int.double(), want[:rows]) and torch.equal(C, (want[:rows] * scale).float())
            imu.imunpack_unpack(plan, A[:rows], B, A_ue, B_eu)
    ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, None, None, ws, fuse=False)
    imu.imunpack_recombine(plan, ws, 1.0, 1.0, C_int, None)
    assert torch.equal(C_int.double(), want[:rows])


@pytest.mark.parametrize("n,d,h,b,levels,few,splits,blev,halves", [
    (257, 128, 8200, 8, 1, 0, 0, 1, True),         # a single k-tile; the second half of a tile of rows is padding
    # two k-tiles, rows of one and two levels, split columns (12100 rows of B, 48 tiles, are for the small tiles: 19.5 us, 25.8 in half tiles)
    (130, 129, 24100, 8, 1, 9, 40, 2, True),
    (4127, 380, 2049, 8, 2, 3, 0, 1, True),        # three k-tiles, more half tiles than two to a CU
    (1000, 1300, 8193, 5, 4, 11, 8180, 2, True),   # four levels a row, columns evenly laid out
    (1000, 1300, 2100, 5, 2, 11, 2095, 3, True),   # ... in four levels
    (3003, 7700, 2890, 8, 1, 0, 0, 1, False),      # whole tiles: 61 k-tiles
    (3003, 7700, 2890, 8, 1, 30, 25, 2, False),
    (1502, 7700, 2890, 8, 2, 3, 0, 1, False),
    (1502, 7700, 1440, 8, 2, 3, 1438, 2, False),
])
def test_half_tiles_and_whole_ones(imu, n, d, h, b, levels, few, splits, blev, halves):
    """Tiles of 128 x 256, which most products take, and of 256 x 256, for long contractions: fp32 results, from registers or
    through LDS, are those of the call that also writes int64, bit for bit, and nothing around C is touched; a product
    whose sums might leave int32 is refused by the launch that has already begun to load it."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + d + h + levels)
    Aq, Bq = _rows_of_levels(rng, n, d, s, levels, few), rng.integers(-(s - 1), s, size=(h, d)).astype(np.int32)
    if splits:
        Bq[rng.choice(h, splits, replace=False), 5] = -3 * s ** (blev - 1)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, b, ROW, ROW)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    C_both = torch.full((n, h), -1.0, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, C_int, C_both, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == 1 and imu.imunpack_diag_gemm_halves(plan) == int(halves)
    around = torch.full((n * h + 2 * 4096,), -1.0, device="cuda")
    C = around[4096:-4096].view(n, h)
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None, fuse=True)
    assert torch.equal(C, C_both)
    assert bool((around[:4096] == -1).all()) and bool((around[-4096:] == -1).all())
    rows = np.unique(np.concatenate([np.arange(0, n, 61), [n // 2, n - 1]]))
    assert np.array_equal(C_int[torch.from_numpy(rows).cuda()].cpu().numpy(), oracle.int_gemm(Aq[rows], Bq))


@pytest.mark.parametrize("n,d,h,b,lev_a,few_a,lev_b,few_b,parts,halves", [
    (338, 64, 481, 5, 3, 60, 5, 0, 0, 0),       # one k-tile, results through LDS in half tiles: small tiles
    (148, 76, 1919, 5, 1, 60, 4, 0, 0, 0),
    (173, 149, 3036, 3, 3, 60, 2, 7, 0, 0),     # the same where rows of B have two levels each
    (130, 129, 12100, 8, 1, 9, 1, 40, 0, 0),    # a few rows of two levels on either side
    (1576, 800, 3072, 8, 1, 0, 1, 0, 1, 1),     # 84 tiles without levels: half tiles
    (776, 97, 972, 6, 3, 0, 3, 0, 1, 1),        # 120 with three levels a row on both sides: four rounds of small tiles
])
def test_small_tiles_and_half_tiles_of_few_large_ones(imu, n, d, h, b, lev_a, few_a, lev_b, few_b, parts, halves):
    """At most 128 tiles, by levels of either side: which kernel runs, and its results."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + d + h)
    Aq, Bq = _rows_of_levels(rng, n, d, s, lev_a, few_a), _rows_of_levels(rng, h, d, s, lev_b, few_b)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, b, ROW, ROW)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C_int, C = torch.full((n, h), -1, dtype=torch.int64, device="cuda"), torch.full((n, h), -1.0, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == parts and imu.imunpack_diag_gemm_halves(plan) == halves
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, C_int, None, None, fuse=True)
    want = oracle.int_gemm(Aq, Bq)
    assert np.array_equal(C_int.cpu().numpy(), want)
    ref = oracle.dequantize(want, 0.013, 0.0021)
    assert (np.abs(C.cpu().numpy().astype(np.float64) - ref) <= REL_TOL * np.abs(ref)).all()


@pytest.mark.parametrize("n,d,h,b,levels,few,blev,halves", [
    (1500, 130, 1499, 3, 1, 0, 4, 0),     # four levels of every row of B, two k-tiles: folded in the registers of whole tiles
    (700, 300, 1500, 3, 2, 0, 4, 0),      # ... and two of every row of A
    (400, 300, 1500, 3, 4, 3, 4, 0),      # ... and four, but three rows with three
    (1500, 300, 1500, 3, 1, 9, 4, 1),     # rows of A of one and two levels in a chunk go through LDS
    (700, 300, 1500, 3, 3, 0, 4, 1),      # so do three levels
    (700, 300, 1500, 8, 2, 0, 4, 1),      # sums that binary64 does not hold
    (1000, 3072, 2000, 3, 1, 0, 4, 0),    # 128 tiles, 24 k-tiles
    (1000, 3073, 2000, 3, 1, 0, 4, 1),    # ... 25
    (3000, 5889, 3000, 3, 1, 0, 4, 0),    # a little more than two rounds, 47 k-tiles
])
def test_four_levels_of_every_column_fold_in_whole_tiles(imu, n, d, h, b, levels, few, blev, halves):
    """Rows of B of four levels each: in whole tiles a lane has them all, half tiles take them through LDS; either way the fp32
    results are those of the call that also writes int64, bit for bit, which is the oracle's."""
    s = 1 << (b - 1)
    rng = np.random.default_rng(n + d + h + levels)
    Aq, Bq = _rows_of_levels(rng, n, d, s, levels, few), _rows_of_levels(rng, h, d, s, blev, 0)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, b, ROW, ROW)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    C_both, C = (torch.full((n, h), -1.0, device="cuda") for _ in range(2))
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, C_int, C_both, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == 1 and imu.imunpack_diag_gemm_halves(plan) == 1
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None, fuse=True)
    assert imu.imunpack_diag_gemm_parts(plan) == 1 and imu.imunpack_diag_gemm_halves(plan) == halves
    assert torch.equal(C, C_both)
    rows = np.unique(np.concatenate([np.arange(0, n, 61), [n // 2, n - 1]]))
    assert np.array_equal(C_int[torch.from_numpy(rows).cuda()].cpu().numpy(), oracle.int_gemm(Aq[rows], Bq))


def test_half_tiles_refuse_what_may_overflow(imu):
    """The fused launch goes out before the host knows the bounds: a second unpack of larger integers than the first had."""
    n, d, h = 300, 400, 8200
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randint(-127, 128, (n, d), generator=g, device="cuda", dtype=torch.int32)
    B = torch.randint(-127, 128, (h, d), generator=g, device="cuda", dtype=torch.int32)
    plan = imu.Plan()
    for top in (1, 128 ** 3):
        A[:, 7] = 5 * top
        B[:, 7] = 9 * top
        imu.imunpack_plan(A, B, 8, COL, COL, plan=plan)
        A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
        C = torch.full((n, h), -1.0, device="cuda")
        if top == 1:
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, None, C, None, fuse=True)
            assert imu.imunpack_diag_gemm_halves(plan) == 1
        else:
            with pytest.raises(imu.ImunpackError):
                imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, None, C, None, fuse=True)
            assert bool((C == -1).all())
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, None, C, torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda"), fuse=True)
        want = A.double() @ B.double().t()      # exact: below 2^53
        assert torch.equal(C, want.float())


def _few_digits(rng, n, d, h, deep, deep_cols=24):
    """In-Bound integers but for four entries of two digits in every column of B and, if `deep`, five of three in some of
    them, no two of those in one row; a few rows of A have two levels."""
    A = rng.integers(-127, 128, (n, d)).astype(np.int32)
    B = rng.integers(-127, 128, (h, d)).astype(np.int32)
    A[::7, rng.integers(0, d)] = 3000
    for k in range(d):
        B[rng.choice(h, 4, replace=False), k] = rng.integers(128, 128 ** 2, 4) * rng.choice([-1, 1], 4)
    if deep:
        cols = np.arange(deep_cols) * (d // deep_cols)
        at = rng.choice(h, (deep_cols, 5), replace=False)
        B[at, cols[:, None]] = rng.integers(128 ** 2, 128 ** 3, at.shape) * rng.choice([-1, 1], at.shape)
    return torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()


def _plan_of_resident_weights(imu, A, B, sa):
    """The first plan in keep-weights mode, where products of any number of rows have lists."""
    plan = imu.imunpack_plan(A, B, 8, sa, BOTH)
    plan.keep_weights()
    return imu.imunpack_plan(A, B, 8, sa, BOTH, plan=plan)


@pytest.mark.parametrize("n,d,h,deep,parts", [
    (20, 1700, 6400, False, 0),    # 64 x 64 tiles: a single exponent group beside the lists
    (20, 1700, 6400, True, 0),     # ... columns of exponent 2 before them
    (150, 1670, 6465, True, 0),
    (2000, 1660, 6400, False, 1),  # 256 x 256 tiles
    (2000, 1660, 6400, True, 1),
    (400, 5800, 13000, True, 2),   # ... cut along the contraction (2: in two parts or more)
])
def test_no_stored_column_has_the_exponent_of_the_lists(imu, n, d, h, deep, parts):
    """Every column of exponent 1 is taken from lists: the shift from the groups above to the lowest one is that over two
    exponents, with the lists in between."""
    A, B = _few_digits(np.random.default_rng(n + d), n, d, h, deep, 200 if parts == 2 else 24)
    want = A.double() @ B.double().t()      # exact: below 2^53
    plan = _plan_of_resident_weights(imu, A, B, ROW)
    col_exp = plan.export()[5].numpy()
    assert int((col_exp == 1).sum()) == imu.imunpack_diag_list_columns(plan) > d // 2 and (int(col_exp.max()) == 2) == deep
    A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
    C = torch.full((n, h), 3.5, device="cuda")
    C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, 0.013, 0.0021, None, C, None)
    assert min(imu.imunpack_diag_gemm_parts(plan), 2) == parts
    imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
    scale = float(np.float32(0.013)) * float(np.float32(0.0021))
    assert torch.equal(C_int.double(), want) and torch.equal(C, (want * scale).float())


@pytest.mark.parametrize("n,d,h,deep", [(20, 1700, 6400, True), (2000, 1660, 6400, False)])
def test_first_unpack_of_a_plan_with_lists_in_a_graph(imu, n, d, h, deep):
    """The graph holds the unpack that comes first after the plan; its replays, and an unpack outside it, leave the same operands, and
    the fused GEMM behind each of them gives the same integers."""
    A, B = _few_digits(np.random.default_rng(n), n, d, h, deep)
    want = A.double() @ B.double().t()
    plan = _plan_of_resident_weights(imu, A, B, ROW)
    assert imu.imunpack_diag_list_columns(plan) > d // 2
    ba, bb, _ = plan.unpacked_bytes()
    A_ue, B_eu = (torch.zeros(x, dtype=torch.int8, device="cuda") for x in (ba, bb))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        imu.imunpack_unpack(plan, A, B, A_ue, B_eu)
    ws = torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda")
    for turn in range(4):
        A_ue.zero_()
        if turn < 3:
            graph.replay()
        else:
            imu.imunpack_unpack(plan, A, B, A_ue, B_eu)
        torch.cuda.synchronize()
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, ws)
        assert torch.equal(C_int.double(), want)


def test_unpack_beside_a_gemm_of_the_same_plan(imu):
    """The plan's operands are unpacked into a second pair of buffers on one stream while GEMMs on the first pair run on another: neither
    the lists nor the transposed copy of A's columns, which the plan holds, change under them."""
    n, d, h = 2000, 1660, 6400
    A, B = _few_digits(np.random.default_rng(1), n, d, h, True)
    want = A.double() @ B.double().t()
    plan = _plan_of_resident_weights(imu, A, B, ROW)
    assert imu.imunpack_diag_list_columns(plan) > d // 2
    A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
    A2, B2 = torch.zeros_like(A_ue), torch.zeros_like(B_eu)
    outs = [torch.full((n, h), -1, dtype=torch.int64, device="cuda") for _ in range(8)]
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for C_int in outs:
        with torch.cuda.stream(second):
            imu.imunpack_unpack(plan, A, B, A2, B2)
        with torch.cuda.stream(first):
            imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
    torch.cuda.synchronize()
    for C_int in outs:
        assert torch.equal(C_int.double(), want)
    imu.imunpack_gemm(plan, A2, B2, 1.0, 1.0, outs[0].zero_(), None, None)
    assert torch.equal(outs[0].double(), want)


@pytest.mark.parametrize("n", [16, 1900])
def test_lists_with_weights_that_stay_resident(imu, n):
    """Keep-weights mode: the lists belong to the unpacking of B.  Taken over (into the same buffer, into another one), made anew when
    other columns of A are split, taken over again; the statistics are the caller's."""
    d, h, b = 1700, 6400, 8
    A, B = _few_digits(np.random.default_rng(2), n, d, h, True)
    other = torch.randint(-127, 128, (n, d), device="cuda", dtype=torch.int32)
    other[:, 3] = 5000
    st_b = imu.imunpack_scan(B, b, imu.Stats.empty(h, d, B.device, imu.Stats.default_ob_cap(h, d)))
    plan = imu.imunpack_plan(A, B, b, COL, BOTH, imu.imunpack_scan(A, b), st_b)
    plan.keep_weights()
    B_eu = None
    for X, buffer, reused in ((A, 0, False), (A.flip(0).contiguous(), 0, True), (A, 1, True), (other, 1, False), (other.flip(0).contiguous(), 1, True),
                              (A, 0, False), (A, 0, True)):
        imu.imunpack_plan(X, B, b, COL, BOTH, imu.imunpack_scan(X, b), st_b, plan)
        assert plan.weights_reused() == reused and imu.imunpack_diag_list_columns(plan) > d // 2
        ba, bb, bw = plan.unpacked_bytes()
        if B_eu is None or B_eu[0].numel() < bb:
            B_eu = [torch.zeros(bb + 2 ** 20, dtype=torch.int8, device="cuda") for _ in range(2)]
        A_ue = torch.zeros(ba, dtype=torch.int8, device="cuda")
        for _ in range(2):                  # the second unpack of a plan writes B_eu whatever was taken over
            imu.imunpack_unpack(plan, X, B, A_ue, B_eu[buffer])
            C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
            imu.imunpack_gemm(plan, A_ue, B_eu[buffer], 1.0, 1.0, C_int, None, None)
            assert torch.equal(C_int.double(), X.double() @ B.double().t())


def test_lists_that_outgrow_their_places(imu):
    """Thirty heavy hitters in each of 32 rows side by side, forty in every column: the columns are split, and the list of those rows is
    far longer than the average that the plan makes room for.  It is made again with more."""
    n, d, h = 40, 1600, 24000
    rng = np.random.default_rng(3)
    A, B = (rng.integers(-127, 128, (r, d)).astype(np.int32) for r in (n, h))
    for k in range(d):
        B[64 + rng.choice(h - 64, 39, replace=False), k] = rng.integers(128, 128 ** 2, 39)
    for r in range(32, 64):
        B[r, rng.choice(d, 30, replace=False)] = -300
    A, B = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    want = A.double() @ B.double().t()
    plan = _plan_of_resident_weights(imu, A, B, ROW)
    for _ in range(2):
        assert imu.imunpack_diag_list_columns(plan) == d
        A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
        assert torch.equal(C_int.double(), want)
        imu.imunpack_plan(A, B, 8, ROW, BOTH, plan=plan)
        assert plan.weights_reused()


def test_bounds_of_a_first_unpack_in_a_graph(imu):
    """Every replay of a graph that holds a plan's first unpack measures the bounds afresh, also where it leaves the second operand's
    unpacking, which a plan in keep-weights mode took over, as it is."""
    rng = np.random.default_rng(8)
    Aq, Bq = (rand_ints(rng, r, 400, 128, 0.003, 2) for r in (130, 200))
    want = oracle.int_gemm(Aq, Bq)
    Qa, Qb = torch.from_numpy(Aq).cuda(), torch.from_numpy(Bq).cuda()
    plan = imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH)
    plan.keep_weights()
    imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH, plan=plan)
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    bounds = plan.bounds()
    for taken_over in (False, True):
        plan.keep_weights(taken_over)
        imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH, plan=plan)
        if taken_over:                      # the plan that the next one takes it over from
            imu.imunpack_unpack(plan, Qa, Qb, A_ue, B_eu)
            imu.imunpack_plan(Qa, Qb, 8, BOTH, BOTH, plan=plan)
        assert plan.weights_reused() == taken_over
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            imu.imunpack_unpack(plan, Qa, Qb, A_ue, B_eu)
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        assert plan.bounds() == bounds
        C_int = torch.full(want.shape, -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
        assert np.array_equal(C_int.cpu().numpy(), want)


def test_lists_of_weights_survive_more_rows_of_activations(imu):
    """The rows of A do not concern B's unpacking: an activation whose rows all split, twice the physical rows of the one before, takes it
    over, lists and all."""
    n, d, h, b = 700, 1700, 6400, 8
    A, B = _few_digits(np.random.default_rng(4), n, d, h, False)
    split = A.clone()
    split[:, 11] = 4000
    plan = imu.imunpack_plan(A, B, b, ROW, BOTH)
    plan.keep_weights()
    for X, reused in ((A, False), (split, True), (A, True)):
        imu.imunpack_plan(X, B, b, ROW, BOTH, plan=plan)
        assert plan.weights_reused() == reused and imu.imunpack_diag_list_columns(plan) > d // 2
        A_ue, B_eu = imu.imunpack_unpack(plan, X, B)
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, None)
        assert torch.equal(C_int.double(), X.double() @ B.double().t())


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("roomy", [False, True])
def test_more_columns_than_the_layout_with_lists_holds(imu, keep, roomy):
    """Every column of A in three levels: more column slots than the layout in LDS, which alone knows lists, has room for.  On a new plan
    object, which learns of them by the room it lacks, and on one that has the room."""
    n, d, h = 33, 4100, 1100
    A, B = _few_digits(np.random.default_rng(5), n, d, h, False)
    A[torch.arange(d, device="cuda") % n, torch.arange(d, device="cuda")] = 20000
    want = A.double() @ B.double().t()
    plan = imu.Plan()
    if roomy:
        imu.imunpack_plan(A, B[:1090], 8, COL, BOTH, plan=plan)
    imu.imunpack_plan(A, B, 8, COL, BOTH, plan=plan)
    plan.keep_weights(keep)
    for turn in range(3):
        assert imu.imunpack_diag_list_columns(plan) == 0 and plan.dims()[1] > 12288 and plan.weights_reused() == (keep and turn == 2)
        A_ue, B_eu = imu.imunpack_unpack(plan, A, B)
        C_int = torch.full((n, h), -1, dtype=torch.int64, device="cuda")
        imu.imunpack_gemm(plan, A_ue, B_eu, 1.0, 1.0, C_int, None, torch.empty(plan.unpacked_bytes()[2] // 8, dtype=torch.int64, device="cuda"))
        assert torch.equal(C_int.double(), want)
        imu.imunpack_plan(A, B, 8, COL, BOTH, plan=plan)


def test_batch_of_one_with_lists(imu):
    """A batch of one product, and one large enough for lists on every call, takes the one-product launch with them: the same bits as the
    calling sequence, and the exact product."""
    n, d, h = 4100, 2100, 8200
    g = torch.Generator(device="cuda").manual_seed(3)
    A, B = torch.randn((n, d), generator=g, device="cuda"), torch.randn((h, d), generator=g, device="cuda") * 0.02
    A[:, ::300] *= 100.0
    B[torch.rand((h, d), generator=g, device="cuda") < 0.001] *= 20.0
    got = imu.imunpack_gemm_batched(A[None], B[None], 95.0, 31.0, 31.0, 8, ROW, BOTH, ctx=imu.BatchContext())[0]
    steps = [float(imu.imunpack_rtn_step(X, 95.0, 31.0)[0].item()) for X in (A, B)]
    (Qa, *_), (Qb, *_) = (imu.imunpack_quantize(X, s, 8) for X, s in zip((A, B), steps))
    plan = imu.imunpack_plan(Qa, Qb, 8, ROW, BOTH)
    assert imu.imunpack_diag_list_columns(plan) > d // 2
    A_ue, B_eu = imu.imunpack_unpack(plan, Qa, Qb)
    C = torch.empty((n, h), device="cuda")
    imu.imunpack_gemm(plan, A_ue, B_eu, steps[0], steps[1], None, C, None)
    assert torch.equal(got, C) and torch.equal(C, (Qa.double() @ Qb.double().t() * (steps[0] * steps[1])).float())
