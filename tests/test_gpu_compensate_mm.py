"""The compensation of many tokens.  Row layout (on the matrix cores, and in list
order): each number of waves per task, remainders in tokens, columns and list
positions, lists longer than a wave holds, tokens without entries.  GEMM layout: one and four columns a
lane, lists longer than a wave's registers, and per-column codebooks with the
GEMM before it (more than 96 tokens).  And the split by channel where it is
taken, i.e. past 10^9 list entries x columns.

Bound: a sum of 2k products r * c in fp32: (2k + 2) 2^-24 sum |r c|, times
s_j; twice that is allowed.  The split's heavy channels hold r over the token's
scale as an fp16 pair, whose low half ends in the subnormals: 2^-25 max |r|
sum |c| more."""
import numpy as np
import pytest

from oracle import oasis_oracle as O
from paper_2507_23035_amd import oasis, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # n, d_in, d_out, k
    (33, 256, 100, 4),        # 6 waves a task: five tiles of 8 tokens, the last of one
    (65, 512, 1000, 64),      # 36 tasks, whole groups of 8
    (200, 520, 8191, 5),      # 3 waves a task, unaligned rows of y, partial groups
    (500, 264, 4100, 9),      # 2 waves a task
    (800, 256, 6700, 3),      # 1 wave a task, one round
    (1000, 256, 20000, 6),    # several slabs a wave, the last run shorter
    (40, 2048, 300, 900),     # lists longer than a wave holds
]


def reference(mx, mn, r, w, s_w, pair=False):
    ch = np.concatenate([mx, mn], 1)
    n, d_in = ch.shape[0], w.shape[0]
    dense = np.zeros((n, d_in))
    for i in range(n):
        ok = (ch[i] >= 0) & (ch[i] < d_in)
        np.add.at(dense[i], ch[i][ok], r[i][ok].astype(np.float64))
    ref = (torch.from_numpy(dense) @ torch.from_numpy(w)).numpy() * s_w
    mag = (torch.from_numpy(np.abs(dense)) @ torch.from_numpy(np.abs(w))).numpy() * s_w
    rest = np.abs(r).max(1, keepdims=True) * np.abs(w).max() * ch.shape[1] * s_w
    return ref, 2.0 * ((ch.shape[1] + 2) * 2.0 ** -24 * mag + (2.0 ** -25 * rest if pair else 0.0))


def inputs(n, d_in, d_out, k):
    rng = np.random.default_rng(n + k)
    w_idx = rng.integers(0, 16, (d_in, d_out), dtype=np.uint8)
    cb = np.sort(rng.standard_normal(16)).astype(np.float16)
    s_w = rng.uniform(0.5, 2.0, d_out).astype(np.float32)
    order = np.argsort(rng.random((n, d_in)), axis=1)[:, : 2 * k].astype(np.int32)
    mx, mn = order[:, :k].copy(), order[:, k:].copy()
    r = (rng.standard_normal((n, 2 * k)) * np.exp(rng.uniform(-6, 6, (n, 1)))).astype(np.float32)
    mn[::3, -1] = -1            # an unused place
    r[1::4, 0] = 0.0            # compensated through the other list
    r[n // 2] = 0.0             # a token without live entries
    r[3, 0] = 1.0e30            # far beyond fp16
    r[5] *= 1.0e-30             # far below it
    return w_idx, cb, s_w, mx, mn, r


def upload(v):
    return torch.from_numpy(np.ascontiguousarray(v)).to(torch.device("cuda:0"))


def check(call, ref, bound, n, d_out):
    y = torch.full((n, d_out), float("nan"), device="cuda:0")
    call(y, False)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= bound), np.nanmax(np.abs(got - ref) / (bound + 1e-300))
    y.fill_(0.5)
    call(y, True)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref - 0.5) <= bound + 2.0 ** -23 * (np.abs(ref) + 1.0))


def rows_call(fused, lists, w_idx, lut, ts):
    """Y' from the row layout: the matrix-core kernel through the fused call with
    tokens of scale 0 (Y* = 0), or the call that sums in list order."""
    n, (d_in, _) = lists[0].shape[0], w_idx.shape
    idx_wr = upload(oasis.pack_weight_rows(w_idx).view(np.int32))
    if not fused:
        return lambda y, acc: oasis.outlier_compensate_rows(*lists, idx_wr, lut, 4, ts, d_in, y=y,
                                                            accumulate=acc)
    idx_w = upload(oasis.pack_weight_indices(w_idx).view(np.int32))
    codes = torch.zeros((n, d_in // 2), dtype=torch.uint8, device="cuda:0")
    t = torch.zeros(n, device="cuda:0")
    return lambda y, acc: oasis.lut_gemm_compensated_rows(codes, t, idx_w, idx_wr, ts, lut, 4, 4,
                                                          *lists, y=y, accumulate=acc)


@pytest.mark.parametrize("n,d_in,d_out,k", CASES)
@pytest.mark.parametrize("fused", [True, False])
def test_compensate_rows(n, d_in, d_out, k, fused):
    print(f"case compensate_mm n={n} d_in={d_in} d_out={d_out} k={k} fused={fused}", flush=True)
    w_idx, cb, s_w, mx, mn, r = inputs(n, d_in, d_out, k)
    lut = oasis.build_lut(cb, 4, cb, 4)
    ref, bound = reference(mx, mn, r, cb.astype(np.float64)[w_idx], s_w.astype(np.float64))
    lists = [upload(v) for v in (mx, mn, r)]
    check(rows_call(fused, lists, w_idx, lut, upload(s_w)), ref, bound, n, d_out)


@pytest.mark.parametrize("n,d_in,d_out,k", [(40, 512, 300, 20), (70, 2048, 77, 300)])
def test_compensate_rows_sums_in_list_order(n, d_in, d_out, k):
    """outlier_compensate_rows: one fp32 fma per entry in list order, then s_j, bit
    for bit (each fma emulated in fp64 as one rounding of an exact sum: entries
    of 13 bits and one magnitude, where the product has 24 bits)."""
    print(f"case list order n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    w_idx, cb, s_w, mx, mn, r = inputs(n, d_in, d_out, k)
    rng = np.random.default_rng(k)
    r = (rng.integers(4096, 8192, r.shape) * rng.choice([-1.0, 1.0], r.shape) / 4096).astype(np.float32)
    r[n // 2] = 0.0
    ch, acc = np.concatenate([mx, mn], 1), np.zeros((n, d_out), dtype=np.float32)
    c = cb.astype(np.float64)
    for e in range(2 * k):
        live = ch[:, e] >= 0
        step = acc[live] + r[live, e, None].astype(np.float64) * c[w_idx[ch[live, e]]]
        acc[live] = step.astype(np.float32)
    lut = oasis.build_lut(np.arange(16).astype(np.float16), 4, cb, 4)
    y = torch.full((n, d_out), float("nan"), device="cuda:0")
    rows_call(False, [upload(v) for v in (mx, mn, r)], w_idx, lut, upload(s_w))(y, False)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), acc * s_w)


@pytest.mark.parametrize("n,d_in,d_out,k", [
    (33, 256, 100, 4),        # 6 waves a task
    (500, 264, 4100, 9),      # fewer
    (1100, 2048, 5000, 100),  # one, compacted lists of the split by channel
])
def test_small_entries_beside_a_massive_one(n, d_in, d_out, k):
    """A token's small entries stay as they are beside one of 2^20 to 2^34 times
    their size: where that one meets a centroid of 0 the column is their sum alone.
    The bound is that of the fp32 sum, with no term for the residuals' format."""
    w_idx, cb, s_w, mx, mn, r = inputs(n, d_in, d_out, k)
    rng = np.random.default_rng(k)
    mx[mx < 16] += 16                      # (a channel may occur twice)
    mn[(mn >= 0) & (mn < 16)] += 16
    mx[:, 1] = rng.integers(0, 16, n)      # the massive entry's channel
    r = (rng.standard_normal((n, 2 * k)) * np.exp2(rng.uniform(-14, 0, (n, 2 * k)))).astype(np.float32)
    r[:, 1] = rng.choice([-1.0, 1.0], n) * 2.0 ** 20
    cb[7] = 0.0
    w_idx[:16, ::3] = 7
    split = n * 2 * k * d_out > 10 ** 9
    print(f"case compensate_mm range n={n} d_in={d_in} d_out={d_out} k={k} split={split}", flush=True)
    w = cb.astype(np.float64)[w_idx]
    ch = np.concatenate([mx, mn], 1)
    dense, absd = np.zeros((n, d_in)), np.zeros((n, d_in))
    for i in range(n):
        ok = ch[i] >= 0
        np.add.at(dense[i], ch[i][ok], r[i][ok].astype(np.float64))
        np.add.at(absd[i], ch[i][ok], np.abs(r[i][ok].astype(np.float64)))
    ref = (torch.from_numpy(dense) @ torch.from_numpy(w)).numpy() * s_w.astype(np.float64)
    mag = (torch.from_numpy(absd) @ torch.from_numpy(np.abs(w))).numpy() * s_w.astype(np.float64)
    bound = 2.0 * (2 * k + 2) * 2.0 ** -24 * mag
    assert 0.0 < np.median(np.abs(ref[:, ::3])) < 2.0 ** 8   # the columns in question
    lut = oasis.build_lut(np.arange(16).astype(np.float16), 4, cb, 4)
    idx_wr, idx_w = upload(oasis.pack_weight_rows(w_idx).view(np.int32)), upload(
        oasis.pack_weight_indices(w_idx).view(np.int32))
    lists, ts = [upload(v) for v in (mx, mn, r)], upload(s_w)
    codes = torch.zeros((n, d_in // 2), dtype=torch.uint8, device="cuda:0")
    t = torch.zeros(n, device="cuda:0")    # Y* = 0
    args = (codes, t, idx_w, idx_wr, ts, lut, 4, 4, *lists)
    y = (oasis.lut_gemm_compensated_split if split else oasis.lut_gemm_compensated_rows)(*args)
    torch.cuda.synchronize()
    err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= bound), np.max(err / (bound + 1e-300))


@pytest.mark.parametrize("n,d_in,d_out,k", [(33, 256, 100, 4), (800, 256, 6700, 3)])
@pytest.mark.parametrize("fused", [True, False])
def test_infinite_residual_rows(n, d_in, d_out, k, fused):
    """An infinite residual gives infinities with its weights' signs; the other
    tokens of its tile stay as they are."""
    print(f"case compensate_mm inf n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    w_idx, cb, s_w, mx, mn, r = inputs(n, d_in, d_out, k)
    assert np.all(cb != 0)
    r[10, 0] = 1.0
    ref, bound = reference(mx, mn, r, cb.astype(np.float64)[w_idx], s_w.astype(np.float64))
    r[10, 0] = np.inf
    lut = oasis.build_lut(cb, 4, cb, 4)
    y = torch.full((n, d_out), float("nan"), device="cuda:0")
    rows_call(fused, [upload(v) for v in (mx, mn, r)], w_idx, lut, upload(s_w))(y, False)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    assert np.array_equal(got[10], np.inf * np.sign(cb.astype(np.float64)[w_idx[mx[10, 0]]]))
    rest = np.arange(n) != 10
    assert np.all(np.abs(got - ref)[rest] <= bound[rest])


@pytest.mark.parametrize("n,d_in,d_out,k", [
    (33, 64, 7, 2),           # one column a lane, most lanes past d_out
    (100, 520, 130, 40),      # a workgroup per token and 64 columns: 20 entries a wave
    (700, 520, 130, 40),      # one column a lane, 80 entries: a second pass of 16
    (2100, 264, 260, 3),      # four columns a lane, 16-byte stores, a partial slab
    (700, 256, 777, 33),      # four columns a lane, unaligned rows, 66 entries
])
def test_compensate_gemm_layout(n, d_in, d_out, k):
    print(f"case compensate_cols n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    w_idx, cb, s_w, mx, mn, r = inputs(n, d_in, d_out, k)
    lut = oasis.build_lut(cb, 4, cb, 4)
    idx_w, ts = upload(oasis.pack_weight_indices(w_idx).view(np.int32)), upload(s_w)
    ref, bound = reference(mx, mn, r, cb.astype(np.float64)[w_idx], s_w.astype(np.float64))
    lists = [upload(v) for v in (mx, mn, r)]
    check(lambda y, acc: oasis.outlier_compensate(*lists, idx_w, lut, 4, ts, d_in, y=y,
                                                  accumulate=acc), ref, bound, n, d_out)


@pytest.mark.parametrize("n,d_in,d_out,k", [
    (97, 72, 37, 4),          # a masked last block, most waves without one, 37 of 64 columns
    (130, 1024, 300, 0),      # two token tiles, no lists
    (300, 584, 1001, 20),     # unaligned rows of y
    (1100, 512, 544, 8),      # four columns a lane in the compensation
])
def test_percol_many_tokens(n, d_in, d_out, k):
    print(f"case percol n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    L = synth.make_layer(synth.custom(n, d_in, d_out, k, seed=n))
    cols = synth.percol_codebooks(L)
    q = O.quantize_act(L.x, L.cb_a, 4, k)
    w = np.take_along_axis(cols.astype(np.float64).T, L.w_idx.astype(np.int64), axis=0)
    a = L.cb_a.astype(np.float64)[q["a"]] * q["t"].astype(np.float64)[:, None]
    s_w = L.s_w.astype(np.float64)
    ref = (torch.from_numpy(a) @ torch.from_numpy(w)).numpy() * s_w
    mag = (torch.from_numpy(np.abs(a)) @ torch.from_numpy(np.abs(w))).numpy() * s_w
    bound = 2.0 * (d_in + 2) * 2.0 ** -24 * mag
    if k:
        comp, more = reference(q["max_idx"], q["min_idx"], q["residual"], w, s_w)
        ref, bound = ref + comp, bound + more + 2.0 ** -22 * (np.abs(comp) + mag)
    lut = oasis.build_lut(L.cb_a, 4, L.cb_w, 4)
    idx_w, ts = upload(oasis.pack_weight_indices(L.w_idx).view(np.int32)), upload(L.s_w)
    args = [upload(O.pack_act_indices(q["a"])), upload(q["t"]), idx_w, ts, lut, upload(cols), 4, 4,
            *[upload(q[key]) for key in ("max_idx", "min_idx", "residual")]]
    check(lambda y, acc: oasis.lut_gemm_compensated_percol(*args, y=y, accumulate=acc), ref, bound,
          n, d_out)


@pytest.mark.parametrize("n,d_in,d_out,k", [(128, 4096, 512, 32), (100, 11008, 320, 88)])
def test_percol_error_of_one_gemm(n, d_in, d_out, k):
    """One call past 96 tokens is no further from 64 bits than calls of 32 tokens
    (2-norms over 30000 and more outputs, whose ratio is steady to a few per cent)."""
    print(f"case percol error n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    L = synth.make_layer(synth.custom(n, d_in, d_out, k, seed=n))
    cols = synth.percol_codebooks(L)
    q = O.quantize_act(L.x, L.cb_a, 4, k)
    w = np.take_along_axis(cols.astype(np.float64).T, L.w_idx.astype(np.int64), axis=0)
    a = L.cb_a.astype(np.float64)[q["a"]] * q["t"].astype(np.float64)[:, None]
    s_w = L.s_w.astype(np.float64)
    ref = (torch.from_numpy(a) @ torch.from_numpy(w)).numpy() * s_w
    ref += reference(q["max_idx"], q["min_idx"], q["residual"], w, s_w)[0]
    lut = oasis.build_lut(L.cb_a, 4, L.cb_w, 4)
    idx_w, ts = upload(oasis.pack_weight_indices(L.w_idx).view(np.int32)), upload(L.s_w)
    act, t, cb = upload(O.pack_act_indices(q["a"])), upload(q["t"]), upload(cols)
    lists = [upload(q[key]) for key in ("max_idx", "min_idx", "residual")]

    def error(step):
        y = torch.cat([oasis.lut_gemm_compensated_percol(act[i:i + step], t[i:i + step], idx_w, ts,
                                                         lut, cb, 4, 4, *(v[i:i + step] for v in lists))
                       for i in range(0, n, step)])
        return np.linalg.norm(y.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)

    one, launches = error(n), error(32)
    assert one <= 1.05 * launches, (one, launches)


@pytest.mark.parametrize("n,d_in,d_out,k,mode", [
    (2000, 256, 4000, 64, O.SCALE_NONE),    # residuals over t past 2^15 leave the GEMM
    (1100, 1088, 2000, 256, O.SCALE_ABSMAX),  # more heavy channels than the dense part takes
    (2000, 264, 4000, 64, O.SCALE_ABSMAX),  # d_in not a multiple of 64: split, then the GEMM
    (400, 320, 16101, 80, O.SCALE_ABSMAX),  # the fewest tokens, unaligned rows of y
])
@pytest.mark.parametrize("accumulate", [False, True])
def test_split_is_taken(n, d_in, d_out, k, mode, accumulate):
    """The split by channel inside the GEMM, at sizes past the rule that skips it."""
    assert n * 2 * k * d_out > 10 ** 9
    L = synth.make_layer(synth.custom(n, d_in, d_out, k, seed=77, dist="normal", outlier_count=5,
                                      outlier_scale=6.0))
    if mode == O.SCALE_NONE:
        L.x[:, 7] = np.float16(40000.0)
        L.x[::2, 9] = np.float16(-40000.0)
    print(f"case split n={n} d_in={d_in} d_out={d_out} k={k} mode={mode}", flush=True)
    dev = torch.device("cuda:0")
    q = O.quantize_act(L.x, L.cb_a, 4, k, mode)
    t = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to(dev)
    idx_w = t(oasis.pack_weight_indices(L.w_idx).view(np.int32))
    idx_wr = t(oasis.pack_weight_rows(L.w_idx).view(np.int32))
    lut = oasis.build_lut(L.cb_a, 4, L.cb_w, 4)
    ws = torch.full((oasis.split_workspace_bytes(n, d_in, d_out, k),), 0x5A, dtype=torch.uint8,
                    device=dev)
    y = torch.full((n, d_out), 0.5 if accumulate else float("nan"), device=dev)
    oasis.lut_gemm_compensated_split(t(O.pack_act_indices(q["a"])), t(q["t"]), idx_w, idx_wr,
                                     t(L.s_w), lut, 4, 4, t(q["max_idx"]), t(q["min_idx"]),
                                     t(q["residual"]), y=y, accumulate=accumulate, workspace=ws)
    torch.cuda.synchronize()
    w = L.cb_w.astype(np.float64)[L.w_idx]
    a = L.cb_a.astype(np.float64)[q["a"]] * q["t"].astype(np.float64)[:, None]
    comp, bound = reference(q["max_idx"], q["min_idx"], q["residual"], w, L.s_w.astype(np.float64),
                            pair=True)
    main = (torch.from_numpy(a) @ torch.from_numpy(w)).numpy() * L.s_w
    mag = (torch.from_numpy(np.abs(a)) @ torch.from_numpy(np.abs(w))).numpy() * L.s_w
    bound = bound + 2.0 * (d_in + 2) * 2.0 ** -24 * mag
    if accumulate:  # 0.5 added once, one more rounding
        main = main + 0.5
        bound = bound + 2.0 ** -23 * (np.abs(main + comp) + 0.5)
    err = np.abs(y.cpu().numpy().astype(np.float64) - main - comp)
    assert np.all(err <= bound), (err / bound).max()


@pytest.mark.parametrize("n,d_in,d_out,k", [(2000, 256, 4000, 64), (1100, 1088, 2000, 256)])
def test_split_replays_match_eager(n, d_in, d_out, k):
    """The split by channel inside the GEMM (both GEMM kernels) captured once and
    replayed three times, y and the workspace poisoned and an eager call made in
    between: every replay equals the eager call bit for bit."""
    assert n * 2 * k * d_out > 10 ** 9
    print(f"case split graph n={n} d_in={d_in} d_out={d_out} k={k}", flush=True)
    L = synth.make_layer(synth.custom(n, d_in, d_out, k, seed=78))
    x = upload(L.x.view(np.int16))
    idx_w = upload(oasis.pack_weight_indices(L.w_idx).view(np.int32))
    idx_wr = upload(oasis.pack_weight_rows(L.w_idx).view(np.int32))
    s_w = upload(L.s_w)
    lut, q = oasis.build_lut_quantize_act(L.cb_a, 4, L.cb_w, 4, x, k)
    ws = torch.empty(oasis.split_workspace_bytes(n, d_in, d_out, k), dtype=torch.uint8,
                     device="cuda:0")
    y = torch.empty((n, d_out), dtype=torch.float32, device="cuda:0")

    def step():
        oasis.build_lut_quantize_act(L.cb_a, 4, L.cb_w, 4, x, k, lut=lut, out=q)
        oasis.lut_gemm_compensated_split(q["idx_act"], q["act_scale"], idx_w, idx_wr, s_w, lut, 4,
                                         4, q["max_idx"], q["min_idx"], q["residual"], y=y,
                                         workspace=ws)

    step()
    torch.cuda.synchronize()
    want = y.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        y.fill_(float("nan"))
        ws.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
        step()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
