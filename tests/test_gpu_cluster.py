"""GPU parity: clustering, error table, allocation and packing against the CPU oracle.

Bar: labels, thresholds, allocations, packed codes and codebooks bit-exact;
centroids and errors within 1e-5 relative.  A decision whose oracle
margin is below 1e-9 may legitimately fall the other way (the two sides sum in
different orders); the oracle counts such decisions per (row, bit width), only
those entries are excused from the exact comparison, and they are still checked
for self-consistency through the oracle's functions (tests/parity_util.py).
On config 0 the count must be zero.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import parity_util
import skim_synth

pytestmark = pytest.mark.gpu

RTOL = 1e-5


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rel_close(got, ref, rtol=RTOL):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    scale = np.maximum(np.abs(ref), 1e-300)
    return np.abs(got - ref) <= rtol * scale + 0.0


def check_table(ctx, W, S, alpha=None, iters=30, bmin=1, bmax=4, require_no_near=False):
    """Error table against the oracle, entry by entry (parity_util.compare_table).  Returns the oracle's result,
    the GPU's, and the number of (row, bit width) entries excused from the exact comparison."""
    ref = oracle.error_table(W, S, alpha, bmin=bmin, bmax=bmax, T=iters, count_near=True)
    out = ctx.error_table(dev(W), dev(S), None if alpha is None else dev(alpha), bmin=bmin, bmax=bmax, iters=iters)
    torch.cuda.synchronize()
    E = out["E"].cpu().numpy()
    ca = out["centroids_all"].cpu().numpy()
    ua = out["upper_all"].cpu().numpy()
    if require_no_near:
        assert ref["near"].tolist() == [0, 0]
    st = parity_util.compare_table(W, S, alpha, ref, E, ca, ua, bmin=bmin, bmax=bmax)
    return ref, out, st["excused"]


def check_rows(ctx, W, S, bits, alpha=None, iters=30):
    """cluster_rows against the oracle: rows without a near-tie bit-exact (labels, thresholds), the others a
    consistent clustering of their own (labels follow from the thresholds, centroids and error from the labels)."""
    cr = ctx.cluster_rows(dev(W), dev(S), dev(bits), alpha=None if alpha is None else dev(alpha), iters=iters)
    torch.cuda.synchronize()
    rr = oracle.cluster_rows(W, S, bits, alpha=alpha, T=iters, count_near=True)
    clean = rr["near_rows"] == 0
    lab = cr["labels"].cpu().numpy()
    up = cr["upper"].cpu().numpy().astype(np.float64)
    assert np.array_equal(lab[clean], rr["labels"][clean])
    assert np.array_equal(up[clean], rr["upper"][clean])
    parity_util.check_rows_self_consistent(W, S, alpha, bits, lab, cr["centroids"].cpu().numpy(), up,
                                           cr["err"].cpu().numpy(), rows=np.flatnonzero(~clean))
    return cr, rr, clean


def test_config0_error_table_allocation_labels_and_pack(ctx, gpu_lib):
    W, S = skim_synth.make_ws(0)
    ref, out, excused = check_table(ctx, W, S, require_no_near=True)
    assert excused == 0
    E = out["E"].cpu().numpy()
    # allocation to 3.0 bits through the library's allocator on the GPU's table
    bits, spent, budget = gpu_lib.greedy_allocate(E, 3.0)
    g = oracle.greedy(ref["E"], 3.0, count_near=True)
    assert g["near"] == 0
    assert np.array_equal(bits, g["bits"]) and spent == g["spent"] == 1536 and budget == 1536
    # K-means at the allocated widths: labels bit-exact
    dbits = dev(bits)
    cr = ctx.cluster_rows(dev(W), dev(S), dbits)
    torch.cuda.synchronize()
    rr = oracle.cluster_rows(W, S, bits, count_near=True)
    assert int(rr["near_rows"].sum()) == 0
    assert np.array_equal(cr["labels"].cpu().numpy(), rr["labels"])
    assert np.array_equal(cr["upper"].cpu().numpy().astype(np.float64), rr["upper"])
    assert rel_close(cr["err"].cpu().numpy(), rr["err"]).all()
    np.testing.assert_allclose(cr["centroids"].cpu().numpy(), rr["centroids"], rtol=RTOL, atol=1e-14)
    # the per-bit blocks of the table hold the same clustering (no second K-means needed)
    sel = ctx.select_allocated(dbits, out)
    torch.cuda.synchronize()
    assert torch.equal(sel["centroids"], cr["centroids"]) and torch.equal(sel["upper"], cr["upper"])
    assert torch.equal(sel["err"], cr["err"])
    # pack from thresholds
    pk = ctx.pack(dev(W), dbits, sel["centroids"], sel["upper"], want_dW=True, bits_host=bits)
    torch.cuda.synchronize()
    rp = oracle.pack(W, bits, rr["labels"], rr["centroids"], want_dW=True)
    assert np.array_equal(pk["codes"].cpu().numpy().view(np.uint32), rp["codes"])
    assert np.array_equal(pk["group_word_offset"].cpu().numpy(), rp["group_word_offset"])
    assert np.array_equal(pk["row_perm"].cpu().numpy(), rp["row_perm"])
    assert np.array_equal(pk["codebooks"].cpu().numpy().view(np.uint16), rp["codebooks"])
    assert np.array_equal(pk["dW"].cpu().numpy(), rp["dW"])


@pytest.mark.parametrize("m", [16, 17, 33, 100, 255, 256, 257, 1000, 2049, 4095, 4097])
def test_ragged_row_lengths(ctx, m):
    W, S = skim_synth.make_ws_small(m, 24, m)
    ref, out, excused = check_table(ctx, W, S)
    assert excused <= 1


@pytest.mark.parametrize("m", [11264, 11808, 12289, 14000, 16384])
def test_rows_whose_running_sums_are_kept_for_groups_of_16_chunks(ctx, m):
    """Rows of one sort on either side of the length from which the iterations keep their running sums for wider groups,
    with an element that outweighs the rest, a row of one value and part-filled last groups."""
    W, S = skim_synth.make_ws_small(m, 6, m, dup_frac=0.05)
    S[1, m // 3] = 1e12
    W[4] = 0.25
    ref, out, excused = check_table(ctx, W, S)
    bits = np.array([1, 2, 3, 4, 3, 2], np.uint8)
    check_rows(ctx, W, S, bits)


@pytest.mark.parametrize("m", [16385, 16400, 20000, 32768])
def test_rows_longer_than_one_lds_sort(ctx, m):
    W, S = skim_synth.make_ws_small(m, 6, m, dup_frac=0.05)
    S[2] = 0.0                      # no sensitivity mass: unit weights on the merged path too
    W[3, : m // 2] = np.sort(W[3, : m // 2])        # first half entirely below / interleaved with the second
    ref, out, excused = check_table(ctx, W, S)
    assert excused <= 6          # entries, as counted by the oracle on these inputs (2, 3, 6, 4)
    bits = np.array([1, 2, 3, 4, 3, 2], np.uint8)
    check_rows(ctx, W, S, bits)


def test_duplicates_zero_sensitivities_and_dead_rows(ctx):
    W, S = skim_synth.make_ws_small(7, 64, 300, dup_frac=0.3, zero_s_frac=0.4)
    S[3] = 0.0                      # a row without any sensitivity mass -> unit weights
    W[5] = np.float32(0.25)         # a constant row: every cluster but the first is empty
    W[6, :150] = np.float32(-1.0)   # two distinct values only
    W[6, 150:] = np.float32(2.0)
    W[7] = np.round(W[7] * 200) / 200   # few distinct values, many exact ties in the sort
    W[8, ::2] = 0.0
    W[8, 1::4] = -0.0               # both zeros are one value
    ref, out, excused = check_table(ctx, W, S)
    assert excused <= 4          # rows of few distinct values put elements exactly between two centroids
    bits = (np.arange(64) % 4 + 1).astype(np.uint8)
    check_rows(ctx, W, S, bits)


def test_heavy_element_rows_exercise_rank_repair(ctx):
    W, S = skim_synth.make_ws_small(9, 32, 500)
    S[np.arange(32), np.arange(32) * 13 % 500] = 1e9     # one element carries nearly all mass
    S[4, -1] = 1e12
    S[5, np.argmax(W[5])] = 1e12                          # the largest element: ranks are pushed down
    S[6, np.argmin(W[6])] = 1e12
    ref, out, excused = check_table(ctx, W, S)
    assert excused <= 1


@pytest.mark.parametrize("iters", [1, 2, 7])
def test_iteration_counts(ctx, iters):
    W, S = skim_synth.make_ws_small(40 + iters, 40, 777)
    check_table(ctx, W, S, iters=iters)


def test_bit_range_subset(ctx):
    W, S = skim_synth.make_ws_small(50, 16, 400)
    check_table(ctx, W, S, bmin=2, bmax=3)
    check_table(ctx, W, S, bmin=4, bmax=4)
    check_table(ctx, W, S, bmin=1, bmax=1)


def test_scaled_clustering(ctx):
    W, S = skim_synth.make_ws_small(60, 48, 640)
    al = skim_synth.make_alpha(3, 640, spread=0.2)
    ref, out, excused = check_table(ctx, W, S, alpha=al)
    assert excused <= 1
    bits = np.full(48, 3, np.uint8)
    cr, rr, clean = check_rows(ctx, W, S, bits, alpha=al)
    # pack with alpha: thresholds live in the scaled domain
    pk = ctx.pack(dev(W), dev(bits), cr["centroids"], cr["upper"], alpha=dev(al), want_dW=True, bits_host=bits)
    torch.cuda.synchronize()
    if clean.all():
        rp = oracle.pack(W, bits, rr["labels"], rr["centroids"], alpha=al, want_dW=True)
        assert np.array_equal(pk["codes"].cpu().numpy().view(np.uint32), rp["codes"])
        assert np.array_equal(pk["codebooks"].cpu().numpy().view(np.uint16), rp["codebooks"])
        assert np.array_equal(pk["dW"].cpu().numpy(), rp["dW"])


def test_row_stride(ctx):
    W, S = skim_synth.make_ws_small(70, 20, 512)
    Wd, Sd = dev(W), dev(S)
    out = ctx.error_table(Wd[:, :300], Sd[:, :300])       # ld = 512, m = 300
    torch.cuda.synchronize()
    ref = oracle.error_table(W[:, :300], S[:, :300], count_near=True)
    clean = ref["near_rows"] == 0
    assert rel_close(out["E"].cpu().numpy()[clean], ref["E"][clean]).all()


def test_many_rows_of_repeated_values_take_the_network_row_after_row(ctx):
    """Every row holds 24 distinct weights, each about ten times over (4 to 20 times): the value bins of the sort
    overflow in every row, so every row of a workgroup is attempted by the bucket path and then either finished by
    its third pass or dropped and sorted by the network (there are many more rows than resident workgroups).
    Results must not depend on which path sorted a row or on what the row before it left behind."""
    n, m = 30000, 256
    rng = np.random.default_rng(77)
    vals = (rng.standard_normal((n, 24)) * 0.02).astype(np.float32)
    pick = rng.integers(0, 24, (n, m))
    W = np.take_along_axis(vals, pick, axis=1)
    S = (rng.standard_normal((n, m)) ** 2).astype(np.float32)
    rows = np.r_[0:64, 14000:14064, n - 64:n]      # the oracle's comparison on a sample of rows, the GPU on all
    out = ctx.error_table(dev(W), dev(S))
    torch.cuda.synchronize()
    ref = oracle.error_table(W[rows], S[rows], count_near=True)
    E = out["E"].cpu().numpy()[rows]
    ca = out["centroids_all"].cpu().numpy()[rows]
    ua = out["upper_all"].cpu().numpy()[rows]
    st = parity_util.compare_table(W[rows], S[rows], None, ref, E, ca, ua)
    assert st["clean"].mean() > 0.5, "too few entries compared exactly"
    # the same rows on their own (one row per workgroup: the first attempt of the bucket path, then the network)
    alone = ctx.error_table(dev(W[rows]), dev(S[rows]))
    torch.cuda.synchronize()
    assert np.array_equal(alone["E"].cpu().numpy(), E)
    assert np.array_equal(alone["upper_all"].cpu().numpy(), ua)
    assert np.array_equal(alone["centroids_all"].cpu().numpy(), ca)


@pytest.mark.parametrize("where", ["start", "middle", "end"])
@pytest.mark.parametrize("m", [1000, 4096, 11008])
def test_rows_with_one_value_9_to_20_times_over(ctx, m, where):
    """Smooth rows in which one value occurs k times, k = 9 .. 20, starting at every alignment to the sort's
    16-slot windows (the rank of the repeated value moves from row to row; at either end of the row or in the
    middle): the value's bin holds k keys, more than
    the two register passes of the bucket path put in order (9 they still do).  Up to 17 the third pass finishes the row, beyond
    that the network does; either way the table must be the oracle's."""
    rng = np.random.default_rng(4100 + m + len(where))
    ks = list(range(9, 21))
    n = len(ks) * 16
    W = (rng.standard_normal((n, m)) * 0.02).astype(np.float32)
    S = (rng.standard_normal((n, m)) ** 2).astype(np.float32)
    for i in range(n):
        k = ks[i // 16]
        order = np.argsort(W[i], kind="stable")
        # rank at which the run of equal values starts: at the least weights of the row, in the middle, or so that
        # the run ends within the last 16 ranks (the last, possibly part-filled, window of the sort)
        r = {"start": i % 16, "middle": (m // 3) + (i % 16), "end": m - k - (i % 16)}[where]
        cols = order[r:r + k]
        W[i, cols] = W[i, order[r]]
    ref, out, excused = check_table(ctx, W, S)
    assert excused <= n // 8


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_weights_converted_from_a_16_bit_format(ctx, fmt):
    """Weights that were rounded to bfloat16 / float16 and widened again: every row holds each value many times
    over, and the sort spreads equal weights over its value bins by their sensitivity.  Rows long enough to fill
    the bins, more rows than workgroups (so that the carried bin map is exercised), oracle on a sample of rows."""
    n, m = 600, 11008
    rng = np.random.default_rng(5)
    W = (rng.standard_normal((n, m)) * 0.02).astype(np.float32)
    mask = rng.random((n, m)) < 0.005
    W = np.where(mask, (rng.standard_normal((n, m)) * 0.2).astype(np.float32), W)
    if fmt == "bf16":
        W = torch.from_numpy(W).bfloat16().float().numpy()
    else:
        W = W.astype(np.float16).astype(np.float32)
    S = (rng.standard_normal((n, m)) ** 2).astype(np.float32)
    S[5, ::3] = 0.0                                   # sensitivities with exact zeros in one row
    W[7] = -np.abs(W[7])                              # a row of negative weights only
    out = ctx.error_table(dev(W), dev(S))
    torch.cuda.synchronize()
    rows = np.r_[0:24, 300:316, n - 8:n]
    ref = oracle.error_table(W[rows], S[rows], count_near=True)
    st = parity_util.compare_table(W[rows], S[rows], None, ref, out["E"].cpu().numpy()[rows],
                                   out["centroids_all"].cpu().numpy()[rows], out["upper_all"].cpu().numpy()[rows])
    # (repeated values make exact ties common: the oracle excuses most entries above one bit, and those are held
    # to the self-consistency checks; the one-bit entries and the rest are compared exactly)
    assert st["clean"].mean() > 0.1, "too few entries compared exactly"
    bits = rng.integers(1, 5, len(rows)).astype(np.uint8)
    check_rows(ctx, W[rows], S[rows], bits)


@pytest.mark.parametrize("m", [64, 200, 1040])
@pytest.mark.parametrize("values", [3, 5, 17, 40])
def test_centroids_that_start_on_equal_weights(ctx, m, values):
    """Rows of few distinct weights whose sensitivity lies on a few neighbouring ranks: runs of 2 to 16 positions with the same
    value, at the bottom, in the middle and at the top of every bit width, over the first iterations and until they stay."""
    rng = np.random.default_rng(100 * m + values)
    n = 24
    W = rng.choice((np.arange(values, dtype=np.float32) - values // 2) / 8.0, (n, m)).astype(np.float32)
    S = rng.random((n, m)).astype(np.float32)
    for i in range(n):          # most of the row's mass on one value
        S[i, W[i] == np.unique(W[i])[(i * values // n) % len(np.unique(W[i]))]] *= 1000.0 ** (i % 3)
    for iters in (1, 2, 30):
        check_table(ctx, W, S, iters=iters)
    check_rows(ctx, W, S, rng.integers(1, 5, n).astype(np.uint8))


@pytest.mark.parametrize("m", [18, 2047, 2052, 4100])
@pytest.mark.parametrize("offset", [0, 1])
def test_labels_at_any_alignment(ctx, m, offset):
    """The label pass with 16- and 4-byte accesses and the one column by column give the same labels, scaled or not."""
    n = 9
    W, S = skim_synth.make_ws_small(m, n, m)
    bits = dev(np.arange(n).astype(np.uint8) % 4 + 1)
    buf = torch.zeros((n, m + 7), device="cuda")
    buf[:, offset:offset + m] = dev(W)
    Sb = torch.zeros((n, m + 7), device="cuda")
    Sb[:, offset:offset + m] = dev(S)
    for al in (None, dev(skim_synth.make_alpha(3, m))):
        a = ctx.cluster_rows(dev(W), dev(S), bits, alpha=al)
        b = ctx.cluster_rows(buf[:, offset:offset + m], Sb[:, offset:offset + m], bits, alpha=al)
        lab = torch.zeros(n * m + 4, dtype=torch.uint8, device="cuda")[offset:offset + n * m].view(n, m)
        c = ctx.cluster_rows(dev(W), dev(S), bits, alpha=al, out=dict(a, labels=lab))
        torch.cuda.synchronize()
        wt = dev(W) if al is None else dev(W) / al
        for i in range(n):
            K = 1 << (i % 4 + 1)
            up = a["upper"][i, :K]
            order = torch.argsort(up, stable=True)
            want = order[torch.searchsorted(up[order], wt[i])].to(torch.uint8)
            assert torch.equal(a["labels"][i], want)
        assert torch.equal(a["labels"], b["labels"]) and torch.equal(a["labels"], c["labels"])


def test_pack_mixed_bits_matches_oracle_layout(ctx):
    n, m = 97, 1111
    W, S = skim_synth.make_ws_small(80, n, m)
    bits = np.random.default_rng(0).integers(1, 5, n).astype(np.uint8)
    cr = ctx.cluster_rows(dev(W), dev(S), dev(bits))
    torch.cuda.synchronize()
    rr = oracle.cluster_rows(W, S, bits, count_near=True)
    pk = ctx.pack(dev(W), dev(bits), cr["centroids"], cr["upper"], bits_host=bits)
    torch.cuda.synchronize()
    # pack is compared on the GPU's own labels (isolates the packer from clustering near-ties)
    rp = oracle.pack(W, bits, cr["labels"].cpu().numpy(), cr["centroids"].cpu().numpy())
    assert np.array_equal(pk["codes"].cpu().numpy().view(np.uint32), rp["codes"])
    assert np.array_equal(pk["group_word_offset"].cpu().numpy(), rp["group_word_offset"])
    assert np.array_equal(pk["row_perm"].cpu().numpy(), rp["row_perm"])
    assert np.array_equal(pk["codebooks"].cpu().numpy().view(np.uint16), rp["codebooks"])
    clean = rr["near_rows"] == 0
    assert np.array_equal(cr["labels"].cpu().numpy()[clean], rr["labels"][clean])


def test_validation_mode_reports_values_the_method_is_undefined_on(gpu_lib):
    W, S = skim_synth.make_ws_small(91, 6, 200)
    al = skim_synth.make_alpha(2, 200)
    c = gpu_lib.Context(0)
    try:
        c.validate_enable(True)
        c.error_table(dev(W), dev(S), dev(al))                      # clean inputs pass
        for arr, name, val in [("W", "W", np.nan), ("W", "W", np.inf), ("S", "S", -1.0), ("S", "S", np.nan),
                               ("alpha", "alpha", 0.0), ("alpha", "alpha", -np.inf)]:
            Wb, Sb, ab = W.copy(), S.copy(), al.copy()
            {"W": Wb, "S": Sb, "alpha": ab}[arr].flat[137] = val
            with pytest.raises(gpu_lib.SkimError, match=name) as ei:
                c.error_table(dev(Wb), dev(Sb), dev(ab))
            assert ei.value.status == -6
        with pytest.raises(gpu_lib.SkimError):
            Sb = S.copy()
            Sb[5, 199] = -0.5                                       # the last element of the last row
            c.cluster_rows(dev(W), dev(Sb), dev(np.full(6, 2, np.uint8)))
        c.validate_enable(False)
        Sb = S.copy()
        Sb[0, 0] = -1.0
        c.error_table(dev(W), dev(Sb))                              # off (the default): not looked for, no error
        torch.cuda.synchronize()
    finally:
        c.close()


def test_argument_errors(ctx, gpu_lib):
    W, S = skim_synth.make_ws_small(90, 4, 64)
    with pytest.raises(gpu_lib.SkimError):
        ctx.error_table(dev(W)[:, :8], dev(S)[:, :8])              # m < 2^bmax
    with pytest.raises(gpu_lib.SkimError):
        ctx.error_table(dev(W), dev(S), bmin=0)
    with pytest.raises(gpu_lib.SkimError):
        ctx.error_table(dev(W), dev(S), iters=0)
    big = torch.zeros((1, gpu_lib.MAX_M + 1), dtype=torch.float32, device="cuda")
    with pytest.raises(gpu_lib.SkimError):
        ctx.error_table(big, big)
    with pytest.raises(gpu_lib.SkimError):
        gpu_lib.greedy_allocate(np.zeros((4, 4)), 5.0)


@pytest.mark.parametrize("n,m,with_alpha", [(37, 100, False), (64, 257, True), (130, 1500, True), (16, 11008, False),
                                            (3, 16, True), (9, 4096, True)])
def test_unpack_and_dequant_matvec_match_oracle(ctx, gpu_lib, n, m, with_alpha):
    """The packed model read back on the GPU: dense weights bit-exact, matrix-vector product (float64
    accumulation, different summation order) to 1e-12 of the sum of magnitudes."""
    W, S = skim_synth.make_ws_small(77, n, m)
    al = skim_synth.make_alpha(5, m) if with_alpha else None
    rng = np.random.default_rng(n * 1000 + m)
    bits = rng.integers(1, 5, n).astype(np.uint8)
    Wd, Sd, bd = dev(W), dev(S), dev(bits)
    ald = None if al is None else dev(al)
    cr = ctx.cluster_rows(Wd, Sd, bd, alpha=ald)
    pk = ctx.pack(Wd, bd, cr["centroids"], cr["upper"], alpha=ald, bits_host=bits)
    x = rng.standard_normal(m).astype(np.float32)
    Wq = ctx.unpack(pk, m, alpha=ald)
    y = ctx.dequant_matvec(pk, m, dev(x), alpha=ald)
    torch.cuda.synchronize()
    args = (pk["codes"].cpu().numpy().view(np.uint32), pk["group_word_offset"].cpu().numpy(),
            pk["row_perm"].cpu().numpy(), pk["codebooks"].cpu().numpy().view(np.uint16), m)
    ref = oracle.unpack(*args, alpha=al)
    assert np.array_equal(Wq.cpu().numpy(), ref)
    yref = oracle.dequant_matvec(*args, x, alpha=al)
    scale = np.abs(ref.astype(np.float64)) @ np.abs(x.astype(np.float64))
    assert np.all(np.abs(y.cpu().numpy() - yref) <= 1e-12 * scale)
    # the float32 reader: same product, float32 fused multiply-adds in its own order
    yf = ctx.dequant_matvec_f32(pk, m, dev(x), alpha=ald)
    torch.cuda.synchronize()
    assert np.all(np.abs(yf.cpu().numpy().astype(np.float64) - yref) <= 1e-5 * scale)
    # x at an address that is no multiple of 16: the kernel with 4-byte loads
    xo = torch.zeros(m + 1, dtype=torch.float32, device="cuda")
    xo[1:] = dev(x)
    y2 = ctx.dequant_matvec(pk, m, xo[1:], alpha=ald)
    yf2 = ctx.dequant_matvec_f32(pk, m, xo[1:], alpha=ald)
    torch.cuda.synchronize()
    assert np.all(np.abs(y2.cpu().numpy() - yref) <= 1e-12 * scale)
    assert np.all(np.abs(yf2.cpu().numpy().astype(np.float64) - yref) <= 1e-5 * scale)


@pytest.mark.parametrize("m", [1, 3, 31, 257, 1022, 4099, 4160])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_unpack_at_any_alignment(ctx, gpu_lib, m, offset):
    """Rows shorter than four columns up to more than one round of a workgroup, the matrix at any multiple of four bytes:
    bit-exact, and nothing written outside the matrix."""
    n = 23
    rng = np.random.default_rng(m)
    bits = np.repeat(np.arange(1, 5), 6)[:n].astype(np.uint8)[rng.permutation(n)]
    W = rng.standard_normal((n, m)).astype(np.float32)
    cent = np.sort(rng.standard_normal((n, 16)), axis=1)
    upper = np.full((n, 16), -np.inf, np.float32)
    for i in range(n):
        K = 1 << bits[i]
        upper[i, :K] = cent[i, :K]
        upper[i, K - 1] = 10.0
    pk = ctx.pack(dev(W), dev(bits), dev(cent), dev(upper), bits_host=bits)
    al = skim_synth.make_alpha(5, m)
    args = (pk["codes"].cpu().numpy().view(np.uint32), pk["group_word_offset"].cpu().numpy(),
            pk["row_perm"].cpu().numpy(), pk["codebooks"].cpu().numpy().view(np.uint16), m)
    for alpha in (None, al):
        ald = None if alpha is None else dev(alpha)
        buf = torch.full((n * m + 8,), 7.0, device="cuda")
        ctx._check(ctx.lib.skim_unpack(ctx.h, pk["codes"].data_ptr(), pk["group_word_offset"].data_ptr(), pk["row_perm"].data_ptr(),
                                       pk["codebooks"].data_ptr(), ald.data_ptr() if ald is not None else None, n, m,
                                       buf.data_ptr() + 4 * offset))
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[offset:offset + n * m].reshape(n, m), oracle.unpack(*args, alpha=alpha))
        assert np.all(got[:offset] == 7.0) and np.all(got[offset + n * m:] == 7.0)


@pytest.mark.parametrize("n,m", [(3200, 64), (1537, 1001), (900, 4097), (700, 8224), (2, 40000),
                                 (15376, 4096), (16000, 4001)])      # (stores that pass the caches by)
def test_unpack_of_several_rows_and_segments_a_workgroup(ctx, n, m):
    """One to three rows a workgroup (the last round part-filled), one to ten segments of a row: bit-exact against the codes looked up one
    by one on the device."""
    g = torch.Generator(device="cuda").manual_seed(n)
    bits = (torch.arange(n, device="cuda") % 4 + 1).to(torch.uint8)
    cent = torch.sort(torch.randn((n, 16), device="cuda", generator=g), dim=1)[0].double()
    K = (1 << bits.long())[:, None]
    slot = torch.arange(16, device="cuda")[None, :]
    upper = torch.where(slot < K - 1, cent.float(), torch.full_like(cent, 1e30).float())
    W = torch.randn((n, m), device="cuda", generator=g)
    al = dev(skim_synth.make_alpha(5, m))
    pk = ctx.pack(W, bits, cent, upper, alpha=al, bits_host=bits.cpu().numpy())
    label = torch.minimum((upper[:, None, :] < (W / al)[:, :, None]).logical_and(slot[None] < K[:, :, None]).sum(2), K - 1) if n * m < 4e6 else None
    got = ctx.unpack(pk, m, alpha=al)
    if label is None:        # (the masks of all weights at once would be large)
        label = torch.cat([torch.minimum((upper[i:i + 100, None, :] < (W[i:i + 100] / al)[:, :, None]).logical_and(slot[None] < K[i:i + 100, :, None]).sum(2),
                                         K[i:i + 100] - 1) for i in range(0, n, 100)])
    assert torch.equal(got, al * cent.float().half().float().gather(1, label))


@pytest.mark.parametrize("n,m", [(1, 5), (3, 33), (5, 8225), (2051, 2088), (4100, 4128), (8200, 2049), (600, 16411), (300, 32768)])
def test_matvec_shapes(ctx, n, m):
    """Sizes at which a workgroup takes 2, 4 or 8 rows (part-filled last ones; bit widths changing inside one) and one or
    several rounds of columns, against the float64 product with the unpacked matrix."""
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randn((n, m), device="cuda", generator=g)
    bits = (torch.arange(n, device="cuda") % 4 + 1).to(torch.uint8)
    cent = torch.sort(torch.randn((n, 16), device="cuda", generator=g), dim=1)[0].double()
    upper = cent.float()
    pk = ctx.pack(W, bits, cent, upper, bits_host=bits.cpu().numpy())
    al = dev(skim_synth.make_alpha(5, m))
    x = torch.randn(m, device="cuda", generator=g)
    Wq = ctx.unpack(pk, m, alpha=al).double()
    ref, scale = Wq @ x.double(), Wq.abs() @ x.double().abs()
    y, yf = ctx.dequant_matvec(pk, m, x, alpha=al), ctx.dequant_matvec_f32(pk, m, x, alpha=al)
    torch.cuda.synchronize()
    assert bool(((y - ref).abs() <= 1e-12 * scale).all())
    assert bool(((yf.double() - ref).abs() <= 1e-5 * scale).all())


@pytest.mark.parametrize("n,m,bound", [(2048, 11008, 1.65e-9), (2048, 22016, 1.35e-9), (1024, 100000, 0.85e-9)])
def test_float32_matvec_adds_in_short_chains(ctx, n, m, bound):
    """The float32 product may not run one chain of additions through a lane's columns: its error, against the sum of the
    products' magnitudes, would not fall with the length of the row as that of a sum of short chains does.  rms over the
    rows: 1.40e-9, 1.05e-9, 0.59e-9 (1.59e-9, 1.16e-9, 0.62e-9 with 32 columns a chain pair), with one chain 1.98e-9, 1.87e-9,
    1.73e-9; four seeds agree to 7 %, and the bound lies between."""
    g = torch.Generator(device="cuda").manual_seed(m)
    bits = (torch.arange(n, device="cuda") % 4 + 1).to(torch.uint8)
    cent = torch.sort(torch.randn((n, 16), device="cuda", generator=g), dim=1)[0].double()
    pk = ctx.pack(torch.randn((n, m), device="cuda", generator=g), bits, cent, cent.float(), bits_host=bits.cpu().numpy())
    x = torch.randn(m, device="cuda", generator=g)
    Wq = ctx.unpack(pk, m).double()
    ref, scale = Wq @ x.double(), Wq.abs() @ x.double().abs()
    err = (ctx.dequant_matvec_f32(pk, m, x).double() - ref) / scale
    rms = float((err * err).mean().sqrt())
    assert rms <= bound, f"{rms:.3e}"


@pytest.mark.parametrize("n", [1, 15, 16, 17, 16384, 16385, 33000])
@pytest.mark.parametrize("offset", [0, 3])
def test_pack_row_order(ctx, n, offset):
    """Positions of the packed rows against a stable sort by bit width: fewer rows than the plan's workgroup has threads, and
    more (a thread then counts several), rows left out among them (bits 0 and 7), the bits at any address."""
    m = 16
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randn((n, m), device="cuda", generator=g)
    cent = torch.sort(torch.randn((n, 16), device="cuda", generator=g), dim=1)[0].double()
    buf = torch.zeros(n + 8, dtype=torch.uint8, device="cuda")
    bits = buf[offset:offset + n]
    bits.copy_(torch.randint(0, 6, (n,), device="cuda", generator=g))
    bits[bits == 5] = 7
    b = bits.cpu().numpy()
    codes = torch.zeros(n, 4, dtype=torch.int32, device="cuda")
    gwo, perm = torch.zeros(6, dtype=torch.int64, device="cuda"), torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cbs = torch.zeros(n * 16, dtype=torch.int16, device="cuda")
    ctx.ensure_workspace(n, m)
    up = cent.float()
    ctx._check(ctx.lib.skim_pack(ctx.h, W.data_ptr(), None, n, m, m, bits.data_ptr(), cent.data_ptr(), up.data_ptr(),
                                 codes.data_ptr(), gwo.data_ptr(), perm.data_ptr(), cbs.data_ptr(), None))
    torch.cuda.synchronize()
    want = np.concatenate([np.flatnonzero(b == q) for q in (1, 2, 3, 4)])
    got = perm.cpu().numpy()
    assert np.array_equal(got[:len(want)], want) and np.all(got[len(want):] == -1)
    sizes = [int((b == q).sum()) * ((m * q + 31) // 32) for q in (1, 2, 3, 4)]
    assert gwo.cpu().numpy().tolist() == [0] + np.cumsum([0] + sizes).tolist()


def _tables(rng, n, kind):
    if kind == "smooth":
        g = np.sort(rng.random((n, 3)), axis=1)[:, ::-1] * rng.random((n, 1))
    elif kind == "ties":
        g = rng.integers(0, 4, (n, 3)).astype(np.float64)          # many equal reductions, some zero
    elif kind == "nonmonotone":
        g = rng.standard_normal((n, 3))                            # reductions of any sign and order
    else:
        g = np.zeros((n, 3))
    E = np.empty((n, 4))
    E[:, 3] = rng.random(n)
    for j in (2, 1, 0):
        E[:, j] = E[:, j + 1] + g[:, j]
    return E


@pytest.mark.parametrize("kind", ["smooth", "ties", "nonmonotone", "flat"])
@pytest.mark.parametrize("n,avg", [(1, 2.0), (7, 1.0), (7, 4.0), (100, 2.5), (1000, 3.2), (4096, 3.2), (22016, 2.25)])
def test_device_greedy_equals_host_and_oracle(ctx, gpu_lib, kind, n, avg):
    """Alg. 1 on the device: same bits as the host function and as the oracle's linear-scan loop on the same
    table, including tables full of ties, reductions of either sign, and the two ends of the budget."""
    rng = np.random.default_rng(n * 7 + len(kind))
    E = _tables(rng, n, kind)
    out = ctx.greedy_allocate_device(dev(E), avg)
    torch.cuda.synchronize()
    bits_h, spent, budget = gpu_lib.greedy_allocate(E, avg)
    got = out["bits"].cpu().numpy()
    info = out["info"].cpu().numpy()
    assert np.array_equal(got, bits_h)
    assert info[8] == spent == budget == info[9]
    assert np.array_equal(info[:8], np.bincount(bits_h, minlength=8))
    if n <= 4096:
        assert np.array_equal(got, oracle.greedy(E, avg)["bits"])


@pytest.mark.parametrize("kind", ["smooth", "ties", "nonmonotone", "dead rows"])
@pytest.mark.parametrize("n", [63, 1024, 1025, 4097, 8193, 12288, 12289])
@pytest.mark.parametrize("bmin,bmax", [(1, 4), (2, 3), (3, 7)])
def test_device_greedy_where_the_rows_per_thread_change(ctx, gpu_lib, kind, n, bmin, bmax):
    """Tables at the ends of the ranges that the variants with the keys in registers serve, and beyond them (more rows,
    more than three upgrades per row): the host function's bits, for budgets from one upgrade to all but one.  Dead rows:
    reductions of zero next to values over forty orders of magnitude (the keys crowd at either end of their range)."""
    rng = np.random.default_rng(n + bmax + len(kind))
    nb = bmax - bmin + 1
    if kind == "dead rows":
        E = np.cumsum(10.0 ** rng.uniform(-40, 0, (n, nb)), axis=1)[:, ::-1].copy()
        E[rng.random(n) < 0.3] = 0.0
    else:
        E = np.concatenate([_tables(rng, n, kind) for _ in range(2)], axis=1)[:, :nb].copy()
    for up in (1, n // 3, (nb - 1) * n // 2, (nb - 1) * n - 1):
        avg = bmin + up / n
        out = ctx.greedy_allocate_device(dev(E), avg, bmin=bmin, bmax=bmax)
        torch.cuda.synchronize()
        bits_h, spent, budget = gpu_lib.greedy_allocate(E, avg, bmin=bmin, bmax=bmax)
        assert np.array_equal(out["bits"].cpu().numpy(), bits_h)
        info = out["info"].cpu().numpy()
        assert info[8] == spent == budget == info[9]
        assert np.array_equal(info[:8], np.bincount(bits_h, minlength=8))


@pytest.mark.parametrize("kind", ["smooth", "ties", "nonmonotone", "flat"])
@pytest.mark.parametrize("n,avg,bmin,bmax", [(1, 2.0, 1, 4), (7, 1.0, 1, 4), (7, 4.0, 1, 4), (100, 2.5, 1, 4),
                                             (129, 3.2, 1, 4), (1000, 3.2, 1, 4), (4096, 3.2, 1, 4),
                                             (3000, 3.999, 1, 4), (5000, 3.4, 3, 4), (300, 2.5, 2, 3)])
def test_dp_allocation_equals_oracle(ctx, kind, n, avg, bmin, bmax):
    """The exact allocation: same bits, same total, same spent bits as the oracle's recurrence (same order of
    additions and the same tie rules, so nothing is left to rounding).  The sizes put the states in one
    workgroup (n <= 2600 at three extra bits) and in several, and the rows in one launch and in many."""
    rng = np.random.default_rng(n * 11 + len(kind))
    E = np.ascontiguousarray(_tables(rng, n, kind)[:, bmin - 1:bmax])
    out = ctx.dp_allocate(dev(E), avg, bmin=bmin, bmax=bmax)
    torch.cuda.synchronize()
    ref = oracle.dp_allocate(E, avg, bmin=bmin, bmax=bmax)
    info = out["info"].cpu().numpy()
    assert np.array_equal(out["bits"].cpu().numpy(), ref["bits"])
    assert info[0] == ref["total"] and info[1] == ref["spent"] and info[2] == ref["budget"]
    if kind in ("smooth",):
        # reductions that shrink with the bits: Alg. 1 reaches the same optimum
        g = ctx.greedy_allocate_device(dev(E), avg, bmin=bmin, bmax=bmax)
        gb = g["bits"].cpu().numpy()
        tot = E[np.arange(n), gb - bmin].sum()
        assert tot == pytest.approx(ref["total"], rel=1e-12)


def test_dp_allocation_rejects_bad_arguments(ctx):
    E = dev(np.zeros((10, 4)))
    with pytest.raises(Exception):
        ctx.dp_allocate(E, 0.5)
    with pytest.raises(Exception):
        ctx.dp_allocate(E, 4.5)
    assert ctx.lib.skim_dp_allocate_scratch_bytes(10, 1, 6, 2.0) == 0      # more than three bits apart
    out = ctx.dp_allocate(E, 2.0)
    torch.cuda.synchronize()
    assert np.all(out["bits"].cpu().numpy() == 1) and out["info"][0].item() == 0.0   # nothing to gain: no bit spent


def _optimal_close(got, ref, W, S, alpha=None):
    """An entry is a difference of float64 prefix sums of s w^2: absolute error of a few ulps of the row's whole
    second moment, on top of the relative tolerance of the other floating-point outputs."""
    scale = np.empty(W.shape[0])
    for i in range(W.shape[0]):
        w, s = (W[i], S[i]) if alpha is None else oracle.scale_row(W[i], S[i], alpha)
        s = s.astype(np.float64) if np.any(s > 0) else np.ones(len(s))
        scale[i] = np.sum(s * w.astype(np.float64) ** 2)
    return np.abs(got - ref) <= RTOL * np.abs(ref) + 1e-12 * scale[:, None], scale[:, None]


@pytest.mark.parametrize("n,m,dup,zs", [(24, 16, 0.0, 0.0), (24, 100, 0.2, 0.3), (20, 257, 0.0, 0.0), (12, 1000, 0.05, 0.1),
                                        (6, 2049, 0.0, 0.0)])
def test_optimal_clustering_error_matches_oracle(ctx, n, m, dup, zs):
    """The exact floor of the clustering error against the oracle's O(K m^2) programme (the GPU fills each layer
    by halving with the monotone-cut bounds): same values, and never above what the Lloyd iterations reach."""
    W, S = skim_synth.make_ws_small(m + n, n, m, dup_frac=dup, zero_s_frac=zs)
    S[1] = 0.0                                   # no mass: unit weights
    W[2] = np.float32(0.5)                       # one value: nothing to lose
    W[3] = np.round(W[3] * 50) / 50              # few distinct values
    got = ctx.kmeans_optimal(dev(W), dev(S))
    table = ctx.error_table(dev(W), dev(S))["E"]
    torch.cuda.synchronize()
    got, table = got.cpu().numpy(), table.cpu().numpy()
    ref = oracle.kmeans_optimal_table(W, S)
    close, scale = _optimal_close(got, ref, W, S)
    assert np.all(close)
    assert np.all(got[2] <= 1e-12 * scale[2]) and np.all(np.diff(got, axis=1) <= 1e-12 * scale)
    assert np.all(got <= table * (1 + 1e-9) + 1e-12 * scale)


def test_optimal_clustering_error_scaled_inputs_and_bit_subset(ctx):
    W, S = skim_synth.make_ws_small(77, 16, 300)
    rng = np.random.default_rng(5)
    alpha = rng.uniform(0.5, 2.0, 300).astype(np.float32)
    got = ctx.kmeans_optimal(dev(W), dev(S), alpha=dev(alpha), bmin=2, bmax=3)
    torch.cuda.synchronize()
    ref = oracle.kmeans_optimal_table(W, S, alpha=alpha, bmin=2, bmax=3)
    assert got.shape == (16, 2) and np.all(_optimal_close(got.cpu().numpy(), ref, W, S, alpha)[0])


@pytest.mark.parametrize("m,bmax", [(14000, 1), (16400, 2)])
def test_optimal_clustering_error_long_rows(ctx, m, bmax):
    """Rows too long for the cuts to sit in LDS (they move to the caller's scratch), and rows sorted in two halves."""
    W, S = skim_synth.make_ws_small(m, 2, m, dup_frac=0.02)
    got = ctx.kmeans_optimal(dev(W), dev(S), bmin=1, bmax=bmax)
    torch.cuda.synchronize()
    ref = oracle.kmeans_optimal_table(W, S, bmin=1, bmax=bmax)
    close, _ = _optimal_close(got.cpu().numpy(), ref, W, S)
    assert np.all(close)


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes_and_flavours(ctx, seed):
    """Seeded sweep over combinations the targeted tests cover one at a time: row count (odd and even: two rows
    share a wavefront), ragged length, duplicated values, zero sensitivities, heavy elements, column scaling,
    iteration count and bit range."""
    rng = np.random.default_rng(9000 + seed)
    n = int(rng.integers(1, 48))
    m = int(rng.choice([16, 31, 64, 100, 333, 1024, 1500, 3001, 5000]))
    W, S = skim_synth.make_ws_small(500 + seed, n, m, dup_frac=float(rng.choice([0.0, 0.1, 0.5])),
                                    zero_s_frac=float(rng.choice([0.0, 0.2, 0.9])))
    if seed % 3 == 0:
        S[np.arange(n), rng.integers(0, m, n)] = 1e8                 # one element carries the mass
    if seed % 4 == 1:
        S[rng.integers(0, n)] = 0.0                                  # a row without mass
    alpha = rng.uniform(0.5, 2.0, m).astype(np.float32) if seed % 2 else None
    bmin = int(rng.integers(1, 4))
    bmax = int(rng.integers(bmin, 5))
    iters = int(rng.choice([1, 3, 30]))
    ref, out, excused = check_table(ctx, W, S, alpha=alpha, iters=iters, bmin=bmin, bmax=bmax)
    assert excused <= 2
    bits = rng.integers(1, 5, n).astype(np.uint8)
    check_rows(ctx, W, S, bits, alpha=alpha, iters=iters)


# (the last piece of 4 or 8 keys partly filled; 251, 256, 513 and 750 pieces: the search tree with and without a fourth level; two rows a
# workgroup, the last one alone; rows in pieces of 4 and of 8 keys)
@pytest.mark.parametrize("m,n,tiled,piece", [(1003, 41, 6600, 4), (1024, 40, 6600, 4), (2050, 41, 1700, 4), (3000, 900, 1100, 8),
                                             (4100, 37, 600, 4)])
def test_rows_kept_in_lds_agree_with_the_iterations_over_global_memory(ctx, m, n, tiled, piece):
    """A small matrix has its rows in LDS while they iterate, a larger one does not: the same rows in either.  Bounds
    (assignments) are equal; sums are taken in another order: centroids within 1e-13 of the row's largest weight times the number
    of iterations, errors within 1e-13 of the row's second moment."""
    rng = np.random.default_rng(m)
    W = (rng.standard_normal((n, m)) * 0.02).astype(np.float32)
    W = np.where(rng.random((n, m)) < 0.005, W * 10, W).astype(np.float32)
    S = (rng.standard_t(3, (n, m)) ** 2).astype(np.float32)
    W[1] = torch.from_numpy(W[1]).to(torch.bfloat16).float().numpy()        # every value many times
    W[2], S[2] = np.concatenate([W[2, : m // 2], -W[2, : m - m // 2]]), 1.0  # midpoints that cancel
    W[3] = 0.25                                                              # one value
    W[4] = np.where(np.arange(m) % 3 == 0, 1.0, -1.0)
    S[5] = 0.0
    S[6] = np.where(np.arange(m) % 50 == 0, S[6], 0.0)                       # clusters without mass
    big = np.float32(np.finfo(np.float32).max)
    W[7] = rng.uniform(-1, 1, m).astype(np.float32) * big
    W[7, ::100] = big
    W[8] = rng.random(m).astype(np.float32) * np.float32(1e-38)
    S[9] = np.float32(10.0) ** rng.integers(-18, 6, m)
    Wd, Sd = dev(W), dev(S)
    reps = -(-tiled // n)
    assert [ctx.lib.skim_cluster_pieces(ctx.h, ctypes.c_int64(k), ctypes.c_int64(m)) for k in (n, reps * n)] == [piece, 0]
    Wt, St = Wd.repeat(reps, 1), Sd.repeat(reps, 1)
    bits = torch.from_numpy(rng.integers(1, 5, n).astype(np.uint8)).cuda()
    few, many = ctx.error_table(Wd, Sd), ctx.error_table(Wt, St)
    rows_few, rows_many = ctx.cluster_rows(Wd, Sd, bits), ctx.cluster_rows(Wt, St, bits.repeat(reps))
    torch.cuda.synchronize()
    assert torch.equal(few["upper_all"], many["upper_all"][:n]) and torch.equal(few["upper_all"], many["upper_all"][-n:])
    assert torch.equal(rows_few["labels"], rows_many["labels"][:n])
    w, s = Wd.double(), Sd.double()
    s = torch.where(s.sum(1, keepdim=True) > 0, s, torch.ones_like(s))
    scale, moment = w.abs().amax(1, keepdim=True), (s * w * w).sum(1, keepdim=True)
    assert bool(((few["centroids_all"] - many["centroids_all"][:n]).abs() <= 3e-12 * scale).all())
    assert bool(((few["E"] - many["E"][:n]).abs() <= 1e-13 * moment).all())
    assert bool(((rows_few["centroids"] - rows_many["centroids"][:n]).abs() <= 3e-12 * scale).all())


@pytest.mark.parametrize("n,m", [(2100, 4096), (2100, 4095), (700, 8200), (5000, 520), (600, 12287), (3, 4000)])
def test_rows_shared_out_by_claims_or_in_fixed_shares(ctx, n, m):
    """Many and few rows a workgroup, 16-byte and 4-byte loads with 8, 12 and 16 slots: every call after the first
    finds the counter of the units as the first did, and a row's thresholds do not depend on the others.  Its centroids and errors do in
    their last digits, where the number of rows decides how the iterations add up (bounds as in the test above)."""
    W, S = skim_synth.make_ws_small(n, min(n, 300), m)
    reps = -(-n // len(W))
    Wd, Sd = dev(W).repeat(reps, 1)[:n].contiguous(), dev(S).repeat(reps, 1)[:n].contiguous()
    first = ctx.error_table(Wd, Sd)
    alone = ctx.error_table(Wd[:64].contiguous(), Sd[:64].contiguous())
    for _ in range(2):
        again = ctx.error_table(Wd, Sd)
        assert all(torch.equal(first[k], again[k]) for k in ("E", "centroids_all", "upper_all"))
    k = min(n, 64)
    assert torch.equal(first["upper_all"][:k], alone["upper_all"][:k])
    assert torch.equal(first["upper_all"], first["upper_all"][:300].repeat(reps, 1)[:n])
    w, s = Wd[:k].double(), Sd[:k].double()
    scale, moment = w.abs().amax(1, keepdim=True), (s * w * w).sum(1, keepdim=True)
    assert bool(((first["centroids_all"][:k] - alone["centroids_all"][:k]).abs() <= 3e-12 * scale).all())
    assert bool(((first["E"][:k] - alone["E"][:k]).abs() <= 1e-13 * moment).all())


# (pieces of 4 keys with three and four levels of the search tree, pieces of 8; even and odd rows of a workgroup)
@pytest.mark.parametrize("n,m,tiled", [(41, 512, 41), (40, 1003, 6600), (7, 3000, 1100), (5, 6007, 600), (5, 13001, 5)])
def test_clusters_of_tiny_mass_beside_a_heavy_element(ctx, n, m, tiled):
    """Rows whose sensitivities differ by up to 1e34, kept in LDS and (with more of them, or longer ones) not: the light clusters are
    smaller than the last digit of the running sums' low word where that holds something in between, and their sums must not come from
    a difference of two of those.  Against the oracle."""
    rng = np.random.default_rng(m)
    W, S = skim_synth.make_ws_small(77 + m, n, m)
    S = S + np.float32(0.01)
    order = np.argsort(W, axis=1)
    for i in range(n):
        heavy = order[i, rng.integers(m // 4, 3 * m // 4)]
        if i % 4 == 0:                      # heavy, in between, light
            S[i, heavy] = 1e32
            S[i, order[i, : 32]] *= np.float32(1e17)
        elif i % 4 == 1:
            S[i] *= np.float32(1e-12)
            S[i, order[i, m // 2: m // 2 + 16]] = rng.uniform(1e20, 2e20, 16)
            S[i, order[i, : m // 8]] *= np.float32(1e16)
        elif i % 4 == 2:                    # everything below the median light, the rest of many magnitudes
            S[i, order[i, : m // 2]] *= np.float32(1e-34)
            S[i, order[i, m // 2:]] = np.float32(10.0) ** rng.uniform(-24, 6, m - m // 2)
        else:                               # 1e-6 of everything, and keys without mass
            S[i, heavy] = 1e9
            S[i, rng.random(m) < 0.3] = 0.0
    _, _, excused = check_table(ctx, W, S)
    assert excused <= n // 8
    check_rows(ctx, W, S, rng.integers(1, 5, n).astype(np.uint8))
    reps = -(-tiled // n)
    check_table(ctx, np.tile(W, (reps, 1)), np.tile(S, (reps, 1)))


# (rows in LDS in pieces of 4 and of 8 keys, over global memory with running sums of 4 and of 16 chunks: with four wavefronts for the errors, the
# last of them without keys; one wavefront; an odd number of rows; widths that are flagged and widths that are not)
@pytest.mark.parametrize("n,m", [(5, 520), (41, 2050), (900, 3000), (3, 9001), (5, 20000), (2601, 4700), (1601, 17000)])
def test_errors_of_rows_of_few_values(ctx, n, m):
    """Rows of 3 or 12 distinct values, whose errors drown in the cancellation of the second moments at some widths or all: every entry is the sum of
    s (w - c)^2 over the row with the centroids and thresholds of the same call, to 1e-12."""
    gen = torch.Generator(device="cuda").manual_seed(m)
    values = torch.randn((n, 12), device="cuda", generator=gen)
    values[::2, 3:] = values[::2, :1]
    W = values.gather(1, torch.randint(0, 12, (n, m), device="cuda", generator=gen))
    W[1] += torch.randn(m, device="cuda", generator=gen)           # one ordinary row
    S = torch.randn((n, m), device="cuda", generator=gen).square()
    out = ctx.error_table(W, S)
    w, s = W.double(), S.double()
    for b in range(1, 5):
        sl = slice((1 << b) - 2, (2 << b) - 2)
        best = torch.full_like(W, float("inf"))
        c = torch.zeros_like(w)
        for up, ck in zip(out["upper_all"][:, sl].T, out["centroids_all"][:, sl].T):
            closer = (up[:, None] >= W) & (up[:, None] < best)
            best = torch.where(closer, up[:, None], best)
            c = torch.where(closer, ck[:, None], c)
        ref = (s * (w - c) ** 2).sum(1)
        # (the second moments serve from 1e-9 of them up and are good to 1e-16 of themselves, a few times over)
        ok = (out["E"][:, b - 1] - ref).abs() <= torch.where(ref >= 0.99e-9 * (s * w * w).sum(1), 1e-6 * ref, 1e-12 * ref)
        assert bool(ok.all()), f"b={b}: rows {torch.nonzero(~ok).flatten()[:5].tolist()}"
