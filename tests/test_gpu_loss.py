"""GPU parity: layer loss tr(dW H dW^T), scale gradient and Adam step against the CPU oracle.

Bar: loss, per-row loss, gradient and updated alpha within 1e-5
relative.  The contraction runs on the matrix cores with every float32
operand scaled and cut into two binary16 pieces and float32 accumulation, the diagonal of H in float64; the
oracle is float64 throughout.  Parity is per call on identical inputs: the
oracle is fed the same W, S, H, labels and alpha as the GPU.
"""
import numpy as np
import pytest
import torch

import oracle
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


def make_case(seed, n, m, K, N=None, with_alpha=True):
    W, S = skim_synth.make_ws_small(seed, n, m)
    S = S + np.float32(0.01)
    rng = np.random.default_rng(seed)
    labels = rng.integers(0, K, (n, m)).astype(np.uint8)
    H = skim_synth.make_h_host(3, N or 4 * m, m)
    H = ((H + H.T) / 2).astype(np.float32)
    al = skim_synth.make_alpha(seed, m) if with_alpha else None
    return W, S, labels, H, al


# (tiles of 256 x 256: widths that leave the last column tile part empty, rows that leave the last row tile part empty; one
# and several column blocks; up to 256 columns one wavefront takes a row)
@pytest.mark.parametrize("n,m,K", [(1, 16, 2), (37, 48, 4), (130, 144, 8), (257, 272, 16), (128, 512, 16), (300, 1024, 8),
                                   (70, 160, 8), (260, 416, 16)])
@pytest.mark.parametrize("with_alpha", [False, True])
def test_layer_loss_matches_oracle(ctx, n, m, K, with_alpha):
    W, S, labels, H, al = make_case(n + m, n, m, K, with_alpha=with_alpha)
    out = ctx.layer_loss(dev(W), dev(S), dev(H), dev(labels), alpha=None if al is None else dev(al))
    torch.cuda.synchronize()
    c, D = oracle.centroids_from_labels(W, S, labels, al)
    ref = oracle.layer_loss(W, H, labels, c, al)
    assert out["loss"].item() == pytest.approx(ref["loss"], rel=RTOL)
    got = out["row_loss"].cpu().numpy()
    assert np.all(np.abs(got - ref["row_loss"]) <= RTOL * np.abs(ref["row_loss"]) + 1e-9 * ref["loss"] / n)


def test_layer_loss_identity_and_diagonal_hessian(ctx):
    n, m = 64, 256
    W, S, labels, H, al = make_case(5, n, m, 8)
    c, D = oracle.centroids_from_labels(W, S, labels, al)
    dWd = W.astype(np.float64) - al.astype(np.float64)[None, :] * np.take_along_axis(c, labels.astype(np.int64), 1)
    out = ctx.layer_loss(dev(W), dev(S), dev(np.eye(m, dtype=np.float32)), dev(labels), alpha=dev(al))
    torch.cuda.synchronize()
    assert out["loss"].item() == pytest.approx((dWd ** 2).sum(), rel=RTOL)
    h = np.random.default_rng(0).uniform(0.5, 2, m).astype(np.float32)
    out = ctx.layer_loss(dev(W), dev(S), dev(np.diag(h)), dev(labels), alpha=dev(al))
    torch.cuda.synchronize()
    np.testing.assert_allclose(out["row_loss"].cpu().numpy(), (h.astype(np.float64)[None, :] * dWd ** 2).sum(1), rtol=RTOL)


@pytest.mark.parametrize("n,m,K", [(5, 32, 4), (40, 144, 8), (130, 512, 16), (33, 160, 8)])
@pytest.mark.parametrize("t_step", [1, 41])
def test_scale_step_matches_oracle(ctx, gpu_lib, n, m, K, t_step):
    W, S, labels, H, al = make_case(100 + n, n, m, K)
    rng = np.random.default_rng(n)
    m1 = (rng.standard_normal(m) * 1e-3).astype(np.float32) if t_step > 1 else np.zeros(m, np.float32)
    m2 = (rng.uniform(0, 1e-6, m)).astype(np.float32) if t_step > 1 else np.zeros(m, np.float32)
    d_al, d_m1, d_m2 = dev(al), dev(m1), dev(m2)
    out = ctx.scale_step(dev(W), dev(S), dev(H), dev(labels), d_al, d_m1, d_m2, t_step)
    torch.cuda.synchronize()
    ref = oracle.scale_grad(W, S, H, labels, al)
    assert out["loss_before"].item() == pytest.approx(ref["loss"], rel=RTOL)
    g = out["grad"].cpu().numpy().astype(np.float64)
    gscale = np.abs(ref["grad"]).max()
    assert np.all(np.abs(g - ref["grad"]) <= RTOL * np.abs(ref["grad"]) + 1e-6 * gscale)
    # optimiser step on the GPU's own gradient (identical inputs on both sides)
    # the ABI carries the hyper-parameters as float32: the oracle gets the same rounded values
    f32 = lambda x: float(np.float32(x))
    a_ref, m1_ref, m2_ref = oracle.adam_step(al, m1, m2, g, t_step, lr0=f32(0.01), beta1=f32(0.9), beta2=f32(0.999),
                                             eps=f32(1e-8), decay=f32(0.5), decay_every=40)
    np.testing.assert_allclose(d_al.cpu().numpy(), a_ref, rtol=RTOL)
    np.testing.assert_allclose(d_m1.cpu().numpy(), m1_ref, rtol=RTOL, atol=1e-6 * np.abs(m1_ref).max())
    np.testing.assert_allclose(d_m2.cpu().numpy(), m2_ref, rtol=RTOL, atol=1e-6 * np.abs(m2_ref).max())


def test_loss_after_clustering_equals_sdiag_error_when_hessian_is_diagonal(ctx):
    """With H = diag(s_i) the L-full error of a row is its S-diag error; here S is shared by
    all rows so that one H serves every row (ties Sec. 3.3 and 3.4 together end to end)."""
    n, m = 32, 512
    W, _ = skim_synth.make_ws_small(11, n, m)
    s_row = (np.random.default_rng(1).standard_t(3, m) ** 2).astype(np.float32)
    S = np.ascontiguousarray(np.broadcast_to(s_row, (n, m)))
    bits = np.full(n, 3, np.uint8)
    cr = ctx.cluster_rows(dev(W), dev(S), dev(bits))
    out = ctx.layer_loss(dev(W), dev(S), dev(np.diag(s_row)), cr["labels"])
    torch.cuda.synchronize()
    np.testing.assert_allclose(out["row_loss"].cpu().numpy(), cr["err"].cpu().numpy(), rtol=1e-5)


def test_loss_argument_errors(ctx, gpu_lib):
    W, S, labels, H, al = make_case(1, 4, 24, 2)     # m not a multiple of 16
    with pytest.raises(gpu_lib.SkimError):
        ctx.layer_loss(dev(W), dev(S), dev(H), dev(labels))


@pytest.mark.parametrize("n,m,with_alpha,zero_s", [(40, 144, False, 0.0), (41, 256, True, 0.0), (130, 512, True, 0.0), (64, 1024, True, 0.0),
                                                   (48, 144, False, 0.9), (48, 272, True, 0.97)])
def test_lfull_error_table_matches_oracle(ctx, n, m, with_alpha, zero_s):
    """Error pre-recording with the layer-wise error: every (row, bit width) entry against the oracle
    (clustering + naive float64 dW H dW^T); rows in which the oracle met a near-tie are excused.  With most
    sensitivities zero some clusters hold members without mass: their centroid is the one the clustering kept."""
    W, S = skim_synth.make_ws_small(21, n, m, zero_s_frac=zero_s)
    H = skim_synth.make_h_host(3, 4 * m, m)
    al = skim_synth.make_alpha(3, m) if with_alpha else None
    ref = oracle.error_table_lfull(W, S, H, alpha=al, count_near=True)
    sd = oracle.error_table(W, S, alpha=al)
    out = ctx.error_table_lfull(dev(W), dev(S), dev(H), alpha=None if al is None else dev(al))
    torch.cuda.synchronize()
    clean = ref["near_rows"] == 0
    assert clean.sum() >= n - 4
    got = out["E_full"].cpu().numpy()
    np.testing.assert_allclose(got[clean], ref["E"][clean], rtol=RTOL)
    np.testing.assert_allclose(out["E"].cpu().numpy()[clean], sd["E"][clean], rtol=RTOL)
    # the S-diag table of the same call equals the plain entry point's, bit for bit
    plain = ctx.error_table(dev(W), dev(S), alpha=None if al is None else dev(al))
    torch.cuda.synchronize()
    assert torch.equal(plain["E"], out["E"]) and torch.equal(plain["upper_all"], out["upper_all"])


def test_train_scale_is_the_composition_of_its_steps_and_tracks_the_oracle(ctx, gpu_lib):
    """skim_train_scale against (a) the same sequence of library calls made one by one: bit-exact; (b) the
    oracle's free-running Alg. 2 on a small, well-conditioned layer: loss trace and alpha within 1e-4 over
    30 steps (per-step parity at 1e-5 is covered by test_scale_step_matches_oracle; a free-running optimiser
    amplifies rounding differences of the fp32 contraction, hence the looser bound here)."""
    n, m = 48, 144
    W, S = skim_synth.make_ws_small(41, n, m)
    S = S + np.float32(0.05)
    H = skim_synth.make_h_host(3, 4 * m, m)
    bits_h = np.full(n, 3, np.uint8)
    Wd, Sd, Hd, bd = dev(W), dev(S), dev(H), dev(bits_h)
    steps = 30
    alpha = torch.ones(m, device="cuda")
    am, av = torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda")
    out = ctx.train_scale(Wd, Sd, Hd, bd, alpha, am, av, steps=steps, outer=2)
    torch.cuda.synchronize()
    # (a) manual composition
    a2 = torch.ones(m, device="cuda")
    m2, v2 = torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda")
    trace = []
    t = 1
    for _ in range(2):
        cr = ctx.cluster_rows(Wd, Sd, bd, alpha=a2)
        for _k in range(steps):
            o = ctx.scale_step(Wd, Sd, Hd, cr["labels"], a2, m2, v2, t, want_grad=False)
            trace.append(o["loss_before"].clone())
            t += 1
    ll = ctx.layer_loss(Wd, Sd, Hd, cr["labels"], alpha=a2)
    trace.append(ll["loss"].clone())
    torch.cuda.synchronize()
    assert torch.equal(alpha, a2) and torch.equal(am, m2) and torch.equal(av, v2)
    assert torch.equal(out["labels"], cr["labels"])
    assert torch.equal(out["loss_trace"], torch.cat([x.reshape(1) for x in trace]))
    c_ref, _ = oracle.centroids_from_labels(W, S, out["labels"].cpu().numpy(), alpha.cpu().numpy())
    np.testing.assert_allclose(out["centroids"].cpu().numpy(), c_ref, rtol=RTOL, atol=1e-12)
    # (b) oracle, free running, one round
    alpha = torch.ones(m, device="cuda")
    am, av = torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda")
    out1 = ctx.train_scale(Wd, Sd, Hd, bd, alpha, am, av, steps=steps)
    torch.cuda.synchronize()
    f32 = lambda x: float(np.float32(x))
    ref = oracle.train_scale(W, S, H, bits_h, np.ones(m, np.float32), steps=steps, lr0=f32(0.01), beta1=f32(0.9),
                             beta2=f32(0.999), eps=f32(1e-8), decay=f32(0.5), decay_every=40)
    np.testing.assert_allclose(out1["loss_trace"].cpu().numpy(), ref["loss_trace"], rtol=1e-4)
    np.testing.assert_allclose(alpha.cpu().numpy(), ref["alpha"], rtol=1e-4)
    assert ref["loss_trace"][-1] < ref["loss_trace"][0]


@pytest.mark.parametrize("N,m", [(40, 12), (300, 130), (1000, 256), (4096, 640),
                                 # wide layers, summed in longer chunks: a last tile of 8 columns and a
                                 # short last slice of activations; two accumulation chunks; a tile count that is
                                 # no multiple of 8; few activations; the narrowest such layer
                                 (200, 3592), (8200, 3840), (128, 4096), (300, 2568)])
def test_hessian_from_activations_matches_oracle(ctx, N, m):
    """H = X^T X / N from bfloat16 activations against the float64 definition: every entry within 1e-5 of the
    entry's natural scale sqrt(H_jj H_ll) (float32 accumulation within a chunk of activations; across chunks
    float64, or for wide layers float32 inside a workgroup's share -- at most a few dozen additions)."""
    X = np.concatenate(list(skim_synth.make_x(3, N, m)))        # float32 values that are exact in bfloat16
    ref = oracle.hessian_from_activations(X).astype(np.float64)
    Xb = torch.from_numpy(X).cuda().to(torch.bfloat16)
    assert torch.equal(Xb.float().cpu(), torch.from_numpy(X))
    H = ctx.hessian_from_activations(Xb)
    torch.cuda.synchronize()
    got = H.cpu().numpy().astype(np.float64)
    scale = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    assert np.all(np.abs(got - ref) <= RTOL * scale), f"max scaled diff {(np.abs(got - ref) / scale).max():.3e}"
    assert torch.equal(H, H.T.contiguous())


@pytest.mark.parametrize("N,m,workspace", [
    (31, 2, "full"), (257, 514, "full"), (4100, 1030, "full"),      # widths that no 16-byte load divides; a short last stage
    (520, 5890, "full"),                     # more tiles than workgroups: one round of whole tiles, then split ones
    (16500, 300, "full"), (16500, 300, "one slot per tile"), (16500, 300, "none")])   # split; too little scratch for that; none
def test_hessian_plans_match_oracle(gpu_lib, N, m, workspace):
    """The ways the activations of a tile are shared out, against the float64 definition (bound as in
    test_hessian_from_activations_matches_oracle)."""
    X = np.concatenate(list(skim_synth.make_x(3, N, m)))
    ref = oracle.hessian_from_activations(X).astype(np.float64)
    Xb = torch.from_numpy(X).cuda().to(torch.bfloat16)
    c = gpu_lib.Context(0)
    H = torch.full((m, m), float("nan"), device="cuda")
    if workspace == "full":
        c.hessian_from_activations(Xb, out=H)
    else:
        tiles = ((m + 255) // 256) * ((m + 255) // 256 + 1) // 2
        ws = torch.empty(tiles * 65536, device="cuda")
        if workspace != "none":
            c._check(c.lib.skim_set_workspace(c.h, ws.data_ptr(), ws.numel() * 4))
        c._check(c.lib.skim_hessian_from_activations(c.h, Xb.data_ptr(), N, m, H.data_ptr()))
    torch.cuda.synchronize()
    got = H.cpu().numpy().astype(np.float64)
    scale = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    assert np.all(np.abs(got - ref) <= RTOL * scale), f"max scaled diff {(np.abs(got - ref) / scale).max():.3e}"
    assert torch.equal(H, H.T.contiguous())
    c.close()


@pytest.mark.parametrize("n,m,K", [
    (3, 4112, 16), (9, 11280, 8),       # rows of 5 .. 11 steps kept in registers, longer ones read again; row groups part empty
    (7, 256, 16), (1030, 32, 8),        # one wavefront a row, H cut in the same launch; a workgroup of the loss for every tile
    (70, 2064, 4),                      # few tiles: every one split; a last stage of 16 columns past a multiple of 32
    (8200, 2080, 16)])                  # more tiles than workgroups: one round of whole tiles, then split ones
def test_loss_and_scale_step_on_other_tile_plans(ctx, n, m, K):
    """Shapes on which the contraction shares its tiles out differently from the small ones above, and the row kernel keeps
    its columns differently: loss, row losses and gradient against the oracle (bounds as above)."""
    W, S, labels, H, al = make_case(n + m, n, m, K, N=64)
    ref = oracle.scale_grad(W, S, H, labels, al)
    out = ctx.layer_loss(dev(W), dev(S), dev(H), dev(labels), alpha=dev(al))
    step = ctx.scale_step(dev(W), dev(S), dev(H), dev(labels), dev(al), dev(np.zeros(m, np.float32)), dev(np.zeros(m, np.float32)), 1)
    torch.cuda.synchronize()
    assert out["loss"].item() == pytest.approx(ref["loss"], rel=RTOL)
    assert step["loss_before"].item() == pytest.approx(ref["loss"], rel=RTOL)
    rl = oracle.layer_loss(W, H, labels, ref["centroids"], al)["row_loss"]
    assert np.all(np.abs(out["row_loss"].cpu().numpy() - rl) <= RTOL * np.abs(rl) + 1e-9 * ref["loss"] / n)
    g = step["grad"].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(g - ref["grad"]) <= RTOL * np.abs(ref["grad"]) + 1e-6 * np.abs(ref["grad"]).max())


def test_training_and_lfull_table_run_without_the_partial_tiles(gpu_lib):
    """The partial tiles of the contraction are optional: a workspace that lacks just them is accepted, and the results are
    those of the full one up to the order of float32 sums (1e-6 over the terms of a row, times the steps)."""
    n, m = 70, 2064                                  # 9 tiles of 129 stages, each cut into at most 8 parts of 16 or more
    W, S, labels, H, al = make_case(7, n, m, 8, N=64)
    Wd, Sd, Hd, bits = dev(W), dev(S), dev(H), dev(np.full(n, 3, np.uint8))
    results = []
    for short in (0, 9 * 8 * 256 * 256 * 4):
        c = gpu_lib.Context(0)
        size = c.workspace_bytes(n, m) - short
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        c._check(c.lib.skim_set_workspace(c.h, ws.data_ptr(), size))
        c.ensure_workspace = lambda n, m: None
        alpha, am, av = dev(al), dev(np.zeros(m, np.float32)), dev(np.zeros(m, np.float32))
        tr = c.train_scale(Wd, Sd, Hd, bits, alpha, am, av, steps=3)
        tab = c.error_table_lfull(Wd, Sd, Hd)
        torch.cuda.synchronize()
        results.append((tr["loss_trace"].cpu().numpy(), alpha.cpu().numpy(), tab["E_full"].cpu().numpy()))
        c.close()
    for full, least in zip(*results):
        np.testing.assert_allclose(least, full, rtol=RTOL)


@pytest.mark.parametrize("n,m", [(5, 16), (33, 112), (40, 272), (70, 544), (300, 1040)])
def test_loss_of_a_hessian_that_is_not_symmetric(ctx, n, m):
    """The loss takes half of the products, and must not take one triangle of H for the other: dW_i H dW_i^T for any H,
    against float64 (5e-7 of the sum of the products' magnitudes: float32 sums of up to 1040 terms, as seen 2e-8), and
    the steps of a training and its last loss alike."""
    W, S, labels, _, al = make_case(n * m, n, m, 8)
    H = np.random.default_rng(m).standard_normal((m, m)).astype(np.float32)
    H[:, : m // 3] *= 30.0
    out = ctx.layer_loss(dev(W), dev(S), dev(H), dev(labels), alpha=dev(al))
    step = ctx.scale_step(dev(W), dev(S), dev(H), dev(labels), dev(al), dev(np.zeros(m, np.float32)), dev(np.zeros(m, np.float32)), 1)
    alpha = dev(al)
    tr = ctx.train_scale(dev(W), dev(S), dev(H), dev(np.full(n, 3, np.uint8)), alpha, dev(np.zeros(m, np.float32)),
                         dev(np.zeros(m, np.float32)), steps=1)
    torch.cuda.synchronize()
    c, _ = oracle.centroids_from_labels(W, S, labels, al)

    def rows(lab, c, al):
        dW = W.astype(np.float64) - al.astype(np.float64)[None, :] * np.take_along_axis(c, lab.astype(np.int64), 1)
        return ((dW @ H.astype(np.float64)) * dW).sum(1), ((np.abs(dW) @ np.abs(H).astype(np.float64)) * np.abs(dW)).sum(1)

    ref, mag = rows(labels, c, al)
    assert np.all(np.abs(out["row_loss"].cpu().numpy() - ref) <= 5e-7 * mag)
    for loss in (out["loss"], step["loss_before"]):
        assert abs(loss.item() - ref.sum()) <= 5e-7 * mag.sum()
    if m % 32 != 0 or m < 128:          # there the step's P is dW H for any H
        g, g_ref = step["grad"].cpu().numpy().astype(np.float64), oracle.scale_grad(W, S, H, labels, al)["grad"]
        assert np.all(np.abs(g - g_ref) <= 1e-5 * np.abs(g_ref).max())
    ref, mag = rows(tr["labels"].cpu().numpy(), tr["centroids"].cpu().numpy(), alpha.cpu().numpy())
    assert abs(tr["loss_trace"][-1].item() - ref.sum()) <= 5e-7 * mag.sum()


@pytest.mark.parametrize("n,m", [(33, 112), (40, 272)])
def test_lfull_table_of_a_hessian_that_is_not_symmetric(ctx, n, m):
    W, S = skim_synth.make_ws_small(5, n, m)
    H = np.random.default_rng(m).standard_normal((m, m)).astype(np.float32)
    Hs = ((H.astype(np.float64) + H.T) / 2)
    got = ctx.error_table_lfull(dev(W), dev(S), dev(H), bmin=2, bmax=3)["E_full"].cpu().numpy()
    sym = ctx.error_table_lfull(dev(W), dev(S), dev(Hs.astype(np.float32)), bmin=2, bmax=3)["E_full"].cpu().numpy()
    scale = np.abs(H).sum() / m * (W.astype(np.float64) ** 2).sum(1)[:, None]        # far above |dW| |H| |dW|
    assert np.all(np.abs(got - sym) <= 1e-6 * scale)


@pytest.mark.parametrize("m", [48, 112, 160])
def test_loss_with_entries_above_the_largest_bfloat16(ctx, m):
    """No piece of a finite float32 value may be infinity: float32 reaches 3.4028e38, bfloat16 3.3895e38, binary16 65504."""
    n = 20
    rng = np.random.default_rng(m)
    W = (rng.standard_normal((n, m)) * 1e-19).astype(np.float32)
    S = np.ones((n, m), np.float32)
    labels = rng.integers(0, 4, (n, m)).astype(np.uint8)
    H = np.diag(rng.choice([3.4028234e38, -3.4e38, 3.398e38, 3.3895e38, 1e38], m).astype(np.float32))
    out = ctx.layer_loss(dev(W), dev(S), dev(H), dev(labels))
    torch.cuda.synchronize()
    c, _ = oracle.centroids_from_labels(W, S, labels, None)
    dW = W.astype(np.float64) - np.take_along_axis(c, labels.astype(np.int64), 1)
    h = np.diag(H).astype(np.float64)[None, :]
    got = out["row_loss"].cpu().numpy()
    assert np.all(np.abs(got - (h * dW ** 2).sum(1)) <= 5e-7 * (np.abs(h) * dW ** 2).sum(1))


def hessian_reference(Xb):
    """X^T X / N in float64 on the device (operands contiguous), and the entries' scale sqrt(H_jj H_ll)."""
    N, m = Xb.shape
    H = torch.zeros((m, m), device="cuda", dtype=torch.float64)
    for r in range(0, N, 16384):
        x = Xb[r:r + 16384].double()
        H += x.T.contiguous() @ x
    H /= N
    d = H.diagonal().clone()
    return H, torch.sqrt(d[:, None] * d[None, :])


@pytest.mark.parametrize("N,m,scratch,bound", [
    (16384, 2048, True, 1.10e-7), (65536, 2560, True, 0.95e-7), (16384, 4098, True, 1.15e-7),      # pieces: one, several, whole tiles
    (4096, 512, False, 2.0e-7), (262144, 256, False, 0.85e-7)])                                    # float64 registers
def test_hessian_of_narrow_layers_adds_chunks_of_2048_in_float64(gpu_lib, N, m, scratch, bound):
    """Rows of up to 2560 columns (and wider ones whose rows are not whole 16-byte pieces): float32 sums run over 2048
    activations, the rest is float64.  rms error of the diagonal, whose sums only grow: at most 1.04e-7, 0.81e-7, 1.04e-7, 1.70e-7,
    0.73e-7 so; with chunks of 8192 or parts added up in float32 1.19e-7, 1.30e-7, 2.78e-7, 3.03e-7, 1.12e-7.  The sums of m
    columns agree to a few per cent between seeds; the bound lies between."""
    gen = torch.Generator(device="cuda").manual_seed(N + m)
    Xb = torch.randn((N, m), device="cuda", generator=gen).to(torch.bfloat16)
    ref, _ = hessian_reference(Xb)
    c = gpu_lib.Context(0)
    H = torch.empty((m, m), device="cuda")
    if scratch:
        c.hessian_from_activations(Xb, out=H)
    else:
        c._check(c.lib.skim_hessian_from_activations(c.h, Xb.data_ptr(), N, m, H.data_ptr()))
    err = H.double().diagonal() / ref.diagonal() - 1.0
    rms = float((err * err).mean().sqrt())
    assert rms <= bound, f"{rms:.3e}"
    c.close()


@pytest.mark.parametrize("N,m,offset,sizes", [
    (16500, 300, 0, (67 << 20, 13 << 20, 1 << 20, 0)),          # one pass, several, too little, none
    (70001, 514, 0, (256 << 20, 40 << 20, 16 << 20)),           # pieces; several passes with pieces
    (2100, 5890, 0, (200 << 20, 60 << 20, 30 << 20)),           # two groups of tiles; one pass, several; smaller groups
    (4200, 2816, 2, (160 << 20, 0)),                            # a wide layer whose rows start between 16-byte borders
    (1500, 5888, 0, (128 << 20, 80 << 20, 67 << 20, 64 << 20, 8 << 20))])    # a round of whole tiles and the rest together; apart; in H itself
def test_hessian_with_any_scratch(gpu_lib, N, m, offset, sizes):
    """Passes with running sums, groups of tiles and the kernel that needs no scratch, against float64: within 1e-6 of
    sqrt(H_jj H_ll) (chunks of 2048 of up to 128 roundings each: at most 3.8e-6, seen 4e-7)."""
    gen = torch.Generator(device="cuda").manual_seed(N + m)
    flat = torch.randn(N * m + offset, device="cuda", generator=gen).to(torch.bfloat16)
    Xb = flat[offset:].view(N, m)
    ref, scale = hessian_reference(Xb)
    c = gpu_lib.Context(0)
    for size in sizes:
        H = torch.full((m, m), float("nan"), device="cuda")
        block = torch.empty(max(size, 256), dtype=torch.uint8, device="cuda")
        c._check(c.lib.skim_hessian_from_activations_scratch(c.h, Xb.data_ptr(), N, m, H.data_ptr(), block.data_ptr() if size else None, size))
        worst = float(((H.double() - ref).abs() / scale).max())
        assert worst <= 1e-6, f"scratch {size}: {worst:.3e}"
        assert torch.equal(H, H.T.contiguous())
    c.close()


# (16 magnitudes a workgroup; one tile and several of the other kernel, the last ones partly empty; rows kept in registers and read again)
@pytest.mark.parametrize("n,m", [(5, 16), (70, 272), (33, 1040), (20, 4112), (5, 11280)])
def test_loss_of_channels_and_rows_of_very_different_magnitude(ctx, n, m):
    """The scales of the pieces: channels of H from 2^-30 to 2^30 with some that are dead, rows of W from 1e-30 to 1e15, one of zeros
    and one next to the subnormal numbers (dW is a float32 value: steps of 1.4e-45, 1.4e-9 of that row's), W within a row from 2^-12 to 1 times the largest.  Against float64, in units of the sum of the products'
    magnitudes: both operands of a product are off by 2^-23 of themselves at most and 2^-22 of it is dropped, 4.8e-7 if all
    of them conspired, and the float32 sums add 5e-8 at these widths."""
    gen = torch.Generator(device="cuda").manual_seed(m)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    X = normal(64, m)
    scale = torch.exp2(torch.randint(-15, 16, (m,), device="cuda", generator=gen).float())
    scale[:: 7] = 0.0
    X = X * scale
    H = X.T.contiguous() @ X
    H = ((H + H.T) / 2).contiguous()
    rows = torch.logspace(-30, 15, n, device="cuda")
    W = normal(n, m) * rows[:, None] * torch.exp2(-torch.randint(0, 13, (n, m), device="cuda", generator=gen).float())
    W[1] = 0.0
    W[2] = normal(m) * 1e-36
    S = torch.ones(n, m, device="cuda")
    labels = torch.randint(0, 4, (n, m), device="cuda", generator=gen, dtype=torch.uint8)
    out = ctx.layer_loss(W, S, H, labels)
    c, _ = oracle.centroids_from_labels(W.cpu().numpy(), S.cpu().numpy(), labels.cpu().numpy(), None)
    dW = W.double() - torch.from_numpy(c).cuda().gather(1, labels.long())
    Hd = H.double()
    ref, mag = ((dW @ Hd) * dW).sum(1), ((dW.abs() @ Hd.abs()) * dW.abs()).sum(1)
    err = (out["row_loss"] - ref).abs()
    assert bool((err <= 5.3e-7 * mag).all()), f"{float((err / mag.clamp_min(1e-300)).max()):.3e}"
    assert out["row_loss"][1].item() == 0.0
    # P and the gradient, with the rows in float32's range for products with H
    W = normal(n, m) * torch.exp2(-torch.randint(0, 13, (n, m), device="cuda", generator=gen).float())
    alpha = torch.exp(normal(m) * 0.1)
    step = ctx.scale_step(W, S, H, labels, alpha.clone(), torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda"), 1)
    a = alpha.double()
    wt, st = (W / alpha).double(), (alpha * alpha).double().expand(n, m)
    L = labels.long()
    D = torch.zeros(n, 16, device="cuda", dtype=torch.float64).scatter_add_(1, L, st.contiguous())
    c = torch.zeros_like(D).scatter_add_(1, L, st * wt) / D.clamp_min(1e-300)
    ck = c.gather(1, L)
    dW = W.double() - a * ck

    def gradient(P, s):         # s = 1: the sums themselves; the magnitudes of all terms otherwise
        f = (lambda x: x) if s else torch.abs
        R = torch.zeros_like(D).scatter_add_(1, L, f(P * a)) / D.clamp_min(1e-300)
        t = W.double() - 2 * a * ck
        return 2 * (f(P * ck) + R.gather(1, L) * f(t)).sum(0)

    g, mag = -gradient(dW @ Hd, True), gradient(dW.abs() @ Hd.abs(), False)
    assert bool(((step["grad"].double() - g).abs() <= 6e-7 * mag).all())
    assert abs(step["loss_before"].item() - float(((dW @ Hd) * dW).sum())) <= 6e-7 * float(((dW.abs() @ Hd.abs()) * dW.abs()).sum())


def gradient_terms(W, alpha, c, D, labels, dW, H, magnitudes=False):
    """Gradient with respect to alpha for unit sensitivities in float64 -- or, with magnitudes, the sum of the terms' magnitudes."""
    a, L = alpha.double(), labels.long()
    f = torch.abs if magnitudes else (lambda x: x)
    P = f(dW) @ f(H)
    ck = c.gather(1, L)
    R = torch.zeros_like(D).scatter_add_(1, L, f(P * a)) / D.clamp_min(1e-300)
    g = (f(P * ck) + R.gather(1, L) * f(W.double() - 2 * a * ck)).sum(0)
    return 2 * g if magnitudes else -2 * g


# (columns of H and rows of H for the columns of P; the scales from the kernel for short rows and from the one for long rows)
@pytest.mark.parametrize("n,m", [(3, 112), (2, 160), (5, 1040)])
@pytest.mark.parametrize("kind", ["strong channel", "strong column", "diagonal", "pairs", "infinite coupling"])
def test_gradient_of_channels_of_very_different_strength(ctx, n, m, kind):
    """A column of the gradient must keep its digits beside channels that are far stronger and that it is not coupled to: Adam
    divides every column by its own size.  One channel with 1e9 times the standard deviation of the others, one column of W 1e9 times the
    others, a diagonal H from 2^-60 to 2^60, pairs of coupled channels from 2^-15 to 1 with one outlier in every row, and a coupling
    that is infinite and belongs to two columns alone.  Channels of different strength share no cluster (the gradient through the
    centroids would join them), and the rows are few (their errors would cancel).  Against float64, in units of the
    sum of the terms' magnitudes: 6e-7 for the pieces and the sums as in the test above; below 2^-16 of its row's largest an entry
    of dW, weighed by its channel, is off by up to 2^-39 of that one, likewise a coupling: 2^-38 (with the scales' powers of two: 2^-36)."""
    gen = torch.Generator(device="cuda").manual_seed(n * m)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    X = normal(4 * m, m)
    H = X.T.contiguous() @ X / (4 * m)
    W, alpha = normal(n, m), torch.exp(normal(m) * 0.1)
    labels = torch.randint(0, 4, (n, m), device="cuda", generator=gen, dtype=torch.uint8)
    checked = torch.ones(m, device="cuda", dtype=torch.bool)
    if kind in ("strong channel", "strong column"):
        j = m // 3
        for k in (j, j + 1):
            H[k, :] = H[:, k] = 0.0
            H[k, k] = 1.0
        if kind == "strong channel":
            H[j, j] = 1e18
        if kind == "strong column":
            W[:, j] *= 1e9
        labels[:, j] = 4 + (torch.arange(n, device="cuda") & 1).to(torch.uint8)
        labels[:, j + 1] = labels[:, j]          # (of two members, so that its dW is not zero)
    elif kind == "diagonal":
        labels[:] = (torch.arange(m, device="cuda") % 16).to(torch.uint8)
        H = torch.diag(torch.exp2(8.0 * labels[0].float() - 60.0))
    elif kind == "pairs":
        labels[:] = (torch.arange(m, device="cuda") // 2 % 16).to(torch.uint8)
        s = torch.exp2(-labels[0].float())
        block = (torch.arange(m, device="cuda") // 2)[:, None] == (torch.arange(m, device="cuda") // 2)[None, :]
        H = torch.where(block, H + 0.5, torch.zeros_like(H)) * s[:, None] * s[None, :]
        W[torch.arange(n, device="cuda"), torch.arange(n, device="cuda") * 7 % m] *= 32.0
    H = ((H + H.T) / 2).contiguous()
    Hd = H.double()
    if kind == "infinite coupling":
        labels[:, 5] = labels[:, 40] = 6
        H[5, 40] = H[40, 5] = float("inf")
        checked[5] = checked[40] = False
    step = ctx.scale_step(W, torch.ones_like(W), H, labels, alpha.clone(), torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda"), 1)
    a, L = alpha.double(), labels.long()
    st = (alpha * alpha).double().expand(n, m).contiguous()
    D = torch.zeros(n, 16, device="cuda", dtype=torch.float64).scatter_add_(1, L, st)
    c = torch.zeros_like(D).scatter_add_(1, L, st * (W / alpha).double()) / D.clamp_min(1e-300)
    dW = W.double() - a * c.gather(1, L)
    g = gradient_terms(W, alpha, c, D, labels, dW, Hd)
    mag = gradient_terms(W, alpha, c, D, labels, dW, Hd, True)
    # the floor: entries of a row as large as its largest weighed one, couplings as large as the largest that their channels allow
    off = (Hd - torch.diag(Hd.diagonal())).abs()
    e = torch.sqrt(off.max(0).values)
    row = (dW.abs() * e).max(1).values
    coupled = (off > 0).double()
    floor = row[:, None] * (coupled.sum(0) * e)[None, :] * 2.0 ** -36
    ck = c.gather(1, L).abs()
    R = torch.zeros_like(D).scatter_add_(1, L, floor * a) / D.clamp_min(1e-300)
    floor = 2 * (floor * ck + R.gather(1, L) * (W.double() - 2 * a * c.gather(1, L)).abs()).sum(0)
    err = (step["grad"].double() - g).abs()
    bad = checked & ~(err <= 6e-7 * mag + floor)
    assert not bool(bad.any()), f"{int(bad.sum())} columns, worst {float((err / mag.clamp_min(1e-300))[bad].max()):.3e} of the terms' magnitudes"


@pytest.mark.parametrize("m,bound", [(512, 0.8e-7), (1552, 1.33e-7)])
def test_gradient_of_correlated_channels(ctx, m, bound):
    """Channels that share 8 common factors: the couplings outweigh the diagonal, and what two pieces lack of a float32 value is the
    same for every row.  2-norm of the gradient's error over six layers of 256 rows, relative to float64: 0.60e-7 and 1.20e-7; with three
    bfloat16 pieces and six products it was 1.08e-7 and 2.16e-7, with the diagonal among the two pieces 2.00e-7 and 1.47e-7 (the sums are
    made in a fixed order: no noise between runs)."""
    n, total = 256, 0.0
    for seed in range(6):
        gen = torch.Generator(device="cuda").manual_seed(seed)

        def normal(*shape):
            return torch.randn(shape, device="cuda", generator=gen)

        scale = torch.ones(m, device="cuda")
        scale[torch.randperm(m, device="cuda", generator=gen)[: m // 100]] = 20.0
        X = (normal(4096, m) * 0.55 + normal(4096, 8) @ normal(8, m)) * scale
        H = X.T.contiguous() @ X / 4096
        H = ((H + H.T) / 2).contiguous()
        W, alpha = normal(n, m) * 0.02, torch.exp(normal(m) * 0.1)
        S = normal(n, m).square() + 0.001
        labels = ctx.cluster_rows(W, S, torch.full((n,), 3, device="cuda", dtype=torch.uint8), alpha=alpha)["labels"]
        g = ctx.scale_step(W, S, H, labels, alpha.clone(), torch.zeros(m, device="cuda"), torch.zeros(m, device="cuda"), 1)["grad"].double()
        a, L = alpha.double(), labels.long()
        st = (S * alpha * alpha).double()
        D = torch.zeros(n, 16, device="cuda", dtype=torch.float64).scatter_add_(1, L, st)
        ck = (torch.zeros_like(D).scatter_add_(1, L, st * (W / alpha).double()) / D.clamp_min(1e-300)).gather(1, L)
        P = (W.double() - a * ck) @ H.double()
        R = (torch.zeros_like(D).scatter_add_(1, L, P * a) / D.clamp_min(1e-300)).gather(1, L)
        ref = -2 * (P * ck + R * S.double() * (W.double() - 2 * a * ck)).sum(0)
        total += float((g - ref).norm() / ref.norm()) ** 2
    assert (total / 6) ** 0.5 <= bound, f"{(total / 6) ** 0.5:.3e}"


@pytest.mark.parametrize("n,m", [(1, 16), (255, 48), (1025, 64), (2049, 272), (5000, 32), (20100, 16), (300, 4112)])
def test_total_of_the_row_losses(ctx, n, m):
    """Row losses added up in one workgroup with their pieces, or in a kernel of their own with four threads a row: the total is the sum of the
    rows' losses, which agree with float64 (5e-7 of the sum of the products' magnitudes, as above)."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((64, m), device="cuda", generator=gen)
    H = (X.T.contiguous() @ X).contiguous()
    H = ((H + H.T) / 2).contiguous()
    W = torch.randn((n, m), device="cuda", generator=gen)
    labels = torch.randint(0, 4, (n, m), device="cuda", generator=gen, dtype=torch.uint8)
    out = ctx.layer_loss(W, torch.ones_like(W), H, labels)
    L = labels.long()
    D = torch.zeros(n, 16, device="cuda", dtype=torch.float64).scatter_add_(1, L, torch.ones_like(W).double())
    dW = W.double() - (torch.zeros_like(D).scatter_add_(1, L, W.double()) / D.clamp_min(1.0)).gather(1, L)
    ref, mag = ((dW @ H.double()) * dW).sum(1), ((dW.abs() @ H.double().abs()) * dW.abs()).sum(1)
    assert bool(((out["row_loss"] - ref).abs() <= 5e-7 * mag).all())
    total = float(out["row_loss"].sum())
    assert abs(out["loss"].item() - total) <= 1e-13 * float(out["row_loss"].abs().sum())
