"""GPU parity of the routed global-attention layer against the fp64 oracle.

Every test runs the HIP path through the C ABI (paper_2609_23733_amd.vp) and
the oracle on the same seeded inputs, then compares:
  - mode-router logits: |diff| <= 1e-5 (fp32 GEMV of 1024 terms);
  - modes and buckets: bit-exact (inputs are generated with logit margins
    >= 1e-3, or planted saliencies >= 1e-3 away from the thresholds);
  - router outputs q_pool, s, C, mean: max |diff| <= 1e-4 * RMS;
  - Y: max |Y - Y_oracle| <= tol * RMS with tol = 1e-4 for fp32 operands and
    2e-2 for bf16 operands (the stated bounds), where RMS is the smaller of
    the head's own RMS and the RMS of the compared layer output over all
    heads, so that the check holds under either reading of "output RMS".
    When Y is stored as bf16 the bound adds the half-ulp of
    round-to-nearest-even, 2^-8 |Y_oracle|, elementwise.
"""
import math
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2609_23733_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def log(msg):
    sys.stdout.write("[gpu-case] %s\n" % msg)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_23733_amd import vp
    vp.load_library()


def run_gpu(x, rule=oracle.RULE_ARGMAX, y_dtype=None, act=0, pool=oracle.POOL_GATED,
            surr_variant=oracle.SURR_EQ7):
    from paper_2609_23733_amd import vp
    layer = vp.RoutedLayer(x, rule=rule, y_dtype=y_dtype, act=act, pool=pool,
                           surr_variant=surr_variant)
    layer.step()
    torch.cuda.synchronize()
    return layer


def rms(a):
    return float(np.sqrt(np.mean(np.square(a))))


def check_router(layer, ref, rule):
    st = layer.state
    for name, g, r in (("q_pool", st.q_pool, ref["q_pool"]), ("ctx", st.ctx, ref["C"]),
                       ("vmean", st.vmean, ref["mean"])):
        g = g.cpu().numpy().astype(np.float64)
        for h in range(g.shape[0]):
            err = np.abs(g[h] - r[h]).max()
            assert err <= 1e-4 * max(rms(r[h]), 1e-30), (name, h, err, rms(r[h]))
    s = st.score.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(s, ref["s"], rtol=1e-4)
    if rule in (oracle.RULE_ARGMAX, oracle.RULE_ARGMAX_BINARY) and ref["logits"] is not None:
        lg = layer.logits.cpu().numpy().astype(np.float64)
        assert np.abs(lg - ref["logits"]).max() <= 1e-5
    modes = layer.modes.cpu().numpy()
    np.testing.assert_array_equal(modes, ref["modes"])
    counts, lst = oracle.buckets(ref["modes"])
    b = layer.buckets.cpu().numpy()
    np.testing.assert_array_equal(b[:3], counts)
    np.testing.assert_array_equal(b[3:3 + len(lst)], lst)
    assert b[19] == 0


def check_y(Yg, Yo, dtype, y_bf16, heads=None, label=""):
    """Yg: GPU rows [R, H, d] (float64); Yo: oracle rows [R, H, d]."""
    tol = TOL[dtype]
    H = Yo.shape[1]
    heads = list(range(H) if heads is None else heads)
    layer_rms = rms(Yo[:, heads, :])
    worst = 0.0
    for h in heads:
        r = Yo[:, h, :]
        half_ulp = 2.0 ** -8 * np.abs(r) if y_bf16 else 0.0
        bound = tol * min(rms(r), layer_rms) + half_ulp
        err = np.abs(Yg[:, h, :] - r)
        ratio = float((err / np.maximum(bound, 1e-300)).max())
        worst = max(worst, ratio)
        assert (err <= bound).all(), "%s head %d: max err %.3e, rms %.3e (layer %.3e), " \
            "ratio %.3f" % (label, h, err.max(), rms(r), layer_rms, ratio)
    log("%s worst err/bound = %.3f" % (label, worst))


def oracle_layer(x, rule=oracle.RULE_ARGMAX, rows=None, full_rows_sel=None, act=0,
                 pool=oracle.POOL_GATED, surr_variant=oracle.SURR_EQ7):
    return oracle.routed_layer(x.Q, x.K, x.V, x.W, x.U, x.w, x.surr, u=x.u, Wr=x.Wr, br=x.br,
                               rule=rule, rows=rows, full_rows_sel=full_rows_sel, act=act,
                               pool=pool, surr_variant=surr_variant)


# ------------------------------------------------------------- small layers

@pytest.mark.parametrize("wl", ["s2_f32", "s8_bf16"])
def test_workload_layer_parity(wl):
    cfg = synth.WORKLOADS[wl]
    log("workload %s" % wl)
    x = synth.make_layer(cfg["S"], dtype=cfg["dtype"], n_full=cfg["n_full"], key=(1, 0),
                         qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    rows = None if cfg["S"] <= 2 else synth.sample_rows(x.N, 768, synth.derive_seed(1, 0, 20))
    ref = oracle_layer(x, rows=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    Yg = layer.Y.double().cpu().numpy()
    if rows is not None:
        Yg = Yg[rows]
    check_y(Yg, ref["Y"], cfg["dtype"], False, label=wl)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P", [1, 2, 63, 64, 65, 255, 257, 1000])
def test_ragged_token_counts(dtype, P):
    """Token counts around the 64-key and 256/128-query tiles, sharp inputs
    (attention far from uniform), every mode present."""
    log("ragged P=%d %s" % (P, dtype))
    modes = np.array([2, 1, 0, 2, 2, 1, 0, 0, 1, 2, 0, 1, 2, 0, 1, 2], np.uint8)
    x = synth.make_layer(1, P, dtype=dtype, key=(2, P), sharp=True, modes=modes,
                         qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], dtype, False, label="P=%d" % P)


@pytest.mark.parametrize("P", [15, 64, 1024, 1025, 4097, 8192, 32705, 32769])
def test_router_chunk_counts(P):
    """Chunks of the router's reductions and their combine (64 groups of threads, up to 8
    chunks each): 1, 4, 64, 65, 171, 256, 512 and 505 routing chunks, 1, 1, 8, 9, 33, 64,
    64 and 52 pooling chunks, with ragged last ones."""
    log("router chunks P=%d" % P)
    x = synth.make_layer(1, P, dtype="bf16", key=(14, P), sharp=True,
                         modes=np.zeros(16, np.uint8), qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    rows = np.arange(4)
    ref = oracle_layer(x, rows=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y[:4].double().cpu().numpy(), ref["Y"], "bf16", False, label="P=%d" % P)


@pytest.mark.parametrize("dtype,P", [("bf16", 300), ("f32", 300), ("bf16", 5000)])
def test_router_key_of_minus_infinity(dtype, P):
    """An infinite key whose logit is -inf has weight 0 wherever it stands (the first tokens
    of a chunk's threads, others, the last one; one position per head), and a head of such
    keys alone has no weights: NaN, which Eq.4 sends to FULL with the flag set."""
    from paper_2609_23733_amd import vp
    log("router minus infinity %s P=%d" % (dtype, P))
    x = synth.make_layer(1, P, dtype=dtype, key=(66, P), sharp=True)
    qp = oracle.router_pool(x.Q, x.W, x.U, x.w)
    at = [0, 1, 2, 3, 4, 7, 8, 15, 16, 17, 31, 32, P // 2, P - 2, P - 1]
    for h, i in enumerate(at):
        x.K[i, h, 5] = -float("inf") * float(np.sign(qp[h, 5]))
    x.K[:, 15, 5] = -float("inf") * float(np.sign(qp[15, 5]))
    layer = run_gpu(x, rule=oracle.RULE_THRESHOLD)
    st = layer.state
    for h in range(15):
        t = x.K[:, h].double().numpy() @ qp[h] / 8
        p = np.exp(t - t.max())
        ctx = p @ x.V[:, h].double().numpy() / p.sum()
        assert abs(float(st.score[h]) * p.sum() - 1) <= 1e-4, (h, float(st.score[h]))
        err = np.abs(st.ctx[h].double().cpu().numpy() - ctx).max()
        assert err <= 1e-4 * rms(ctx), (h, err)
    assert np.isnan(float(st.score[15])) and int(layer.modes[15]) == 2
    assert int(layer.buckets[19]) & 1


@pytest.mark.parametrize("H", [1, 3, 5, 8])
def test_fewer_heads(H):
    log("H=%d" % H)
    modes = np.array(([2, 1, 0] * 6)[:H], np.uint8)
    x = synth.make_layer(2, 150, dtype="bf16", key=(3, H), sharp=True, H=H, modes=modes,
                         qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", False, label="H=%d" % H)


def test_bf16_output_and_relu():
    log("bf16 output, relu")
    x = synth.make_layer(2, 700, dtype="bf16", key=(4, 0), sharp=True, n_full=6,
                         qkv_device="cuda")
    for act in (0, 1):
        layer = run_gpu(x, y_dtype=torch.bfloat16, act=act)
        ref = oracle_layer(x, act=act)
        check_router(layer, ref, oracle.RULE_ARGMAX)
        check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", True, label="act=%d" % act)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("wscale", [1.0, 20.0])
def test_pooling_weight_scale(dtype, wscale):
    """Gated pooling (Eq.1-2) with the pooling vector w as drawn (|w|_1 log2 e
    near 6: every exponential of the pooling logits fits fp32 without a
    reference point) and scaled by 20 (near 115: the pooling sums keep a
    running maximum)."""
    log("pooling weights x%g %s" % (wscale, dtype))
    x = synth.make_layer(2, 700, dtype=dtype, key=(13, 0), sharp=True, n_full=6,
                         qkv_device="cuda")
    x.w = (x.w.float() * wscale).to(x.w.dtype)
    l1 = x.w.float().abs().sum(dim=1) * 1.4426950408889634
    assert ((l1 < 60) if wscale == 1.0 else (l1 > 60)).all(), l1
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], dtype, False,
            label="pool w x%g %s" % (wscale, dtype))


@pytest.mark.parametrize("case,P", [("plain", 1025), ("plain", 1088), ("plain", 1151),
                                    ("columns", 1100), ("huge", 1100), ("one inf", 1100)])
def test_fp32_split_full_heads(case, P):
    """fp32 FULL heads past 1,024 tokens (operands as sums of two fp16 values)
    against the oracle, every row: token counts on both sides of whole 64-key tiles
    and 128-query items; V's features over 15 decades (each keeps its own
    precision); K and V past the split's range, and one infinite value of V, whose
    heads run on fp32 MFMAs.  Per feature, 2-norm error <= 1e-6 of its norm
    plus 2e-7 of sqrt(1 / N) |v| (a feature's near-uniform average cancels to
    that size): exp2 to 1 ulp and sums of N weights, each rounded to 2^-24, leave
    a few 1e-7 (3e-7 observed with fp32 MFMAs)."""
    from paper_2609_23733_amd import vp
    log("fp32 split %s P=%d" % (case, P))
    x = synth.make_layer(1, P, dtype="f32", n_full=5, n_surr=0, key=(61, P), sharp=True)
    heads = np.nonzero(x.modes == 2)[0]
    if case == "columns":
        x.V *= torch.logspace(-12, 3, 64)
    elif case == "huge":
        x.K *= 2.0 ** 70
        x.Q *= 2.0 ** -70
        x.V *= 2.0 ** 80
    elif case == "one inf":
        x.V[17, int(heads[1]), 5] = float("inf")
    layer = run_gpu(x, y_dtype=torch.float32)
    Y = layer.Y.double().cpu().numpy()
    for h in heads:
        ref = oracle.full_rows(x.Q, x.K, x.V, int(h))
        g = Y[:, h, :]
        if case == "one inf" and h == heads[1]:
            assert not np.isfinite(g[:, 5]).any()
            g, ref = np.delete(g, 5, 1), np.delete(ref, 5, 1)
        scale = np.abs(x.V[:, int(h)].double().numpy()).max(0) if case != "one inf" else 1.0
        err = np.linalg.norm(g - ref, axis=0)
        bound = 1e-6 * np.linalg.norm(ref, axis=0) + (2e-7 * scale if case != "one inf" else 2e-7)
        assert (err <= bound).all(), (case, int(h), float((err / bound).max()))


@pytest.mark.parametrize("scale", [64.0, 4096.0, 16384.0])
def test_fp32_large_logits(scale):
    """fp32 FULL heads past 1,024 tokens with logits up to about 2^15, 2^27 and 2^31 (log2
    units), where half an ulp of a softmax reference point reaches 64: every row whose two
    largest logits lie further apart than fp32 dot products can move them (64 roundings of
    2^-24 of sum |q k| each, both logits) and 40 is that key's value row, to 1e-6."""
    log("fp32 large logits x%g" % scale)
    P = 1100
    x = synth.make_layer(1, P, dtype="f32", n_full=3, n_surr=0, key=(62, P), sharp=True)
    x.Q *= scale
    x.K *= scale
    Y = run_gpu(x, y_dtype=torch.float32).Y.double().cpu().numpy()
    for h in np.nonzero(x.modes == 2)[0]:
        q, k, v = (t[:, int(h)].double().numpy() for t in (x.Q, x.K, x.V))
        t = C_LOG2 * (q @ k.T)
        moved = C_LOG2 * 2.0 ** -17 * (np.abs(q) @ np.abs(k).T).max(1)
        top2 = np.sort(t, axis=1)[:, -2:]
        sure = top2[:, 1] - top2[:, 0] > moved + 40
        assert sure.mean() > 0.5 if scale == 64 else sure.mean() > 0.9
        g, ref = Y[sure, h], v[t.argmax(1)[sure]]
        lost = int((~np.isfinite(Y[:, h])).any(1).sum())
        assert lost == 0, (scale, int(h), lost)
        ratio = float((np.abs(g - ref) / (1e-6 * np.abs(ref) + 2.0 ** -30 * np.abs(v).max())).max())
        assert ratio <= 1, (scale, int(h), ratio)


@pytest.mark.parametrize("case,b", [("features", 12), ("features", 16), ("features", 20),
                                    ("features", 24), ("rows", 8), ("rows", 16), ("rows", 24),
                                    ("cells", 20)])
def test_fp32_split_unequal_sizes(case, b):
    """fp32 FULL heads past 1,024 tokens whose operands differ much in size: half of K's
    features 2^-b and Q's 2^b times the others (the same logits), and value rows, or half of
    their features, 2^-b of the others that get all the weight (the others' logits are 80
    below).  Bound as in test_fp32_split_full_heads, with the size of the rows that have the
    weight."""
    log("fp32 unequal sizes %s 2^%d" % (case, b))
    P = 1100
    x = synth.make_layer(1, P, dtype="f32", n_full=3, n_surr=0, key=(63, P), sharp=True)
    if case == "features":
        x.K[:, :, :32] *= 2.0 ** -b
        x.Q[:, :, :32] *= 2.0 ** b
    else:
        x.Q[:, :, 0] = 30.0
        x.K[0::2, :, 0] = 0.0
        x.K[1::2, :, 0] = -16.0
        x.V[0::2, :, :64 if case == "rows" else 32] *= 2.0 ** -b
    Y = run_gpu(x, y_dtype=torch.float32).Y.double().cpu().numpy()
    for h in np.nonzero(x.modes == 2)[0]:
        ref = oracle.full_rows(x.Q, x.K, x.V, int(h))
        err = np.linalg.norm(Y[:, h] - ref, axis=0)
        scale = np.abs(x.V[0::2, int(h)].double().numpy()).max(0)
        ratio = float((err / (1e-6 * np.linalg.norm(ref, axis=0) + 2e-7 * scale)).max())
        log("  head %d worst err/bound %.3f" % (h, ratio))
        assert ratio <= 1, (case, b, int(h), ratio)


@pytest.mark.parametrize("H", [1, 2, 3, 5])
def test_fp32_split_few_heads(H):
    """fp32 FULL heads past 1,024 tokens with fewer heads than 16 (other strides and
    workspace offsets), every row."""
    log("fp32 split H=%d" % H)
    x = synth.make_layer(1, 1374, dtype="f32", key=(64, H), H=H, sharp=True,
                         modes=np.full(H, 2, np.uint8))
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "f32", False, label="H=%d" % H)


def test_fp32_mixed_items():
    """fp32 FULL heads of 4,200 tokens (33 items of 128 queries a head, 528 in all: one whole
    round of the 512 workgroups and 16 split over them), every other head past the split's
    range: workgroups go from one loop to the other.  The first, a middle and the last item."""
    log("fp32 mixed items")
    P = 4200
    x = synth.make_layer(1, P, dtype="f32", key=(65, P), sharp=True,
                         modes=np.full(16, 2, np.uint8))
    x.K[:, 1::2] *= 2.0 ** 70
    x.Q[:, 1::2] *= 2.0 ** -70
    rows = np.concatenate([np.arange(128), 2048 + np.arange(128), np.arange(4096, P)])
    layer = run_gpu(x, y_dtype=torch.float32)
    Y = layer.Y[torch.from_numpy(rows).to(layer.Y.device)].double().cpu().numpy()
    ref = np.stack([oracle.full_rows(x.Q, x.K, x.V, h, rows=rows) for h in range(16)], 1)
    check_y(Y, ref, "f32", False, label="mixed items")


def test_single_token():
    """N = 1: FULL returns v, MEAN returns v, s = 1 (every head FULL under Eq.4)."""
    log("N=1")
    x = synth.make_layer(1, 1, dtype="f32", key=(5, 0), n_full=16, qkv_device="cuda")
    layer = run_gpu(x, rule=oracle.RULE_THRESHOLD, y_dtype=torch.float32)
    np.testing.assert_array_equal(layer.modes.cpu().numpy(), np.full(16, 2, np.uint8))
    np.testing.assert_allclose(layer.Y.cpu().numpy(), x.V.cpu().numpy(), rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(layer.state.score.cpu().numpy(), 1.0, rtol=1e-6)


# --------------------------------------------------- threshold rule (Eq.4)

def planted_inputs(N, targets, dtype, seed=0):
    """All queries equal within a head (q_pool = q), one planted key per head
    with logit L_h chosen so that s_h = targets[h]; see the oracle pins."""
    H = len(targets)
    rng = np.random.default_rng(seed)
    Q = np.zeros((N, H, 64), np.float32)
    Q[:, :, 0] = 1.0
    K = (rng.normal(size=(N, H, 64)) * 0.125).astype(np.float32)
    K[:, :, 0] = 0.0
    V = (rng.normal(size=(N, H, 64)) * 0.125).astype(np.float32)
    for h, s in enumerate(targets):
        L = math.log(s * (N - 1) / (1.0 - s))
        K[(h * 97) % N, h, 0] = 8.0 * L
    x = synth.make_layer(1, N, dtype=dtype, key=(6, N), H=H, n_full=0)
    td = synth.torch_dtype(dtype)
    x.Q = torch.from_numpy(Q).to(td)
    x.K = torch.from_numpy(K).to(td)
    x.V = torch.from_numpy(V).to(td)
    return x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_threshold_rule_planted_saliency(dtype):
    N = 2748
    log("threshold planted %s" % dtype)
    # at least 4e-3 from tau_low and 2e-2 from tau_high before rounding, so
    # that bf16 rounding of the planted key (<= 3e-3 in s) keeps 1e-3
    targets = [0.22, 0.18, 0.014, 0.006, 0.6, 0.05, 0.1, 0.3,
               0.015, 0.005, 0.25, 0.12, 0.9, 0.02, 0.17, 0.23]
    x = planted_inputs(N, targets, dtype)
    ref = oracle_layer(x, rule=oracle.RULE_THRESHOLD)
    # margins after rounding to the stored dtype
    assert (np.minimum(np.abs(ref["s"] - 0.2), np.abs(ref["s"] - 0.01)) >= 1e-3).all()
    layer = run_gpu(x.to("cuda"), rule=oracle.RULE_THRESHOLD, y_dtype=torch.float32)
    check_router(layer, ref, oracle.RULE_THRESHOLD)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], dtype, False, label="planted")


def test_assign_boundaries_and_nan():
    from paper_2609_23733_amd import vp
    log("assign boundaries")
    tl, th = np.float32(0.01), np.float32(0.2)
    s = np.array([th, tl, np.nextafter(th, 0), np.nextafter(tl, 1), 1.0, 0.0, np.nan, 0.05],
                 np.float32)
    modes, buckets = vp.assign_heads(torch.from_numpy(s).cuda(), vp.RULE_THRESHOLD)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(modes.cpu().numpy(), [2, 0, 1, 1, 2, 0, 2, 1])
    b = buckets.cpu().numpy()
    np.testing.assert_array_equal(b[:3], [2, 3, 3])
    np.testing.assert_array_equal(b[3:11], [1, 5, 2, 3, 7, 0, 4, 6])
    assert b[19] & 1
    lg = np.array([[1, 1, 0], [0, 2, 2], [3, 3, 3], [0, 0, 1], [np.nan, 0, 0], [-1, -2, -3]],
                  np.float32)
    modes, buckets = vp.assign_heads(torch.from_numpy(lg).cuda(), vp.RULE_ARGMAX)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(modes.cpu().numpy(), oracle.assign(lg.astype(np.float64), 1))


# ---------------------------------------------------- robustness and order

def test_deterministic_bitwise():
    log("determinism")
    x = synth.make_layer(4, 1374, dtype="bf16", key=(7, 0), n_full=6, qkv_device="cuda")
    a = run_gpu(x)
    Y1 = a.Y.clone()
    q1 = a.state.q_pool.clone()
    a.step()
    torch.cuda.synchronize()
    assert torch.equal(Y1, a.Y)
    assert torch.equal(q1, a.state.q_pool)


def test_permutation_equivariance_gpu():
    log("permutation")
    modes = np.array([2, 1, 0, 2] * 4, np.uint8)
    x = synth.make_layer(2, 300, dtype="f32", key=(8, 0), sharp=True, modes=modes,
                         qkv_device="cuda")
    a = run_gpu(x, y_dtype=torch.float32)
    Ya = a.Y.double().cpu().numpy()
    pi = torch.from_numpy(np.random.default_rng(0).permutation(x.N)).cuda()
    xp = synth.make_layer(2, 300, dtype="f32", key=(8, 0), sharp=True, modes=modes,
                          qkv_device="cuda")
    xp.Q, xp.K, xp.V = x.Q[pi].contiguous(), x.K[pi].contiguous(), x.V[pi].contiguous()
    b = run_gpu(xp, y_dtype=torch.float32)
    Yb = b.Y.double().cpu().numpy()
    ref = Ya[pi.cpu().numpy()]
    for h in range(16):
        assert np.abs(Yb[:, h] - ref[:, h]).max() <= 1e-4 * rms(ref[:, h])


# ------------------------------------------ seeded random configurations

def _random_configurations(n, seed=4242):
    """n seeded draws over the layer's small-shape space: views, tokens per
    view (ragged around the 64-key and query tiles), head count, a mode per
    head, operand dtype, Y dtype, activation and input sharpness."""
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(n):
        H = int(rng.integers(1, 17))
        cases.append(dict(i=i, S=int(rng.integers(1, 4)), P=int(rng.integers(1, 600)), H=H,
                          dtype=("f32", "bf16")[int(rng.integers(0, 2))],
                          y_bf16=bool(rng.integers(0, 2)), act=int(rng.integers(0, 2)),
                          sharp=bool(rng.integers(0, 2)),
                          modes=rng.integers(0, 3, size=H).astype(np.uint8)))
    return cases


@pytest.mark.parametrize("c", _random_configurations(12), ids=lambda c: "r%d" % c["i"])
def test_random_configurations(c):
    """Router state, modes, buckets and every output row against the oracle
    on a seeded random configuration."""
    label = "random %d: S=%d P=%d H=%d %s y=%s act=%d sharp=%d modes=%s" % (
        c["i"], c["S"], c["P"], c["H"], c["dtype"], "bf16" if c["y_bf16"] else "f32", c["act"],
        c["sharp"], "".join(str(int(m)) for m in c["modes"]))
    log(label)
    x = synth.make_layer(c["S"], c["P"], dtype=c["dtype"], key=(40, c["i"]), sharp=c["sharp"],
                         H=c["H"], modes=c["modes"], qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.bfloat16 if c["y_bf16"] else torch.float32, act=c["act"])
    ref = oracle_layer(x, act=c["act"])
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], c["dtype"], c["y_bf16"],
            label="random %d" % c["i"])


# ------------------------------------------------- full-size workloads

@pytest.mark.parametrize("wl,n_full", [("s32_bf16", 4), ("s32_bf16", 16), ("s100_bf16", 4),
                                       ("s100_bf16", 16), ("s500_bf16", 1), ("s500_bf16", 6)])
def test_full_size_sampled(wl, n_full):
    """The benchmark workloads at full size, in the benchmark's launch
    configuration (bf16 operands, bf16 Y): router and modes on all tokens,
    SURR and MEAN heads on every row, FULL heads on sampled query rows."""
    cfg = synth.WORKLOADS[wl]
    log("full size %s n_full=%d" % (wl, n_full))
    x = synth.make_layer(cfg["S"], dtype="bf16", n_full=n_full, key=(cfg["S"], 0),
                         qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.bfloat16)
    rows = synth.sample_rows(x.N, 96, synth.derive_seed(cfg["S"], 0, 20))
    ref = oracle_layer(x, rows=rows, full_rows_sel=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    Yg = layer.Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    full = [h for h in range(16) if ref["modes"][h] == 2]
    for h in full:
        ref["Y"][:, h, :] = ref["Y_full_rows"][h]
    check_y(Yg, ref["Y"], "bf16", True, label="%s/%d" % (wl, n_full))


@pytest.mark.parametrize("wl,n_full", [("s32_bf16", 4), ("s32_bf16", 16), ("s100_bf16", 4),
                                       ("s500_bf16", 6)])
def test_full_size_sampled_f32_output(wl, n_full):
    """The benchmark workloads at full size with fp32 Y, so that the
    comparison is the bf16-operand bar alone: max |err| <= 2e-2 * min(head
    RMS, layer RMS) with no output rounding term.  At these sizes most FULL
    work items run whole (one workgroup over all key tiles) and the rest in
    the split tail; the sampled rows include the last one."""
    cfg = synth.WORKLOADS[wl]
    log("full size fp32 Y %s n_full=%d" % (wl, n_full))
    x = synth.make_layer(cfg["S"], dtype="bf16", n_full=n_full, key=(cfg["S"], 0),
                         qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    rows = synth.sample_rows(x.N, 128, synth.derive_seed(cfg["S"], 1, 20))
    ref = oracle_layer(x, rows=rows, full_rows_sel=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    Yg = layer.Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    for h in range(16):
        if ref["modes"][h] == 2:
            ref["Y"][:, h, :] = ref["Y_full_rows"][h]
    check_y(Yg, ref["Y"], "bf16", False, label="%s/%d fp32 Y" % (wl, n_full))


@pytest.mark.parametrize("S,y_bf16", [(32, False), (100, True)])
def test_full_size_sharp(S, y_bf16):
    """Full-size layers whose FULL heads attend sharply (Q, K ~ N(0, 1): logit
    spread of several log2 units, as heads routed FULL by Eq.4 have), so every
    work item's Cauchy-Schwarz bound exceeds the zero-reference window and
    the running-reference-point path carries the whole FULL stage."""
    log("full size sharp S=%d y=%s" % (S, "bf16" if y_bf16 else "f32"))
    x = synth.make_layer(S, dtype="bf16", n_full=4, key=(S, 3), sharp=True, qkv_device="cuda")
    full = [h for h in range(16) if x.modes[h] == 2]
    qn = torch.linalg.vector_norm(x.Q[:, full].float(), dim=2) * C_LOG2      # [N, 4]
    kn = torch.linalg.vector_norm(x.K[:, full].float(), dim=2).amax(dim=0)   # [4]
    nq = -(-x.N // 512)
    qmax = torch.stack([qn[t * 512:(t + 1) * 512].amax(dim=0) for t in range(nq)])
    assert (qmax * kn > FAST_BOUND).all()
    layer = run_gpu(x, y_dtype=torch.bfloat16 if y_bf16 else torch.float32)
    rows = synth.sample_rows(x.N, 128, synth.derive_seed(S, 3, 20))
    ref = oracle_layer(x, rows=rows, full_rows_sel=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    Yg = layer.Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    for h in full:
        ref["Y"][:, h, :] = ref["Y_full_rows"][h]
    check_y(Yg, ref["Y"], "bf16", y_bf16, label="sharp S=%d" % S)


def test_full_size_wide():
    """S = 32 with sharp Q and K scaled by 1.3: every FULL work item's bound
    (about 30 log2 units) exceeds the window of the zero-reference modes, so
    the whole FULL stage runs with running reference points (WIDE items);
    fp32 Y at the strict bar on 128 sampled rows, the last one among them."""
    S = 32
    log("full size wide S=%d" % S)
    x = synth.make_layer(S, dtype="bf16", n_full=4, key=(S, 6), sharp=True, qkv_device="cuda")
    x.Q = (x.Q.float() * 1.3).to(torch.bfloat16)
    x.K = (x.K.float() * 1.3).to(torch.bfloat16)
    b = item_bounds(x)
    assert (b > EXT_BOUND).all(), b.min()
    layer = run_gpu(x, y_dtype=torch.float32)
    rows = synth.sample_rows(x.N, 128, synth.derive_seed(S, 6, 20))
    ref = oracle_layer(x, rows=rows, full_rows_sel=rows)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    Yg = layer.Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    for h in range(16):
        if ref["modes"][h] == 2:
            ref["Y"][:, h, :] = ref["Y_full_rows"][h]
    check_y(Yg, ref["Y"], "bf16", False, label="wide S=%d" % S)


def test_element_offsets_past_2_32():
    """N = 3053 x 1374 = 4,194,822 tokens: element offsets token * 1024 + 64 h
    + i pass 2^32 from token 2^22 on.  The last head runs FULL (the largest
    offsets), head 14 SURR and head 13 MEAN; fp32 Y.  Sampled rows straddle
    the boundary (tokens 2^22 - 1, 2^22 and the last one among them).  The
    oracle sees one head at a time ([N, 1, d] slices): router state of the
    three heads (Eq.1-3, Eq.5 context and value mean), the FULL head's rows,
    the SURR head's rows (Eq.5-7 with the oracle's C_h) and the MEAN head's
    rows."""
    S, P = 3053, 1374
    N = S * P
    assert N * 16 * 64 > 2 ** 32
    modes = np.array([1, 0] * 7 + [1, 2], np.uint8)
    hf, hs, hm = 15, 14, 13
    log("element offsets past 2^32: N=%d" % N)
    x = synth.make_layer(S, P, dtype="bf16", key=(S, 5), modes=modes, qkv_device="cuda")
    layer = run_gpu(x, y_dtype=torch.float32)
    np.testing.assert_array_equal(layer.modes.cpu().numpy(), modes)
    b = 2 ** 22
    rows = np.unique(np.concatenate([
        synth.sample_rows(N, 20, synth.derive_seed(S, 5, 20)),
        np.array([0, b - 1, b, b + 1, N - 2, N - 1])])).astype(np.int64)
    Yg = layer.Y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    st = layer.state
    ref = {}
    for h in (hf, hs, hm):
        sl = slice(h, h + 1)
        Qh, Kh, Vh = (t[:, sl].float().cpu() for t in (x.Q, x.K, x.V))
        qp = oracle.router_pool(Qh, x.W[sl], x.U[sl], x.w[sl])
        s, C, mean = oracle.router_route(Kh, Vh, qp)
        for name, g, r in (("q_pool", st.q_pool[h], qp[0]), ("ctx", st.ctx[h], C[0]),
                           ("vmean", st.vmean[h], mean[0])):
            g = g.cpu().numpy().astype(np.float64)
            err = np.abs(g - r).max()
            assert err <= 1e-4 * max(rms(r), 1e-30), (name, h, err, rms(r))
        np.testing.assert_allclose(float(st.score[h]), s[0], rtol=1e-4)
        if h == hf:
            ref[h] = oracle.full_rows(Qh, Kh, Vh, 0, rows)
        elif h == hs:
            surr = {k: v[sl] for k, v in x.surr.items()}
            ref[h] = oracle.surr_rows(Vh, C[0], surr, 0, rows)
        else:
            ref[h] = np.broadcast_to(mean[0], (rows.shape[0], 64))
        del Qh, Kh, Vh
    for h in (hf, hs, hm):
        r = ref[h]
        err = np.abs(Yg[:, h, :] - r)
        bound = TOL["bf16"] * rms(r)
        log("offsets past 2^32: head %d worst err/bound = %.3f" % (h, float(err.max() / bound)))
        assert (err <= bound).all(), (h, float(err.max()), bound)
    # MEAN rows are the head's value mean itself, wherever they lie
    np.testing.assert_array_equal(
        Yg[:, hm, :], np.broadcast_to(st.vmean[hm].cpu().numpy().astype(np.float64),
                                      (rows.shape[0], 64)))


# ------------------------------------ softmax reference point (FULL, bf16)

C_LOG2 = 1.4426950408889634 / 8.0
# Logit bound (log2 units) up to which a work item runs in the FULL kernel's
# fastest mode (reference point 0, no overflow test); the cases below that
# must leave that mode assert bounds above it.
FAST_BOUND = 10.0


def tile_bounds(x, bq=256):
    """Per 256-query tile and head: max_i |c q_i| * max_j |k_j| (log2 units),
    the Cauchy-Schwarz bound on the tile's logits."""
    q = torch.linalg.vector_norm(x.Q.float(), dim=2).cpu().numpy() * C_LOG2   # [N, H]
    k = torch.linalg.vector_norm(x.K.float(), dim=2).cpu().numpy().max(axis=0)  # [H]
    nt = -(-x.N // bq)
    return np.stack([q[t * bq:(t + 1) * bq].max(axis=0) * k for t in range(nt)])


FULL8 = np.array([2, 2, 1, 0, 2, 2, 1, 0, 2, 2, 1, 0, 2, 2, 1, 0], np.uint8)


# Logit bound (log2 units) up to which a work item keeps the zero reference
# point until a weight overflows fp16.
EXT_BOUND = 24.0


def item_bounds(x):
    """Per 512-query work item and FULL head: the Cauchy-Schwarz logit bound."""
    return tile_bounds(x, bq=512)[:, x.modes == 2]


def test_zero_reference_overflow_moves():
    """Logit bounds between 10 and 24 (zero reference point kept while the
    weights fit fp16), with one key per FULL head planted in tile 5 along
    that head's largest query, 20 log2 units above 0: that query's weights
    overflow fp16 mid-sequence and its reference point moves there."""
    log("zero reference point: planted overflow")
    x = synth.make_layer(1, 1500, dtype="bf16", key=(11, 0), sharp=True, modes=FULL8,
                         qkv_device="cuda")
    x.K = (x.K.float() * 0.8).to(torch.bfloat16)
    for h in np.nonzero(x.modes == 2)[0]:
        q = x.Q[:, h].float()
        i0 = int(torch.linalg.vector_norm(q, dim=1).argmax())
        qn = float(torch.linalg.vector_norm(q[i0]))
        x.K[5 * 64 + 7, h] = (q[i0] / qn * (20.0 / (C_LOG2 * qn))).to(torch.bfloat16)
        logit = float((x.Q[i0, h].float() @ x.K[5 * 64 + 7, h].float())) * C_LOG2
        assert 19.5 < logit < 20.5, logit
    b = item_bounds(x)
    assert ((b > FAST_BOUND) & (b <= EXT_BOUND)).all(), b
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", False, label="planted overflow")


def test_zero_reference_low_first_tile():
    """Queries with positive components and first-tile keys pointing against
    them (k = -(7/8) (1, ..., 1) plus small noise): every query's first-tile
    maximum lies below -4 log2 units, so its reference point starts there;
    later keys (random signs) raise the row maxima by about ten log2 units,
    and queries whose weights then overflow fp16 move their reference point."""
    log("zero reference point: low first tile")
    x = synth.make_layer(1, 1500, dtype="bf16", key=(12, 0), sharp=True, modes=FULL8,
                         qkv_device="cuda")
    x.Q = (x.Q.float().abs() * 0.9).to(torch.bfloat16)
    x.K[:64] = (-7.0 / 8.0 + 0.05 * x.K[:64].float()).to(torch.bfloat16)
    q, k = x.Q.float().cpu(), x.K[:64].float().cpu()
    first = torch.stack([q[:, h] @ k[:, h].T for h in range(16)]).amax(dim=2) * C_LOG2
    assert (first[torch.from_numpy(x.modes == 2)] < -4).all(), first.max()
    b = item_bounds(x)
    assert ((b > FAST_BOUND) & (b <= EXT_BOUND)).all(), b
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", False, label="low first tile")


@pytest.mark.parametrize("P,n_full,few", [(2500, 16, True), (9001, 1, False), (4700, 2, False)])
def test_combined_parts(P, n_full, few):
    """Items of FULL heads split over workgroups, on both sides of the combine's rule (units
    of 64 queries below 8 parts an item, of 8 queries and two groups of parts from there):
    every query of the first, a middle and the (ragged) last item.  One key per head planted
    as in test_zero_reference_overflow_moves: some parts of one query have their own
    reference point, the others 0."""
    log("combined parts P=%d full=%d" % (P, n_full))
    modes = np.zeros(16, np.uint8)
    modes[16 - n_full:] = 2
    x = synth.make_layer(1, P, dtype="bf16", key=(13, P), sharp=True, modes=modes,
                         qkv_device="cuda")
    x.K = (x.K.float() * 0.7).to(torch.bfloat16)
    nkt, items = -(-P // 64), -(-P // 512) * n_full
    tail = items % 256
    parts = min(256, tail * nkt)
    assert tail and (parts < 8 * tail) == few
    heads = np.nonzero(modes == 2)[0]
    rows = [np.arange(512), 512 * (P // 1024) + np.arange(512), np.arange(P // 512 * 512, P)]
    for h in heads:
        q = x.Q[:, h].float()
        i0 = int(torch.linalg.vector_norm(q, dim=1).argmax())
        qn = float(torch.linalg.vector_norm(q[i0]))
        x.K[21 * 64 + 7, h] = (q[i0] / qn * (20.0 / (C_LOG2 * qn))).to(torch.bfloat16)
        rows.append(np.array([i0]))
    b = item_bounds(x)
    assert ((b > FAST_BOUND) & (b <= EXT_BOUND)).all(), b
    rows = np.unique(np.concatenate(rows))
    layer = run_gpu(x, y_dtype=torch.float32)
    Y = layer.Y[torch.from_numpy(rows).to(layer.Y.device)].double().cpu().numpy()
    ref = np.zeros_like(Y)
    for h in heads:
        ref[:, h] = oracle.full_rows(x.Q, x.K, x.V, int(h), rows=rows)
    check_y(Y, ref, "bf16", False, heads=heads, label="parts P=%d full=%d" % (P, n_full))


def test_reference_point_mixed_launch():
    """Query tiles whose logits are provably small (reference point 0: bound
    at most 14 in log2 units) and tiles that need the running reference point,
    in one launch: sharp queries halved, then queries 256..511 and one query of
    tile 4 scaled by 16 (both exact in bf16)."""
    log("reference point: mixed tiles")
    x = synth.make_layer(1, 1500, dtype="bf16", key=(9, 0), sharp=True, modes=FULL8,
                         qkv_device="cuda")
    x.Q *= 0.5
    x.Q[256:512] *= 16
    x.Q[1100] *= 16
    b = tile_bounds(x)
    big = np.zeros(b.shape[0], bool)
    big[[1, 4]] = True
    assert (b[big] > 48).all() and (b[~big] < 13).all(), b
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", False, label="mixed")


@pytest.mark.parametrize("P,grow_to,qs", [(1500, 8.0, 4.0), (4097, 8.0, 4.0),
                                          (1500, 2.2, 1.0), (4097, 2.2, 1.0)])
def test_reference_point_moves(P, grow_to, qs):
    """Key norms grow along the sequence (x1 to x`grow_to`) and queries are
    scaled by `qs`, so logits exceed every earlier reference point several
    times: the running reference point moves and O, l are rescaled; ragged
    last tile.  (8, 4): logit bounds above 380, weights overflow fp16 at
    once; (2.2, 1): bounds between 24 and 44, the row maxima creep up tile
    by tile."""
    log("reference point: growing logits P=%d grow=%g q*%g" % (P, grow_to, qs))
    x = synth.make_layer(1, P, dtype="bf16", key=(10, P), sharp=True, modes=FULL8,
                         qkv_device="cuda")
    grow = torch.linspace(1.0, grow_to, x.N, device=x.K.device)[:, None, None]
    x.K = (x.K.float() * grow).to(torch.bfloat16)
    x.Q *= qs
    b = tile_bounds(x, bq=512)[:, x.modes == 2]
    assert (b > (64 if grow_to > 4 else FAST_BOUND)).all(), b
    layer = run_gpu(x, y_dtype=torch.float32)
    ref = oracle_layer(x)
    check_router(layer, ref, oracle.RULE_ARGMAX)
    check_y(layer.Y.double().cpu().numpy(), ref["Y"], "bf16", False,
            label="grow P=%d x%g q*%g" % (P, grow_to, qs))
