"""GPU parity of the backward pass: ae_attn_backward (through the C ABI, fed by the HIP forward pass's output and
row statistic) against the fp64 backward oracle on the same seeded bf16 inputs.  Bar as for the forward pass
(bf16 operands, bf16 weights and score gradients into the second MFMAs, fp32 accumulation): max-abs <= 1e-2 and
mean-abs <= 1e-3, relative to max(1, the largest |reference| of the row)."""
import math

import numpy as np
import pytest
import torch

from oracle import attention_backward
from paper_2502_15349_amd.workloads import C2, Workload, make_grad, make_inputs

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS = 1e-2, 1e-3
DIMS = [(64, 64), (128, 128), (128, 256), (192, 128)]


@pytest.fixture(scope="module")
def A():
    from paper_2502_15349_amd import ae_attn
    return ae_attn


def hip_backward(A, w, Q, K, V, dO, out_dtype=None):
    dev = torch.device("cuda:0")
    Qd, Kd, Vd, dOd = Q.to(dev), K.to(dev), V.to(dev), dO.to(dev)
    stats = torch.empty((w.B, w.H_q, w.L_q), dtype=torch.float32, device=dev) if w.norm in ("softmax", "abssum", "abs_of_sum") else None
    O = A.run_workload(w, Qd, Kd, Vd, stats=stats, out_dtype=out_dtype)
    dQ, dK, dV = A.attention_backward(Qd, Kd, Vd, O, dOd, stats, scale=w.scale_value, score_mod=w.score_mod, bias=w.bias,
                                      gamma=w.gamma(), norm=w.norm, mask=w.mask, window=w.window)
    torch.cuda.synchronize()
    return [x.cpu().double().numpy() for x in (dQ, dK, dV)]


def oracle_backward(w, Q, K, V, dO):
    return attention_backward(Q, K, V, dO, scale=w.scale_value, score_mod=w.score_mod, bias=w.bias, gamma=w.gamma(),
                              norm=w.norm, mask=w.oracle_mask())


def check(got, ref, what):
    assert np.isfinite(got).all(), f"{what}: non-finite gradient"
    rs = np.maximum(np.abs(ref).max(axis=-1, keepdims=True), 1.0)
    err = np.abs(got - ref) / rs
    print(f"{what}: max_abs {err.max():.3e} mean_abs {err.mean():.3e} |ref|max {np.abs(ref).max():.3e}", flush=True)
    assert err.max() <= MAX_ABS, f"{what}: max-abs {err.max():.3e}"
    assert err.mean() <= MEAN_ABS, f"{what}: mean-abs {err.mean():.3e}"


def run_case(A, w, out_dtype=None, positive_scores=False):
    print(f"case {w}", flush=True)
    Q, K, V = make_inputs(w)
    if positive_scores:   # |q|, |k|: every score positive, so that a signed row sum does not cancel
        Q, K = Q.abs(), K.abs()
    dO = make_grad(w)
    got, ref = hip_backward(A, w, Q, K, V, dO, out_dtype), oracle_backward(w, Q, K, V, dO)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        check(g, r, f"{w.name} {name}")


VARIANTS = {
    "softmax": dict(),
    "softmax_causal": dict(mask="causal"),
    "softmax_bias_causal": dict(score_mod="bias", bias=0.75, mask="causal"),
    "softmax_negative_scale": dict(scale=-0.11, mask="causal"),
    "sigmoid_causal": dict(score_mod="bias", norm="sigmoid", mask="causal", bias=-math.log(300.0)),
    "sigmoid": dict(norm="sigmoid", score_mod="bias", bias=-3.0),
    # no normalization: ReLU attention, and the bare (biased) scores as weights
    "relu": dict(score_mod="relu", norm="none", scale=0.01),
    "relu_causal": dict(score_mod="relu", norm="none", mask="causal", scale=0.01),
    "none_bias_causal": dict(score_mod="bias", bias=0.02, norm="none", mask="causal", scale=0.005),
    # retention (per-head decay, abs-sum normalizers): rows above the clamp, and (tiny scale) below it
    "retnet_abssum": dict(score_mod="head_decay", norm="abssum", mask="causal", decay=True),
    "retnet_abs_of_sum": dict(score_mod="head_decay", norm="abs_of_sum", mask="causal", decay=True),
    "retnet_abssum_below_clamp": dict(score_mod="head_decay", norm="abssum", mask="causal", decay=True, scale=0.0005),
    "decay_nonorm": dict(score_mod="head_decay", norm="none", mask="causal", decay=True, scale=0.01),
    "abssum_plain": dict(norm="abssum"),
    # (|sum| as normalizer: a bias that keeps the row sums away from cancellation, where the statistic itself --
    # and with it every gradient of the row -- is ill-conditioned)
    "abs_of_sum_bias_causal": dict(norm="abs_of_sum", score_mod="bias", bias=3.0, mask="causal"),
}


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("variant", sorted(VARIANTS))
def test_backward_small_ragged(A, dims, variant):
    # 3 own tiles with a ragged tail on either side, 5-6 LDS tiles with a ragged tail, grouped heads 2:1
    # The |sum| normalizer with zero-mean scores divides by a row sum that cancels (sum |s'| can be 50 x |sum s'|):
    # the operator itself is ill-conditioned there, gradients reach hundreds and no bf16 path meets an absolute bar.
    # With decay (no bias to shift the scores) it is therefore run on |q|, |k|.
    run_case(A, Workload(variant, 40, 2, 4, 2, 300, 333, dims[0], dims[1], **VARIANTS[variant]),
             positive_scores=variant == "retnet_abs_of_sum")


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"d{d[0]}_{d[1]}")
def test_backward_abs_of_sum_decay_unnarrowed(A, dims):
    """The |sum| normalizer with decay on the plain N(0, 1) inputs (no |q|, |k|): the row sums cancel (sum |s'| is
    some 50 x |sum s'|), so the operator amplifies every rounding of its inputs by that factor and gradients reach
    hundreds; an absolute bar means nothing here.  Relative bar instead, per tensor: the largest error at most 2 % of
    the largest |reference|, the mean error at most 2 % of the mean |reference| (bf16 weights carry 2^-9 relative
    rounding each; amplified by the cancellation of the row sum, percent-level agreement is what the arithmetic
    supports)."""
    w = Workload("retnet_abs_of_sum_raw", 40, 2, 4, 2, 300, 333, dims[0], dims[1], score_mod="head_decay", norm="abs_of_sum",
                 mask="causal", decay=True)
    print(f"case {w}", flush=True)
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    got, ref = hip_backward(A, w, Q, K, V, dO), oracle_backward(w, Q, K, V, dO)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        assert np.isfinite(g).all()
        err = np.abs(g - r)
        print(f"{w.name} {name}: max err {err.max():.3e} of max |ref| {np.abs(r).max():.3e}; mean err {err.mean():.3e} of mean |ref| "
              f"{np.abs(r).mean():.3e}", flush=True)
        assert err.max() <= 2e-2 * np.abs(r).max() and err.mean() <= 2e-2 * np.abs(r).mean(), name


@pytest.mark.parametrize("Lq,Lk", [(1, 1), (1, 200), (200, 1), (31, 33), (64, 64), (128, 128), (129, 257), (500, 130),
                                    (130, 500), (257, 129)])
@pytest.mark.parametrize("mask", ["none", "causal"])
def test_backward_lengths(A, Lq, Lk, mask):
    # L_q != L_k in both directions (causal: bottom-right aligned; with L_q > L_k the first rows see no key and
    # must get zero gradient), single rows, exact tile multiples
    run_case(A, Workload(f"len{Lq}x{Lk}{mask}", 41, 1, 3, 1, Lq, Lk, 64, 64, mask=mask))
    run_case(A, Workload(f"len{Lq}x{Lk}{mask}sig", 42, 1, 2, 2, Lq, Lk, 128, 128, mask=mask, norm="sigmoid", score_mod="bias", bias=-2.0))
    run_case(A, Workload(f"len{Lq}x{Lk}{mask}relu", 45, 1, 2, 1, Lq, Lk, 64, 64, mask=mask, norm="none", score_mod="relu", scale=0.02))


@pytest.mark.parametrize("dims", [(128, 128), (128, 256), (192, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("Lq,Lk", [(32, 129), (33, 32), (65, 160), (95, 96), (161, 97), (192, 127), (129, 161)])
def test_backward_pairs_of_wavefronts(A, dims, Lq, Lk):
    """The kernels with a pair of wavefronts per 32 own rows walk tiles of 32 rows through a ring of five stages: walks
    of one to six tiles per query head, three query heads one after the other (the copies run three tiles ahead, over
    the seam between heads), last tiles of 1, 31 and 32 rows, own rows that fill one to four of the pairs; with a row
    statistic and without, the factor of the abs-sum form carrying the sign of the score, ReLU's a mask.  (Without a mask every
    length runs on pairs; the causal ones of up to 128 rows on single wavefronts, see test_backward_short_walks.)"""
    for kw in (dict(), dict(norm="sigmoid", score_mod="bias", bias=-3.0), dict(norm="abssum"), dict(score_mod="relu", norm="none", scale=0.01),
               dict(norm="sigmoid", score_mod="bias", bias=-3.0, mask="causal"),
               dict(score_mod="head_decay", norm="abssum", mask="causal", decay=True)):
        run_case(A, Workload("bwd_pairs", 46, 1, 3, 1, Lq, Lk, dims[0], dims[1], **kw))


@pytest.mark.parametrize("dims", [(128, 128), (128, 256), (192, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("Lq,Lk,window,g", [(64, 65, 500, 1), (65, 64, 500, 1), (128, 128, 500, 1), (129, 128, 500, 1), (128, 129, 500, 1), (400, 333, 7, 1), (333, 400, 33, 2),
                                            (400, 420, 96, 1), (420, 400, 97, 1), (520, 540, 256, 1), (540, 520, 257, 1), (300, 333, 128, 2),
                                            (333, 300, 129, 2), (300, 310, 299, 1), (400, 420, 128, 1), (420, 400, 129, 1), (64, 64, 500, 2), (32, 33, 500, 2)])
def test_backward_short_walks(A, dims, Lq, Lk, window, g):
    """Head dims whose registers leave room for one workgroup per CU: causal walks of up to 64 rows (128 without normalization), times
    the q heads of a group on the key side, and at 128/128 windows of up to 128 run on single wavefronts, longer ones on pairs.  Both
    sides of each limit, windows that hide whole tiles from some waves and not from others, L_q and L_k either way."""
    for kw in (dict(), dict(norm="sigmoid", score_mod="bias", bias=-3.0), dict(norm="none", scale=0.01)):
        run_case(A, Workload(f"short{window}", 48, 1, g, 1, Lq, Lk, dims[0], dims[1], mask="sliding_window", window=window, **kw))


@pytest.mark.parametrize("window", [1, 7, 64, 100, 333, 5000])
@pytest.mark.parametrize("Lq,Lk", [(300, 333), (333, 300), (700, 700)])
def test_backward_sliding_window(A, window, Lq, Lk):
    # windows shorter than a sub-tile, spanning a few tiles, and wider than the keys (= the causal mask); the walk
    # of either kernel starts and ends at the tiles the window allows
    run_case(A, Workload(f"win{window}_{Lq}x{Lk}", 47, 1, 4, 2, Lq, Lk, 128, 128, mask="sliding_window", window=window))
    run_case(A, Workload(f"win{window}_{Lq}x{Lk}sig", 48, 2, 2, 2, Lq, Lk, 64, 64, mask="sliding_window", window=window,
                         norm="sigmoid", score_mod="bias", bias=-1.0))


@pytest.mark.parametrize("dims,kw", [((128, 128), dict(mask="causal")), ((128, 128), dict(mask="sliding_window", window=64)), ((128, 128), dict()),
                                     ((64, 64), dict(mask="causal")), ((192, 128), dict(mask="causal")),
                                     ((128, 256), dict(score_mod="head_decay", norm="abssum", mask="causal", decay=True))],
                         ids=["d128_causal", "d128_window", "d128", "d64", "d192", "d128_256_abssum"])
def test_backward_batch_entries_do_not_depend_on_the_launches(A, dims, kw):
    # seven batch entries at once, where some head dims take a launch for each side, and one at a time, where both sides
    # share one: the same values.  (64/64 and 192/128 share one either way at this size -- beyond their lines is the test below --
    # and show that the workgroups' places in the grid leave the values alone)
    w = Workload("launches", 47, 7, 8, 8, 1000, 1030, dims[0], dims[1], **kw)
    dev = torch.device("cuda:0")
    Q, K, V = (t.to(dev) for t in make_inputs(w))
    dO = make_grad(w).to(dev)
    stats = torch.empty((w.B, w.H_q, w.L_q), dtype=torch.float32, device=dev)
    O = A.run_workload(w, Q, K, V, stats=stats)
    args = dict(scale=w.scale_value, score_mod=w.score_mod, bias=w.bias, gamma=w.gamma(), norm=w.norm, mask=w.mask, window=w.window)
    whole = A.attention_backward(Q, K, V, O, dO, stats, **args)
    for b in range(w.B):
        part = A.attention_backward(*(t[b:b + 1].contiguous() for t in (Q, K, V, O, dO, stats)), **args)
        torch.cuda.synchronize()
        for x, y in zip(whole, part):
            assert torch.equal(x[b:b + 1], y)


@pytest.mark.parametrize("dims,mask,B,H,L", [((64, 64), "none", 8, 16, 2048), ((64, 64), "causal", 8, 16, 3500), ((192, 128), "causal", 2, 64, 4095)],
                         ids=["d64", "d64_causal", "d192_causal"])
def test_backward_calls_of_much_work_take_a_launch_for_each_side(A, dims, mask, B, H, L):
    # all batch entries at once stand beyond the line, one at a time in front of it: the same values
    g = torch.Generator("cuda").manual_seed(49)
    Q, K, V, dO = (torch.randn(B, H, L, D, generator=g, device="cuda", dtype=torch.bfloat16) for D in (dims[0], dims[0], dims[1], dims[1]))
    stats = torch.empty((B, H, L), dtype=torch.float32, device="cuda")
    args = dict(scale=dims[0] ** -0.5, mask=mask)
    O = A.attention_forward(Q, K, V, stats=stats, **args)
    whole = A.attention_backward(Q, K, V, O, dO, stats, **args)
    for b in range(B):
        part = A.attention_backward(*(t[b:b + 1].contiguous() for t in (Q, K, V, O, dO, stats)), **args)
        for x, y in zip(whole, part):
            assert torch.equal(x[b:b + 1], y)


@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (192, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("mask", ["none", "causal"])
@pytest.mark.parametrize("n", [1, 2, 3, 6])
def test_heads_do_not_depend_on_their_number(A, dims, mask, n):
    # eight k/v heads, one per XCD, against the first n of them, whose workgroups are shared out over 8, 4, 8 and 4 XCDs: every
    # workgroup is there once and the values are the same, forwards and backwards
    w = Workload("heads", 48, 1, 16, 8, 1500, 1530, dims[0], dims[1], mask=mask)
    dev = torch.device("cuda:0")
    Q, K, V = (t.to(dev) for t in make_inputs(w))
    dO = make_grad(w).to(dev)

    def both(nq, nkv):
        q, k, v, g = Q[:, :nq].contiguous(), K[:, :nkv].contiguous(), V[:, :nkv].contiguous(), dO[:, :nq].contiguous()
        stats = torch.empty((1, nq, w.L_q), dtype=torch.float32, device=dev)
        O = A.attention_forward(q, k, v, stats=stats, scale=w.scale_value, mask=mask)
        return (O, stats) + tuple(A.attention_backward(q, k, v, O, g, stats, scale=w.scale_value, mask=mask))

    for x, y in zip(both(2 * n, n), both(16, 8)):
        assert torch.equal(x, y[:, :x.shape[1]])


@pytest.mark.parametrize("dims", [(64, 64), (128, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("mask", ["none", "causal"])
@pytest.mark.parametrize("n,L", [(9, 1100), (9, 2100), (13, 2100), (25, 1100), (33, 1100), (33, 2100)])
def test_heads_of_many_groups_do_not_depend_on_their_number(A, dims, mask, n, L):
    # groups that are cut into parts and groups that stay whole, on both sides of the lines between them, against eight at a time
    g = torch.Generator("cuda").manual_seed(50)
    Q, K, V, dO = (torch.randn(1, n, L, D, generator=g, device="cuda", dtype=torch.bfloat16) for D in (dims[0], dims[0], dims[1], dims[1]))
    args = dict(scale=dims[0] ** -0.5, mask=mask)

    def both(h0, h1):
        q, k, v, do = (t[:, h0:h1].contiguous() for t in (Q, K, V, dO))
        stats = torch.empty((1, h1 - h0, L), dtype=torch.float32, device="cuda")
        O = A.attention_forward(q, k, v, stats=stats, **args)
        return (O, stats) + tuple(A.attention_backward(q, k, v, O, do, stats, **args))

    whole = both(0, n)
    for h0 in (0, n - 8):
        for x, y in zip(whole, both(h0, h0 + 8)):
            assert torch.equal(x[:, h0:h0 + 8], y)


def test_backward_more_heads_than_the_decay_table(A):
    # handles without a per-head decay may have more query heads than the decay table holds (256): the kernels of
    # the linear normalizations must not read the table then
    run_case(A, Workload("heads260_none", 49, 1, 260, 130, 70, 90, 64, 64, norm="none", scale=0.01, mask="causal"))
    run_case(A, Workload("heads260_abssum", 50, 1, 260, 260, 40, 40, 64, 64, norm="abssum"))


def test_backward_bf16_forward_output(A):
    # delta is formed from the forward output as stored: also when that is bf16
    run_case(A, Workload("bf16_O", 43, 1, 4, 2, 260, 260, 128, 128, mask="causal"), out_dtype=torch.bfloat16)


def test_backward_strided_inputs(A):
    # Q, K, V as [B, L, H, D] memory viewed as [B, H, L, D]
    w = Workload("strided", 44, 2, 4, 2, 200, 230, 128, 128, mask="causal")
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    dev = torch.device("cuda:0")
    Qd, Kd, Vd = (x.to(dev).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for x in (Q, K, V))
    stats = torch.empty((w.B, w.H_q, w.L_q), dtype=torch.float32, device=dev)
    O = A.run_workload(w, Qd, Kd, Vd, stats=stats)
    got = A.attention_backward(Qd, Kd, Vd, O, dO.to(dev), stats, scale=w.scale_value, mask=w.mask)
    torch.cuda.synchronize()
    ref = oracle_backward(w, Q, K, V, dO)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        check(g.cpu().double().numpy(), r, f"strided {name}")


def test_backward_full_size_c2_one_group(A):
    """The benchmark shape (4 x 32/8 heads x 2048 x 128, causal softmax) at full size; the oracle checks one
    (batch, k/v head) group: its four query heads' dQ and the group's dK, dV."""
    w = C2
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    got = hip_backward(A, w, Q, K, V, dO)
    b, hk, g = 2, 5, w.H_q // w.H_kv
    hs = slice(hk * g, hk * g + g)
    ref = attention_backward(Q[b:b + 1, hs], K[b:b + 1, hk:hk + 1], V[b:b + 1, hk:hk + 1], dO[b:b + 1, hs],
                             scale=w.scale_value, norm="softmax", mask="causal")
    check(got[0][b:b + 1, hs], ref[0], "C2 dQ")
    check(got[1][b:b + 1, hk:hk + 1], ref[1], "C2 dK")
    check(got[2][b:b + 1, hk:hk + 1], ref[2], "C2 dV")


def test_backward_seeded_random_shapes(A):
    """40 seeded draws over shapes (ragged, L_q != L_k in both directions), head grouping, head dims,
    normalization / modification / mask, each against the backward oracle."""
    rng = np.random.default_rng(20250305)
    combos = [("softmax", "none"), ("softmax", "bias"), ("sigmoid", "bias"), ("none", "relu"), ("none", "none"),
              ("abssum", "none"), ("abssum", "head_decay"), ("none", "head_decay")]
    for case in range(40):
        dims = DIMS[int(rng.integers(len(DIMS)))]
        norm, mod = combos[int(rng.integers(len(combos)))]
        g = int(rng.choice([1, 2, 4]))
        H_kv = int(rng.integers(1, 3))
        Lq, Lk = int(rng.integers(1, 500)), int(rng.integers(1, 600))
        mask = "causal" if mod == "head_decay" else str(rng.choice(["none", "causal", "sliding_window"]))
        if mask == "sliding_window" and (mod == "relu" or norm == "abssum"):
            mask = "causal"
        w = Workload(f"rand{case}", 500 + case, int(rng.integers(1, 3)), g * H_kv, H_kv, Lq, Lk, dims[0], dims[1],
                     score_mod=mod, norm=norm, mask=mask, window=int(rng.integers(1, 400)) if mask == "sliding_window" else 0,
                     decay=(mod == "head_decay"), bias=float(rng.uniform(-2, 1)) if norm != "none" else 0.01,
                     scale=(0.01 if norm == "none" else None))
        run_case(A, w)


def test_backward_hip_graph_replays(A):
    """ae_attn_backward allocates nothing: its launches are captured into a HIP graph and replayed four
    times with new dO values and eager work in between; every replay must equal the eager call bit for bit."""
    dev = torch.device("cuda:0")
    w = Workload("graph_bwd", 46, 1, 4, 2, 300, 420, 128, 128, mask="causal")
    Q, K, V = (x.to(dev) for x in make_inputs(w))
    dO0 = make_grad(w).to(dev)
    stats = torch.empty((w.B, w.H_q, w.L_q), dtype=torch.float32, device=dev)
    O = A.run_workload(w, Q, K, V, stats=stats)
    h = A.ae_attn_create(B=w.B, H_q=w.H_q, H_kv=w.H_kv, L_q=w.L_q, L_k=w.L_k, D_qk=w.D_qk, D_v=w.D_v,
                         scale=w.scale_value, mask=w.mask)
    ws = torch.empty(A.ae_attn_backward_workspace_bytes(h), dtype=torch.uint8, device=dev)
    ws_e = torch.empty_like(ws)
    dO = dO0.clone()
    outs_g = [torch.zeros(x.shape, dtype=torch.float32, device=dev) for x in (Q, K, V)]
    outs_e = [torch.zeros(x.shape, dtype=torch.float32, device=dev) for x in (Q, K, V)]

    def launch(outs, wsp, stream):
        A.ae_attn_backward(h, Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), dO.data_ptr(), stats.data_ptr(),
                           outs[0].data_ptr(), outs[1].data_ptr(), outs[2].data_ptr(), wsp.data_ptr(), wsp.numel(),
                           stream.cuda_stream)

    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        launch(outs_g, ws, side)
    torch.cuda.synchronize()
    for replay in range(4):
        if replay:
            dO.copy_((dO0.float() * (1.0 + 0.3 * replay)).to(torch.bfloat16).roll(replay, dims=2))
        for x in outs_g:
            x.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        launch(outs_e, ws_e, torch.cuda.current_stream())
        torch.cuda.synchronize()
        for name, a, b in zip(("dQ", "dK", "dV"), outs_g, outs_e):
            assert torch.equal(a, b), f"replay {replay}: {name} differs from the eager call"
    del graph
    A.ae_attn_destroy(h)


@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (192, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("norm", ["softmax", "sigmoid", "none"])
@pytest.mark.parametrize("mask", ["none", "causal"])
def test_backward_bias_tensor(A, dims, norm, mask):
    """dQ, dK, dV with an additive bias tensor (per batch and head / shared over the batch / over both) on a ragged,
    grouped shape; the bias rows are padded to a multiple of 8 on the device."""
    from paper_2502_15349_amd.workloads import make_bias_tensor
    dev = torch.device("cuda:0")
    w = Workload(f"bwd_bias_{norm}_{mask}", 63, 2, 4, 2, 300, 333, dims[0], dims[1], score_mod="bias_tensor", norm=norm,
                 mask=mask, scale=(0.01 if norm == "none" else None))
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    Qd, Kd, Vd, dOd = Q.to(dev), K.to(dev), V.to(dev), dO.to(dev)
    for per_batch, per_head in ((True, True), (False, True), (False, False)):
        bt = make_bias_tensor(w, per_batch, per_head)
        if norm == "none":
            bt = (bt.float() * 0.01).to(torch.bfloat16)
        print(f"case {w.name} dims {dims} bias shape {tuple(bt.shape)}", flush=True)
        btd = torch.zeros(bt.shape[:3] + (336,), dtype=torch.bfloat16, device=dev)
        btd[..., :w.L_k] = bt.to(dev)
        btv = btd[..., :w.L_k]
        stats = torch.empty((w.B, w.H_q, w.L_q), dtype=torch.float32, device=dev) if norm == "softmax" else None
        O = A.run_workload(w, Qd, Kd, Vd, stats=stats, bias_tensor=btv)
        got = A.attention_backward(Qd, Kd, Vd, O, dOd, stats, scale=w.scale_value, score_mod="bias_tensor", norm=norm,
                                   mask=mask, bias_tensor=btv, want_dbias=True)
        torch.cuda.synchronize()
        ref = attention_backward(Q, K, V, dO, scale=w.scale_value, score_mod="bias_tensor", norm=norm, mask=mask, bias_tensor=bt,
                                 with_dbias=True)
        for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
            check(g.cpu().double().numpy(), r, f"{w.name} {tuple(bt.shape)} {name}")
        # The bias gradient is dS' itself, element by element, stored as bf16.  Where one weight dominates a row,
        # dS' = P (dP - delta) is a difference of nearly equal numbers of size |dO| |V| (~ 8 here), and delta comes
        # from the forward output as stored (bf16 weights in its sum): single elements are off by a few 1e-2 where
        # the sums that form dQ, dK, dV average such errors out.  Bar: max-abs 3e-2, mean-abs 1e-3, relative to
        # max(1, largest |reference| of the row).
        gB, rB = got[3].float().cpu().double().numpy(), ref[3]
        errB = np.abs(gB - rB) / np.maximum(np.abs(rB).max(axis=-1, keepdims=True), 1.0)
        print(f"{w.name} {tuple(bt.shape)} dBias: max_abs {errB.max():.3e} mean_abs {errB.mean():.3e}", flush=True)
        assert np.isfinite(gB).all() and errB.max() <= 3e-2 and errB.mean() <= MEAN_ABS


@pytest.mark.parametrize("dims", [(64, 64), (128, 128), (192, 128)], ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("norm", ["softmax", "sigmoid", "none"])
@pytest.mark.parametrize("Lq,Lk", [(64, 64), (64, 65), (65, 64), (61, 128), (64, 129)])
def test_backward_bias_tensor_short_walks(A, dims, norm, Lq, Lk):
    """Causal walks of up to 128 rows (keys; queries times the two q heads of a group) with a bias tensor run on single
    wavefronts at 128/128 (64/64 likewise, 192/128 on pairs); both sides of the limit."""
    from paper_2502_15349_amd.workloads import make_bias_tensor
    dev = torch.device("cuda:0")
    w = Workload(f"bwd_bias_short_{norm}", 65, 2, 4, 2, Lq, Lk, dims[0], dims[1], score_mod="bias_tensor", norm=norm, mask="causal",
                 scale=(0.01 if norm == "none" else None))
    print(f"case {w}", flush=True)
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    bt = make_bias_tensor(w, True, True)
    if norm == "none":
        bt = (bt.float() * 0.01).to(torch.bfloat16)
    btd = torch.zeros(bt.shape[:3] + ((Lk + 7) // 8 * 8,), dtype=torch.bfloat16, device=dev)
    btd[..., :Lk] = bt.to(dev)
    Qd, Kd, Vd, dOd = (t.to(dev) for t in (Q, K, V, dO))
    stats = torch.empty((2, 4, Lq), dtype=torch.float32, device=dev) if norm == "softmax" else None
    O = A.run_workload(w, Qd, Kd, Vd, stats=stats, bias_tensor=btd[..., :Lk])
    got = A.attention_backward(Qd, Kd, Vd, O, dOd, stats, scale=w.scale_value, score_mod="bias_tensor", norm=norm, mask="causal",
                               bias_tensor=btd[..., :Lk], want_dbias=True)
    torch.cuda.synchronize()
    ref = attention_backward(Q, K, V, dO, scale=w.scale_value, score_mod="bias_tensor", norm=norm, mask="causal", bias_tensor=bt, with_dbias=True)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        check(g.cpu().double().numpy(), r, f"{w.name} {name}")
    gB, rB = got[3].float().cpu().double().numpy(), ref[3]  # (the bars of test_backward_bias_tensor)
    errB = np.abs(gB - rB) / np.maximum(np.abs(rB).max(axis=-1, keepdims=True), 1.0)
    assert np.isfinite(gB).all() and errB.max() <= 3e-2 and errB.mean() <= MEAN_ABS


@pytest.mark.parametrize("B,H,H_kv,Lq,Lk", [(2, 64, 64, 400, 385), (3, 40, 40, 385, 520), (2, 96, 24, 260, 500), (4, 20, 20, 767, 800)])
@pytest.mark.parametrize("norm", ["softmax", "sigmoid", "none"])
def test_backward_bias_tensor_by_number_of_workgroups(A, B, H, H_kv, Lq, Lk, norm):
    """64/64 with a bias tensor: a side whose walks are 384 rows or longer (half of them with the causal mask) runs on pairs of
    wavefronts while it has at most 32 workgroups per XCD (48), on single ones beyond.  Workgroups per XCD of the four shapes,
    query side / key side: 64 / 64, 60 / 75, 72 / 24, 60 / 70; of one batch entry alone 32 / 32, 20 / 25, 36 / 12, 18 / 21.  The two
    forms sum in one order: the whole batch gives the bits of its entries alone, but for sigmoid, whose factors
    dP P (1 - P) are multiplied in another order: 2^-23 relative, which turns one bf16 rounding of dS' (2^-9) in 2^13; the
    root of the mean square over all is 2^-9 2^-6.5 = 2e-5, held to ten times that.  The entries alone are held to the
    oracle on the first group of heads."""
    from paper_2502_15349_amd.workloads import make_bias_tensor
    dev = torch.device("cuda:0")
    w = Workload("bwd_bias_many", 64, B, H, H_kv, Lq, Lk, 64, 64, score_mod="bias_tensor", norm=norm, mask="causal" if B == 4 else "none",
                 scale=(0.01 if norm == "none" else None))
    print(f"case {w}", flush=True)
    Q, K, V = (t.to(dev) for t in make_inputs(w))
    dO = make_grad(w).to(dev)
    bt = make_bias_tensor(w, False, True)
    if norm == "none":
        bt = (bt.float() * 0.01).to(torch.bfloat16)
    btd = torch.zeros(bt.shape[:3] + ((Lk + 7) // 8 * 8,), dtype=torch.bfloat16, device=dev)
    btd[..., :Lk] = bt.to(dev)
    btv = btd[..., :Lk]
    stats = torch.empty((B, H, Lq), dtype=torch.float32, device=dev) if norm == "softmax" else None
    O = A.run_workload(w, Q, K, V, stats=stats, bias_tensor=btv)

    def grads(sl):
        out = A.attention_backward(Q[sl], K[sl], V[sl], O[sl], dO[sl], None if stats is None else stats[sl], scale=w.scale_value,
                                   score_mod="bias_tensor", norm=norm, mask=w.mask, bias_tensor=btv, want_dbias=True)
        torch.cuda.synchronize()
        return [g.float() for g in out]
    whole, parts = grads(slice(0, B)), [grads(slice(b, b + 1)) for b in range(B)]
    for n, name in enumerate(("dQ", "dK", "dV", "dBias")):
        ref = torch.cat([q[n] for q in parts])
        assert torch.isfinite(ref).all()
        if norm == "sigmoid":
            assert (whole[n] - ref).norm() <= 2e-4 * ref.norm(), name
        else:
            assert torch.equal(whole[n], ref), name
    n = H // H_kv
    ref = attention_backward(Q[:1, :n].cpu(), K[:1, :1].cpu(), V[:1, :1].cpu(), dO[:1, :n].cpu(), scale=w.scale_value, score_mod="bias_tensor",
                             norm=norm, mask=w.mask, bias_tensor=bt[:, :n])
    for name, g, r in zip(("dQ", "dK", "dV"), (whole[0][:1, :n], whole[1][:1, :1], whole[2][:1, :1]), ref):
        check(g.cpu().double().numpy(), r, f"{w.name} {name}")


SELECTING = {
    "retention": dict(score_mod="head_decay", norm="abssum", mask="causal", decay=True),
    "abs_of_sum": dict(norm="abs_of_sum", score_mod="bias", bias=3.0, mask="causal"),
    "decay_nonorm": dict(score_mod="head_decay", norm="none", mask="causal", decay=True, scale=0.01),
    "none_window": dict(norm="none", mask="sliding_window", window=40, scale=0.01),
    "none_bias_tensor": dict(norm="none", score_mod="bias_tensor", mask="causal", scale=0.01),
    "relu": dict(score_mod="relu", norm="none", scale=0.01),
    "relu_causal": dict(score_mod="relu", norm="none", mask="causal", scale=0.01),
}


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("form", sorted(SELECTING))
def test_backward_hidden_entries_stay_zero(A, dims, form):
    """The retention, no-normalization and ReLU forms select the score gradient 0 of a hidden (or clipped) entry: an
    infinite value row changes dQ of no query that does not see it (or clips it), an infinite row of dO changes dK of no
    key hidden from that query, not by a bit."""
    if form == "none_bias_tensor" and dims == (128, 256):
        pytest.skip("the bias tensor does not come with head dims 128/256")
    dev = torch.device("cuda:0")
    w = Workload("bwd_select", 47, 1, 4, 2, 150, 163, dims[0], dims[1], **SELECTING[form])
    Q, K, V = (t.to(dev) for t in make_inputs(w))
    dO = make_grad(w).to(dev)
    bt = torch.zeros((1, 1, 150, 168), dtype=torch.bfloat16, device=dev)[..., :163] if form == "none_bias_tensor" else None
    stats = torch.empty((1, 4, 150), dtype=torch.float32, device=dev) if w.norm in ("abssum", "abs_of_sum") else None
    O = A.run_workload(w, Q, K, V, stats=stats, bias_tensor=bt)

    def grads(V, dO):
        out = A.attention_backward(Q, K, V, O if stats is not None else None, dO, stats, scale=w.scale_value, score_mod=w.score_mod,
                                   bias=w.bias, gamma=w.gamma(), norm=w.norm, mask=w.mask, window=w.window, bias_tensor=bt,
                                   want_dbias=bt is not None)
        torch.cuda.synchronize()
        return out

    i = torch.arange(150, device=dev).view(-1, 1) + 13
    j = torch.arange(163, device=dev).view(1, -1)
    zero = torch.zeros((1, 4, 150, 163), dtype=torch.bool, device=dev)
    if w.mask != "none":
        zero |= j > i
    if w.mask == "sliding_window":
        zero |= j <= i - w.window
    if w.score_mod == "relu":
        zero |= (Q.double() @ K.double().repeat_interleave(2, 1).transpose(2, 3)) < 0
    clean = grads(V, dO)
    Vx = V.clone()
    Vx[0, :, 100, 3] = float("inf")
    got = grads(Vx, dO)
    free = zero[:, :, :, 100]
    assert free.any() and torch.equal(got[0][free], clean[0][free])
    assert not torch.isfinite(got[0][~free]).all()
    if bt is not None:
        assert torch.equal(got[3][free], clean[3][free])
    dOx = dO.clone()
    dOx[0, ::2, 60, 3] = float("inf")  # one q head of each group
    got = grads(V, dOx)
    free = zero[:, ::2, 60, :]
    assert free.any() and torch.equal(got[1][free], clean[1][free])
    assert not torch.isfinite(got[1][~free]).all()


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("norm", ["abssum", "abs_of_sum", "none"])
@pytest.mark.parametrize("L", [100, 300])  # (one wavefront per 32 rows, and the pairs, where a head dim has both)
def test_backward_vanished_decay_passes_infinities_on(A, dims, norm, L):
    """An entry is left out because it is hidden, not because its decay vanishes: with a rate of 1e-4 the factor is 0 in 32 bits from ten
    tokens on, and an infinite value row or row of dO still reaches every query or key that sees it, in tiles that are visible as a whole
    and in those on the diagonal alike (the oracle's product in 64 bits is infinite), and no other."""
    dev = torch.device("cuda:0")
    w = Workload("vanished", 48, 1, 4, 2, L, L, dims[0], dims[1], mask="causal")
    Q, K, V = (t.to(dev) for t in make_inputs(w))
    dO = make_grad(w).to(dev)
    args = dict(scale=w.scale_value, score_mod="head_decay", gamma=[1e-4] * 4, norm=norm, mask="causal")
    stats = torch.empty((1, 4, L), dtype=torch.float32, device=dev) if norm != "none" else None
    O = A.attention_forward(Q, K, V, stats=stats, **args)
    t = torch.arange(L, device=dev)
    Vx = V.clone()
    Vx[0, :, 35, 3] = float("inf")  # (queries 46 to 63 share a tile of the diagonal with it, later ones do not)
    bad = ~torch.isfinite(A.attention_backward(Q, K, Vx, O, dO, stats, **args)[0]).all(-1)
    assert torch.equal(bad, (t >= 35).expand_as(bad))
    dOx = dO.clone()
    dOx[0, :, 60, 3] = float("inf")
    bad = ~torch.isfinite(A.attention_backward(Q, K, V, O, dOx, stats, **args)[1]).all(-1)
    assert torch.equal(bad, (t <= 60).expand_as(bad))


def test_more_workgroups_than_one_launch_holds(A):
    # 8.4 million heads of one token: either side of the backward pass has 2^31 threads, both together more than a launch holds.  With
    # s = scale q . k and d = scale v . dO (64 terms each, summed in 32 bits: 2^-18 of the sum of their absolute values), rounded to
    # bf16 (2^-9): dQ = d k, dK = d q, dV = s dO
    B, H, D = 131073, 64, 64
    g = torch.Generator("cuda").manual_seed(90)
    Q, K, V, dO = (torch.randn(B, H, 1, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    dQ, dK, dV = A.attention_backward(Q, K, V, None, dO, None, scale=0.1, norm="none")
    n = 10000
    for b0 in range(0, B, n):
        q, k, v, do = (t[b0:b0 + n].double() for t in (Q, K, V, dO))
        s, d = 0.1 * (q * k).sum(-1, keepdim=True), 0.1 * (v * do).sum(-1, keepdim=True)
        es, ed = 0.1 * (q * k).abs().sum(-1, keepdim=True), 0.1 * (v * do).abs().sum(-1, keepdim=True)
        for name, got, w, e, x in (("dQ", dQ, d, ed, k), ("dK", dK, d, ed, q), ("dV", dV, s, es, do)):
            assert ((got[b0:b0 + n].double() - w * x).abs() <= (2.0 ** -8 * w.abs() + 2.0 ** -17 * e) * x.abs() + 1e-7).all(), (name, b0)


def decay_rates_bound(Q, K, V, dO, gam, scale, norm):
    """Element by element, what the gradients of an attention with decay may be away from those in 64 bits.  Units: u = 2^-8, the rounding of
    P and dS' to bfloat16 (eight significant bits, to nearest), an eighth more for the 32-bit factors and sums; v = 2^-16, 256 roundings of 2^-24 in a product of
    up to 256 terms.  |dP - delta| may be far below |dP| and |delta|, and delta has the roundings of the forward pass's P.  Factors
    below 2^-126 are 0 in 32 bits: with sums below 2^26, 2^-100."""
    u, v, f64 = 1.125 * 2.0 ** -8, 2.0 ** -16, torch.float64
    g = Q.shape[1] // K.shape[1]
    q, do = Q.to(f64), dO.to(f64)
    k, val = (t.to(f64).repeat_interleave(g, 1) for t in (K, V))
    dist = torch.arange(Q.shape[2]).view(-1, 1) + K.shape[2] - Q.shape[2] - torch.arange(K.shape[2])
    dec = torch.where(dist >= 0, torch.tensor(gam, dtype=f64).view(-1, 1, 1) ** dist.clamp(min=0), 0.0)
    s = q @ k.transpose(2, 3) * scale * dec
    n = torch.ones_like(s[..., :1])
    if norm != "none":
        n = (s.abs() if norm == "abssum" else s).sum(-1, keepdim=True).abs().clamp(min=1.0)
    f, p = dec / n, s / n  # what dP - delta and q . k are multiplied with; P
    e_p = u * p.abs() + v * f * scale * (q.abs() @ k.abs().transpose(2, 3))
    dp, e_dp = (do @ val.transpose(2, 3)).abs(), v * (do.abs() @ val.abs().transpose(2, 3))
    e_delta = 0.0 if norm == "none" else (e_p * dp + 2 * p.abs() * e_dp).sum(-1, keepdim=True)
    delta = 0.0 if norm == "none" else (p * (do @ val.transpose(2, 3))).sum(-1, keepdim=True).abs()
    e_ds = u * f * (dp + delta) + f * (e_dp + e_delta)
    fold = lambda t: t.view(t.shape[0], -1, g, *t.shape[2:]).sum(2)
    return tuple(t + 2.0 ** -100 for t in (scale * (e_ds @ k.abs()), fold(scale * (e_ds.transpose(2, 3) @ q.abs())), fold(e_p.transpose(2, 3) @ do.abs())))


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"d{d[0]}_{d[1]}")
@pytest.mark.parametrize("norm", ["abssum", "abs_of_sum", "none"])
def test_backward_decay_rates(A, dims, norm):
    """Decay rates above one, of one, and so small that a factor vanishes within a tile: tiles that are visible as a whole form the factors
    as products (one exponential per lane times constants), the others one by one.  Heads with small rates share a k/v head, and every
    element has a bound of its own: the gradients of the rate above one are a thousand times the others'."""
    w = Workload("rates", 990, 2, 4, 2, 200, 330, *dims, score_mod="head_decay", norm=norm, mask="causal")
    gam = [1.02, 1.0, 0.05, 1e-4]
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    dev = torch.device("cuda:0")
    args = dict(scale=w.scale_value, score_mod="head_decay", gamma=gam, norm=norm, mask="causal")
    Qd, Kd, Vd = Q.to(dev), K.to(dev), V.to(dev)
    stats = None if norm == "none" else torch.empty((2, 4, 200), dtype=torch.float32, device=dev)
    O = A.attention_forward(Qd, Kd, Vd, stats=stats, **args)
    got = A.attention_backward(Qd, Kd, Vd, O, dO.to(dev), stats, **args)
    ref = attention_backward(Q, K, V, dO, **args)
    bounds = decay_rates_bound(Q, K, V, dO, gam, w.scale_value, norm)
    for name, x, r, bound in zip(("dQ", "dK", "dV"), got, ref, bounds):
        err = np.abs(x.cpu().double().numpy() - r) / bound.numpy()
        for h in range(r.shape[1]):
            share = np.linalg.norm(bound.numpy()[:, h]) / np.linalg.norm(r[:, h])
            print(f"{norm} {dims} {name} head {h}: {err[:, h].max():.3f} of the bound, which is {share:.4f} of the norm", flush=True)
            assert share < 0.02 or gam[h * 4 // r.shape[1]] >= 1  # (a bound that zeros would not meet)
        assert err.max() <= 1.0, (name, err.max())
        # The large rates' bound adds up what mostly cancels.  Of the norm, which they dominate: the roundings of the weights, of dS' and,
        # through delta, of the forward weights, less than 2^-9 each in the root mean square.
        err = np.linalg.norm(x.cpu().double().numpy() - r) / np.linalg.norm(r)
        assert err <= 3 * 2.0 ** -9, (name, err)
