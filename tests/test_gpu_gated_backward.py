"""GPU parity of the backward pass of the recurrent pattern with per-token gates (ae_gated_backward, through the C
ABI) against the fp64 token-by-token backward oracle on the same seeded inputs.

Bars.  dQ, dK, dV: as for the forward pass -- max-abs <= 1e-2 and mean-abs <= 1e-3 relative to max(1, the largest
|reference| of the row); each is one run of the forward kernel on other operands (bf16 operands, bf16 weights and
state into the MFMAs, fp32 accumulation).

dlog_decay and dkey_gate are one number per token, and a bar of their own is derived from the arithmetic.  With
G_ij = P_ij dP_ij (forward weight times its gradient), q_i . dq_i is the sum of row i of G, k_j . dk_j the sum of
column j, dkey_gate_j = k_j . dk_j / g_j, and dlog_decay_t = sum_{i >= t} (q_i . dq_i - k_i . dk_i).  Row sums and
column sums come out of different runs of the kernel, each of which rounds its weights (and the carried state, and
the weighted values that update it) to bf16: every term G_ij carries an independent relative error of up to 2^-9
per rounding, about 2^-9 in standard deviation for the three together.  A sum of such terms is off by 2^-9 times the
root of the sum of their squares.  The tests form G from the inputs (its entries are what the model needs, not an
expected value) and hold
    dkey_gate_j   to  3 x 2^-9 x sum_i |G_ij| / g_j                                         (+ 1e-4 absolute),
    dlog_decay_t  to  8 x 2^-9 x sqrt(sum_{i >= t} (sum_j G_ij^2 + sum_j G_ji^2))           (+ 1e-3 absolute).
The first is the worst case of the three roundings (a column of G has few terms of weight, and the rounded state and
the rounded weighted values are shared by many of them, so their errors add up coherently rather than at random).
The second is eight standard deviations of the model: a long sum over many tokens, near enough to Gaussian, with
the same shared roundings fattening its tails (measured: the mean error is 0.8 standard deviations, as the model
says; the worst of some 10^5 tokens 7.1).  At the benchmark size, where G does not fit, the root of a sum of squares is
replaced by max(|sum|, rms of such sums over the head): for terms of random sign the two are of one size.  The errors
of unrelated pairs (i, j >= t) do not cancel in the suffix sum as their exact values do, which is why the bar grows
with the root of the number of later tokens; an implementation that forms both sums from one set of rounded weights
would not need that.
"""
import math

import numpy as np
import pytest
import torch

from oracle.gated_recurrent_backward_oracle import gated_recurrent_backward as oracle_backward
from oracle.gated_recurrent_backward_oracle import gated_recurrent_backward_head
from paper_2502_15349_amd.workloads import Workload, make_gates, make_grad, make_inputs

pytestmark = pytest.mark.gpu
MAX_ABS, MEAN_ABS = 1e-2, 1e-3


@pytest.fixture(scope="module")
def A():
    from paper_2502_15349_amd import ae_attn
    return ae_attn


def check_rows(got, ref, what):
    assert np.isfinite(got).all(), what
    rs = np.maximum(np.abs(ref).max(axis=-1, keepdims=True), 1.0)
    err = np.abs(got - ref) / rs
    print(f"{what}: max_abs {err.max():.3e} mean_abs {err.mean():.3e} |ref|max {np.abs(ref).max():.3e}", flush=True)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (what, err.max(), err.mean())


def inputs(cid, B, H, H_qk, L, dqk, dv, kind):
    Q, K, _ = make_inputs(Workload("gq", cid, B, H_qk, H_qk, L, L, dqk, dqk))
    wv = Workload("gv", cid, B, H, H, L, L, dv, dv)
    _, _, V = make_inputs(wv)
    dO = make_grad(wv)
    la, kg = make_gates(B, H, L, 1000 * cid + 5, kind)
    return Q, K, V, la, kg, dO


def run(A, Q, K, V, la, kg, dO, scale):
    dev = torch.device("cuda:0")
    r = A.gated_recurrent_backward(Q.to(dev), K.to(dev), V.to(dev), la.to(dev), None if kg is None else kg.to(dev), dO.to(dev),
                                   scale=scale)
    torch.cuda.synchronize()
    return [None if t is None else t.cpu().double().numpy() for t in r]


U = 2.0 ** -9


def check_tokens(got, bound, ref, what):
    """Per-token quantities [.., L] against the derived bound (same shape)."""
    assert np.isfinite(got).all(), what
    ratio = np.abs(got - ref) / bound
    print(f"{what}: worst error / bound {ratio.max():.3f}, mean {ratio.mean():.3f} |ref|max {np.abs(ref).max():.3e}", flush=True)
    assert ratio.max() <= 1.0, (what, ratio.max())


def token_bounds_proxy(qdq, kdk):
    """The bar of dlog_decay where G is too large to form: qdq, kdk are the oracle's q_i . dq_i and k_i . dk_i [L]."""
    def floored(x):
        return np.maximum(np.abs(x), np.sqrt(np.mean(x ** 2, axis=-1, keepdims=True)))
    return 8 * U * np.sqrt(np.cumsum((floored(qdq) ** 2 + floored(kdk) ** 2)[..., ::-1], axis=-1)[..., ::-1]) + 1e-3


def head_bounds(q, k, v, la, g, dO, scale):
    """One value head: G_ij = P_ij dP_ij from the inputs, and from it the bars of dlog_decay and dkey_gate [L]."""
    L = q.shape[0]
    B = np.cumsum(la)
    expo = B[:, None] - B[None, :]
    A = np.where(np.tril(np.ones((L, L), dtype=bool)), np.exp(np.minimum(expo, 0.0)), 0.0)
    gg = np.ones(L) if g is None else g
    G = scale * A * (q @ k.T) * gg[None, :] * (dO @ v.T)
    row2, col2 = np.sum(G * G, axis=1), np.sum(G * G, axis=0)
    b_dla = 8 * U * np.sqrt(np.cumsum((row2 + col2)[::-1])[::-1]) + 1e-3
    b_dkg = 3 * U * np.sum(np.abs(G), axis=0) / np.abs(gg) + 1e-4
    return b_dla, b_dkg


def all_bounds(Q, K, V, la, kg, dO, scale):
    Bn, H, L = la.shape
    grp = H // Q.shape[1]
    b_dla, b_dkg = np.zeros((Bn, H, L)), np.zeros((Bn, H, L))
    for b in range(Bn):
        for h in range(H):
            b_dla[b, h], b_dkg[b, h] = head_bounds(Q[b, h // grp], K[b, h // grp], V[b, h], la[b, h], None if kg is None else kg[b, h],
                                                   dO[b, h], scale)
    return b_dla, b_dkg


def compare(got, ref, what, with_gate, dots):
    dQ, dK, dV, dla, dkg = got
    check_rows(dQ, ref["dQ"], what + " dQ")
    check_rows(dK, ref["dK"], what + " dK")
    check_rows(dV, ref["dV"], what + " dV")
    b_dla, b_dkg = dots
    check_tokens(dla, b_dla, ref["dlog_decay"], what + " dlog_decay")
    if with_gate:
        check_tokens(dkg, b_dkg, ref["dkey_gate"], what + " dkey_gate")
    else:
        assert dkg is None


def oracle_all(Q, K, V, la, kg, dO, scale):
    n = [Q.float().numpy().astype(np.float64), K.float().numpy().astype(np.float64), V.float().numpy().astype(np.float64),
         la.numpy().astype(np.float64), None if kg is None else kg.numpy().astype(np.float64), dO.float().numpy().astype(np.float64)]
    return oracle_backward(*n, scale=scale), all_bounds(*n, scale)


@pytest.mark.parametrize("dqk,dv", [(64, 64), (128, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("kind", ["gated_retention", "mamba2"])
@pytest.mark.parametrize("L", [1, 63, 64, 65, 200, 513])
def test_matches_oracle(A, dqk, dv, kind, L):
    Q, K, V, la, kg, dO = inputs(900 + L % 7, 2, 3, 3, L, dqk, dv, kind)
    scale = 1.0 / math.sqrt(dqk)
    print(f"case {kind} {dqk}/{dv} L {L}", flush=True)
    got = run(A, Q, K, V, la, kg, dO, scale)
    ref, dots = oracle_all(Q, K, V, la, kg, dO, scale)
    compare(got, ref, f"{kind} {dqk}/{dv} L={L}", kg is not None, dots)


@pytest.mark.parametrize("dqk,dv", [(128, 64), (64, 64)])
def test_grouped_query_key_heads(A, dqk, dv):
    # Mamba2's structure at a reduced head count: B and C shared by the value heads of a group; dQ and dK are sums
    # over the group
    Q, K, V, la, kg, dO = inputs(910, 1, 8, 2, 300, dqk, dv, "mamba2")
    got = run(A, Q, K, V, la, kg, dO, 1.0)
    ref, dots = oracle_all(Q, K, V, la, kg, dO, 1.0)
    compare(got, ref, f"mamba2 groups {dqk}/{dv}", True, dots)


@pytest.mark.parametrize("dqk", [64, 128])
@pytest.mark.parametrize("H,H_qk,heads", [(256, 128, 2), (384, 128, 3), (320, 64, 3)])
@pytest.mark.parametrize("kind,L", [("gated_retention", 64), ("mamba2", 130), ("mamba2", 193)])
def test_several_heads_per_workgroup(A, dqk, H, H_qk, heads, kind, L):
    # more value heads than compute units: a workgroup takes two or three heads of a group in turn (of five: three, then two)
    Q, K, V, la, kg, dO = inputs(930 + L % 7, 2, H, H_qk, L, dqk, 64, kind)
    h = A.ae_gated_create(B=2, H=H, H_qk=H_qk, L=L, D_qk=dqk, D_v=64, scale=0.1)
    parts = -(-(H // H_qk) // heads)
    assert A.ae_gated_backward_workspace_bytes(h) == (2 * H * L * 4 + 255) // 256 * 256 + 2 * 2 * H_qk * parts * L * dqk * 4
    A.ae_gated_destroy(h)
    dQ, dK, dV, dla, dkg = run(A, Q, K, V, la, kg, dO, 0.1)
    # The same with every head given its own copy of its q/k head, which is the path of one head per workgroup (held to the oracle
    # above): the same products from the same operands, so what is left is the order of sums in 32 bits -- 2^-23 of the sum of
    # the absolute terms for every addition.
    grp = H // H_qk
    Qx, Kx = (t.repeat_interleave(grp, dim=1) for t in (Q, K))
    eQ, eK, eV, ela, ekg = run(A, Qx, Kx, V, la, kg, dO, 0.1)
    eps = 2.0 ** -23

    def close(got, ref, bound, what):
        ratio = np.abs(got - ref) / (bound + 1e-30)
        print(f"{heads} heads per workgroup {kind} {dqk}/64 L={L} {what}: worst error / bound {ratio.max():.3f}", flush=True)
        assert np.isfinite(got).all() and ratio.max() <= 1.0, (what, ratio.max())

    for name, g, e in (("dQ", dQ, eQ), ("dK", dK, eK)):
        e = e.reshape(2, H_qk, grp, L, dqk)
        close(g, e.sum(axis=2), 2 * grp * eps * np.abs(e).sum(axis=2) + 1e-7, name)
    assert np.array_equal(dV, eV)
    q, k = Qx.double().numpy(), Kx.double().numpy()
    rows_q, rows_k = np.abs(q * eQ).sum(axis=-1), np.abs(k * eK).sum(axis=-1)
    if kg is not None:
        close(dkg, ekg, 2 * dqk * eps * rows_k / kg.double().numpy() + 1e-7, "dkey_gate")
    close(dla, ela, (2 * dqk * eps * (rows_q + rows_k) + 1e-7)[..., ::-1].cumsum(axis=-1)[..., ::-1] + 2 * eps * np.abs(ela), "dlog_decay")


@pytest.mark.parametrize("dqk,dv,B,H,H_qk,L", [(64, 64, 1, 3, 3, 200), (128, 64, 2, 6, 2, 129), (128, 64, 2, 132, 22, 130), (64, 128, 1, 2, 2, 64),
                                               (128, 128, 1, 2, 2, 1061)])
def test_gate_multiplies_finished_rows_of_dv(A, dqk, dv, B, H, H_qk, L):
    # the key gate of token j is a factor of row j of dV and of nothing that is summed into it: one product in 32 bits, so dV is
    # that of a call without gates times the gates, bit for bit -- whole and cut walks, one head per workgroup and two
    Q, K, V, la, kg, dO = inputs(950 + L % 7, B, H, H_qk, L, dqk, dv, "mamba2")
    dV, bare = (run(A, Q, K, V, la, g, dO, 0.1)[2] for g in (kg, None))
    assert np.array_equal(dV, (bare.astype(np.float32) * kg.numpy()[..., None]).astype(np.float64))


@pytest.mark.parametrize("dqk,dv", [(64, 64), (128, 64), (64, 128), (128, 128)])
def test_batch_entries_do_not_depend_on_the_launches(A, dqk, dv):
    # 180 (batch, head) pairs: more workgroups than compute units, of which (64/64) two share one; 60 at a time have one each
    Q, K, V, la, kg, dO = inputs(940, 3, 60, 60, 321, dqk, dv, "mamba2")
    whole = run(A, Q, K, V, la, kg, dO, 0.1)
    for b in range(3):
        part = run(A, *(t[b:b + 1].contiguous() for t in (Q, K, V, la, kg, dO)), 0.1)
        for x, y in zip(whole, part):
            assert np.array_equal(x[b:b + 1], y)


@pytest.mark.parametrize("dqk", [64, 128])
@pytest.mark.parametrize("H,H_qk,L", [(32, 8, 130), (80, 1, 130), (61, 1, 64), (62, 1, 65), (62, 2, 1), (62, 2, 129)])
def test_four_heads_per_workgroup(A, dqk, H, H_qk, L):
    # Groups of 4 (one workgroup each: no sums are left), 80, 61, 62 and 31 value heads, taken four at a time and, in
    # the last part, four, one, two or three, against the same heads with a q/k head each: sums of n values x in 32 bits, each operation within 2^-24 of its
    # result, so within 2^-23 n of the sum of |x|; the row products k . x have dqk terms.
    B, n = 8, H // H_qk
    Q, K, V, la, kg, dO = (t.cuda() for t in inputs(950, B, H, H_qk, L, dqk, 64, "mamba2"))
    h = A.ae_gated_create(B=B, H=H, H_qk=H_qk, L=L, D_qk=dqk, D_v=64, scale=0.1)
    rows = (B * H * L * 4 + 255) // 256 * 256
    parts = (A.ae_gated_backward_workspace_bytes(h) - rows) // (2 * B * H_qk * L * dqk * 4)
    A.ae_gated_destroy(h)
    assert parts == (n + 3) // 4
    dQ, dK, dV, dla, dkg = A.gated_recurrent_backward(Q, K, V, la, kg, dO, scale=0.1)
    Qx, Kx = (t.repeat_interleave(n, dim=1) for t in (Q, K))
    eQ, eK, eV, ela, ekg = A.gated_recurrent_backward(Qx, Kx, V, la, kg, dO, scale=0.1)
    assert torch.equal(dV, eV)
    for got, ref in ((dQ, eQ), (dK, eK)):
        ref = ref.double().view(B, H_qk, n, L, dqk)
        assert ((got.double() - ref.sum(dim=2)).abs() <= 2.0 ** -23 * n * ref.abs().sum(dim=2) + 1e-30).all()
    terms = (Kx.double() * eK.double()).abs().sum(-1) / kg.double()  # of k . x, where eK = g x
    assert ((dkg.double() - ekg.double()).abs() <= 2.0 ** -23 * dqk * terms + 1e-30).all()
    later = ((Qx.double() * eQ.double()).abs().sum(-1) + (Kx.double() * eK.double()).abs().sum(-1)).flip(-1).cumsum(-1).flip(-1)
    assert ((dla.double() - ela.double()).abs() <= 2.0 ** -23 * (dqk + 2) * later + 1e-30).all()


@pytest.mark.parametrize("dqk,dv,H,H_qk", [(128, 128, 2, 2), (64, 64, 3, 3), (128, 64, 4, 1)])
@pytest.mark.parametrize("kind", ["gated_retention", "mamba2"])
@pytest.mark.parametrize("L", [1061, 2560])
def test_few_heads_long_sequence(A, dqk, dv, H, H_qk, kind, L):
    # shapes whose walks the library cuts into segments (6 and 20 here, the last one short), forwards and backwards
    Q, K, V, la, kg, dO = inputs(920 + L % 5, 1, H, H_qk, L, dqk, dv, kind)
    scale = 1.0 / math.sqrt(dqk)
    got = run(A, Q, K, V, la, kg, dO, scale)
    ref, dots = oracle_all(Q, K, V, la, kg, dO, scale)
    compare(got, ref, f"segments {kind} {dqk}/{dv} L={L}", kg is not None, dots)


def test_strong_decay_and_no_decay(A):
    # per-token decays of e^-8, none at all (gradients are plain suffix sums), and a slow decay broken by single
    # tokens of e^-30
    w = Workload("dec", 913, 1, 3, 3, 260, 260, 64, 64)
    Q, K, V = make_inputs(w)
    dO = make_grad(w)
    la = torch.full((1, 3, 260), -8.0)
    la[:, 1] = 0.0
    la[:, 2] = -0.01
    la[:, 2, 5::37] = -30.0
    got = run(A, Q, K, V, la, None, dO, 0.125)
    ref, dots = oracle_all(Q, K, V, la, None, dO, 0.125)
    compare(got, ref, "decay e^-8 / none / resets", False, dots)


def test_sampled_heads_at_benchmark_size(A):
    # 8 x 32 heads x 8192 tokens, 128/128, gated retention: three heads against the oracle
    B, H, L = 8, 32, 8192
    Q, K, V, la, kg, dO = inputs(914, B, H, H, L, 128, 128, "gated_retention")
    scale = 1.0 / math.sqrt(128)
    dQ, dK, dV, dla, _ = run(A, Q, K, V, la, kg, dO, scale)
    for b, h in ((0, 0), (3, 17), (7, 31)):
        ref = gated_recurrent_backward_head(Q[b, h].float().numpy(), K[b, h].float().numpy(), V[b, h].float().numpy(), la[b, h].numpy(),
                                            None, dO[b, h].float().numpy(), scale=scale)
        check_rows(dQ[b, h], ref["dq"], f"benchmark size ({b},{h}) dQ")
        check_rows(dK[b, h], ref["dk"], f"benchmark size ({b},{h}) dK")
        check_rows(dV[b, h], ref["dv"], f"benchmark size ({b},{h}) dV")
        qn, kn = Q[b, h].float().numpy().astype(np.float64), K[b, h].float().numpy().astype(np.float64)
        b_dla = token_bounds_proxy(np.sum(qn * ref["dq"], axis=-1), np.sum(kn * ref["dk"], axis=-1))
        check_tokens(dla[b, h], b_dla, ref["dlog_decay"], f"benchmark size ({b},{h}) dlog_decay")


def test_one_workgroup_per_compute_unit_again_at_many_tokens(A):
    # 64/64: the three walks of 256 pairs x 4096 fill three rounds of one workgroup per compute unit each; those of 128 pairs share
    B, H, L = 8, 32, 4096
    g = torch.Generator("cuda").manual_seed(91)
    Q, K, V, dO = (torch.randn(B, H, L, 64, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    la = torch.nn.functional.logsigmoid(torch.randn(B, H, L, generator=g, device="cuda")) / 16
    whole = A.gated_recurrent_backward(Q, K, V, la, None, dO, scale=0.125)
    for b in (0, 4):
        part = A.gated_recurrent_backward(*(t[b:b + 4].contiguous() for t in (Q, K, V, la)), None, dO[b:b + 4].contiguous(), scale=0.125)
        for x, y in zip(whole[:4], part[:4]):
            assert torch.equal(x[b:b + 4], y)


@pytest.mark.parametrize("B,H_qk", [(59375, 64), (89063, 32)])
def test_more_workgroups_than_one_launch_holds(A, B, H_qk):
    # 3.8 and 5.7 million (batch, head) pairs of one token, 64 heads each (alone, or in groups of two): the three walks have more than
    # 2^32 threads.  With s = q . k, d = v . dO (64 terms each, summed in 32 bits: 2^-18 of the sum of their absolute values) and weights
    # in bf16 (2^-9 of themselves): dq = scale g d k, dk = scale g d q, dv = scale g s dO, dg = scale s d, and no gradient of the decay
    # but the difference of two such products.
    H, D = 64, 64
    g = torch.Generator("cuda").manual_seed(89)
    Q, K = (torch.randn(B, H_qk, 1, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    V, dO = (torch.randn(B, H, 1, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    kg = torch.rand(B, H, 1, generator=g, device="cuda")
    dQ, dK, dV, dla, dkg = A.gated_recurrent_backward(Q, K, V, torch.zeros(B, H, 1, device="cuda"), kg, dO, scale=0.1)
    n, grp = 5000, H // H_qk
    for b0 in range(0, B, n):
        q, k, v, do, w = (t[b0:b0 + n].double() for t in (Q, K, V, dO, kg.unsqueeze(-1)))
        qx, kx = (t.repeat_interleave(grp, dim=1) for t in (q, k))
        s, d = 0.1 * (qx * kx).sum(-1, keepdim=True), (v * do).sum(-1, keepdim=True)
        es, ed = 0.1 * (qx * kx).abs().sum(-1, keepdim=True), (v * do).abs().sum(-1, keepdim=True)

        def close(got, ref, size, terms, what):
            assert ((got[b0:b0 + n].double() - ref).abs() <= 2.0 ** -8 * size + 2.0 ** -17 * terms + 1e-6).all(), (what, b0)

        def group(x):
            return x.reshape(x.shape[0], H_qk, grp, 1, -1).sum(dim=2)

        close(dV, w * s * do, (w * s * do).abs(), w * es * do.abs(), "dV")
        close(dQ, group(0.1 * w * d * kx), group((0.1 * w * d * kx).abs()), group(0.1 * w * ed * kx.abs()), "dQ")
        close(dK, group(0.1 * w * d * qx), group((0.1 * w * d * qx).abs()), group(0.1 * w * ed * qx.abs()), "dK")
        close(dkg, (s * d)[..., 0], (es * d.abs())[..., 0], (es * ed)[..., 0], "dkey_gate")
        close(dla, torch.zeros_like((s * d)[..., 0]), 2 * (w * es * d.abs())[..., 0], 2 * (w * es * ed)[..., 0], "dlog_decay")
