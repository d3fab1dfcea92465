"""GPU parity of the HyperNEAT path (tn_cppn_query, tn_substrate_forward,
tn_substrate_backward, tn_cppn_backward) against the float64 oracle. Every
oracle input is synthetic or the oracle's own: substrate kernels get seeded
synthetic bfloat16 weights, inputs and activations; threshold decisions on the
oracle side are its own float64 ones, and where such a decision could differ
from the GPU's float32 one (|w_ref| within the forward tolerance of the
threshold: "ambiguous") the upstream gradient is set to 0 on both sides, or
the bound carries the flip.

CPPN values (before the threshold): the forward tolerance of test_gpu_forward,
|w - w_ref| <= 1e-5 * cond + 2^-100. Stored weights: bit-exact round to
nearest even of the GPU's own thresholded float32 value; threshold decisions
equal the oracle's except where |w_ref| lies within the forward tolerance of
the threshold (counted, not compared: both sides take the decision in their own
precision there).
Substrate: with the GPU's bfloat16 weights and inputs as exact float64 values
(their products are exact in float32), float32 accumulation of K = 1024 terms
errs by at most K * 2^-24 = 2^-14 times the sum of the terms' magnitudes, so
|h - tanh(z_ref)| <= 2^-14 * sum_s |x_s w_s| + 2^-21 (the last term: tanh's
own error from the hardware exp and reciprocal), and y against bf16(h) W2
within 2^-14 * sum_t |bf16(h_t) w_t|. End to end against the float64 oracle
with float64 weights (the GPU's threshold decisions): |y - y_ref| <= 2^-7 *
error_scale: the four bfloat16 roundings take at most 2^-8 of it (pinned in
test_oracle_hyperneat), the accumulations and the CPPN's float32 error (below
1e-5 relative) stay inside the remaining factor of two.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import host, to_device
from helpers import population_from_rows
from oracle import hyperneat as hn

pytestmark = pytest.mark.gpu
GRID, NOUT, THR = 32, 8, 0.2


def _bf16_bits(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    nan = np.isnan(np.asarray(x, np.float32))
    r = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    r[nan] = 0x7FC0
    return r


def _bits16(t):
    return host(t.view(torch.int16)).view(np.uint16)


def _bf16_value(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def _query(P, seed=5):
    import paper_2504_08339_amd as tn
    pop = synth.cppn_population(seed=seed, P=P)
    dp = to_device(pop)
    tr = tn.transform(dp)
    w1t, w2t, r1, r2 = tn.cppn_query(dp, tr, GRID, NOUT, THR, raw=True)
    return tn, pop, dp, tr, w1t, w2t, r1, r2


def _check_genome(pop, g, r1, r2, w1b, w2b):
    gen = oracle.decode(pop, g)
    tr = oracle.transform(gen)
    grid, outs = hn.grid_coords(GRID), hn.row_coords(NOUT)
    ambiguous = 0
    for src_xy, dst_xy, raw, wb in ((grid, grid, r1[g], w1b[g]), (grid, outs, r2[g], w2b[g])):
        ref, cond = oracle.forward(gen, tr, hn.query_inputs(src_xy, dst_xy), with_cond=True)
        ref = ref[:, 0].reshape(len(src_xy), len(dst_xy)).T      # [t][s]
        cond = cond[:, 0].reshape(len(src_xy), len(dst_xy)).T
        tol = 1e-5 * cond + 2.0 ** -100
        if tr.status:
            assert np.isnan(raw).all()
            continue
        err = np.abs(raw.astype(np.float64) - ref)
        assert np.all(err <= tol), (g, float(err.max()))
        kept = np.where(np.abs(raw) < THR, np.float32(0), raw)
        assert np.array_equal(wb, _bf16_bits(kept))   # consistency of the two outputs
        near = np.abs(np.abs(ref) - THR) <= tol
        ambiguous += int(near.sum())
        same = (np.abs(raw) < THR) == (np.abs(ref) < THR)
        assert np.all(same | near)
        # the stored weight against the oracle's thresholded value: one bfloat16
        # rounding (2^-8 relative) plus the float32 error, away from the threshold
        want = hn.threshold(ref, THR)
        diff = np.abs(_bf16_value(wb) - want)
        assert np.all((diff <= 2.0 ** -8 * np.abs(want) + tol) | near), g
    return ambiguous


def test_cppn_query_matches_oracle():
    tn, pop, dp, tr, w1t, w2t, r1, r2 = _query(6)
    r1, r2 = host(r1), host(r2)
    w1b, w2b = _bits16(w1t), _bits16(w2t)
    assert w1b.shape == (6, 1024, 1024) and w2b.shape == (6, 8, 1024)
    amb = sum(_check_genome(pop, g, r1, r2, w1b, w2b) for g in range(pop.P))
    print("threshold decisions within tolerance of 0.2:", amb)
    assert (w1b != 0).any() and (w1b == 0).any()      # the threshold did something


def test_cppn_query_flagged_and_shape_errors():
    import paper_2504_08339_amd as tn
    from helpers import population_from_rows
    good = [[k, 0.0, 1.0, 0, 0] for k in range(5)] + [[5, 0.1, 1.0, 2, 0]]
    cyc = good + [[7, 0.0, 1.0, 2, 0], [8, 0.0, 1.0, 2, 0]]
    pop = population_from_rows([(good, [[0, 5, 1.0, 1], [4, 5, 0.5, 1]]),
                                (cyc, [[7, 8, 1.0, 1], [8, 7, 1.0, 1], [8, 5, 1.0, 1]])], 5, 1,
                               N_max=12, C_max=6)
    dp = to_device(pop)
    tr = tn.transform(dp)
    w1t, w2t, r1, r2 = tn.cppn_query(dp, tr, 8, 2, THR, raw=True)
    assert host(tr.status)[1] != 0
    assert np.isnan(host(r1)[1]).all() and np.all(_bits16(w1t)[1] == 0x7FC0)
    assert np.isfinite(host(r1)[0]).all()
    with pytest.raises(tn.TNError):
        tn.cppn_query(dp, tr, 6, 2, THR)               # 36 nodes: not a multiple of 64
    xor = to_device(synth.xor_population(P=2))
    with pytest.raises(tn.TNError):
        tn.cppn_query(xor, tn.transform(xor), 8, 2, THR)   # not a 5 -> 1 CPPN
    u1 = torch.zeros((2, 64, 64), device="cuda")
    u2 = torch.zeros((2, 2, 64), device="cuda")
    dW, db = tn.cppn_backward(dp, tr, u1, u2, 8, 2, THR)
    assert np.isnan(host(dW)[1]).all() and np.isnan(host(db)[1]).all()
    assert np.all(host(dW)[0] == 0.0) and np.all(host(db)[0] == 0.0)


def _synthetic_weights(P, seed):
    """Seeded bfloat16 substrate weights, about half zero (as after a
    threshold), as device tensors of bfloat16 bits and their float64 values."""
    rng = np.random.default_rng(seed)
    S = GRID * GRID
    w1 = rng.standard_normal((P, S, S)).astype(np.float32) * np.float32(0.05)
    w1[rng.random(w1.shape) < 0.5] = 0.0
    w2 = rng.standard_normal((P, NOUT, S)).astype(np.float32) * np.float32(0.05)
    b1, b2 = _bf16_bits(w1), _bf16_bits(w2)
    t1 = torch.from_numpy(b1.view(np.int16)).cuda().view(torch.bfloat16)
    t2 = torch.from_numpy(b2.view(np.int16)).cuda().view(torch.bfloat16)
    return t1, t2, _bf16_value(b1), _bf16_value(b2)


def _bf16_input(shape, seed):
    X = np.random.default_rng(seed).standard_normal(shape).astype(np.float32)
    bits = _bf16_bits(X)
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16), _bf16_value(bits)


@pytest.mark.parametrize("shared", [True, False])
def test_substrate_forward_matches_oracle(shared):
    """h against tanh(X W1) in float64 on the same bfloat16 values (float32
    accumulation of K = 1024 exact products: 2^-14 of the magnitudes, plus
    tanh's 2^-21); y against the oracle's bf16(H) W2, where the GPU rounds its
    own float32 h: the two roundings can differ by one bfloat16 step per term
    (2^-8 of |H| |W2|) besides the accumulation's 2^-14."""
    import paper_2504_08339_amd as tn
    P, B = 4, 100
    w1t, w2t, W1, W2 = _synthetic_weights(P, 15)
    xb, Xv = _bf16_input((B, GRID * GRID) if shared else (P, B, GRID * GRID), 8)
    h, y = tn.substrate_forward(w1t, w2t, xb, GRID, NOUT, THR)
    h, y = host(h), host(y)
    for g in range(P):
        Xg = Xv if shared else Xv[g]
        H, _ = hn.substrate_forward(Xg, W1[g].T, W2[g].T)
        S1 = np.abs(Xg) @ np.abs(W1[g]).T
        assert np.all(np.abs(h[g] - H) <= 2.0 ** -14 * S1 + 2.0 ** -21), g
        Hb = _bf16_value(_bf16_bits(H.astype(np.float32)))
        mag = np.abs(Hb) @ np.abs(W2[g]).T
        assert np.all(np.abs(y[g] - Hb @ W2[g].T) <= (2.0 ** -8 + 2.0 ** -14) * mag + 1e-30), g


@pytest.mark.parametrize("grid,B", [(8, 1), (8, 129), (16, 127), (24, 128), (32, 257)])
def test_substrate_product_forms_agree(grid, B):
    """The product by LDS-direct loads (aligned operands) and by registers
    (inputs shifted by one element) take the same sums: equal bits, at sizes
    that fill a tile of 128 rows and columns, miss it and pass it; hidden
    values and, above 128 rows, the weight gradient."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(B)
    S, P = grid * grid, 3
    bf = lambda *shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).cuda() \
        .to(torch.bfloat16)
    w1t, w2t, x = bf(P, S, S) * 0.1, bf(P, 5, S) * 0.1, bf(P, B, S)
    shifted = torch.empty(P * B * S + 1, dtype=torch.bfloat16, device="cuda")[1:].view(P, B, S)
    shifted.copy_(x)
    h, _ = tn.substrate_forward(w1t, w2t, x, grid, 5, THR)
    h2, _ = tn.substrate_forward(w1t, w2t, shifted, grid, 5, THR)
    assert torch.equal(h.view(torch.int32), h2.view(torch.int32))
    ref = torch.tanh(torch.stack([x[g].float() @ w1t[g].float().T for g in range(P)]).double())
    assert (h - ref).abs().max() < 1e-4
    if B > 128:
        dy = torch.from_numpy(rng.standard_normal((P, B, 5)).astype(np.float32)).cuda()
        dw1t, _ = tn.substrate_backward(w2t, x, h, dy, grid, 5, THR)
        dz = (torch.stack([dy[g] @ w2t[g].float() for g in range(P)]) * (1 - h * h)).to(torch.bfloat16)
        want = torch.stack([dz[g].double().T @ x[g].double() for g in range(P)])
        size = torch.stack([dz[g].double().abs().T @ x[g].double().abs() for g in range(P)])
        assert ((dw1t - want).abs() <= 2.0 ** -7 * size).all()


@pytest.mark.parametrize("shared", [True, False])
def test_substrate_backward_matches_oracle(shared):
    """Gradients of sum(dY * Y) against the oracle's substrate adjoint on the
    same synthetic h, dY, weights and inputs. dw2t: float32 sums of B <= 128
    terms, |err| <= 2^-17 * sum_b |h dy|; dw1t: dZ rounded to bfloat16 (2^-9)
    plus float32 accumulation, |err| <= 2^-8 * sum_b |dz_b x_b|."""
    import paper_2504_08339_amd as tn
    P, B = 3, 100
    _, w2t, _, W2 = _synthetic_weights(P, 16)
    xb, Xv = _bf16_input((B, GRID * GRID) if shared else (P, B, GRID * GRID), 9)
    rng = np.random.default_rng(12)
    h = np.tanh(rng.standard_normal((P, B, GRID * GRID))).astype(np.float32)
    dy = rng.standard_normal((P, B, NOUT)).astype(np.float32)
    dw1t, dw2t = tn.substrate_backward(w2t, xb, torch.from_numpy(h).cuda(),
                                       torch.from_numpy(dy).cuda(), GRID, NOUT, THR)
    dw1t, dw2t = host(dw1t), host(dw2t)
    for g in range(P):
        Xg = Xv if shared else Xv[g]
        H = h[g].astype(np.float64)
        dY = dy[g].astype(np.float64)
        dW1, dW2 = hn.substrate_backward(Xg, W2[g].T, H, dY)      # [s][t], [t][j]
        b2 = 2.0 ** -17 * (np.abs(H).T @ np.abs(dY)) + 1e-30
        assert np.all(np.abs(dw2t[g].T - dW2) <= b2), g
        dZ = (dY @ W2[g]) * (1.0 - H * H)
        b1 = 2.0 ** -8 * (np.abs(Xg).T @ np.abs(dZ)) + 1e-30            # [s][t]
        assert np.all(np.abs(dw1t[g].T - dW1) <= b1), g


def _oracle_raw(gen, tr, src, dst):
    """The oracle's CPPN values [S][T] and the mask of ambiguous threshold
    decisions (|w| within the forward tolerance of the threshold)."""
    ref, cond = oracle.forward(gen, tr, hn.query_inputs(src, dst), with_cond=True)
    ref = ref[:, 0].reshape(len(src), len(dst))
    cond = cond[:, 0].reshape(len(src), len(dst))
    return ref, np.abs(np.abs(ref) - THR) <= 1e-5 * cond + 2.0 ** -100


def _flip_bound(A1, A2, X, W2, H, tol1, tol2):
    """How far the outputs can move when the ambiguous threshold decisions
    (masks A1 [s][t], A2 [t][j]) go the other way: a weight flips between 0 and
    at most thr + its tolerance; tanh' <= 1."""
    dz = np.abs(X) @ (A1 * (THR + tol1))                          # [B][t]
    return dz @ np.abs(W2) + np.abs(H) @ (A2 * (THR + tol2))     # [B][j]


def _oracle_pipeline(pop, g, grid, n_out, X):
    """The oracle's own substrate for genome g: float64 weights with its own
    threshold decisions, H, Y, the error scale and the flip bound."""
    gen = oracle.decode(pop, g)
    otr = oracle.transform(gen)
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    ref1, cond1 = oracle.forward(gen, otr, hn.query_inputs(src, src), with_cond=True)
    ref2, cond2 = oracle.forward(gen, otr, hn.query_inputs(src, outs), with_cond=True)
    S = grid * grid
    r1, c1 = ref1[:, 0].reshape(S, S), cond1[:, 0].reshape(S, S)
    r2, c2 = ref2[:, 0].reshape(S, n_out), cond2[:, 0].reshape(S, n_out)
    t1, t2 = 1e-5 * c1 + 2.0 ** -100, 1e-5 * c2 + 2.0 ** -100
    A1, A2 = np.abs(np.abs(r1) - THR) <= t1, np.abs(np.abs(r2) - THR) <= t2
    W1, W2 = hn.threshold(r1, THR), hn.threshold(r2, THR)
    H, Y = hn.substrate_forward(X, W1, W2)
    return W1, W2, H, Y, hn.error_scale(X, W1, W2, H), _flip_bound(A1, A2, X, W2, H, t1, t2)


def test_substrate_end_to_end_against_float64():
    """GPU query + substrate forward against the oracle's float64 pipeline
    with its own threshold decisions: |y - y_ref| <= 2^-7 * error_scale (the
    four bfloat16 roundings take 2^-8 of it, pinned in test_oracle_hyperneat;
    accumulation and the CPPN's float32 error stay in the rest) + the effect of
    the ambiguous decisions."""
    tn, pop, dp, tr, w1t, w2t, r1, r2 = _query(3, seed=25)
    xb, Xv = _bf16_input((64, GRID * GRID), 9)
    h, y = tn.substrate_forward(w1t, w2t, xb, GRID, NOUT, THR)
    y = host(y)
    for g in range(pop.P):
        W1, W2, H, Y, scale, flip = _oracle_pipeline(pop, g, GRID, NOUT, Xv)
        assert np.all(np.abs(y[g] - Y) <= 2.0 ** -7 * scale + flip), g


def test_full_size_sampled():
    """1000 CPPNs on the 32 x 32 / 32 x 32 / 8 substrate with 128 inputs per
    genome, as the benchmark runs it; three sampled genomes against the
    oracle's own pipeline (hidden values: one bfloat16 rounding of each weight,
    2^-8, and float32 accumulation, 2^-14, of sum |x w|, plus the ambiguous
    decisions; outputs: the end-to-end bound)."""
    import paper_2504_08339_amd as tn
    pop = synth.cppn_population()
    dp = to_device(pop)
    tr = tn.transform(dp)
    w1t, w2t = tn.cppn_query(dp, tr, GRID, NOUT, THR)
    xb, Xv = _bf16_input((pop.P, 128, GRID * GRID), 5)
    h, y = tn.substrate_forward(w1t, w2t, xb, GRID, NOUT, THR)
    h, y = host(h), host(y)
    assert np.isfinite(y).all()
    for g in (17, 500, 803):
        W1, W2, H, Y, scale, flip = _oracle_pipeline(pop, g, GRID, NOUT, Xv[g])
        mag = np.abs(Xv[g]) @ np.abs(W1)
        src = hn.grid_coords(GRID)
        gen = oracle.decode(pop, g)
        ref1, cond1 = oracle.forward(gen, oracle.transform(gen), hn.query_inputs(src, src),
                                     with_cond=True)
        t1 = 1e-5 * cond1[:, 0].reshape(GRID * GRID, GRID * GRID) + 2.0 ** -100
        A1 = np.abs(np.abs(ref1[:, 0].reshape(GRID * GRID, GRID * GRID)) - THR) <= t1
        dz = np.abs(Xv[g]) @ (A1 * (THR + t1))
        assert np.all(np.abs(h[g] - H) <= (2.0 ** -8 + 2.0 ** -14) * mag + dz + 2.0 ** -21), g
        assert np.all(np.abs(y[g] - Y) <= 2.0 ** -7 * scale + flip), g
        print(f"genome {g}: ambiguous threshold decisions {int(A1.sum())}, "
              f"max |y - y64| / scale {float(np.max(np.abs(y[g] - Y) / scale)):.3e}")


def _cppn_grad_case(grid, n_out, P, seed):
    """Upstream gradients drawn from a seed, set to 0 at the queries whose
    threshold decision is ambiguous by the oracle's own values, fed to both
    sides."""
    import paper_2504_08339_amd as tn
    pop = synth.cppn_population(seed=seed, P=P)
    dp = to_device(pop)
    tr = tn.transform(dp)
    S = grid * grid
    rng = np.random.default_rng(seed)
    u1 = rng.standard_normal((P, S, S)).astype(np.float32)      # [g][t][s]
    u2 = rng.standard_normal((P, n_out, S)).astype(np.float32)  # [g][j][s]
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    raws = []
    for g in range(P):
        gen = oracle.decode(pop, g)
        otr = oracle.transform(gen)
        if otr.status:
            raws.append(None)
            continue
        r1, a1 = _oracle_raw(gen, otr, src, src)      # [s][t]
        r2, a2 = _oracle_raw(gen, otr, src, outs)
        u1[g][a1.T] = 0.0
        u2[g][a2.T] = 0.0
        raws.append((r1, r2))
    dW, db = tn.cppn_backward(dp, tr, torch.from_numpy(u1).cuda(), torch.from_numpy(u2).cuda(),
                              grid, n_out, THR)
    return pop, raws, u1, u2, host(dW), host(db)


def _check_cppn_grads(pop, grid, n_out, raws, u1, u2, dW, db, genomes):
    """Against the oracle's CPPN adjoint with its own threshold decisions:
    |g - g_ref| <= 3e-5 |g_ref| + 1e-5 max|g_ref| per genome (float32 sums
    over up to 2^20 queries of terms that carry the forward's 1e-5 error; the
    worst measured |g - g_ref| / (|g_ref| + max|g_ref|) is 6.4e-6 on the full
    substrate, 1.1e-6 on the small one); returns that worst ratio."""
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    worst = 0.0
    for g in genomes:
        gen = oracle.decode(pop, g)
        tr = oracle.transform(gen)
        if tr.status:
            assert np.isnan(dW[g]).all() and np.isnan(db[g]).all()
            continue
        r1, r2 = raws[g]
        a = hn.cppn_gradient(gen, tr, src, src, r1, u1[g].T.astype(np.float64))
        b = hn.cppn_gradient(gen, tr, src, outs, r2, u2[g].T.astype(np.float64))
        ref_w = np.zeros(pop.C_max)
        ref_b = np.zeros(pop.N_max)
        for row, val in a[0].items():
            ref_w[row] += val + b[0][row]
        for row, val in a[1].items():
            ref_b[row] += val + b[1][row]
        ref = np.concatenate([ref_w, ref_b])
        got = np.concatenate([dW[g], db[g]]).astype(np.float64)
        err = np.abs(got - ref)
        tol = 3e-5 * np.abs(ref) + 1e-5 * np.abs(ref).max()
        assert np.all(err <= tol), (g, float(np.max(err - tol)))
        worst = max(worst, float(np.max(err / (np.abs(ref) + np.abs(ref).max() + 1e-300))))
    return worst


def test_cppn_backward_small_grid():
    pop, raws, u1, u2, dW, db = _cppn_grad_case(8, 2, 8, 31)
    worst = _check_cppn_grads(pop, 8, 2, raws, u1, u2, dW, db, range(pop.P))
    print(f"CPPN adjoint, 8x8 substrate: worst |err| / (|g| + max|g|) {worst:.3e}")
    dead = (pop.conn_in < 0) | (pop.conn_en == 0)
    assert np.all(dW[dead] == 0.0)
    assert np.all(db[pop.node_key < pop.n_in] == 0.0)


def test_cppn_backward_full_substrate():
    pop, raws, u1, u2, dW, db = _cppn_grad_case(GRID, NOUT, 2, 41)
    worst = _check_cppn_grads(pop, GRID, NOUT, raws, u1, u2, dW, db, range(pop.P))
    print(f"CPPN adjoint, 32x32 substrate: worst |err| / (|g| + max|g|) {worst:.3e}")


def test_cppn_backward_both_slot_forms_and_edge_limit():
    """CPPNs of 34 to 70 enabled in-edges: the compact form (at most 48
    in-edges) and the full one (49 to 64) against the oracle, NaN above the
    64 in-edges the adjoint holds."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(61)
    muts = np.array([30, 46, 50, 54, 58, 62, 75, 40])
    pop = synth.grow_population(8, 5, 1, 32, 128, muts, rng,
                                hidden_acts=("sin", "gaussian", "tanh", "abs"),
                                output_acts=("tanh",))
    edges = [int((pop.conn_rows(g)["en"] > 0).sum()) for g in range(pop.P)]
    assert min(edges) <= 48 and any(48 < e <= 64 for e in edges) and max(edges) > 64
    grid, n_out = 8, 2
    dp = to_device(pop)
    tr = tn.transform(dp)
    S = grid * grid
    u1 = rng.standard_normal((pop.P, S, S)).astype(np.float32)
    u2 = rng.standard_normal((pop.P, n_out, S)).astype(np.float32)
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    raws = []
    for g in range(pop.P):
        gen = oracle.decode(pop, g)
        otr = oracle.transform(gen)
        r1, a1 = _oracle_raw(gen, otr, src, src)
        r2, a2 = _oracle_raw(gen, otr, src, outs)
        u1[g][a1.T] = 0.0
        u2[g][a2.T] = 0.0
        raws.append((r1, r2))
    dW, db = tn.cppn_backward(dp, tr, torch.from_numpy(u1).cuda(), torch.from_numpy(u2).cuda(),
                              grid, n_out, THR)
    dW, db = host(dW), host(db)
    over = [g for g in range(pop.P) if edges[g] > 64]
    for g in over:
        assert np.isnan(dW[g]).all() and np.isnan(db[g]).all()
    _check_cppn_grads(pop, grid, n_out, raws, u1, u2, dW, db,
                      [g for g in range(pop.P) if edges[g] <= 64])


def _walk_genomes(rng, aggs):
    """CPPNs around the limits of the walk over sources and targets. Nodes are
    (sources, activation): 's' the source's coordinates, 't' the target's, 'o'
    the constant input, a number an earlier node."""
    tanh, sin = 2, 4
    specs = [
        [("st", tanh)],
        [("s", sin)],                                         # one value per source
        [("t", sin)], [("o", tanh)], [("", sin)],             # per target; constants
        [("s", 5), ("t", 6), ([0, 1], tanh)],
        [("t", sin)] + [([k], (sin, tanh, 5, 6)[k % 4]) for k in range(16)] + [(["s", 3, 16], tanh)],
        [("s", sin), ([0], 5), ("o", 1), ("t", sin), ([1, 2, 3], sin), ("st", 0), ([4, 5], 3)],
    ]
    for n_tanh, n_sin in ((13, 2), (14, 2), (20, 1), (22, 0), (9, 18)):   # 20, 21 positions; 48, 49 rows; 32
        specs.append([(("st", "s", "t", "o")[k % 4] if k < 6 else
                       [k - 1, k - 4, k - 6][:2 if n_sin > 9 else 3], sin if k < n_sin else tanh) for k in range(n_tanh + n_sin)])
    genomes = []
    for g, spec in enumerate(specs):
        keys = list(range(6, 5 + len(spec))) + [5]
        nodes = [[k, 0.0, 1.0, 0, 0] for k in range(5)]
        conns = []
        for i, (srcs, act) in enumerate(spec):
            nodes.append([keys[i], float(rng.normal() * 0.3), float(rng.choice([1.0, 0.75])), act,
                          aggs[(g + i) % len(aggs)]])
            for s in srcs:
                for q in ({"s": (0, 1), "t": (2, 3), "o": (4,)}[s] if isinstance(s, str) else (keys[s],)):
                    conns.append([q, keys[i], float(rng.normal()), 1])
        nodes.sort()
        genomes.append((nodes, conns + [[4, keys[0], 1.0, 0]] if spec[0][0] != "o" else conns))
    return genomes


@pytest.mark.parametrize("aggs", [(0,), (0, 1, 2, 3, 4, 5)])
@pytest.mark.parametrize("grid,n_out", [(8, 130), (16, 1), (24, 7)])
def test_query_walk_equals_the_packed_program(grid, n_out, aggs):
    """Populations of 32 node rows (the walk over sources and targets), padded
    and ragged, give the bits of the same genomes in 33 rows (the packed
    program), with a flagged genome among them; where a mean may round a term
    once instead of twice, values of size 1 agree to 1e-5."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(grid + n_out)
    genomes = _walk_genomes(rng, aggs)
    genomes.append((genomes[0][0] + [[6, 0.0, 1.0, 2, 0]],
                    [[5, 6, 1.0, 1], [6, 5, 1.0, 1], [0, 6, 1.0, 1]]))    # a cycle
    pop = population_from_rows(genomes, 5, 1)
    assert pop.N_max == 32
    rag = synth.to_ragged(pop)
    out = []
    for p in (synth.to_padded(rag, N_max=33, C_max=pop.C_max), pop, rag):
        dp = to_device(p)
        tr = tn.transform(dp)
        assert list(np.flatnonzero(host(tr.status)[:p.P])) == [p.P - 1]
        w1t, w2t, r1, r2 = tn.cppn_query(dp, tr, grid, n_out, THR, raw=True)
        out.append((_bits16(w1t), _bits16(w2t), host(r1), host(r2)))
    for w1, w2, r1, r2 in out[1:]:
        assert np.isnan(r1[-1]).all() and np.isnan(r2[-1]).all() and (w1[-1] == 0x7FC0).all()
        if aggs == (0,):
            assert np.array_equal(w1, out[0][0]) and np.array_equal(w2, out[0][1])
            assert np.array_equal(r1.view(np.uint32), out[0][2].view(np.uint32))
            assert np.array_equal(r2.view(np.uint32), out[0][3].view(np.uint32))
        else:
            np.testing.assert_allclose(r1, out[0][2], rtol=1e-5, atol=1e-5)
            np.testing.assert_allclose(r2, out[0][3], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("grid,n_out", [(8, 70), (16, 3)])
def test_cppn_backward_walk(grid, n_out):
    """The adjoint of the same genomes (both register files, nodes of one value
    per source or target, more target nodes than the table holds) against the
    oracle."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(grid)
    pop = population_from_rows(_walk_genomes(rng, (0,)), 5, 1)
    dp = to_device(pop)
    tr = tn.transform(dp)
    S = grid * grid
    u1 = rng.standard_normal((pop.P, S, S)).astype(np.float32)
    u2 = rng.standard_normal((pop.P, n_out, S)).astype(np.float32)
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    raws = []
    for g in range(pop.P):
        gen = oracle.decode(pop, g)
        otr = oracle.transform(gen)
        r1, a1 = _oracle_raw(gen, otr, src, src)
        r2, a2 = _oracle_raw(gen, otr, src, outs)
        u1[g][a1.T] = 0.0
        u2[g][a2.T] = 0.0
        raws.append((r1, r2))
    dW, db = tn.cppn_backward(dp, tr, torch.from_numpy(u1).cuda(), torch.from_numpy(u2).cuda(),
                              grid, n_out, THR)
    _check_cppn_grads(pop, grid, n_out, raws, u1, u2, host(dW), host(db), range(pop.P))


def test_cppn_backward_through_the_substrate():
    """The whole chain on the GPU (CPPN query -> substrate forward -> substrate
    backward -> CPPN adjoint) against the oracle's float64 chain with its own
    decisions. The genomes and inputs are chosen so that no threshold decision
    is ambiguous (checked on the oracle side); the GPU's bfloat16 weights,
    inputs and dZ put a few 2^-8 on the substrate gradients, so the CPPN
    gradient is held to 2^-5 of the genome's largest component."""
    import paper_2504_08339_amd as tn
    pop = synth.cppn_population(seed=54, P=2)
    grid, n_out = 8, 4
    src, outs = hn.grid_coords(grid), hn.row_coords(n_out)
    for g in range(pop.P):
        gen = oracle.decode(pop, g)
        otr = oracle.transform(gen)
        assert not _oracle_raw(gen, otr, src, src)[1].any()
        assert not _oracle_raw(gen, otr, src, outs)[1].any()
    dp = to_device(pop)
    tr = tn.transform(dp)
    w1t, w2t = tn.cppn_query(dp, tr, grid, n_out, THR)
    xb, Xv = _bf16_input((32, grid * grid), 6)
    h, y = tn.substrate_forward(w1t, w2t, xb, grid, n_out)
    dyn = np.random.default_rng(6).standard_normal((2, 32, n_out)).astype(np.float32)
    dw1t, dw2t = tn.substrate_backward(w2t, xb, h, torch.from_numpy(dyn).cuda(), grid, n_out)
    dW, db = tn.cppn_backward(dp, tr, dw1t, dw2t, grid, n_out)
    dW, db = host(dW), host(db)
    for g in range(pop.P):
        gen = oracle.decode(pop, g)
        otr = oracle.transform(gen)
        ref = hn.hyperneat(gen, otr, grid, n_out, Xv, dyn[g].astype(np.float64), THR)
        rw = np.zeros(pop.C_max)
        rb = np.zeros(pop.N_max)
        for r, v in ref["dw_cppn"].items():
            rw[r] = v
        for r, v in ref["db_cppn"].items():
            rb[r] = v
        want = np.concatenate([rw, rb])
        got = np.concatenate([dW[g], db[g]]).astype(np.float64)
        assert np.all(np.abs(got - want) <= 2.0 ** -5 * np.abs(want).max() + 1e-12), g


@pytest.mark.parametrize("grid", [8, 16, 24])
@pytest.mark.parametrize("B,m,shared,shift", [(1, 1, False, 0), (31, 8, True, 0), (33, 9, False, 0),
                                              (128, 32, False, 0), (129, 8, False, 0),
                                              (40, 17, False, 1)])
def test_substrate_tiles_and_remainders(grid, B, m, shared, shift):
    """Substrate forward and backward against float64 at the edges of their
    tiles: S = 64, 256, 576, batches around 32 and 128 (the fused gradient's
    largest), outputs around 8, 16 and 32, shared inputs, and weights and inputs
    that are only 2-byte aligned. Bars of the substrate tests: K float32
    additions of exact bfloat16 products, dz rounded to bfloat16."""
    import paper_2504_08339_amd as tn
    S, P = grid * grid, 3
    gen = torch.Generator().manual_seed(grid * 1000 + B + m)
    normal = lambda *shape: torch.randn(shape, generator=gen)

    def placed(t):  # on the device, `shift` elements off an aligned start
        flat = torch.zeros(t.numel() + shift, dtype=t.dtype, device="cuda")
        flat[shift:] = t.reshape(-1).cuda()
        return flat[shift:].view(t.shape)

    w1 = torch.tanh(normal(P, S, S)).bfloat16()
    w2 = torch.tanh(normal(P, m, S)).bfloat16()
    x = normal(*((B, S) if shared else (P, B, S))).bfloat16()
    dy = normal(P, B, m)
    dw1, dw2 = placed(w1), placed(w2)
    h, y = tn.substrate_forward(dw1, dw2, placed(x), grid, m)
    g1, g2 = tn.substrate_backward(dw2, placed(x), h, dy.cuda(), grid, m)
    h, y, g1, g2 = (t.cpu().double() for t in (h, y, g1, g2))
    xd, w1d, w2d, d = x.double().expand(P, B, S), w1.double(), w2.double(), dy.double()
    z = xd @ w1d.transpose(1, 2).contiguous()
    scale = xd.abs() @ w1d.abs().transpose(1, 2).contiguous()
    assert ((h - torch.tanh(z)).abs() <= 2.0 ** -14 * scale + 2.0 ** -21).all()
    hb = h.float().bfloat16().double()
    terms = hb.abs() @ w2d.abs().transpose(1, 2).contiguous()
    assert ((y - hb @ w2d.transpose(1, 2).contiguous()).abs() <= 2.0 ** -14 * terms).all()
    ht, dt = h.transpose(1, 2).contiguous(), d.transpose(1, 2).contiguous()
    assert ((g2 - dt @ h).abs() <= 2.0 ** -17 * (dt.abs() @ h.abs()) + 2.0 ** -126).all()
    dz = (d @ w2d) * (1 - h * h)
    dz_terms = (d.abs() @ w2d.abs()) * (1 - h * h)
    dzt = dz.transpose(1, 2).contiguous()
    bar = 2.0 ** -8 * (dz_terms.transpose(1, 2).contiguous() @ xd.abs()) + 2.0 ** -126
    assert ((g1 - dzt @ xd).abs() <= bar).all()


@pytest.mark.parametrize("B", [1, 31, 32, 97, 127, 130])
@pytest.mark.parametrize("m", [3, 9])
def test_substrate_backward_of_infinite_upstreams(B, m):
    """An infinite upstream value in the batch's last row gives the infinities
    (and, where it meets a 0, the NaNs) of dY^T H and dZ^T x, on every side of
    the batch sizes that the gradient kernels round up to."""
    import paper_2504_08339_amd as tn
    grid, P = 8, 3
    S = grid * grid
    gen = torch.Generator().manual_seed(100 * B + m)
    normal = lambda *shape: torch.randn(shape, generator=gen)
    x, w2 = normal(P, B, S).bfloat16(), torch.tanh(normal(P, m, S)).bfloat16()
    h, dy = torch.tanh(normal(P, B, S)), normal(P, B, m)
    h[0, B - 1, 5] = 0.0
    x[0, B - 1, 7] = 0.0
    dy[0, B - 1, 1] = float("inf")
    dy[1, B - 1, m - 1] = float("-inf")
    g1, g2 = tn.substrate_backward(w2.cuda(), x.cuda(), h.cuda(), dy.cuda(), grid, m)
    hd, dd, xd, wd = h.double(), dy.double(), x.double(), w2.double()
    want2 = torch.stack([(dd[g, :, :, None] * hd[g, :, None, :]).sum(0) for g in range(P)])
    dz = torch.stack([(dd[g, :, :, None] * wd[g][None]).sum(1) for g in range(P)]) * (1 - hd * hd)
    want1 = torch.stack([(dz[g, :, :, None] * xd[g, :, None, :]).sum(0) for g in range(P)])
    assert torch.isinf(want2).any() and torch.isnan(want2).any() and torch.isinf(want1).any()
    for got, want in ((g1.cpu().double(), want1), (g2.cpu().double(), want2)):
        fine = torch.isfinite(want)
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(got[~fine & ~torch.isnan(want)], want[~fine & ~torch.isnan(want)])
        assert torch.isfinite(got[fine]).all()


@pytest.mark.parametrize("grid", [8, 24])
@pytest.mark.parametrize("B,m", [(1, 1), (9, 2), (31, 8), (64, 9), (127, 5), (128, 32)])
def test_substrate_backward_bits_do_not_depend_on_alignment(grid, B, m):
    """Inputs that are only 2-byte aligned take the kernels of larger batches:
    the same bits, dw2t summed in ascending batch index."""
    import paper_2504_08339_amd as tn
    S, P = grid * grid, 3
    gen = torch.Generator().manual_seed(grid + 10 * B + m)
    normal = lambda *shape: torch.randn(shape, generator=gen)
    x, w2 = normal(P, B, S).bfloat16().cuda(), torch.tanh(normal(P, m, S)).bfloat16().cuda()
    h, dy = torch.tanh(normal(P, B, S)).cuda(), normal(P, B, m).cuda()
    shifted = torch.empty(P * B * S + 1, dtype=torch.bfloat16, device="cuda")[1:].view(P, B, S)
    shifted.copy_(x)
    a1, a2 = tn.substrate_backward(w2, x, h, dy, grid, m)
    b1, b2 = tn.substrate_backward(w2, shifted, h, dy, grid, m)
    assert torch.equal(a1.view(torch.int32), b1.view(torch.int32))
    assert torch.equal(a2.view(torch.int32), b2.view(torch.int32))


@pytest.mark.parametrize("grid,B,m,scale", [(8, 1, 1, 1.0), (8, 70, 130, 1.0), (16, 64, 8, 1.0),
                                            (16, 65, 17, 1e-3), (24, 129, 10, 1.0),
                                            (32, 40, 16, 1.0), (8, 33, 5, 1e-38)])
def test_substrate_outputs_add_in_ascending_order(grid, B, m, scale):
    """y is one chain of fused multiply-adds in ascending hidden index: every bit
    of it, at the edges of the tiles of 64 rows and 16 outputs and for weights
    down to the smallest magnitudes. The chain here adds the exact product in
    float64 and rounds to float32 once."""
    import paper_2504_08339_amd as tn
    S, P = grid * grid, 2
    gen = torch.Generator().manual_seed(B + m)
    normal = lambda *shape: torch.randn(shape, generator=gen)
    w1, w2, x = (normal(P, S, S) * 0.1).bfloat16(), (normal(P, m, S) * scale).bfloat16(), normal(P, B, S)
    h, y = tn.substrate_forward(w1.cuda(), w2.cuda(), x.bfloat16().cuda(), grid, m)
    hb, wd = host(h.bfloat16().double()), w2.double().numpy()
    acc = np.zeros((P, B, m), np.float32)
    for t in range(S):
        acc = (acc.astype(np.float64) + hb[:, :, t, None] * wd[:, None, :, t]).astype(np.float32)
    assert np.array_equal(host(y).view(np.uint32), acc.view(np.uint32))


@pytest.mark.parametrize("aggs", [(1,), (2,), (3,), (4,), (5,), (0, 1, 2, 3, 4, 5)])
def test_query_walk_bits_of_every_aggregation(aggs):
    """The walk over sources and targets and the packed program round every
    aggregation's terms alike (a term of a mean is rounded before it is added)."""
    import paper_2504_08339_amd as tn
    pop = population_from_rows(_walk_genomes(np.random.default_rng(7), aggs), 5, 1)
    out = []
    for p in (synth.to_padded(synth.to_ragged(pop), N_max=33, C_max=pop.C_max), pop):
        dp = to_device(p)
        out.append([host(t) for t in tn.cppn_query(dp, tn.transform(dp), 8, 70, THR, raw=True)[2:]])
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
