"""GPU parity of tn_forward / tn_forward_loss against the float64 oracle.

Tolerance: |y_gpu - y_ref| <= 1e-5 * cond(y) + 2^-100, where cond is the
first-order error scale the oracle computes alongside the outputs (|y| plus the
local activation slope times the propagated magnitudes |b| + |rho| * sum |w|
cond); it is never below 1e-5 * |y_ref|. The absolute floor 2^-100 covers values
below float32's range: float32 underflows at 2^-126 (normal) / 2^-149
(subnormal), and the floor allows that error to be amplified by up to 2^26
downstream. Flagged genomes must give NaN.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import host, tensor, to_device
from helpers import load_golden, population_from_rows

pytestmark = pytest.mark.gpu
RTOL = 1e-5
ABS_FLOOR = 2.0 ** -100


def gpu_forward(pop, obs):
    import paper_2504_08339_amd as tn
    dp = to_device(pop)
    tr = tn.transform(dp)
    return host(tn.forward(dp, tr, tensor(obs)))


def compare_all(Y, ref, cond, status):
    """Whole-population comparison against oracle_pool references; returns the
    worst |err| / cond over every output of every valid genome."""
    bad_flag = status != 0
    assert np.isnan(Y[bad_flag]).all()
    Yv = Y[~bad_flag].astype(np.float64)
    rv, cv = ref[~bad_flag], cond[~bad_flag]
    err = np.abs(Yv - rv)
    bad = err > RTOL * cv + ABS_FLOOR
    assert not bad.any(), (int(bad.sum()), float(err[bad].max()))
    pos = cv > 0
    return float((err[pos] / cv[pos]).max()) if pos.any() else 0.0


def check(pop, obs, Y, genomes=None):
    """Asserts the bar on every listed genome and returns the worst |err| / cond."""
    idx = range(pop.P) if genomes is None else genomes
    worst = 0.0
    for g in idx:
        gen = oracle.decode(pop, g)
        tr = oracle.transform(gen)
        X = obs if obs.ndim == 2 else obs[g]
        ref, cond = oracle.forward(gen, tr, X, with_cond=True)
        y = Y[g]
        if tr.status:
            assert np.isnan(y).all(), g
            continue
        err = np.abs(y.astype(np.float64) - ref)
        bad = err > RTOL * cond + ABS_FLOOR
        assert not bad.any(), (g, float(err[bad].max()), float(cond[bad].min()))
        pos = cond > 0
        if pos.any():
            worst = max(worst, float((err[pos] / cond[pos]).max()))
    return worst


def test_xor_population_and_fitness():
    import paper_2504_08339_amd as tn
    pop = synth.xor_population()
    X = synth.xor_inputs()
    T = synth.xor_targets()
    dp = to_device(pop)
    tr = tn.transform(dp)
    Y = host(tn.forward(dp, tr, tensor(X)))
    check(pop, X, Y)
    fit, Yl = tn.forward_loss(dp, tr, tensor(X), tensor(T), scale=-1.0, offset=4.0)
    fit = host(fit)
    assert np.array_equal(host(Yl), Y)
    for g in range(pop.P):
        ref = oracle.xor_fitness(oracle.forward_population(pop, X, [g])[0], T)
        assert abs(fit[g] - ref) <= 1e-5 * 4.0


@pytest.mark.parametrize("case", load_golden("hand_networks.json")["cases"],
                         ids=lambda c: c["name"])
def test_hand_networks(case):
    pop = population_from_rows([(case["nodes"], case["conns"])], case["n_in"], case["n_out"])
    X = np.array(case["obs"], np.float32)
    Y = gpu_forward(pop, X)
    np.testing.assert_allclose(Y[0], np.array(case["expected"]), rtol=0,
                               atol=max(case["tol"], 1e-6))


def test_control_tiles_and_ragged_tail():
    pop = synth.control_population(P=64)
    obs = synth.normal_obs(64, 200, 17, 102)   # 3 full tiles + a tail of 8
    Y = gpu_forward(pop, obs)
    worst = check(pop, obs, Y)
    print(f"control tiles: worst |err|/cond {worst:.3e}")


def test_control_full_size_all_genomes():
    """The full control-policy workload (1000 genomes x 1000 observations) in the
    launch configuration the benchmark times; every output of every genome
    against the oracle (computed in parallel worker processes)."""
    import oracle_pool
    pop = synth.control_population()
    obs = synth.normal_obs(pop.P, 1000, 17, 102)
    Y = gpu_forward(pop, obs)
    assert Y.shape == (1000, 1000, 6)
    assert np.isfinite(Y).all()
    ref, cond, st = oracle_pool.forward_reference("control", pop.P)
    worst = compare_all(Y, ref, cond, st)
    print(f"control 1000 x 1000: worst |err|/cond {worst:.3e}")


@pytest.mark.parametrize("B", [130, 300])
def test_all_activations_aggregations_and_response(B):
    """Every activation and aggregation with random responses; 130
    observations run two tiles per wavefront, 300 four."""
    rng = np.random.default_rng(5)
    pop = synth.cppn_population(P=80, seed=77)
    valid = pop.node_key >= 0
    pop.node_act[valid] = rng.integers(0, 7, size=int(valid.sum()))
    pop.node_agg[valid] = rng.integers(0, 6, size=int(valid.sum()))
    pop.node_resp[valid] = rng.uniform(-2, 2, size=int(valid.sum())).astype(np.float32)
    obs = rng.uniform(-1.5, 1.5, size=(80, B, pop.n_in)).astype(np.float32)
    Y = gpu_forward(pop, obs)
    check(pop, obs, Y)


@pytest.mark.parametrize("K,W", [(1, 1), (1, 3), (2, 3), (4, 2), (1, 16)])
def test_lds_engine_wide_nodes_every_aggregation(K, W):
    """The LDS engine on dense random DAGs (many nodes with more than six
    in-edges, through the four-at-a-time in-edge loop and its remainder, some
    with none) with every activation, aggregation and random responses, on 150
    observations (a ragged last tile), against the oracle. Three wavefronts
    split the levels unevenly; sixteen is the largest workgroup (one
    observation per lane)."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(21)
    pop = synth.random_dag_population(40, 5, 3, rng, h_lo=4, h_hi=60, c_lo=5.0, c_hi=9.0,
                                      c_cap=400, disable_p=0.1)
    valid = pop.node_key >= 0
    pop.node_act[valid] = rng.integers(0, 7, size=int(valid.sum()))
    pop.node_agg[valid] = rng.integers(0, 6, size=int(valid.sum()))
    pop.node_resp[valid] = rng.uniform(-1.5, 1.5, size=int(valid.sum())).astype(np.float32)
    obs = rng.uniform(-1.0, 1.0, size=(40, 150, 5)).astype(np.float32)
    dp = to_device(pop)
    tr = tn.transform(dp)
    wide = 0
    for g in range(pop.P):
        c = pop.conn_rows(g)
        wide = max(wide, int(np.bincount(c["out"][c["en"] > 0]).max()))
    assert wide > 6
    Y = host(tn.forward(dp, tr, tensor(obs), engine=tn.TN_ENGINE_LDS, obs_per_lane=K,
                        waves_per_genome=W))
    check(pop, obs, Y)


def test_shared_observations_and_single_row():
    pop = synth.control_population(P=30)
    X = synth.normal_obs(1, 65, 17, 5)[0]
    Y = gpu_forward(pop, X)
    check(pop, X, Y)
    Y1 = gpu_forward(pop, X[:1])
    check(pop, X[:1], Y1)


def test_flagged_genomes_nan_and_loss_nan():
    import paper_2504_08339_amd as tn
    from test_gpu_transform import _malformed
    pop = _malformed()
    X = np.random.default_rng(1).standard_normal((5, 2)).astype(np.float32)
    dp = to_device(pop)
    tr = tn.transform(dp)
    Y = host(tn.forward(dp, tr, tensor(X)))
    check(pop, X, Y)
    loss, _ = tn.forward_loss(dp, tr, tensor(X), tensor(np.zeros((5, 1), np.float32)))
    loss = host(loss)
    st = host(tr.status)
    assert np.array_equal(np.isnan(loss), st != 0)


def test_empty_batch_and_population():
    import paper_2504_08339_amd as tn
    pop = synth.xor_population(P=4)
    dp = to_device(pop)
    tr = tn.transform(dp)
    out = tn.forward(dp, tr, torch.empty((0, 3), dtype=torch.float32, device="cuda"))
    assert out.shape == (4, 0, 1)
    loss, _ = tn.forward_loss(dp, tr, torch.empty((0, 3), dtype=torch.float32, device="cuda"),
                              torch.empty((0, 1), dtype=torch.float32, device="cuda"),
                              scale=-1.0, offset=4.0)
    assert np.all(host(loss) == 4.0)
    empty = synth.subset(pop, [])
    de = to_device(empty)
    te = tn.transform(de)
    assert tn.forward(de, te, tensor(synth.xor_inputs())).shape == (0, 4, 1)


def test_ragged_equals_padded_bitwise():
    pop = synth.batching_population(P=120)
    obs = synth.normal_obs(120, 70, 27, 103)
    Yr = gpu_forward(pop, obs)
    Yp = gpu_forward(synth.to_padded(pop), obs)
    assert np.array_equal(Yr.view(np.uint32), Yp.view(np.uint32))
    check(pop, obs, Yr, list(range(0, 120, 7)))


def test_deterministic():
    pop = synth.control_population(P=100)
    obs = synth.normal_obs(100, 100, 17, 9)
    a = gpu_forward(pop, obs)
    b = gpu_forward(pop, obs)
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_mse_loss_matches_oracle():
    import paper_2504_08339_amd as tn
    pop = synth.differentiation_population(P=64)
    X = synth.uniform_inputs(1024, 4, 104)
    T = synth.target_mlp(X, 32, 2, 204)
    dp = to_device(pop)
    tr = tn.transform(dp)
    loss, Y = tn.forward_loss(dp, tr, tensor(X), tensor(T), scale=1.0 / (1024 * 2))
    loss, Y = host(loss), host(Y)
    check(pop, X, Y)
    for g in range(pop.P):
        ref = oracle.sse_loss(oracle.forward_population(pop, X, [g])[0], T, 1.0 / 2048)
        assert abs(loss[g] - ref) <= 1e-5 * abs(ref) + 1e-7


@pytest.mark.parametrize("K,W", [(1, 1), (1, 4), (2, 4), (4, 2), (2, 8), (1, 16)])
def test_lds_tile_shapes_and_tight_rows_bitwise(K, W):
    """Every LDS tile shape, with rows sized to the population's largest n_rows,
    gives the same bits as the default launch; too few rows gives NaN."""
    import paper_2504_08339_amd as tn
    pop = synth.control_population(P=80)
    obs = synth.normal_obs(80, 300, 17, 7)
    dp = to_device(pop)
    tr = tn.transform(dp)
    xt = tensor(obs)
    ref = host(tn.forward(dp, tr, xt))
    rows = int(host(tr.n_rows).max())
    assert rows < pop.N_max
    lds = dict(engine=tn.TN_ENGINE_LDS, obs_per_lane=K, waves_per_genome=W)
    y = host(tn.forward(dp, tr, xt, rows=rows, **lds))
    assert np.array_equal(y.view(np.uint32), ref.view(np.uint32))
    short = host(tn.forward(dp, tr, xt, rows=rows - 1, **lds))
    need = host(tr.n_rows)[:pop.P]
    assert np.isnan(short[need > rows - 1]).all()
    assert np.array_equal(short[need <= rows - 1].view(np.uint32), ref[need <= rows - 1].view(np.uint32))


@pytest.mark.parametrize("W,rows", [(1, 64), (4, 64), (8, 64), (4, 32), (2, 32), (4, 96), (2, 200),
                                    (1, 50), (4, 50), (8, 50), (2, 100), (4, 100)])
def test_register_engine_bitwise_and_row_limit(W, rows):
    """The register engine gives the LDS engine's bits for every genome whose
    packed program fits its rows and NaN for the others; observations in one
    shared batch and per genome, with a ragged last tile; the files of 50 and
    100 rows (four and two tiles per wavefront) also with a last wavefront
    whose later tiles are empty (333 observations) or that has a single
    partial tile (40)."""
    import paper_2504_08339_amd as tn
    pop = synth.control_population(P=90) if rows in (32, 64) else synth.batching_population(P=90)
    I = pop.n_in
    cases = [synth.normal_obs(90, 333, I, 8), synth.normal_obs(1, 333, I, 9)[0]]
    if rows in (50, 100):
        cases.append(synth.normal_obs(90, 40, I, 10))
    for obs in cases:
        dp = to_device(pop)
        tr = tn.transform(dp)
        xt = tensor(obs)
        ref = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_LDS, obs_per_lane=1,
                              waves_per_genome=4))
        y = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_REG, waves_per_genome=W, rows=rows))
        need = host(tr.prog_rows)[:pop.P]
        assert (need <= rows).any()
        fit = need <= rows
        assert np.array_equal(y[fit].view(np.uint32), ref[fit].view(np.uint32))
        assert np.isnan(y[~fit]).all()


@pytest.mark.parametrize("rows", [50, 100, 200])
def test_register_engine_misaligned_buffers_bitwise(rows):
    """Observations and outputs one float off a 16-byte boundary (views into
    larger buffers): the register engine then stages one float per lane and
    stores outputs one at a time, with the same bits as from aligned buffers
    (16 bytes per lane, four outputs per store)."""
    import paper_2504_08339_amd as tn
    pop = synth.batching_population(P=120)
    obs = synth.normal_obs(pop.P, 300, pop.n_in, 13)
    dp = to_device(pop)
    tr = tn.transform(dp)
    xt = tensor(obs)
    ref = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_REG, rows=rows, waves_per_genome=4))
    big = torch.zeros(obs.size + 1, dtype=torch.float32, device="cuda")
    xo = big[1:].view(obs.shape)
    xo.copy_(xt)
    assert xo.data_ptr() % 16 == 4
    ybig = torch.full((pop.P * 300 * pop.n_out + 1,), 7.0, dtype=torch.float32, device="cuda")
    yo = ybig[1:].view(pop.P, 300, pop.n_out)
    tn.forward(dp, tr, xo, out=yo, engine=tn.TN_ENGINE_REG, rows=rows, waves_per_genome=4)
    y = host(yo)
    fit = host(tr.prog_rows)[:pop.P] <= rows
    assert fit.sum() > 10
    assert np.array_equal(y[fit].view(np.uint32), ref[fit].view(np.uint32))
    assert float(host(ybig[:1])[0]) == 7.0


@pytest.mark.parametrize("rows", [50, 100])
def test_register_file_tiles_agree_bitwise(rows):
    """The tiles a wavefront holds in one register file (four at 50 rows, two
    at 100) each see the same 64 observations here, so their outputs must
    agree bit for bit, and with the LDS engine: a window reading a stale index
    shows up as a tile that disagrees."""
    import paper_2504_08339_amd as tn
    pop = synth.batching_population(P=600)
    base = synth.normal_obs(pop.P, 64, pop.n_in, 12)
    obs = np.concatenate([base] * 8, axis=1)                  # 512 observations
    dp = to_device(pop)
    tr = tn.transform(dp)
    xt = tensor(obs)
    ref = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_LDS, obs_per_lane=1,
                          waves_per_genome=4))
    for W in (1, 4):
        y = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_REG, rows=rows, waves_per_genome=W))
        fit = host(tr.prog_rows)[:pop.P] <= rows
        assert fit.sum() > 100
        tiles = y[fit].reshape(int(fit.sum()), 8, 64, pop.n_out).view(np.uint32)
        assert np.array_equal(tiles, np.broadcast_to(tiles[:, :1], tiles.shape))
        assert np.array_equal(y[fit].view(np.uint32), ref[fit].view(np.uint32))


@pytest.mark.parametrize("name", ["batching", "cppn", "differentiation"])
def test_auto_split_equals_single_engine(name):
    """The library's choice (registers for small programs, LDS for the rest)
    gives the same bits as the LDS engine alone; checked against the oracle on
    sampled genomes, and the fused loss on the same split."""
    import paper_2504_08339_amd as tn
    pop = {"batching": lambda: synth.batching_population(P=160),
           "cppn": lambda: synth.cppn_population(P=160),
           "differentiation": lambda: synth.differentiation_population(P=160)}[name]()
    obs = synth.normal_obs(pop.P, 150, pop.n_in, 31)
    dp = to_device(pop)
    tr = tn.transform(dp)
    xt = tensor(obs)
    auto = host(tn.forward(dp, tr, xt))
    lds = host(tn.forward(dp, tr, xt, engine=tn.TN_ENGINE_LDS, obs_per_lane=1,
                          waves_per_genome=2))
    assert np.array_equal(auto.view(np.uint32), lds.view(np.uint32))
    need = host(tr.prog_rows)[:pop.P]
    if name == "batching":
        assert (need <= 64).any() and (need > 64).any()
    check(pop, obs, auto, list(range(0, pop.P, 9)))
    T = np.random.default_rng(3).standard_normal((150, pop.n_out)).astype(np.float32)
    loss, Y = tn.forward_loss(dp, tr, xt, tensor(T), scale=0.5, offset=1.0)
    loss, Y = host(loss), host(Y)
    assert np.array_equal(Y.view(np.uint32), auto.view(np.uint32))
    ref = 1.0 + 0.5 * ((auto.astype(np.float64) - T) ** 2).sum(axis=(1, 2))
    np.testing.assert_allclose(loss, ref, rtol=2e-5)


@pytest.mark.parametrize("B", [1, 2, 3, 8, 9, 16, 17, 32, 33])
def test_small_batches_equal_the_lds_engine(B):
    """The automatic choice at small batches (lanes over nodes and observations
    up to 16, up to 32 for few genomes) gives the LDS engine's bits on uneven
    ragged genomes and on wide nodes of every aggregation and activation with a
    flagged genome among them; the fused loss agrees with the outputs."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(B)
    keys = list(range(9))
    genomes = []
    for g in range(14):
        nodes = [[k, float(rng.normal()), float(rng.choice([1.0, 0.5, -0.75])),
                  int(rng.integers(0, 7)), g % 6 if k >= 5 else 0] for k in keys]
        nodes += [[20 + h, float(rng.normal()), 1.0, int(rng.integers(0, 7)), (g + h) % 6]
                  for h in range(70)]
        conns = [[i, 20 + h, float(rng.normal() * 0.5), 1] for h in range(70) for i in range(5)
                 if (h + i) % 3]
        conns += [[20 + h, 5 + h % 4, float(rng.normal() * 0.5), int(h % 7 > 0)] for h in range(70)]
        genomes.append((nodes, conns if g else conns + [[5, 20, 1.0, 1], [20, 5, 1.0, 1]]))
    for pop in (population_from_rows(genomes, 5, 4),
                synth.random_dag_population(30, 27, 8, np.random.default_rng(3))):
        dp = to_device(pop)
        tr = tn.transform(dp)
        obs = tensor(rng.normal(size=(pop.P, B, pop.n_in)).astype(np.float32))
        ref = host(tn.forward(dp, tr, obs, engine=tn.TN_ENGINE_LDS))
        Y = host(tn.forward(dp, tr, obs))
        flagged = host(tr.status)[:pop.P] != 0
        assert np.isnan(Y[flagged]).all() and flagged.sum() == (1 if pop.n_in == 5 else 0)
        assert np.array_equal(Y[~flagged].view(np.uint32), ref[~flagged].view(np.uint32))
        target = rng.normal(size=(B, pop.n_out)).astype(np.float32)
        loss, out = tn.forward_loss(dp, tr, obs, tensor(target), scale=-1.0, offset=4.0)
        assert np.array_equal(host(out).view(np.uint32)[~flagged], ref[~flagged].view(np.uint32))
        sse = ((ref[~flagged].astype(np.float64) - target) ** 2).sum((1, 2))
        assert np.allclose(host(loss)[~flagged], 4.0 - sse, rtol=1e-5, atol=1e-5 * sse.max())
        only, none = tn.forward_loss(dp, tr, obs, tensor(target), scale=-1.0, offset=4.0,
                                     store_outputs=False)
        assert none is None and np.array_equal(host(only).view(np.uint32), host(loss).view(np.uint32))
        assert np.isnan(host(loss)[flagged]).all()


@pytest.mark.parametrize("B", [193, 256, 257, 384, 385, 460])
def test_two_tile_genomes_in_the_four_tile_launch(B):
    """The automatic choice from 193 observations on runs genomes of 51 to 100
    program rows two tiles at a time in the launch of those of up to 50: the
    LDS engine's bits, over units that end in each of their four tiles."""
    import paper_2504_08339_amd as tn
    pop = synth.grow_population(24, 17, 6, 128, 512, np.linspace(60, 230, 24).astype(int),
                                np.random.default_rng(B), hidden_acts=("tanh", "sin"),
                                output_acts=("tanh",))
    dp = to_device(pop)
    tr = tn.transform(dp)
    rows = host(tr.prog_rows)[:pop.P]
    assert (rows <= 50).any() and ((rows > 50) & (rows <= 100)).any()
    obs = tensor(np.random.default_rng(1).normal(size=(pop.P, B, 17)).astype(np.float32))
    ref = host(tn.forward(dp, tr, obs, engine=tn.TN_ENGINE_LDS))
    assert np.array_equal(host(tn.forward(dp, tr, obs)).view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("B", [1, 16, 17, 32, 33])
@pytest.mark.parametrize("N,C", [(1024, 4096), (900, 4096), (1024, 2000), (500, 2000)])
def test_small_batches_of_large_capacities(N, C, B):
    """Every capacity within the library's limits is accepted at every small
    batch, by the outputs and by the fused loss: the bits of the register
    engine (most genomes) and of the LDS engine (the larger ones)."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(N + C + B)
    pop = synth.grow_population(9, 17, 6, N, C, np.array([0, 5, 30, 60, 90, 120, 200, 900, 1300]), rng,
                                hidden_acts=("tanh", "sin"), output_acts=("tanh",))
    dp = to_device(pop)
    tr = tn.transform(dp)
    obs = tensor(rng.normal(size=(pop.P, B, pop.n_in)).astype(np.float32))
    need = host(tr.prog_rows)[:pop.P]
    assert (need <= 200).sum() >= 6 and (need > 200).any()
    ref = host(tn.forward(dp, tr, obs, engine=tn.TN_ENGINE_REG, rows=200))
    lds = host(tn.forward(dp, tr, obs, engine=tn.TN_ENGINE_LDS, rows=min(N, 400)))
    ref[need > 200] = lds[need > 200]
    assert not np.isnan(ref).any()
    Y = host(tn.forward(dp, tr, obs))
    assert np.array_equal(Y.view(np.uint32), ref.view(np.uint32))
    target = rng.normal(size=(B, pop.n_out)).astype(np.float32)
    loss, out = tn.forward_loss(dp, tr, obs, tensor(target))
    assert np.array_equal(host(out).view(np.uint32), ref.view(np.uint32))
    sse = ((ref.astype(np.float64) - target) ** 2).sum((1, 2))
    np.testing.assert_allclose(host(loss), sse, rtol=1e-5)


@pytest.mark.parametrize("B", [1, 3, 8, 16])
@pytest.mark.parametrize("ragged", [False, True])
def test_small_batches_by_size_class(B, ragged):
    """Populations too large for one launch at their row capacities (the genomes
    by size class, or all by the other engines at 16 observations): the
    engines' bits for genomes on either side of the classes' lines, a flagged
    genome among them, with the fused loss."""
    import paper_2504_08339_amd as tn
    rng = np.random.default_rng(40 + B)
    few = synth.grow_population(12, 17, 6, 1024, 4096,
                                np.array([0, 40, 120, 300, 330, 360, 700, 1000, 1300, 20, 60, 250]), rng,
                                hidden_acts=("tanh", "sin"), output_acts=("tanh",))
    few.node_key[9, 3] = few.node_key[9, 4]  # a repeated key
    pop = synth.subset(few, [i % 12 for i in range(1603)])
    if ragged:
        pop = synth.to_ragged(pop)
    dp = to_device(pop)
    tr = tn.transform(dp)
    status, need = host(tr.status)[:12], host(tr.prog_rows)[:12]
    assert (status != 0).tolist() == [i == 9 for i in range(12)]
    obs = rng.normal(size=(pop.P, B, pop.n_in)).astype(np.float32)
    large = (need > 200)[np.arange(pop.P) % 12]
    ok = np.arange(pop.P) % 12 != 9
    assert large.any() and not large[9]
    x = tensor(obs)
    ref = host(tn.forward(dp, tr, x, engine=tn.TN_ENGINE_REG, rows=200))
    lds = host(tn.forward(dp, tr, x, engine=tn.TN_ENGINE_LDS, rows=400))
    ref[large] = lds[large]
    assert not np.isnan(ref[ok]).any()
    Y = host(tn.forward(dp, tr, x))
    assert np.array_equal(Y[ok].view(np.uint32), ref[ok].view(np.uint32)) and np.isnan(Y[~ok]).all()
    target = rng.normal(size=(B, pop.n_out)).astype(np.float32)
    loss, out = tn.forward_loss(dp, tr, x, tensor(target))
    assert np.array_equal(host(out)[ok].view(np.uint32), ref[ok].view(np.uint32))
    sse = ((ref[ok].astype(np.float64) - target) ** 2).sum((1, 2))
    np.testing.assert_allclose(host(loss)[ok], sse, rtol=1e-5)
    assert np.isnan(host(loss)[~ok]).all()
