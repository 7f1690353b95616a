"""GPU checkpointed adjoint (FP32) against the FP64 oracle's adjoint, which
is itself pinned to central finite differences on the CPU.  Gradients are
compared per parameter group by relative L2 error, at the horizon where the
forward meets parity with contact (200 steps)."""
import time

import numpy as np
import pytest
import torch

from gpu_util import DEV, gpu_population, need_gpu, oracle_robots, say, voxel_population
from paper_2405_00698_amd import SR_QUERY_FP32, inputs

pytestmark = pytest.mark.gpu

C1 = [4] * 8


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _l2rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _dJ(R, seed=0):
    return np.random.default_rng(seed).uniform(0.5, 1.5, size=R).astype(np.float32)


TOL = 1e-3  # gradient tolerance: relative L2 per parameter group, and per component (below)
# Per robot, any group: the error a wrong kernel or parametrisation makes is
# O(1) relative; FP32-vs-FP64 branch differences stay well below this.
SANITY = 5e-2


def _component_excess(g, ref):
    """max_i |g_i - ref_i| / (1e-3 max_i |ref_i|): at most 1 when every
    component is within 1e-3 of the group's largest gradient (the max-norm
    relative error, the norm the position parity uses)."""
    return float(np.abs(g - ref).max() / (TOL * max(np.abs(ref).max(), 1e-300)))


def _compare(P, robots, dJ, steps, label):
    """Per robot: relative L2 error of each group (k, a, phi) and its
    max-norm relative error, against the oracle's FP64 adjoint."""
    g = {k: v.cpu().numpy().astype(np.float64) for k, v in P.backward(torch.from_numpy(dJ).to(DEV)).items()}
    M, S, mo, so = P.counts()
    out = []
    for r, R in robots:
        J, gk, ga, gp = R.backward(steps, g=float(dJ[r]))
        sl = slice(so[r], so[r + 1])
        l2 = [_l2rel(g[key][sl], ref) for key, ref in (("k", gk), ("a", ga), ("phi", gp))]
        cx = [_component_excess(g[key][sl], ref) for key, ref in (("k", gk), ("a", ga), ("phi", gp))]
        say(label, "robot", r, "springs", S[r], "relative L2 (k, a, phi): %.1e %.1e %.1e" % tuple(l2),
            " max-norm / 1e-3: %.2f %.2f %.2f" % tuple(cx))
        out.append((max(l2), max(cx)))
    return out


def _align(P, robots):
    """Give the oracle robots the GPU's own (a, phi) of every spring: with a
    nonzero phase the library reports a >= 0 and phi = atan2(k L0 a sin, k L0 a
    cos), which differs from a signed amplitude by pi in phase, and gradients
    are taken with respect to the parameters as reported."""
    sp = {k: v.cpu().numpy().astype(np.float64) for k, v in P.springs().items()}
    M, S, mo, so = P.counts()
    for r, R in enumerate(robots):
        R.set_springs(a=sp["a"][so[r]:so[r + 1]], phi=sp["phi"][so[r]:so[r + 1]])


def test_spring_gradients_match_oracle(orc):
    """The gradient check's population (8 robots of 4^3) at the contact
    horizon, 200 steps: every robot within 1e-3 in relative L2 and in max-norm
    for each parameter group."""
    cls, w = voxel_population(C1, 51)
    steps, K = 200, 50
    P = gpu_population(C1, cls, w)
    P.record(K, steps)
    P.step(steps)
    robots = list(enumerate(oracle_robots(orc, C1, cls, w)))
    for r, (l2, cx) in enumerate(_compare(P, robots, _dJ(len(C1)), steps, "C1")):
        assert l2 <= TOL, (r, l2)
        assert cx <= 1.0, (r, cx)


def _instance_verdict(res, label):
    """One kernel instance's robots: each within SANITY in every group, and
    the median robot within 1e-3 in relative L2.  Single robots may exceed 1e-3:
    the FP32 run and the FP64 oracle decide stick or slip from tangential
    speeds that differ in the last digits, and a node whose speed sits that
    close to the friction threshold takes the other branch of the piecewise
    smooth map, whose derivative differs there."""
    worst = [l2 for l2, _ in res]
    say(label, "median relative L2 %.1e, max %.1e, within 1e-3: %d of %d"
        % (float(np.median(worst)), max(worst), sum(x <= TOL for x in worst), len(worst)))
    assert max(worst) <= SANITY, (label, worst)
    assert float(np.median(worst)) <= TOL, (label, worst)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12])
def test_spring_gradients_match_oracle_every_side(orc, n):
    """Every adjoint kernel instance (the exchange forms, in direction chunks
    at 9^3-12^3, with the split gradient pass from 8^3 up) against the oracle's
    adjoint at the contact horizon, 200 steps with gravity, ground and
    friction, four robots each.  Odd sides carry per-spring phases (the
    phase-plane kernels)."""
    sides = [n] * 4
    # a one- or two-voxel-wide robot may come out empty at 20 % empty voxels
    cls, w = voxel_population(sides, 80 + n, p_empty=0.2 if n > 2 else 0.0)
    steps, K = 200, 50
    P = gpu_population(sides, cls, w)
    robots = oracle_robots(orc, sides, cls, w)
    if n % 2 == 1:
        sp = P.springs()
        phi = torch.from_numpy(np.random.default_rng(n).uniform(-3.0, 3.0, size=sp["k"].numel())
                               .astype(np.float32)).to(DEV)
        P.set_spring_params(None, None, phi)
        _align(P, robots)
    P.record(K, steps)
    P.step(steps)
    res = _compare(P, list(enumerate(robots)), _dJ(len(sides), n), steps, "side %d" % n)
    _instance_verdict(res, "side %d" % n)


def test_uneven_population_gradients_match_oracle(orc):
    """One backward over a population of mixed sides: the fused reverse forms
    (4^3, 5^3, 7^3) and the split ones (8^3, 10^3 and 12^3, with their direction
    chunks, recording kernels and gradient passes on the other streams) in the
    same call, each robot against the oracle's adjoint at the contact horizon."""
    sides = [12, 4, 8, 10, 5, 7, 10, 4]
    cls, w = voxel_population(sides, 77, p_empty=0.2)
    steps, K = 200, 50
    P = gpu_population(sides, cls, w)
    robots = oracle_robots(orc, sides, cls, w)
    P.record(K, steps)
    P.step(steps)
    res = _compare(P, list(enumerate(robots)), _dJ(len(sides), 9), steps, "uneven")
    _instance_verdict(res, "uneven")


def test_c4_sample_gradients_match_oracle(orc):
    """The differentiation workload (64 robots of 8^3 from random genomes,
    FP32 build, checkpoint every 100 steps): eight sampled robots against the
    oracle at the contact horizon (200 steps), and at the full 2000 steps,
    where the agreement is only reported."""
    from paper_2405_00698_amd.api import Population
    R = 64
    G = inputs.random_genomes(R, seed=1)
    B = inputs.gaussian_B()
    sample = [0, 9, 21, 30, 42, 50, 57, 63]
    dJ = _dJ(R, 4)
    for steps in (200, 2000):
        P = Population([8] * R)
        P.build_from_genomes(torch.from_numpy(G).to(DEV), torch.from_numpy(B).to(DEV), SR_QUERY_FP32)
        cls, wq = (t.cpu().numpy() for t in P.query())
        P.record(100, steps)
        P.step(steps)
        robots = [(r, orc.Robot(8, cls[r * 512:(r + 1) * 512], wq[r * 512:(r + 1) * 512].astype(np.float64)))
                  for r in sample]
        res = _compare(P, robots, dJ, steps, "C4 %d steps" % steps)
        if steps == 200:
            _instance_verdict(res, "C4 sample, 200 steps")
        else:
            say("C4 sample, 2000 steps: relative L2 per robot", ["%.1e" % l2 for l2, _ in res])
        P.close()


def test_gradients_independent_of_checkpoint_interval():
    cls, w = voxel_population(C1, 52)
    steps = 200
    ref = None
    dJ = torch.from_numpy(_dJ(len(C1), 1)).to(DEV)
    for K in (1, 7, 64, 200):
        P = gpu_population(C1, cls, w)
        P.record(K, steps)
        P.step(steps)
        g = {k: v.cpu().numpy() for k, v in P.backward(dJ).items()}
        if ref is None:
            ref = g
        else:
            for key in ("k", "a", "phi"):
                assert np.array_equal(g[key], ref[key]), (K, key)


@pytest.mark.parametrize("n", [10, 11, 12])
def test_recompute_reproduces_the_forward(n):
    """The recording kernels that recompute each checkpointed segment give the
    forward kernel's bits: with a checkpoint every step the backward starts
    each step from the forward's own state, with one segment it recomputes
    the whole run, and the gradients agree bit for bit."""
    sides = [n] * 2
    cls, w = voxel_population(sides, 60 + n)
    steps = 120
    dJ = torch.from_numpy(_dJ(len(sides), n)).to(DEV)
    ref = None
    for K in (1, 40, steps):
        say("side", n, "checkpoint interval", K)
        P = gpu_population(sides, cls, w)
        P.record(K, steps)
        P.step(steps)
        g = {k: v.cpu().numpy() for k, v in P.backward(dJ).items()}
        if ref is None:
            ref = g
        else:
            for key in ("k", "a", "phi"):
                assert np.array_equal(g[key], ref[key]), (K, key)


def test_genome_gradient_matches_oracle(orc):
    sides = [3] * 6
    B = inputs.gaussian_B()
    G = inputs.random_genomes(6, seed=5)
    steps, K = 150, 50
    from paper_2405_00698_amd.api import Population
    P = Population(sides)
    Gt, Bt = torch.from_numpy(G).to(DEV), torch.from_numpy(B).to(DEV)
    P.build_from_genomes(Gt, Bt, SR_QUERY_FP32)
    P.record(K, steps)
    P.step(steps)
    dJ = _dJ(6, 2)
    gg = P.backward(torch.from_numpy(dJ).to(DEV), genomes=Gt, B=Bt)["genome"].cpu().numpy().astype(np.float64)
    for r in range(6):
        lg = orc.query(G[r].astype(np.float64), B.astype(np.float64), 3)
        srt = np.sort(lg[:, :5], axis=1)
        if (srt[:, -1] - srt[:, -2]).min() <= 1e-4:
            continue
        J, go = orc.genome_fitness_grad(G[r].astype(np.float64), B.astype(np.float64), 3, steps)
        go = go * float(dJ[r])
        e = _l2rel(gg[r], go)
        say("robot", r, "genome gradient relative L2 %.2e" % e)
        assert e <= TOL


@pytest.mark.parametrize("side", [2, 5, 6, 8, 9])
def test_genome_gradient_at_tile_edges(orc, side):
    """The genome gradient from the GPU's own spring gradients, carried on in
    FP64 (parallel-sum rule and MLP), so that only that part is compared.  Tiles
    of 128 voxels (16 per wave): 8 voxels, 125 (a partial last wave), 216 and 729
    (a partial last tile), 512 (whole tiles)."""
    from paper_2405_00698_amd.api import Population
    R, steps, K = 4, 60, 30
    B = inputs.gaussian_B()
    G = inputs.random_genomes(R, seed=60 + side, empty_bias=np.full(R, -3.0 if side == 2 else 0.0))
    P = Population([side] * R)
    Gt, Bt = torch.from_numpy(G).to(DEV), torch.from_numpy(B).to(DEV)
    P.build_from_genomes(Gt, Bt, SR_QUERY_FP32)
    P.record(K, steps)
    P.step(steps)
    g = P.backward(torch.from_numpy(_dJ(R, 2)).to(DEV), genomes=Gt, B=Bt)
    gg = g["genome"].cpu().numpy().astype(np.float64)
    gk, ga = (g[q].cpu().numpy().astype(np.float64) for q in ("k", "a"))
    cls, w = (q.cpu().numpy() for q in P.query())
    _, S, _, so = P.counts()
    for r in range(R):
        vox = slice(r * side ** 3, (r + 1) * side ** 3)
        robot = orc.Robot(side, cls[vox], w[vox].astype(np.float64))
        sp = robot.springs()
        sl = slice(so[r], so[r + 1])
        assert robot.S == S[r]
        # dJ/dk at fixed Z = k a (phases are zero here, and dJ/dIm Z carries no weight)
        gz = ga[sl] / sp["k"]
        dJdw = robot.dJdw(gk[sl] - sp["a"] * gz, gz, np.zeros_like(gz))
        go = orc.mlp_backward(G[r].astype(np.float64), B.astype(np.float64), side, dJdw)
        e = _l2rel(gg[r], go)
        say("side", side, "robot", r, "genome gradient relative L2 %.2e" % e)
        assert e <= TOL


def test_autograd_functions_route_through_the_adjoint():
    from paper_2405_00698_amd.api import GenomeFitness, Population, SpringFitness
    cls, w = voxel_population(C1, 53)
    P = gpu_population(C1, cls, w)
    sp = P.springs()
    k = sp["k"].clone().requires_grad_(True)
    a = sp["a"].clone().requires_grad_(True)
    phi = sp["phi"].clone().requires_grad_(True)
    wts = torch.from_numpy(_dJ(8, 3)).to(DEV)
    fit = SpringFitness.apply(k, a, phi, P, 120, 40)
    (fit * wts).sum().backward()
    P2 = gpu_population(C1, cls, w)
    P2.set_spring_params(k.detach(), a.detach(), phi.detach())
    P2.record(40, 120)
    P2.step(120)
    g = P2.backward(wts)
    assert torch.equal(k.grad, g["k"]) and torch.equal(a.grad, g["a"]) and torch.equal(phi.grad, g["phi"])
    # genome path
    B = torch.from_numpy(inputs.gaussian_B()).to(DEV)
    G = torch.from_numpy(inputs.random_genomes(4, seed=9)).to(DEV).requires_grad_(True)
    P3 = Population([4] * 4)
    f3 = GenomeFitness.apply(G, B, P3, 100, 25)
    f3.sum().backward()
    assert G.grad is not None and torch.isfinite(G.grad).all() and G.grad.abs().sum() > 0


def test_backward_without_recording_is_an_error():
    from paper_2405_00698_amd import _lib
    cls, w = voxel_population(C1, 54)
    P = gpu_population(C1, cls, w)
    P.step(10)
    with pytest.raises(_lib.SoftRobotError):
        P.backward(torch.ones(8, device=DEV))


def test_adjoint_forward_time_ratio_c4():
    """64 robots of 8^3, 2000 steps, checkpoint every 100: time of pop_backward
    (recompute included) over the forward pop_step(2000)."""
    sides = [8] * 64
    B = torch.from_numpy(inputs.gaussian_B()).to(DEV)
    G = torch.from_numpy(inputs.random_genomes(64, seed=1)).to(DEV)
    from paper_2405_00698_amd.api import Population
    P = Population(sides)
    P.build_from_genomes(G, B, SR_QUERY_FP32)
    P.record(100, 2000)
    P.step(200)
    torch.cuda.synchronize()
    P.reset()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    P.step(2000)
    torch.cuda.synchronize()
    tf = time.perf_counter() - t0
    dJ = torch.ones(64, device=DEV)
    P.backward(dJ)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    g = P.backward(dJ)
    torch.cuda.synchronize()
    tb = time.perf_counter() - t0
    say("C4 forward %.4f s  backward %.4f s  ratio %.2f" % (tf, tb, tb / tf))
    assert torch.isfinite(g["k"]).all()
    assert tb / tf < 10.0


@pytest.mark.parametrize("dash", [False, True])
def test_group_gradients_do_not_depend_on_the_other_groups(dash):
    """Side groups are reversed at their own pace through shared segment
    buffers; with a last segment shorter than the others (246 = 4 * 50 + 46)
    each group's spring gradients are the bits it has in a population alone."""
    from paper_2405_00698_amd import table2_params
    params = table2_params() if dash else None
    sides = [6, 7, 8, 9] * 13
    cls, w = voxel_population(sides, 68)
    at = np.concatenate([[0], np.cumsum([n ** 3 for n in sides])])

    def gradients(robots):
        from paper_2405_00698_amd.api import Population
        P = Population([sides[r] for r in robots], params=params)
        P.build_from_voxels(torch.from_numpy(np.concatenate([cls[at[r]:at[r + 1]] for r in robots])).to(DEV),
                            torch.from_numpy(np.concatenate([w[at[r]:at[r + 1]] for r in robots])).to(DEV))
        P.record(50, 246)
        P.step(246)
        out = [g.cpu().numpy() for g in P.backward(torch.ones(len(robots), device=DEV)).values()]
        off = np.concatenate([[0], np.cumsum(P.counts()[1])])
        return {r: [g[off[i]:off[i + 1]] for g in out] for i, r in enumerate(robots)}

    together = gradients(list(range(len(sides))))
    for n in (6, 7, 8, 9):
        alone = gradients([r for r in range(len(sides)) if sides[r] == n])
        for r, g in alone.items():
            for a, b in zip(g, together[r]):
                assert np.array_equal(a, b), (n, r)


@pytest.mark.parametrize("dash", [False, True])
@pytest.mark.parametrize("n", [8, 9, 10, 11, 12])
def test_gradient_pass_forms_give_the_same_bits(n, dash):
    """One segment is summed in tiles of 256 slots; of several, all but the one
    reversed last by the pass beside the reversal (where the side has one).
    Nine robots: a full and a nearly empty row of the tiles' XCD numbering."""
    from paper_2405_00698_amd import table2_params
    from paper_2405_00698_amd.api import Population
    sides = [n] * 9
    cls, w = voxel_population(sides, 69, p_empty=0.3)
    ref = None
    for K in (61, 20, 1):
        P = Population(sides, params=table2_params() if dash else None)
        P.build_from_voxels(torch.from_numpy(cls).to(DEV), torch.from_numpy(w).to(DEV))
        P.record(K, 61)
        P.step(61)
        g = [q.cpu().numpy() for q in P.backward(torch.ones(9, device=DEV)).values()]
        if ref is None:
            ref = g
        else:
            for a, b in zip(g, ref):
                assert np.array_equal(a, b), K


@pytest.mark.parametrize("n,dash", [(1, False), (5, True), (6, True), (7, True), (8, True), (9, True)])
def test_checkpoints_written_ahead_of_the_steps(n, dash):
    """Sides whose step kernel writes the checkpoint in a loop of its own: the
    gradients do not depend on how many checkpoints there are."""
    from paper_2405_00698_amd import table2_params
    from paper_2405_00698_amd.api import Population
    sides = [n] * 3
    cls, w = voxel_population(sides, 72, p_empty=0.0 if n == 1 else 0.3)
    ref = None
    for K in (40, 7, 1):
        P = Population(sides, params=table2_params() if dash else None)
        P.build_from_voxels(torch.from_numpy(cls).to(DEV), torch.from_numpy(w).to(DEV))
        P.record(K, 40)
        P.step(40)
        g = [q.cpu().numpy() for q in P.backward(torch.ones(3, device=DEV)).values()]
        assert np.abs(g[0]).max() > 0
        ref = ref or g
        for a, b in zip(g, ref):
            assert np.array_equal(a, b), K


@pytest.mark.parametrize("dash", [False, True])
@pytest.mark.parametrize("pair", [(8, 12), (5, 11), (4, 6), (9, 10)])
def test_two_group_gradients_are_those_of_each_alone(pair, dash):
    """Two sides share one recomputation stream, one stream of gradient passes and
    the segment buffers.  Two split reverse steps, a fused and a split one, two
    fused ones (with dashpots 9^3 and 10^3 sum beside the reversal in two parts,
    12^3 and 11^3 in tiles); two segments more than buffer sets, the last one
    short, and one step in a segment of its own."""
    from paper_2405_00698_amd import table2_params
    from paper_2405_00698_amd.api import Population
    params = table2_params() if dash else None
    sides = [pair[i % 3 == 0] for i in range(15)]  # ten of the first, five of the second
    cls, w = voxel_population(sides, 73, p_empty=0.25)
    at = np.concatenate([[0], np.cumsum([n ** 3 for n in sides])])

    def gradients(robots, K, steps):
        P = Population([sides[r] for r in robots], params=params)
        P.build_from_voxels(torch.from_numpy(np.concatenate([cls[at[r]:at[r + 1]] for r in robots])).to(DEV),
                            torch.from_numpy(np.concatenate([w[at[r]:at[r + 1]] for r in robots])).to(DEV))
        dJ = torch.tensor([1.0 + 0.1 * r for r in robots], device=DEV)
        out = []
        for _ in range(2):  # the second on the buffers that the first has left
            P.reset()
            P.record(K, steps)
            P.step(steps)
            out.append([g.cpu().numpy() for g in P.backward(dJ).values()])
        for a, b in zip(*out):
            assert np.array_equal(a, b)
        off = np.concatenate([[0], np.cumsum(P.counts()[1])])
        return {r: [g[off[i]:off[i + 1]] for g in out[0]] for i, r in enumerate(robots)}

    for K, steps in ((30, 30 * 4 + 17), (30, 30 * 3 + 1), (40, 25)):
        together = gradients(list(range(len(sides))), K, steps)
        for n in pair:
            alone = gradients([r for r in range(len(sides)) if sides[r] == n], K, steps)
            for r, g in alone.items():
                for a, b in zip(g, together[r]):
                    assert np.array_equal(a, b), (K, steps, n, r)
