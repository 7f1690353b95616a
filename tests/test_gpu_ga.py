"""GPU GA generation against the oracle on identical fitness, genomes and
Philox counters: every integer decision (ranks, elites, tournament winners,
crossover flags) bit-exact; copied genes bitwise; mutated genes within FP32
rounding of the oracle's FP64 value."""
import math

import numpy as np
import pytest
import torch

from gpu_util import DEV, need_gpu, say
from paper_2405_00698_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _run_both(orc, fit, G, **kw):
    from paper_2405_00698_amd.api import GAConfig, ga_generation
    P, L = G.shape
    cfg = GAConfig(**{k: v for k, v in kw.items() if k in ("elite_frac", "tournament_k", "p_cross", "p_mut", "sigma")})
    seed, gen = kw.get("seed", 3), kw.get("generation", 0)
    gin = torch.from_numpy(G).to(DEV)
    gout = torch.empty_like(gin)
    dec = torch.empty((P, 3), dtype=torch.int32, device=DEV)
    ga_generation(torch.from_numpy(fit.astype(np.float32)).to(DEV), gin, gout, cfg, seed=seed, generation=gen,
                  decisions=dec)
    ref, rdec = orc.ga_generation(fit.astype(np.float32).astype(np.float64), G.astype(np.float64),
                                  elite_frac=kw.get("elite_frac", 0.3), k=kw.get("tournament_k", 4),
                                  p_cross_thr=cfg.params.p_cross_thr, p_mut_thr=cfg.params.p_mut_thr,
                                  sigma=float(np.float32(kw.get("sigma", 0.02))), seed=seed, generation=gen)
    return gout.cpu().numpy(), dec.cpu().numpy(), ref, rdec


def _check(G, out, dec, ref, rdec):
    assert np.array_equal(dec, rdec)
    for c in range(G.shape[0]):
        A, B, kind = rdec[c]
        if kind == 0:
            assert np.array_equal(out[c], G[A])
            continue
        src_ok = (out[c] == G[A]) | (out[c] == G[B])
        diff = np.abs(out[c].astype(np.float64) - ref[c])
        # genes that were copied are bitwise the oracle's; mutated ones agree to FP32 rounding
        assert np.all(diff[src_ok & (ref[c] == out[c])] == 0)
        assert np.all(diff <= 1e-6 * np.maximum(1.0, np.abs(ref[c])))


@pytest.mark.parametrize("P,L,k,elite,seed,gen", [(5, 3, 4, 0.3, 3, 0), (33, 300, 4, 0.3, 7, 5),
                                                  (64, 1000, 1, 0.0, 9, 1), (31, 257, 7, 0.5, 11, 2 ** 40),
                                                  (16, 64, 64, 1.0, 1, 3), (1, 5, 4, 0.3, 2, 0)])
def test_ga_matches_oracle(orc, P, L, k, elite, seed, gen):
    g = np.random.default_rng(P + L)
    fit = g.normal(size=P).astype(np.float32)
    if P > 4:
        fit[2] = fit[4]
        fit[3] = np.nan
    G = g.normal(size=(P, L)).astype(np.float32)
    out, dec, ref, rdec = _run_both(orc, fit, G, tournament_k=k, elite_frac=elite, seed=seed, generation=gen,
                                    p_cross=0.4, p_mut=0.1)
    _check(G, out, dec, ref, rdec)


@pytest.mark.parametrize("L", [255, 256, 1793, 2047, 2048, 2049, 3072, 3073, 6145, 18433])
@pytest.mark.parametrize("P", [9, 600])
def test_ga_chunk_edges(orc, L, P):
    """Genome lengths around the 256-gene mask blocks and the workgroups' chunk
    (1024 genes for a few genomes, up to 3072 for many), every gene mutating in
    half of the runs."""
    g = np.random.default_rng(L)
    G = g.normal(size=(P, L)).astype(np.float32)
    fit = g.normal(size=P).astype(np.float32)
    out, dec, ref, rdec = _run_both(orc, fit, G, seed=L, generation=2, p_mut=1.0 if L % 2 else 0.1, p_cross=0.7)
    _check(G, out, dec, ref, rdec)


def test_ga_workload_size_decisions(orc):
    """1024 genomes of 8710 genes (the uneven-batch population)."""
    P, L = 1024, inputs.GENOME_LEN
    G = inputs.random_genomes(P, seed=5)
    fit = np.random.default_rng(1).normal(size=P).astype(np.float32)
    say("GA 1024 x 8710")
    out, dec, ref, rdec = _run_both(orc, fit, G, seed=3, generation=7)
    _check(G, out, dec, ref, rdec)
    moved = (out != G[dec[:, 0]]) & (out != G[dec[:, 1]])
    assert 0.08 < moved[dec[:, 2] != 0].mean() < 0.12


def test_ga_rejects_overlap_and_bad_k():
    from paper_2405_00698_amd import _lib
    from paper_2405_00698_amd.api import GAConfig, ga_generation
    g = torch.zeros((8, 4), device=DEV)
    f = torch.zeros(8, device=DEV)
    with pytest.raises(_lib.SoftRobotError):
        ga_generation(f, g, g, GAConfig())
    with pytest.raises(_lib.SoftRobotError):
        ga_generation(f, g, torch.zeros_like(g), GAConfig(tournament_k=0))
