"""Parity of the HIP sampler, energies and estimator against the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2606_22984_amd as fv
from oracle import estimator, network as net, philox, physics, sampler
from tests.gpu_util import ALL_PRECISIONS, DECISION_TOL, FP32, SITE_TOL, SPLIT, lattice_cfg, make_model, say, to_np
from workloads import ModelConfig, ea_instance, init_params, sk_instance
from workloads.instances import random_spins

pytestmark = pytest.mark.gpu


def _check_samples(theta, cfg, spins, lq, seed, stream, prec, rows=None, b0=0):
    """Teacher-forced decision check and sampled-vs-oracle log q on the given rows."""
    spins = to_np(spins)
    lq = to_np(lq).astype(np.float64)
    assert set(np.unique(spins)).issubset({-1, 1})
    assert np.all(np.isfinite(lq))
    idx = np.arange(spins.shape[0]) if rows is None else np.asarray(rows)
    sub = spins[idx]
    th = net.as_theta(theta)
    pp = net.cond_plus(th, cfg, sub, chunk=8).numpy()
    u = np.concatenate([philox.uniforms(seed, stream, 1, cfg.n_spins, b0 + b) for b in idx])
    wrong = (u < pp) != (sub > 0)
    gap = np.abs(u - pp)
    bad = int((wrong & (gap >= DECISION_TOL[prec])).sum())
    say(f"decision mismatches outside tol: {bad}; mismatches inside: {int(wrong.sum()) - bad}; "
        f"sites with |u-p|<1e-5: {int((gap < 1e-5).sum())} of {gap.size}")
    assert bad == 0
    ref = net.log_q(th, cfg, sub, chunk=8).numpy()
    per_site = np.abs(lq[idx] - ref) / cfg.n_spins
    say(f"max per-site |dlog q| {per_site.max():.3e}")
    assert per_site.max() <= SITE_TOL[prec]


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
@pytest.mark.parametrize("batch", [1024, 1000, 1])
def test_sample_sk16(prec, batch):
    cfg = ModelConfig(16, 32, 2, 2).full_causal()
    say("sk16", prec, batch)
    m, theta = make_model(cfg, batch, prec, seed=3)
    spins, lq = m.sample(batch, seed=77, stream_id=5)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 77, 5, prec)


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
def test_sample_sharp_conditionals(prec):
    """Head scaled x10: conditionals near 0/1 stress the decision and log-softmax tails."""
    cfg = ModelConfig(24, 32, 2, 2).with_mask(5, 3)
    say("sharp", prec)
    m, theta = make_model(cfg, 48, prec, seed=9, style="sharp")
    spins, lq = m.sample(48, seed=1, stream_id=2)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 1, 2, prec)


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
def test_sample_ea2d_L16(prec):
    cfg = lattice_cfg(16, 2, 64, 4, 4)
    assert (cfg.window, cfg.prefix) == (16, 17)
    say("ea2d_L16", prec)
    m, theta = make_model(cfg, 80, prec, seed=11)
    spins, lq = m.sample(70, seed=123, stream_id=9)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 123, 9, prec)


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
def test_sample_ea3d_L10_shape(prec):
    cfg = lattice_cfg(10, 3, 128, 8, 8)
    assert (cfg.window, cfg.prefix) == (100, 101)
    say("ea3d_L10", prec)
    m, theta = make_model(cfg, 40, prec, seed=21, style="default")
    spins, lq = m.sample(40, seed=5, stream_id=1)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 5, 1, prec, rows=[0, 17, 39])


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
def test_sample_sk512_shape(prec):
    cfg = ModelConfig(512, 128, 6, 8).full_causal()
    say("sk512", prec)
    m, theta = make_model(cfg, 20, prec, seed=31, style="default")
    spins, lq = m.sample(20, seed=8, stream_id=4)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 8, 4, prec, rows=[0, 19])


@pytest.mark.parametrize("prec", [SPLIT, FP32])
def test_sample_full_batch_ea3d(prec):
    """Full 3D workload batch (16384 samples, the benchmark's launch), sampled rows checked."""
    cfg = lattice_cfg(10, 3, 128, 8, 8)
    say("ea3d full batch", prec)
    m, theta = make_model(cfg, 16384, prec, seed=21, style="default")
    spins, lq = m.sample(16384, seed=2, stream_id=7)
    torch.cuda.synchronize()
    _check_samples(theta, cfg, spins, lq, 2, 7, prec, rows=[0, 8191, 16383])


def test_sampling_is_deterministic_and_seeded():
    cfg = lattice_cfg(6, 2, 32, 2, 2)
    m, theta = make_model(cfg, 64, FP32)
    a, la = m.sample(64, 4, 4)
    b, lb = m.sample(64, 4, 4)
    c, lc = m.sample(64, 5, 4)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(la, lb)
    assert not torch.equal(a, c)


def test_sample_rejects_bad_batch():
    cfg = ModelConfig(16, 32, 2, 2).full_causal()
    m, _ = make_model(cfg, 8, FP32)
    with pytest.raises(fv.FvanError):
        m.sample(9, 0, 0)


# ---------------------------------------------------------------- energies

@pytest.mark.parametrize("L,D,batch", [(16, 2, 4096), (32, 2, 333), (10, 3, 1), (3, 2, 5)])
def test_energy_pm1_bit_exact(L, D, batch):
    inst = ea_instance(L, D, 1000 + L, "pm1")
    say("energy pm1", L, D, batch)
    spins_np = random_spins(batch, inst.n, 3)
    spins = torch.as_tensor(spins_np, device="cuda")
    c = fv.couplings(inst)
    E = to_np(fv.energy(c, spins)).astype(np.int64)
    ref = physics.energy_edges_int(spins_np, inst.edges_i, inst.edges_j, inst.J)
    assert np.array_equal(E, ref)
    Em = to_np(fv.energy(c, -spins)).astype(np.int64)
    assert np.array_equal(Em, E)


@pytest.mark.parametrize("batch", [16384, 7])
def test_energy_gaussian_3d(batch):
    inst = ea_instance(10, 3, 4000, "gauss")
    spins_np = random_spins(batch, inst.n, 4)
    c = fv.couplings(inst)
    E = to_np(fv.energy(c, torch.as_tensor(spins_np, device="cuda"))).astype(np.float64)
    ref = physics.energy_edges(spins_np, inst.edges_i, inst.edges_j, inst.J.astype(np.float32).astype(np.float64))
    assert np.max(np.abs(E - ref)) / inst.n <= 1e-5


@pytest.mark.parametrize("n,batch", [(512, 8192), (512, 17), (16, 1024), (100, 1)])
def test_energy_dense_sk(n, batch):
    inst = sk_instance(n, 3000 + n)
    spins_np = random_spins(batch, n, 5)
    c = fv.couplings(inst)
    E = to_np(fv.energy(c, torch.as_tensor(spins_np, device="cuda"))).astype(np.float64)
    ref = physics.energy_dense(spins_np, inst.dense.astype(np.float32).astype(np.float64))
    assert np.max(np.abs(E - ref)) / n <= 1e-5


# ---------------------------------------------------------------- estimator

@pytest.mark.parametrize("is_int,batch", [(True, 4096), (False, 16384), (False, 2), (True, 1)])
def test_free_energy_and_weights(is_int, batch):
    rng = np.random.default_rng(batch)
    n, beta = 256, 0.7
    E = rng.integers(-500, 500, batch).astype(np.int32) if is_int else rng.normal(-300, 20, batch).astype(np.float32)
    lq = rng.normal(-150, 5, batch).astype(np.float32)
    Et = torch.as_tensor(E, device="cuda")
    lt = torch.as_tensor(lq, device="cuda")
    stats = to_np(fv.free_energy(Et, lt, beta, n))
    mean, var = estimator.free_energy_stats(E.astype(np.float64), lq.astype(np.float64), beta, n)
    assert abs(stats[0] - mean) <= 1e-12 * abs(mean)
    assert abs(stats[1] - var) <= 1e-9 * max(var, 1e-30) + 1e-300
    w = to_np(fv.reinforce_weights(Et, lt, beta)).astype(np.float64)
    wref = estimator.reinforce_weights(E.astype(np.float64), lq.astype(np.float64), beta)
    assert np.max(np.abs(w - wref)) <= 1e-6 * np.max(np.abs(wref)) + 1e-30
    s1 = to_np(fv.free_energy(Et, lt, beta, n))
    assert np.array_equal(s1, stats)           # fixed-order reduction: bitwise reproducible


def test_free_energy_end_to_end_ea2d():
    """F_q/N from GPU samples, GPU energies and GPU log q vs the oracle re-evaluating E and
    ln q in FP64 on the same samples: |dF_q/N| <= 1e-4."""
    inst = ea_instance(16, 2, 2000, "pm1")
    cfg = lattice_cfg(16, 2, 64, 4, 4)
    for prec in (FP32, SPLIT):
        m, theta = make_model(cfg, 64, prec, seed=2, style="default")
        spins, lq = m.sample(64, 3, 1)
        c = fv.couplings(inst)
        E = fv.energy(c, spins)
        stats = to_np(fv.free_energy(E, lq, 1.0, cfg.n_spins))
        sp = to_np(spins)
        E_ref = physics.energy_edges_int(sp, inst.edges_i, inst.edges_j, inst.J)
        assert np.array_equal(to_np(E).astype(np.int64), E_ref)
        lq_ref = net.log_q(net.as_theta(theta), cfg, sp).numpy()
        mean_ref, _ = estimator.free_energy_stats(E_ref, lq_ref, 1.0, cfg.n_spins)
        say(f"prec {prec}: dF/N = {abs(stats[0] - mean_ref):.3e}")
        assert abs(stats[0] - mean_ref) <= 1e-4


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
def test_free_energy_parity_ea3d(prec):
    """|F_q/N (GPU) - F_q/N (oracle, FP64 on the GPU's samples)| <= 1e-4 at the 3D workload, per beta."""
    inst = ea_instance(10, 3, 4000, "gauss")
    cfg = lattice_cfg(10, 3, 128, 8, 8)
    B = 32
    m, theta = make_model(cfg, B, prec, seed=21, style="default")
    spins, lq = m.sample(B, 6, 2)
    c = fv.couplings(inst)
    E = fv.energy(c, spins)
    sp = to_np(spins)
    E_ref = physics.energy_edges(sp, inst.edges_i, inst.edges_j, inst.J.astype(np.float32).astype(np.float64))
    lq_ref = net.log_q(net.as_theta(theta), cfg, sp, chunk=4).numpy()
    for beta in (0.5, 1.0, 2.0):
        stats = to_np(fv.free_energy(E, lq, beta, cfg.n_spins))
        mean_ref, _ = estimator.free_energy_stats(E_ref, lq_ref, beta, cfg.n_spins)
        dF = abs(stats[0] - mean_ref)
        say(f"prec {prec} beta {beta}: |dF_q/N| = {dF:.3e}")
        assert dF <= 1e-4


@pytest.mark.parametrize("n,batch,offset", [(1, 3, 0), (63, 33, 0), (64, 16, 0), (65, 17, 1), (128, 4096, 0),
                                            (129, 4097, 0), (256, 4095, 1), (257, 100, 0), (512, 33, 0), (513, 20, 0),
                                            (4096, 33, 0)])
def test_energy_dense_tile_edges(n, batch, offset):
    """Dense energies at the edges of the kernel's column blocks and sample tiles, with rows and matrices that
    are not 16-byte aligned (offset: J starts that many floats into its allocation), against FP64.  Bound: every
    partial sum has at most n FP32 terms in a row, within n 2^-24 sum |J_ij| in all."""
    rng = np.random.default_rng(n)
    J = rng.standard_normal((n, n)).astype(np.float32)
    store = torch.zeros(n * n + offset, device="cuda")
    store[offset:] = torch.as_tensor(J.reshape(-1), device="cuda")
    c = fv.CouplingsC(n_spins=n, kind=fv.BONDS_DENSE, degree=0, nbr=None, J=store.data_ptr() + 4 * offset)
    coup = fv.Couplings(n, fv.BONDS_DENSE, 0, None, store, c)
    s = random_spins(batch, n, 3)
    E = to_np(fv.energy(coup, torch.as_tensor(s, device="cuda"))).astype(np.float64)
    x = s.astype(np.float64)
    ref = -0.5 * ((x @ J.astype(np.float64).T) * x).sum(1)
    tol = 0.5 * np.abs(J.astype(np.float64)).sum() * n * 2.0 ** -24 + np.abs(ref) * 2.0 ** -24
    assert np.all(np.abs(E - ref) <= tol)


def test_energy_dense_spins_other_than_pm1():
    """Entries other than +-1 (here 0 and 2) keep the plain definition -1/2 sum J_ij s_i s_j."""
    n, batch = 130, 40
    rng = np.random.default_rng(8)
    inst = sk_instance(n, 5)
    s = random_spins(batch, n, 6)
    s[5, 7], s[20, 0], s[39, 129] = 0, 2, 0
    E = to_np(fv.energy(fv.couplings(inst), torch.as_tensor(s, device="cuda"))).astype(np.float64)
    x, J = s.astype(np.float64), inst.dense.astype(np.float32).astype(np.float64)
    ref = -0.5 * ((x @ J) * x).sum(1)
    assert np.max(np.abs(E - ref)) / n <= 1e-5


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
@pytest.mark.parametrize("d,dh,vocab", [(32, 16, 2), (64, 16, 2), (128, 16, 2), (64, 32, 2), (128, 64, 256)])
def test_samples_do_not_depend_on_the_batch(d, dh, vocab, prec):
    """The samples a workgroup owns (4, 8, 16 or 32) go by the batch; sample b is the same bits in every batch.
    37 visible keys: more than one K/V batch per sample at every width; ragged last workgroups."""
    cfg = ModelConfig(45, d, 2, d // dh, d_token=2 if vocab == 2 else 8, vocab=vocab, window=20, prefix=16)
    batches = (3, 37, 1029, 2051, 4099, 8200)
    m = fv.Model(cfg, batches[-1], prec, init_params(cfg, 3, "random"), workspaces=fv.WS_SAMPLER)
    ref = None
    for B in batches:
        s, lq = (m.sample if vocab == 2 else m.sample_tokens)(B, 11, 2)
        n = min(B, 37)
        if B == 37:
            ref = (s.clone(), lq.clone())
        elif ref is not None:
            assert torch.equal(s[:n], ref[0][:n]) and torch.equal(lq[:n], ref[1][:n]), B
            if B > 1029:
                assert torch.equal(s[:1029], last[0][:1029]) and torch.equal(lq[:1029], last[1][:1029]), B
        last = (s.clone(), lq.clone())


@pytest.mark.parametrize("vocab,batch", [(3, 1), (16, 5), (33, 37), (255, 9), (256, 4099)])
def test_token_head_of_any_vocabulary(vocab, batch):
    """The sampler's ln q against the teacher-forced pass of the same tokens: vocabularies off the
    padding's multiple of 32, and 1 to 16 samples per half workgroup.  Both are FP32 sums of at most
    64 terms per logit: a site's ln q agrees to a few hundred ulp."""
    cfg = ModelConfig(9, 64, 2, 4, d_token=8, vocab=vocab, window=5, prefix=2)
    m = fv.Model(cfg, batch, FP32, init_params(cfg, 4, "random"))
    tok, lq = m.sample_tokens(batch, 21, 1)
    assert int(tok.max()) < vocab
    ref = to_np(m.log_prob_tokens(tok)).astype(np.float64)
    assert np.max(np.abs(to_np(lq).astype(np.float64) - ref)) / cfg.n_spins <= 5e-5


@pytest.mark.parametrize("n,batch,offset", [(1, 3, 0), (12, 17, 0), (13, 17, 1), (63, 33, 0), (64, 16, 0), (65, 17, 1),
                                            (128, 4096, 0), (129, 4097, 0), (256, 4095, 1), (257, 100, 0), (511, 31, 0),
                                            (512, 33, 0), (513, 20, 0), (4096, 33, 0)])
def test_energy_dense_of_unit_couplings_is_exact(n, batch, offset):
    """Couplings of +-1 (n^2 <= 2^24 of them): every partial sum is an integer that FP32 holds, in any order, so the
    energies are equal to the integer ones; an element lost, doubled or taken from another row would show."""
    rng = np.random.default_rng(n + 1)
    up = np.triu(rng.choice(np.array([-1, 1], np.int8), (n, n)), 1)
    J = up + up.T
    store = torch.zeros(n * n + offset, device="cuda")
    store[offset:] = torch.as_tensor(J.reshape(-1).astype(np.float32), device="cuda")
    c = fv.CouplingsC(n_spins=n, kind=fv.BONDS_DENSE, degree=0, nbr=None, J=store.data_ptr() + 4 * offset)
    coup = fv.Couplings(n, fv.BONDS_DENSE, 0, None, store, c)
    s = random_spins(batch, n, 3)
    E = to_np(fv.energy(coup, torch.as_tensor(s, device="cuda"))).astype(np.float64)
    x = s.astype(np.float64)
    assert np.array_equal(E, -0.5 * ((x @ J.astype(np.float64)) * x).sum(1))


@pytest.mark.parametrize("prec", ALL_PRECISIONS)
@pytest.mark.parametrize("d,dh,vocab", [(32, 16, 2), (64, 16, 2), (128, 16, 2), (64, 32, 2), (128, 64, 256)])
def test_samples_of_every_batch_are_those_of_the_largest(d, dh, vocab, prec):
    """Sample b is the same bits in every batch, against the largest (two rounds of 32-sample workgroups): one sample,
    a single ragged 4-sample workgroup, and every workgroup size with a ragged last one."""
    cfg = ModelConfig(45, d, 2, d // dh, d_token=2 if vocab == 2 else 8, vocab=vocab, window=20, prefix=16)
    m = fv.Model(cfg, 8200, prec, init_params(cfg, 3, "random"), workspaces=fv.WS_SAMPLER)
    call = m.sample if vocab == 2 else m.sample_tokens
    ref_s, ref_lq = call(8200, 11, 2)
    assert torch.isfinite(ref_lq).all() and len(torch.unique(ref_s)) > 1
    for B in (1, 3, 37, 1029, 2051, 4099):
        s, lq = call(B, 11, 2)
        assert torch.equal(s, ref_s[:B]) and torch.equal(lq, ref_lq[:B]), B
