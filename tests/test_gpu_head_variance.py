"""GPU-vs-oracle parity of the attention variance used by the offline head
classification (Sec. 4.2), and recovery of the mask planted in the synthetic
workload from the GPU's numbers."""
import numpy as np
import pytest
import torch

from oracle import hack_oracle as ho
from paper_2504_09261_amd import workload as wl
from paper_2504_09261_amd.binding import HackError

pytestmark = pytest.mark.gpu

# Probabilities are float32 values formed from chained-MFMA scores: their relative
# error is a few 1e-6 for ordinary logits; the two moments are accumulated in fp64,
# so sigma = E[A^2] - E[A]^2 inherits that relative error against its larger term.
REL, ABS = 2e-5, 1e-9


def _u():
    from tests import gpu_util
    return gpu_util


def _final_step(cfg, layer):
    data = wl.gen_layer(cfg, layer)
    K = np.concatenate([data[k].k for k in range(1, cfg.n_steps + 1)], axis=2)       # [B, H, T_K, d]
    return data[cfg.n_steps].q, K


def _sigma_gpu(hk, u, cfg, Q, K):
    B, H = Q.shape[0], Q.shape[1]
    rows = [(K[b, h], K[b, h]) for b in range(B) for h in range(H)]
    cache, _ = u.build_cache(rows, cfg.head_dim, cfg.dtype)
    sigma = torch.full((B * H,), -1.0, dtype=torch.float64, device=u.DEV)
    hk.head_variance(u.to_dev(Q, cfg.dtype), cache, cfg.scale, sigma)
    torch.cuda.synchronize()
    return sigma.cpu().numpy()


@pytest.mark.parametrize("cfg_id,layer", [(1, 0), (1, 3)])
def test_head_variance_matches_oracle_and_recovers_the_planted_mask(cfg_id, layer):
    u = _u()
    cfg = wl.get_config(cfg_id, batch=2)
    hk = u.make_hack(cfg)
    Q, K = _final_step(cfg, layer)
    got = _sigma_gpu(hk, u, cfg, Q, K)
    types = wl.head_types(cfg, layer)
    want = np.array([ho.head_variance(Q[b, h].astype(np.float64), K[b, h].astype(np.float64), cfg.scale)
                     for b in range(cfg.batch) for h in range(cfg.heads)])
    assert np.all(np.abs(got - want) <= REL * np.maximum(want, 1e-3) + ABS), float(np.max(np.abs(got - want) / want))
    mean_sigma = got.reshape(cfg.batch, cfg.heads).mean(axis=0)          # "averaged over a validation set"
    assert np.array_equal(ho.classify_heads(mean_sigma, float((types == 0).mean())), types)
    hk.close()


def test_head_variance_ragged_shapes_and_degenerate_cases():
    u = _u()
    rng = np.random.default_rng(9)
    H, B, d, dtype = 3, 2, 128, "bf16"
    for Nk, lens in ((37, [1, 31, 32, 33, 200, 95]), (1, [5, 64, 1, 77, 129, 2]), (130, [130, 259, 7, 64, 63, 400])):
        hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=H * B, max_cache_len=512, max_queries=Nk)
        rows = [(u.rand_values(rng, (n, d), dtype), None) for n in lens]
        rows = [(k, k) for k, _ in rows]
        cache, _ = u.build_cache(rows, d, dtype, pad_rows=3, fill=50.0)   # poison between units
        Q = wl.bf16_to_f32(wl.bf16_round(u.rand_values(rng, (B, H, Nk, d), dtype)))
        sigma = torch.full((H * B,), -1.0, dtype=torch.float64, device=u.DEV)
        hk.head_variance(u.to_dev(Q, dtype), cache, 0.09, sigma)
        torch.cuda.synchronize()
        got = sigma.cpu().numpy()
        for uu in range(H * B):
            b, h = divmod(uu, H)
            want = ho.head_variance(Q[b, h].astype(np.float64), rows[uu][0].astype(np.float64), float(np.float32(0.09)))
            assert abs(got[uu] - want) <= REL * max(want, 1e-3) + ABS, (Nk, uu, got[uu], want)
        if Nk == 1:
            assert np.all(np.abs(got) < 1e-12)                            # one query: no variance
        hk.close()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_head_variance_without_variance(head_dim):
    """One query: exactly zero whatever the keys.  The same query many times over: never negative, and within the fp64
    rounding of the two moments, whose size is at most N sum_j A_j^2 / N <= 1 (2^-53 per sum, some 1e3 of them)."""
    u = _u()
    rng = np.random.default_rng(head_dim)
    lens = [1, 33, 64, 257, 300, 1000]
    hk = u.make_hack(heads=6, head_dim=head_dim, dtype="bf16", max_units=6, max_cache_len=1000, max_queries=70)
    cache, _ = u.build_cache([(k, k) for k in (u.rand_values(rng, (n, head_dim), "bf16") for n in lens)], head_dim, "bf16")
    row = u.rand_values(rng, (1, 6, 1, head_dim), "bf16")
    for Nk in (1, 70):
        sigma = torch.full((6,), -1.0, dtype=torch.float64, device=u.DEV)
        hk.head_variance(u.to_dev(np.repeat(row, Nk, axis=2), "bf16"), cache, 0.125, sigma)
        got = sigma.cpu().numpy()
        assert np.all(got == 0.0) if Nk == 1 else np.all((got >= 0.0) & (got < 1e-12)), (Nk, got)
    hk.close()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("Nk,lens", [(96, [1, 96, 224]), (225, [225, 256, 257]), (257, [320, 353, 640])])
def test_head_variance_pipeline_lengths_and_rising_logits(head_dim, Nk, lens):
    """Lengths around the pipeline's fill, steady loop and drain on both sides, with keys that grow along the cache so
    that pass 1 has to move its reference again and again.  Largest logit about 18 nats: a chained float32 dot product
    is off by at most D 2^-24 times the sum of its |products|, here below 6e-6 nats, which moves a probability by
    as much and sigma by twice that."""
    u = _u()
    rng = np.random.default_rng(100 * Nk + head_dim)
    hk = u.make_hack(heads=3, head_dim=head_dim, dtype="bf16", max_units=3, max_cache_len=640, max_queries=Nk)
    rows = [wl.bf16_to_f32(wl.bf16_round(u.rand_values(rng, (n, head_dim), "bf16") * np.linspace(0.1, 4.0, n, dtype=np.float32)[:, None]))
            for n in lens]
    cache, _ = u.build_cache([(k, k) for k in rows], head_dim, "bf16", pad_rows=3, fill=50.0)
    Q = wl.bf16_to_f32(wl.bf16_round(u.rand_values(rng, (1, 3, Nk, head_dim), "bf16")))
    scale = float(np.float32(head_dim ** -0.5))
    sigma = torch.full((3,), -1.0, dtype=torch.float64, device=u.DEV)
    hk.head_variance(u.to_dev(Q, "bf16"), cache, scale, sigma)
    torch.cuda.synchronize()
    for h in range(3):
        want = ho.head_variance(Q[0, h].astype(np.float64), rows[h].astype(np.float64), scale)
        assert abs(float(sigma[h]) - want) <= REL * max(want, 1e-3) + ABS, (h, float(sigma[h]), want)
    hk.close()


def test_head_variance_full_size_sampled_units_and_errors():
    """The 1024^2 benchmark shape (4096 queries x 10521 keys per unit) on the device;
    two units through the oracle."""
    u = _u()
    cfg = wl.get_config(2)
    hk = u.make_hack(cfg)
    Q, K = _final_step(cfg, 0)
    got = _sigma_gpu(hk, u, cfg, Q, K)
    types = wl.head_types(cfg, 0)
    for uu in (int(np.where(types == 0)[0][0]), cfg.heads + int(np.where(types == 1)[0][0])):
        b, h = divmod(uu, cfg.heads)
        want = ho.head_variance(Q[b, h].astype(np.float64), K[b, h].astype(np.float64), cfg.scale)
        assert abs(got[uu] - want) <= REL * max(want, 1e-3) + ABS, (uu, got[uu], want)
    mean_sigma = got.reshape(cfg.batch, cfg.heads).mean(axis=0)
    assert np.array_equal(ho.classify_heads(mean_sigma, float((types == 0).mean())), types)
    with pytest.raises(HackError):
        hk.head_variance(u.to_dev(Q, cfg.dtype), u.build_cache([(K[0, 0], K[0, 0])] * cfg.n_units, cfg.head_dim, cfg.dtype)[0],
                         -1.0, torch.zeros(cfg.n_units, dtype=torch.float64, device=u.DEV))
    hk.close()
    hk32 = u.make_hack(wl.get_config(0))
    with pytest.raises(HackError):
        c0 = wl.get_config(0)
        hk32.head_variance(torch.zeros((1, c0.heads, 4, c0.head_dim), device=u.DEV),
                           u.build_cache([(np.zeros((4, c0.head_dim), np.float32),) * 2] * c0.heads, c0.head_dim, "f32")[0],
                           0.1, torch.zeros(c0.heads, dtype=torch.float64, device=u.DEV))
    hk32.close()
