"""Per-kernel GPU-vs-oracle parity through the C ABI (ctypes binding).

Bars: kept-index sets and compaction bit-exact; importance within a few float32
ulp of the fp64 oracle; attention within 2e-2 max-abs (bf16) / 1e-4 (fp32).
"""
import numpy as np
import pytest
import torch

from oracle import hack_oracle as ho
from paper_2504_09261_amd import workload as wl
from paper_2504_09261_amd.binding import Cache, HackError

pytestmark = pytest.mark.gpu


def _u():
    from tests import gpu_util
    return gpu_util


# ---------------------------------------------------------------------------
# a3 compact
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
def test_compact_bit_exact_two_sources_and_pos(dtype, d):
    u = _u()
    rng = np.random.default_rng(42 + d)
    H, B, Nk = 4, 2, 37
    U = H * B
    lens = [0, 1, 63, 64, 65, 300, 7, 129]
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=U, max_cache_len=512, max_queries=64)
    rows = [(u.rand_values(rng, (n, d), dtype), u.rand_values(rng, (n, d), dtype)) for n in lens]
    cin, off_in = u.build_cache(rows, d, dtype, pad_rows=3)
    pos_in = np.full(cin.rows, -7, np.int32)
    for o, n in zip(off_in, lens):
        pos_in[o:o + n] = 1000 + np.arange(n)
    cin.pos = torch.from_numpy(pos_in).to(u.DEV)
    k_new, v_new = u.rand_values(rng, (B, H, Nk, d), dtype), u.rand_values(rng, (B, H, Nk, d), dtype)
    keep = [min(n + Nk, k) for n, k in zip(lens, [5, 38, 1, 101, 64, 200, 44, 0])]
    idx_stride = 256
    idx = np.zeros((U, idx_stride), np.int32)
    sel = []
    for uu, (n, k) in enumerate(zip(lens, keep)):
        I = np.sort(rng.choice(n + Nk, size=k, replace=False)).astype(np.int32)
        sel.append(I)
        idx[uu, :k] = I
    off_out, total_out = u.aligned_offsets(keep, pad_rows=5)
    sentinel = 3.0
    Kout = torch.full((total_out, d), sentinel, dtype=hk.torch_dtype, device=u.DEV)
    Vout = torch.full((total_out, d), sentinel, dtype=hk.torch_dtype, device=u.DEV)
    Pout = torch.full((total_out,), -1, dtype=torch.int32, device=u.DEV)
    cout = Cache(Kout, Vout, off_out, np.asarray(keep, np.int32), Pout)
    hk.compact(B, Nk, cin, torch.from_numpy(idx).to(u.DEV), cout, u.to_dev(k_new, dtype), u.to_dev(v_new, dtype),
               pos_new=5000)
    torch.cuda.synchronize()
    Kg, Vg, Pg = u.from_dev(Kout), u.from_dev(Vout), Pout.cpu().numpy()
    touched = np.zeros(total_out, bool)
    for uu in range(U):
        b, h = divmod(uu, H)
        K_in = np.concatenate([rows[uu][0], k_new[b, h]]).astype(np.float64)
        V_in = np.concatenate([rows[uu][1], v_new[b, h]]).astype(np.float64)
        P_in = np.concatenate([1000 + np.arange(lens[uu]), 5000 + np.arange(Nk)])
        Kh, Vh = ho.compact(K_in, V_in, sel[uu])
        o, n = off_out[uu], keep[uu]
        assert np.array_equal(Kg[o:o + n], Kh) and np.array_equal(Vg[o:o + n], Vh)
        assert np.array_equal(Pg[o:o + n], P_in[sel[uu]])
        touched[o:o + n] = True
    assert np.all(Kg[~touched] == sentinel) and np.all(Pg[~touched] == -1)   # nothing written outside
    hk.close()


def test_compact_rejects_overlap_and_bad_ranges():
    u = _u()
    hk = u.make_hack(heads=1, head_dim=64, dtype="bf16", max_units=1, max_cache_len=64, max_queries=8)
    K = torch.zeros((64, 64), dtype=torch.bfloat16, device=u.DEV)
    idx = torch.zeros((1, 64), dtype=torch.int32, device=u.DEV)
    cin = Cache(K, K.clone(), [0], [16])
    with pytest.raises(HackError):       # output on top of rows that are read
        hk.compact(1, 1, cin, idx, Cache(K, cin.v, [8], [4]))
    with pytest.raises(HackError):       # output beyond the array
        hk.compact(1, 1, cin, idx, Cache(K.clone(), K.clone(), [56], [16]))
    with pytest.raises(HackError):       # keeps more rows than exist
        hk.compact(1, 1, cin, idx, Cache(K.clone(), K.clone(), [0], [17]))
    with pytest.raises(HackError):       # misaligned offset
        hk.compact(1, 1, Cache(K, K.clone(), [3], [4]), idx, Cache(K.clone(), K.clone(), [0], [2]))
    hk.close()


# ---------------------------------------------------------------------------
# a2 select
# ---------------------------------------------------------------------------
def _select_case(u, hk, imp_rows, t_in, head_type, budget, n_init, n_recent, H):
    U = len(t_in)
    stride = int(max(t_in))
    stride = (stride + 63) // 64 * 64
    imp = np.zeros((U, stride), np.float32)
    for i, r in enumerate(imp_rows):
        imp[i, :len(r)] = r
    kept = torch.full((U, stride), -1, dtype=torch.int32, device=u.DEV)
    len_out = hk.select(U // H, torch.from_numpy(imp).to(u.DEV), t_in, head_type, budget, n_init, n_recent, kept)
    torch.cuda.synchronize()
    kept = kept.cpu().numpy()
    for i in range(U):
        want = ho.select(imp_rows[i].astype(np.float64), int(head_type[i % H]), int(budget[i]), n_init, n_recent)
        assert len_out[i] == len(want) == min(budget[i], t_in[i])
        assert np.array_equal(kept[i, :len_out[i]], want), f"unit {i}: T={t_in[i]} b={budget[i]} type={head_type[i % H]}"
        assert np.all(kept[i, len_out[i]:] == -1)


def test_select_bit_exact_random_ragged():
    u = _u()
    rng = np.random.default_rng(5)
    H = 8
    hk = u.make_hack(heads=H, head_dim=64, dtype="bf16", max_units=32, max_cache_len=8831, max_queries=4096)
    head_type = np.array([0, 1, 0, 1, 1, 0, 1, 0], np.uint8)
    n_init, n_recent = 5, 64
    t_in = np.array([8831, 8831, 6039, 7981, 65, 64, 1025, 300,  70, 69, 1023, 1024, 4121, 2521, 100, 77], np.int32)
    budget = np.array([1579, 4735, 1943, 3885, 65, 1, 700, 299,   1, 69, 1022, 9999, 3885, 1943, 69, 76], np.int32)
    rows = []
    for T in t_in:
        r = rng.random(T).astype(np.float32) * np.float32(32.0 / T)
        dup = rng.integers(0, T, max(2, T // 10))           # plant exact duplicates around the threshold
        r[dup] = r[dup[0]]
        rows.append(r)
    _select_case(u, hk, rows, t_in, head_type, budget, n_init, n_recent, H)
    # swapped classes
    _select_case(u, hk, rows, t_in, 1 - head_type, budget, n_init, n_recent, H)
    hk.close()


def test_select_ties_and_degenerate_segments():
    u = _u()
    H = 2
    hk = u.make_hack(heads=H, head_dim=64, dtype="bf16", max_units=8, max_cache_len=2048, max_queries=256)
    head_type = np.array([0, 1], np.uint8)
    T = 1500
    flat = np.full(T, np.float32(32.0 / T))
    two = flat.copy()
    two[::3] *= 2
    zeros = np.zeros(T, np.float32)
    tiny = np.full(T, np.float32(1e-39))              # subnormal importance
    rows = [flat, flat, two, two, zeros, zeros, tiny, tiny]
    t_in = np.full(8, T, np.int32)
    for budget in (1, 5, 69, 70, 500, 501, 1499):
        _select_case(u, hk, rows, t_in, head_type, np.full(8, budget, np.int32), 5, 64, H)
    # structural budget below init + recent (small-budget reading) and n_init > T - n_recent
    _select_case(u, hk, rows, t_in, head_type, np.full(8, 40, np.int32), 5, 64, H)
    _select_case(u, hk, [r[:66] for r in rows], np.full(8, 66, np.int32), head_type, np.full(8, 65, np.int32), 5, 64, H)
    hk.close()


@pytest.mark.parametrize("T", [1, 255, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 16384, 16385, 32768])
def test_select_every_size_class_and_digit(T):
    """Both sides of every launch form, with importance whose threshold is settled by the first, second or last digit of
    the keys, in ties of equal keys, and with rows that are not 16-byte aligned: exact."""
    u = _u()
    rng = np.random.default_rng(T)
    pad = 1 if T % 2 else 4           # odd strides take the unaligned loads
    stride = T + pad
    spread = rng.lognormal(-6, 2, T)                                     # fifty octave pieces
    close = (1.0 + rng.integers(0, 1 << 9, T) * 2.0 ** -23)              # equal but for the last nine bits
    few = rng.integers(0, 3, T).astype(np.float64)                       # three values, zero among them
    second = (1.0 + rng.permutation(T) * 2.0 ** -18)                     # inside one first-digit bin up to T = 2^15
    imp_h = np.zeros((4, stride), np.float32)
    for i, x in enumerate((spread, close, few, second)):
        imp_h[i, :T] = x
    hk = u.make_hack(heads=4, head_dim=64, dtype="bf16", max_units=4, max_cache_len=32768, max_queries=16)
    imp = torch.from_numpy(imp_h).to(u.DEV)
    for budget, n_init, n_recent, types in (((T + 1) // 2, 0, 0, [0, 0, 0, 0]), (max(1, T // 3), min(5, T // 4), T // 5, [1, 1, 0, 1]),
                                            (1, 0, 0, [0, 0, 0, 0]), (max(1, T - 1), 0, min(3, T), [0, 1, 1, 0])):
        kept = torch.full((4, stride), -1, dtype=torch.int32, device=u.DEV)
        ln = hk.select(1, imp, [T] * 4, types, [budget] * 4, n_init, n_recent, kept)
        torch.cuda.synchronize()
        for h in range(4):
            want = ho.select(imp_h[h, :T], types[h], budget, n_init, n_recent)
            got = kept[h, :ln[h]].cpu().numpy()
            assert np.array_equal(got, want), (T, h, budget)
            assert torch.all(kept[h, ln[h]:] == -1)
    hk.close()


@pytest.mark.parametrize("T", [4100, 6143, 6144, 6145, 12284, 12287, 12288, 12289])
def test_select_forms_of_6_and_12_keys_a_thread(T):
    test_select_every_size_class_and_digit(T)


def test_select_rejects_bad_arguments():
    u = _u()
    hk = u.make_hack(heads=1, head_dim=64, dtype="bf16", max_units=1, max_cache_len=128, max_queries=16)
    imp = torch.zeros((1, 128), device=u.DEV)
    kept = torch.zeros((1, 128), dtype=torch.int32, device=u.DEV)
    with pytest.raises(HackError):
        hk.select(1, imp, [100], [0], [0], 5, 16, kept)           # budget < 1
    with pytest.raises(HackError):
        hk.select(1, imp, [129], [0], [10], 5, 16, kept)          # T above max_cache_len
    with pytest.raises(HackError):
        hk.select(1, imp, [100], [2], [10], 5, 16, kept)          # bad head class
    with pytest.raises(HackError):
        hk.select(1, imp, [10], [1], [5], 5, 16, kept)            # n_recent > T
    hk.close()


# ---------------------------------------------------------------------------
# a1 score
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d,Nk,lens", [
    ("bf16", 128, 256, [0, 1, 255, 256, 257, 1500, 31, 700]),
    ("bf16", 64, 100, [5, 30, 462, 202, 0, 91, 255, 256]),
    ("bf16", 128, 9, [21, 57, 0, 4, 1000, 250, 256, 3]),        # N_k < 32: every query observes
    ("f32", 64, 100, [5, 30, 462, 202, 0, 91, 255, 256]),
])
def test_score_matches_oracle(dtype, d, Nk, lens):
    u = _u()
    rng = np.random.default_rng(11 + Nk + d)
    H, B = 4, 2
    U = H * B
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=U, max_cache_len=2048, max_queries=256)
    scale = float(np.float32(1.0 / np.sqrt(d)))
    rows = [(u.rand_values(rng, (n, d), dtype), u.rand_values(rng, (n, d), dtype)) for n in lens]
    cin, _ = u.build_cache(rows, d, dtype, pad_rows=2, fill=100.0)      # poison between units
    q = u.rand_values(rng, (B, H, Nk, d), dtype) * 2.0
    k_new = u.rand_values(rng, (B, H, Nk, d), dtype)
    if dtype == "bf16":
        q = wl.bf16_to_f32(wl.bf16_round(q))
    stride = 2048
    imp = torch.full((U, stride), -1.0, device=u.DEV)
    hk.score(torch.from_numpy(q).to(hk.torch_dtype).to(u.DEV), cin, scale, imp, k_new=u.to_dev(k_new, dtype))
    torch.cuda.synchronize()
    got = imp.cpu().numpy().astype(np.float64)
    obs = ho.observation_rows(Nk, 32)
    worst = 0.0
    for uu in range(U):
        b, h = divmod(uu, H)
        K_in = np.concatenate([rows[uu][0], k_new[b, h]]).astype(np.float64)
        want = ho.importance(q[b, h][obs].astype(np.float64), K_in, scale)
        T = K_in.shape[0]
        rel = np.abs(got[uu, :T] - want) / want
        worst = max(worst, rel.max())
        assert np.all(got[uu, T:] == -1.0)
        assert abs(got[uu, :T].sum() - len(obs)) < 1e-4 * len(obs)
    assert worst < (2e-7 if dtype == "f32" else 1e-6), worst
    hk.close()


@pytest.mark.parametrize("d,H,Nk,lens,n_obs,gain", [
    (64, 4, 32, [0, 31, 32, 33], 32, 1.0),                  # exactly one chunk of 64 keys, one less, one more
    (128, 4, 16, [0, 1, 47, 240], 16, 1.0),                 # one tile of 16 keys; half of the observation rows unused
    (64, 2, 9, [3, 1000], 5, 60.0),                         # logits of thousands: only the maximum of a row is left
    (64, 44, 40, [900 + i for i in range(44)], 32, 1.0),    # more than 640 chunks of 64 keys: chunks of 256
    (128, 44, 40, [730 + i for i in range(44)], 7, 1.0),    # ... the last chunk of 256 begins at 768
])
def test_f32_score_chunk_edges(d, H, Nk, lens, n_obs, gain):
    """Logits are fp64 dot products (error ~1e-16 of their terms); 2^x of the reduced argument carries about one float32
    ulp (1.2e-7) per term, the stored importance half another one: 2e-7 relative, plus 1e-13 of a logit in absolute terms."""
    u = _u()
    rng = np.random.default_rng(d + H + Nk)
    hk = u.make_hack(heads=H, head_dim=d, dtype="f32", max_units=H, max_cache_len=1100, max_queries=Nk)
    scale = float(np.float32(gain / np.sqrt(d)))
    rows = [(u.rand_values(rng, (n, d), "f32"),) * 2 for n in lens]
    cin, _ = u.build_cache(rows, d, "f32", pad_rows=2, fill=np.nan)
    q, k_new = u.rand_values(rng, (1, H, Nk, d), "f32"), u.rand_values(rng, (1, H, Nk, d), "f32")
    imp = torch.full((H, 1100), -1.0, device=u.DEV)
    hk.score(u.to_dev(q, "f32"), cin, scale, imp, k_new=u.to_dev(k_new, "f32"), n_obs=n_obs)
    torch.cuda.synchronize()
    got = imp.cpu().numpy().astype(np.float64)
    obs = [(i * Nk) // n_obs for i in range(n_obs)]
    for h in range(H):
        K = np.concatenate([rows[h][0], k_new[0, h]]).astype(np.float64)
        want = ho.importance(q[0, h][obs].astype(np.float64), K, scale)
        assert np.all(np.abs(got[h, :len(K)] - want) <= 2e-7 * want + 1e-30 + (gain > 1) * 1e-10 * want)
        assert np.all(got[h, len(K):] == -1.0)
    hk.close()


def test_score_many_units_split_into_launch_groups_and_repeated_calls():
    """More score work items than the device holds at once: the library must cut
    the launch into groups of whole units.  Calling twice on the same context
    also checks that the normaliser workspace is left clean."""
    u = _u()
    rng = np.random.default_rng(5)
    H, B, d, Nk, dtype = 16, 6, 128, 32, "bf16"
    U = H * B
    lens = [int(x) for x in rng.integers(3900, 4200, U)]
    lens[7], lens[50] = 1, 130                                         # short units among long ones
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=U, max_cache_len=4352, max_queries=Nk)
    scale = float(np.float32(1.0 / np.sqrt(d)))
    rows = [(u.rand_values(rng, (n, d), dtype), None) for n in lens]
    rows = [(k, k) for k, _ in rows]
    cin, _ = u.build_cache(rows, d, dtype)
    q = u.rand_values(rng, (B, H, Nk, d), dtype) * 2.0
    k_new = u.rand_values(rng, (B, H, Nk, d), dtype)
    stride = 4352
    obs = ho.observation_rows(Nk, 32)
    qd, kd = u.to_dev(q, dtype), u.to_dev(k_new, dtype)
    for rep in range(2):
        imp = torch.full((U, stride), -1.0, device=u.DEV)
        hk.score(qd, cin, scale, imp, k_new=kd)
        torch.cuda.synchronize()
        got = imp.cpu().numpy().astype(np.float64)
        T_all = np.array(lens) + Nk
        sums = np.array([got[uu, :T_all[uu]].sum() for uu in range(U)])
        assert np.all(np.abs(sums - len(obs)) < 1e-4 * len(obs)), (rep, sums.min(), sums.max())
        for uu in (0, 7, 50, 51, U // 2, U - 1):
            b, h = divmod(uu, H)
            K_in = np.concatenate([rows[uu][0], k_new[b, h]]).astype(np.float64)
            want = ho.importance(q[b, h][obs].astype(np.float64), K_in, scale)
            assert float(np.max(np.abs(got[uu, :len(want)] - want) / want)) < 1e-6, (rep, uu)
            assert np.all(got[uu, len(want):] == -1.0)
    hk.close()


@pytest.mark.parametrize("d,longest,keys", [(128, 2400, 96), (128, 4800, 192), (64, 5000, 96), (64, 5500, 192), (64, 7000, 256)])
def test_score_items_of_three_and_six_tiles(d, longest, keys):
    """Item sizes between the powers of two, chosen where smaller items do not fit one launch (the last case: 256 keys where 192 would put a
    third work-group on a compute unit): units that end on and around item, tile and work-group boundaries, in one launch, in two
    passes and with fixed scratch (the same bits), against float64."""
    u = _u()
    H, Nk = 64, 40
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + longest)
    t_in = np.full(H, longest, np.int32)
    ends = [41, 95, 96, 97, 191, 192, 193, 383, 384, 385, 767, 768, 769]
    for i, t in enumerate(ends):
        t_in[5 + i] = max(t, Nk + 1)
    t_in[30:40] = longest - np.arange(10) * 11
    lens = (t_in - Nk).astype(np.int32)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    q, kn = (torch.randn((1, H, Nk, d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    K = torch.randn((int(off[-1]), d), generator=gen, device=u.DEV).bfloat16()
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=longest, max_queries=Nk)
    assert hk.score_item_keys(t_in) == keys                    # the size that is under test
    src = Cache(K, K, off[:-1], lens)
    stride = (longest + 63) // 64 * 64
    imps = []
    for form in ("fused", "fused", "two-pass", "static"):
        imp = torch.full((H, stride), -1.0, device=u.DEV)
        if form == "two-pass":
            hk.set_score_mode(1)
        (hk.score_static if form == "static" else hk.score)(q, src, scale, imp, k_new=kn)
        torch.cuda.synchronize()
        imps.append(imp)
    assert all(torch.equal(imps[0], x) for x in imps[1:])
    rows = [i * Nk // 32 for i in range(32)]
    for x in list(range(5, 5 + len(ends))) + [0, 30, 39, 63]:
        k = torch.cat([K[off[x]:off[x] + lens[x]], kn[0, x]]).double()
        want = torch.softmax(scale * (q[0, x, rows].double() @ k.T.contiguous()), -1).sum(0)
        assert float(((imps[0][x, :t_in[x]].double() - want) / want).abs().max()) < 1e-6, (x, int(t_in[x]))   # the bar of the entry point
        assert bool((imps[0][x, t_in[x]:] == -1).all())
    hk.check()
    hk.close()


def test_score_extreme_logits_bf16():
    """Logits of a few hundred nats: the row normalisers live in fp64, so peaked
    rows must still follow the fp64 oracle over 100+ orders of magnitude (entries
    that underflow float32 are compared absolutely; the relative bar is the one
    the arithmetic supports at this logit magnitude, not the 1e-6 of ordinary data).  Beyond +-354 nats the parked logits are clamped: the
    library must say so instead of returning a silently different answer."""
    u = _u()
    rng = np.random.default_rng(21)
    H, B, d, Nk, dtype = 2, 1, 128, 40, "bf16"
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=2, max_cache_len=1024, max_queries=Nk)
    rows = [(u.rand_values(rng, (n, d), dtype) * 4.0, u.rand_values(rng, (n, d), dtype)) for n in (700, 333)]
    cin, _ = u.build_cache(rows, d, dtype)
    q = wl.bf16_to_f32(wl.bf16_round(u.rand_values(rng, (B, H, Nk, d), dtype) * 4.0))
    k_new = u.rand_values(rng, (B, H, Nk, d), dtype) * 4.0
    obs = ho.observation_rows(Nk, 32)
    qd, kd = torch.from_numpy(q).to(hk.torch_dtype).to(u.DEV), u.to_dev(k_new, dtype)
    peak = max(float(np.abs(q[0, uu][obs].astype(np.float64) @ np.concatenate([rows[uu][0], k_new[0, uu]]).T.astype(np.float64)).max())
               for uu in range(2))
    scale = float(np.float32(300.0 / peak))                            # largest |logit| = 300 nats
    imp = torch.full((2, 1024), -1.0, device=u.DEV)
    hk.score(qd, cin, scale, imp, k_new=kd)
    torch.cuda.synchronize()
    hk.check()
    got = imp.cpu().numpy().astype(np.float64)
    for uu in range(2):
        K_in = np.concatenate([rows[uu][0], k_new[0, uu]]).astype(np.float64)
        want = ho.importance(q[0, uu][obs].astype(np.float64), K_in, scale)
        err = np.abs(got[uu, :len(want)] - want)
        # float32 slices of a dot product of magnitude 300 / scale carry ~2.5e-8 * |logit| of absolute
        # error into the logit, i.e. that much relative error into exp(logit): 1e-5 at 300 nats
        assert np.all(err <= 1e-5 * want + 1e-37), (uu, float((err / np.maximum(want, 1e-300)).max()))
        assert abs(got[uu, :len(want)].sum() - len(obs)) < 1e-4 * len(obs)
    # 500 nats: outside the supported range -> reported once, context stays usable
    hk.score(qd, cin, float(np.float32(500.0 / peak)), imp, k_new=kd)
    torch.cuda.synchronize()
    with pytest.raises(HackError) as ei:
        hk.check()
    assert ei.value.status == -3
    hk.check()
    hk.score(qd, cin, scale, imp, k_new=kd)
    torch.cuda.synchronize()
    hk.check()
    hk.close()


def test_score_cache_only_custom_rows_and_inactive_units():
    u = _u()
    rng = np.random.default_rng(3)
    H, B, d, Nk, dtype = 2, 1, 128, 64, "bf16"
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=2, max_cache_len=1024, max_queries=64)
    rows = [(u.rand_values(rng, (n, d), dtype), u.rand_values(rng, (n, d), dtype)) for n in (513, 40)]
    cin, _ = u.build_cache(rows, d, dtype)
    q = u.rand_values(rng, (B, H, Nk, d), dtype)
    q_idx = np.array([63, 0, 5, 5, 17], np.int32)                     # arbitrary rows, repeats allowed
    imp = torch.full((2, 1024), -1.0, device=u.DEV)
    hk.score(u.to_dev(q, dtype), cin, 0.11, imp, q_idx=q_idx, n_obs=5, active=[1, 0])
    torch.cuda.synchronize()
    got = imp.cpu().numpy().astype(np.float64)
    want = ho.importance(q[0, 0][q_idx].astype(np.float64), rows[0][0].astype(np.float64), float(np.float32(0.11)))
    assert float(np.max(np.abs(got[0, :513] - want) / want)) < 1e-6
    assert np.all(got[1] == -1.0)                                     # inactive unit untouched
    with pytest.raises(HackError):
        hk.score(u.to_dev(q, dtype), cin, 0.11, imp, q_idx=[64], n_obs=1)
    with pytest.raises(HackError):
        hk.score(u.to_dev(q, dtype), cin, -1.0, imp)
    hk.close()


# ---------------------------------------------------------------------------
# a4 attention
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d,Nk,lens,tol,kernel", [
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, "tile128"),
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, "split"),
    ("bf16", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 2e-2, "tile128"),
    ("bf16", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 2e-2, "split"),
    ("bf16", 128, 1, [1, 5, 21, 57, 121, 265, 64, 32], 2e-2, "tile128"),
    ("bf16", 128, 1, [1, 5, 21, 57, 121, 265, 64, 32], 2e-2, "split"),
    ("bf16", 64, 33, [3, 31, 32, 96, 97, 160, 2000, 129], 2e-2, "split"),
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, None),
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, "tile128_plain"),
    ("bf16", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 2e-2, "tile128_plain"),
    ("bf16", 128, 130, [96, 97, 192, 193, 224, 225, 256, 289], 2e-2, "tile128"),      # 3 .. 10 key blocks: every
    ("bf16", 64, 130, [96, 97, 192, 193, 224, 225, 256, 289], 2e-2, "tile128"),       # way in and out of the steady loop
    ("bf16", 128, 130, [320, 321, 351, 352, 353, 384, 416, 449], 2e-2, "tile128"),
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, "stream"),           # work items cut into segments,
    ("bf16", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 2e-2, "stream"),          # partial results added up by the
    ("bf16", 128, 130, [96, 97, 192, 193, 224, 225, 256, 289], 2e-2, "stream"),       # work-group that finishes last
    ("bf16", 64, 130, [320, 321, 351, 352, 353, 384, 416, 449], 2e-2, "stream"),
    ("bf16", 128, 1, [1, 5, 21, 57, 121, 265, 64, 32], 2e-2, "stream"),
    ("bf16", 128, 300, [1, 2, 63, 64, 65, 1943, 127, 700], 2e-2, "cut"),              # whole work items, the longest halved
    ("bf16", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 2e-2, "cut"),
    ("bf16", 128, 130, [320, 321, 351, 352, 1353, 384, 416, 2047], 2e-2, "cut"),
    ("f32", 64, 100, [102, 306, 1, 33, 562, 91, 128, 129], 1e-4, None),
    ("f32", 128, 70, [1, 2, 63, 64, 65, 300, 127, 31], 1e-4, None),
])
def test_attention_matches_oracle(dtype, d, Nk, lens, tol, kernel):
    """Both bf16 attention kernels (128-query tiles; 32-query items with the keys split
    over the waves) on the same ragged shapes: fewer keys than waves, one key, block
    boundaries +-1, many blocks per wave, a last query tile with a single query."""
    u = _u()
    rng = np.random.default_rng(17 + Nk + d)
    H, B = 4, 2
    U = H * B
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=U, max_cache_len=2048, max_queries=512,
                     attention=kernel)
    scale = float(np.float32(1.0 / np.sqrt(d)))
    rows = [(u.rand_values(rng, (n, d), dtype) * 1.5, u.rand_values(rng, (n, d), dtype)) for n in lens]
    if dtype == "bf16":
        rows = [(wl.bf16_to_f32(wl.bf16_round(k)), v) for k, v in rows]
    cache, _ = u.build_cache(rows, d, dtype, pad_rows=1, fill=50.0)
    q = u.rand_values(rng, (B, H, Nk, d), dtype)
    # twice with different queries: the second launch reuses whatever scratch the first one left
    for rep in range(2):
        out = torch.full((B, H, Nk, d), 7.0, dtype=hk.torch_dtype, device=u.DEV)
        hk.attn(u.to_dev(q, dtype), cache, scale, out)
        torch.cuda.synchronize()
        got = u.from_dev(out)
        for uu in range(U):
            b, h = divmod(uu, H)
            want = ho.attention(q[b, h].astype(np.float64), rows[uu][0].astype(np.float64),
                                rows[uu][1].astype(np.float64), scale)
            err = np.abs(got[b, h] - want).max()
            assert err < tol, (rep, uu, lens[uu], err)
        q = u.rand_values(rng, (B, H, Nk, d), dtype)
    hk.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Nk,lens", [
    (5, 1, [1, 2, 16, 17, 127]),            # one query; block edges; fewer blocks than waves
    (5, 17, [15, 31, 128, 129, 300]),       # ragged query tile; wave-split edges
    (3, 48, [257, 33, 640]),
    (26, 250, [1 + 13 * i for i in range(26)]),   # more than 384 tiles of 16 queries: the 32-query form, ragged tiles
])
def test_f32_attention_tile_edges(d, H, Nk, lens):
    """Float32 sums of at most 640 terms and one exponential each: within 2e-5 of the fp64 result (outputs are
    averages of values of unit variance; the observed worst is 4e-6)."""
    u = _u()
    rng = np.random.default_rng(5 * d + Nk)
    hk = u.make_hack(heads=H, head_dim=d, dtype="f32", max_units=H, max_cache_len=640, max_queries=Nk)
    q = u.rand_values(rng, (1, H, Nk, d), "f32")
    rows = [(u.rand_values(rng, (n, d), "f32"), u.rand_values(rng, (n, d), "f32")) for n in lens]
    cache, _ = u.build_cache(rows, d, "f32", pad_rows=3, fill=np.nan)   # rows of nobody must not be read into a result
    out = torch.full((1, H, Nk, d), float("nan"), device=u.DEV)
    scale = float(np.float32(1.0 / np.sqrt(d)))
    hk.attn(u.to_dev(q, "f32"), cache, scale, out)
    torch.cuda.synchronize()
    got = u.from_dev(out)[0]
    for h in range(H):
        K, V = (x.astype(np.float64) for x in rows[h])
        s = q[0, h].astype(np.float64) @ K.T * scale
        p = np.exp(s - s.max(1, keepdims=True))
        assert np.abs(got[h] - (p / p.sum(1, keepdims=True)) @ V).max() < 2e-5
    hk.close()


@pytest.mark.parametrize("d", [64, 128])
def test_f32_step_appends_in_the_attention_launch(d):
    """Steps that do not compress: cached rows and position ids are exactly the concatenation, outputs those of hack_attn."""
    u = _u()
    rng = np.random.default_rng(d)
    H = 3
    hk = u.make_hack(heads=H, head_dim=d, dtype="f32", max_units=H, max_cache_len=512, max_queries=196)
    mc = hk.managed_cache([300] * H)
    want_k, want_v = [], []
    for n in (1, 4, 37, 196):
        q, k, v = (torch.from_numpy(u.rand_values(rng, (1, H, n, d), "f32")).to(u.DEV) for _ in range(3))
        out, ref = torch.empty_like(q), torch.empty_like(q)
        hk.step(mc, q, k, v, np.zeros(H, np.uint8), [1 << 30] * H, 5, 0.1, out)
        hk.attn(q, mc.as_cache(), 0.1, ref)
        want_k.append(k[0])
        want_v.append(v[0])
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    off, ln = mc.view()
    K, V = torch.cat(want_k, 1), torch.cat(want_v, 1)
    for h in range(H):
        assert torch.equal(mc.k[off[h]:off[h] + ln[h]], K[h]) and torch.equal(mc.v[off[h]:off[h] + ln[h]], V[h])
        assert torch.equal(mc.pos[off[h]:off[h] + ln[h]].cpu(), torch.arange(238, dtype=torch.int32))
    mc.close()
    hk.close()


def test_cut_and_streamed_attention_launches_agree_with_whole_work_items():
    """Random unit counts, cache lengths and query counts: the 128-query kernel with every cut the pair
    model likes, and in its streamed form (equal runs of key blocks), against the same kernel on whole
    work items.  The partial results of a cut work item are added up in float32, so the outputs agree to
    a bf16 rounding of the output; each form runs many times on its context (every launch meets the
    counters and partial-result slots the one before it left)."""
    u = _u()
    rng = np.random.default_rng(2024)
    for case in range(8):
        d = int(rng.choice([64, 128]))
        H, B = int(rng.integers(1, 9)), int(rng.integers(1, 6))
        U = H * B
        Nk = int(rng.integers(1, 900))
        lens = rng.integers(1, int(rng.choice([64, 700, 6000])) + 1, size=U).astype(np.int32)
        off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)])[:-1].astype(np.int64)
        rows = int(((lens + 7) // 8 * 8).sum())
        K = (torch.randn((rows, d), device=u.DEV) * 1.5).to(torch.bfloat16)
        V = torch.randn((rows, d), device=u.DEV).to(torch.bfloat16)
        q = torch.randn((B, H, Nk, d), device=u.DEV).to(torch.bfloat16)
        # Many launches back to back, alternating between two sets of queries: a part that was read before its
        # writer's stores had arrived would be the other query set's, far outside the tolerance.
        q2 = torch.randn((B, H, Nk, d), device=u.DEV).to(torch.bfloat16)
        outs = {}
        for kernel in ("tile128", "cut", "stream"):
            hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=U, max_cache_len=6000, max_queries=900,
                             attention=kernel)
            o, o2 = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
            first = None
            for it in range(1 if kernel == "tile128" else 24):
                hk.attn(q, Cache(K, V, off, lens), float(1.0 / np.sqrt(d)), o)
                hk.attn(q2, Cache(K, V, off, lens), float(1.0 / np.sqrt(d)), o2)
                if first is None:
                    first = (o.clone(), o2.clone())
                else:      # the parts are added up in a fixed order: every launch gives the same bits
                    assert torch.equal(o, first[0]) and torch.equal(o2, first[1]), (case, kernel, it)
                o.fill_(7.0)
                o2.fill_(7.0)
            o, o2 = first
            torch.cuda.synchronize()
            outs[kernel] = (o.float().cpu().numpy(), o2.float().cpu().numpy())
            hk.close()
        for kernel in ("cut", "stream"):
            for which in (0, 1):
                assert np.isfinite(outs[kernel][which]).all(), (case, kernel)
                err = float(np.abs(outs[kernel][which] - outs["tile128"][which]).max())
                assert err < 2e-2, (case, kernel, which, d, U, Nk, int(lens.max()), err)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Nk,lens", [
    (3, 33, [1, 32, 33]), (3, 5, [640, 640, 31]), (4, 40, [641, 1, 32, 2049]), (2, 100, [672, 700]), (3, 64, [1, 897, 4001]),
    (65, 128, [641] * 65), (64, 128, [641] * 63 + [7]),     # 260 and 256 work items, the line between four and eight waves
    (48, 128, [641] * 47 + [7]), (32, 224, [1025] * 31 + [9]), (32, 224, [1024] * 32),   # ... and at head_dim 128: 240 and 256 items + units
])
def test_key_split_attention_block_and_wave_edges(d, H, Nk, lens):
    """Key-split work items of one block, of fewer and of more blocks than waves, with four and with eight waves."""
    u = _u()
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + len(lens))
    lens = np.asarray(lens, np.int32)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    q = torch.randn((1, H, Nk, d), generator=gen, device=u.DEV).bfloat16()
    K, V = (torch.randn((int(off[-1]), d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=int(lens.max()), max_queries=Nk, attention="split")
    out = torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, off[:-1], lens), scale, out)
    torch.cuda.synchronize()
    for h in range(H):
        k, v = (x[off[h]:off[h] + lens[h]].double() for x in (K, V))
        want = torch.softmax(scale * (q[0, h].double() @ k.T.contiguous()), -1) @ v
        # P and O are rounded to bf16: 2^-8 of the largest value each
        assert float((out[0, h].double() - want).abs().max()) < 2e-2, (h, int(lens[h]))
    hk.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("U,Nk,lens", [
    (7, 15, [1, 32, 64, 33, 128, 129, 300]), (5, 16, [32, 31, 96, 160, 17]), (5, 17, [32, 1, 128, 255, 64]), (5, 31, [32, 63, 65, 127, 256]),
    (3, 48, [32, 700, 1]), (9, 33, [700] * 8 + [32]),
    (192, 17, [32, 200, 3]), (193, 17, [32, 129, 64]),      # 192 and 200 work items (dealt to eight XCDs): the lines between 16 and 32 queries,
    (384, 16, [32, 45, 97]), (385, 16, [32, 128, 20]),      # 384 and 392,
    (64, 32, [641, 32, 900]), (65, 20, [641, 32, 64]),      # 64 and 72 and
    (128, 31, [641, 32, 64]), (129, 32, [641, 5, 256]),     # 128 and 136 with eight waves
])
def test_key_split_attention_with_16_and_32_queries_a_work_group(d, U, Nk, lens):
    """Single blocks (exactly full ones among them), rows of queries on either side of 16 and 32, and work items on both sides of the lines at
    which a work-group takes half of one: attention, a step that appends (its last Nk rows are new) and one that compresses give the same bits,
    within the rounding of the probabilities and the output to bf16."""
    u = _u()
    gen = torch.Generator(u.DEV)
    gen.manual_seed(U + Nk)
    lens = np.resize(np.asarray(lens, np.int32), U)
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=U, head_dim=d, dtype="bf16", max_units=U, max_cache_len=int(lens.max()) + Nk, max_queries=max(Nk, int(lens.max())), attention="split")
    q, kn, vn = (torch.randn((1, U, Nk, d), generator=gen, device=u.DEV).bfloat16() for _ in range(3))

    def check(out, cache, what):
        off, ln = cache.view()
        for x in list(range(min(U, 12))) + [U - 1]:
            k, v = (t[off[x]:off[x] + ln[x]].double() for t in (cache.k, cache.v))
            p = torch.softmax(scale * (q[0, x].double() @ k.T.contiguous()), -1)
            # every probability, their sum and the output carry 2^-9 each; float32 scores and sums are far below
            bound = 3 * 2.0 ** -9 * (p @ v.abs()) * 1.02 + 1e-4
            assert bool(((out[0, x].double() - p @ v).abs() <= bound).all()), (what, x, int(ln[x]))

    types, never = np.zeros(U, np.uint8), np.full(U, 10**6, np.int32)
    # rows in front of the steps: one step for all units, compressed to their lengths
    first = max(int(lens.max()), 2)
    k0, v0 = (torch.randn((1, U, first, d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    mc = hk.managed_cache(np.maximum(np.maximum(lens, 2) + Nk, first))
    hk.step(mc, k0, k0, v0, types, np.where(lens < first, lens, 10**6).astype(np.int32), 5, scale, torch.empty_like(k0))
    assert list(mc.view()[1]) == list(lens)
    out, want = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    hk.attn(q, mc.as_cache(), scale, out)
    torch.cuda.synchronize()
    check(out, mc, "attention")
    for what, budget in (("compressing", np.maximum(lens, 2)), ("appending", never)):
        hk.step(mc, q, kn, vn, types, budget, 5, scale, out)
        hk.attn(q, mc.as_cache(), scale, want)
        torch.cuda.synchronize()
        assert torch.equal(out, want), what
        check(out, mc, what)
    hk.check()
    mc.close()
    hk.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("waves,queries", [(4, 16), (4, 32), (8, 16), (8, 32)])
def test_key_split_attention_moving_reference_and_minus_infinity(d, waves, queries):
    """Scores that rise and fall by 20 bits with every block of every wave, and first, last and all but one of the blocks at -inf, in
    work-groups of four and eight waves and of 16 and 32 queries."""
    u = _u()
    U = {(4, 16): 12, (4, 32): 200 if d == 128 else 392, (8, 16): 12, (8, 32): 100 if d == 128 else 136}[waves, queries]
    Nk, longest = 20, 32 * waves * 5
    kinds = ["grows", "shrinks", "no start", "one key", "no end"]
    some = [longest, longest - 1, longest - 31, 32 * waves * 2 + 1, 32 * waves + 33, 32 * waves]
    lens = np.array([some[i // 5 % 6] for i in range(U)], np.int32)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + waves + queries)
    q = torch.randn((1, U, Nk, d), generator=gen, device=u.DEV)
    q[..., 0] = 4.0
    q = q.bfloat16()
    scale = float(np.float32(d ** -0.5))
    K, V = (torch.zeros((int(off[-1]), d), dtype=torch.bfloat16, device=u.DEV) for _ in range(2))
    for h in range(U):
        k, v = (torch.randn((int(lens[h]), d), generator=gen, device=u.DEV) for _ in range(2))
        K[off[h]:off[h] + lens[h]], V[off[h]:off[h] + lens[h]] = u.walked_keys(k, v, waves, kinds[h % 5], scale)
    hk = u.make_hack(heads=U, head_dim=d, dtype="bf16", max_units=U, max_cache_len=longest, max_queries=Nk, attention="split")
    out = torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, off[:-1], lens), scale, out)
    torch.cuda.synchronize()
    moves = 0
    for h in range(min(U, 60)):
        k, v = (x[off[h]:off[h] + lens[h]].double() for x in (K, V))
        logits = scale * (q[0, h].double() @ k.T.contiguous())
        if h % 5 == 0:
            got = u.reference_moves(logits, waves)
            assert got == (int(lens[h]) + 31) // 32 - waves, (h, got)      # in every block but the first ones
            moves += got
        p = torch.softmax(logits, -1)
        # every probability, their sum and the output carry 2^-9 each; float32 scores (of up to 42 nats) and sums are far below
        bound = 3 * 2.0 ** -9 * (p @ v.abs()) * 1.02 + 1e-4
        assert bool(((out[0, h].double() - p @ v).abs() <= bound).all()), (h, kinds[h % 5], int(lens[h]))
    assert moves > 0
    hk.check()
    hk.close()


@pytest.mark.parametrize("d,T,waves", [(64, 640, 4), (128, 600, 4), (64, 1504, 8), (128, 1304, 8)])
def test_key_split_attention_rounds_no_coarser_than_its_probabilities(d, T, waves):
    """The error against float64 is that of probabilities rounded to bf16 in units of the largest score so far, each wave's largest one exactly.
    (Rounded in units of the first block's scores, probabilities just below the largest lose up to a bit: 1.08 to 1.2 times the error.)"""
    u = _u()
    U, Nk = 8, 64
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + T)
    q = (2 * torch.randn((1, U, Nk, d), generator=gen, device=u.DEV)).bfloat16()
    K, V = (torch.randn((U * T, d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=U, head_dim=d, dtype="bf16", max_units=U, max_cache_len=T, max_queries=Nk, attention="split")
    out = torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, np.arange(U, dtype=np.int64) * T, np.full(U, T, np.int32)), scale, out)
    torch.cuda.synchronize()
    off, as_rounded = 0.0, 0.0
    for h in range(U):
        k, v = K[h * T:(h + 1) * T], V[h * T:(h + 1) * T]
        want = torch.softmax(scale * (q[0, h].double() @ k.double().T.contiguous()), -1) @ v.double()
        off += float((out[0, h].double() - want).square().sum())
        as_rounded += float((u.attention_with_rounded_probabilities(q[0, h], k, v, scale, waves).double() - want).square().sum())
    assert off ** 0.5 < 1.02 * as_rounded ** 0.5       # the same roundings; float32 scores and sums are 2^-15 of them
    hk.close()


# the forms of the 128-query kernel (halves: head_dim 128)
TILE_FORMS = [(d, n, f) for d, n in ((64, 130), (128, 33), (128, 257)) for f in ("tile128", "stream", "halves") if d == 128 or f != "halves"]


@pytest.mark.parametrize("d,Nk,form", TILE_FORMS)
def test_tile_attention_block_edges_and_moving_reference(d, Nk, form):
    """One to ten key blocks, full and ragged, in the 128-query kernel, with keys of one size, and with keys that grow from block to block in
    the order in which a work item or a half walks them, by more than its reference leaves room for: every query moves it in every stage."""
    u = _u()
    lens = [1, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 288, 289, 320]
    lens = np.array([n for n in lens if n > 32 or form != "halves"], np.int32)   # either half needs a block
    H = len(lens)
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + Nk)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    q = torch.randn((1, H, Nk, d), generator=gen, device=u.DEV)
    q[..., 0] = 4.0
    q = q.bfloat16()
    K, V = (torch.randn((int(off[-1]), d), generator=gen, device=u.DEV) for _ in range(2))
    scale = float(np.float32(d ** -0.5))
    grown = K.clone()
    walks = []   # per unit: the blocks of a whole item (last one first), or those of either half
    for h in range(H):
        nb = (int(lens[h]) + 31) // 32
        parts = [(0, (nb + 1) // 2), ((nb + 1) // 2, nb)] if form == "halves" else [(0, nb)]
        walks.append([[hi - 1] + list(range(lo, hi - 1)) for lo, hi in parts])
        for walk in walks[h]:
            for step, b in enumerate(walk):
                rows = slice(int(off[h]) + 32 * b, int(off[h]) + min(32 * b + 32, int(lens[h])))
                grown[rows] *= 0.25
                grown[rows, 0] = (step - 5) * 18 / (4.0 * scale)    # 18 nats a block, 26 of the 16 bits that the reference leaves
    hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=int(lens.max()), max_queries=Nk, attention=form)
    V = V.bfloat16()
    for K, grows in ((K.bfloat16(), False), (grown.bfloat16(), form != "stream")):   # (a stream's segments start where its cuts fall)
        out = torch.full_like(q, 7.0)
        hk.attn(q, Cache(K, V, off[:-1], lens), scale, out)
        torch.cuda.synchronize()
        for h in range(H):
            k, v = (x[off[h]:off[h] + lens[h]].double() for x in (K, V))
            logits = scale * (q[0, h].double() @ k.T.contiguous())
            for walk in walks[h] if grows else []:
                tops = torch.stack([logits[:, 32 * b:32 * b + 32].amax(1) for b in walk])
                assert len(walk) < 2 or float((tops[1:] - tops[:-1]).min()) > 12, h    # 16 bits are 11.1 nats
            want = torch.softmax(logits, -1) @ v
            # P and O are rounded to bf16: 2^-8 of the largest value each, |V| up to 4.5
            assert float((out[0, h].double() - want).abs().max()) < 4e-2, (h, int(lens[h]))
    hk.close()


@pytest.mark.parametrize("d,Nk,form", TILE_FORMS)
def test_tile_attention_where_whole_blocks_score_minus_infinity(d, Nk, form):
    """Keys that score -inf for every query fill the block that a work item, a segment or a half begins with: what is left decides."""
    u = _u()
    lens = np.array([33, 65, 129, 289, 64, 320, 77, 160, 225, 288], np.int32)
    H = len(lens)
    gen = torch.Generator(u.DEV)
    gen.manual_seed(d + Nk)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    q = torch.randn((1, H, Nk, d), generator=gen, device=u.DEV)
    q[..., 0] = q[..., 0].abs() + 0.1
    q = q.bfloat16()
    K, V = (torch.randn((int(off[-1]), d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    for h in range(H):
        n, k = int(lens[h]), K[off[h]:off[h] + lens[h]]
        if h < 6:
            k[(n - 1) // 32 * 32:, 0] = -torch.inf    # the last block, of one key, full
        elif h == 6:
            k[torch.arange(n, device=u.DEV) != 40, 0] = -torch.inf
        elif h == 7:
            k[:96, 0] = -torch.inf                    # the first of its halves
        else:
            k[32:, 0] = -torch.inf
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=int(lens.max()), max_queries=Nk, attention=form)
    out = torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, off[:-1], lens), scale, out)
    torch.cuda.synchronize()
    for h in range(H):
        k, v = (x[off[h]:off[h] + lens[h]].double() for x in (K, V))
        want = torch.softmax(scale * (q[0, h].double() @ k.T.contiguous()), -1) @ v
        # P and O are rounded to bf16: 2^-8 of the largest value each, |V| up to 4.5
        assert float((out[0, h].double() - want).abs().max()) < 4e-2, (h, int(lens[h]))   # (a NaN is not)
    hk.close()


@pytest.mark.parametrize("form", ["tile128", "tile128_plain"])
@pytest.mark.parametrize("d", [64, 128])
def test_tile_attention_over_more_rows_than_32_bits_of_bytes(d, form):
    """A unit whose keys take more than 4 GiB: the one key that matters lies behind them, in a block that is not the last one."""
    u = _u()
    line = 2**32 // (2 * d)
    n, at = line + 100, line + 40
    K, V = (torch.zeros((n + 4, d), dtype=torch.bfloat16, device=u.DEV) for _ in range(2))
    K[at] = 8.0     # 8 sqrt(d) = 64 nats and more above all other keys, of which there are e^17
    V[at] = torch.arange(d, device=u.DEV).bfloat16()
    q = torch.ones((1, 1, 1, d), dtype=torch.bfloat16, device=u.DEV)
    hk = u.make_hack(heads=1, head_dim=d, dtype="bf16", max_units=1, max_cache_len=64, max_queries=1, attention=form)
    out = torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, np.zeros(1, np.int64), np.array([n], np.int32)), float(np.float32(d ** -0.5)), out)
    torch.cuda.synchronize()
    assert torch.equal(out[0, 0, 0], V[at])
    hk.close()


@pytest.mark.parametrize("forced,H,Nk,lens", [
    (True, 3, 1, [33, 64, 65]), (True, 4, 127, [96, 97, 128, 129]), (True, 3, 128, [160, 191, 193]), (True, 5, 129, [224, 225, 256, 321, 1000]),
    (False, 20, 832, [865] * 10 + [897, 900] * 5),       # 140 work items of 128 queries: halves by the library's own rule
    (False, 20, 832, [864] + [40] * 19),                 # one block short of it
])
def test_attention_with_the_keys_in_two_halves(forced, H, Nk, lens, monkeypatch):
    """Odd and even numbers of blocks, halves of a single ragged block, steady loops entered by neither, one or both halves."""
    u = _u()
    if forced:
        monkeypatch.setenv("HACK_ATTN_PIPE", "2")
        monkeypatch.setenv("HACK_ATTN_SPLIT_ITEMS", "0")
    d = 128
    gen = torch.Generator(u.DEV)
    gen.manual_seed(Nk + len(lens))
    lens = np.asarray(lens, np.int32)
    off = np.concatenate([[0], np.cumsum((lens + 7) // 8 * 8)]).astype(np.int64)
    q = torch.randn((1, H, Nk, d), generator=gen, device=u.DEV).bfloat16()
    K, V = (torch.randn((int(off[-1]), d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    K[off[0]:off[0] + 16] *= 12      # the halves' references lie far apart
    scale = float(np.float32(d ** -0.5))
    hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=int(lens.max()), max_queries=Nk)
    assert hk.attn_variant(1, Nk) == 0
    out, again = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    hk.attn(q, Cache(K, V, off[:-1], lens), scale, out)
    hk.attn(q, Cache(K, V, off[:-1], lens), scale, again)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    for h in range(H):
        k, v = (x[off[h]:off[h] + lens[h]].double() for x in (K, V))
        want = torch.softmax(scale * (q[0, h].double() @ k.T.contiguous()), -1) @ v
        # P and O are rounded to bf16: 2^-8 of the largest value each, |V| up to 4.5
        assert float((out[0, h].double() - want).abs().max()) < 4e-2, (h, int(lens[h]))
    hk.close()


@pytest.mark.parametrize("tiles,T", [(65, 1541), (72, 1280), (73, 1249), (80, 1300), (129, 1281), (81, 1300)])
def test_last_round_of_equal_work_items_in_pieces(tiles, T):
    """Eight units of one length whose work items fill the device once or twice and leave 1, 8, 9, 16, 1 (cut in four, four, three, two,
    four) or 17 (left whole) an XCD: against whole work items, and every launch with the bits of the first."""
    u = _u()
    H, d, Nk = 8, 128, tiles * 128 - 5
    gen = torch.Generator(u.DEV)
    gen.manual_seed(tiles)
    q = torch.randn((1, H, Nk, d), generator=gen, device=u.DEV).bfloat16()
    stride = (T + 7) // 8 * 8
    K, V = (torch.randn((H * stride, d), generator=gen, device=u.DEV).bfloat16() for _ in range(2))
    kv = Cache(K, V, np.arange(H, dtype=np.int64) * stride, np.full(H, T, np.int32))
    scale = float(np.float32(d ** -0.5))
    outs = {}
    for name in (None, "tile128"):
        hk = u.make_hack(heads=H, head_dim=d, dtype="bf16", max_units=H, max_cache_len=T, max_queries=Nk, attention=name)
        out = torch.full_like(q, 7.0)
        hk.attn(q, kv, scale, out)
        for _ in range(5):
            again = torch.full_like(q, 7.0)
            hk.attn(q, kv, scale, again)
            assert torch.equal(out, again)
        outs[name] = out.float()
        hk.close()
    # both round P and O to bf16
    assert float((outs[None] - outs["tile128"]).abs().max()) < 1e-2
    assert torch.equal(outs[None], outs["tile128"]) == (tiles == 81)


def test_attention_rejects_empty_unit_and_bad_scale():
    u = _u()
    hk = u.make_hack(heads=1, head_dim=64, dtype="bf16", max_units=1, max_cache_len=64, max_queries=8)
    K = torch.zeros((64, 64), dtype=torch.bfloat16, device=u.DEV)
    q = torch.zeros((1, 1, 8, 64), dtype=torch.bfloat16, device=u.DEV)
    with pytest.raises(HackError):
        hk.attn(q, Cache(K, K.clone(), [0], [0]), 0.1, q.clone())
    with pytest.raises(HackError):
        hk.attn(q, Cache(K, K.clone(), [0], [8]), float("nan"), q.clone())
    with pytest.raises(HackError):
        hk.attn(torch.zeros((1, 1, 9, 64), dtype=torch.bfloat16, device=u.DEV), Cache(K, K.clone(), [0], [8]), 0.1, q)
    hk.close()


def test_attention_variant_query_matches_the_documented_rule(monkeypatch):
    u = _u()
    hk = u.make_hack(heads=16, head_dim=128, dtype="bf16", max_units=32, max_cache_len=256, max_queries=4096)
    # 32-query work items of a launch: B*H*ceil(N_k/32); the key-split kernel serves launches up to 512 of them at d = 128
    assert [hk.attn_variant(2, n) for n in (1, 64, 400, 512, 513, 576, 4096)] == [1, 1, 1, 1, 0, 0, 0]
    assert hk.attn_variant(1, 1024) == 1 and hk.attn_variant(1, 1025) == 0
    hk.close()
    hk = u.make_hack(heads=30, head_dim=64, dtype="bf16", max_units=960, max_cache_len=256, max_queries=256)
    assert hk.attn_variant(32, 64) == 1 and hk.attn_variant(32, 100) == 0     # 1920 and 3840 items against 2048 at d = 64
    assert hk.attn_variant(6, 256) == 1 and hk.attn_variant(8, 256) == 0      # 1440 and 1920 against 1500 where tiles of 128 queries are full
    assert hk.attn_variant(8, 224) == 1                                        # 1680; they are not
    hk.close()
    monkeypatch.setenv("HACK_ATTN_SPLIT_ITEMS", "2048")                       # a limit that is given is taken as it is
    hk = u.make_hack(heads=30, head_dim=64, dtype="bf16", max_units=960, max_cache_len=256, max_queries=256)
    assert hk.attn_variant(8, 256) == 1 and hk.attn_variant(9, 256) == 0      # 1920 and 2160 items
    hk.close()
    hk = u.make_hack(heads=2, head_dim=64, dtype="f32", max_units=2, max_cache_len=64, max_queries=16)
    assert hk.attn_variant(1, 1) == 0                                          # fp32 contexts have one attention kernel
    with pytest.raises(HackError):
        hk.attn_variant(0, 4)
    hk.close()


def test_score_give_up_is_contained_reported_and_recovered(monkeypatch):
    """The in-kernel wait of the fused bf16 score kernel is bounded.  A host-side test hook makes
    one work-group of every fused launch withhold its row sums and sets a small poll limit, so the
    work-groups of that unit give up deterministically while every kernel still exits normally.
    Then: the condition is raised; a fused launch queued after the failing one does not consume
    what it left in the exchange slots (it writes nothing); the call that reports the failure
    re-arms the workspace and switches the context to the two-pass form; the same context then
    gives the right importance again."""
    u = _u()
    monkeypatch.setenv("HACK_SCORE_SPIN_LIMIT", "8")
    monkeypatch.setenv("HACK_SCORE_TEST_SKIP_PUBLISH", "3")
    rng = np.random.default_rng(9)
    H, d, dtype, Nk, L = 4, 128, "bf16", 64, 8000
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=H, max_cache_len=8192, max_queries=Nk)
    monkeypatch.delenv("HACK_SCORE_SPIN_LIMIT")
    monkeypatch.delenv("HACK_SCORE_TEST_SKIP_PUBLISH")
    assert hk.score_mode() == 0
    K = u.rand_values(rng, (H * L, d), dtype)
    Kd = u.to_dev(K, dtype)
    cin = Cache(Kd, Kd, np.arange(H, dtype=np.int64) * L, np.full(H, L, np.int32))
    q = u.rand_values(rng, (1, H, Nk, d), dtype)
    qd = u.to_dev(q, dtype)
    scale = 0.05
    imp1 = torch.full((H, 8192), -1.0, device=u.DEV)
    imp2 = torch.full((H, 8192), -1.0, device=u.DEV)
    # a few milliseconds of other work first, so that both score calls are queued before the first one runs
    # (the host looks at the fault word at every entry)
    big = torch.randn((8192, 8192), device=u.DEV, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for _ in range(8):
        big = (big @ big).clamp_(-1, 1)
    hk.score(qd, cin, scale, imp1)           # one unit of this launch never gets all its sums
    hk.score(qd, cin, scale, imp2)           # queued behind it: must leave without reading the slots
    torch.cuda.synchronize()
    assert torch.all(imp2 == -1.0)           # nothing was formed from stale sums
    with pytest.raises(HackError) as ei:
        hk.check()
    assert ei.value.status == -4
    assert hk.score_mode() == 1              # recovered into the form without in-kernel waits
    hk.check()                               # reported once
    imp3 = torch.full((H, 8192), -1.0, device=u.DEV)
    hk.score(qd, cin, scale, imp3)
    torch.cuda.synchronize()
    hk.check()
    got = imp3.cpu().numpy().astype(np.float64)
    obs = ho.observation_rows(Nk, 32)
    for uu in range(H):
        want = ho.importance(q[0, uu][obs].astype(np.float64), K[uu * L:(uu + 1) * L].astype(np.float64), scale)
        assert float(np.max(np.abs(got[uu, :L] - want) / want)) < 1e-6, uu
        assert np.all(got[uu, L:] == -1.0)
    hk.close()
    # a fresh context without the hook works in the fused form on the same inputs, with the same bits
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=H, max_cache_len=8192, max_queries=Nk)
    imp4 = torch.full((H, 8192), -1.0, device=u.DEV)
    hk.score(qd, cin, scale, imp4)
    torch.cuda.synchronize()
    hk.check()
    assert hk.score_mode() == 0 and torch.equal(imp3, imp4)
    hk.close()


def test_a_score_waits_long_for_work_that_shares_the_device(monkeypatch):
    """How long a fused score launch waits before it gives up and costs its context the fused form: a work-group withholds its
    sums, and the default limit of polls has to last 80 ms (91 ms with the poll of 0.35 us that it was first chosen for)."""
    u = _u()
    monkeypatch.setenv("HACK_SCORE_TEST_SKIP_PUBLISH", "3")
    hk = u.make_hack(heads=4, head_dim=64, dtype="bf16", max_units=4, max_cache_len=8192, max_queries=64)
    monkeypatch.delenv("HACK_SCORE_TEST_SKIP_PUBLISH")
    L = 8000
    k = torch.ones((4 * L, 64), device=u.DEV, dtype=torch.bfloat16)
    q = torch.ones((1, 4, 64, 64), device=u.DEV, dtype=torch.bfloat16)
    imp = torch.empty((4, 8192), device=u.DEV)
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    begin.record()
    hk.score(q, Cache(k, k, np.arange(4, dtype=np.int64) * L, np.full(4, L, np.int32)), 0.05, imp)
    end.record()
    torch.cuda.synchronize()
    with pytest.raises(HackError):
        hk.check()
    assert 80.0 < begin.elapsed_time(end) < 1000.0
    hk.close()


def test_score_two_pass_form_matches_fused_bit_for_bit_and_holds_any_number_of_items():
    """hack_set_score_mode: the two-pass form (no in-kernel waits) gives the same importance bit
    for bit, also where the fused form has to cut the work into several launches, and switching
    back and forth leaves the exchange workspace usable."""
    u = _u()
    rng = np.random.default_rng(15)
    H, B, d, Nk, dtype = 16, 5, 128, 48, "bf16"
    U = H * B
    lens = [int(x) for x in rng.integers(3500, 4200, U)]
    lens[3], lens[40] = 0, 77
    hk = u.make_hack(heads=H, head_dim=d, dtype=dtype, max_units=U, max_cache_len=4352, max_queries=Nk)
    rows = [(u.rand_values(rng, (n, d), dtype),) * 2 for n in lens]
    cin, _ = u.build_cache(rows, d, dtype)
    q, k_new = u.rand_values(rng, (B, H, Nk, d), dtype) * 1.5, u.rand_values(rng, (B, H, Nk, d), dtype)
    qd, kd = u.to_dev(wl.bf16_to_f32(wl.bf16_round(q)), dtype), u.to_dev(k_new, dtype)
    scale = float(np.float32(1.0 / np.sqrt(d)))
    out = []
    for mode in (0, 1, 0, 1):
        hk.set_score_mode(mode)
        imp = torch.full((U, 4352), -1.0, device=u.DEV)
        hk.score(qd, cin, scale, imp, k_new=kd)
        torch.cuda.synchronize()
        hk.check()
        out.append(imp)
    for o in out[1:]:
        assert torch.equal(out[0], o)
    got = out[1].cpu().numpy().astype(np.float64)
    obs = ho.observation_rows(Nk, 32)
    qh = wl.bf16_to_f32(wl.bf16_round(q))
    for uu in (0, 3, 40, U - 1):
        b, h = divmod(uu, H)
        K_in = np.concatenate([rows[uu][0], k_new[b, h]]).astype(np.float64)
        want = ho.importance(qh[b, h][obs].astype(np.float64), K_in, scale)
        assert float(np.max(np.abs(got[uu, :len(want)] - want) / want)) < 1e-6, uu
    hk.close()
