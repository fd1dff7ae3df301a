"""GPU tests of single kernels at the sizes where their tiling can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2604_10900_amd as cask  # noqa: E402
from oracle import ref  # noqa: E402
from synth import caches  # noqa: E402
from tests import parity  # noqa: E402
from tests.test_gpu_parity import _attend_check  # noqa: E402

W = caches.WORKLOADS
B = cask.binding


def _note(*a):
    print(*a, flush=True)


def _units(lens, prefixes, seed=3, **kw):
    """A ragged batch, one generator group per unit."""
    parts = [caches.make(caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=1, prefix=p, decode=n - p, wid=300 + i, **kw), seed=seed)
             for i, (n, p) in enumerate(zip(lens, prefixes))]
    row_off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    return dict(K=torch.cat([c["K"] for c in parts]), V=torch.cat([c["V"] for c in parts]), Q=torch.cat([c["Q"] for c in parts]),
                row_off=row_off, prefix_len=torch.tensor(prefixes, dtype=torch.int32))


SCORE_FORMS = {"chosen": 0, "narrow": B.PATH_NARROW_ROWS, "wide": B.PATH_WIDE_ROWS | B.PATH_NO_FUSED_SWEEPS,
               "one_launch": B.PATH_FORCE_FUSED_SWEEPS}


@pytest.mark.parametrize("form", sorted(SCORE_FORMS))
@pytest.mark.parametrize("G,Wn,causal,splits", [(4, 64, 1, 0), (7, 100, 1, 3), (1, 17, 1, 0), (4, 128, 0, 2)])
def test_scores_with_64_channels(G, Wn, causal, splits, form):
    """bf16 scores with d = 64 (four k-steps a tile): units of a window, a tile, a stage and a block of
    rows and one more, in every form of the sweeps.  Bar: 1e-4 of the unit's largest score, as for
    d = 128 (fp32 sums of 64 exact products, the same two-level row sums)."""
    lens = [Wn, Wn + 1, 129, 256, 257, 1025, 1599, 4097]
    pref = [0, 1, 0, 40, 100, 0, 333, 50]
    c = _units(lens, pref, head_dim=64, q_per_kv=G, window=Wn)
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=G, window=Wn, causal=causal, budget=Wn + 60,
                    path_flags=SCORE_FORMS[form], score_splits=splits)
    row_off, _, K, _, Q = parity.host_arrays(c)
    b = parity.to_device(c, p)
    s = cask.score(b)
    s2 = cask.score(b, torch.full_like(s, 7.0))
    torch.cuda.synchronize()
    assert torch.equal(s, s2)
    _note(form, G, Wn, causal, "score error / max", parity.check_scores(s.cpu().numpy(), ref.score(parity.ref_params(p), row_off, K, Q), row_off))


@pytest.mark.parametrize("G,Wn,n,units", [(1, 128, 2000, 8), (2, 32, 3000, 12), (4, 64, 5378, 6), (5, 100, 1500, 12)])
def test_scores_with_64_channels_keep_the_precision_of_the_vector_kernel(G, Wn, n, units):
    """bf16 scores with d = 64 against 64-bit sums: 2-norm of the error over 2-norm of the result.  Two
    roundings count: that of a row's log-sum-exp (8 to 32 in base 2: half an ulp of it, uniform, 2.7e-7 to
    5.5e-7 x ln 2) and that of a term's distance from the row's reference, as much again if the reference
    lies as far off; a score is the mean over rows, so both shrink with the rows that see the key.
    Reference near the largest logit: 1.7e-7 to 2.6e-7; at the row's first: 3.3e-7 to 4.2e-7."""
    c = _units([n] * units, [n // 8] * units, head_dim=64, q_per_kv=G, window=Wn)
    K, Q = c["K"].double().reshape(units, n, 64), c["Q"].double().reshape(units, Wn * G, 64)
    x = Q @ K.transpose(1, 2).contiguous() / 8.0
    sees = n - Wn + torch.arange(Wn * G) // G
    x.masked_fill_(torch.arange(n)[None, None] > sees[None, :, None], float("-inf"))
    want = torch.softmax(x, dim=2).mean(dim=1).reshape(-1)
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=G, window=Wn, budget=Wn + 60)
    got = cask.score(parity.to_device(c, p)).cpu().double()
    err = float((got - want).norm() / want.norm())
    _note(G, Wn, n, units, "error", err)
    assert err < 3e-7


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,Wn,causal,splits", [(4, 64, 1, 0), (7, 100, 1, 3), (1, 17, 1, 0), (4, 128, 0, 64), (1, 33, 0, 1)])
def test_fp32_scores_on_the_matrix_tiles(G, Wn, causal, splits, d):
    """fp32 scores: units of a window, a 32-row tile, a workgroup's 128 rows and one more.  Bar: 1e-5 of
    the unit's largest score (logits of up to 128 products and sums of at most a few thousand terms
    in fp32, relative errors below 3e-6 in all)."""
    lens = [Wn, Wn + 1, 129, 128, 160, 257, 1025, 1599, 4097]
    pref = [0, 1, 0, 0, 40, 100, 0, 333, 50]
    c = _units(lens, pref, head_dim=d, q_per_kv=G, window=Wn)
    noise = torch.Generator().manual_seed(d)
    c = {k: (v.float() * (1 + 1e-3 * torch.randn(v.shape, generator=noise)) if k in ("K", "V", "Q") else v) for k, v in c.items()}
    p = cask.Params(dtype=cask.F32, head_dim=d, q_per_kv=G, window=Wn, causal=causal, budget=Wn + 60, score_splits=splits)
    row_off, _, K, _, Q = parity.host_arrays(c)
    b = parity.to_device(c, p)
    s = cask.score(b)
    s2 = cask.score(b, torch.full_like(s, 7.0))
    torch.cuda.synchronize()
    assert torch.equal(s, s2)
    _note(d, G, Wn, causal, "score error / max",
          parity.check_scores(s.cpu().numpy(), ref.score(parity.ref_params(p), row_off, K, Q), row_off, rel=1e-5))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,G,stride,n", [(128, 7, 1025, 12), (64, 16, 530, 12), (128, 17, 97, 12), (64, 1, 2000, 3), (128, 5, 9001, 3)])
def test_attention_tiles_splits_and_rows_past_the_end(d, G, stride, n, dtype):
    """cask_attend at lengths around a 16- or 32-row tile and a round of eight waves, up to 17 heads
    (two passes), units split over several workgroups (the longer strides with few units), counts on
    part of the rows; rows past a unit's length hold NaN and must not be seen.  Tolerance: derived at
    _attend_check."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(17)
    cand = [1, 15, 16, 17, 31, 32, 33, 255, 256, 257, 511, 513, 1024, 4097]
    lens = np.array([min(stride, cand[i % len(cand)]) for i in range(n - 2)] + [stride, max(1, stride - 1)], dtype=np.int32)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(d + G)
    Q = (1.5 * torch.randn(n, G, d, generator=g)).to(dt).to(dev)
    Kc = torch.randn(n, stride, d, generator=g).to(dt)
    Vc = torch.randn(n, stride, d, generator=g).to(dt)
    pitch = max(1, stride - 40)
    count = rng.integers(1, 20, (n, pitch)).astype(np.int32)
    padded = np.ones((n, stride), dtype=np.int32)
    padded[:, :pitch] = count
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=1, budget=stride)
    rp = parity.ref_params(p)
    Qh, Kh, Vh = caches.host_bits(Q), caches.host_bits(Kc), caches.host_bits(Vc)
    for i, L in enumerate(lens):
        Kc[i, L:] = float("nan")
        Vc[i, L:] = float("nan")
    Kc, Vc = Kc.to(dev), Vc.to(dev)
    split = B.load().cask_attend_workspace_bytes(B.C.byref(p.c()), n, stride) > 0
    assert split or stride < 2000
    for cnt, pad in ((None, None), (count, padded)):
        got = cask.attend(p, Q, Kc, Vc, torch.from_numpy(lens).to(dev), count=None if cnt is None else torch.from_numpy(cnt).to(dev))
        torch.cuda.synchronize()
        _note(dtype, d, G, stride, split, _attend_check(p, rp, got, ref.attend(rp, Qh, Kh, Vh, lens, count=pad), Qh, Kh, Vh, lens, pad))


def _attend_inputs(dtype, d, G, stride, n, seed):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    Q, K, V = ((s * torch.randn(*shape, generator=g, device="cuda:0")).to(dt)
               for s, shape in ((1.5, (n, G, d)), (1.0, (n, stride, d)), (1.0, (n, stride, d))))
    rng = np.random.default_rng(seed)
    lens = np.where(rng.random(n) < 0.3, rng.integers(1, stride + 1, n), stride - rng.integers(0, min(stride, 40), n)).astype(np.int32)
    lens[0] = stride
    count = rng.integers(1, 20, (n, stride)).astype(np.int32)
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=1, budget=stride)
    return p, Q, K, V, lens, count


def _attend_some(p, got, Q, K, V, lens, count, units):
    """Units `units` of a result against the oracle."""
    rp = parity.ref_params(p)
    Qh, Kh, Vh = (caches.host_bits(x[units]) for x in (Q, K, V))
    cnt = None if count is None else count[units]
    return _attend_check(p, rp, got[units], ref.attend(rp, Qh, Kh, Vh, lens[units], count=cnt), Qh, Kh, Vh, lens[units], cnt)


@pytest.mark.parametrize("dtype,d,G,stride,n", [
    # four waves per workgroup (512 workgroups or more)
    ("bf16", 128, 7, 97, 513), ("bf16", 64, 3, 161, 600), ("f32", 128, 17, 33, 520), ("f32", 64, 2, 300, 512), ("bf16", 128, 4, 2050, 128),
    # long fp32 units of 64 channels: eight waves however many units
    ("f32", 64, 2, 769, 512),
    # long fp32 units of 128 channels: eight waves between 257 and 511 workgroups
    ("f32", 128, 1, 3201, 390),
    # caches beyond 256 MB: non-temporal loads, four and eight waves
    ("bf16", 128, 4, 1101, 512), ("bf16", 128, 2, 1801, 300), ("bf16", 64, 4, 1001, 1100), ("bf16", 64, 1, 2201, 500),
    ("f32", 128, 3, 551, 512), ("f32", 128, 4, 1001, 300), ("f32", 128, 2, 1101, 257), ("f32", 64, 4, 601, 1024), ("f32", 64, 2, 1101, 512)])
def test_attention_forms_of_many_units_and_large_caches(dtype, d, G, stride, n):
    """Every wave count and load policy of cask_attend; a tenth of a large call's units is compared (all of a
    small one's).  Rows behind a unit's length hold NaN.  Tolerance: derived at _attend_check."""
    p, Q, K, V, lens, count = _attend_inputs(dtype, d, G, stride, n, seed=stride)
    past = torch.arange(stride, device=K.device)[None] >= torch.from_numpy(lens).to(K.device)[:, None]
    clean = K.clone(), V.clone()
    K[past] = float("nan")
    V[past] = float("nan")
    large = n * stride * d * K.element_size() * 2 > 256 << 20
    units = list(range(0, n, n // 12 if large or n * stride > 60000 else 1)) + [n - 1]
    for cnt in (None, count):
        got = cask.attend(p, Q, K, V, torch.from_numpy(lens).to(K.device), count=None if cnt is None else torch.from_numpy(cnt).to(K.device))
        torch.cuda.synchronize()
        assert torch.isfinite(got).all()
        _note(dtype, d, G, stride, n, "large" if large else "", _attend_some(p, got, Q, *clean, lens, cnt, units))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,G,stride,n", [(128, 5, 9001, 3), (64, 16, 2000, 7), (64, 17, 1800, 100)])
def test_attention_of_long_units_with_and_without_a_workspace(d, G, stride, n, dtype):
    """Few long units through cask_attend, and through cask_attend_ws with no workspace and with one a byte
    short: one launch each, the same bits, against the oracle and within its bar of the split result."""
    p, Q, K, V, lens, count = _attend_inputs(dtype, d, G, stride, n, seed=7)
    lib, dev = B.load(), K.device
    cp = p.c()
    need = lib.cask_attend_workspace_bytes(B.C.byref(cp), n, stride)
    assert need > 0
    ln, cn = torch.from_numpy(lens).to(dev), torch.from_numpy(count).to(dev)
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    st = torch.cuda.current_stream().cuda_stream
    args = [B.C.byref(cp), n, Q.data_ptr(), K.data_ptr(), V.data_ptr(), stride, ln.data_ptr(), cn.data_ptr(), stride]
    outs = [torch.full_like(Q, 7.0) for _ in range(4)]
    assert lib.cask_attend(*args, outs[0].data_ptr(), st) == 0
    assert lib.cask_attend_ws(*args, outs[1].data_ptr(), None, 0, st) == 0
    assert lib.cask_attend_ws(*args, outs[2].data_ptr(), ws.data_ptr(), need - 1, st) == 0
    assert lib.cask_attend_ws(*args, outs[3].data_ptr(), ws.data_ptr(), need, st) == 0
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    units = list(range(min(n, 8)))
    for o in (outs[0], outs[3]):
        _note(dtype, d, G, stride, n, _attend_some(p, o, Q, K, V, lens, count, units))
    assert torch.equal(outs[3], cask.attend(p, Q, K, V, ln, count=cn))


@pytest.mark.parametrize("d,G,n,units", [(128, 7, 2000, 12), (128, 4, 300, 24), (64, 3, 1000, 24), (64, 8, 4097, 6)])
def test_fp32_attention_keeps_the_precision_of_short_sums(d, G, n, units):
    """fp32 cask_attend against 64-bit sums: 2-norm of the error over 2-norm of the result.  A weight is
    off by ln 2 times its base-2 logit's error, and the logits that count are about 10 here.  A logit
    of d products in chains of eight, the chains added in pairs, passes about 8 / 2 + log2(d / 8) = 8
    roundings of 2^-25 x 10 / sqrt(3) at full size, most of them smaller: below ln 2 x 4.8e-7 = 3.4e-7;
    the value sums add less than 2e-7, in squares: 4e-7.  (One chain of d products: 4.5e-7 to 8.5e-7.)"""
    dev = torch.device("cuda:0")
    g = torch.Generator().manual_seed(n + d)
    Q = 1.2 * torch.randn(units, G, d, generator=g)
    K = torch.randn(units, n, d, generator=g)
    Q += 0.35 * K[:, n // 2][:, None] + 0.35 * K[:, n // 3][:, None]     # two rows that hold much of the weight
    V = torch.randn(units, n, d, generator=g)
    count = torch.randint(1, 4, (units, n), generator=g, dtype=torch.int32)
    p = cask.Params(dtype=cask.F32, head_dim=d, q_per_kv=G, window=1, budget=n)
    for cnt in (None, count):
        x = Q.double() @ K.double().transpose(1, 2) / d ** 0.5
        if cnt is not None:
            x = x + cnt.double().log()[:, None, :]
        want = torch.softmax(x, dim=2) @ V.double()
        got = cask.attend(p, Q.to(dev), K.to(dev), V.to(dev), torch.full((units,), n, dtype=torch.int32, device=dev),
                          count=None if cnt is None else cnt.to(dev)).cpu().double()
        err = float((got - want).norm() / want.norm())
        _note(d, G, n, cnt is not None, "largest logit", round(float(x.max()) * 1.4427, 1), "error", err)
        assert err < 4e-7


@pytest.mark.parametrize("radius", [0, 70])
@pytest.mark.parametrize("tau", [0.3, -2.0])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
def test_consolidation_at_the_edges_of_tiles_and_seed_blocks(d, dtype, tau, radius):
    """cask_consolidate with role arrays of the caller: donor ranges around a 32-row tile and a
    workgroup's rows, seed counts around a 32-row step and a 128-row block, up to every second row
    (tau = -2: every donor folds).  A donor may differ only where its two best cosines, or best and
    threshold, lie within 1e-4 in the oracle (fp32 sums of 64 or 128 products: errors below 2e-5)."""
    Wn = 16
    lens = [Wn + 1, Wn + 33, 160, 161, 289, 544, 1057, 2100]
    pref = [0, 1, 16, 0, 17, 16, 1, 333]
    seeds = [1, 1, 31, 33, 127, 128, 129, 800]
    c = _units(lens, pref, head_dim=d, q_per_kv=2, window=Wn, cluster_frac=0.5)
    if dtype == "f32":
        c = {k: (v.float() if k in ("K", "V", "Q") else v) for k, v in c.items()}
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=2, window=Wn, budget=900,
                    sim_threshold=tau, merge_radius=radius)
    row_off, prefix_len, K, V, Q = parity.host_arrays(c)
    rng = np.random.default_rng(d)
    total = int(row_off[-1])
    role = np.full(total, ref.DONOR, dtype=np.uint8)
    for u, (n, P, M) in enumerate(zip(lens, pref, seeds)):
        lo = int(row_off[u])
        role[lo:lo + P] = ref.PREFIX_KEEP
        role[lo + n - Wn:lo + n] = ref.RECENT
        role[lo + P + rng.choice(n - Wn - P, size=min(M, n - Wn - P), replace=False)] = ref.SEED
    s = rng.random(total).astype(np.float32)
    want, best, second = ref.consolidate(parity.ref_params(p), row_off, prefix_len, K, s, role, want_sims=True)
    b = parity.to_device(c, p)
    got = cask.consolidate(b, torch.from_numpy(s).to(b.device), torch.from_numpy(role).to(b.device))
    torch.cuda.synchronize()
    assert (want >= 0).sum() > 800
    _note(d, dtype, tau, radius, "excused", parity.check_assign_excused(got.cpu().numpy(), want, best, second, float(np.float32(tau)), "edges"))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("longest,units,G,Wn,causal", [
    (256, 40, 7, 64, 1), (384, 40, 7, 64, 0), (511, 40, 7, 65, 1), (640, 40, 8, 57, 1), (641, 40, 7, 64, 1), (600, 140, 5, 60, 1),
    (96, 2, 1, 17, 1), (512, 3, 7, 128, 1), (768, 3, 5, 100, 0), (769, 2, 7, 33, 1), (1024, 3, 4, 64, 1)])
def test_scores_of_short_units_in_one_sweep(longest, units, G, Wn, causal, d):
    """Units of at most 1024 rows, whose event scores them in one launch: four waves (more than 256
    workgroups) or eight, every number of key tiles per wave, lengths around a tile and down to the
    window, a last block of window rows that is not full, and a batch that takes two sweeps; the scores of the event against the oracle
    (bar as above: 1e-4 of the unit's largest score)."""
    cand = [longest, Wn, Wn + 1, longest - 1, longest // 2 + 1, (longest + Wn) // 2, max(Wn, longest - 32), max(Wn, 129)]
    lens = [min(longest, cand[i % len(cand)]) for i in range(units)]
    c = _units(lens, [i % 3 * 5 if n > Wn + 10 else 0 for i, n in enumerate(lens)], head_dim=d, q_per_kv=G, window=Wn)
    p = cask.Params(dtype=cask.BF16, head_dim=d, q_per_kv=G, window=Wn, causal=causal, budget=max(Wn + 5, longest // 2))
    row_off, _, K, _, Q = parity.host_arrays(c)
    b = parity.to_device(c, p)
    s = cask.compress(b).scores.clone()
    s2 = cask.compress(b).scores
    torch.cuda.synchronize()
    assert torch.equal(s, s2)
    err = parity.check_scores(s.cpu().numpy(), ref.score(parity.ref_params(p), row_off, K, Q), row_off)
    _note(d, longest, units, "score error / max", err)
    assert err < 5e-6   # fp32 sums of at most 1024 terms, two levels of exponentials: relative errors of a few 2^-20


def test_hidden_keys_keep_their_scores_when_a_window_row_is_nan():
    """A window row that holds NaN spoils the keys it sees and no others."""
    Wn, G, n = 40, 2, 300
    c = _units([n, n], [0, 0], head_dim=128, q_per_kv=G, window=Wn)
    p = cask.Params(dtype=cask.BF16, head_dim=128, q_per_kv=G, window=Wn, budget=n)
    clean = cask.compress(parity.to_device(c, p)).scores.clone()
    c["Q"][0, 9, 1] = float("nan")
    got = cask.compress(parity.to_device(c, p)).scores
    torch.cuda.synchronize()
    last = n - Wn + 9                      # the last key that window row sees
    assert torch.isnan(got[:last + 1]).all()
    assert torch.equal(got[last + 1:], clean[last + 1:])


@pytest.mark.parametrize("dtype,d,form", [("bf16", 64, f) for f in sorted(SCORE_FORMS)] + [("f32", 64, "chosen"), ("f32", 128, "chosen"),
                                                                                         ("bf16", 64, "short"), ("bf16", 128, "short")])
@pytest.mark.parametrize("G,Wn", [(1, 17), (2, 33), (7, 100), (4, 64)])
def test_a_key_at_minus_infinity_scores_zero(G, Wn, dtype, d, form):
    """Keys whose logit is -inf for every window row that sees them get the score 0 and leave the others
    theirs, also where W * G does not fill the last tile of window rows (the tile's spare places must
    not multiply zeros with the infinity)."""
    lens = [300, 449] if form == "short" else [257, 1500, 700]
    c = _units(lens, [0] * len(lens), head_dim=d, q_per_kv=G, window=Wn)
    if dtype == "f32":
        c = {k: (v.float() if k in ("K", "V", "Q") else v) for k, v in c.items()}
    c["Q"][..., 0] = c["Q"][..., 0].abs() + 0.125
    spots = [int(c["row_off"][u]) + r for u, n in enumerate(lens) for r in (5, n // 2, n - 1)]
    c["K"][spots, 0] = float("-inf")
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60,
                    path_flags=SCORE_FORMS.get(form, 0))
    b = parity.to_device(c, p)
    got = (cask.compress(b).scores if form == "short" else cask.score(b)).cpu()
    want = torch.empty(got.shape, dtype=torch.float64)
    for u, n in enumerate(lens):
        lo = int(c["row_off"][u])
        x = c["Q"][u].double().reshape(-1, d) @ c["K"][lo:lo + n].double().t().contiguous() / d ** 0.5
        x.masked_fill_(torch.arange(n)[None] > n - Wn + torch.arange(Wn * G)[:, None] // G, float("-inf"))
        want[lo:lo + n] = torch.softmax(x, dim=1).mean(dim=0)
    assert not torch.isnan(want).any()
    assert (got[spots] == 0).all()
    assert float((got.double() - want).abs().max()) <= 1e-4 * float(want.max())


@pytest.mark.parametrize("units", [3, 131])
@pytest.mark.parametrize("d,R,budget,core,prefix_budget", [(128, -1, 300, -1, 100), (64, 40, 257, 64, 65), (128, 33, 129, 0, 64)])
def test_tail_of_short_units_at_the_edges_of_rank_pieces(d, R, budget, core, prefix_budget, units):
    """Whole events on units of at most 1024 rows: prefix and decode ranges of 63, 64, 65, ... rows
    (pieces of the rank count), ranks asked for in both, with the copying workgroups (few units) and
    without; rows, roles, folds and statuses element by element against the oracle."""
    Wn = 32
    cand = [(200, 0), (64 + Wn, 1), (Wn + 129, 64), (Wn + 128, 63), (320, 65), (512, 128), (1024, 129), (1000, 300), (577, 449), (Wn, 0)]
    lens, pref = zip(*[cand[(i * 3 + units) % len(cand)] for i in range(units)])
    if units > 10:   # (the oracle's time: mostly the shorter ones)
        lens, pref = zip(*[(n, q) if i % 10 == 0 else (min(n, 330), min(q, 66)) for i, (n, q) in enumerate(zip(lens, pref))])
    c = _units(list(lens), list(pref), head_dim=d, q_per_kv=2, window=Wn, cluster_frac=0.6)
    p = cask.Params(dtype=cask.BF16, head_dim=d, q_per_kv=2, window=Wn, recent=R, budget=budget, core=core, prefix_budget=prefix_budget)
    _note(d, budget, units, parity.full_check(c, p))


@pytest.mark.parametrize("longest", [640, 641])
@pytest.mark.parametrize("units", [4, 130])
def test_rank_pieces_of_batches_up_to_and_beyond_640_rows(units, longest):
    """The rank count's two piece sizes (the batch's longest unit decides), with and without the copying
    workgroups: prefix-only units, prefixes and traces of a piece, a block and one row more or less."""
    Wn = 32
    cand = [(longest, 300), (64 + Wn, 64 + Wn), (longest, longest), (Wn + 33, 31), (Wn + 257, 129), (Wn + 160, 32), (400, 255)]
    lens, pref = zip(*[cand[i % len(cand)] for i in range(units)])
    c = _units(list(lens), list(pref), head_dim=128, q_per_kv=2, window=Wn, cluster_frac=0.6)
    p = cask.Params(dtype=cask.BF16, head_dim=128, q_per_kv=2, window=Wn, budget=90, prefix_budget=40)
    _note(units, longest, parity.full_check(c, p))


@pytest.mark.parametrize("merged", [0.02, 0.9])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
def test_group_diagnostics_around_a_round_of_rows(d, dtype, merged):
    """Dispersion and lost mass of units around a wave's 64 rows, a workgroup's 1024 and its 8192 in
    flight, with few and with nearly all rows assigned to a slot.  Bar 2e-5: distances of fp32 terms
    (64 bands, relative error below 1e-5 in all), summed in double."""
    Wn, B_ = 16, 40
    lens = [Wn, 63, 64, 65, 1023, 1025, 8191, 8193, 9300]
    c = _units(lens, [0] * len(lens), head_dim=d, q_per_kv=1, window=Wn)
    f32 = dtype == "f32"
    if f32:
        c = {k: (v.float() if k in ("K", "V", "Q") else v) for k, v in c.items()}
    p = cask.Params(dtype=cask.F32 if f32 else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=B_)
    row_off, _, K, _, _ = parity.host_arrays(c)
    rng = np.random.default_rng(d)
    total = int(row_off[-1])
    s = rng.random(total).astype(np.float32)
    a = np.where(rng.random(total) < merged, rng.integers(0, B_, total), -1).astype(np.int32)
    Ko = torch.randn(len(lens), B_, d, generator=torch.Generator().manual_seed(d)).to(torch.float32 if f32 else torch.bfloat16)
    want_d, want_l = ref.group_diagnostics(parity.ref_params(p), row_off, K, s, a, caches.host_bits(Ko))
    b = parity.to_device(c, p)
    got_d, got_l = cask.group_diagnostics(b, torch.from_numpy(s).to(b.device), torch.from_numpy(a).to(b.device), Ko.to(b.device))
    torch.cuda.synchronize()
    np.testing.assert_allclose(got_d.cpu().numpy(), want_d, rtol=2e-5, atol=1e-6)
    np.testing.assert_allclose(got_l.cpu().numpy(), want_l, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("spread", ["outlier", "binades", "clusters"])
@pytest.mark.parametrize("N,P", [(6144, 100), (6145, 6000), (18432, 16384), (18433, 9000), (25601, 40), (36864, 20000), (36865, 300), (40000, 37000)])
def test_ranks_where_the_bins_are_uneven(N, P, spread):
    """Roles and kept rows on injected scores at the edges of the selection's instances (6, 12, 18, 25, 36
    keys a thread, then a chunk of keys at a time): two outliers that leave everything else in one
    bin of the first histogram, sixty binades, and clusters a few ulps wide with ties in them."""
    rng = np.random.default_rng(N + len(spread))
    lens, pref = [N, 1200], [P, 200]
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(row_off[-1])
    if spread == "outlier":
        sc = (1.0 + rng.permutation(total) / total).astype(np.float32)
        sc[[5, N + 5]], sc[[9, N + 9]] = 3e38, -3e38
    elif spread == "binades":
        sc = (2.0 ** rng.uniform(-60, 0, total)).astype(np.float32)
    else:
        sc = (2.0 ** rng.integers(-3, 3, total)).astype(np.float32)
        sc = (sc.view(np.uint32) + rng.integers(0, 200, total).astype(np.uint32)).view(np.float32)
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=1, window=64, budget=900, sim_threshold=2.0)
    rp, prefix = parity.ref_params(p), np.array(pref, dtype=np.int32)
    role_w, _ = ref.prefix_evict(rp, row_off, prefix, sc)
    role_w, _ = ref.partition(rp, row_off, prefix, sc, role_w)
    K = torch.from_numpy(rng.standard_normal((total, 64)).astype(np.float32)).to(torch.bfloat16).cuda()
    b = cask.Batch(p, torch.from_numpy(row_off), torch.from_numpy(prefix), K, K, torch.zeros(2, 64, 1, 64, dtype=torch.bfloat16, device="cuda"))
    sd = torch.from_numpy(sc).cuda()
    role, _ = cask.prefix_evict(b, sd)
    role, _ = cask.partition(b, sd, role)
    out = cask.compress(b, scores=sd)
    rho = cask.mass_diagnostics(b, sd, role, out.out_mass, out.out_len)
    torch.cuda.synchronize()
    assert np.array_equal(role.cpu().numpy(), role_w)
    kept = np.isin(role_w, [1, 2, 3, 5])
    for u in range(2):
        rows = np.nonzero(kept[row_off[u]: row_off[u + 1]])[0]
        assert int(out.out_len[u]) == len(rows) == 900
        assert np.array_equal(out.out_src[u].cpu().numpy(), rows)
        want = np.full(lens[u], -1)
        want[rows] = np.arange(len(rows))
        assert np.array_equal(out.assign[row_off[u]: row_off[u + 1]].cpu().numpy(), want)
    if spread != "outlier":
        want_rho = ref.mass_diagnostics(rp, row_off, sc, role_w, out.out_mass.cpu().numpy(), out.out_len.cpu().numpy())
        np.testing.assert_allclose(rho.cpu().numpy(), want_rho, rtol=2e-6)


@pytest.mark.parametrize("kind", ["zeros", "two", "ulps", "end_of_a_bin"])
@pytest.mark.parametrize("N,P", [(4096, 30), (9217, 5000), (36864, 300), (36865, 20000)])
def test_ranks_where_many_rows_share_a_value(N, P, kind):
    """Roles where a bin of the first histogram holds one value thousands of times, two values an ulp apart, or a
    thousand different keys up to its very end, with the rank between its last two and others right behind it."""
    rng = np.random.default_rng(N)
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=1, window=64, budget=900, sim_threshold=2.0)
    C = cask.plan(p, P, N)["core"]
    if kind == "zeros":
        sc = np.where(rng.random(N) < 0.95, 0.0, rng.random(N))
    elif kind == "two":
        sc = np.where(rng.random(N) < 0.5, 1e-4, 2e-4)
    elif kind == "ulps":
        sc = (np.float32(1.0).view(np.uint32) + rng.integers(0, 2, N).astype(np.uint32)).view(np.float32)
        sc[[3, N - 70]], sc[[4, N - 71]] = 3e38, -3e38
    else:
        least = int(np.float32(2.0 ** -20).view(np.uint32))
        end = least + 40 * 65536                                       # bins of 2^16 from the smallest key on
        top = least + 2 ** 27 - 1 - np.arange(C - 71)
        behind, last = end + np.arange(70), np.array([end - 1, end - 3])
        below = np.concatenate([[end - 65536 + 0x8003], end - 65536 + 0x8003 + rng.integers(0, 0x7000, 1100), [least]])
        keys = np.concatenate([top, behind, last, below])
        n = N - 64 - P
        keys = np.concatenate([keys, least + rng.integers(0, 30 * 65536, n - len(keys))]).astype(np.uint32)
        sc = np.zeros(N, dtype=np.float32)
        sc[P: P + n] = rng.permutation(keys).view(np.float32)
    sc = sc.astype(np.float32)
    rp, row_off, prefix = parity.ref_params(p), np.array([0, N], dtype=np.int64), np.array([P], dtype=np.int32)
    role_w, _ = ref.prefix_evict(rp, row_off, prefix, sc)
    role_w, _ = ref.partition(rp, row_off, prefix, sc, role_w)
    K = torch.zeros(N, 64, dtype=torch.bfloat16, device="cuda")
    b = cask.Batch(p, torch.from_numpy(row_off), torch.from_numpy(prefix), K, K, torch.zeros(1, 64, 1, 64, dtype=torch.bfloat16, device="cuda"))
    sd = torch.from_numpy(sc).cuda()
    role, _ = cask.prefix_evict(b, sd)
    role, _ = cask.partition(b, sd, role)
    src = cask.compress(b, scores=sd).out_src[0]
    torch.cuda.synchronize()
    assert np.array_equal(role.cpu().numpy(), role_w)
    assert np.array_equal(src.cpu().numpy(), np.nonzero(np.isin(role_w, [1, 2, 3, 5]))[0])


def _scores64(c, units, n, d, G, Wn):
    """Scores in 64 bits, on the CPU."""
    K, Q = c["K"].double().reshape(units, n, d), c["Q"].double().reshape(units, Wn * G, d)
    x = Q @ K.transpose(1, 2).contiguous() / d ** 0.5
    x.masked_fill_(torch.arange(n)[None, None] > (n - Wn + torch.arange(Wn * G) // G)[None, :, None], float("-inf"))
    return torch.softmax(x, dim=2).mean(dim=1).reshape(-1)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,Wn,n,units,kind", [(4, 64, 4096, 4, "plain"), (2, 32, 1000, 6, "plain"), (7, 100, 1531, 3, "plain"),
                                               (4, 64, 1000, 4, "small_keys"), (4, 64, 1000, 4, "past_bf16")])
def test_fp32_scores_from_bf16_terms(G, Wn, n, units, kind, d):
    """fp32 scores against 64-bit sums, 2-norm of the error over 2-norm of the result.  The products of three
    bf16 terms leave 2^-24 of a product; what counts are the roundings of a logit (two large partial sums
    of sixteen channels at a time) and of the log-sum-exp (half an ulp at 8 to 16 in base 2: 3.4e-7 to
    6.9e-7 x ln 2, uniform, shrinking with the rows that see a key): measured 1.2e-7 to 3.1e-7.  small_keys:
    keys 2^-100 of the queries' inverse (their third terms stay normal numbers); past_bf16: finite keys that
    round to infinity in bf16 take the wave's share to the fp32 tiles."""
    c = _units([n] * units, [n // 8] * units, head_dim=d, q_per_kv=G, window=Wn)
    noise = torch.Generator().manual_seed(d + n)
    c = {k: (v.float() * (1 + 1e-3 * torch.randn(v.shape, generator=noise)) if k in ("K", "V", "Q") else v) for k, v in c.items()}
    if kind == "small_keys":
        c["K"], c["Q"] = c["K"] * 2.0 ** -100, c["Q"] * 2.0 ** 100
    elif kind == "past_bf16":
        c["Q"][..., 5] *= 2.0 ** -126
        c["K"][:, 5] *= 2.0 ** 20
        c["K"][[3, 40, n - Wn - 2, 2 * n - Wn + 1], 5] = torch.tensor([3.4e38, -3.4e38, 3.4e38, 3.4e38])
    want = _scores64(c, units, n, d, G, Wn)
    assert bool(torch.isfinite(want).all())
    p = cask.Params(dtype=cask.F32, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60)
    got = cask.score(parity.to_device(c, p)).cpu().double()
    err = float((got - want).norm() / want.norm())
    _note(G, Wn, n, units, kind, d, "error", err)
    assert err < 4e-7


@pytest.mark.parametrize("budget,h,d,prefix,rows", [(320, 7, 128, 0, 1500), (321, 7, 128, 0, 1500), (320, 7, 64, 40, 900), (256, 1, 128, 30, 1200),
                                                    (192, 2, 64, 0, 700), (300, 7, 128, 20, 330)])
def test_dedup_walk_with_every_row_in_lds(budget, h, d, prefix, rows):
    """De-duplicated seeding of bf16 units where the walk covers at most 448 rows (budget 320, h = 7: exactly;
    321: the general kernel), a few blocks of 64 and one, and a scratch shorter than the walk; roles and
    events against the oracle, at a threshold that no decision of the walk comes close to."""
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=3, prefix=prefix, decode=rows, budget=budget, head_dim=d, window=32, cluster_frac=0.6)
    c = caches.make(w, seed=5 + budget)
    row_off, prefix_len, K, V, Q = parity.host_arrays(c)
    for dt in (0.0, 0.013, -0.017, 0.031, -0.029, 0.047):
        p = parity.params_of(w, sim_threshold=0.8 + dt, seed_dedup=h)
        rp = parity.ref_params(p)
        scores = ref.score(rp, row_off, K, Q)
        role0, _ = ref.prefix_evict(rp, row_off, prefix_len, scores)
        if ref.partition_keys(rp, row_off, prefix_len, K, scores, role0)[2].min() >= 1e-3:
            break
    else:
        pytest.fail("no clear threshold for this cache")
    _note(budget, h, d, parity.full_check(c, p))


@pytest.mark.parametrize("units,N,P,budget,tau,dtype,d", [(3, 8292, 100, 160, -1.0, "bf16", 128), (3, 8293, 100, 160, -1.0, "bf16", 128),
                                                          (131, 1200, 0, 90, 0.2, "bf16", 64), (70, 1100, 60, 130, -1.0, "f32", 64),
                                                          (2, 3000, 2000, 700, -1.0, "f32", 128), (5, 1500, 0, 65, -1.0, "bf16", 128)])
def test_grouping_and_fold_in_one_launch(units, N, P, budget, tau, dtype, d):
    """Whole events where every donor, or most, fold: two to eight workgroups a unit, lists in LDS and in memory
    (a share's 1024 donors), groups folded by one wave and by four, a decode trace that just fills a
    workgroup's rows (8192) and one row more (two launches), a single seed; against the oracle."""
    Wn = 32
    kw = dict(head_dim=d, q_per_kv=1, window=Wn, cluster_frac=0.5)
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=units, prefix=P, decode=N - P, budget=budget, **kw)
    c = caches.make(w, seed=units + N)
    if dtype == "f32":
        c = {k: (v.float() if k in ("K", "V", "Q") else v) for k, v in c.items()}
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=budget, sim_threshold=tau)
    _note(units, N, budget, parity.full_check(c, p, expect_folds=True))


@pytest.mark.parametrize("units,N,P,budget,dtype,d,radius,scale", [(3, 700, 40, 230, "bf16", 128, 0, 1.0), (2, 289, 1, 120, "bf16", 128, 90, 1.0),
                                                                    (9, 1100, 300, 380, "bf16", 64, 0, 1.0), (2, 600, 20, 320, "f32", 128, 100, 1.0),
                                                                    (2, 500, 0, 200, "f32", 64, 0, 1e16), (2, 500, 0, 200, "f32", 128, 0, 1e-14),
                                                                    (1, 500, 0, 200, "bf16", 128, 0, 1e17)])
def test_band_distance_screen(units, N, P, budget, dtype, d, radius, scale):
    """Kappa geometry with thresholds among the nearest distances (no donor folds, some, most, all), so that
    the screen decides on pairs near the bar: blocks of 32 seeds and remainders, last tiles of rows, keys
    whose squares are at either end of the range where the screen holds; against the oracle."""
    Wn = 32
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=units, prefix=P, decode=N - P, budget=budget, head_dim=d, q_per_kv=1, window=Wn,
                      cluster_frac=0.5)
    c = caches.make(w, seed=units + N)
    c["K"] = (c["K"].float() * scale).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    c["Q"] = (c["Q"].float() / scale).to(c["K"].dtype)
    c["V"] = c["V"].to(c["K"].dtype)
    band = torch.rand(d // 2, generator=torch.Generator().manual_seed(d)) ** 2
    band[5] = 0.0
    kw = dict(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=budget, merge_geometry=1,
              band_weight=band.cuda(), merge_radius=radius)
    row_off, prefix_len, K, V, Q = parity.host_arrays(c)
    rp = parity.ref_params(cask.Params(dist_threshold=1e30, **kw))
    want = ref.compress(rp, row_off, prefix_len, K, V, Q)
    near = -ref.consolidate(rp, row_off, prefix_len, K, want["scores"], want["role"], want_sims=True)[1][want["role"] == 4]
    near = np.sort(near[np.isfinite(near)])
    for share in (0.0, 0.05, 0.5, 0.95, 1.0):
        theta = float(near[int(share * (len(near) - 1))]) * (0.5 if share == 0.0 else 1.001)
        _note(units, N, dtype, d, scale, "theta", theta, parity.full_check(c, cask.Params(dist_threshold=theta, **kw)))


@pytest.mark.parametrize("dtype,d,G,Wn", [("bf16", 128, 7, 64), ("bf16", 64, 3, 50), ("f32", 64, 2, 40)])
def test_ragged_units_and_key_splits(dtype, d, G, Wn):
    """Units of very different lengths, more than eight of them (parts of a unit are turned round from unit to
    unit), several row blocks, the library's own key splits, an odd and an even number of them; scores and a
    whole event's merges against the oracle.  Bar of the scores: 1e-4 of the largest, as everywhere."""
    lens = [2700, 130, 1100, 260, 2048, 513, 65 + Wn, 1900, 400, 2600, 700, 150, 1300, 2100, 320, 900, 1025, 180, 2500]
    c = _units(lens, [n // 7 for n in lens], head_dim=d, q_per_kv=G, window=Wn)
    if dtype == "f32":
        c = {k: (v.float() if k in ("K", "V", "Q") else v) for k, v in c.items()}
    row_off, prefix_len, K, V, Q = parity.host_arrays(c)
    kw = dict(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60)
    want = ref.score(parity.ref_params(cask.Params(**kw)), row_off, K, Q)
    for splits, form in ((0, 0), (1, 0), (2, 0), (3, 0), (4, 0), (3, B.PATH_WIDE_ROWS), (4, B.PATH_WIDE_ROWS)):
        p = cask.Params(score_splits=splits, path_flags=form | B.PATH_NO_FUSED_SWEEPS, **kw)
        got = cask.score(parity.to_device(c, p)).cpu().numpy()
        for u in range(len(lens)):
            sl = slice(row_off[u], row_off[u + 1])
            assert np.abs(got[sl] - want[sl]).max() <= 1e-4 * want[sl].max(), (splits, form, u)
    _note(dtype, d, parity.full_check(c, cask.Params(**kw)))


@pytest.mark.parametrize("N", [4096, 4097, 8192, 8193])
def test_roles_indexed_at_the_edges_of_the_instances(N):
    """Slots and seed ordinals from given roles (consolidation on its own, and events with de-duplicated
    seeding) for units of four and eight rows a thread, one row more, and one of 150 rows beside each."""
    c = _units([N, 150], [300, 20], head_dim=64, q_per_kv=1, window=32)
    kw = dict(head_dim=64, q_per_kv=1, window=32, budget=140)
    _note(N, parity.full_check(c, cask.Params(sim_threshold=0.3, **kw)))
    p = cask.Params(sim_threshold=2.0, seed_dedup=2, **kw)   # no cosine reaches it: every walk is decided by rank alone
    _note(N, parity.full_check(c, p))


@pytest.mark.parametrize("units,longest,rest", [(512, 6000, 1100), (300, 9000, 1500)])
def test_key_splits_do_not_follow_the_other_units_lengths(units, longest, rest):
    """A unit's scores are the same bits whether the other units of the batch are as long as it or much shorter
    (with the number of units and the longest unit the same): the order of its sums is not theirs to choose."""
    at = [0, units // 3, units - 1]   # the units that have the longest length in both batches
    G, Wn, d = 2, 32, 64
    g = torch.Generator(device="cuda").manual_seed(units)
    K3 = torch.randn(3, longest, d, generator=g, device="cuda").to(torch.bfloat16)
    Q = torch.randn(units, Wn, G, d, generator=g, device="cuda").to(torch.bfloat16)
    p = cask.Params(dtype=cask.BF16, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60)
    got = []
    for other in (longest, rest):
        lens = [longest if u in at else other for u in range(units)]
        row_off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
        K = torch.randn(int(row_off[-1]), d, generator=g, device="cuda").to(torch.bfloat16)
        for k, u in zip(K3, at):
            K[int(row_off[u]): int(row_off[u + 1])] = k
        s = cask.score(cask.Batch(p, row_off, torch.zeros(units, dtype=torch.int32), K, K, Q))
        got.append([s[int(row_off[u]): int(row_off[u + 1])].clone() for u in at])
    torch.cuda.synchronize()
    for u, a, b in zip(at, *got):
        assert torch.equal(a, b), u


@pytest.mark.parametrize("units,n,G,Wn", [(171, 5248, 6, 64), (303, 2817, 4, 128), (611, 1456, 7, 64), (128, 5378, 7, 128)])
def test_narrow_sweeps_of_64_channels_sum_in_the_wide_forms_order(units, n, G, Wn):
    """Batches that take the narrow form where the model prefers the wide one (their own best key splits would be
    2, 2, 1 and 1 for 4, 5, 2 and 1): the scores are the wide form's, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(n)
    K = torch.randn(units * n, 64, generator=g, device="cuda").to(torch.bfloat16)
    Q = torch.randn(units, Wn, G, 64, generator=g, device="cuda").to(torch.bfloat16)
    row_off = torch.arange(units + 1, dtype=torch.int64) * n
    got = []
    for flags in (0, B.PATH_WIDE_ROWS):
        p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=G, window=Wn, budget=Wn + 60, path_flags=flags)
        got.append(cask.score(cask.Batch(p, row_off, torch.zeros(units, dtype=torch.int32), K, K, Q)))
    torch.cuda.synchronize()
    assert torch.equal(*got)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_band_distance_screen_at_the_worst_rounding_to_bf16(dtype, d):
    """Keys whose weighted channels all lie half a bf16 ulp above a power of two, where rounding takes the most
    off (2^-8 of a value, 2^-7 of a product): equal keys are at distance 0, and the screen must let them
    through at a small threshold.  Copies are spread over forty patterns of signs; against the oracle."""
    rng = np.random.default_rng(d)
    N, Wn, M, n_core = 700, 32, 40, 30
    pattern = rng.choice([-1.0, 1.0], (M, d)).astype(np.float32)
    free = rng.permutation(N - Wn)
    core, seeds = free[:n_core], free[n_core:n_core + M]
    which = rng.integers(0, M, N)
    which[seeds] = rng.permutation(M)
    K = pattern[which] * np.float32(2.0) ** (which % 5)[:, None].astype(np.float32)
    up = np.float32(1 + 2.0 ** -8)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    if dtype == "f32":
        K = K * up
    band = torch.full((d // 2,), float(up) if dtype == "bf16" else 1.0)
    s = (1e-3 * (1.0 + rng.permutation(N))).astype(np.float32) / N
    s[core] = 0.5 + 1e-3 * np.arange(n_core, dtype=np.float32)
    s[seeds] = 0.25 + 1e-3 * np.arange(M, dtype=np.float32)
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=Wn + n_core + M, core=n_core,
                    prefix_budget=0, merge_geometry=1, band_weight=band.cuda(), dist_threshold=0.25)
    rp = parity.ref_params(p)
    c = dict(K=torch.from_numpy(K).to(dt), V=torch.from_numpy(K).to(dt), Q=torch.zeros(1, Wn, 1, d, dtype=dt),
             row_off=torch.tensor([0, N], dtype=torch.int64), prefix_len=torch.zeros(1, dtype=torch.int32))
    row_off, prefix_len, Kb, Vb, Qb = parity.host_arrays(c)
    want = ref.compress(rp, row_off, prefix_len, Kb, Vb, Qb, scores=s)
    assert int((want["role"] == ref.SEED).sum()) == M and int((want["assign"] >= 0).sum()) == N   # every donor folds
    out = cask.compress(parity.to_device(c, p), scores=torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(out.assign.cpu().numpy(), want["assign"])


@pytest.mark.parametrize("form", ["chosen", "wide", "one_launch"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("keys,splits", [((100, 104), 1), ((100, 300), 2), ((110, 300), 1)])
def test_scores_where_only_the_sum_of_shares_leaves_the_range(keys, splits, dtype, d, form):
    """Two keys 127.5 octaves above all others, seen by two lanes or by two key splits: each share of a row's sum
    still fits fp32 against its first logit, their total does not.  Every row then gives half its mass to
    either key, 2^-129 to any other."""
    N, Wn, G = 512, 40, 2
    K = torch.zeros(N, d)
    K[list(keys), 3] = 127.5
    Q = torch.zeros(1, Wn, G, d)
    Q[..., 3] = 1.0
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    c = dict(K=K.to(dt), V=K.to(dt), Q=Q.to(dt), row_off=torch.tensor([0, N], dtype=torch.int64), prefix_len=torch.zeros(1, dtype=torch.int32))
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60,
                    softmax_scale=float(np.log(2.0)), score_splits=splits, path_flags=SCORE_FORMS[form])
    got = cask.score(parity.to_device(c, p)).cpu().double()
    want = torch.zeros(N, dtype=torch.float64)
    want[list(keys)] = 0.5
    assert float((got - want).abs().max()) < 1e-4   # (a log-sum-exp of 128.5 in fp32: 2^-17 of an octave)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("small", ["keys", "queries"])
@pytest.mark.parametrize("e", [100, 112, 118])
def test_fp32_scores_at_the_lower_end_of_the_range(e, small, d):
    """One operand near 2^-e, the other near 2^e: from about 2^-109 on the smaller one's terms do not all fit bf16,
    and the larger one sends its workgroups to the fp32 tiles.  Error against 64-bit sums as for ordinary
    values (bound: test_fp32_scores_from_bf16_terms)."""
    G, Wn, n, units = 4, 64, 1000, 4
    c = _units([n] * units, [n // 8] * units, head_dim=d, q_per_kv=G, window=Wn)
    noise = torch.Generator().manual_seed(d + e)
    c = {k: (v.float() * (1 + 1e-3 * torch.randn(v.shape, generator=noise)) if k in ("K", "V", "Q") else v) for k, v in c.items()}
    s = e if small == "queries" else -e
    c["K"], c["Q"] = c["K"] * 2.0 ** s, c["Q"] * 2.0 ** -s
    want = _scores64(c, units, n, d, G, Wn)
    p = cask.Params(dtype=cask.F32, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60)
    got = cask.score(parity.to_device(c, p)).cpu().double()
    err = float((got - want).norm() / want.norm())
    _note(e, small, d, "error", err)
    assert err < 4e-7


@pytest.mark.parametrize("N", [36864, 36865])
def test_more_than_32767_seeds_in_one_chunk_of_the_walk(N):
    """A unit that keeps 34 000 seeds and next to nothing else: the walk's packed count of seeds passes the sign
    bit of a word (36 864 rows are its largest chunk; one row more takes the keys in chunks)."""
    rng = np.random.default_rng(N)
    Wn, M = 32, 34000
    sc = rng.permutation(N).astype(np.float32)
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=1, window=Wn, budget=Wn + M, core=0, prefix_budget=0, sim_threshold=2.0)
    K = torch.from_numpy(rng.standard_normal((N, 64)).astype(np.float32)).to(torch.bfloat16).cuda()
    b = cask.Batch(p, torch.tensor([0, N], dtype=torch.int64), torch.zeros(1, dtype=torch.int32), K, K,
                   torch.zeros(1, Wn, 1, 64, dtype=torch.bfloat16, device="cuda"))
    out = cask.compress(b, scores=torch.from_numpy(sc).cuda())
    torch.cuda.synchronize()
    top = np.argsort(-sc[: N - Wn], kind="stable")[:M]
    rows = np.concatenate([np.sort(top), np.arange(N - Wn, N)])
    assert int(out.out_len[0]) == M + Wn and np.array_equal(out.out_src[0].cpu().numpy(), rows)
    want = np.full(N, -1)
    want[rows] = np.arange(M + Wn)
    assert np.array_equal(out.assign.cpu().numpy(), want)
    assert torch.equal(out.K_out[0].cpu(), K.cpu()[rows])


def test_diagnostics_are_tensors_of_their_own():
    """Dispersion and lost mass share no storage: either can be resized, saved or kept without the other."""
    c = _units([700, 900], [40, 0], head_dim=64, q_per_kv=1, window=32)
    b = parity.to_device(c, cask.Params(head_dim=64, q_per_kv=1, window=32, budget=140))
    out = cask.compress(b)
    for t in B.group_diagnostics(b, out.scores, out.assign, out.K_out):
        assert t._base is None and t.untyped_storage().nbytes() == 2 * 4


def test_grouping_and_fold_with_the_most_seeds_a_share_can_hold():
    """129 units and more take two workgroups each; with 1024 seeds a unit either holds 512, the largest workspace
    in LDS that grouping and fold in one launch ask for (no limit is raised for it); against the oracle."""
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=130, prefix=0, decode=1300, budget=1056, core=16, head_dim=64, q_per_kv=1, window=16,
                      cluster_frac=0.5)
    p = parity.params_of(w, sim_threshold=0.3)
    assert cask.plan(p, 0, 1300)["seeds"] == 1024
    _note(parity.full_check(caches.make(w, seed=77), p, expect_folds=True))


@pytest.mark.parametrize("decode,launches", [(8100, 1), (8300, 2)])
def test_stage_timing_of_the_fold(decode, launches):
    """Every donor folds: with up to 8192 decode rows the grouping launch folds too and the last stage is an empty
    event pair, with more the last stage is the folding launch (empty pairs cost some microseconds, the fold of
    16 000 rows several times that)."""
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=2, prefix=0, decode=decode)
    b = parity.to_device(caches.make(w), parity.params_of(w, sim_threshold=-1.0))
    out = cask.compress(b)
    torch.cuda.synchronize()
    B.timing_enable(20)
    for _ in range(20):
        cask.compress(b, out)
    ms, n = B.timing_read()
    B.timing_enable(0)
    _note(decode, {k: round(v * 1e3, 1) for k, v in ms.items()}, "us a call")
    assert n == 20 and ms["gather"] > 2 * ms["index_roles"]      # (the walk runs in the selection: an empty pair)
    if launches == 1:
        assert ms["emit"] < 2 * ms["index_roles"]
    else:
        assert ms["emit"] > 2 * ms["index_roles"]


def _planted_folds(rng, N, Wn, n_core, M, sizes, d, zero=False):
    """A unit whose seed j has exactly sizes[j] donors (its key, scaled): K, V, scores.  `zero`: all scores are zero,
    so that rank is by row, and every group is averaged by its rows' counts."""
    K = rng.integers(-4, 5, (N, d)).astype(np.float32)
    V = rng.integers(-4, 5, (N, d)).astype(np.float32)
    s = (1e-3 * (1.0 + rng.permutation(N))).astype(np.float32) / N       # distinct, small
    free = np.arange(N - Wn) if zero else rng.permutation(N - Wn)
    core, seeds, rest = free[:n_core], free[n_core:n_core + M], rng.permutation(free[n_core + M:])
    s[core] = 0.5 + 1e-3 * np.arange(n_core, dtype=np.float32)
    s[seeds] = 0.25 + 1e-3 * np.arange(M, dtype=np.float32)
    at = 0
    for j, n in enumerate(sizes):
        K[rest[at:at + n]] = K[seeds[j]] * np.where(np.arange(n) % 2 == 1, 2.0, 1.0)[:, None]   # cosine 1 with that seed
        at += n
    return K, V, np.zeros_like(s) if zero else s


@pytest.mark.parametrize("longest", [8100, 8300])
@pytest.mark.parametrize("n_fold,dtype,d", [(1, "bf16", 128), (63, "f32", 64), (64, "bf16", 128), (64, "f32", 128), (65, "bf16", 64), (65, "f32", 128)])
def test_step_folds_in_one_launch_and_in_two(n_fold, dtype, d, longest):
    """Groups of 1, 63, 64, 65, 200 and 1500 donors, a unit where n_fold donors fold (the short list's 64 entries),
    and a unit without score mass, all as a step with counts in and out and rows behind the budget: up to 8192
    rows of decode trace one launch groups and folds, with more two do.  Scores injected; against the oracle."""
    Wn, n_core, M = 64, 20, 16
    rng = np.random.default_rng(n_fold + longest)
    spread = [n_fold // M + (j < n_fold % M) for j in range(M)]
    made = [_planted_folds(rng, 3000, Wn, n_core, M, [1, 63, 64, 65, 200, 1500], d), _planted_folds(rng, 2000, Wn, n_core, M, spread, d),
            _planted_folds(rng, longest, Wn, n_core, M, [3, 70, 64, 0, 900], d, zero=True)]
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    K, V, s = (np.concatenate(x) for x in zip(*made))
    cnt = rng.integers(1, 20, len(s)).astype(np.int32)
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=Wn + n_core + M, core=n_core,
                    prefix_budget=0, sim_threshold=0.999)
    S = p.budget + 37
    c = dict(K=torch.from_numpy(K).to(dt), V=torch.from_numpy(V).to(dt), Q=torch.zeros(3, Wn, 1, d, dtype=dt),
             row_off=torch.tensor(np.cumsum([0] + [len(m[0]) for m in made]), dtype=torch.int64), prefix_len=torch.zeros(3, dtype=torch.int32))
    row_off, plen, Kb, Vb, Qb = parity.host_arrays(c)
    rp = parity.ref_params(p)
    want = ref.compress_step(rp, row_off, plen, Kb, Vb, Qb, in_count=cnt, scores=s, out_stride_rows=S)
    folded = [int((want["assign"][row_off[u]:row_off[u + 1]] >= 0).sum() - want["out_len"][u]) for u in range(3)]
    assert folded == [1893, n_fold, 1037], folded
    b = parity.to_device(c, p)
    for rep in range(2):
        out = cask.Outputs(b)
        Ko = torch.zeros(3, S, d, dtype=dt, device="cuda")
        Vo = torch.zeros_like(Ko)
        oc = torch.zeros(3, p.budget, dtype=torch.int32, device="cuda")
        cask.compress_step(b, Ko, Vo, out, in_count=torch.from_numpy(cnt).cuda(), out_count=oc, scores=torch.from_numpy(s).cuda())
        torch.cuda.synchronize()
        got = dict(K_out=caches.host_bits(Ko), V_out=caches.host_bits(Vo), out_len=out.out_len.cpu().numpy(), out_src=out.out_src.cpu().numpy(),
                   out_mass=out.out_mass.cpu().numpy(), assign=out.assign.cpu().numpy(), status=out.status.cpu().numpy(), count=oc.cpu().numpy())
        assert rep == 0 or all(np.array_equal(got[k], first[k]) for k in got)          # the same bits on a second run
        first = got
    for k in ("out_len", "out_src", "assign", "status"):
        assert np.array_equal(got[k], want[k]), k
    assert np.array_equal(got["count"], want["out_count"])
    assert not got["K_out"][:, p.budget:].any() and not got["V_out"][:, p.budget:].any()   # rows behind the output stay untouched
    assert parity.check_values(p, got, want, Kb.reshape(-1, d), Vb.reshape(-1, d), row_off) == 6 + min(n_fold, M) + 4


@pytest.mark.parametrize("longest", [8100, 8300])
def test_dedup_step_in_one_launch_and_in_two(longest):
    """De-duplicated seeding (fewer seeds than places may result), counts in and out, a row stride beyond the budget;
    grouping and fold in one launch and in two, on injected scores against the oracle."""
    c = _units([1500, longest], [70, 0], cluster_frac=0.6)
    row_off, plen, K, V, Q = parity.host_arrays(c)
    cnt = np.random.default_rng(12).integers(1, 6, int(row_off[-1])).astype(np.int32)
    for dt in (0.0, 0.013, -0.017, 0.031, -0.029, 0.047):
        p = cask.Params(dtype=cask.BF16, head_dim=128, q_per_kv=c["Q"].shape[2], window=c["Q"].shape[1], budget=320, sim_threshold=0.8 + dt, seed_dedup=4)
        rp = parity.ref_params(p)
        s = ref.score(rp, row_off, K, Q)
        role0, _ = ref.prefix_evict(rp, row_off, plen, s)
        if ref.partition_keys(rp, row_off, plen, K, s, role0)[2].min() >= 1e-3:
            break
    else:
        pytest.fail("no clear threshold for this cache")
    S = 448
    want = ref.compress_step(rp, row_off, plen, K, V, Q, in_count=cnt, scores=s, out_stride_rows=S)
    _, best, second = ref.consolidate(rp, row_off, plen, K, s, want["role"], want_sims=True)
    b = parity.to_device(c, p)
    out = cask.Outputs(b)
    Ko = torch.zeros(2, S, 128, dtype=torch.bfloat16, device="cuda")
    Vo, oc = torch.zeros_like(Ko), torch.zeros(2, p.budget, dtype=torch.int32, device="cuda")
    cask.compress_step(b, Ko, Vo, out, in_count=torch.from_numpy(cnt).cuda(), out_count=oc, scores=torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    got = dict(K_out=caches.host_bits(Ko), V_out=caches.host_bits(Vo), out_len=out.out_len.cpu().numpy(), out_src=out.out_src.cpu().numpy(),
               out_mass=out.out_mass.cpu().numpy(), assign=out.assign.cpu().numpy())
    assert np.array_equal(got["out_len"], want["out_len"])
    for u in range(2):
        L, sl = int(want["out_len"][u]), slice(row_off[u], row_off[u + 1])
        assert np.array_equal(got["out_src"][u, :L], want["out_src"][u, :L])
        excused = parity.check_assign_excused(got["assign"][sl], want["assign"][sl], best[sl], second[sl], float(np.float32(p.sim_threshold)), f"unit {u}")
        if excused == 0:
            assert np.array_equal(oc.cpu().numpy()[u, :L], want["out_count"][u, :L])
    assert parity.check_values(p, got, want, K.reshape(-1, 128), V.reshape(-1, 128), row_off) >= 5


@pytest.mark.parametrize("P", [0, 1, 4096, 4097, 6145, 36865])
def test_prefix_stage_of_units_much_longer_than_their_prefixes(P):
    """Stage 1 alone takes the instance of the selection that its longest prefix needs, whatever the units hold
    behind it: edges of the instances, ties at the rank, a unit without a prefix; roles behind a prefix are
    left as they are."""
    rng = np.random.default_rng(P)
    lens, pref = [40000, 3000, 20000], [P, min(P, 900), 0]
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    sc = np.floor(rng.random(int(row_off[-1])) * 300).astype(np.float32) / 300
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=1, window=64, budget=900, prefix_budget=600)
    prefix = np.array(pref, dtype=np.int32)
    want, _ = ref.prefix_evict(parity.ref_params(p), row_off, prefix, sc)
    K = torch.zeros(int(row_off[-1]), 64, dtype=torch.bfloat16, device="cuda")
    b = cask.Batch(p, torch.from_numpy(row_off), torch.from_numpy(prefix), K, K, torch.zeros(3, 64, 1, 64, dtype=torch.bfloat16, device="cuda"))
    role, _ = cask.prefix_evict(b, torch.from_numpy(sc).cuda(), torch.full((int(row_off[-1]),), 77, dtype=torch.uint8, device="cuda"))
    role = role.cpu().numpy()
    for u in range(3):
        lo, mid, hi = row_off[u], row_off[u] + pref[u], row_off[u + 1]
        assert np.array_equal(role[lo:mid], want[lo:mid]) and (role[mid:hi] == 77).all()


@pytest.mark.parametrize("D", [64, 65, 4096, 4097, 6145, 36865])
def test_decode_stage_of_units_much_longer_than_their_traces(D):
    """Stage 2 alone reads its keys from behind the prefix and takes the instance that its longest trace needs:
    edges of the instances, ties at the ranks, a unit that is all trace, one whose trace is all kept; roles in
    front are left as they are."""
    rng = np.random.default_rng(D)
    lens, trace = [40000, 3000, 20000], [D, min(D, 3000), min(D, 700)]
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    prefix = np.array([n - t for n, t in zip(lens, trace)], dtype=np.int32)
    sc = np.floor(rng.random(int(row_off[-1])) * 300).astype(np.float32) / 300
    p = cask.Params(dtype=cask.BF16, head_dim=64, q_per_kv=1, window=64, budget=900, prefix_budget=100)
    want, _ = ref.partition(parity.ref_params(p), row_off, prefix, sc, np.full(int(row_off[-1]), 77, dtype=np.uint8))
    K = torch.zeros(int(row_off[-1]), 64, dtype=torch.bfloat16, device="cuda")
    b = cask.Batch(p, torch.from_numpy(row_off), torch.from_numpy(prefix), K, K, torch.zeros(3, 64, 1, 64, dtype=torch.bfloat16, device="cuda"))
    role, _ = cask.partition(b, torch.from_numpy(sc).cuda(), torch.full((int(row_off[-1]),), 77, dtype=torch.uint8, device="cuda"))
    assert np.array_equal(role.cpu().numpy(), want)


@pytest.mark.parametrize("theta,radius", [(float("inf"), 0), (1e6, 60), (999999.0, 60)])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
def test_band_distances_without_a_screen(dtype, d, theta, radius):
    """Thresholds that fold every donor (within the radius) into its nearest seed: the form without the screen, from
    1e6 on, and the last threshold with it; blocks of 32 seeds and a remainder, a last tile of rows."""
    Wn = 32
    w = caches.scaled(W["cfg2"], n_layers=1, n_kv_heads=2, prefix=30, decode=590, budget=230, head_dim=d, q_per_kv=1, window=Wn, cluster_frac=0.5)
    c = caches.make(w, seed=d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    c = {k: (v.to(dt) if k in ("K", "V", "Q") else v) for k, v in c.items()}
    band = torch.rand(d // 2, generator=torch.Generator().manual_seed(d)) ** 2
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=1, window=Wn, budget=230, core=100, merge_geometry=1,
                    band_weight=band.cuda(), dist_threshold=theta, merge_radius=radius)
    _note(dtype, d, theta, parity.full_check(c, p, expect_folds=True))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,Wn,splits", [(2, 16, 0), (1, 4, 3), (4, 64, 0)])
def test_fp32_scores_with_steep_logits(G, Wn, splits, d):
    """Keys thirty times as long: logits hundreds of octaves apart, so that most sums leave the range of their
    first reference and are taken again.  A logit has the same bits in both sweeps, so that its own rounding
    cancels in the one key that has a row's mass; what is left is half an ulp of the row's log-sum-exp L, twice
    (as it is rounded, and as a maximum that it is added to): at most 2^-24 |L| ln 2 of a score."""
    n, units = 1200, 3
    g = torch.Generator().manual_seed(d + Wn)
    K, Q = 30.0 * torch.randn(units * n, d, generator=g), 4.0 * torch.randn(units, Wn, G, d, generator=g)
    c = dict(K=K, V=K, Q=Q, row_off=torch.arange(units + 1, dtype=torch.int64) * n, prefix_len=torch.zeros(units, dtype=torch.int32))
    want = _scores64(c, units, n, d, G, Wn)
    top = float((Q.double().reshape(units, -1, d) @ K.double().reshape(units, n, d).transpose(1, 2).contiguous()).max() / d ** 0.5 / np.log(2.0))
    p = cask.Params(dtype=cask.F32, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60, score_splits=splits)
    got = cask.score(parity.to_device(c, p)).cpu().double()
    err = float((got - want).norm() / want.norm())
    _note(G, Wn, d, "largest logit", top, "octaves, error", err, "bound", 2.0 ** -24 * top * np.log(2.0))
    assert err < 2.0 ** -24 * top * np.log(2.0)


@pytest.mark.parametrize("form", ["chosen", "wide", "one_launch"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("late,splits", [(100, 1), (104, 1), (300, 2)])
def test_scores_of_a_share_far_below_another_ones_reference(late, splits, dtype, d, form):
    """A lane (a key split) whose first logits are 0 and whose sum then reaches 2^119, beside a lane that starts at
    127: the first one's reference lies 127 to 143 octaves below the second's, beyond what fp32's exponent
    takes in one step, and its key still has 1/257 of every row."""
    N, Wn, G = 512, 40, 2
    K = torch.zeros(N, d)
    first = 0 if late == 100 else 4   # (a lane holds keys 0 - 3, or 4 - 7, of every eight)
    K[first, 3], K[late, 3] = 127.0, 119.0
    Q = torch.zeros(1, Wn, G, d)
    Q[..., 3] = 1.0
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    c = dict(K=K.to(dt), V=K.to(dt), Q=Q.to(dt), row_off=torch.tensor([0, N], dtype=torch.int64), prefix_len=torch.zeros(1, dtype=torch.int32))
    p = cask.Params(dtype=cask.F32 if dtype == "f32" else cask.BF16, head_dim=d, q_per_kv=G, window=Wn, budget=Wn + 60,
                    softmax_scale=float(np.log(2.0)), score_splits=splits, path_flags=SCORE_FORMS[form])
    got = cask.score(parity.to_device(c, p)).cpu().double()
    want = torch.zeros(N, dtype=torch.float64)
    want[first], want[late] = 256.0 / 257.0, 1.0 / 257.0
    assert float((got - want).abs().max()) < 2e-5   # (a log-sum-exp of 127 in fp32, and a logit of 127: 2^-18 of an octave each)
