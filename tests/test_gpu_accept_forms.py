"""The two forms in which the accept pass keeps the shifted row p_hat ~ exp(z/T + eta (q - p)): multiples of the kept
exponentials up to eta = 20, logarithms above.  Both around the switch, with every slice size, at low temperature (where
exponentials underflow), with masked parts of the vocabulary (-inf and the lowest float), with and without supplied row
statistics, and with every exchange recomputed: against the oracle, and bit for bit between the runs."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2502_20330_amd import binding
from paper_2502_20330_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _masked(acc, kind):
    zt, zd = acc.target_logits, acc.draft_logits
    low = {"none": None, "inf": -np.inf, "lowest": np.finfo(np.float32).min}[kind]
    if low is None:
        return acc
    # a whole slice of either row and scattered entries; never a drafted token
    for z in (zt, zd):
        z[:, :, 16384:33000] = low
        z[:, :, 5::97] = low
    keep = np.arange(zt.shape[2])
    keep = keep[(keep % 97 != 5) & ((keep < 16384) | (keep >= 33000))]
    rng = np.random.default_rng(9)
    best = keep[np.argsort(-zd[:, :, keep], axis=-1)[..., :6]]
    acc.draft_tokens[:] = np.take_along_axis(best, rng.integers(0, 6, acc.draft_tokens.shape)[..., None], -1)[..., 0]
    return acc


def _chunk_stats(z, chunk, T):
    rows = z.reshape(-1, z.shape[-1]).astype(np.float64)
    n = -(-rows.shape[1] // chunk)
    rows = np.pad(rows, ((0, 0), (0, n * chunk - rows.shape[1])), constant_values=-np.inf).reshape(len(rows), n, chunk)
    m = rows.max(-1)
    with np.errstate(invalid="ignore", over="ignore"):
        e = np.where(np.isfinite(rows), np.exp((rows - np.where(np.isfinite(m), m, 0.0)[..., None]) / T), 0.0)
    return torch.from_numpy(np.stack([m, e.sum(-1)], -1).astype(np.float32)).cuda()


@pytest.mark.parametrize("slice_entries", [4096, 8192, 10240, 16384, 0])    # 0: the library's choice at 24 sequences, 10240 or 16384
@pytest.mark.parametrize("eta,T,mask", [(20.0, 0.1, "none"), (20.5, 0.1, "none"), (20.0, 1.0, "inf"), (20.5, 1.0, "inf"),
                                        (1.0, 0.1, "lowest"), (50.0, 0.7, "lowest"), (0.0, 0.05, "inf")])
def test_both_forms_match_the_oracle_and_each_other(slice_entries, eta, T, mask):
    cfg = wl.scaled(wl.CONFIGS["llama8b_32k"], batch=4 if slice_entries else 24, vocab=50257, gamma_choices=(2, 4), eta=eta, temperature=T, name="forms")
    acc = _masked(wl.gen_accept_inputs(cfg, salt=31), mask)
    r = gu.rapid()
    runs = []
    try:
        r.set_option(binding.OPT_ACCEPT_SLICE, slice_entries)
        for wait in (100, 0, 2):
            r.set_option(binding.OPT_ACCEPT_WAIT_US, wait)
            gpu, ref = gu.run_accept_case(acc, eta=eta, temperature=T)
            runs.append(gpu)
            assert wait > 0 or r.accept_status()[1] > 0           # the exchanges were recomputed
        r.set_option(binding.OPT_ACCEPT_WAIT_US, 100)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        for side in ((True, True), (True, False), (False, True)):
            out = r.rapid_accept(dev(acc.target_logits), dev(acc.draft_logits), dev(acc.draft_tokens), eta, dev(acc.uniforms),
                                 gammas=dev(acc.gammas), temperature=T,
                                 target_stats=_chunk_stats(acc.target_logits, 1000, T) if side[0] else None,
                                 draft_stats=_chunk_stats(acc.draft_logits, 1000, T) if side[1] else None)
            torch.cuda.synchronize()
            runs.append(tuple(t.cpu().numpy() for t in out))
    finally:
        r.set_option(binding.OPT_ACCEPT_WAIT_US, 100)
        r.set_option(binding.OPT_ACCEPT_SLICE, 0)
    for other in runs[1:3]:
        assert all(np.array_equal(x.view(np.int32), y.view(np.int32)) for x, y in zip(runs[0], other))
    for gpu in runs:
        st = gu.compare_accept(gpu, ref, acc.gammas, cfg.gamma_max)
        assert st["n_mismatch"] == 0 and st["token_mismatch"] == 0 and st["exempt_sequences"] == 0, st
        # fp32 arguments of the exponentials: |z - max| / T up to 30 / 0.05 at 2^-24, a few times over
        assert st["max_ratio_rel_err"] <= 1e-4, st


@pytest.mark.parametrize("V", [1, 3, 4095, 4097, 8193, 50257])
def test_greedy_ties_masks_and_row_ends(V):
    """Equal maxima in one thread, across threads and across slices (lowest index), rows that are -inf from some point on
    or throughout, maxima at the ends of rows of any alignment."""
    rng = np.random.default_rng(V)
    B, g = 5, 3
    zt = rng.integers(-3, 4, (B, g + 1, V)).astype(np.float32)             # many ties
    zd = rng.integers(-3, 4, (B, g, V)).astype(np.float32)
    zt[1, :, V // 2:] = -np.inf
    zt[2, 1] = -np.inf
    zd[3, 0] = -np.inf
    zt[4, :, -1] = 9.0
    zt[4, 2, 0] = 9.0
    tok = np.argmax(zd, -1).astype(np.int32)
    u = rng.random((B, g + 1), dtype=np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n, toks, _ = gu.rapid().rapid_accept(dev(zt), dev(zd), dev(tok), 1.0, dev(u), temperature=0.0)
    torch.cuda.synchronize()
    n, toks = n.cpu().numpy(), toks.cpu().numpy()
    with np.errstate(invalid="ignore"):
        for b in range(B):
            want = g
            for k in range(g):
                a, c = zt[b, k, tok[b, k]] - zt[b, k].max(), zd[b, k, tok[b, k]] - zd[b, k].max()
                rho = np.inf if a > c else (0.0 if a < c else 1.0)         # (a NaN gap compares as equal)
                if not u[b, k] <= min(1.0, rho):
                    want = k
                    break
            assert n[b] == want, (b, n, want)
            assert list(toks[b, :want]) == list(tok[b, :want]) and toks[b, want] == int(np.argmax(zt[b, want]))
            assert np.all(toks[b, want + 1:] == -1)


@pytest.mark.parametrize("batch,V,slices", [(1, 20000, 20), (1, 100001, 49), (6, 100001, 25), (15, 50257, 50), (24, 50257, 13), (44, 50257, 17), (48, 50257, 10),
                                            (600, 1030, 1)])
def test_every_build_of_the_draw_and_its_give_up_path(batch, V, slices):
    """Vocabularies and batches that select 256 threads of 4 (one and up to three workgroups per compute unit) and 8 entries, 512 of 8 (one round of one
    and of two workgroups per compute unit), 256 of 12 (up to three) and 20, a row end inside a thread's entries; with every exchange recomputed the results are the same bits, and it is every one:
    each of a sequence's `slices` workgroups gives up on all slices in each of the draw's exchanges (three, one for a bonus row)."""
    cfg = wl.scaled(wl.CONFIGS["llama8b_32k"], batch=batch, vocab=V, gamma_choices=(0, 1), draft_noise_std=2.0, name="draws")
    acc = wl.gen_accept_inputs(cfg, salt=V)
    r = gu.rapid()
    runs = []
    try:
        for wait in (100, 0, 2):
            r.set_option(binding.OPT_ACCEPT_WAIT_US, wait)
            gpu, ref = gu.run_accept_case(acc, eta=cfg.eta)
            runs.append(gpu)
            if wait == 0:
                bonus = int((gpu[0] == acc.gammas).sum())
                assert gu.draw_giveups(r) == slices ** 2 * (3 * (batch - bonus) + bonus)
    finally:
        r.set_option(binding.OPT_ACCEPT_WAIT_US, 100)
    for other in runs[1:]:
        assert all(np.array_equal(x.view(np.int32), y.view(np.int32)) for x, y in zip(runs[0], other))
    st = gu.compare_accept(runs[0], ref, acc.gammas, cfg.gamma_max)
    assert st["n_mismatch"] == 0 and st["token_mismatch"] == 0 and st["exempt_sequences"] == 0, st


@pytest.mark.parametrize("batch,V,slices", [(61, 50257, 13), (65, 49152, 12), (1025, 1030, 1)])
def test_draws_beyond_one_round_of_workgroups(batch, V, slices):
    """The build of 16 entries (17 and 16 slices of 12 entries a sequence no longer fit four workgroups to a compute unit): slices that end
    inside a thread's entries and with the row, and one slice per sequence; the give-up path included."""
    test_every_build_of_the_draw_and_its_give_up_path(batch, V, slices)


@pytest.mark.parametrize("g", [1023, 1024, 1100, 20000])
def test_greedy_with_thousands_of_drafted_positions(g):
    """More positions than the decision keeps arg-maxima for in LDS: all accepted, and rejected at the last one."""
    rng = np.random.default_rng(g)
    V = 7
    zt = rng.standard_normal((2, g + 1, V)).astype(np.float32)
    zd = zt[:, :g].copy()
    tok = np.argmax(zd, -1).astype(np.int32)
    tok[1, g - 1] = -5                                        # outside the vocabulary: rejected
    u = np.full((2, g + 1), 0.5, dtype=np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n, toks, _ = gu.rapid().rapid_accept(dev(zt), dev(zd), dev(tok), 1.0, dev(u), temperature=0.0)
    torch.cuda.synchronize()
    n, toks = n.cpu().numpy(), toks.cpu().numpy()
    assert list(n) == [g, g - 1]
    for b in range(2):
        np.testing.assert_array_equal(toks[b, :n[b]], tok[b, :n[b]])
        assert toks[b, n[b]] == int(np.argmax(zt[b, n[b]])) and np.all(toks[b, n[b] + 1:] == -1)


@pytest.mark.parametrize("eta", [1e6, 2.2e7, 6e7, 1e8, 2e8, 3e8, 1e12, 1e30])
def test_shift_of_any_size(eta):
    """A shift eta (q - p) far past the range of the exponential.  Token 0 (q = 0.9, p = 0.5) takes all of p_hat, so its residual
    max(p - p_hat, p - q, 0) is 0 and it is never drawn after a reject; the others (q < p) keep p, the draw is theirs.  The
    last token, p = q = 1e-30, keeps p_hat's normaliser above zero whatever the shift makes of token 0."""
    V, B = 101, 64
    p = np.concatenate([[0.5], np.full(99, 0.5 / 99), [1e-30]])
    q = np.concatenate([[0.9], np.full(99, 0.1 / 99), [1e-30]])
    zt = np.broadcast_to(np.log(p).astype(np.float32), (B, 2, V))
    zd = np.broadcast_to(np.log(q).astype(np.float32), (B, 1, V))
    u = np.stack([np.full(B, 0.5), (np.arange(B) + 0.5) / B], 1).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n, toks, ratio = gu.rapid().rapid_accept(dev(zt), dev(zd), torch.full((B, 1), 3, dtype=torch.int32, device="cuda"), eta,
                                             dev(u), tail_alpha=0.0)
    torch.cuda.synchronize()
    assert not n.any() and not ratio.any()                     # p_hat of the drafted token is 0
    want = 1 + np.floor(u[:, 1] * 99)                          # 99 equal weights, and u stays clear of their edges
    np.testing.assert_array_equal(toks[:, 0].cpu().numpy(), want)


@pytest.mark.parametrize("eta", [0.0, 1.0, 20.0, 25.0])
@pytest.mark.parametrize("slice_entries", [4096, 8192, 10240, 16384])
def test_a_nan_logit_costs_its_slice_only(slice_entries, eta):
    """One NaN in a target row, a draft row or both: sums leave out the slice that holds it, so the ratio stays finite and the
    accept test can still reject (a NaN ratio would accept every draft).  Expected ratios in float64 with that slice taken
    out; the tail rule is off, so that no maximum enters."""
    V, g, at = 50257, 3, 20000
    rng = np.random.default_rng(3)
    zt = (4 * rng.standard_normal((3, g + 1, V))).astype(np.float32)
    zd = (zt[:, :g] + rng.standard_normal((3, g, V))).astype(np.float32)
    tok = np.argsort(-zd, -1)[..., 5].astype(np.int32)
    u = np.full((3, g + 1), 0.999, dtype=np.float32)
    zt[[0, 2], 1, at] = np.nan
    zd[[1, 2], 1, at] = np.nan
    want = np.empty((3, g))
    size = 8192 if slice_entries == 10240 and eta > 20 else slice_entries
    lo = at // size * size
    for b in range(3):
        for k in range(g):
            t, d = zt[b, k].astype(np.float64), zd[b, k].astype(np.float64)
            with np.errstate(invalid="ignore"):
                et, ed = np.exp(t - np.nanmax(t)), np.exp(d - np.nanmax(d))
            out = np.zeros(V, dtype=bool)
            out[lo:lo + size] = True
            p = et / (et[~out] if np.isnan(t).any() else et).sum()
            q = ed / (ed[~out] if np.isnan(d).any() else ed).sum()
            f = p * np.exp(eta * (q - p))
            ph = f / (f[~out] if np.isnan(t).any() or np.isnan(d).any() else f).sum()
            want[b, k] = ph[tok[b, k]] / q[tok[b, k]]
    assert np.all(np.isfinite(want)) and np.all(np.abs(np.minimum(want, 1) - 0.999) > 1e-3) and (want[:, 1] < 0.9).any()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    r = gu.rapid()
    try:
        r.set_option(binding.OPT_ACCEPT_SLICE, slice_entries)
        for wait in (100, 0):
            r.set_option(binding.OPT_ACCEPT_WAIT_US, wait)
            n, toks, ratio = r.rapid_accept(dev(zt), dev(zd), dev(tok), eta, dev(u), tail_alpha=0.0)
            torch.cuda.synchronize()
            np.testing.assert_allclose(ratio.cpu().numpy(), want, rtol=1e-4)
            for b in range(3):
                fail = np.flatnonzero(want[b] < 0.999)
                assert int(n[b]) == (fail[0] if len(fail) else g)
    finally:
        r.set_option(binding.OPT_ACCEPT_WAIT_US, 100)
        r.set_option(binding.OPT_ACCEPT_SLICE, 0)


@pytest.mark.parametrize("slice_entries", [4096, 8192, 10240, 16384])
@pytest.mark.parametrize("supplied", [False, True])
def test_slices_are_combined_in_float64(slice_entries, supplied):
    """Every slice of a target row holds one value, a different distance below the maximum, and eta = 0: sums inside a slice
    are whole numbers, so all that rounds is the way from the slices' scale to the row's.  With that in float64 the ratio is
    the float64 value to the last bit of its own float32 (2^-24), where float32 exponentials of distances up to 12 are off
    by as much as half a unit of 2^-20 in the argument."""
    rng = np.random.default_rng(6)
    B, W = 32, 4
    V = W * slice_entries
    a = rng.uniform(0.5, 12.0, (B, 2, W))
    a[:, :, 0] = 0.0
    zt = np.repeat(-a.astype(np.float32), slice_entries, -1)
    zt[:, :, 1:slice_entries] = -np.inf                       # the maximum itself: one entry, so that the others weigh
    zd = np.zeros((B, 1, V), dtype=np.float32)
    tok = rng.integers(slice_entries, V, (B, 1)).astype(np.int32)
    u = rng.random((B, 2), dtype=np.float32)
    e = np.exp(zt[:, 0].astype(np.float64))
    want = np.take_along_axis(e, tok, -1) / e.sum(-1, keepdims=True) * V
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    r = gu.rapid()
    try:
        r.set_option(binding.OPT_ACCEPT_SLICE, slice_entries)
        stats = _chunk_stats(zt, slice_entries, 1.0) if supplied else None
        _, _, ratio = r.rapid_accept(dev(zt), dev(zd), dev(tok), 0.0, dev(u), tail_alpha=0.0, target_stats=stats)
        torch.cuda.synchronize()
    finally:
        r.set_option(binding.OPT_ACCEPT_SLICE, 0)
    err = np.abs(ratio.cpu().numpy().astype(np.float64) / want - 1)
    bound = 2.0 ** -24 + 1e-12
    if supplied:                                              # the entries then carry the distance themselves, in float32
        bound += 2.0 ** -20
    assert err.max() <= bound, err.max()


@pytest.mark.parametrize("eta", [0.5, 20.0, 30.0])
@pytest.mark.parametrize("excess", [0.0, 60.0, 100.0, 124.0, 400.0])
def test_the_maximum_of_an_empty_chunk_does_not_count(eta, excess):
    """Supplied statistics may hold empty chunks (sum 0), whatever stands in their maximum: here `excess` powers of two above
    the row's own, far enough for float32 exponentials relative to it to run out of range.  Same results as the oracle's."""
    cfg = wl.scaled(wl.CONFIGS["llama8b_32k"], batch=6, vocab=20000, gamma_choices=(2, 3), eta=eta, draft_noise_std=1.0, name="empty")
    acc = wl.gen_accept_inputs(cfg, salt=8)
    acc.target_logits -= 40                                   # rows whose maxima are below 0, where a zeroed pair lies above them
    acc.draft_logits -= 40
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()

    def stats(z):
        st = _chunk_stats(z, 700, 1.0)
        empty = torch.zeros_like(st[:, :2])
        empty[..., 0] = st[..., 0].amax(1, keepdim=True) + excess * np.log(2)
        return torch.cat([empty[:, :1], st, empty[:, 1:]], 1).contiguous()

    ref = gu.run_accept_case(acc, eta=eta)[1]
    for sides in ((True, True), (True, False), (False, True)):
        got = gu.rapid().rapid_accept(dev(acc.target_logits), dev(acc.draft_logits), dev(acc.draft_tokens), eta, dev(acc.uniforms),
                                      gammas=dev(acc.gammas), target_stats=stats(acc.target_logits) if sides[0] else None,
                                      draft_stats=stats(acc.draft_logits) if sides[1] else None)
        torch.cuda.synchronize()
        res = gu.compare_accept(tuple(t.cpu().numpy() for t in got), ref, acc.gammas, cfg.gamma_max)
        assert res["n_mismatch"] == 0 and res["token_mismatch"] == 0 and res["exempt_sequences"] == 0, res
        assert res["max_ratio_rel_err"] <= 1e-4, res


@pytest.mark.parametrize("B,g,V", [(256, 0, 300), (256, 3, 300), (257, 0, 300), (257, 3, 300), (300, 11, 900), (2100, 2, 65), (40, 17, 900)])
def test_greedy_decision_of_any_number_of_waves(B, g, V):
    """The decision's waves follow the drafted positions (at most 16) and the batch (four from 257 sequences on)."""
    rng = np.random.default_rng(B + g)
    zt = rng.standard_normal((B, g + 1, V)).astype(np.float32)
    zd = (zt[:, :g] + 0.2 * rng.standard_normal((B, g, V))).astype(np.float32)
    tok = np.argmax(zd, -1).astype(np.int32)
    u = rng.random((B, g + 1), dtype=np.float32)
    gam = rng.integers(0, g + 1, B).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n, toks, ratio = gu.rapid().rapid_accept(dev(zt), dev(zd), dev(tok), 1.0, dev(u), gammas=dev(gam), temperature=0.0)
    torch.cuda.synchronize()
    ref = oracle.accept_greedy(zt, zd, tok, u, gammas=gam)
    np.testing.assert_array_equal(n.cpu().numpy(), ref.n_accepted)
    np.testing.assert_array_equal(toks.cpu().numpy(), ref.out_tokens)
    live = np.arange(g)[None, :] < gam[:, None]
    np.testing.assert_array_equal(ratio.cpu().numpy().astype(np.float64)[live], ref.ratio[live])


@pytest.mark.parametrize("T", [1.0, 0.0])
def test_ratios_past_a_sequences_drafts(T):
    """rapid_accept_filled writes all of a ratio buffer, 0 past a sequence's own drafts, whatever it held (here NaN); the binding calls it
    for a buffer that it makes.  A buffer of the caller's keeps what it holds there."""
    cfg = wl.scaled(wl.CONFIGS["llama8b_32k"], batch=6, vocab=5003, gamma_choices=(0, 1, 3), draft_noise_std=2.0, name="ratios")
    acc = wl.gen_accept_inputs(cfg, salt=7)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    gam = dev(np.asarray(acc.gammas, dtype=np.int32))
    zt, zd, tok, u = (dev(x) for x in (acc.target_logits, acc.draft_logits, acc.draft_tokens, acc.uniforms))
    r = gu.rapid()
    B, g = acc.draft_tokens.shape
    past = torch.arange(g, device="cuda")[None] >= gam[:, None]
    assert past.any() and not past.all()

    def buffers(fill):
        return (torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, g + 1), dtype=torch.int32, device="cuda"),
                torch.full((B, g), fill, device="cuda"))
    n, toks, mine = buffers(7.0)
    r.rapid_accept(zt, zd, tok, 1.0, u, gammas=gam, temperature=T, outs=(n, toks, mine))
    assert torch.equal(mine[past], torch.full_like(mine[past], 7.0))
    filled = buffers(float("nan"))
    ws = torch.zeros(r.lib.rapid_accept_workspace_bytes(r._ctx, B, g, zt.shape[2]), dtype=torch.uint8, device="cuda")
    rc = r.lib.rapid_accept_filled(r._ctx, B, g, zt.shape[2], zt.data_ptr(), zd.data_ptr(), tok.data_ptr(), gam.data_ptr(), 1.0, T, 0.1,
                                   u.data_ptr(), None, 0, None, 0, *(t.data_ptr() for t in filled), ws.data_ptr(), ws.numel(),
                                   torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    for out in (filled, r.rapid_accept(zt, zd, tok, 1.0, u, gammas=gam, temperature=T)):
        assert torch.equal(out[0], n) and torch.equal(out[1], toks)
        assert torch.equal(out[2][~past].view(torch.int32), mine[~past].view(torch.int32))
        assert torch.equal(out[2][past].view(torch.int32), torch.zeros_like(out[2][past]).view(torch.int32))


@pytest.mark.parametrize("V", [4096, 8192, 12289])
def test_greedy_rows_at_the_borders_of_slices(V):
    """One slice, two, and four with one entry in the last."""
    test_greedy_ties_masks_and_row_ends(V)


@pytest.mark.parametrize("V", [41120, 41123])
def test_greedy_batches_past_the_caches(V):
    """A call on more than 80 MiB of logits, whose rows are read with the streaming hint, against the same sequences in calls below
    the line; rows with ties, masks and a NaN, rows that are not 16-byte aligned."""
    B, g = 172, 1
    assert B * (2 * g + 1) * V * 4 > 80 << 20 > 86 * (2 * g + 1) * V * 4
    gen = torch.Generator(device="cuda").manual_seed(V)
    t = torch.randn(B, g + 1, V, device="cuda", generator=gen)
    t[::3] = t[::3].mul_(2).round_()
    t[5, :, 1000:] = -torch.inf
    t[7, 0, V - 1] = torch.nan
    d = torch.where(torch.rand(B, g, V, device="cuda", generator=gen) < 0.5, t[:, :g], t[:, :g] - 1).contiguous()
    tok = d.nan_to_num(-9).argmax(-1).to(torch.int32)
    u = torch.rand(B, g + 1, device="cuda", generator=gen)
    whole = gu.rapid().rapid_accept(t, d, tok, 0.5, u, temperature=0.0)
    for lo in (0, 86):
        part = gu.rapid().rapid_accept(*(x[lo:lo + 86] for x in (t, d, tok)), 0.5, u[lo:lo + 86], temperature=0.0)
        for a, b in zip(whole, part):
            assert torch.equal(a[lo:lo + 86].view(torch.int32), b.view(torch.int32))
    assert 0 < int(whole[0].sum()) < B
