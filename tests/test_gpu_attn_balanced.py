"""Attention of ragged batches whose total length the caller passes (balanced shares of the token stream, one
workgroup per compute unit) against the float64 oracle: lengths at the edges of a 128-token quantum and of a share,
sequences without tokens, more sequences than lanes of a wave or than shares, every layout and row count.

The hint and the bound of the lengths alone choose the route, so cases of few tokens, which the library would leave to the fixed
grid, pass larger ones than are true."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2502_20330_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _lens(kind, B, rng):
    if kind == "edges":                       # around multiples of 128 and of the shares
        base = np.array([11, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 4095, 4097, 6000])
        return np.concatenate([[6000], rng.choice(base, B - 1)])
    if kind == "one_long":                    # one sequence holds nearly all tokens
        return np.concatenate([[20011], rng.integers(11, 60, B - 1)])
    if kind == "long_last":
        return np.concatenate([rng.integers(11, 60, B - 1), [20011]])
    if kind == "empty":                       # sequences without tokens between the others, first and last included
        n = rng.integers(100, 3000, B)
        n[::3] = 0
        n[-1] = 0
        n[B // 2] = 5000
        return n
    return np.concatenate([[700], rng.integers(11, 300, B - 1)])      # short


CASES = [  # kind, batch, query heads, kv heads, head_dim, gamma choices, page, head-major
    ("edges", 6, 32, 8, 128, (4, 8), 16, True),
    ("edges", 9, 32, 8, 128, (0, 10), 0, False),
    ("edges", 5, 4, 1, 64, (4,), 0, True),
    ("edges", 7, 28, 4, 128, (9, 10), 64, True),      # 77 rows: two row teams of 3 + 2 blocks
    ("edges", 4, 64, 8, 128, (10, 11), 0, False),     # 96 rows: 3 + 3
    ("one_long", 8, 16, 8, 64, (3,), 16, False),
    ("long_last", 12, 32, 8, 128, (8,), 0, True),
    ("empty", 10, 32, 8, 128, (8,), 16, True),
    ("short", 70, 8, 2, 128, (2, 5), 0, True),        # more sequences than lanes
    ("short", 150, 16, 8, 128, (1,), 16, False),      # more sequences than shares per head
    ("edges", 5, 3, 3, 128, (4,), 0, False),          # 84 groups for 3 heads
]


def _quanta_needed(batch, hkv, d, n_cu=256):
    """Host rule: tokens in quanta of 128 from which a ragged batch runs on balanced shares."""
    groups = n_cu // hkv & ~1
    assert groups >= 16 and batch <= 256
    return (2 if d == 64 else 1) * (2 * groups + batch)


def _balanced_route(q, k, pt, lens, max_ctx, hkv):
    """(hint, max_ctx, page table) that select balanced shares: the true ones where they do."""
    B, _, _, d = q.shape
    hint = max(int(lens.astype(np.int64).clip(0).sum()), 128 * _quanta_needed(B, hkv, d))
    bound = max(max_ctx, -(-hint * 100 // (85 * B)))
    if pt is not None and bound > pt.shape[1] * k.shape[1]:
        pt = torch.nn.functional.pad(pt, (0, -(-bound // k.shape[1]) - pt.shape[1]), value=-1).contiguous()
    r = gu.rapid()
    nsplit = -(-bound // r.verify_attn_chunk(r.attn_shape(q, k, bound, page_table=pt, ctx_sum_hint=hint)))
    assert hint * 10 < B * bound * 9 and (256 // hkv & ~1) + B - 1 <= B * nsplit
    return hint, bound, pt


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c[:5]))
def test_balanced_shares_match_the_oracle(case):
    kind, B, hq, hkv, d, gch, page, head_major = case
    rng = np.random.default_rng([77, B, hq])
    lens = _lens(kind, B, rng).astype(np.int32)
    gam = rng.choice(np.asarray(gch, dtype=np.int32), size=B).astype(np.int32)
    gam = np.where(lens > 0, np.minimum(gam, np.maximum(lens, 1) - 1), gam).astype(np.int32)
    cfg = wl.scaled(wl.CONFIGS["ragged_paged"], name="balanced", batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                    gamma_choices=gch, paged=page > 0, page_size=max(page, 1))
    max_ctx = int(lens.max())
    table, n_pages = None, 0
    if page:
        need = -(-lens // page)
        n_pages = int(need.sum()) + 2
        perm = rng.permutation(n_pages).astype(np.int32)
        table = np.full((B, int(need.max())), -1, dtype=np.int32)
        at = 0
        for b, n in enumerate(need):
            table[b, :n] = perm[at:at + n]
            at += n
    inp = wl.gen_attn_inputs(cfg, layer=3, seqs=wl.Sequences(lens, gam, table, n_pages, max_ctx))
    q, k, v = gu.bf16_to_dev(inp.q), gu.bf16_to_dev(inp.k), gu.bf16_to_dev(inp.v)
    if head_major:
        k, v = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (k, v))
    pt = torch.from_numpy(table).cuda() if page else None
    ctx = torch.from_numpy(lens).cuda()
    hint, bound, wide_pt = _balanced_route(q, k, pt, lens, max_ctx, hkv)
    r = gu.rapid()
    got = []
    for h in (hint, hint, 0):                 # twice (the workspace then holds old partials), and the fixed grid of splits
        lse = torch.zeros((B, hq, cfg.q_max), dtype=torch.float32, device="cuda")
        out = r.rapid_verify_attn(q, k, v, ctx, gammas=torch.from_numpy(gam).cuda(), page_table=wide_pt if h else pt,
                                  max_ctx=bound if h else max_ctx, softmax_scale=cfg.softmax_scale, lse_out=lse, ctx_sum_hint=h)
        torch.cuda.synchronize()
        got.append((gu.bf16_to_host(out), lse.cpu().numpy().astype(np.float64)))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    bs, ts, hs, ps = wl.kv_strides(cfg, inp.seqs)
    lay = oracle.KVLayout(bs, ts, hs, page, ps, table.shape[1] if page else 0)
    live = lens > 0
    ref_lens = np.where(live, lens, 1).astype(np.int32)
    ref_gam = np.where(live, gam, 0).astype(np.int32)
    ref_table = np.maximum(table, 0) if page else None
    ref, ref_lse = oracle.verify_attn(inp.q, inp.k, inp.v, ref_lens, lay, Hkv=hkv, scale=cfg.softmax_scale,
                                      gammas=ref_gam, page_table=ref_table, want_lse=True)
    for out, lse in got:
        gu.assert_attn_close(out[live], ref[live], str(case))
        assert not out[~live].any()                                    # no tokens: zeros
        for b in np.flatnonzero(live):
            n = gam[b] + 1
            assert np.max(np.abs(lse[b, :, :n] - ref_lse[b, :, :n])) < 1e-4     # fp32 sums of bf16 products


def _flat_case(B, lens, max_ctx, hint, d=128, hkv=8, hq=16, eff=None):
    """A contiguous token-major batch of equal capacity, true lengths `lens` (`eff` as the kernels clamp them)."""
    eff = np.asarray(lens if eff is None else eff, dtype=np.int32)
    cfg = wl.scaled(wl.CONFIGS["llama8b_32k"], name="flat", batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, gamma_choices=(3,),
                    ctx=(max_ctx, max_ctx))
    inp = wl.gen_attn_inputs(cfg)
    lse = torch.zeros((B, hq, 4), dtype=torch.float32, device="cuda")
    out = gu.rapid().rapid_verify_attn(gu.bf16_to_dev(inp.q), gu.bf16_to_dev(inp.k), gu.bf16_to_dev(inp.v),
                                       torch.from_numpy(np.asarray(lens, dtype=np.int32)).cuda(), max_ctx=max_ctx,
                                       softmax_scale=cfg.softmax_scale, lse_out=lse, ctx_sum_hint=hint)
    torch.cuda.synchronize()
    got, lse = gu.bf16_to_host(out), lse.cpu().numpy().astype(np.float64)
    bs, ts, hs, _ = wl.kv_strides(cfg, inp.seqs)
    live = eff > 0
    ref, ref_lse = oracle.verify_attn(inp.q, inp.k, inp.v, np.where(live, eff, 4).astype(np.int32), oracle.KVLayout(bs, ts, hs),
                                      Hkv=hkv, scale=cfg.softmax_scale, gamma=3, want_lse=True)
    gu.assert_attn_close(got[live], ref[live], "flat")
    assert np.max(np.abs(lse[live] - ref_lse[live])) < 1e-4
    assert not got[~live].any()


def test_lengths_out_of_range_are_clamped():
    """Lengths are device data: one above the bound counts as the bound, a negative one as 0, in the shares as in the sums."""
    lens = [1500, 1500 + 7000, 800, -5, 1500, 20, -2 ** 31, 2 ** 31 - 1, 700, 1111]
    eff = [1500, 1500, 800, 0, 1500, 20, 0, 1500, 700, 1111]
    hint = 11000
    assert hint // 128 >= _quanta_needed(10, 8, 128) and hint * 10 < 10 * 1500 * 9
    _flat_case(10, lens, 1500, hint, eff=eff)


@pytest.mark.parametrize("lens,hint", [([2000] * 10, 11000), ([2000, 5, 5, 5, 5, 5, 5, 5, 5, 5], 17500), ([4] * 10, 11000)])
def test_a_wrong_hint_only_chooses_the_route(lens, hint):
    """Hints far below and far above the true sum."""
    assert hint // 128 >= _quanta_needed(10, 8, 128) and hint * 10 < 10 * 2000 * 9
    _flat_case(10, lens, 2000, hint)


@pytest.mark.parametrize("B", [255, 256, 257])
def test_the_largest_batch_of_balanced_shares_and_the_next(B):
    lens = np.random.default_rng(B).integers(4, 600, B)
    lens[[0, 70, B - 1]] = 600, 0, 599
    hint = max(int(lens.sum()), 128 * _quanta_needed(min(B, 256), 4, 64))
    assert hint * 10 < B * 600 * 9
    _flat_case(B, lens, 600, hint, d=64, hkv=4, hq=4)
