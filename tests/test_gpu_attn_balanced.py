"""Attention of ragged batches whose total length the caller passes (balanced shares of the token stream, one
workgroup per compute unit) against the float64 oracle: lengths at the edges of a 128-token quantum and of a share,
sequences without tokens, more sequences than lanes of a wave or than shares, every layout and row count."""
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
    ctx, hint = torch.from_numpy(lens).cuda(), int(lens.astype(np.int64).sum())
    assert hint * 10 < B * max_ctx * 9
    r = gu.rapid()
    got = []
    for h in (hint, hint, 0):                 # twice (the workspace then holds old partials), and the fixed grid of splits
        lse = torch.zeros((B, hq, cfg.q_max), dtype=torch.float32, device="cuda")
        out = r.rapid_verify_attn(q, k, v, ctx, gammas=torch.from_numpy(gam).cuda(), page_table=pt, max_ctx=max_ctx,
                                  softmax_scale=cfg.softmax_scale, lse_out=lse, ctx_sum_hint=h)
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
