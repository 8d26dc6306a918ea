"""Output head at row pitches that are multiples of 4 KiB and next to them: logits against float64, statistics against
the written logits, and every logit summed in one order wherever its weight row lies in the vocabulary."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2502_20330_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,vocab,rows", [(2048, 1600, 1), (2048, 2005, 17), (2176, 1600, 9), (4096, 4100, 9),
                                               (4096, 16, 3), (6144, 3000, 33), (8192, 2500, 96)])
def test_slab_rotation(hidden, vocab, rows):
    h, w = wl.gen_lm_head_inputs(rows, hidden, vocab, salt=hidden + rows)
    hd, wd = gu.bf16_to_dev(h), gu.bf16_to_dev(w)
    r = gu.rapid()
    logits, stats = r.rapid_lm_head(hd, wd, temperature=0.7)
    torch.cuda.synchronize()
    ref = hd.double().cpu() @ wd.double().cpu().t()
    got = logits.double().cpu()
    assert torch.all((got - ref).abs() <= 5e-5 + 1e-5 * ref.abs())        # `hidden` fp32 additions of exact products
    chunk = r.lm_head_chunk(vocab, rows)
    st = stats.double().cpu().numpy()
    for c in range(st.shape[1]):
        z = got.numpy()[:, c * chunk:(c + 1) * chunk]
        np.testing.assert_array_equal(st[:, c, 0], z.max(-1))
        np.testing.assert_allclose(st[:, c, 1], np.exp((z - z.max(-1, keepdims=True)) / 0.7).sum(-1), rtol=2e-5)


@pytest.mark.parametrize("hidden,vocab,rows", [(1024, 5003, 1), (2048, 5003, 9), (4096, 5003, 17), (6144, 5003, 33),
                                               (8192, 5003, 9), (2176, 20011, 72)])
def test_equal_weight_rows_give_equal_logits(hidden, vocab, rows):
    """Tied or padding embeddings: rows of W with the same bits, in every workgroup, wave and block of the grid, must tie
    exactly, or rounding and not the lowest index decides a greedy token (and the token of a draw depends on the place of a
    row in the vocabulary).  The ties then go through the greedy limit of the accept pass."""
    h, w = wl.gen_lm_head_inputs(rows, hidden, 7, salt=hidden)
    idx = torch.arange(vocab, device="cuda") % 7
    hd, wd = gu.bf16_to_dev(h), gu.bf16_to_dev(w)[idx].contiguous()
    r = gu.rapid()
    logits, _ = r.rapid_lm_head(hd, wd)
    assert torch.equal(logits, logits[:, idx])
    u = torch.rand(rows, 1, device="cuda")
    _, tok, _ = r.rapid_accept(logits.view(rows, 1, vocab), torch.empty(rows, 0, vocab, device="cuda"),
                               torch.empty(rows, 0, dtype=torch.int32, device="cuda"), 0.0, u, temperature=0.0)
    ref = (hd.double() @ wd[:7].double().t()).argmax(-1)
    assert torch.equal(tok[:, 0].long(), ref)


@pytest.mark.parametrize("hidden,vocab,eta", [(2048, 32000, 1.0), (4096, 20003, 0.25)])
def test_head_and_accept_against_float64_logits(hidden, vocab, eta):
    """The chain of the output head and the accept pass on its statistics against the oracle's accept on float64 logits:
    what rounding of the logits may decide is counted, everything else has to agree.  With D = max |logit - float64|,
    probabilities move by at most 2 D relative, those of p_hat by 2 D + eta 2 D, so an accept ratio moves by less than
    (4 + 2 eta) D of itself and an edge of the normalised residual (the positive part of p - p_hat and p - q, of total
    weight W) by less than (8 + 4 eta) D / W; twice that is left for the float32 row statistics."""
    B, g = 16, 4
    rows = B * (g + 1)
    h, w = wl.gen_lm_head_inputs(rows, hidden, vocab, salt=41)
    hd, wd = gu.bf16_to_dev(h), gu.bf16_to_dev(w)
    z, st = gu.rapid().rapid_lm_head(hd, wd)
    z64 = (hd.double() @ wd.double().t()).view(B, g + 1, vocab)
    D = float((z.double().view_as(z64) - z64).abs().max())
    assert D < 1e-4
    rng = np.random.default_rng(hidden)
    zt = z64.float().cpu().numpy()
    zd = (zt[:, :g] + rng.standard_normal((B, g, vocab))).astype(np.float32)
    tok = np.argmax(zd + rng.gumbel(size=zd.shape), -1).astype(np.int32)
    u = rng.random((B, g + 1), dtype=np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n, out, _ = gu.rapid().rapid_accept(z.view(B, g + 1, vocab), dev(zd), dev(tok), eta, dev(u), target_stats=st)
    torch.cuda.synchronize()
    n, out = n.cpu().numpy(), out.cpu().numpy()
    ref = oracle.accept(zt, zd, tok, u, eta=eta)
    ties = 0
    for b in range(B):
        if np.any(ref.accept_margin[b] <= 2 * (4 + 2 * eta) * D):
            ties += 1
            continue
        m, W = int(ref.n_accepted[b]), 1.0
        assert n[b] == m
        if m < g:
            p, q, ph = oracle.distributions(z64[b, m].cpu().numpy(), zd[b, m], eta=eta)
            W = np.maximum(np.maximum(p - ph, p - q), 0.0).sum()
        if ref.draw_margin[b] <= 2 * (8 + 4 * eta) * D / W:
            ties += 1
            continue
        np.testing.assert_array_equal(out[b], ref.out_tokens[b])
    print(f"[head + accept against float64 logits] D = {D:.1e}, near ties {ties} of {B}")
    # a worst case of all logits off by D at once: a drawn token whose own weight is below it (a quarter to a third of the draws
    # from such a vocabulary) cannot be told from its neighbour; the others, the majority, are compared
    assert ties < B // 2


@pytest.mark.parametrize("hidden", [256, 1792, 2048, 2304, 4096, 128, 2176])
@pytest.mark.parametrize("vocab", [16, 1601, 12317])
def test_every_row_count_gives_the_same_logits(hidden, vocab):
    """The builds for one to six row blocks, edges of the blocks on both sides, slabs in one piece and in two (2048, 4096),
    ranges of one and of four vocabulary blocks, that is at most one for a wave: against float64, and a row's logits do
    not depend on how many rows are in the call."""
    h, w = wl.gen_lm_head_inputs(96, hidden, vocab, salt=hidden + vocab)
    hd, wd = gu.bf16_to_dev(h), gu.bf16_to_dev(w)
    ref = hd.double().cpu() @ wd.double().cpu().t()
    r = gu.rapid()
    whole, _ = r.rapid_lm_head(hd, wd)
    # products of bf16 are exact in float32, `hidden` additions of them round by 2^-24 of the running sum each
    assert torch.all((whole.double().cpu() - ref).abs() <= 5e-5 + 1e-5 * ref.abs())
    for rows in (1, 15, 16, 17, 33, 48, 49, 64, 65, 80, 81):
        logits, stats = r.rapid_lm_head(hd[:rows].contiguous(), wd)
        assert torch.equal(logits, whole[:rows]), rows
        chunk = r.lm_head_chunk(vocab, rows)
        pad = torch.nn.functional.pad(logits, (0, stats.shape[1] * chunk - vocab), value=-np.inf)
        z = pad.view(rows, stats.shape[1], chunk)
        assert torch.equal(stats[..., 0], z.amax(-1)), rows
        torch.testing.assert_close(stats[..., 1].double(), torch.exp(z.double() - z.double().amax(-1, True)).sum(-1),
                                   rtol=2e-5, atol=0)


@pytest.mark.parametrize("hidden", [1280, 2048, 4096, 6144, 8192, 12288, 16384, 18432, 24576, 32768])
def test_pitches_at_which_a_slab_is_two_runs(hidden):
    """The order of the sum over the hidden dimension: slabs of 256, or, where rows of W are a multiple of 4 KiB but no
    power of two from 16 KiB on, of 128 and the 128 that lie 2 KiB further on.  With 2^30 first, -2^30 at 1024 and 1 at 128, the 1 is lost
    unless the other two meet before it is added."""
    w = torch.zeros(1601, hidden, dtype=torch.bfloat16, device="cuda")
    w[:, 0], w[:, 1024], w[:, 128] = 2.0 ** 30, -2.0 ** 30, 1.0
    two_runs = 2 * hidden % 4096 == 0 and 2 * hidden not in (1 << 14, 1 << 15, 1 << 16)
    for rows in (1, 17, 48, 49, 96):
        logits, _ = gu.rapid().rapid_lm_head(torch.ones(rows, hidden, dtype=torch.bfloat16, device="cuda"), w)
        assert torch.all(logits == float(two_runs)), rows


@pytest.mark.parametrize("hidden", [256, 1792, 2048, 8192])
@pytest.mark.parametrize("vocab,blocks", [(33001, 9), (57001, 14), (68001, 17), (131072, 32)])
def test_waves_with_many_vocabulary_blocks(hidden, vocab, blocks):
    """The steady state of the builds for four to six row blocks: two to eight vocabulary blocks a wave, unevenly among the
    waves or evenly, so that loads of a slab of h are waited for by count or drained, and units of W requested before or after
    them; at 8192 also the line between the two kernels (4 NR blocks).  Against float64, and the same bits as in a
    call of fewer rows."""
    r = gu.rapid()
    assert r.lm_head_chunk(vocab, 96) == 16 * blocks
    g = torch.Generator(device="cuda").manual_seed(hidden + vocab)
    h = torch.randn(96, hidden, device="cuda", generator=g).bfloat16()
    w = (torch.randn(vocab, hidden, device="cuda", generator=g, dtype=torch.bfloat16) * (4 / hidden ** 0.5))
    few = [r.rapid_lm_head(h[i:i + 16].contiguous(), w)[0] for i in range(0, 96, 16)]
    whole = torch.cat(few)
    for at in range(0, vocab, 16384):
        ref = h.double() @ w[at:at + 16384].double().t().contiguous()
        assert torch.all((whole[:, at:at + 16384].double() - ref).abs() <= 5e-5 + 1e-5 * ref.abs())
    for rows in (48, 49, 64, 65, 80, 81, 96):
        logits, stats = r.rapid_lm_head(h[:rows].contiguous(), w)
        assert torch.equal(logits, whole[:rows]), rows
        z = torch.nn.functional.pad(logits, (0, stats.shape[1] * 16 * blocks - vocab), value=-np.inf).view(rows, -1, 16 * blocks)
        assert torch.equal(stats[..., 0], z.amax(-1)), rows
