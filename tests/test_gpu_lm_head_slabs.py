"""Output head at row pitches that are multiples of 4 KiB, where workgroups start at different slabs of the hidden
dimension and wrap around, and next to them: logits against float64, statistics against the written logits."""
import numpy as np
import pytest
import torch

import gpu_util as gu
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
