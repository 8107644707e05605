"""Logits go to any 4-byte aligned device buffer: a contiguous view at any
element offset receives the same bits as an aligned tensor, on every LM-head
kernel (9 rows weight-streaming, 40 and 105 rows gemm_mid, 144 rows tiled), and
nothing around it is written."""

import numpy as np
import pytest

from workloads import ModelConfig, make_weights, tokens as wt

pytestmark = pytest.mark.gpu

WIDE = ModelConfig("wide", 1, 4096, 32, 2, 128, 4128, 4096, 5.0e5, max_pos=1024)


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_01019_amd as hvd
    gm = hvd.Model(WIDE, make_weights(WIDE, seed=11, gain_std=0.1))
    kv = hvd.KVCache(gm, max_seqs=3, n_pages=48)
    prompts = [wt.uniform_context(wt.rng_for("context", 950 + b), 30 + 7 * b, WIDE.vocab) for b in range(3)]
    yield torch, kv, prompts
    kv.close()
    gm.close()


@pytest.mark.parametrize("ks", [(8,), (39,), (34, 34, 34), (47, 47, 47)])
def test_offset_views_receive_the_same_logits(setup, ks):
    torch, kv, prompts = setup
    ids, rows, V = list(range(len(ks))), sum(ks) + len(ks), WIDE.vocab
    drafts = [wt.random_chain(wt.rng_for("draft", 950 + b), k, V) for b, k in zip(ids, ks)]
    want = torch.empty((rows, V), dtype=torch.float32, device="cuda")
    for offset in (0, 1, 2, 3):
        buf = torch.full((rows * V + 8,), -7.0, dtype=torch.float32, device="cuda")
        view = buf[offset: offset + rows * V].view(rows, V)
        assert view.data_ptr() % 16 == 4 * offset
        for b in ids:
            kv.prefill(b, prompts[b])
        print(f"{rows} rows, offset {offset}", flush=True)
        kv.verify(ids, [len(prompts[b]) - 1 for b in ids], drafts, logits=view if offset else want)
        for b in ids:
            kv.seq_free(b)
        if offset:
            assert torch.equal(view, want)
            assert (buf[:offset] == -7).all() and (buf[offset + rows * V:] == -7).all()
    assert np.isfinite(want.cpu().numpy()).all()
