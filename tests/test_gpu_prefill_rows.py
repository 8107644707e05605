"""GPU parity of the large-batch GEMMs at the row counts where their work plan
changes: prompts whose prefill is one chunk of a few row tiles (K split with
equal and unequal runs), of several tiles (whole tiles plus shared ones) and
two chunks, each followed by a verify that reads every cached position, and a
verify of several sequences whose rows start anywhere in a page.

Two layers of model width 1024 (8 q / 2 kv heads of 128, SwiGLU 4096, vocab
2048), random norm gains.  Tolerances as everywhere: logits max-abs 2e-2;
argmax, accepted length and next token exact except near ties."""

import numpy as np
import pytest

import oracle
from tests._parity import Report, check_step
from workloads import ModelConfig, make_weights, tokens as wt

pytestmark = pytest.mark.gpu

CFG = ModelConfig("rows", 2, 1024, 8, 2, 128, 4096, 2048, 5.0e5, max_pos=2304)


@pytest.fixture(scope="module")
def model():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_01019_amd as hvd
    w = make_weights(CFG, seed=23, gain_std=0.1)
    return torch, oracle.OracleModel(CFG, w, dtype=np.float32), hvd.Model(CFG, w)


@pytest.mark.parametrize("n", [130, 257, 390, 1001, 2200])
def test_prefill_then_verify(model, n):
    import paper_2606_01019_amd as hvd
    torch, om, gm = model
    kv = hvd.KVCache(gm, max_seqs=4, n_pages=4 * 160)
    rng = wt.rng_for("context", 300, n)
    # one long prompt, and three short ones verified with it: their rows start
    # at positions that are no multiple of 8, and there are more than 128
    prompts = [wt.uniform_context(rng, m, CFG.vocab) for m in (n, 3, 14, 45)]
    drafts = [wt.random_chain(rng, k, CFG.vocab) for k in (40, 35, 33, 29)]
    for b, p in enumerate(prompts):
        kv.prefill(b, p)
    rows = sum(len(d) + 1 for d in drafts)
    print(f"prompt {n}: verify of {rows} rows", flush=True)
    lg = torch.empty((rows, CFG.vocab), dtype=torch.float32, device="cuda")
    a, nx = kv.verify(list(range(4)), [len(p) - 1 for p in prompts], drafts, logits=lg)
    lg = lg.cpu().numpy().astype(np.float64)
    rep, at = Report(), 0
    for b, (p, d) in enumerate(zip(prompts, drafts)):
        res = oracle.verify(om, oracle.prefill(om, p), d)
        check_step(rep, res, lg[at:at + len(d) + 1], int(a[b]), int(nx[b]), d)
        at += len(d) + 1
    print(rep)
    kv.close()


def test_chunk_rows_above_a_short_rotary_table():
    """HVD_OPT_PREFILL_ROWS may exceed max_pos: a chunk has at most the prompt's
    rows.  512-row chunks of a 95-token prompt leave what one 96-row chunk leaves."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_01019_amd as hvd
    short = ModelConfig("short", 2, 256, 4, 4, 64, 1024, 4096, 1.0e4, max_pos=100, max_draft=4)
    gm = hvd.Model(short, make_weights(short, seed=29, gain_std=0.1))
    kv = hvd.KVCache(gm, max_seqs=1, n_pages=8)
    prompt = wt.uniform_context(wt.rng_for("context", 301), 95, short.vocab)
    out = []
    for rows in (0, 16, 128, 512, 2048):
        kv.set_option(hvd.hvd.HVD_OPT_PREFILL_ROWS, rows)
        print(f"chunks of {rows} rows", flush=True)
        kv.prefill(0, prompt)
        lg = torch.empty((5, short.vocab), dtype=torch.float32, device="cuda")
        kv.verify([0], [94], [np.asarray([1, 2, 3, 4])], logits=lg)
        out.append(lg.cpu())
        kv.seq_free(0)
    for lg in out:
        assert float((lg - out[0]).abs().max()) <= 2e-3
    for bad in (-16, 8, 24, 4096):
        with pytest.raises(hvd.HvdError):
            kv.set_option(hvd.hvd.HVD_OPT_PREFILL_ROWS, bad)
    kv.close()
    gm.close()
