"""GPU parity of the large-batch GEMMs at the row counts where their work plan
changes: prompts whose prefill is one chunk of a few row tiles (K split with
equal runs), one of many and two chunks, each followed by a verify that reads
every cached position, and a verify of several sequences whose rows start
anywhere in a page; and verifies of 1536 and 2000 rows whose plans deal K steps
out in unequal runs, hand a workgroup a shared tile and a whole one after it,
and do both at once.

Two layers of model width 1024 (8 q / 2 kv heads of 128, SwiGLU 4096, vocab
2048) or 3072 (24 / 6 heads, SwiGLU 5632), random norm gains.  Tolerances as everywhere: logits max-abs 2e-2;
argmax, accepted length and next token exact except near ties."""

import ctypes

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


SHARED = ModelConfig("shared", 2, 3072, 24, 6, 128, 5632, 2048, 5.0e5, max_pos=256)


@pytest.fixture(scope="module")
def shared():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_01019_amd as hvd
    w = make_weights(SHARED, seed=31, gain_std=0.1)
    return torch, oracle.OracleModel(SHARED, w, dtype=np.float32), hvd.Model(SHARED, w)


def _plan_kinds(rows, N, K, single=False):
    """Of the plan of a GEMM: whether runs are unequal, and whether whole tiles stand beside shared ones."""
    from paper_2606_01019_amd.build import HOST_LIB
    out = (ctypes.c_int32 * 4)()
    ctypes.CDLL(HOST_LIB).hvdh_tiled_plan(-(-rows // 16), N, K // 32, int(single), 256, ctypes.c_int64(128 << 20), out)
    tile, n_wg, n_shared, n_sk = out
    tiles = -(-rows // (128, 128, 256, 256, 128)[tile]) * (N // (128, 256, 256, 256, 256)[tile])
    return bool(n_shared and n_sk % n_shared), 0 < n_shared < tiles


@pytest.mark.parametrize("batch, k, pair", [(24, 63, True), (24, 63, False), (32, 62, True)])
def test_shared_tiles_match_oracle(shared, batch, k, pair):
    """Verifies, since their logits show every row: 24 sequences of 64 rows, 32 of 62 or 63."""
    import paper_2606_01019_amd as hvd
    torch, om, gm = shared
    c = SHARED
    ks = [k] * 24 if batch == 24 else [k - b % 2 for b in range(batch)]
    rows = sum(ks) + batch
    kinds = {"o": _plan_kinds(rows, c.d_model, c.q_dim), "gateup": _plan_kinds(rows, 2 * c.ffn_dim, c.d_model, not pair)}
    if rows == 1536:
        assert kinds["o"] == (True, False) and kinds["gateup"] == (False, True)
    else:
        assert rows == 2000 and kinds["gateup"] == (True, True)
    kv = hvd.KVCache(gm, max_seqs=batch, n_pages=batch * 8)
    if pair:
        kv.set_mlp_single(False)
    rng = wt.rng_for("context", 302, rows)
    prompts = [wt.uniform_context(rng, 3 + b, c.vocab) for b in range(batch)]
    drafts = [wt.random_chain(rng, n, c.vocab) for n in ks]
    for b, p in enumerate(prompts):
        kv.prefill(b, p)
    print(f"verify of {rows} rows, pair {pair}: {kinds}", flush=True)
    lg = torch.empty((rows, c.vocab), dtype=torch.float32, device="cuda")
    a, nx = kv.verify(list(range(batch)), [len(p) - 1 for p in prompts], drafts, logits=lg)
    lg = lg.cpu().numpy().astype(np.float64)
    rep, at = Report(), 0
    for b, (p, d) in enumerate(zip(prompts, drafts)):
        res = oracle.verify(om, oracle.prefill(om, p), d)
        check_step(rep, res, lg[at:at + len(d) + 1], int(a[b]), int(nx[b]), d)
        at += len(d) + 1
    print(rep)
    kv.close()
