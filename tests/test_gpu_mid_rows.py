"""GPU parity of verifies of 33 to 144 rows on a decoder wide enough for the
shared-activation GEMM (gemm_mid takes GEMMs of K >= 4096 and at least 4096
columns from three row tiles on): every row-tile count of a row block, two row
blocks, the fewest and the most rows of a tile, K splits, column blocks of 64
and 128 and a short last K slot (the down GEMM has 129 K steps), the MLP and
LM-head GEMMs single-pass and on the hi + lo pair.

Tolerances as everywhere: logits max-abs 2e-2; argmax, accepted length and next
token exact except near ties."""

import numpy as np
import pytest

import oracle
from tests._parity import Report, check_step
from workloads import ModelConfig, make_weights, tokens as wt

pytestmark = pytest.mark.gpu

WIDE = ModelConfig("wide", 1, 4096, 32, 2, 128, 4128, 4096, 5.0e5, max_pos=1024)
# draft lengths per sequence: 33, 48, 49, 65, 96, 97 and 128 rows; 144 (two row blocks)
BATCHES = ((32,), (47,), (48,), (64,), (47, 47), (47, 48), (63, 63), (47, 47, 47))


@pytest.fixture(scope="module")
def wide():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = make_weights(WIDE, seed=11, gain_std=0.1)
    om = oracle.OracleModel(WIDE, w)
    ctxs = [wt.uniform_context(wt.rng_for("context", 900 + b), 40 + 7 * b, WIDE.vocab) for b in range(3)]
    cases = {}
    for ks in BATCHES:
        seqs = []
        for b, k in enumerate(ks):
            st = oracle.prefill(om, ctxs[b])
            d = wt.random_chain(wt.rng_for("draft", 900 + 100 * b + k), k, WIDE.vocab)
            seqs.append((st, d, oracle.verify(om, st, d)))
        cases[ks] = seqs
    return torch, w, ctxs, cases


@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("max_mt", [8, 16])
def test_rows_match_oracle(wide, pair, max_mt):
    import paper_2606_01019_amd as hvd
    torch, w, ctxs, cases = wide
    gm = hvd.Model(WIDE, w)
    kv = hvd.KVCache(gm, max_seqs=3, n_pages=96)
    try:
        kv.set_option(hvd.hvd.HVD_OPT_SKINNY_MAX_MT, max_mt)
        if pair:
            kv.set_mlp_single(False)
            kv.set_option(hvd.hvd.HVD_OPT_LM_SINGLE, 0)
        rep = Report()
        for ks, seqs in cases.items():
            print(f"pair {pair}, {sum(ks) + len(ks)} rows", flush=True)
            ids = list(range(len(ks)))
            for b in ids:
                kv.prefill(b, ctxs[b])
            lg = torch.empty((sum(ks) + len(ks), WIDE.vocab), dtype=torch.float32, device="cuda")
            a, n = kv.verify(ids, [s.ctx for s, _, _ in seqs], [d for _, d, _ in seqs], logits=lg)
            out, at = lg.cpu().numpy().astype(np.float64), 0
            for b, (_, d, res) in enumerate(seqs):
                check_step(rep, res, out[at: at + len(d) + 1], int(a[b]), int(n[b]), d)
                at += len(d) + 1
            for b in ids:
                kv.seq_free(b)
        print(rep)
    finally:
        kv.close()
        gm.close()
