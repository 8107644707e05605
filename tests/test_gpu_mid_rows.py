"""GPU parity of verifies of 33 to 144 rows on a decoder wide enough for the
shared-activation GEMM (gemm_mid takes GEMMs of K >= 4096 and at least 4096
columns from three row tiles on): every row-tile count of a row block, two row
blocks, the fewest and the most rows of a tile and a short last K slot (the down GEMM has 129 K steps), the MLP
and LM-head GEMMs single-pass and on the hi + lo pair, under the launch policy
(column blocks of 64 here); then every GEMM on column blocks of 64 and of 128,
unsplit and with three and eight K splits, on the workspace, on the static
scratch of hvd_verify_noalloc (whose 8 MiB cut the eight splits) and replayed
from a graph.

Tolerances as everywhere: logits max-abs 2e-2; argmax, accepted length and next
token exact except near ties."""

import ctypes

import numpy as np
import pytest

import oracle
from tests._parity import Report, check_step
from workloads import ModelConfig, make_weights, tokens as wt

pytestmark = pytest.mark.gpu

WIDE = ModelConfig("wide", 1, 4096, 32, 2, 128, 4128, 4096, 5.0e5, max_pos=1024)
# draft lengths per sequence: 33, 48, 49, 65, 96, 97 and 128 rows; 144 (two row blocks)
BATCHES = ((32,), (47,), (48,), (64,), (47, 47), (47, 48), (63, 63), (47, 47, 47))
# gate/up has 520 strips here, a multiple of 8, so every GEMM can take 128 columns
# per workgroup; the down GEMM's 130 K steps leave its last single-pass slot short
WIDE8 = ModelConfig("wide8", 1, 4096, 32, 2, 128, 4160, 4096, 5.0e5, max_pos=1024)
BATCHES8 = ((32,), (64,), (47, 47), (47, 48), (63, 63), (47, 47, 47))  # 3, 5, 6, 7, 8 and two times 5 row tiles


def _cases(cfg, batches):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = make_weights(cfg, seed=11, gain_std=0.1)
    om = oracle.OracleModel(cfg, w)
    ctxs = [wt.uniform_context(wt.rng_for("context", 900 + b), 40 + 7 * b, cfg.vocab) for b in range(3)]
    cases = {}
    for ks in batches:
        seqs = []
        for b, k in enumerate(ks):
            st = oracle.prefill(om, ctxs[b])
            d = wt.random_chain(wt.rng_for("draft", 900 + 100 * b + k), k, cfg.vocab)
            seqs.append((st, d, oracle.verify(om, st, d)))
        cases[ks] = seqs
    return torch, w, ctxs, cases


@pytest.fixture(scope="module")
def wide():
    return _cases(WIDE, BATCHES)


@pytest.fixture(scope="module")
def wide8():
    return _cases(WIDE8, BATCHES8)


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


@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("strips", [4, 8])
@pytest.mark.parametrize("splits", [1, 3, 8])
def test_column_blocks_and_splits_match_oracle(wide8, strips, splits, pair):
    import paper_2606_01019_amd as hvd
    from paper_2606_01019_amd.build import HOST_LIB
    torch, w, ctxs, cases = wide8
    host = ctypes.CDLL(HOST_LIB)
    out = (ctypes.c_int32 * 4)()
    c = WIDE8
    for mt in (3, 5, 6, 7, 8, 9):  # what the options below make of the plan
        for N, K in ((c.q_dim + 2 * c.kv_dim, c.d_model), (c.d_model, c.q_dim), (2 * c.ffn_dim, c.d_model),
                     (c.d_model, c.ffn_dim), (c.vocab, c.d_model)):
            assert host.hvdh_mid_plan(mt, N, K, 1, ctypes.c_int64(128 << 20), strips, splits, out)
            assert tuple(out) == (strips, splits, -(-mt // 8), mt if mt <= 8 else 5)
    assert host.hvdh_mid_plan(8, 4096, 4096, 1, ctypes.c_int64(8 << 20), strips, 8, out) and out[1] == 4
    gm = hvd.Model(c, w)
    kv = hvd.KVCache(gm, max_seqs=3, n_pages=96)
    try:
        kv.set_option(hvd.hvd.HVD_OPT_SKINNY_MAX_MT, 16)
        for family in hvd.hvd.GEMM_FAMILIES:
            kv.set_gemm_shape(family, strips, splits)
        if pair:
            kv.set_mlp_single(False)
            kv.set_option(hvd.hvd.HVD_OPT_LM_SINGLE, 0)
        rep = Report()
        for ks, seqs in cases.items():
            ids = list(range(len(ks)))
            for b in ids:
                kv.prefill(b, ctxs[b])
            lens = [s.ctx for s, _, _ in seqs]

            def step(how):
                print(f"strips {strips}, splits {splits}, pair {pair}, {sum(ks) + len(ks)} rows: {how}", flush=True)
                kv.set_graphs(how == "graph")
                lg = torch.empty((sum(ks) + len(ks), c.vocab), dtype=torch.float32, device="cuda")
                a, n = kv.verify(ids, lens, [d for _, d, _ in seqs], logits=lg, noalloc=how == "noalloc")
                for b in ids:  # cancel the uncommitted verify
                    kv.truncate(b, lens[b], int(ctxs[b][-1]))
                return lg.cpu().numpy(), a, n

            eager = step("eager")
            for lg, a, n in (eager, step("noalloc")):
                at = 0
                for b, (_, d, res) in enumerate(seqs):
                    check_step(rep, res, lg[at: at + len(d) + 1].astype(np.float64), int(a[b]), int(n[b]), d)
                    at += len(d) + 1
            for _ in range(3):  # captured, then replayed
                for got, ref in zip(step("graph"), eager):
                    assert np.array_equal(got, ref)
            kv.set_graphs(False)
            for b in ids:
                kv.seq_free(b)
        print(rep)
    finally:
        kv.close()
        gm.close()
