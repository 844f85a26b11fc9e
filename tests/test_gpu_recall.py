"""GPU parity of the recall point (Sec. 4.2 step-level scheduling, Eq. 10 as
printed): after a step's prefill, all of its query tokens -- through every
layer and query head -- select one working set.  Scores and selection through
the C ABI against the oracle, as in tests/parity.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_04852_amd import kvmem as K
from paper_2609_04852_amd import workload as W
from paper_2609_04852_amd.step import RecallState
from parity import assert_index_bitwise, check_scores, check_selection, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    K.lib()
    yield
    torch.cuda.synchronize()


def run_recall(cfg, seed, check_index=True):
    log(f"[case] recall {cfg.name} seed={seed} L={cfg.n_layers} M={cfg.n_blocks} n_q={cfg.n_q} "
        f"Hkv={cfg.n_kv_heads} Hq={cfg.n_q_heads} d={cfg.head_dim} Bt={cfg.block_tokens} mode={cfg.mode}")
    w = W.generate(cfg, seed, with_values=False)
    b2p = w.block_to_page
    S, Rr = cfg.sink_blocks, cfg.n_recent
    index_ref = np.stack([oracle.mean_k(oracle_pool(cfg, k), b2p) for k in w.k_pool])
    mode = oracle.MEAN_ALL if cfg.mode == W.MEAN_ALL else oracle.MAX_GROUP
    rel = oracle.block_relevance(w.q[0], index_ref, S, Rr, mode)
    k_eff = oracle.k_eff(cfg.budget_tokens, cfg.budget_tokens, cfg.block_tokens, cfg.n_blocks, S, Rr)
    vb_ref, _ = oracle.select(rel, S, Rr, k_eff, b2p)
    log("  gpu: index + select")
    st = RecallState(cfg, w.k_pool, b2p)
    st.build_index()
    torch.cuda.synchronize()
    if check_index:
        for l in range(cfg.n_layers):
            assert_index_bitwise(st.index_rows(l), index_ref[l])
    n_view = st.select(torch.from_numpy(np.ascontiguousarray(w.q[0])).cuda())
    torch.cuda.synchronize()
    assert n_view == S + k_eff + Rr
    vb, vpg = st.view_blocks.cpu().numpy(), st.view_pages.cpu().numpy()
    stats = check_selection(vb, vpg, rel, b2p, S, Rr, k_eff, ref_view=vb_ref)
    worst = check_scores(st.scores.cpu().numpy(), rel, S, Rr)
    log(f"  selection ok: {stats}, worst score rel err {worst:.2e}")
    return st, w


def oracle_pool(cfg, pool):
    return oracle.decode_fp8(pool, cfg.kv_scale) if cfg.kv_dtype == "fp8" else pool


RECALL_SHAPES = [
    # L, Hkv, Hq, d, Bt, M, S, Rr, n_q, mode, extra blocks
    (2, 2, 8, 128, 32, 700, 0, 8, 32, W.MEAN_ALL, 90),    # 128 rows per KV head and layer
    (3, 1, 4, 64, 16, 1500, 2, 16, 16, W.MEAN_ALL, 200),  # 64 rows, d64, a ragged last tile
    (1, 4, 16, 128, 64, 333, 0, 2, 8, W.MAX_GROUP, 40),    # 32 rows, one selection per KV head
    (2, 8, 32, 128, 16, 2100, 1, 40, 128, W.MEAN_ALL, 300),  # 512 rows: row partitions of the sum
    (1, 2, 8, 64, 16, 400, 0, 4, 256, W.MAX_GROUP, 50),      # 1,024 rows per selection: partitions of the max
]


@pytest.mark.parametrize("shape", RECALL_SHAPES, ids=[f"r{i}" for i in range(len(RECALL_SHAPES))])
def test_recall_shapes(shape):
    L, hkv, hq, d, bt, m, s, rr, nq, mode, extra = shape
    cfg = W.small_config(n_layers=L, n_kv_heads=hkv, n_q_heads=hq, head_dim=d, block_tokens=bt, kv_dtype="bf16",
                         history_tokens=m * bt, recent_tokens=rr * bt, sink_blocks=s,
                         budget_tokens=(s + rr + extra) * bt, n_q=nq, mode=mode, n_planted=3)
    run_recall(cfg, 31)


def test_recall_fp8():
    cfg = W.small_config(n_layers=2, n_kv_heads=4, n_q_heads=16, head_dim=128, block_tokens=32, kv_dtype="fp8",
                         kv_scale=float(np.float32(8 / 448)), history_tokens=900 * 32, recent_tokens=8 * 32,
                         budget_tokens=120 * 32, n_q=64, n_planted=3)
    run_recall(cfg, 32)


def test_recall_1m():
    run_recall(W.CONFIGS["1m_recall"], W.CONFIGS["1m_recall"].seed)


# rows per KV head around the edges of the 32-row waves and of the four
# workgroup shapes, with sinks and recent blocks that leave ragged first and
# last index tiles, a single tile, and one with no whole tile
ROW_SHAPES = [
    # G, n_q, d, M, S, Rr, mode
    (1, 17, 128, 64, 0, 1, W.MAX_GROUP),
    (1, 32, 64, 200, 3, 5, W.MEAN_ALL),
    (3, 11, 128, 331, 70, 9, W.MEAN_ALL),   # 33 rows, the first tile all sinks
    (4, 16, 64, 130, 1, 2, W.MAX_GROUP),    # 64 rows
    (5, 13, 128, 193, 0, 64, W.MEAN_ALL),   # 65 rows
    (8, 16, 128, 257, 2, 3, W.MAX_GROUP),   # 128 rows
    (1, 129, 64, 100, 30, 40, W.MEAN_ALL),  # 129 rows, no tile whole
    (7, 41, 128, 640, 0, 16, W.MEAN_ALL),   # 287 rows: a second, nearly empty row group
]


@pytest.mark.parametrize("shape", ROW_SHAPES, ids=[f"rows{s[0] * s[1]}_d{s[2]}" for s in ROW_SHAPES])
def test_rows_per_head(shape):
    G, nq, d, m, s, rr, mode = shape
    cfg = W.small_config(n_layers=2 if G != 1 else 1, n_kv_heads=2, n_q_heads=2 * G, head_dim=d, block_tokens=16,
                         kv_dtype="bf16", history_tokens=m * 16, recent_tokens=rr * 16, sink_blocks=s,
                         budget_tokens=(s + rr + max(1, (m - s - rr) // 5)) * 16, n_q=nq, mode=mode, n_planted=2)
    run_recall(cfg, 41)


def test_rows_wide_range():
    """Logits from rows whose elements span 40 binades: index blocks scaled by
    2^-20 .. 2^20 and queries scaled the other way, elements down to 2^-30 of
    their row's largest.  The fixed-point digits must leave the correctly rounded
    logits' accuracy (scores within the parity bound)."""
    r = np.random.default_rng(5)
    d, m, nq, hq = 128, 256, 24, 2
    geom = K.Geom(1, hq, d, 16, K.KVMEM_F32)
    index = r.standard_normal((m, 1, d)) * 2.0 ** r.integers(-15, 1, (m, 1, d))
    index = (index * 2.0 ** r.integers(-20, 21, (m, 1, 1))).astype(np.float32)
    q = r.standard_normal((1, nq, hq, d)) * 2.0 ** r.integers(-15, 1, (1, nq, hq, d))
    q = (q * 2.0 ** -20.0).astype(np.float32)
    _check_scores_of_rows(geom, q, index, 1e-6)


def test_rows_not_finite():
    """An index row with a NaN or an infinity, or a query with one, gives what
    the plain softmax gives: NaN scores where a logit is NaN or +inf, weight 0
    where it is -inf."""
    r = np.random.default_rng(6)
    d, m, nq, hq = 64, 200, 20, 1
    geom = K.Geom(1, hq, d, 16, K.KVMEM_F32)
    q = np.abs(r.standard_normal((1, nq, hq, d))).astype(np.float32)
    base = r.standard_normal((m, 1, d)).astype(np.float32)
    neg = base.copy()
    neg[7, 0, 5] = -np.inf  # every logit of block 7 is -inf: never selected, the others unchanged
    s = _check_scores_of_rows(geom, q, neg, 1e-6)
    assert s[0, 7] == 0.0
    for bad in (np.nan, np.inf):
        x = base.copy()
        x[11, 0, 3] = bad
        assert np.isnan(_scores_of_rows(geom, q, x)).all()
    q[0, 3, 0, 1] = np.nan
    assert np.isnan(_scores_of_rows(geom, q, base)).all()


def _scores_of_rows(geom, q, index):
    m, d = index.shape[0], index.shape[2]
    tiles = -(-m // 64)
    rows = np.zeros((tiles * 64, 1, d), np.float32)
    rows[:m] = index
    tiled = np.ascontiguousarray(rows.reshape(tiles, 64, 1, d // 4, 4).transpose(0, 2, 3, 1, 4))
    ti = torch.from_numpy(tiled).cuda()
    tq = torch.from_numpy(q).cuda()
    b2p = torch.arange(m, dtype=torch.int32, device="cuda")
    scores = torch.empty((1, m), dtype=torch.float32, device="cuda")
    k = m // 4
    vb = torch.empty((1, k + 1), dtype=torch.int32, device="cuda")
    ws = torch.empty(K.kvmem_select_workspace_bytes(geom, 1, q.shape[1], m, 0, 1, K.KVMEM_REDUCE_MEAN_ALL),
                     dtype=torch.uint8, device="cuda")
    K.kvmem_select(geom, tq, ti, m, 0, 1, (k + 1) * 16, (k + 1) * 16, K.KVMEM_REDUCE_MEAN_ALL, 0.0, b2p, vb,
                   torch.empty_like(vb), ws, scores)
    torch.cuda.synchronize()
    return scores.cpu().numpy()[:, :m - 1]


def _check_scores_of_rows(geom, q, index, rtol):
    got = _scores_of_rows(geom, q, index)
    s = np.einsum("lmhd,bd->mhb", q.astype(np.float64), np.where(np.isfinite(index), index, 0)[:-1, 0].astype(np.float64))
    s /= np.sqrt(q.shape[-1])
    s = np.where(np.isneginf(index[:-1, 0]).any(-1)[None, None], -np.inf, s)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    ref = p.sum(0).mean(0)[None]
    big = ref > 1e-30
    assert np.abs(got[big] / ref[big] - 1).max() <= rtol
    assert np.abs(got[~big]).max(initial=0.0) <= 1e-29
    return got
