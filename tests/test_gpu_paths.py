"""Every kernel instance and step branch the library dispatches to, reached through
the C ABI and held to the oracle: the generic scan at every rank and both query
types, the specialised scans for each (rank, group size, query type, wave steps),
the attention kernels for every pairing of query and KV types and every split
shape, both selection paths (fast, and the block-level path with survivors
re-read from memory), and the fused step's build-list branches (wider bases,
fp32 KV, KIVI before and after the build, the KV write).  Tolerances as in the
other parity tests: page LSE 1e-3 absolute, output 2e-3 rel-L2, tables by the
gap rule."""
import numpy as np
import pytest
import torch

from oracle import locks_oracle as O
from paper_2607_24555_amd import locks as B
from tests._gpu_common import (LSE_TOL, OUT_TOL, Dev, check_attention_on_table, check_sel_lse,
                               check_table, ids_of, near_tie_overlap, rel_l2)
from workloads import WorkloadSpec, build_workload, gather_unit

pytestmark = pytest.mark.gpu

DT = {"bf16": B.LOCKS_BF16, "fp32": B.LOCKS_FP32}


def _dev(name, S, G, Hkv, lens, rank, budget, kv, q, basis=B.LOCKS_BASIS_INT4, seed=21,
         spare=0, on_gpu=False):
    print(f"[paths {name}] S={S} G={G} Hkv={Hkv} lens={lens[:4]} r={rank} b={budget} kv={kv} "
          f"q={q} basis={basis}", flush=True)
    spec = WorkloadSpec(name, S, G * Hkv, Hkv, list(lens), rank, budget, kv, q,
                        spare_pages_per_seq=spare)
    d = Dev(build_workload(spec, seed, device="cuda" if on_gpu else "cpu"))
    if basis != B.LOCKS_BASIS_INT4:
        d.cfg.basis = basis
        d.ws = B.alloc_workspace(d.cfg, d.device)
    return d


def _scores_against_oracle(d, store, recs):
    cfg, G = d.cfg, d.cfg.group
    all_lse = torch.full((cfg.num_seqs, cfg.num_q_heads, cfg.max_pages_per_seq), float("nan"),
                         device=d.device)
    B.score_pages(cfg, d.q, store, d.pt, d.sl, d.ws, all_lse)
    torch.cuda.synchronize()
    worst = 0.0
    refs = {}
    basis = B.BASIS_NAMES[cfg.basis]
    for (s, h), rec in recs.items():
        k, v, qg = d.unit(s, h)
        ref = O.decode_step(qg, k, v, rec, cfg.rank, cfg.budget_tokens, basis)
        refs[(s, h)] = (k, v, qg, ref)
        n_c = k.shape[0] // 16
        if n_c:
            got = all_lse[s, h * G:(h + 1) * G, :n_c].double().cpu().numpy()
            worst = max(worst, float(np.max(np.abs(got - ref["s_hat"]))))
    assert worst <= LSE_TOL, worst
    return refs, worst


def _step_against_oracle(d, refs, ids, sel, out, lse):
    cfg, G = d.cfg, d.cfg.group
    results, worst = [], 0.0
    for (s, h), (k, v, qg, ref) in refs.items():
        n_c, n = k.shape[0] // 16, -(-k.shape[0] // 16)
        got = ids_of(ids[s, h].tolist())
        results.append(check_table(got, ref, n, cfg.k))
        hs = slice(h * G, (h + 1) * G)
        worst = max(worst, check_attention_on_table(qg, k, v, got, out[s, hs].double().cpu().numpy(),
                                                    lse[s, hs].double().cpu().numpy()))
        check_sel_lse(sel[s, hs].double().cpu().numpy(), got, ref["s_hat"], n_c)
    return near_tie_overlap(results), worst


def _attend_on_oracle_tables(d, refs):
    cfg, G = d.cfg, d.cfg.group
    ids = torch.full((cfg.num_seqs, cfg.num_kv_heads, cfg.k), -1, dtype=torch.int32)
    for (s, h), (_, _, _, ref) in refs.items():
        ids[s, h, :len(ref["ids"])] = torch.tensor(ref["ids"], dtype=torch.int32)
    out, lse = B.sparse_attend(cfg, d.q, d.k, d.v, d.pt, d.sl, ids.to(d.device), d.ws)
    dout, dlse = B.dense_attend(cfg, d.q, d.k, d.v, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    worst = 0.0
    for (s, h), (k, v, qg, ref) in refs.items():
        hs = slice(h * G, (h + 1) * G)
        o = out[s, hs].double().cpu().numpy()
        worst = max(worst, max(rel_l2(o[g], ref["out"][g]) for g in range(G)))
        np.testing.assert_allclose(lse[s, hs].double().cpu().numpy(), ref["lse"], atol=LSE_TOL)
        o_d, l_d = O.dense_step(qg, k, v)
        od = dout[s, hs].double().cpu().numpy()
        worst = max(worst, max(rel_l2(od[g], o_d[g]) for g in range(G)))
        np.testing.assert_allclose(dlse[s, hs].double().cpu().numpy(), l_d, atol=LSE_TOL)
    assert worst <= OUT_TOL, worst
    return worst


@pytest.mark.parametrize("q", ["bf16", "fp32"])
@pytest.mark.parametrize("rank", list(range(1, 16)))
def test_generic_scan_every_rank(rank, q):
    """Two-head groups: the generic matrix-core scan at every rank but 8, which has its own."""
    d = _dev("generic", 1, 2, 2, [16 * 130 + 5], rank, 256, q, q)
    store, recs = d.oracle_summaries()
    _, worst = _scores_against_oracle(d, store, recs)
    print(f"[paths generic] r={rank} q={q}: max |hat s err| {worst:.2e}")


@pytest.mark.parametrize("G,rank,page", [(16, 8, 16), (16, 8, 32), (16, 8, 64), (8, 8, 16),
                                         (4, 8, 16), (4, 8, 64), (16, 4, 16), (4, 2, 16)])
def test_scores_of_heads_with_different_query_ranges(G, rank, page):
    """Heads of one group whose largest query elements lie in different powers of two:
    each head's scores keep that head's own query scale."""
    spec = WorkloadSpec("ranges", 1, 2 * G, 2, [page * 150 + 3], rank, 256, "bf16", "bf16",
                        page_size=page)
    d = Dev(build_workload(spec, 5))
    f = torch.tensor([1.0, 0.3, 1.7, 0.07, 0.9, 0.51, 1.2, 0.013])
    q = d.w.q.float() * f.repeat(2 * G // 8 + 1)[:2 * G, None]
    d.w.q = q.to(torch.bfloat16)
    d.q = d.w.q.cuda()
    store, recs = d.oracle_summaries()
    out = B.score_pages(d.cfg, d.q, store, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    for (s, h), rec in recs.items():
        k, v, qg = d.unit(s, h)
        ref = O.decode_step(qg, k, v, rec, rank, 256, "int4", page)["s_hat"]
        n_c = k.shape[0] // page
        got = out[s, h * G:(h + 1) * G, :n_c].double().cpu().numpy()
        np.testing.assert_allclose(got, ref[:, :n_c], atol=LSE_TOL, rtol=0)


def _rank8_against_oracle(d, page, units, rtol=0.0):
    """Page scores and selected tables of rank-8 units against the oracle."""
    cfg, G = d.cfg, d.cfg.group
    store, recs = d.oracle_summaries(units)
    lse = torch.full((cfg.num_seqs, cfg.num_q_heads, cfg.max_pages_per_seq), float("nan"),
                     device=d.device)
    ids, _ = B.select(cfg, d.q, store, d.pt, d.sl, d.ws, out_all_lse=lse)
    torch.cuda.synchronize()
    for (s, h), rec in recs.items():
        k, v, qg = d.unit(s, h)
        ref = O.decode_step(qg, k, v, rec, 8, cfg.budget_tokens, "int4", page)
        n_c, n = k.shape[0] // page, -(-k.shape[0] // page)
        got = lse[s, h * G:(h + 1) * G].double().cpu().numpy()
        np.testing.assert_allclose(got[:, :n_c], ref["s_hat"][:, :n_c], atol=LSE_TOL, rtol=rtol)
        assert np.isnan(got[:, n_c:]).all()
        if not rtol:
            check_table(ids_of(ids[s, h].tolist()), ref, n, cfg.k)


@pytest.mark.parametrize("steps", [1, 4])
@pytest.mark.parametrize("G,page,q", [(1, 16, "fp32"), (3, 16, "bf16"), (4, 32, "bf16"),
                                      (5, 32, "bf16"), (7, 16, "bf16"), (8, 16, "fp32"),
                                      (8, 32, "bf16"), (6, 64, "bf16"), (9, 64, "bf16"),
                                      (12, 16, "bf16"), (16, 16, "fp32"), (16, 32, "bf16")])
def test_rank8_scan_groups_and_tile_edges(G, page, q, steps):
    """The rank-8 scans at every head-column width, page size and query type, with
    sequences that end on and around the edges of 16-page steps and of a wave's pages,
    in grids small enough for one step per wave and large enough for four."""
    edges = [page * n + e for n, e in ((1, 0), (15, 3), (16, 0), (17, 1), (63, 0), (64, 5),
                                       (65, 0), (130, 2), (0, 5))]
    if steps == 1:
        S, Hkv, lens = len(edges), 2, edges
    else:      # 260 blocks of 256 (sub-)pages: four steps per wave
        S, Hkv = 65, 4
        lens = (edges * 8)[:S]
    spec = WorkloadSpec("groups", S, G * Hkv, Hkv, lens, 8, page * 10, "bf16", q, page_size=page)
    d = Dev(build_workload(spec, 17))
    _rank8_against_oracle(d, page, {(s, h) for s in range(len(edges)) for h in (0, Hkv - 1)})


@pytest.mark.parametrize("G,page", [(4, 16), (7, 64), (8, 16), (16, 16), (16, 32)])
def test_rank8_scan_of_widely_spread_logits(G, page):
    """Pages whose logits spread over more than the range of a float32 exponential:
    the scan's sums are then taken with the max shifted out (scores of several
    hundred nats, so float32 rounding enters relative to them)."""
    spec = WorkloadSpec("spread", 2, 2 * G, 2, [page * 70 + 1, page * 5], 8, page * 10, "bf16",
                        "bf16", page_size=page)
    d = Dev(build_workload(spec, 19))
    d.w.q = (d.w.q.float() * 60).to(torch.bfloat16)
    d.q = d.w.q.cuda()
    _rank8_against_oracle(d, page, {(s, h) for s in (0, 1) for h in (0, 1)}, rtol=2e-6)


@pytest.mark.parametrize("G,page", [(4, 16), (3, 32), (8, 64), (16, 16), (12, 64)])
def test_rank8_scan_of_uncentred_coefficients(G, page):
    """Records whose coefficient rows do not sum to zero: all of a page's logits may lie
    hundreds of nats above or below its centroid's, where no sum of exponentials is in
    float32's range without a shift.  Some pages keep their own rows."""
    spec = WorkloadSpec("uncentred", 2, 2 * G, 2, [page * 70 + 1, page * 5], 8, page * 10, "bf16",
                        "bf16", page_size=page)
    d = Dev(build_workload(spec, 37))
    d.w.q = (d.w.q.float() * 60).to(torch.bfloat16)
    d.q = d.w.q.cuda()
    store, recs = d.oracle_summaries()
    out = torch.empty(2, 2 * G, d.cfg.max_pages_per_seq, device=d.device)
    off = 64 * 8
    for (s, h), rec in recs.items():
        rec = rec.copy()
        c = rec[:, off:off + 8 * page].reshape(-1, page, 8)
        c[::3] = c[::3, :1]                       # every token the page's first row
        rec[:, off:off + 8 * page] = c.reshape(rec.shape[0], -1)
        recs[(s, h)] = rec
        store[d.w.page_table[s, :rec.shape[0]].long().to(d.device), h] = torch.from_numpy(rec).to(d.device)
    B.score_pages(d.cfg, d.q, store, d.pt, d.sl, d.ws, out)
    torch.cuda.synchronize()
    spread = 0.0
    for (s, h), rec in recs.items():
        k, v, qg = d.unit(s, h)
        ref = O.decode_step(qg, k, v, rec, 8, d.cfg.budget_tokens, "int4", page)["s_hat"]
        n_c = k.shape[0] // page
        got = out[s, h * G:(h + 1) * G, :n_c].double().cpu().numpy()
        np.testing.assert_allclose(got, ref[:, :n_c], atol=LSE_TOL, rtol=2e-6)
        spread = max(spread, np.abs(ref).max())
    assert spread > 100.0


def _rank8_scores(G, page, q_dtype, edit, seed=41):
    """Page scores of rank-8 units and their 64-bit values, after edit(workload) changed
    its tensors."""
    spec = WorkloadSpec("digits", 2, 2 * G, 2, [page * 70 + 1, page * 5], 8, page * 10, "bf16",
                        q_dtype, page_size=page)
    w = build_workload(spec, seed)
    edit(w)
    d = Dev(w)
    store, recs = d.oracle_summaries()
    out = B.score_pages(d.cfg, d.q, store, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    got, want = [], []
    for (s, h), rec in recs.items():
        k, v, qg = d.unit(s, h)
        n_c = k.shape[0] // page
        got.append(out[s, h * G:(h + 1) * G, :n_c].double().cpu().numpy())
        with np.errstate(invalid="ignore"):           # queries that are not finite
            ref = O.decode_step(qg, k, v, rec, 8, d.cfg.budget_tokens, "int4", page)
        want.append(ref["s_hat"][:, :n_c])
    return got, want


# every head-column width of the rank-8 scans, without the four- and sixteen-head groups
# (whose queries are held in 20 bits of the head's largest element)
WIDE_QUERY = [(1, 16, "fp32"), (3, 16, "bf16"), (2, 32, "fp32"), (3, 64, "bf16"), (8, 16, "bf16"),
              (7, 16, "fp32"), (5, 32, "bf16"), (6, 64, "fp32"), (9, 16, "fp32"), (15, 32, "bf16"),
              (12, 64, "fp32")]


@pytest.mark.parametrize("G,page,q", WIDE_QUERY)
def test_scores_of_a_query_with_a_dominant_channel(G, page, q):
    """One query channel 1,000 times the others, on which the keys are zero: the scores rest
    on elements 2^-13 of the largest.  Held: 2^-31 of the largest element (8 x 1,024) per
    channel, over 127 channels of keys of up to 16, over sqrt(128), and the roundings of
    scores of up to 100."""
    def edit(w):
        w.k_cache[..., 0] = 0
        w.q[..., 0] = 1024.0 * w.q.float().abs().amax(-1).clamp(max=8.0).to(w.q.dtype)
    got, want = _rank8_scores(G, page, q, edit)
    tol = 2.0 ** -31 * 8192 * 16 * 127 / 128 ** 0.5 + 2.0 ** -21 * 100
    err = max(np.abs(a - b).max() for a, b in zip(got, want))
    assert np.abs(want[0]).max() <= 100
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("G,page", [(g, p) for g, p, q in WIDE_QUERY if q == "fp32"])
def test_scores_of_fp32_queries_keep_float32(G, page):
    """fp32 queries that bf16 does not hold: the mean error over the pages is within half a
    unit in the last place of the largest score, which the roundings of the score's own
    sums (a handful, of either sign) leave on average."""
    def edit(w):
        gen = torch.Generator().manual_seed(3)
        w.q *= 1 + 0.01 * torch.rand(w.q.shape, generator=gen)
    got, want = _rank8_scores(G, page, "fp32", edit)
    err = np.concatenate([np.abs(a - b).ravel() for a, b in zip(got, want)])
    top = max(np.abs(b).max() for b in want)
    print(f"[paths fp32 queries] G={G} page={page}: mean {err.mean():.2e} max {err.max():.2e} of {top:.1f}")
    assert err.mean() <= 2.0 ** -24 * top, (err.mean(), top)


@pytest.mark.parametrize("G,page,q", WIDE_QUERY)
def test_scores_of_huge_queries(G, page, q):
    """Queries of 1e6 (projections past float16's range): scores stay relative to float32."""
    def edit(w):
        w.q = (w.q.float() * 1e6).to(w.q.dtype)
    got, want = _rank8_scores(G, page, q, edit)
    for a, b in zip(got, want):
        np.testing.assert_allclose(a, b, rtol=0, atol=2.0 ** -21 * max(np.abs(x).max() for x in want))


@pytest.mark.parametrize("G,page,q", WIDE_QUERY)
def test_scores_of_a_query_that_is_not_finite(G, page, q):
    """A NaN or an infinity in a head's query makes that head's scores NaN and leaves the
    other heads' as they are, up to the rounding of sums that are then taken with their max
    shifted out (four units in the last place)."""
    base, _ = _rank8_scores(G, page, q, lambda w: None)

    def edit(w):
        w.q[0, 0, 5] = float("nan")
        w.q[0, G + G // 2, 127] = float("-inf")
    got, _ = _rank8_scores(G, page, q, edit)
    bad = {(0, 0), (1, G // 2)}                       # (KV head, head of its group) of sequence 0
    for i, (a, b) in enumerate(zip(got, base)):
        s, h = divmod(i, 2)
        for g in range(G):
            if s == 0 and (h, g) in bad:
                assert np.isnan(a[g]).all()
            else:
                np.testing.assert_allclose(a[g], b[g], rtol=2.0 ** -21, atol=0)


@pytest.mark.parametrize("G,rank,heads", [(1, 8, 20480), (9, 8, 20480), (4, 2, 50048)])
def test_scores_of_blocks_past_16_mib(G, rank, heads):
    """So many KV heads that one block's records pass 2^24 bytes: each head's scores equal
    those of the same head in a store of 64 heads (the same records, the same sums)."""
    cfg = B.Config(1, 64 * G, 64, rank, 256, 4, 4)
    gen = torch.Generator().manual_seed(11)
    k = torch.randn(4, 64, 16, 128, generator=gen).to(torch.bfloat16).cuda()
    q = torch.randn(1, 64 * G, 128, generator=gen).to(torch.bfloat16).cuda()
    pt = torch.tensor([[2, 0, 3, 1]], dtype=torch.int32).cuda()
    sl = torch.tensor([4 * 16], dtype=torch.int32).cuda()
    store = B.alloc_summaries(cfg, "cuda")
    B.build_summaries(cfg, k, pt, sl, store)
    want = B.score_pages(cfg, q, store, pt, sl, B.alloc_workspace(cfg, "cuda"))
    n = heads // 64
    big = B.Config(1, heads * G, heads, rank, 256, 4, 4)
    assert heads * store.shape[-1] >= 1 << 24
    got = B.score_pages(big, q.repeat(1, n, 1), store.repeat(1, n, 1), pt, sl,
                        B.alloc_workspace(big, "cuda"))
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    torch.testing.assert_close(got.view(n, 64 * G, 4), want.expand(n, -1, -1), rtol=0, atol=1e-5)


@pytest.mark.parametrize("G,rank,q", [(4, 8, "bf16"), (16, 8, "fp32"), (4, 2, "bf16")])
def test_scores_with_an_unaligned_query(G, rank, q):
    """A query tensor that starts one element past a 16-byte boundary scores the same bits."""
    d = _dev("unaligned", 1, G, 2, [16 * 90 + 3], rank, 256, "bf16", q)
    store, _ = d.oracle_summaries()
    want = B.score_pages(d.cfg, d.q, store, d.pt, d.sl, d.ws)
    buf = torch.empty(d.q.numel() + 1, dtype=d.q.dtype, device=d.device)
    buf[1:] = d.q.flatten()
    got = B.score_pages(d.cfg, buf[1:].view(d.q.shape), store, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    assert torch.equal(got[..., :90], want[..., :90])


STEP_CASES = {
    # name: (G, rank, kv dtype, q dtype)
    "G16-r2": (16, 2, "bf16", "bf16"),
    "G16-r4": (16, 4, "bf16", "bf16"),
    "G16-r2-fp32": (16, 2, "fp32", "fp32"),
    "G16-r4-fp32q": (16, 4, "bf16", "fp32"),
    "G16-r8-fp32q": (16, 8, "bf16", "fp32"),
    "G4-r2-fp32q": (4, 2, "bf16", "fp32"),
    "G4-r4-fp32kv": (4, 4, "fp32", "bf16"),
    "G4-r4-fp32": (4, 4, "fp32", "fp32"),
    "G4-r8-fp32q": (4, 8, "bf16", "fp32"),
}


@pytest.mark.parametrize("name", sorted(STEP_CASES))
def test_step_kernel_variants(name):
    """Scan, fused step, attention on the oracle's tables and the dense baseline for
    the specialised scans and every pairing of query and KV types."""
    G, rank, kv, q = STEP_CASES[name]
    d = _dev(name, 1, G, 2, [16 * 1100 + 3], rank, 2048, kv, q)
    store, recs = d.oracle_summaries()
    refs, err = _scores_against_oracle(d, store, recs)
    ids, sel, out, lse = B.decode_step(d.cfg, d.q, d.k, d.v, d.pt, d.sl, store, d.ws)
    torch.cuda.synchronize()
    ov, worst = _step_against_oracle(d, refs, ids, sel, out, lse)
    worst_a = _attend_on_oracle_tables(d, refs)
    print(f"[paths {name}] hat s err {err:.2e}; step near-tie overlap {ov:.4f}, rel-L2 "
          f"{worst:.2e}; attend/dense on oracle tables rel-L2 {worst_a:.2e}")


BIG_CASES = {
    # four 16-page steps per scan wave, fp32 queries
    "G16-r8-fp32q-4steps": (2, 16, 2, [16 * 16384 + 7, 16 * 16000 + 2], 8),
    "G4-r8-fp32q-4steps": (1, 4, 8, [16 * 8192 + 5], 8),
}


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", sorted(BIG_CASES))
def test_step_four_step_scans_fp32_queries(name):
    S, G, Hkv, lens, rank = BIG_CASES[name]
    d = _dev(name, S, G, Hkv, lens, rank, 2048, "bf16", "fp32", on_gpu=True)
    store, recs = d.oracle_summaries()
    refs, err = _scores_against_oracle(d, store, recs)
    ids, sel, out, lse = B.decode_step(d.cfg, d.q, d.k, d.v, d.pt, d.sl, store, d.ws)
    torch.cuda.synchronize()
    ov, worst = _step_against_oracle(d, refs, ids, sel, out, lse)
    print(f"[paths {name}] hat s err {err:.2e}; near-tie overlap {ov:.4f}; rel-L2 {worst:.2e}")


SPLIT_CASES = {
    # 32 (seq, KV head) units of 128 table entries: two entries per attention wave
    "two-per-wave": (4, [16 * 256 + 9, 16 * 300, 16 * 129 + 1, 16 * 400 + 15]),
    # 128 units: eight entries per wave
    "eight-per-wave": (16, [16 * 260 + 3 * i for i in range(16)]),
}


@pytest.mark.parametrize("name", sorted(SPLIT_CASES))
def test_attention_split_shapes(name):
    S, lens = SPLIT_CASES[name]
    d = _dev(name, S, 4, 8, lens, 8, 2048, "bf16", "bf16", on_gpu=True)
    store, recs = d.oracle_summaries()
    refs, _ = _scores_against_oracle(d, store, recs)
    ids, sel, out, lse = B.decode_step(d.cfg, d.q, d.k, d.v, d.pt, d.sl, store, d.ws)
    torch.cuda.synchronize()
    ov, worst = _step_against_oracle(d, refs, ids, sel, out, lse)
    worst_a = _attend_on_oracle_tables(d, refs)
    print(f"[paths {name}] step rel-L2 {worst:.2e}, near-tie overlap {ov:.4f}; attend on "
          f"oracle tables {worst_a:.2e}")


@pytest.mark.timeout(600)
def test_block_level_selection_rereads_survivors():
    """A 4096-token budget over 33,001 pages: the block-level selection path, whose
    final cut holds more survivors than its registers and re-reads them."""
    d = _dev("many-survivors", 1, 2, 1, [16 * 33000 + 5], 8, 4096, "bf16", "bf16", on_gpu=True)
    store, recs = d.oracle_summaries()
    refs, _ = _scores_against_oracle(d, store, recs)
    ids, sel, out, lse = B.decode_step(d.cfg, d.q, d.k, d.v, d.pt, d.sl, store, d.ws)
    ids2, sel2 = B.select(d.cfg, d.q, store, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids2)
    ov, worst = _step_against_oracle(d, refs, ids, sel, out, lse)
    print(f"[paths many-survivors] near-tie overlap {ov:.4f}, rel-L2 {worst:.2e}")


BUILD_CASES = {
    # name: (kv, q, basis, kivi stage or None, budget, kv write inside the step)
    "int8-basis": ("bf16", "bf16", B.LOCKS_BASIS_INT8, None, 256, False),
    "bf16-basis-kivi-post": ("bf16", "bf16", B.LOCKS_BASIS_BF16, B.LOCKS_KIVI_POST, 256, False),
    "fp32-kv": ("fp32", "fp32", B.LOCKS_BASIS_INT4, None, 256, True),
    "fp32-q-kivi-pre": ("bf16", "fp32", B.LOCKS_BASIS_INT4, B.LOCKS_KIVI_PRE, 256, True),
    "block-select-kv-write": ("bf16", "bf16", B.LOCKS_BASIS_INT4, None, 4096, True),
    "int8-basis-kv-write-kivi-pre": ("bf16", "bf16", B.LOCKS_BASIS_INT8, B.LOCKS_KIVI_PRE, 256,
                                     True),
}


@pytest.mark.parametrize("name", sorted(BUILD_CASES))
def test_step_build_list_branches(name):
    """A fused step with a build list (and optionally KIVI and the new token's KV
    write) on the step branches other than the overlapped int4 build: it must equal,
    bit for bit, the same work done by the separate entry points in order (KV
    write, KIVI PRE, build, KIVI POST, then a step without a list), and its output
    must match the oracle's attention over its own table on the final caches."""
    kv, q, basis, stage, budget, write = BUILD_CASES[name]
    rank = 4
    lens = [16 * 300 - 1, 16 * 200 + 9, 16 * 150 + 15]   # the new token fills page 299 of seq 0
    d = _dev(name, 3, 4, 2, lens, rank, budget, kv, q, basis=basis, spare=1)
    cfg = d.cfg
    dev = d.device
    store = B.alloc_summaries(cfg, dev)
    B.build_summaries(cfg, d.k, d.pt, d.sl, store)
    kivi = None if stage is None else B.Kivi(4, 32, stage)
    gen = torch.Generator().manual_seed(5)
    kt = torch.bfloat16 if kv == "bf16" else torch.float32
    k_new = torch.randn(3, 2, 128, generator=gen).to(kt).to(dev) if write else None
    v_new = torch.randn(3, 2, 128, generator=gen).to(kt).to(dev) if write else None
    new_lens = [L + 1 if write else L for L in lens]
    sl = torch.tensor(new_lens, dtype=torch.int32, device=dev)
    listed = [(s, L // 16 - 1) for s, L in enumerate(new_lens)] + [(1, 3), (2, 77)]
    bl = torch.tensor(listed, dtype=torch.int32, device=dev)
    blocks = torch.tensor([int(d.w.page_table[s, j]) for s, j in listed], device=dev).long()
    store[blocks] = 0                                   # the build must rewrite them
    # reference: the separate entry points in the step's order
    rk, rv, rstore = d.k.clone(), d.v.clone(), store.clone()
    if write:
        B.append_kv(cfg, k_new, v_new, rk, rv, d.pt, sl)
    if kivi is not None and stage == B.LOCKS_KIVI_PRE:
        B.kivi_quantize(cfg, kivi, rk, rv, d.pt, sl, bl)
    B.build_summaries(cfg, rk, d.pt, sl, rstore, build_list=bl)
    if kivi is not None and stage == B.LOCKS_KIVI_POST:
        B.kivi_quantize(cfg, kivi, rk, rv, d.pt, sl, bl)
    r_ids, r_sel, r_out, r_lse = B.decode_step(cfg, d.q, rk, rv, d.pt, sl, rstore, d.ws)
    torch.cuda.synchronize()
    ws2 = B.alloc_workspace(cfg, dev)
    ids, sel, out, lse = B.decode_step(cfg, d.q, d.k, d.v, d.pt, sl, store, ws2, build_list=bl,
                                       kivi=kivi, k_new=k_new, v_new=v_new)
    torch.cuda.synchronize()
    assert torch.equal(d.k, rk) and torch.equal(d.v, rv)
    assert torch.equal(store, rstore)
    assert torch.equal(ids, r_ids)
    assert torch.equal(out, r_out) and torch.equal(lse, r_lse)
    assert torch.equal(torch.nan_to_num(sel, nan=-7.0), torch.nan_to_num(r_sel, nan=-7.0))
    # the output against the oracle's attention over the step's table, final caches
    d.w.k_cache, d.w.v_cache = d.k, d.v
    d.w.spec.seq_lens = new_lens
    G = cfg.group
    worst = 0.0
    for s in range(cfg.num_seqs):
        for h in range(cfg.num_kv_heads):
            k, v, qg = gather_unit(d.w, s, h)
            got = ids_of(ids[s, h].tolist())
            assert len(got) == min(cfg.k, -(-new_lens[s] // 16))
            hs = slice(h * G, (h + 1) * G)
            worst = max(worst, check_attention_on_table(qg, k, v, got, out[s, hs].double().cpu().numpy(),
                                                        lse[s, hs].double().cpu().numpy()))
    print(f"[paths {name}] equals the separate calls bit for bit; rel-L2 on its tables "
          f"{worst:.2e}")


@pytest.mark.parametrize("G,page", [(4, 16), (7, 16), (16, 64), (2, 32)])
def test_dense_attention_of_ragged_batches(G, page):
    """Dense attention in blocks of eight units, two a wave, most of them past their
    sequence's end: empty sequences, single tokens, lengths on and around a wave's and a
    block's units."""
    lens = [16 * 64, 0, 1, 16 * 64 + 1, 16 * 16 - 1, 7000, 16 * 256, 16 * 3 + 9]
    spec = WorkloadSpec("dense", len(lens), 2 * G, 2, lens, 8, 16 * page, "bf16", "bf16",
                        page_size=page)
    d = Dev(build_workload(spec, 23))
    out, lse = B.dense_attend(d.cfg, d.q, d.k, d.v, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    for s in range(len(lens)):
        for h in range(2):
            k, v, qg = d.unit(s, h)
            o, l = O.dense_step(qg, k, v)
            hs = slice(h * G, (h + 1) * G)
            got = out[s, hs].double().cpu().numpy()
            if lens[s] == 0:
                assert not got.any() and torch.isneginf(lse[s, hs]).all()
                continue
            assert max(rel_l2(got[g], o[g]) for g in range(G)) <= OUT_TOL
            np.testing.assert_allclose(lse[s, hs].double().cpu().numpy(), l, atol=LSE_TOL)


@pytest.mark.parametrize("S,Hkv,G,budget,page,q,splits", [
    (1, 1, 1, 256, 16, "fp32", 16),       # a unit a block
    (1, 1, 7, 4096, 32, "bf16", 64),      # 256 units: at most 64 splits
    (2, 2, 16, 4096, 16, "bf16", 64),     # 1,024 blocks with the heads' further blocks
    (4, 2, 16, 2048, 16, "fp32", 32),     # 128 units, 2,048 blocks in 64 splits
    (4, 2, 3, 2048, 64, "bf16", 64),
])
def test_fp32_sparse_attention_splits(S, Hkv, G, budget, page, q, splits):
    """Sparse attention over fp32 caches: the splits that its rule takes (counted in the
    partials that the call leaves behind), and its output over given tables, one of them
    padded and one with a partial last page, against 64 bits."""
    k = budget // page
    n = max(64, 2 * k)
    gen = torch.Generator(device="cuda").manual_seed(13)
    kc, vc = (torch.randn(S * n, Hkv, page, 128, generator=gen, device="cuda") for _ in range(2))
    qq = torch.randn(S, Hkv * G, 128, generator=gen, device="cuda").to(torch.bfloat16 if q == "bf16" else torch.float32)
    pt = torch.randperm(S * n, generator=gen, device="cuda").int().view(S, n)
    sl = torch.full((S,), n * page - 5, dtype=torch.int32, device="cuda")
    ids = torch.stack([torch.randperm(n - 1, generator=gen, device="cuda")[:k].sort()[0]
                       for _ in range(S * Hkv)]).int().view(S, Hkv, k)
    ids[..., -1] = n - 1
    ids[-1, -1, -3:] = -1
    cfg = B.Config(S, Hkv * G, Hkv, 8, budget, n, S * n, B.LOCKS_FP32, DT[q], page_size=page)
    ws = B.alloc_workspace(cfg, "cuda")
    ws.view(torch.int32).fill_(0x7fedcba9)            # a NaN that no partial is
    out, lse = B.sparse_attend(cfg, qq, kc, vc, pt, sl, ids, ws)
    torch.cuda.synchronize()
    written = (ws.view(torch.int32) != 0x7fedcba9).sum().item()
    assert written == S * Hkv * G * splits * 130, written / (S * Hkv * G * 130)
    for s in range(S):
        for h in range(Hkv):
            mine = ids[s, h][ids[s, h] >= 0].long()
            kd, vd = (x[pt[s, mine].long(), h].reshape(-1, 128).double() for x in (kc, vc))
            live = (mine[:, None] * page + torch.arange(page, device="cuda")).view(-1) < sl[s]
            z = torch.matmul(qq[s, h * G:(h + 1) * G].double(), kd.t().contiguous()) / 128 ** 0.5
            z = z.masked_fill(~live, -float("inf"))
            want = torch.matmul(torch.softmax(z, -1), vd)
            got = out[s, h * G:(h + 1) * G].double()
            assert ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item() <= 1e-5
            assert (lse[s, h * G:(h + 1) * G].double() - torch.logsumexp(z, -1)).abs().max().item() <= 1e-5


@pytest.mark.parametrize("name,G,page,copies,pool,splits", [
    ("half", 4, 16, 1, 16640, 10),          # 520 blocks, and a pool that can fill them
    ("half", 2, 32, 1, 16640, 10),
    ("whole, small pool", 1, 16, 1, 16000, 5),      # the pool fills 500 of the 520 at most
    ("whole, large grid", 4, 16, 2, 16000, 5),      # 1,040 blocks
    ("whole, no room", 16, 64, 1, 16640, 5),        # halved partials exceed the workspace
])
def test_dense_attention_splits_of_long_batches(name, G, page, copies, pool, splits):
    """Dense attention whose blocks hold 256 units, and where its rule halves them, 128,
    several of them a sequence (counted in the partials that the call leaves behind): empty
    sequences, single tokens, lengths on and just past a wave's and a block's units, odd
    counts of units.  pool: 16-token units per KV head in the cache."""
    lens = [20480, 0, 1, 1024, 1025, 4096, 4097, 2048, 2049, 16 * 129, 16 * 385 + 5, 20479, 12345]
    Hkv, sub = 8, page // 16
    S, nb, mp = len(lens) * copies, pool // sub, 20480 // page
    gen = torch.Generator(device="cuda").manual_seed(7)
    k, v = (torch.randn(nb, Hkv, page, 128, generator=gen, device="cuda", dtype=torch.bfloat16)
            for _ in range(2))
    q = torch.randn(len(lens), Hkv * G, 128, generator=gen, device="cuda").to(torch.bfloat16)
    pt = torch.randperm(nb, generator=gen, device="cuda")[torch.arange(len(lens) * mp, device="cuda") % nb]
    pt = pt.int().view(len(lens), mp)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    cfg = B.Config(S, Hkv * G, Hkv, 8, 2 * page, mp, nb, page_size=page)
    ws = B.alloc_workspace(cfg, "cuda")
    ws.view(torch.int32).fill_(0x7fedcba9)            # a NaN that no partial is
    out, lse = B.dense_attend(cfg, q.repeat(copies, 1, 1), k, v, pt.repeat(copies, 1), sl.repeat(copies), ws)
    torch.cuda.synchronize()
    written = torch.nonzero(ws.view(torch.int32) != 0x7fedcba9).max().item() + 1
    assert written == S * Hkv * G * splits * 130, written / (S * Hkv * G * 130)
    for c in range(1, copies):
        assert torch.equal(out[c * len(lens):(c + 1) * len(lens)], out[:len(lens)])
    for s, L in enumerate(lens):
        if L == 0:
            assert not out[s].any() and torch.isneginf(lse[s]).all()
            continue
        n = -(-L // page)
        kd, vd = (x[pt[s, :n].long()].transpose(0, 1).reshape(Hkv, n * page, 128)[:, :L].double()
                  for x in (k, v))
        z = torch.matmul(q[s].double().view(Hkv, G, 128), kd.transpose(1, 2).contiguous()) / 128 ** 0.5
        want_l = torch.logsumexp(z, -1).view(-1)
        want = torch.matmul(torch.softmax(z, -1), vd).view(-1, 128)
        err = (out[s].double() - want).norm(dim=-1) / want.norm(dim=-1)
        assert err.max().item() <= OUT_TOL, (s, L, err.max().item())
        assert (lse[s].double() - want_l).abs().max().item() <= LSE_TOL


@pytest.mark.parametrize("G,copies", [(4, 1), (4, 86), (2, 86), (4, 172), (16, 172)])
def test_selection_chunk_sizes(G, copies):
    """Selection in chunks of 512, 1,024 and 2,048 pages (the size grows with the
    batch): three sequences that end just past a chunk, inside one and below the budget,
    repeated until the grid takes the size.  The first copy is held to the oracle, the
    others equal it."""
    d = _dev("chunks", 3, G, 2, [16 * 2050 + 5, 16 * 1025 + 1, 16 * 40], 8, 2048, "bf16", "bf16")
    store, recs = d.oracle_summaries()
    refs, _ = _scores_against_oracle(d, store, recs)
    d.cfg.num_seqs = 3 * copies
    d.q, d.pt, d.sl = d.q.repeat(copies, 1, 1), d.pt.repeat(copies, 1), d.sl.repeat(copies)
    d.ws = B.alloc_workspace(d.cfg, d.device)
    ids, sel, out, lse = B.decode_step(d.cfg, d.q, d.k, d.v, d.pt, d.sl, store, d.ws)
    ids2, sel2 = B.select(d.cfg, d.q, store, d.pt, d.sl, d.ws)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids2)
    for t in (ids, sel, out, lse):
        c = t.view(torch.int32).view(copies, 3, *t.shape[1:])  # bits: open pages' scores are NaN
        assert torch.equal(c, c[:1].expand_as(c))
    _step_against_oracle(d, refs, ids, sel, out, lse)


@pytest.mark.parametrize("G,page,q,kv,copies", [
    (1, 16, "fp32", "fp32", 1), (3, 32, "bf16", "fp32", 1), (5, 16, "fp32", "bf16", 1),
    (16, 64, "fp32", "fp32", 1), (5, 16, "fp32", "fp32", 172), (1, 16, "bf16", "fp32", 172),
    (4, 16, "bf16", "bf16", 172), (16, 32, "bf16", "bf16", 172)])
def test_attention_head_groups_and_whole_lists(G, page, q, kv, copies):
    """Attention of fp32 tensors at every count of heads a block can hold, and lists that
    one block takes whole (many sequences): lengths around a page, a single token, an empty
    sequence, list entries left open; K and V 4 or 2 bytes off a 16-byte boundary where the
    vector-ALU kernel reads them."""
    lens = [page * 9 + 3, 1, 0, page * 8]
    spec = WorkloadSpec("groups", len(lens), 2 * G, 2, lens, 8, 12 * page, kv, q, page_size=page)
    d = Dev(build_workload(spec, 29))
    c = d.cfg
    ids = torch.full((len(lens), 2, c.k), -1, dtype=torch.int32, device=d.device)
    for s, L in enumerate(lens):
        n = -(-L // page)
        ids[s, :, :n] = torch.arange(n, device=d.device)
    want = [[O.dense_step(*(d.unit(s, h)[i] for i in (2, 0, 1))) if lens[s] else None
             for h in range(2)] for s in range(len(lens))]
    if kv == "fp32" or q == "fp32":
        def off(t):
            buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
            buf[1:] = t.flatten()
            return buf[1:].view(t.shape)
        d.k, d.v, d.q = off(d.k), off(d.v), off(d.q)
    c.num_seqs = len(lens) * copies
    d.q, d.pt, d.sl = d.q.repeat(copies, 1, 1) if copies > 1 else d.q, \
        d.pt.repeat(copies, 1), d.sl.repeat(copies)
    d.ws = B.alloc_workspace(c, d.device)
    for out, lse in (B.sparse_attend(c, d.q, d.k, d.v, d.pt, d.sl, ids.repeat(copies, 1, 1), d.ws),
                     B.dense_attend(c, d.q, d.k, d.v, d.pt, d.sl, d.ws)):
        torch.cuda.synchronize()
        for t in (out, lse):
            x = t.view(copies, len(lens), *t.shape[1:])
            assert torch.equal(x, x[:1].expand_as(x))
        for s in range(len(lens)):
            for h in range(2):
                hs = slice(h * G, (h + 1) * G)
                got = out[s, hs].double().cpu().numpy()
                if not lens[s]:
                    assert not got.any() and torch.isneginf(lse[s, hs]).all()
                    continue
                o, l = want[s][h]
                assert max(rel_l2(got[g], o[g]) for g in range(G)) <= OUT_TOL
                np.testing.assert_allclose(lse[s, hs].double().cpu().numpy(), l, atol=LSE_TOL)
