"""GPU parity, all KV resident in HBM: metadata, block scores, top-k
selection and sparse attention against the CPU oracle, through the C ABI.

Cases span several tiles with ragged tails, sequences shorter than k, an
empty sequence, GQA groups of 1, 4, 7 and 16, blocks of 8, 16 and 32
tokens, k equal to and above the block count (dense attention), exact score
ties, and the tiny and Llama-3-8B-shaped workloads at their full sizes.
"""
import math
import zlib

import numpy as np
import pytest
import torch

import gpu_util as gu
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ss():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2509_24626_amd import binding
    binding.lib()
    return binding


CASES = {
    # name: B, Hq, Hkv, blk, nblk_max, k, n_plant, nblk
    "tiny-b2-h8kv2-ctx4k": (2, 8, 2, 16, 256, 16, 8, None),
    "ragged-short-empty": (3, 8, 2, 16, 40, 16, 0, [40, 7, 0]),
    "gqa7-blk8-ragged": (2, 28, 4, 8, 300, 24, 0, [300, 123]),
    "gqa1-blk32": (2, 4, 4, 32, 64, 8, 0, None),
    "gqa16-blk16": (1, 32, 2, 16, 100, 10, 0, None),
    "k-equals-blocks": (2, 8, 2, 16, 20, 20, 0, None),
    "k-above-blocks": (2, 8, 2, 16, 20, 32, 0, [20, 13]),
}



def _random_cases(n, seed):
    """Seeded extra shapes: heads and group size (1 to 16), block size,
    nblk_max, k (1 to 200, often above some sequences' block counts) and
    ragged block counts, empty sequences included."""
    rng = np.random.default_rng(seed)
    out = {}
    for i in range(n):
        Hkv = int(rng.choice([1, 2, 4, 8]))
        G = int(rng.choice([1, 2, 4, 7, 16]))
        blk = int(rng.choice([8, 16, 32]))
        nmax = int(rng.integers(1, 700))
        k = int(rng.choice([1, 5, 16, 64, 200]))
        B = int(rng.integers(1, 6))
        nblk = [int(x) for x in rng.integers(0, nmax + 1, size=B)]
        out[f"random-{seed}-{i}"] = (B, Hkv * G, Hkv, blk, nmax, k, 0, nblk)
    return out


CASES.update(_random_cases(8, 17))

_cache = {}


def workload(name):
    if name not in _cache:
        B, Hq, Hkv, blk, nmax, k, npl, nblk = CASES[name]
        print(f"[gpu] workload {name}: B={B} Hq={Hq} Hkv={Hkv} blk={blk} nblk_max={nmax} k={k}", flush=True)
        _cache[name] = gu.HbmWorkload(B, Hq, Hkv, blk, nmax, k, seed=zlib.crc32(name.encode()) % 1000, n_plant=npl, nblk=nblk)
    return _cache[name]


def oracle_meta(oracle_impl, w):
    return oracle_impl.build_metadata(w.kv_host, w.unit_off_host, w.nblk_host, w.B, w.Hkv, w.nblk_max, w.blk, w.d)


def valid_rows_equal(a, b, nblk):
    for bb in range(a.shape[0]):
        n = int(nblk[bb])
        np.testing.assert_array_equal(a[bb, :, :n], b[bb, :, :n])


@pytest.mark.parametrize("name", list(CASES))
def test_metadata_bitexact(ss, oracle_impl, name):
    w = workload(name)
    meta = gu.run_metadata(ss, w)
    torch.cuda.synchronize()
    valid_rows_equal(gu.u16(meta), oracle_meta(oracle_impl, w), w.nblk_host)


@pytest.mark.parametrize("name", list(CASES))
def test_scores_and_selection(ss, oracle_impl, name):
    w = workload(name)
    meta = gu.run_metadata(ss, w)
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    sel = torch.empty(w.B, w.Hkv, w.k, dtype=torch.int32, device="cuda")
    ss.ss_score_topk(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, w.k, scores, sel)
    torch.cuda.synchronize()
    om = oracle_meta(oracle_impl, w)
    S = oracle_impl.score(w.q_host, om, w.nblk_host, w.Hq, w.Hkv, w.nblk_max, w.d)
    osel = oracle_impl.select(S, w.nblk_host, w.k)
    worst = gu.check_scores(scores.cpu().numpy(), S, w.q_host, om, w.nblk_host, w.Hq // w.Hkv)
    diff = gu.check_selection(sel.cpu().numpy(), osel, S, w.nblk_host, w.k)
    print(f"[gpu] {name}: worst relative score error {worst:.2e}; units with tie-band differences {len(diff)}")


@pytest.mark.parametrize("name", list(CASES))
def test_metadata_mean_bitexact(ss, oracle_impl, name):
    """Mean-key metadata: the exact mean of each block's keys rounded once to bf16, bit-exact."""
    w = workload(name)
    meta = torch.empty(w.B, w.Hkv, w.nblk_max, w.d, dtype=torch.int16, device="cuda")
    ss.ss_build_metadata_mean(w.kv, w.unit_off, w.nblk, w.B, w.Hkv, w.nblk_max, w.blk, w.d, meta)
    torch.cuda.synchronize()
    om = oracle_impl.build_metadata_mean(w.kv_host, w.unit_off_host, w.nblk_host, w.B, w.Hkv, w.nblk_max, w.blk, w.d)
    valid_rows_equal(gu.u16(meta), om, w.nblk_host)


def test_metadata_mean_rounds_once(ss):
    """The hand-worked mean-key fixture (golden/mean_key_rounding.txt) on the
    GPU, through ss_build_metadata_mean and through the fill path of
    ss_append_kv: a mean 2^-25 above a rounding midpoint (which a rounding
    through fp32 would tie the other way), exact midpoints tying to even
    both ways, and a negative mean.  The fixture's 4 channels repeat over
    the 128."""
    import pins
    fx = pins.read_fixture("mean_key_rounding.txt")
    blk, d = int(fx["blk"][0]), 128
    rows = [[float(x) for x in fx["token_0_to_29"]]] * 30 + [[float(x) for x in fx["token_30"]],
                                                              [float(x) for x in fx["token_31"]]]
    K = torch.tensor(np.tile(np.array(rows), (1, d // 4)), dtype=torch.float32).to(torch.bfloat16)  # [blk][d]
    assert torch.equal(K.float(), torch.tensor(np.tile(np.array(rows), (1, d // 4)), dtype=torch.float32))
    want = np.tile(np.array([float(x) for x in fx["mean_key"]]), d // 4)
    rec = torch.zeros(2 * blk * d, dtype=torch.bfloat16)
    rec[:blk * d] = K.reshape(-1)
    rec = rec.cuda()
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    meta = torch.zeros(1, 1, 1, d, dtype=torch.int16, device="cuda")
    ss.ss_build_metadata_mean(rec, torch.zeros(1, dtype=torch.int64, device="cuda"), one, 1, 1, 1, blk, d, meta)
    got = meta.view(torch.bfloat16).float().cpu().numpy().reshape(-1)
    np.testing.assert_array_equal(got, want)
    # the same block filled token by token: its metadata row is written by the append of token 31
    length = torch.zeros(1, dtype=torch.int32, device="cuda")
    nblk = torch.zeros(1, dtype=torch.int32, device="cuda")
    open_rec = torch.zeros(1, 1, 2 * blk * d, dtype=torch.int16, device="cuda")
    meta2 = torch.zeros(1, 1, 1, d, dtype=torch.int16, device="cuda")
    for t in range(blk):
        kv = torch.zeros(1, 1, 2, d, dtype=torch.bfloat16)
        kv[0, 0, 0] = K[t]
        ss.ss_append_kv(kv.cuda(), length, nblk, 1, 1, blk, d, 1, open_rec, meta2, None, meta_kind=ss.SS_META_MEAN)
    torch.cuda.synchronize()
    assert int(nblk.item()) == 1 and int(length.item()) == blk
    got2 = meta2.view(torch.bfloat16).float().cpu().numpy().reshape(-1)
    np.testing.assert_array_equal(got2, want)


@pytest.mark.parametrize("kind,agg", [(0, 1), (1, 0), (1, 1)], ids=["cuboid-sum", "mean-max", "mean-sum"])
@pytest.mark.parametrize("name", list(CASES))
def test_score_variants_and_selection(ss, oracle_impl, name, kind, agg):
    w = workload(name)
    if kind == 0:
        meta = gu.run_metadata(ss, w)
        om = oracle_meta(oracle_impl, w)
    else:
        meta = torch.empty(w.B, w.Hkv, w.nblk_max, w.d, dtype=torch.int16, device="cuda")
        ss.ss_build_metadata_mean(w.kv, w.unit_off, w.nblk, w.B, w.Hkv, w.nblk_max, w.blk, w.d, meta)
        om = oracle_impl.build_metadata_mean(w.kv_host, w.unit_off_host, w.nblk_host, w.B, w.Hkv, w.nblk_max, w.blk,
                                             w.d)
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    sel = torch.empty(w.B, w.Hkv, w.k, dtype=torch.int32, device="cuda")
    ss.ss_score_blocks_variant(w.q, meta, kind, agg, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, scores)
    ss.ss_select_topk(scores, w.nblk, w.B, w.Hkv, w.nblk_max, w.k, sel)
    torch.cuda.synchronize()
    S = oracle_impl.score_variant(w.q_host, om, kind, agg, w.nblk_host, w.Hq, w.Hkv, w.nblk_max, w.d)
    osel = oracle_impl.select(S, w.nblk_host, w.k)
    worst = gu.check_scores_variant(scores.cpu().numpy(), S, w.q_host, om, w.nblk_host, w.Hq // w.Hkv, kind, agg)
    diff = gu.check_selection(sel.cpu().numpy(), osel, S, w.nblk_host, w.k)
    print(f"[gpu] {name} kind={kind} agg={agg}: worst relative score error {worst:.2e}; tie-band units {len(diff)}")


def test_score_variant_rejects_unknown_kind(ss):
    w = workload("tiny-b2-h8kv2-ctx4k")
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    for kind, agg in ((2, 0), (0, 2), (-1, 0)):
        with pytest.raises(ss.SparseServeError):
            ss.ss_score_blocks_variant(w.q, scores, kind, agg, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, scores)


@pytest.mark.parametrize("name", list(CASES))
def test_attention_on_oracle_selection(ss, oracle_impl, name):
    w = workload(name)
    om = oracle_meta(oracle_impl, w)
    S = oracle_impl.score(w.q_host, om, w.nblk_host, w.Hq, w.Hkv, w.nblk_max, w.d)
    osel = oracle_impl.select(S, w.nblk_host, w.k)
    out = gu.run_attention(ss, w, torch.from_numpy(osel).cuda())
    torch.cuda.synchronize()
    ref = oracle_impl.attention(w.q_host, w.kv_host, w.unit_off_host, osel, w.Hkv, w.blk)
    err = np.abs(out.cpu().numpy() - ref).max()
    print(f"[gpu] {name}: attention max abs error {err:.2e}")
    assert err <= gu.ATTN_TOL


@pytest.mark.parametrize("name", ["tiny-b2-h8kv2-ctx4k", "gqa7-blk8-ragged", "ragged-short-empty"])
def test_end_to_end_step(ss, oracle_impl, name):
    """GPU selection feeds GPU attention; units whose selection equals the
    oracle's must match the oracle's attention."""
    w = workload(name)
    meta = gu.run_metadata(ss, w)
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    sel = torch.empty(w.B, w.Hkv, w.k, dtype=torch.int32, device="cuda")
    ss.ss_score_topk(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, w.k, scores, sel)
    out = gu.run_attention(ss, w, sel).cpu().numpy()
    om = oracle_meta(oracle_impl, w)
    S = oracle_impl.score(w.q_host, om, w.nblk_host, w.Hq, w.Hkv, w.nblk_max, w.d)
    osel = oracle_impl.select(S, w.nblk_host, w.k)
    ref = oracle_impl.attention(w.q_host, w.kv_host, w.unit_off_host, osel, w.Hkv, w.blk)
    gsel = sel.cpu().numpy()
    G = w.Hq // w.Hkv
    compared = 0
    for b in range(w.B):
        for g in range(w.Hkv):
            if np.array_equal(gsel[b, g], osel[b, g]):
                compared += 1
                assert np.abs(out[b, g * G:(g + 1) * G] - ref[b, g * G:(g + 1) * G]).max() <= gu.ATTN_TOL
    assert compared >= w.units - 1


def test_planted_blocks_are_selected(ss):
    """Sanity (not parity): on the tiny workload every planted block is
    among the selected blocks of its KV head."""
    B, Hq, Hkv, blk, nmax, k, npl, _ = CASES["tiny-b2-h8kv2-ctx4k"]
    seed = zlib.crc32(b"tiny-b2-h8kv2-ctx4k") % 1000
    w = workload("tiny-b2-h8kv2-ctx4k")
    meta = gu.run_metadata(ss, w)
    scores = torch.empty(B, Hkv, nmax, dtype=torch.float32, device="cuda")
    sel = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
    ss.ss_score_topk(w.q, meta, w.nblk, B, Hq, Hkv, nmax, 128, k, scores, sel)
    gsel = sel.cpu().numpy()
    for b in range(B):
        for g in range(Hkv):
            planted = synth.gen.planted_blocks(nmax, npl, seed, 0, b, g, "cuda").cpu().numpy()
            assert set(planted.tolist()) <= set(gsel[b, g].tolist())


def test_scores_at_the_largest_block_count(ss, oracle_impl):
    """Scoring and selection at 65536 blocks per unit (the largest supported)
    with a ragged second sequence: each wave's staged tiles past a
    sequence's end read zeros through the buffer bounds and nothing is
    written past the end; scores and selection match the oracle."""
    rng = np.random.default_rng(21)
    B, Hq, Hkv, nmax, k = 2, 8, 2, 65536, 128
    nblk = np.array([65536, 40001], np.int32)
    a = torch.from_numpy(rng.standard_normal((B, Hkv, nmax, 128)).astype(np.float32))
    c = torch.from_numpy(rng.standard_normal((B, Hkv, nmax, 128)).astype(np.float32))
    meta = torch.stack([torch.minimum(a, c), torch.maximum(a, c)], 3).bfloat16().cuda().contiguous()
    del a, c
    q = torch.from_numpy(rng.standard_normal((B, Hq, 128)).astype(np.float32)).bfloat16().cuda()
    scores = torch.full((B, Hkv, nmax), 7.0, dtype=torch.float32, device="cuda")
    sel = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
    ss.ss_score_topk(q, meta, torch.from_numpy(nblk).cuda(), B, Hq, Hkv, nmax, 128, k, scores, sel)
    torch.cuda.synchronize()
    q_host = gu.u16(q)
    meta_host = gu.u16(meta)
    S = oracle_impl.score(q_host, meta_host, nblk, Hq, Hkv, nmax, 128)
    got = scores.cpu().numpy()
    assert np.all(got[1, :, 40001:] == 7.0), "scores written past the sequence's end"
    gu.check_scores(got, S, q_host, meta_host, nblk, Hq // Hkv)
    gu.check_selection(sel.cpu().numpy(), oracle_impl.select(S, nblk, k), S, nblk, k)


def test_topk_exact_ties(ss, oracle_impl):
    """Scores drawn from a handful of values (massive exact ties, +0 and -0,
    negatives): the GPU selection must equal the oracle's bit for bit."""
    rng = np.random.default_rng(5)
    for B, Hkv, nmax, k, nblk in [(2, 3, 1000, 37, [1000, 999]), (1, 2, 5000, 512, [5000]),
                                  (2, 2, 300, 300, [300, 17]), (1, 1, 16384, 512, [16384]),
                                  (3, 1, 64, 1, [64, 1, 2]), (1, 2, 4096, 128, [4096]), (1, 1, 30000, 700, [30000])]:
        vals = np.array([-3.5, -0.0, 0.0, 1.25, 1.25000012, 7.0, 246.0], np.float32)
        sc = vals[rng.integers(0, len(vals), size=(B, Hkv, nmax))]
        sel = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
        ss.ss_select_topk(torch.from_numpy(sc).cuda(), torch.tensor(nblk, dtype=torch.int32, device="cuda"), B, Hkv,
                          nmax, k, sel)
        ref = oracle_impl.select(sc.astype(np.float64), np.array(nblk, np.int32), k)
        np.testing.assert_array_equal(sel.cpu().numpy(), ref)


def test_topk_random_scores_match(ss, oracle_impl):
    """Continuous random scores (no ties) at the workloads' block counts and
    in every workgroup-width class of the kernel (up to 65536 blocks)."""
    rng = np.random.default_rng(6)
    for nmax, k in [(256, 16), (2048, 128), (4096, 128), (8192, 128), (16384, 512), (700, 699), (40000, 256),
                    (65536, 128)]:
        sc = (246 + 21 * rng.standard_normal((2, 2, nmax))).astype(np.float32)
        sel = torch.empty(2, 2, k, dtype=torch.int32, device="cuda")
        ss.ss_select_topk(torch.from_numpy(sc).cuda(), torch.full((2,), nmax, dtype=torch.int32, device="cuda"), 2, 2,
                          nmax, k, sel)
        ref = oracle_impl.select(sc.astype(np.float64), np.full(2, nmax, np.int32), k)
        np.testing.assert_array_equal(sel.cpu().numpy(), ref)


def test_topk_clustered_scores(ss, oracle_impl):
    """Score rows whose first radix digit takes one or a few values (a narrow
    band with far outliers, mixed signs, a single value with one larger),
    rows shorter than k and empty rows: the selections equal the oracle's."""
    rng = np.random.default_rng(11)
    B, Hkv, nmax, k = 4, 4, 8192, 128
    rows = []
    band = 30 + 1e-3 * rng.standard_normal(nmax)
    out = band.copy()
    out[::97] += 5e4  # 85 outliers, then the band
    rows.append(out)
    rows.append(0.5 * rng.standard_normal(nmax))  # mixed signs around zero
    one = np.full(nmax, 7.0)
    one[4000] = 8.0
    rows.append(one)  # massive ties below one larger value
    rows.append(np.concatenate([np.full(nmax // 2, -1.0), 1e-30 * np.arange(nmax // 2)]))  # subnormals and -1
    rows.append(np.where(rng.random(nmax) < 0.02, 1e6, 1.0) + 1e-3 * rng.standard_normal(nmax))  # ~164 above the rest
    rows.append(np.round(rng.standard_normal(nmax), 1))  # few distinct values
    while len(rows) < B * Hkv:
        rows.append(246 + 21 * rng.standard_normal(nmax))
    sc = np.stack(rows).reshape(B, Hkv, nmax).astype(np.float32)
    for nblk in ([nmax] * B, [nmax, 100, 0, 129]):
        sel = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
        ss.ss_select_topk(torch.from_numpy(sc).cuda(), torch.tensor(nblk, dtype=torch.int32, device="cuda"), B, Hkv,
                          nmax, k, sel)
        ref = oracle_impl.select(sc.astype(np.float64), np.array(nblk, np.int32), k)
        np.testing.assert_array_equal(sel.cpu().numpy(), ref)


def test_attention_skips_invalid_slots(ss, oracle_impl):
    """-1 entries anywhere and slots >= slot_limit are skipped."""
    w = workload("gqa1-blk32")  # B=2, Hq=Hkv=4, blk 32, 64 blocks, k=8
    slots = np.array([[[3, -1, 7, 70, 0, -1, 63, 5],
                       [-1, -1, -1, -1, -1, -1, -1, -1],
                       [64, 65, 1000, -1, 2, -1, -1, -1],
                       [10, 11, 12, 13, 14, 15, 16, 17]],
                      [[1, 2, 3, 4, 5, 6, 64, 65],
                       [10, -1, 11, -1, 12, -1, 13, -1],
                       [-1, -1, -1, -1, -1, -1, -1, 9],
                       [63, 62, 61, 60, 59, 58, 57, 56]]], np.int32)
    out = gu.run_attention(ss, w, torch.from_numpy(slots).cuda(), slot_limit=64).cpu().numpy()
    ora_slots = np.where(slots >= 64, -1, slots)
    ref = oracle_impl.attention(w.q_host, w.kv_host, w.unit_off_host, ora_slots, w.Hkv, w.blk)
    assert np.abs(out - ref).max() <= gu.ATTN_TOL
    assert np.all(out[0, 1] == 0)  # every entry skipped -> zero output


def test_attention_bounds_slots_by_unit_capacity(ss, oracle_impl):
    """With per-unit capacities, a slot at or above its unit's own capacity
    is skipped even when it lies below slot_limit.  The over-capacity slots
    sit in units that are not last, so each one addresses bytes inside the
    allocation (in the unit's 64-record region): reading it would not fault,
    and would change the output."""
    w = workload("gqa1-blk32")  # B=2, Hq=Hkv=4, blk 32, 64 records per unit, k=8
    cap = np.array([64, 10, 0, 30, 64, 5, 64, 20], np.int32)
    slots = np.array([[[3, 9, 7, 40, 0, 63, 62, 5],
                       [9, 10, 11, 40, 0, 1, 2, -1],
                       [0, 1, 2, 3, 4, 5, 6, 7],
                       [29, 30, 31, 50, 1, -1, 2, 3]],
                      [[1, 2, 3, 4, 5, 6, 64, 65],
                       [4, 5, 6, 7, 8, 0, 1, 63],
                       [10, -1, 11, -1, 12, -1, 13, 60],
                       [19, 20, 21, 0, 22, 1, 2, 3]]], np.int32)
    assert np.any((slots >= cap.reshape(2, 4, 1)) & (slots < 64))
    out = gu.run_attention(ss, w, torch.from_numpy(slots).cuda(), slot_limit=64,
                           capacity=torch.from_numpy(cap).cuda()).cpu().numpy()
    ora_slots = np.where((slots >= cap.reshape(2, 4, 1)) | (slots >= 64), -1, slots)
    ref = oracle_impl.attention(w.q_host, w.kv_host, w.unit_off_host, ora_slots, w.Hkv, w.blk)
    assert np.abs(out - ref).max() <= gu.ATTN_TOL
    assert np.all(out[0, 2] == 0)  # capacity 0: every entry skipped
    # without the capacities the same slots are read (the bound is what skips them)
    out_nocap = gu.run_attention(ss, w, torch.from_numpy(slots).cuda(), slot_limit=64).cpu().numpy()
    assert np.abs(out_nocap[0, 1] - ref[0, 1]).max() > 1e-3


def test_runs_are_bitwise_deterministic(ss):
    w = workload("gqa7-blk8-ragged")
    meta = gu.run_metadata(ss, w)
    res = []
    for _ in range(2):
        scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
        sel = torch.empty(w.B, w.Hkv, w.k, dtype=torch.int32, device="cuda")
        ss.ss_score_topk(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, w.k, scores, sel)
        out = gu.run_attention(ss, w, sel)
        res.append((sel.cpu().numpy(), out.cpu().numpy()))
    np.testing.assert_array_equal(res[0][0], res[1][0])
    np.testing.assert_array_equal(res[0][1].view(np.uint32), res[1][1].view(np.uint32))


def test_kernel_timing_hook(ss):
    """ss_time_next_kernel: the attached events bracket exactly one kernel
    (within the stream-recorded bracket around the same call), the call's
    result is unchanged, and the setting is consumed by that launch."""
    w = workload("gqa7-blk8-ragged")
    meta = gu.run_metadata(ss, w)
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    ref = torch.empty_like(scores)
    ss.ss_score_blocks(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, ref)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    torch.cuda.synchronize()
    ev[0].record()
    ss.ss_time_next_kernel(ev[1], ev[2])
    ss.ss_score_blocks(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, scores)
    ev[3].record()
    torch.cuda.synchronize()
    inner, outer = ev[1].elapsed_time(ev[2]), ev[0].elapsed_time(ev[3])
    print(f"[gpu] kernel {inner * 1e3:.1f} us inside a {outer * 1e3:.1f} us bracket", flush=True)
    assert 0 < inner <= outer
    assert ev[0].elapsed_time(ev[1]) >= 0 and ev[2].elapsed_time(ev[3]) >= 0
    valid_rows_equal(scores.cpu().numpy(), ref.cpu().numpy(), w.nblk_host)
    # consumed: the next launch does not touch the events again
    ss.ss_score_blocks(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, scores)
    torch.cuda.synchronize()
    assert ev[1].elapsed_time(ev[2]) == inner
    ss.ss_time_next_kernel(None, None)


def test_llama3_8b_shape_full_size(ss, oracle_impl):
    """The Llama-3-8B-shaped single layer at full size (B=32, 32/8 heads,
    32k context, blk 16, k=128, 64 planted blocks per head), every unit
    checked against the oracle."""
    cfg = synth.get(1)
    print(f"[gpu] {cfg.name}: generating", flush=True)
    w = gu.HbmWorkload(cfg.B, cfg.Hq, cfg.Hkv, cfg.blk, cfg.nblk_max, cfg.k, seed=0, n_plant=cfg.n_plant)
    meta = gu.run_metadata(ss, w)
    scores = torch.empty(w.B, w.Hkv, w.nblk_max, dtype=torch.float32, device="cuda")
    sel = torch.empty(w.B, w.Hkv, w.k, dtype=torch.int32, device="cuda")
    ss.ss_score_topk(w.q, meta, w.nblk, w.B, w.Hq, w.Hkv, w.nblk_max, w.d, w.k, scores, sel)
    out = gu.run_attention(ss, w, sel).cpu().numpy()
    gmeta = gu.u16(meta)
    print(f"[gpu] {cfg.name}: oracle", flush=True)
    om = oracle_meta(oracle_impl, w)
    np.testing.assert_array_equal(gmeta, om)
    S = oracle_impl.score(w.q_host, om, w.nblk_host, w.Hq, w.Hkv, w.nblk_max, w.d)
    osel = oracle_impl.select(S, w.nblk_host, w.k)
    gu.check_scores(scores.cpu().numpy(), S, w.q_host, om, w.nblk_host, w.Hq // w.Hkv)
    diff = gu.check_selection(sel.cpu().numpy(), osel, S, w.nblk_host, w.k)
    ref = oracle_impl.attention(w.q_host, w.kv_host, w.unit_off_host, osel, w.Hkv, w.blk)
    G = w.Hq // w.Hkv
    worst = 0.0
    for b in range(w.B):
        for g in range(w.Hkv):
            if (b, g) not in diff:
                worst = max(worst, float(np.abs(out[b, g * G:(g + 1) * G] - ref[b, g * G:(g + 1) * G]).max()))
    # attention on the oracle's own selection covers every unit
    out2 = gu.run_attention(ss, w, torch.from_numpy(osel).cuda()).cpu().numpy()
    worst2 = float(np.abs(out2 - ref).max())
    print(f"[gpu] {cfg.name}: tie-band units {len(diff)}, attention err {worst:.2e} / {worst2:.2e}")
    assert worst <= gu.ATTN_TOL and worst2 <= gu.ATTN_TOL


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("blk,Hkv,tokens,token_major", [(8, 3, 1003, True), (16, 2, 37, False), (32, 1, 999, True),
                                                        (8, 8, 90011, False), (16, 8, 90011, True),
                                                        (32, 8, 90011, True), (16, 8, 90011, False)])
def test_metadata_launch_shapes(ss, kind, blk, Hkv, tokens, token_major):
    """Metadata of two sequences, one a few blocks short of the other, from
    token-major KV and from block records, with fewer keys than kLargeBytes
    and with more (90011 tokens of 8 heads, both sequences: 352 MiB); block
    counts that end inside a wave's group.  Bit-exact against min/max over
    totalOrder keys and the fp64 mean rounded once, computed here; rows past
    a sequence's count keep what they held."""
    d, B = 128, 2
    n = tokens // blk
    nblk = torch.tensor([n, n - min(n - 1, 5)], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(tokens * 64 + blk)
    shape = (B, n * blk, Hkv, 2, d) if token_major else (B, Hkv, n, 2, blk, d)
    kv = torch.randn(shape, generator=g, device="cuda").bfloat16()
    kv.view(-1)[::97] = -0.0
    kv.view(-1)[::89] = 0.0
    rec = blk * 2 * d * 2
    if token_major:
        row, step = Hkv * 2 * d * 2, blk * Hkv * 2 * d * 2
        off = [b * n * step + h * 2 * d * 2 for b in range(B) for h in range(Hkv)]
        keys = kv[:, :, :, 0].unflatten(1, (n, blk)).permute(0, 3, 1, 2, 4)
    else:
        row, step = d * 2, rec
        off = [(b * Hkv + h) * n * rec for b in range(B) for h in range(Hkv)]
        keys = kv[:, :, :, 0]
    off = torch.tensor(off, dtype=torch.int64, device="cuda")
    meta = torch.full((B, Hkv, n) + ((2, d) if kind == 0 else (d,)), 0x7ABC, dtype=torch.int16, device="cuda")
    print(f"[gpu] metadata kind {kind}, blk {blk}, {Hkv} heads, {tokens} tokens, token-major {token_major}", flush=True)
    ss.ss_build_metadata_strided(kv, off, nblk, B, Hkv, n, blk, d, step, row, kind, meta)
    for b in range(B):
        m = int(nblk[b])
        k = keys[b, :, :m].contiguous()
        if kind == 0:
            bits = k.view(torch.int16)
            order = torch.where(bits < 0, bits ^ 0x7FFF, bits)  # totalOrder as signed integers
            lo, hi = order.amin(2), order.amax(2)
            want = torch.stack([torch.where(x < 0, x ^ 0x7FFF, x) for x in (lo, hi)], 2)
        else:
            x = (k.double().sum(2) / blk).view(torch.int64)  # to 8 significant bits, ties to even
            x = ((x + ((1 << 44) - 1) + ((x >> 45) & 1)) >> 45) << 45
            want = x.view(torch.float64).bfloat16().view(torch.int16)
        assert torch.equal(meta[b, :, :m], want)
        assert bool((meta[b, :, m:] == 0x7ABC).all())


@pytest.mark.parametrize("blk,Hkv,B,n,token_major", [
    (8, 8, 513, 4, False), (8, 3, 1400, 1, False), (16, 1, 4096, 2, True), (32, 8, 512, 1, False),  # half a wave a unit
    (8, 8, 512, 4, False), (8, 5, 819, 1, True), (16, 8, 511, 2, False),                              # just fewer units
    (8, 7, 67, 70, False), (16, 8, 700, 3, False), (32, 2, 1400, 3, False), (8, 8, 1, 4097, False),   # by size
    (8, 8, 2100, 5, True), (32, 3, 1400, 5, True)])                                                # and by size past the cache
def test_metadata_rows_across_units(ss, blk, Hkv, B, n, token_major):
    """Many units of few blocks, whose blocks share waves, on either side of
    the lines from which they do: counts of 0 to n in turn, so that units
    begin, end and are missing anywhere in a wave, also in the last one.
    Bit-exact against min/max over totalOrder keys; the rows past a count
    keep what they held."""
    d = 128
    nblk = torch.tensor([(3 * b + b // 7) % (n + 1) for b in range(B)], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(blk * 10000 + B)
    shape = (B, n * blk, Hkv, 2, d) if token_major else (B, Hkv, n, 2, blk, d)
    kv = torch.randn(shape, generator=g, device="cuda").bfloat16()
    kv.view(-1)[::97] = -0.0
    if token_major:
        row, step = Hkv * 2 * d * 2, blk * Hkv * 2 * d * 2
        off = [b * n * step + h * 2 * d * 2 for b in range(B) for h in range(Hkv)]
        keys = kv[:, :, :, 0].unflatten(1, (n, blk)).permute(0, 3, 1, 2, 4)
    else:
        row, step = d * 2, blk * 2 * d * 2
        off = [u * n * step for u in range(B * Hkv)]
        keys = kv[:, :, :, 0]
    off = torch.tensor(off, dtype=torch.int64, device="cuda")
    meta = torch.full((B, Hkv, n, 2, d), 0x7ABC, dtype=torch.int16, device="cuda")
    print(f"[gpu] metadata of {B} x {Hkv} units of {n} blocks of {blk}, token-major {token_major}", flush=True)
    ss.ss_build_metadata_strided(kv, off, nblk, B, Hkv, n, blk, d, step, row, 0, meta)
    bits = keys.contiguous().view(torch.int16)
    order = torch.where(bits < 0, bits ^ 0x7FFF, bits)  # totalOrder as signed integers
    want = torch.stack([torch.where(x < 0, x ^ 0x7FFF, x) for x in (order.amin(3), order.amax(3))], 3)
    live = torch.arange(n, device="cuda")[None] < nblk[:, None]
    want = torch.where(live[:, None, :, None, None], want, torch.full_like(want, 0x7ABC))
    assert torch.equal(meta, want)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("blk,Hkv,n,values", [(16, 4, 10300, True), (8, 2, 41100, True), (16, 1, 41000, True),
                                              (32, 2, 10300, False), (16, 3, 800, True)])
def test_metadata_heads_one_after_another(ss, kind, blk, Hkv, n, values):
    """Keys whose heads lie one after another, [head][token][K, V][d] or, for
    two heads, keys alone with the heads side by side (the same stride): on
    either side of the line to keys that come from HBM, with the heads'
    waves in either order.  Bit-exact as above."""
    d = 128
    g = torch.Generator(device="cuda").manual_seed(n + Hkv)
    if values:
        kv = torch.randn(Hkv, n, blk, 2, d, generator=g, device="cuda").bfloat16()
        keys, row = kv[:, :, :, 0], 2 * d * 2
        off = [h * n * blk * row for h in range(Hkv)]
    else:
        kv = torch.randn(n, blk, Hkv, d, generator=g, device="cuda").bfloat16()
        keys, row = kv.permute(2, 0, 1, 3), Hkv * d * 2
        off = [h * d * 2 for h in range(Hkv)]
    off = torch.tensor(off, dtype=torch.int64, device="cuda")
    nblk = torch.tensor([n - 3], dtype=torch.int32, device="cuda")
    meta = torch.full((Hkv, n) + ((2, d) if kind == 0 else (d,)), 0x7ABC, dtype=torch.int16, device="cuda")
    print(f"[gpu] metadata kind {kind}, {Hkv} heads of {n} blocks of {blk}, values between {values}", flush=True)
    ss.ss_build_metadata_strided(kv, off, nblk, 1, Hkv, n, blk, d, blk * row, row, kind, meta)
    k = keys.contiguous()
    if kind == 0:
        bits = k.view(torch.int16)
        order = torch.where(bits < 0, bits ^ 0x7FFF, bits)
        want = torch.stack([torch.where(x < 0, x ^ 0x7FFF, x) for x in (order.amin(2), order.amax(2))], 2)
    else:
        x = (k.double().sum(2) / blk).view(torch.int64)
        x = ((x + ((1 << 44) - 1) + ((x >> 45) & 1)) >> 45) << 45
        want = x.view(torch.float64).bfloat16().view(torch.int16)
    assert torch.equal(meta[:, :n - 3], want[:, :n - 3]) and bool((meta[:, n - 3:] == 0x7ABC).all())


@pytest.mark.parametrize("n", [1, 2, 63, 65, 256, 257, 512, 513, 1024, 1025, 2049, 4097, 8193, 16385, 65536])
def test_topk_launch_shapes_and_extremes(ss, oracle_impl, n):
    """Either side of the launch shapes' row lengths, rows one score short of
    the row's room among them; rows of the largest and smallest floats with
    infinities (so that the keys span all 32 bits), of subnormals, of one
    value, of neighbouring floats, of outliers above a tight band, and one
    with more equal scores at its bound than the last search takes; every k
    from one block to all of them.  Equal to the oracle's selection."""
    rng = np.random.default_rng(n)
    near = np.arange(n, dtype=np.uint32)
    rng.shuffle(near)
    rows = np.stack([
        np.where(rng.random(n) < 0.5, np.float32(-np.inf), np.finfo(np.float32).max * rng.uniform(-1, 1, n)),
        np.where(rng.random(n) < 0.01, np.float32(np.inf), np.float32(-np.inf)),
        rng.integers(-50, 50, n) * np.float32(1e-45),
        np.full(n, np.float32(-3.0)),
        (np.float32(246).view(np.uint32) + near).view(np.float32),
        np.where(np.arange(n) % 97 == 5, np.float32(5e4), np.float32(30)) + 1e-3 * rng.standard_normal(n),
        np.where(rng.random(n) < 0.9, np.float32(1), rng.standard_normal(n)),
        246 + 21 * rng.standard_normal(n)]).astype(np.float32)
    B, Hkv = 4, 2
    sc = rows.reshape(B, Hkv, n)
    nblk = np.array([n, max(n - 1, 0), n, n // 2], np.int32)
    for k in sorted({1, max(n // 3, 1), max(n - 1, 1), n, n + 3, min(n, 128)}):
        sel = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
        ss.ss_select_topk(torch.from_numpy(sc).cuda(), torch.from_numpy(nblk).cuda(), B, Hkv, n, k, sel)
        ref = oracle_impl.select(sc.astype(np.float64), nblk, k)
        np.testing.assert_array_equal(sel.cpu().numpy(), ref, err_msg=f"n={n} k={k}")


@pytest.mark.parametrize("n", [300, 1000, 2048, 5000, 16384])
def test_topk_clusters_at_the_bound(ss, oracle_impl, n):
    """Clusters of scores around the bound of just fewer, as many and more
    than the last search takes (64), of distinct, of few and of equal values,
    inside a range so wide that one interval holds them all; whole numbers on
    either side of zero, and scores that are mostly zero.  Equal to the
    oracle's selection."""
    rng = np.random.default_rng(n)
    sizes = [63, 64, 65, 129, 280]
    rows, ks = [], []
    for c in sizes:
        for kind in range(3):
            x = np.full(n, -1e30, np.float32)
            at = rng.permutation(n)
            x[at[:10]] = 1e30
            near = 1 + np.arange(c) * np.float32(2.0 ** -22)
            x[at[10:10 + c]] = near if kind == 0 else near[rng.integers(0, 3, c)] if kind == 1 else near[0]
            rows.append(x)
            ks.append(10 + c // 2)
    for x in ((50 * rng.standard_normal(n)).round(), rng.integers(0, 200, n), np.maximum(rng.standard_normal(n), 0),
              rng.standard_normal(n), rng.integers(0, 3, n)):
        rows.append(x.astype(np.float32))
        ks.append(128)
    sc = np.stack(rows)[:, None]
    nblk = np.full(len(rows), n, np.int32)
    for k in sorted(set(ks) | {100}):
        sel = torch.empty(len(rows), 1, k, dtype=torch.int32, device="cuda")
        ss.ss_select_topk(torch.from_numpy(sc).cuda(), torch.from_numpy(nblk).cuda(), len(rows), 1, n, k, sel)
        ref = oracle_impl.select(sc.astype(np.float64), nblk, k)
        np.testing.assert_array_equal(sel.cpu().numpy(), ref, err_msg=f"n={n} k={k}")


@pytest.mark.parametrize("units,G,blk,k", [(1, 16, 8, 1), (3, 4, 16, 15), (3, 4, 16, 31), (2, 7, 16, 32), (5, 7, 8, 65),
                                           (1, 5, 16, 700), (95, 4, 16, 96), (96, 4, 16, 97), (96, 1, 32, 48),
                                           (143, 4, 16, 40), (144, 4, 16, 40), (256, 2, 8, 33), (257, 2, 16, 40),
                                           (341, 1, 16, 33), (383, 2, 16, 32), (384, 2, 16, 32), (511, 1, 16, 33),
                                           (512, 1, 16, 33)])
def test_attention_launch_shapes(ss, units, G, blk, k):
    """Either side of the lines between one workgroup of 8 waves per unit,
    one of 4 waves, and splits; entries that are not selected in between, a
    unit with none, and steps that do not divide among waves and splits.
    Against float64 on the GPU: products are exact and sums 32-bit, so the
    probabilities' 16 bits bound the error, 2^-15 of the largest |V|."""
    d, slots = 128, k + 3
    g = torch.Generator(device="cuda").manual_seed(units * 1000 + k)
    kv = torch.randn(units, slots, 2, blk * d, generator=g, device="cuda").bfloat16()
    q = torch.randn(units, G, d, generator=g, device="cuda").bfloat16()
    sel = torch.rand(units, slots, generator=g, device="cuda").topk(k, dim=1).indices.to(torch.int32)
    sel[torch.rand(units, k, generator=g, device="cuda") < 0.1] = -1
    sel[units // 2] = -1
    cap = torch.full((units,), slots, dtype=torch.int32, device="cuda")
    cap[0] = slots - 2  # two slots of the first unit's region are not its own
    off = torch.arange(units, dtype=torch.int64, device="cuda") * slots * 2 * blk * d * 2
    out = torch.empty(units, G, d, device="cuda")
    wsb = ss.ss_sparse_attention_workspace(units, G, 1, d, blk, k)
    ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device="cuda")
    print(f"[gpu] attention: {units} units, G {G}, blk {blk}, k {k}", flush=True)
    ss.ss_sparse_attention(q, kv, off, sel, cap, slots, units, G, 1, d, blk, k, d ** -0.5, out, ws, wsb)
    worst = 0.0
    for u in range(units):
        s = sel[u][(sel[u] >= 0) & (sel[u] < cap[u])].long()
        if s.numel() == 0:
            assert bool((out[u] == 0).all())
            continue
        K = kv[u, s, 0].reshape(-1, d).double()
        V = kv[u, s, 1].view(-1, d, blk).transpose(1, 2).reshape(-1, d).double()
        p = ((q[u].double() @ K.t().contiguous()) * d ** -0.5).softmax(-1)
        worst = max(worst, float((out[u].double() - p @ V).abs().max()))
    assert worst <= 2.0 ** -15 * float(kv.abs().max()), worst


@pytest.mark.parametrize("units,G,blk,k", [(1, 1, 16, 5), (16, 2, 8, 11), (17, 2, 8, 10), (9, 3, 16, 7), (9, 3, 32, 3),
                                           (300, 16, 8, 1), (4, 7, 8, 15), (8, 1, 16, 9), (9, 1, 16, 9),
                                           (64, 4, 16, 10), (65, 4, 16, 10), (128, 4, 8, 25), (129, 4, 8, 25),
                                           (200, 8, 16, 23), (200, 8, 16, 24), (3, 2, 16, 24), (2, 1, 32, 64),
                                           (383, 1, 32, 48), (384, 1, 16, 95), (384, 1, 16, 96), (512, 1, 16, 96)])
def test_attention_plan_lines(ss, units, G, blk, k):
    """Either side of the lines between one workgroup of 4 and of 8 waves per
    unit (by heads, block size, steps and units) and of the first splits."""
    test_attention_launch_shapes(ss, units, G, blk, k)


@pytest.mark.parametrize("units,k,splits", [(8, 128, 8), (4, 100, 7), (16, 511, 31), (24, 128, 8)])
def test_attention_with_less_workspace(ss, units, k, splits):
    """A workspace smaller than the query's, down to the least one (two 4-wave
    workgroups a CU of 16 steps or more each: `splits`), is served with as many
    splits as it holds: the same output within the 16 bits of a probability,
    nothing written past the end."""
    G, blk, d = 4, 16, 128
    g = torch.Generator(device="cuda").manual_seed(units + k)
    kv = torch.randn(units, k, 2, blk * d, generator=g, device="cuda").bfloat16()
    q = torch.randn(units, G, d, generator=g, device="cuda").bfloat16()
    sel = torch.arange(k, dtype=torch.int32, device="cuda").repeat(units, 1)
    off = torch.arange(units, dtype=torch.int64, device="cuda") * k * 2 * blk * d * 2
    one = units * G * (d + 2) * 4
    full = ss.ss_sparse_attention_workspace(units, G, 1, d, blk, k)
    assert full >= splits * one
    got = []
    for size in (full, (full + splits * one) // 2, splits * one):
        print(f"[gpu] attention: {units} units, k {k}, workspace {size} of {full}", flush=True)
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        out = torch.empty(units, G, d, device="cuda")
        ss.ss_sparse_attention(q, kv, off, sel, None, k, units, G, 1, d, blk, k, d ** -0.5, out, ws, size)
        assert bool((ws[size:] == 0x5A).all())
        got.append(out)
    for out in got[1:]:
        assert float((out - got[0]).abs().max()) <= 2.0 ** -15 * float(kv.abs().max())


@pytest.mark.parametrize("units,k,limit", [(8, 128, 32), (8, 128, 16), (8, 128, 8), (44, 256, 32), (1, 512, 32),
                                           (64, 128, 32), (128, 128, 32)])
def test_attention_merge_keeps_infinities(ss, units, k, limit):
    """A channel whose 32-bit sums overflow is infinite in every split's
    partial, and so is the output: the merge multiplies no partial that it is
    to leave out (0 * inf is no number).  19 splits, 16, 8, 5, 32, 4 and 2 or
    about as many, by kernels that read 4, 8, 16 or 32 partials."""
    G, blk, d = 4, 16, 128
    g = torch.Generator(device="cuda").manual_seed(units + limit)
    kv = torch.randn(units, k, 2, blk * d, generator=g, device="cuda").bfloat16()
    kv[:, :, 1].view(units, k, d, blk)[:, :, 5] = 3e38
    kv[:, :, 1].view(units, k, d, blk)[:, :, 77] = -3e38
    q = torch.zeros(units, G, d, device="cuda").bfloat16()  # every probability alike
    sel = torch.arange(k, dtype=torch.int32, device="cuda").repeat(units, 1)
    off = torch.arange(units, dtype=torch.int64, device="cuda") * k * 2 * blk * d * 2
    size = min(ss.ss_sparse_attention_workspace(units, G, 1, d, blk, k), limit * units * G * (d + 2) * 4)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    out = torch.empty(units, G, d, device="cuda")
    print(f"[gpu] attention with overflowing sums: {units} units, k {k}, at most {limit} splits", flush=True)
    ss.ss_sparse_attention(q, kv, off, sel, None, k, units, G, 1, d, blk, k, d ** -0.5, out, ws, size)
    assert bool((out[:, :, 5] == float("inf")).all()) and bool((out[:, :, 77] == float("-inf")).all())
    rest = torch.ones(d, dtype=torch.bool)
    rest[[5, 77]] = False
    assert bool(out[:, :, rest].isfinite().all())


@pytest.mark.parametrize("kind,agg", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("nblk,G", [((1, 15, 0), 1), ((16, 17, 31), 4), ((33, 48, 32), 7), ((1000, 40, 999), 16),
                                    ((40000, 65, 39985), 2)])
def test_score_tile_edges(ss, kind, agg, nblk, G):
    """Block counts on either side of a tile (16) and of a workgroup (32),
    sequences that end before a workgroup begins, and a launch of more
    workgroups than the chip holds at once (two heads of 40000 blocks).
    Against float64 on the GPU within the summation bound of 256 exact
    products; scores past a sequence's count keep what they held."""
    B, Hkv, n, d = len(nblk), 2, max(nblk), 128
    g = torch.Generator(device="cuda").manual_seed(n * 8 + G)
    lo = torch.randn(B, Hkv, n, d, generator=g, device="cuda").bfloat16()
    meta = lo if kind else torch.stack([lo, (lo.float() + torch.rand(lo.shape, generator=g, device="cuda")).bfloat16()], 3)
    q = torch.randn(B, Hkv * G, d, generator=g, device="cuda").bfloat16()
    nb = torch.tensor(nblk, dtype=torch.int32, device="cuda")
    scores = torch.full((B, Hkv, n), 7.5, device="cuda")
    print(f"[gpu] scores of {nblk} blocks, G {G}, kind {kind}, agg {agg}", flush=True)
    ss.ss_score_blocks_variant(q, meta.contiguous(), kind, agg, nb, B, Hkv * G, Hkv, n, d, scores)
    w = q.double().view(B, Hkv, G, d)
    if kind:
        per, mag = torch.matmul(lo.double(), w.transpose(2, 3).contiguous()), lo.double().abs()
    else:
        m = meta.double()
        per = torch.matmul(m[:, :, :, 0], w.clamp(max=0).transpose(2, 3).contiguous())
        per += torch.matmul(m[:, :, :, 1], w.clamp(min=0).transpose(2, 3).contiguous())
        mag = m.abs().amax(3)
    want = per.sum(-1) if agg else per.amax(-1)
    bound = (2 * d + G) * 2.0 ** -24 * torch.matmul(mag, w.abs().transpose(2, 3).contiguous()).sum(-1)
    for b in range(B):
        k = nblk[b]
        assert bool(((scores[b, :, :k].double() - want[b, :, :k]).abs() <= bound[b, :, :k]).all())
        assert bool((scores[b, :, k:] == 7.5).all())


@pytest.mark.parametrize("kind,agg", [(0, 0), (1, 1)])
@pytest.mark.parametrize("B,n", [(95, 64), (96, 32), (96, 33), (97, 63), (96, 64), (96, 65), (3071, 256), (3072, 65),
                                 (3073, 129), (3072, 256), (3072, 257), (5, 1023), (300, 100), (37, 192), (40, 639),
                                 (9, 1024), (70, 1024), (9, 1025), (9, 2048), (9, 2049)])
def test_score_rows_of_any_length(ss, kind, agg, B, n):
    """Rows of lengths from nothing to all, two heads a sequence, on either
    side of the numbers of rows (192, 6144) and blocks (33 to 64, 256) from
    which one workgroup takes a row, and rows of 4, 6, 20, 32, 33, 64 and 65
    chunks, which are taken in an order that differs from row to row up to 32
    (mean keys: 64)."""
    nblk = torch.randint(0, n + 1, (B,), generator=torch.Generator().manual_seed(B + n)).tolist()
    nblk[0], nblk[1], nblk[-1] = n, 0, n - 1
    test_score_tile_edges(ss, kind, agg, tuple(nblk), 4)


@pytest.mark.parametrize("kind,agg", [(0, 0), (1, 1)])
@pytest.mark.parametrize("B,Hkv,n", [(17, 7, 1000), (29, 7, 50), (13, 5, 700), (9, 3, 224), (11, 12, 1024), (1, 11, 96),
                                     (1000, 7, 70)])
def test_score_batch_matches_single_rows(ss, kind, agg, B, Hkv, n):
    """Heads and chunks a row in numbers that are no powers of two, rows that
    one workgroup takes and chunks in another order, against a call for each
    row by itself, which has none of them: bit for bit."""
    G, d = 3, 128
    g = torch.Generator(device="cuda").manual_seed(B + n)
    meta = torch.randn(B, Hkv, n, 2 - kind, d, generator=g, device="cuda").bfloat16()
    q = torch.randn(B, Hkv, G, d, generator=g, device="cuda").bfloat16()
    nb = torch.randint(0, n + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    got, want = (torch.full((B, Hkv, n), 7.5, device="cuda") for _ in range(2))
    print(f"[gpu] scores of {B} x {Hkv} rows of {n}, kind {kind}", flush=True)
    ss.ss_score_blocks_variant(q, meta, kind, agg, nb, B, Hkv * G, Hkv, n, d, got)
    for b in range(0, B, max(1, B // 30)):
        for h in range(Hkv):
            ss.ss_score_blocks_variant(q[b, h], meta[b, h], kind, agg, nb[b:], 1, G, 1, n, d, want[b, h])
        assert torch.equal(got[b], want[b]), b


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("B,Hkv,G", [(3, 2, 4), (64, 4, 1), (257, 1, 7), (2, 1, 16)])
def test_score_topk_in_one_launch(ss, n, B, Hkv, G):
    """ss_score_topk over rows around the lengths that one launch takes, with
    as many units as CUs and one more, against ss_score_blocks followed by
    ss_select_topk: scores and selections bit for bit, scores past a count
    and everything else untouched.  Repeated metadata rows give exact ties;
    counts of 0, of one block and of all, and more wanted than there are."""
    d = 128
    g = torch.Generator(device="cuda").manual_seed(n * 1000 + B)
    lo = torch.randn(B, Hkv, n, d, generator=g, device="cuda").bfloat16()
    lo[:, :, n // 2:] = lo[:, :, :n - n // 2]
    meta = torch.stack([lo, lo + 1], 3).contiguous()
    q = torch.randn(B, Hkv * G, d, generator=g, device="cuda").bfloat16()
    nb = torch.randint(0, n + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    nb[0], nb[-1] = n, min(n, 1)
    for k in sorted({1, max(n // 3, 1), n + 2}):
        one = torch.full((B, Hkv, n), 7.5, device="cuda"), torch.full((B, Hkv, k), -5, dtype=torch.int32, device="cuda")
        two = one[0].clone(), one[1].clone()
        ss.ss_score_topk(q, meta, nb, B, Hkv * G, Hkv, n, d, k, *one)
        ss.ss_score_blocks(q, meta, nb, B, Hkv * G, Hkv, n, d, two[0])
        ss.ss_select_topk(two[0], nb, B, Hkv, n, k, two[1])
        assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1]), (n, B, Hkv, G, k)
