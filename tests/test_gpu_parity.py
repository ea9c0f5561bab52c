"""GPU parity: every step of the HIP path against the CPU oracle, through the C ABI.

Bars (written out here): decisions and matched indices bit-exact except rows whose
oracle similarity lies within 1e-3 of the threshold (counted); similarities within 1e-5;
hit rows exact copies; computed rows within 1e-4 (fp32) / 2e-2 (bf16) relative, measured
per sequence as max|gpu - oracle| / max|oracle|.
"""
import sys

import numpy as np
import pytest
import torch

import gemm_rule
from oracle import llmc_oracle as O
from paper_2512_16843_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    from paper_2512_16843_amd import llmc
    assert torch.cuda.is_available(), "these tests need the GPU"
    llmc.lib()
    return llmc


def npf(t):
    return t.detach().float().cpu().numpy()


def f32(x):
    return float(np.float32(x))


def rel_err_rows(got, want):
    got = np.asarray(got, dtype=np.float64).reshape(got.shape[0], -1)
    want = np.asarray(want, dtype=np.float64).reshape(want.shape[0], -1)
    return np.abs(got - want).max(axis=1) / np.maximum(np.abs(want).max(axis=1), 1e-30)


def oracle_bank_from_gpu(bank, dtype):
    ob = O.Bank(bank.n_slots, bank.k, bank.S, bank.d, dtype, n_act_slots=bank.n_act_slots)
    ob.fp = npf(bank.fp)
    ob.inv_norm = npf(bank.inv_norm)
    ob.act = npf(bank.act)
    if bank.act_slot is not None:
        ob.act_slot = bank.act_slot.cpu().numpy()
    ob.last_used = bank.last_used.cpu().numpy().astype(np.uint64)
    ob.hits = bank.hits.cpu().numpy().astype(np.uint32)
    ob.valid = bank.valid.cpu().numpy()
    return ob


# ---------------------------------------------------------------------------
# step 1: fingerprint
# ---------------------------------------------------------------------------

def run_fingerprint(L, h, P, bias):
    B, S, d = h.shape
    k = P.shape[1]
    fp = torch.empty((B, k), dtype=h.dtype, device="cuda")
    inv = torch.empty((B,), dtype=torch.float32, device="cuda")
    ws = torch.empty((L.llmc_fingerprint_workspace_bytes(B, S, d),), dtype=torch.uint8, device="cuda")
    L.llmc_fingerprint(h, P, bias, fp, inv, ws)
    torch.cuda.synchronize()
    return fp, inv


@pytest.mark.parametrize("dtype,B,S,d,k,use_bias", [
    ("f32", 8, 32, 128, 64, False),      # tiny-encoder shape
    ("f32", 3, 1, 64, 32, True),         # S = 1
    ("bf16", 5, 33, 768, 256, True),     # ragged token chunk
    ("bf16", 7, 384, 768, 256, False),   # BERT-base row shape, several chunks
    ("bf16", 4, 1024, 768, 256, False),  # GPT-2 row shape
    ("bf16", 9, 128, 1024, 256, False),  # BERT-large row shape
])
def test_fingerprint_matches_oracle(L, dtype, B, S, d, k, use_bias):
    say(f"fingerprint {dtype} B={B} S={S} d={d} k={k} bias={use_bias}")
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = np.random.Generator(np.random.PCG64(B * 1000 + S))
    h = torch.from_numpy(g.standard_normal((B, S, d)).astype(np.float32) + 0.3).to(tdt).cuda()
    P = W.make_projection(d, k, tdt, seed=3)[0].cuda()
    bias = torch.from_numpy(g.standard_normal(k).astype(np.float32) * 0.1).cuda() if use_bias else None
    fp, inv = run_fingerprint(L, h, P, bias)
    q, qinv = O.fingerprint(npf(h), npf(P), None if bias is None else npf(bias), dtype)
    got = npf(fp)
    if dtype == "f32":
        np.testing.assert_allclose(got, q, rtol=0, atol=2e-6)
    else:
        # the key is a quantised code decided after an fp32 (device) / fp64 (oracle) sum: codes agree
        # except where the value sits on a rounding boundary, and then they differ by one bf16 step
        diff = got != q
        assert diff.mean() < 5e-3, diff.mean()
        step = np.maximum(np.abs(q), 2.0 ** -126) * 2.0 ** -7
        assert np.all(np.abs(got - q)[diff] <= step[diff])
    # the stored inverse norm is that of the key the device actually stored
    np.testing.assert_allclose(npf(inv), O.inv_norm(got), rtol=3e-7, atol=0)
    np.testing.assert_allclose(npf(inv), qinv, rtol=1e-4)


@pytest.mark.parametrize("name,base,kw,n_prefix", [
    ("f32 encoder", "TINY_ENCODER", dict(B=5, S=32), 8),
    ("f32 decoder", "TINY_ENCODER", dict(B=4, S=40, arch=1, gelu=1, ln_eps=1e-5), 13),       # ragged prefix, causal, LN1 first
    ("f32 whole sequence", "TINY_ENCODER", dict(B=3, S=32), 32),
    ("bf16 bert-base rows", "BERT_BASE", dict(B=6, n_layers=1), 32),
    ("bf16 gpt2 rows", "GPT2_SMALL", dict(B=3, n_layers=1), 100),                             # not a multiple of the key tile
])
def test_fingerprint_with_prefix_attention_statistics_matches_oracle(L, name, base, kw, n_prefix):
    """llmc_fingerprint_prefix (token average + mean of the block's self-attention outputs over the first tokens,
    one linear map) against the oracle.  The map of the attention feature is scaled so that both features carry
    comparable weight in the key.  fp32: 1e-5 absolute on the unit-norm key.  bf16: the attention feature passes
    through three bf16 products (QKV, softmax-weighted values, output projection), each rounded to 2^-9 relative, so
    it arrives with about 1e-2 relative error and, carrying about half of the key's length, moves the key's direction by
    at most about 1e-2: cosine with the oracle's key above 1 - 1e-4, components within 1.5e-3."""
    say(f"fingerprint with prefix attention statistics: {name}, first {n_prefix} tokens")
    cfg = W.scaled(getattr(W, base), n_layers=1, **{k_: v for k_, v in kw.items() if k_ != "n_layers"})
    dtype = cfg.dtype
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    ids = W.make_sources(cfg, cfg.B, seed=1)
    h = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    wnp = {k_: npf(v) for k_, v in ws[0].items()}
    g = np.random.Generator(np.random.PCG64(41))
    a_ref = O.prefix_attention_mean(npf(h), wnp, cfg.arch, cfg.n_heads, cfg.ln_eps, n_prefix)
    p_ref = npf(h).astype(np.float64).mean(axis=1)
    ratio = float(np.linalg.norm(p_ref) / max(np.linalg.norm(a_ref), 1e-30))
    P2 = np.concatenate([g.standard_normal((cfg.d, cfg.k)), ratio * g.standard_normal((cfg.d, cfg.k))]) / np.sqrt(cfg.k)
    P2t = torch.from_numpy(P2.astype(np.float32)).to(cfg.torch_dtype).cuda()
    bias = torch.from_numpy((g.standard_normal(cfg.k) * 0.01 * np.linalg.norm(p_ref[0])).astype(np.float32)).cuda()
    layer = L.layer_from_weights(cfg, ws[0])
    fp = torch.empty((cfg.B, cfg.k), dtype=cfg.torch_dtype, device="cuda")
    inv = torch.empty((cfg.B,), dtype=torch.float32, device="cuda")
    wsb = torch.empty((L.llmc_fingerprint_prefix_workspace_bytes(layer.desc(), cfg.B, cfg.S, n_prefix),), dtype=torch.uint8,
                      device="cuda")
    L.llmc_fingerprint_prefix(layer.desc(), h, n_prefix, P2t, bias, fp, inv, wsb)
    torch.cuda.synchronize()
    q, qinv = O.fingerprint_prefix(npf(h), npf(P2t), npf(bias), dtype, wnp, cfg.arch, cfg.n_heads, cfg.ln_eps, n_prefix)
    got = npf(fp)
    # the attention feature carries weight: without it the key would be far from the one computed
    q_plain, _ = O.fingerprint(npf(h), npf(P2t)[:cfg.d], npf(bias), dtype)
    assert np.abs(q_plain - q).max() > 2e-2
    err = np.abs(got - q).max()
    cos = (got.astype(np.float64) * q).sum(axis=1) / np.linalg.norm(got.astype(np.float64), axis=1) / np.linalg.norm(q, axis=1)
    say(f"  max |key - oracle| {err:.2e}, min cosine {cos.min():.7f}")
    if dtype == "f32":
        assert err < 1e-5
    else:
        assert err < 1.5e-3 and cos.min() > 1 - 1e-4
    np.testing.assert_allclose(npf(inv), O.inv_norm(got), rtol=3e-7, atol=0)
    # the call is a function of each sequence alone
    if cfg.B >= 3:
        fp1 = torch.empty((1, cfg.k), dtype=cfg.torch_dtype, device="cuda")
        inv1 = torch.empty((1,), dtype=torch.float32, device="cuda")
        L.llmc_fingerprint_prefix(layer.desc(), h[2:3].contiguous(), n_prefix, P2t, bias, fp1, inv1, wsb)
        torch.cuda.synchronize()
        assert torch.equal(fp1[0], fp[2]) and torch.equal(inv1[0], inv[2])


def test_fingerprint_is_position_and_batch_independent(L):
    say("fingerprint determinism across batch position and size")
    g = np.random.Generator(np.random.PCG64(77))
    h = torch.from_numpy(g.standard_normal((12, 384, 768)).astype(np.float32)).to(torch.bfloat16).cuda()
    P = W.make_projection(768, 256, torch.bfloat16, seed=3)[0].cuda()
    fp_a, inv_a = run_fingerprint(L, h, P, None)
    perm = torch.from_numpy(g.permutation(12)).cuda()
    fp_b, inv_b = run_fingerprint(L, h[perm].contiguous(), P, None)
    assert torch.equal(fp_a[perm], fp_b) and torch.equal(inv_a[perm], inv_b)
    fp_c, inv_c = run_fingerprint(L, h[3:4].contiguous(), P, None)
    assert torch.equal(fp_c[0], fp_a[3]) and torch.equal(inv_c[0], inv_a[3])


@pytest.mark.parametrize("k", [32, 96, 288, 992])
def test_fingerprint_key_lengths_that_do_not_fill_wavefronts(L, k):
    """Norms are sums over wavefronts.  32 and 96 columns end inside one (their 128 and 384 threads of work do not); 288 and
    992 columns give 1008 and 992 threads of work, which threads without any fill up to whole wavefronts."""
    say(f"fingerprint f32 k={k}")
    g = np.random.Generator(np.random.PCG64(k))
    h = torch.from_numpy(g.standard_normal((3, 70, 192)).astype(np.float32)).cuda()
    P = W.make_projection(192, k, torch.float32, seed=3)[0].cuda()
    fp, inv = run_fingerprint(L, h, P, None)
    q, _ = O.fingerprint(npf(h), npf(P), None, "f32")
    assert np.abs(npf(fp) - q).max() < 1e-5            # unit keys from sums of 192 products
    np.testing.assert_allclose(npf(inv), O.inv_norm(npf(fp)), rtol=3e-7, atol=0)


def test_fingerprint_zero_input(L):
    say("fingerprint of an all-zero sequence")
    h = torch.zeros((2, 5, 128), dtype=torch.float32, device="cuda")
    P = W.make_projection(128, 64, torch.float32, seed=3)[0].cuda()
    fp, inv = run_fingerprint(L, h, P, None)
    assert torch.all(fp == 0) and torch.all(inv == 0)


def test_inv_norm(L):
    say("inv_norm")
    g = np.random.Generator(np.random.PCG64(5))
    x = torch.from_numpy(g.standard_normal((1001, 256)).astype(np.float32)).to(torch.bfloat16).cuda()
    x[17] = 0
    out = torch.empty((1001,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(x, out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(npf(out), O.inv_norm(npf(x)))


# ---------------------------------------------------------------------------
# steps 2-3: match + threshold
# ---------------------------------------------------------------------------

def make_bank(L, keys, valid=None, S=1, d=64, dtype=torch.bfloat16, policy=None, act=None, act_slot=None, A=None):
    N, k = keys.shape
    bank = L.Bank(N, k, S, d, dtype, "cuda", n_act_slots=A, policy=L.EVICT_LRU if policy is None else policy,
                  act_slot=act_slot)
    bank.fp.copy_(keys)
    L.llmc_inv_norm(bank.fp, bank.inv_norm)
    bank.valid.copy_(torch.ones(N, dtype=torch.uint8) if valid is None else valid)
    if act is not None:
        bank.act.copy_(act)
    bank.refresh()
    torch.cuda.synchronize()
    return bank


def run_match(L, bank, q, qinv, tau):
    B = q.shape[0]
    idx = torch.empty((B,), dtype=torch.int32, device="cuda")
    sim = torch.empty((B,), dtype=torch.float32, device="cuda")
    hit = torch.empty((B,), dtype=torch.uint8, device="cuda")
    tie = torch.empty((B,), dtype=torch.uint8, device="cuda")
    ws = torch.empty((L.llmc_match_workspace_bytes(bank, B),), dtype=torch.uint8, device="cuda")
    L.llmc_match(bank, q, qinv, tau, idx, sim, hit, tie, ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), npf(sim), hit.cpu().numpy().astype(bool), tie.cpu().numpy()


def check_match(L, bank, q, tau, dtype):
    qinv = torch.empty((q.shape[0],), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(q, qinv)
    idx, sim, hit, tie = run_match(L, bank, q, qinv, tau)
    ob = oracle_bank_from_gpu(bank, dtype)
    oidx, osim = O.match(npf(q), npf(qinv), ob.fp, ob.inv_norm, ob.valid)
    ohit = O.threshold(osim, f32(tau))
    near_tau = np.abs(osim - f32(tau)) < 1e-3
    assert np.array_equal(idx, oidx), (np.nonzero(idx != oidx)[0][:10], idx[idx != oidx][:10], oidx[idx != oidx][:10])
    fin = np.isfinite(osim)
    np.testing.assert_allclose(sim[fin], osim[fin], rtol=0, atol=1e-5)
    assert np.all(np.isneginf(sim[~fin]))
    assert np.array_equal(hit[~near_tau], ohit[~near_tau])
    return dict(idx=idx, sim=sim, hit=hit, tie=tie, near_tau=int(near_tau.sum()), oracle_sim=osim)


def unit_rows(g, n, k):
    x = g.standard_normal((n, k))
    return x / np.linalg.norm(x, axis=1, keepdims=True)


@pytest.mark.parametrize("N,B,k", [(1000, 37, 64), (130, 5, 256), (4096, 200, 256), (64, 1, 32),
                                   # more than 256 queries: the skewed 8-wavefront kernel, ragged banks, one-tile splits
                                   (1000, 300, 64), (5000, 513, 128), (130, 260, 256), (70000, 700, 256)])
def test_match_bf16_random_bank_with_holes(L, N, B, k):
    say(f"match bf16 random N={N} B={B} k={k}")
    g = np.random.Generator(np.random.PCG64(N + B))
    keys = torch.from_numpy(unit_rows(g, N, k).astype(np.float32)).to(torch.bfloat16).cuda()
    valid = torch.from_numpy((g.random(N) > 0.15).astype(np.uint8))
    bank = make_bank(L, keys, valid)
    qn = unit_rows(g, B, k)
    # a third of the queries are noisy copies of bank keys (some of them of FREE slots)
    for b in range(0, B, 3):
        j = int(g.integers(0, N))
        qn[b] = npf(keys[j]) + 0.05 * g.standard_normal(k) / np.sqrt(k)
    q = torch.from_numpy(qn.astype(np.float32)).to(torch.bfloat16).cuda()
    r = check_match(L, bank, q, 0.9, "bf16")
    assert np.all(valid.numpy()[r["idx"]] == 1)
    bank.close()


@pytest.mark.parametrize("dtype,N,B,k", [("bf16", 5000, 40, 64), ("bf16", 5000, 300, 256), ("bf16", 3000, 9, 96),
                                          ("f32", 2000, 7, 64)])
def test_match_many_near_identical_keys_in_different_blocks(L, dtype, N, B, k):
    """Five keys that differ from one another by a few units in the last place of a few elements (cosines within
    about 1e-6 of each other: beyond what the fp32 bulk pass can order), spread over different 32-row blocks of the
    bank, plus exact duplicates.  Two kept candidate groups cannot always decide such a query: the row must be
    FLAGGED (near-tie flag 2), its slot must be one the oracle sees within 2e-5 of its maximum, and its similarity
    within 2e-5 of the oracle's; every other row is exact."""
    say(f"match {dtype} N={N} B={B} k={k}: five near-identical keys in different blocks")
    g = np.random.Generator(np.random.PCG64(N + k))
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    keys = torch.from_numpy(unit_rows(g, N, k).astype(np.float32)).to(tdt)
    base = keys[11].clone()
    spots = [7, 100, 1033, 2 * N // 3, N - 3]
    step = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -8         # cosines between variants differ by about 1e-6
    variants = []
    for v, j in enumerate(spots):
        x = base.float().clone()
        for e in range(3):
            i = (5 * v + 11 * e) % k
            x[i] = x[i] * (1.0 + step * (1 + (v + e) % 2))
        keys[j] = x.to(tdt)
        variants.append(keys[j].clone())
    keys[300] = keys[1033]                                    # exact duplicates
    keys[1032] = keys[spots[3]]
    valid = torch.ones(N, dtype=torch.uint8)
    valid[100] = 0                                            # one of the five is a free slot
    bank = make_bank(L, keys.cuda(), valid, dtype=tdt)
    qn = unit_rows(g, B, k).astype(np.float32)
    q = torch.from_numpy(qn).to(tdt)
    for b, v in enumerate([0, 2, 3, 4, 1]):                   # the first five queries are the variants themselves
        q[b] = variants[v]
    q = q.cuda()
    qinv = torch.empty((B,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(q, qinv)
    idx, sim, hit, tie = run_match(L, bank, q, qinv, 0.9)
    ob = oracle_bank_from_gpu(bank, dtype)
    oidx, osim = O.match(npf(q), npf(qinv), ob.fp, ob.inv_norm, ob.valid)
    wide = O.near_tie_sets(npf(q), npf(qinv), ob.fp, ob.inv_norm, ob.valid, gap=2e-5)
    assert np.all(tie[:5] == 2), tie[:8]
    assert np.all(tie[5:] < 2)
    for b in range(B):
        if tie[b] == 2:
            assert idx[b] in wide[b] and abs(sim[b] - osim[b]) < 2e-5
            assert len(wide[b]) >= 5
        else:
            assert idx[b] == oidx[b] and abs(sim[b] - osim[b]) < 1e-5
    assert np.all(hit[:5])
    bank.close()


def test_match_duplicates_self_and_negative_best(L):
    say("match bf16 duplicates across tiles / self hit / all-negative similarities")
    g = np.random.Generator(np.random.PCG64(3))
    N, k = 700, 128
    kn = unit_rows(g, N, k).astype(np.float32)
    keys = torch.from_numpy(kn).to(torch.bfloat16)
    keys[650] = keys[20]
    keys[333] = keys[20]
    keys[334] = keys[200]
    bank = make_bank(L, keys.cuda())
    q = torch.stack([keys[650], keys[334], keys[5], -keys[7]]).cuda()
    r = check_match(L, bank, q, 0.95, "bf16")
    assert r["idx"].tolist()[:3] == [20, 200, 5]
    np.testing.assert_allclose(r["sim"][:3], 1.0, atol=1e-6)
    assert r["hit"].tolist()[:3] == [True, True, True] and r["tie"][0] and r["tie"][1]
    # with only one key left valid, the best similarity of -key is negative, and it is still reported
    v = torch.zeros(N, dtype=torch.uint8)
    v[7] = 1
    bank.valid.copy_(v)
    bank.refresh()
    r = check_match(L, bank, q[3:4].contiguous(), 0.0, "bf16")
    assert r["idx"][0] == 7 and r["sim"][0] < -0.99 and not r["hit"][0]
    bank.close()


def test_match_empty_bank_and_zero_query(L):
    say("match: empty bank, zero query")
    g = np.random.Generator(np.random.PCG64(4))
    keys = torch.from_numpy(unit_rows(g, 256, 64).astype(np.float32)).to(torch.bfloat16).cuda()
    bank = make_bank(L, keys, torch.zeros(256, dtype=torch.uint8))
    q = keys[:3].contiguous()
    r = check_match(L, bank, q, -2.0, "bf16")
    assert np.all(r["idx"] == -1) and not r["hit"].any()
    v = torch.ones(256, dtype=torch.uint8)
    v[:9] = 0
    bank.valid.copy_(v)
    bank.refresh()
    z = torch.zeros((1, 64), dtype=torch.bfloat16, device="cuda")
    r = check_match(L, bank, z, 0.0, "bf16")
    assert r["idx"][0] == 9 and r["sim"][0] == 0 and not r["hit"][0]      # first valid slot, similarity 0, 0 > 0 false
    bank.close()


def test_match_f32(L):
    say("match f32 N=256 k=64 (tiny-encoder bank shape)")
    g = np.random.Generator(np.random.PCG64(6))
    keys = torch.from_numpy(unit_rows(g, 256, 64).astype(np.float32)).cuda()
    valid = torch.from_numpy((g.random(256) > 0.1).astype(np.uint8))
    bank = make_bank(L, keys, valid, dtype=torch.float32)
    qn = unit_rows(g, 8, 64)
    qn[0] = npf(keys[100]) + 0.01 * g.standard_normal(64)
    qn[1] = npf(keys[3])
    q = torch.from_numpy(qn.astype(np.float32)).cuda()
    r = check_match(L, bank, q, 0.95, "f32")
    bank.close()


@pytest.mark.parametrize("N,B,k", [(1, 1, 32), (31, 3, 64), (129, 16, 96), (1000, 17, 256), (4097, 70, 128),
                                   (300, 65, 1024)])
def test_match_f32_edges(L, N, B, k):
    """Sizes around the 32-row fragments, the 128-row blocks and the two query blockings (16 and 64)."""
    say("match f32 N=%d B=%d k=%d with holes" % (N, B, k))
    g = np.random.Generator(np.random.PCG64(1000 + N))
    keys = torch.from_numpy(unit_rows(g, N, k).astype(np.float32)).cuda()
    valid = g.random(N) > 0.2
    valid[N // 2] = True
    bank = make_bank(L, keys, torch.from_numpy(valid.astype(np.uint8)), dtype=torch.float32)
    qn = unit_rows(g, B, k)
    near = np.nonzero(valid)[0][-min(B, int(valid.sum())):]
    qn[:len(near)] = npf(keys)[near] + 0.01 * g.standard_normal((len(near), k))
    check_match(L, bank, torch.from_numpy(qn.astype(np.float32)).cuda(), 0.9, "f32")
    bank.close()


@pytest.mark.parametrize("N,B,k,splits", [
    (16500, 2048, 64, 43),   # 129 blocks of 128 rows, three to a workgroup; the last block has 116 rows
    (16300, 130, 32, 7),     # 128 blocks, 19 to a workgroup and 14 in the last split, which the workspace allows
])
def test_match_f32_several_blocks_per_workgroup(L, N, B, k, splits):
    """A workgroup that walks several bank blocks: the running best of a query over ascending groups, equal keys in
    different blocks of one split, more near-identical keys than the two groups that are decided exactly, a short last
    split."""
    say(f"match f32 N={N} B={B} k={k} in {splits} splits")
    g = np.random.Generator(np.random.PCG64(N + B))
    kn = unit_rows(g, N, k).astype(np.float32)
    per = -(-((N + 127) // 128) // splits) * 128             # rows of a split
    assert per >= 256 and N % per > 128                       # several blocks, also in the last split
    valid = g.random(N) > 0.2
    base = (0, per, N - N % per)                              # first, second and last split
    for i, b0 in enumerate(base):
        # the same key in the split's first and second block; in the second split twice in its second block
        kn[b0 + 150] = kn[b0 + 7]
        valid[[b0 + 7, b0 + 150]] = (i != 1, True)
        if i == 1:
            kn[b0 + 200] = kn[b0 + 7]
            valid[b0 + 200] = True
    for j in (40, 100, 170, 230):                             # a step of fp32 in a few elements: cosines within 1e-6
        kn[j] = kn[1]
        kn[j, j % k] = np.nextafter(kn[j, j % k], np.float32(9.0), dtype=np.float32)
    valid[[1, 40, 100, 170, 230]] = True
    keys = torch.from_numpy(kn).cuda()
    bank = make_bank(L, keys, torch.from_numpy(valid.astype(np.uint8)), dtype=torch.float32)
    qn = unit_rows(g, B, k).astype(np.float32)
    near = np.concatenate([[b0 + 7 for b0 in base], np.nonzero(valid)[0][-60:]])
    qn[:len(near)] = kn[near]
    qn[3:len(near)] += (0.01 * g.standard_normal((len(near) - 3, k))).astype(np.float32)
    qn[B - 1] = kn[1]
    q = torch.from_numpy(qn).cuda()
    qinv = torch.empty((B,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(q, qinv)
    res = []
    # 20 bytes per query and split; and the size that is asked for, which leaves the number of splits to the library
    for size in (20 * B * splits, L.llmc_match_workspace_bytes(bank, B)):
        ws = torch.empty((size,), dtype=torch.uint8, device="cuda")
        idx = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        sim = torch.empty((B,), dtype=torch.float32, device="cuda")
        hit = torch.empty((B,), dtype=torch.uint8, device="cuda")
        tie = torch.empty((B,), dtype=torch.uint8, device="cuda")
        L.llmc_match(bank, q, qinv, 0.9, idx, sim, hit, tie, ws)
        torch.cuda.synchronize()
        res.append([npf(x) for x in (idx, sim, hit, tie)])
    ob = oracle_bank_from_gpu(bank, "f32")
    oidx, osim = O.match(npf(q), npf(qinv), ob.fp, ob.inv_norm, ob.valid)
    for idx, sim, hit, tie in res:
        assert np.all(tie[:B - 1] < 2) and tie[B - 1] == 2    # only the last query has more than two groups in reach
        assert np.array_equal(idx[:B - 1], oidx[:B - 1])
        assert idx[:3].tolist() == [7, per + 150, N - N % per + 7]
        assert np.all(tie[:3] == 1)                           # the runner-up lies in another group of the same split
        assert int(idx[B - 1]) in (1, 40, 100, 170, 230)
        assert np.abs(sim - osim).max() < 1e-5
        assert np.array_equal(hit != 0, osim > 0.9)
    for a, b in zip(*res):                                    # how the bank is split changes nothing
        assert np.array_equal(a, b)
    bank.close()


@pytest.mark.parametrize("live", [(7,), (7, 300)])
def test_match_f32_best_score_that_overflows(L, live):
    """Keys and queries of 1e25: every product of a query and a live key overflows to -inf in the bulk pass, and the best
    of these entries is still the answer."""
    say(f"match f32, scores that overflow to -inf, live slots {live}")
    g = np.random.Generator(np.random.PCG64(8))
    N, k = 320, 64
    keys = torch.from_numpy((1e25 * np.abs(unit_rows(g, N, k))).astype(np.float32)).cuda()
    valid = torch.zeros(N, dtype=torch.uint8)
    valid[list(live)] = 1
    bank = make_bank(L, keys, valid, dtype=torch.float32)
    r = check_match(L, bank, -keys[[7, 300, 11]], 0.9, "f32")
    assert set(r["idx"].tolist()) <= set(live) and not r["hit"].any()
    bank.close()


def test_match_f32_workspace_of_a_larger_batch_serves_smaller_ones(L):
    """The size reported for fp32 keys rises with the batch, and a workspace of one candidate record (20 bytes) per query
    is enough: fewer splits of the bank, the same results.  One byte less is refused."""
    N, k = 131072, 32
    say(f"match f32 workspaces N={N} k={k}: sized for 129 queries, used for 128")
    g = np.random.Generator(np.random.PCG64(77))
    keys = torch.from_numpy(unit_rows(g, N, k).astype(np.float32)).cuda()
    bank = make_bank(L, keys, dtype=torch.float32)
    sizes = [L.llmc_match_workspace_bytes(bank, B) for B in (1, 16, 17, 64, 65, 128, 129, 256, 257, 4096, 262144, 300000)]
    assert sizes == sorted(sizes)
    B = 128
    q = torch.from_numpy((npf(keys[:B]) + 0.1 * unit_rows(g, B, k)).astype(np.float32)).cuda()
    qinv = torch.empty((B,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(q, qinv)
    least = (20 * B + 255) // 256 * 256
    res = []
    for size in (L.llmc_match_workspace_bytes(bank, B), L.llmc_match_workspace_bytes(bank, B + 1), least):
        ws = torch.empty((size,), dtype=torch.uint8, device="cuda")
        idx = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        sim = torch.empty((B,), dtype=torch.float32, device="cuda")
        L.llmc_match(bank, q, qinv, 0.9, idx, sim, None, None, ws)
        torch.cuda.synchronize()
        res.append((idx, sim))
    assert res[0][0].tolist() == list(range(B))
    for idx, sim in res[1:]:
        assert torch.equal(idx, res[0][0]) and torch.equal(sim, res[0][1])
    with pytest.raises(L.LlmcError) as e:
        L.llmc_match(bank, q, qinv, 0.9, idx, sim, None, None, torch.empty((least - 1,), dtype=torch.uint8, device="cuda"))
    assert e.value.status == L.ERR_WORKSPACE
    bank.close()


def test_match_clustered_bank_scaled_stress(L):
    say("match bf16 clustered bank 128 clusters x 256, 1024 queries (scaled copy of the stress config)")
    data = W.make_clustered_bank(128, 256, 256, 0.05, 1024, seed=5)
    bank = make_bank(L, data["bank"].cuda())
    q = data["queries"].cuda()
    r = check_match(L, bank, q, 0.95, "bf16")
    inside = data["q_cluster"].numpy() >= 0
    cl = data["cluster"].numpy()
    assert np.array_equal(cl[r["idx"][inside]], data["q_cluster"].numpy()[inside])
    assert r["hit"][inside].mean() > 0.99 and r["hit"][~inside].mean() < 0.01
    say(f"  hit rate {r['hit'].mean():.3f}, near-tie rows {int(r['tie'].sum())}, near-tau rows {r['near_tau']}")
    bank.close()


# ---------------------------------------------------------------------------
# sign-bit keys and their Hamming match (integer work: bit-exact)
# ---------------------------------------------------------------------------

def words(t):
    """int32 device tensor of key words -> uint32 numpy"""
    return t.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("dtype,B,S,d,k,use_bias", [
    ("f32", 8, 32, 128, 64, False), ("bf16", 5, 37, 768, 256, False), ("bf16", 3, 128, 1024, 512, True),
    ("f32", 2, 9, 64, 96, True), ("bf16", 70, 16, 192, 32, False),
])
def test_fingerprint_bits_match_oracle_signs(L, dtype, B, S, d, k, use_bias):
    say(f"sign-bit fingerprint {dtype} B={B} S={S} d={d} k={k} bias={use_bias}")
    g = np.random.Generator(np.random.PCG64(B * 1000 + k))
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    h = torch.from_numpy(g.standard_normal((B, S, d)).astype(np.float32)).to(tdt).cuda()
    P = torch.from_numpy((g.standard_normal((d, k)) / np.sqrt(k)).astype(np.float32)).to(tdt).cuda()
    bias = torch.from_numpy(0.05 * g.standard_normal(k).astype(np.float32)).cuda() if use_bias else None
    bits = torch.empty((B, k // 32), dtype=torch.int32, device="cuda")
    ws = torch.empty((L.llmc_fingerprint_workspace_bytes(B, S, d),), dtype=torch.uint8, device="cuda")
    L.llmc_fingerprint_bits(h, P, bias, bits, ws)
    torch.cuda.synchronize()
    v = O.simhash_projection(npf(h), npf(P), None if bias is None else npf(bias))
    want = v >= 0
    got = O.unpack_bits(words(bits), k)
    # the sign is decided in the kernel's fp32 arithmetic: projections within 1e-5 of the vector's scale of zero may differ
    scale = np.sqrt((v * v).mean(axis=1, keepdims=True))
    near_zero = np.abs(v) < 1e-5 * scale
    assert np.array_equal(got[~near_zero], want[~near_zero])
    say(f"  {int(near_zero.sum())} of {v.size} projections near zero, {int((got != want).sum())} signs differ there")
    # the same input gives the same key wherever it sits
    bits2 = torch.empty((1, k // 32), dtype=torch.int32, device="cuda")
    L.llmc_fingerprint_bits(h[B - 1:B].contiguous(), P, bias, bits2, ws)
    torch.cuda.synchronize()
    assert torch.equal(bits2[0], bits[B - 1])


def run_match_bits(L, bank_bits, valid, q_bits, max_h):
    N, W = bank_bits.shape
    B = q_bits.shape[0]
    idx = torch.empty((B,), dtype=torch.int32, device="cuda")
    dist = torch.empty((B,), dtype=torch.int32, device="cuda")
    hit = torch.empty((B,), dtype=torch.uint8, device="cuda")
    ws = torch.empty((L.llmc_match_bits_workspace_bytes(N, W * 32, B),), dtype=torch.uint8, device="cuda")
    L.llmc_match_bits(bank_bits, valid, q_bits, max_h, idx, dist, hit, ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), dist.cpu().numpy(), hit.cpu().numpy().astype(bool)


@pytest.mark.parametrize("N,B,k", [(1000, 37, 64), (130, 5, 256), (4099, 300, 256), (64, 1, 32), (777, 260, 128),
                                   (50000, 513, 512), (333, 9, 96), (2500, 40, 1024),
                                   # many queries of 256-bit keys: the scan runs on the matrix cores
                                   (4099, 600, 256), (4096, 512, 256), (70001, 1030, 256), (9000, 513, 256)])
def test_match_bits_is_exact(L, N, B, k):
    say(f"Hamming match N={N} B={B} k={k}")
    g = np.random.Generator(np.random.PCG64(N * 7 + B))
    W_ = k // 32
    bank = g.integers(0, 2 ** 32, size=(N, W_), dtype=np.uint64).astype(np.uint32)
    q = g.integers(0, 2 ** 32, size=(B, W_), dtype=np.uint64).astype(np.uint32)
    valid = (g.random(N) > 0.15).astype(np.uint8)
    # a third of the queries are bank keys with a few bits flipped (some of FREE slots), some exact duplicates in the bank
    for b in range(0, B, 3):
        j = int(g.integers(0, N))
        q[b] = bank[j]
        for _ in range(int(g.integers(0, 6))):
            i = int(g.integers(0, k))
            q[b, i // 32] ^= np.uint32(1 << (i % 32))
    if N > 40:
        bank[N - 1] = bank[3]
        bank[N // 2] = bank[3]
        q[B - 1] = bank[3]
        valid[[3, N // 2, N - 1]] = 1
    max_h = O.max_hamming(f32(0.95), k)
    idx, dist, hit = run_match_bits(L, torch.from_numpy(bank.view(np.int32)).cuda(), torch.from_numpy(valid).cuda(),
                                    torch.from_numpy(q.view(np.int32)).cuda(), max_h)
    oidx, odist = O.match_bits(q, bank, valid, k)
    assert np.array_equal(idx, oidx), (np.nonzero(idx != oidx)[0][:8], idx[idx != oidx][:8], oidx[idx != oidx][:8])
    assert np.array_equal(dist, odist)
    assert np.array_equal(hit, O.threshold_bits(oidx, odist, max_h))
    if N > 40:
        assert idx[B - 1] == 3 and dist[B - 1] == 0 and hit[B - 1]
    say(f"  {int(hit.sum())} hits within {max_h} bits")


@pytest.mark.parametrize("n_distinct", [1, 5, 64])
def test_match_bits_with_many_queries_breaks_ties_to_the_lowest_slot(L, n_distinct):
    say(f"Hamming match on the matrix cores: a bank of {n_distinct} distinct keys repeated through every tile, free slots between")
    g = np.random.Generator(np.random.PCG64(900 + n_distinct))
    N, B, k = 6000, 700, 256
    distinct = g.integers(0, 2 ** 32, size=(n_distinct, 8), dtype=np.uint64).astype(np.uint32)
    if n_distinct > 1:
        distinct[1] = 0                       # the all-zero key: no common set bit with anything
        distinct[2] = 0xFFFFFFFF              # and the all-ones key
    bank = distinct[g.integers(0, n_distinct, size=N)]
    valid = (g.random(N) > 0.4).astype(np.uint8)
    q = distinct[g.integers(0, n_distinct, size=B)].copy()
    for b in range(0, B, 2):                  # half of the queries a few bits away: equal distances to every copy
        for _ in range(int(g.integers(1, 9))):
            i = int(g.integers(0, k))
            q[b, i // 32] ^= np.uint32(1 << (i % 32))
    q[B - 1] = 0
    q[B - 2] = 0xFFFFFFFF
    max_h = O.max_hamming(f32(0.95), k)
    idx, dist, hit = run_match_bits(L, torch.from_numpy(bank.view(np.int32)).cuda(), torch.from_numpy(valid).cuda(),
                                    torch.from_numpy(q.view(np.int32)).cuda(), max_h)
    oidx, odist = O.match_bits(q, bank, valid, k)
    assert np.array_equal(idx, oidx), (np.nonzero(idx != oidx)[0][:8], idx[idx != oidx][:8], oidx[idx != oidx][:8])
    assert np.array_equal(dist, odist)
    assert np.array_equal(hit, O.threshold_bits(oidx, odist, max_h))
    # nothing valid at all: every query reports no neighbour, also from this scan
    idx, dist, hit = run_match_bits(L, torch.from_numpy(bank.view(np.int32)).cuda(),
                                    torch.zeros(N, dtype=torch.uint8).cuda(), torch.from_numpy(q.view(np.int32)).cuda(), k)
    assert np.all(idx == -1) and np.all(dist == O.NO_MATCH_DIST) and not hit.any()
    # one valid slot, the last one
    v = np.zeros(N, np.uint8)
    v[N - 1] = 1
    idx, dist, hit = run_match_bits(L, torch.from_numpy(bank.view(np.int32)).cuda(), torch.from_numpy(v).cuda(),
                                    torch.from_numpy(q.view(np.int32)).cuda(), k)
    oidx, odist = O.match_bits(q, bank, v, k)
    assert np.all(idx == N - 1) and np.array_equal(dist, odist) and hit.all()


def test_match_bits_empty_bank_and_thresholds(L):
    say("Hamming match: empty bank, max_hamming -1 and k")
    g = np.random.Generator(np.random.PCG64(12))
    N, B, k = 300, 7, 64
    bank = g.integers(0, 2 ** 32, size=(N, 2), dtype=np.uint64).astype(np.uint32)
    q = bank[:B].copy()
    tb, tq = torch.from_numpy(bank.view(np.int32)).cuda(), torch.from_numpy(q.view(np.int32)).cuda()
    idx, dist, hit = run_match_bits(L, tb, torch.zeros(N, dtype=torch.uint8).cuda(), tq, k)
    assert np.all(idx == -1) and np.all(dist == O.NO_MATCH_DIST) and not hit.any()
    ones = torch.ones(N, dtype=torch.uint8).cuda()
    idx, dist, hit = run_match_bits(L, tb, ones, tq, -1)        # tau >= 1: nothing hits, not even an identical key
    assert np.array_equal(idx, np.arange(B)) and np.all(dist == 0) and not hit.any()
    idx, dist, hit = run_match_bits(L, tb, ones, tq, k)
    assert hit.all()
    v = torch.zeros(N, dtype=torch.uint8)
    v[N - 1] = 1
    idx, dist, hit = run_match_bits(L, tb, v.cuda(), tq, k)
    assert np.all(idx == N - 1)


@pytest.mark.parametrize("N,B,k", [(3000, 50, 64), (777, 9, 128), (20000, 300, 256), (5000, 33, 512)])
def test_lsh_bucketed_match_is_exact_against_the_oracle(L, N, B, k):
    say(f"bucketed Hamming lookup N={N} B={B} k={k}")
    g = np.random.Generator(np.random.PCG64(N + k))
    W_ = k // 32
    bank = g.integers(0, 2 ** 32, size=(N, W_), dtype=np.uint64).astype(np.uint32)
    # few distinct values in band 0 of many keys: big buckets, candidates without being near
    bank[: N // 2, 0] = (bank[: N // 2, 0] & np.uint32(0xFFFF0000)) | np.uint32(0x1234)
    q = g.integers(0, 2 ** 32, size=(B, W_), dtype=np.uint64).astype(np.uint32)
    valid = (g.random(N) > 0.15).astype(np.uint8)
    for b in range(0, B, 2):
        j = int(g.integers(0, N))
        q[b] = bank[j]
        for _ in range(int(g.integers(0, 5))):
            i = int(g.integers(0, k))
            q[b, i // 32] ^= np.uint32(1 << (i % 32))
    q[1, 0] = (q[1, 0] & np.uint32(0xFFFF0000)) | np.uint32(0x1234)     # falls into the big bucket
    tb = torch.from_numpy(bank.view(np.int32)).cuda()
    tq = torch.from_numpy(q.view(np.int32)).cuda()
    tv = torch.from_numpy(valid).cuda()
    index = torch.empty((L.llmc_lsh_index_bytes(N, k),), dtype=torch.uint8, device="cuda")
    L.llmc_lsh_build(tb, tv, index)
    idx = torch.empty((B,), dtype=torch.int32, device="cuda")
    dist = torch.empty((B,), dtype=torch.int32, device="cuda")
    hit = torch.empty((B,), dtype=torch.uint8, device="cuda")
    cmpd = torch.empty((B,), dtype=torch.int32, device="cuda")
    max_h = O.max_hamming(f32(0.95), k)
    L.llmc_match_bits_lsh(tb, index, tq, max_h, idx, dist, hit, cmpd)
    torch.cuda.synchronize()
    oidx, odist, _ = O.match_bits_lsh(q, bank, valid, k)
    assert np.array_equal(idx.cpu().numpy(), oidx)
    assert np.array_equal(dist.cpu().numpy(), odist)
    assert np.array_equal(hit.cpu().numpy().astype(bool), O.threshold_bits(oidx, odist, max_h))
    # bucket members visited: over the bands, the valid slots equal to the query in that band
    want = np.zeros(B, np.int64)
    for band in range(k // 16):
        w, sh = band // 2, np.uint32(16 * (band % 2))
        qv = (q[:, w] >> sh) & np.uint32(0xFFFF)
        bv = (bank[:, w] >> sh) & np.uint32(0xFFFF)
        want += ((qv[:, None] == bv[None, :]) & (valid[None, :] == 1)).sum(axis=1)
    assert np.array_equal(cmpd.cpu().numpy(), want)
    # rebuilt after a change of validity, the lookup follows
    valid2 = valid.copy()
    gone = oidx[oidx >= 0][:5]
    valid2[gone] = 0
    L.llmc_lsh_build(tb, torch.from_numpy(valid2).cuda(), index)
    L.llmc_match_bits_lsh(tb, index, tq, max_h, idx, dist, hit, None)
    torch.cuda.synchronize()
    oidx2, odist2, _ = O.match_bits_lsh(q, bank, valid2, k)
    assert np.array_equal(idx.cpu().numpy(), oidx2) and np.array_equal(dist.cpu().numpy(), odist2)
    say(f"  {int((oidx >= 0).sum())} of {B} queries have candidates; visited per query: median {int(np.median(want))}, max {int(want.max())} of {N}")


def test_bit_keys_follow_the_cosine_match_on_a_clustered_bank(L):
    say("sign-bit keys of a clustered bank: the Hamming neighbour lies in the query's cluster, like the cosine neighbour")
    data = W.make_clustered_bank(64, 128, 256, 0.05, 512, seed=5)
    keys = data["bank"].cuda()                              # [8192, 256] bf16 unit vectors, 64 clusters
    qv = data["queries"].cuda()
    g = np.random.Generator(np.random.PCG64(21))
    kb = 256
    P = torch.from_numpy((g.standard_normal((256, kb)) / np.sqrt(kb)).astype(np.float32)).to(torch.bfloat16).cuda()
    N, B = keys.shape[0], qv.shape[0]
    ws = torch.empty((L.llmc_fingerprint_workspace_bytes(N, 1, 256),), dtype=torch.uint8, device="cuda")
    bank_bits = torch.empty((N, kb // 32), dtype=torch.int32, device="cuda")
    q_bits = torch.empty((B, kb // 32), dtype=torch.int32, device="cuda")
    L.llmc_fingerprint_bits(keys.view(N, 1, 256), P, None, bank_bits, ws)     # each key as a one-token sequence
    L.llmc_fingerprint_bits(qv.view(B, 1, 256), P, None, q_bits, ws)
    max_h = O.max_hamming(f32(0.95), kb)
    idx, dist, hit = run_match_bits(L, bank_bits, torch.ones(N, dtype=torch.uint8).cuda(), q_bits, max_h)
    oidx, odist = O.match_bits(words(q_bits), words(bank_bits), np.ones(N, np.uint8), kb)
    assert np.array_equal(idx, oidx) and np.array_equal(dist, odist)
    inside = data["q_cluster"].numpy() >= 0
    cl = data["cluster"].numpy()
    agree = (cl[idx[inside]] == data["q_cluster"].numpy()[inside]).mean()
    say(f"  within-cluster queries matched into their cluster: {agree:.3f}; hits {hit[inside].mean():.3f} inside, "
        f"{hit[~inside].mean():.3f} outside (max_hamming {max_h})")
    assert agree > 0.99 and hit[inside].mean() > 0.95 and hit[~inside].mean() < 0.01


# ---------------------------------------------------------------------------
# step 4: gather
# ---------------------------------------------------------------------------

def test_gather_hits_is_exact_copy_with_shared_value_rows(L):
    say("gather with an act_slot map")
    g = np.random.Generator(np.random.PCG64(8))
    N, A, S, d = 64, 8, 33, 128
    keys = torch.from_numpy(unit_rows(g, N, 32).astype(np.float32)).to(torch.bfloat16).cuda()
    act = torch.from_numpy(g.standard_normal((A, S, d)).astype(np.float32)).to(torch.bfloat16).cuda()
    act_slot = torch.from_numpy((np.arange(N) % A).astype(np.int32)).cuda()
    bank = make_bank(L, keys, S=S, d=d, act=act, act_slot=act_slot, A=A)
    B = 10
    idx = torch.from_numpy(g.integers(0, N, B).astype(np.int32)).cuda()
    rows = torch.tensor([0, 2, 3, 7, 9, 1, 1, 1, 1, 1], dtype=torch.int32, device="cuda")
    n = torch.tensor([5], dtype=torch.int32, device="cuda")
    out = torch.full((B, S, d), -7.0, dtype=torch.bfloat16, device="cuda")
    L.llmc_gather_hits(bank, idx, rows, n, B, out)
    torch.cuda.synchronize()
    for b in range(B):
        if b in (0, 2, 3, 7, 9):
            assert torch.equal(out[b], act[int(idx[b]) % A])
        else:
            assert torch.all(out[b] == -7.0)
    bank.close()


# ---------------------------------------------------------------------------
# step 5: the block f_l on its own (uncached layer)
# ---------------------------------------------------------------------------

def small_cfg(arch, dtype, d=128, heads=2, dff=256, S=33, B=5, **kw):
    return W.scaled(W.TINY_ENCODER, arch=arch, dtype=dtype, d=d, n_heads=heads, d_ff=dff, S=S, B=B, n_layers=1,
                    gelu=O.GELU_ERF if arch == 0 else O.GELU_TANH, ln_eps=1e-12 if arch == 0 else 1e-5, **kw)


@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("dtype,d,heads,dff,S,B", [
    ("f32", 128, 2, 512, 32, 8),
    ("f32", 64, 1, 64, 7, 3),
    ("bf16", 128, 2, 256, 33, 5),      # 165 tokens: ragged against the 128-row tile
    ("bf16", 768, 12, 3072, 130, 2),   # model-sized widths, several k steps, S past one query block
])
def test_uncached_layer_matches_oracle(L, arch, dtype, d, heads, dff, S, B):
    say(f"plain layer arch={arch} {dtype} d={d} heads={heads} dff={dff} S={S} B={B}")
    from paper_2512_16843_amd.engine import GatedStack
    cfg = small_cfg(arch, dtype, d, heads, dff, S, B)
    ws = W.make_layer_weights(cfg, seed=11)
    g = np.random.Generator(np.random.PCG64(S))
    h0 = torch.from_numpy(g.standard_normal((B, S, d)).astype(np.float32)).to(cfg.torch_dtype).cuda()
    st = GatedStack(cfg, ws, W.make_projection(d, cfg.k, cfg.torch_dtype), cached_layers=[])
    out = st.forward(h0, tau=0.5)
    torch.cuda.synchronize()
    wnp = {k: npf(v) for k, v in ws[0].items()}
    want = np.stack([O.layer_forward(npf(h0[b]), wnp, arch, heads, cfg.ln_eps, cfg.gelu) for b in range(B)])
    err = rel_err_rows(npf(out), want)
    say(f"  max rel err {err.max():.3e}")
    assert err.max() < TOL[dtype]
    cnt = st.hit_counts()
    assert cnt[0, L.CNT_MISS] == B and cnt[0, L.CNT_HIT] == 0


# ---------------------------------------------------------------------------
# the gated stack, free-running in fp32 (tiny-encoder config, whole run incl. bank build)
# ---------------------------------------------------------------------------

def build_banks_gpu(L, st, h_src, tick=1):
    """All-miss pass with insertion over the source sequences, batch by batch."""
    Bn = st.B
    outs = []
    for s in range(0, h_src.shape[0], Bn):
        outs.append([o.clone() for o in st.forward(h_src[s:s + Bn].contiguous(), tau=2.0,
                                                   flags=L.INSERT_ON_MISS, tick=tick, keep_all=True)])
    torch.cuda.synchronize()
    return outs


def test_tiny_encoder_free_running_with_bank_build(L):
    say("tiny encoder fp32: bank build + gated queries, free running")
    from paper_2512_16843_amd.engine import GatedStack
    cfg = W.TINY_ENCODER
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, torch.float32, seed=3, n_layers=cfg.n_layers)
    src = W.make_sources(cfg, cfg.n_bank, seed=1)
    h_src = W.embed(torch.from_numpy(src), tok, pos, torch.float32)
    st = GatedStack(cfg, ws, Ps)
    build_banks_gpu(L, st, h_src.cuda())
    # oracle builds its own banks from the same inputs
    wnp = [{k: npf(v) for k, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    obanks = [O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, "f32") for _ in range(cfg.n_layers)]
    for s in range(0, cfg.n_bank, cfg.B):
        O.infer(h_src[s:s + cfg.B].numpy(), obanks, Pnp, [None] * cfg.n_layers, wnp, cfg.arch, cfg.n_heads,
                cfg.ln_eps, cfg.gelu, tau=2.0, flags=O.FLAG_INSERT_ON_MISS, tick=1)
    for l in range(cfg.n_layers):
        b = st.banks[l]
        assert torch.all(b.valid == 1)
        np.testing.assert_allclose(npf(b.fp), obanks[l].fp, atol=3e-6)
        assert rel_err_rows(npf(b.act), obanks[l].act).max() < TOL["f32"]
        assert torch.all(b.last_used == 1) and torch.all(b.hits == 0)
    # queries: half near-duplicates (1-2 substitutions), half fresh
    ids, srcmap = W.make_substitution_queries(cfg, src, n_dup=cfg.B // 2, n_subst=(1, 2), seed=2)
    h0 = W.embed(torch.from_numpy(ids), tok, pos, torch.float32)
    tau = 0.95
    outs = st.forward(h0.cuda(), tau=tau, keep_all=True)
    torch.cuda.synchronize()
    _, res = O.infer(h0.numpy(), obanks, Pnp, [None] * cfg.n_layers, wnp, cfg.arch, cfg.n_heads, cfg.ln_eps,
                     cfg.gelu, tau=f32(tau))
    n_near = 0
    for l in range(cfg.n_layers):
        g = st.gate[l]
        r = res[l]
        near = np.abs(r.sim - f32(tau)) < 1e-3
        n_near += int(near.sum())
        hit = g.hit.cpu().numpy().astype(bool)
        assert np.array_equal(hit[~near], r.hit[~near])
        assert np.array_equal(g.idx.cpu().numpy()[~near], r.idx[~near])
        np.testing.assert_allclose(npf(g.sim), r.sim, atol=1e-5)
        ok = ~near
        err = rel_err_rows(npf(outs[l])[ok], r.h_out[ok])
        assert err.max() < TOL["f32"], err
        cnt = st.hit_counts()[l]
        assert cnt[L.CNT_HIT] == hit.sum() and cnt[L.CNT_MISS] == cfg.B - hit.sum()
        say(f"  layer {l}: hits {int(hit.sum())}/{cfg.B}, near-threshold rows {int(near.sum())}, max err {err.max():.2e}")
        if near.any():
            break       # a row excused at this layer may legitimately diverge afterwards
    st.close()


def test_gated_invariants_on_gpu(L):
    say("tau > 1 equals the uncached path bit for bit; resubmitted sources hit at 1 with stored values")
    from paper_2512_16843_amd.engine import GatedStack
    cfg = W.scaled(W.TINY_ENCODER, n_bank=64)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, torch.float32, seed=3, n_layers=cfg.n_layers)
    src = W.make_sources(cfg, 64, seed=1)
    h_src = W.embed(torch.from_numpy(src), tok, pos, torch.float32).cuda()
    st = GatedStack(cfg, ws, Ps)
    build_banks_gpu(L, st, h_src)
    plain = GatedStack(cfg, ws, Ps, cached_layers=[])
    ids, _ = W.make_substitution_queries(cfg, src, n_dup=4, n_subst=1, seed=9)
    h0 = W.embed(torch.from_numpy(ids), tok, pos, torch.float32).cuda()
    a = st.forward(h0, tau=1.0 + 1e-3).clone()
    b = plain.forward(h0, tau=0.0).clone()
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert st.hit_counts()[:, L.CNT_HIT].sum() == 0
    outs = st.forward(h_src[8:16].contiguous(), tau=0.95, keep_all=True)
    torch.cuda.synchronize()
    for l in range(cfg.n_layers):
        assert torch.all(st.gate[l].hit == 1)
        assert st.gate[l].idx.cpu().tolist() == list(range(8, 16))
        np.testing.assert_allclose(npf(st.gate[l].sim), 1.0, atol=1e-6)
        assert torch.equal(outs[l], st.banks[l].act[8:16])
    # a permuted, smaller batch gives the same rows bit for bit (row independence)
    small = GatedStack(cfg, ws, Ps, cached_layers=[], B=3)
    c = small.forward(h0[[5, 0, 2]].contiguous(), tau=0.0)
    torch.cuda.synchronize()
    assert torch.equal(c, b[[5, 0, 2]])
    st.close(); plain.close(); small.close()


# ---------------------------------------------------------------------------
# step 6: insertion and LRU
# ---------------------------------------------------------------------------

def test_bank_insert_and_evict_direct(L):
    say("bank insert / evict against the oracle bank, device-side counts")
    g = np.random.Generator(np.random.PCG64(12))
    N, k, S, d = 40, 32, 3, 64
    bank = L.Bank(N, k, S, d, torch.bfloat16, "cuda")
    ob = O.Bank(N, k, S, d, "bf16")
    counters = torch.zeros((L.CNT_WORDS,), dtype=torch.int32, device="cuda")
    for tick in range(1, 12):
        mmax = 16
        m = int(g.integers(0, mmax + 1))
        keys = torch.from_numpy(unit_rows(g, mmax, k).astype(np.float32)).to(torch.bfloat16).cuda()
        inv = torch.empty((mmax,), dtype=torch.float32, device="cuda")
        L.llmc_inv_norm(keys, inv)
        acts = torch.from_numpy(g.standard_normal((mmax, S, d)).astype(np.float32)).to(torch.bfloat16).cuda()
        rows = torch.from_numpy(g.permutation(mmax).astype(np.int32)).cuda()
        dm = torch.tensor([m], dtype=torch.int32, device="cuda")
        slots = torch.full((mmax,), -5, dtype=torch.int32, device="cuda")
        L.llmc_bank_insert(bank, keys, inv, acts, rows, dm, mmax, tick, slots, counters)
        # touch a few random valid entries (what a hit does), same on both sides
        torch.cuda.synchronize()
        r = rows.cpu().numpy()[:m]
        oslots, _ = ob.insert(npf(keys)[r], npf(inv)[r], npf(acts)[r], tick)
        assert slots.cpu().tolist() == oslots + [-1] * (mmax - m)
        live = np.nonzero(ob.valid)[0]
        touched = g.choice(live, size=min(3, len(live)), replace=False)
        ob.touch(touched.tolist(), tick + 100)
        bank.last_used[torch.from_numpy(touched).cuda()] = tick + 100
        bank.hits[torch.from_numpy(touched).cuda()] += 1
        if tick % 4 == 0:
            vm = int(g.integers(1, 6))
            vic = torch.empty((8,), dtype=torch.int32, device="cuda")
            L.llmc_bank_evict(bank, torch.tensor([vm], dtype=torch.int32, device="cuda"), 8, vic)
            torch.cuda.synchronize()
            assert vic.cpu().tolist() == ob.evict(vm) + [-1] * (8 - vm)
        torch.cuda.synchronize()
        assert np.array_equal(bank.valid.cpu().numpy(), ob.valid)
        v = ob.valid.astype(bool)
        assert np.array_equal(bank.last_used.cpu().numpy().astype(np.uint64)[v], ob.last_used[v])
        assert np.array_equal(bank.hits.cpu().numpy().astype(np.uint32)[v], ob.hits[v])
        assert np.array_equal(npf(bank.fp)[v], ob.fp[v])
        assert np.array_equal(npf(bank.act)[v], ob.act[v])
        assert np.array_equal(npf(bank.inv_norm)[v], ob.inv_norm[v])
    assert int(counters[L.CNT_EVICTED]) > 0 and int(counters[L.CNT_INSERTED]) > N
    bank.close()


@pytest.mark.parametrize("N,big_ticks", [(3000, False), (10000, True), (40000, False), (40000, True), (70000, True)])
def test_slot_selection_at_size(L, N, big_ticks):
    """Victims and insertion slots over banks of every size class of the selection kernel (keys held in registers
    up to 49,152 slots, re-read beyond), with ticks that do or do not reach the high bytes of the recency key."""
    say(f"slot selection N={N} big_ticks={big_ticks}")
    g = np.random.Generator(np.random.PCG64(N + int(big_ticks)))
    k, S, d = 32, 1, 64
    bank = L.Bank(N, k, S, d, torch.bfloat16, "cuda")
    ob = O.Bank(N, k, S, d, "bf16")
    valid = (g.random(N) > 0.002).astype(np.uint8)
    hi = (1 << 31) - 10 if big_ticks else 300
    lu = g.integers(0, hi, size=N).astype(np.uint64)
    lu[g.integers(0, N, size=N // 3)] = 7                       # many equal recencies: the slot number decides
    ob.valid[:] = valid
    ob.last_used[:] = lu
    bank.valid.copy_(torch.from_numpy(valid))
    bank.last_used.copy_(torch.from_numpy(lu.astype(np.int64)))
    bank.refresh()
    # eviction of 150 entries
    vic = torch.empty((256,), dtype=torch.int32, device="cuda")
    L.llmc_bank_evict(bank, torch.tensor([150], dtype=torch.int32, device="cuda"), 256, vic)
    torch.cuda.synchronize()
    assert vic.cpu().tolist() == ob.evict(150) + [-1] * 106
    assert np.array_equal(bank.valid.cpu().numpy(), ob.valid)
    # insertion of 400 rows: the free slots (evicted ones included) by ascending index first, then LRU victims
    m = 400
    keys = torch.from_numpy(unit_rows(g, m, k).astype(np.float32)).to(torch.bfloat16).cuda()
    inv = torch.empty((m,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(keys, inv)
    acts = torch.from_numpy(g.standard_normal((m, S, d)).astype(np.float32)).to(torch.bfloat16).cuda()
    slots = torch.empty((m,), dtype=torch.int32, device="cuda")
    counters = torch.zeros((L.CNT_WORDS,), dtype=torch.int32, device="cuda")
    tick = hi + 1
    L.llmc_bank_insert(bank, keys, inv, acts, None, None, m, tick, slots, counters)
    torch.cuda.synchronize()
    oslots, n_ev = ob.insert(npf(keys), npf(inv), npf(acts), tick)
    assert slots.cpu().tolist() == oslots
    assert int(counters[L.CNT_EVICTED]) == n_ev and int(counters[L.CNT_INSERTED]) == m
    assert np.array_equal(bank.valid.cpu().numpy(), ob.valid)
    bank.close()


def test_decayed_hits_policy_stream_against_oracle(L):
    """Staleness-aware replacement on the device, step by step against the oracle bank: hits recorded by the gate's
    own compaction kernel (through llmc_layer_forward_gated would need a model; here hits are recorded the way that
    kernel does it and the halving, the selection and the eviction counters come from the library)."""
    say("decayed-hits replacement: scripted stream of hits, insertions and evictions")
    g = np.random.Generator(np.random.PCG64(31))
    N, k, S, d, half_life = 48, 32, 2, 64, 4
    bank = L.Bank(N, k, S, d, torch.bfloat16, "cuda", policy=L.EVICT_DECAYED_HITS, half_life=half_life)
    ob = O.Bank(N, k, S, d, "bf16", decayed_hits=True, half_life=half_life)
    counters = torch.zeros((L.CNT_WORDS,), dtype=torch.int32, device="cuda")
    for tick in range(1, 40):
        mmax = 12
        m = int(g.integers(0, mmax + 1)) if tick % 2 == 1 else 0
        keys = torch.from_numpy(unit_rows(g, mmax, k).astype(np.float32)).to(torch.bfloat16).cuda()
        inv = torch.empty((mmax,), dtype=torch.float32, device="cuda")
        L.llmc_inv_norm(keys, inv)
        acts = torch.from_numpy(g.standard_normal((mmax, S, d)).astype(np.float32)).to(torch.bfloat16).cuda()
        slots = torch.full((mmax,), -5, dtype=torch.int32, device="cuda")
        dm = torch.tensor([m], dtype=torch.int32, device="cuda")
        # the insert call brings the hit counts to this tick's epoch first (also with m = 0)
        L.llmc_bank_insert(bank, keys, inv, acts, None, dm, mmax, tick, slots, counters)
        torch.cuda.synchronize()
        oslots, _ = ob.insert(npf(keys)[:m], npf(inv)[:m], npf(acts)[:m], tick)
        assert slots.cpu().tolist() == oslots + [-1] * (mmax - m), (tick, slots.cpu().tolist(), oslots)
        # hits of this tick (after the halving): some entries several times
        live = np.nonzero(ob.valid)[0]
        hit_slots = g.choice(live, size=min(5, len(live)), replace=True).tolist() if len(live) else []
        ob.touch(hit_slots, tick)
        for j in hit_slots:
            bank.last_used[j] = tick
            bank.hits[j] += 1
        if tick % 5 == 0:
            vm = int(g.integers(1, 4))
            vic = torch.empty((4,), dtype=torch.int32, device="cuda")
            L.llmc_bank_evict(bank, torch.tensor([vm], dtype=torch.int32, device="cuda"), 4, vic)
            torch.cuda.synchronize()
            assert vic.cpu().tolist() == ob.evict(vm) + [-1] * (4 - vm)
        torch.cuda.synchronize()
        v = ob.valid.astype(bool)
        assert np.array_equal(bank.valid.cpu().numpy(), ob.valid)
        assert np.array_equal(bank.hits.cpu().numpy().astype(np.uint32)[v], ob.hits[v]), tick
        assert np.array_equal(bank.last_used.cpu().numpy().astype(np.uint64)[v], ob.last_used[v])
    assert int(counters[L.CNT_EVICTED]) > 0
    bank.close()


def test_gated_stream_with_decayed_hits_policy(L):
    """The gated layer itself with INSERT_ON_MISS | UPDATE_LRU on banks ranked by decayed hits: slots taken, hit counts
    and recency after every batch against the oracle (tiny fp32 encoder, so decisions are far from the threshold)."""
    from paper_2512_16843_amd.engine import GatedStack
    say("gated stream, decayed-hits banks: repeated and fresh sequences over 10 batches")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=6, n_bank=10)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, policy=L.EVICT_DECAYED_HITS, half_life=3)
    obanks = [O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, "f32", decayed_hits=True, half_life=3) for _ in range(cfg.n_layers)]
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    pool = W.make_sources(cfg, 14, seed=1)
    g = np.random.Generator(np.random.PCG64(32))
    flags = L.INSERT_ON_MISS | L.UPDATE_LRU
    evicted = 0
    for tick in range(1, 11):
        ids = pool[g.integers(0, 6 if tick < 5 else 14, size=cfg.B)]      # early batches revisit a few sources
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
        st.forward(h0, tau=0.99, flags=flags, tick=tick)
        torch.cuda.synchronize()
        _, res = O.infer(npf(h0), obanks, Pnp, [None] * cfg.n_layers, wnp, cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu,
                         tau=f32(0.99), flags=O.FLAG_INSERT_ON_MISS | O.FLAG_UPDATE_LRU, tick=tick, out_dtype="f32")
        for l in range(cfg.n_layers):
            gate, r, bk, ob = st.gate[l], res[l], st.banks[l], obanks[l]
            near = np.abs(r.sim - f32(0.99)) < 1e-3
            assert not near.any()
            assert np.array_equal(gate.hit.cpu().numpy().astype(bool), r.hit)
            n_miss = int((~r.hit).sum())
            assert gate.slots.cpu().tolist()[:n_miss] == r.slots, (tick, l)
            v = ob.valid.astype(bool)
            assert np.array_equal(bk.valid.cpu().numpy(), ob.valid)
            assert np.array_equal(bk.hits.cpu().numpy().astype(np.uint32)[v], ob.hits[v]), (tick, l)
            assert np.array_equal(bk.last_used.cpu().numpy().astype(np.uint64)[v], ob.last_used[v])
            evicted += r.n_evicted
    assert evicted > 0
    st.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_divergence_monitor_against_oracle(L, dtype):
    """Sampled hit rows are recomputed; cached values that drifted are replaced by the fresh output, the others
    stay bit for bit; duplicates of one entry are decided by the lowest row.  Oracle banks are copies of the GPU's."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"divergence monitor {dtype}: drifted and clean cached values, duplicate rows, with and without insertion")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=8, n_bank=24) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=2, B=8, S=40, n_bank=24)
    tol = TOL[dtype]
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, reval_every=2, drift_bound=0.05)
    src = W.make_sources(cfg, 16, seed=1)
    for s0 in (0, 8):
        st.forward(W.embed(torch.from_numpy(src[s0:s0 + 8]), tok, pos, cfg.torch_dtype).cuda(), tau=2.0,
                   flags=L.INSERT_ON_MISS, tick=1)
    torch.cuda.synchronize()
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    g = np.random.Generator(np.random.PCG64(41))
    # queries: sources 0..5, source 3 again twice (duplicates of one entry), one fresh sequence
    ids = np.concatenate([src[[0, 1, 2, 3, 3, 5, 3]], W.make_sources(cfg, 1, seed=9)], axis=0)
    h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    # drift some cached values of layer 0 on the device: slots of sources 1, 3 and 5
    for j in (1, 3, 5):
        st.banks[0].act[j] += torch.from_numpy((0.5 * g.standard_normal((cfg.S, cfg.d))).astype(np.float32)).to(cfg.torch_dtype).cuda()
    for tick, flags in ((4, L.REVALIDATE | L.UPDATE_LRU), (5, L.REVALIDATE | L.INSERT_ON_MISS)):
        obanks = [oracle_bank_from_gpu(b, dtype) for b in st.banks]
        act_before = [b.act.clone() for b in st.banks]
        outs = st.forward(h0, tau=0.9, flags=flags, tick=tick, keep_all=True)
        torch.cuda.synchronize()
        oflags = O.FLAG_REVALIDATE | (O.FLAG_UPDATE_LRU if flags & L.UPDATE_LRU else 0) | \
            (O.FLAG_INSERT_ON_MISS if flags & L.INSERT_ON_MISS else 0)
        for l in range(cfg.n_layers):
            h_prev = h0 if l == 0 else outs[l - 1]
            ob = obanks[l]
            r = O.gated_layer(npf(h_prev), ob, Pnp[l], None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu,
                              f32(0.9), flags=oflags, tick=tick, out_dtype=dtype, reval_every=2, drift_bound=0.05)
            gate, bk = st.gate[l], st.banks[l]
            assert not (np.abs(r.sim - f32(0.9)) < 1e-3).any()
            hit = gate.hit.cpu().numpy().astype(bool)
            assert np.array_equal(hit, r.hit) and np.array_equal(gate.idx.cpu().numpy()[hit], r.idx[hit])
            cnt = gate.counters.cpu().numpy()
            assert cnt[L.CNT_REVALIDATED] == len(r.revalidated) and cnt[L.CNT_DIVERGED] == len(r.refreshed), (l, cnt, r.refreshed)
            assert cnt[L.CNT_COMPUTED] == cnt[L.CNT_MISS] + cnt[L.CNT_REVALIDATED] and cnt[L.CNT_HIT] + cnt[L.CNT_MISS] == cfg.B
            for d_ in r.divergence:
                assert abs(d_ - 0.05) > 0.02          # decisions of this test sit far from the bound
            got = npf(outs[l])
            for b in range(cfg.B):
                if hit[b] and b not in r.revalidated:
                    assert torch.equal(outs[l][b], act_before[l][int(r.idx[b])])
                else:                                 # computed: misses and recomputed hits
                    assert rel_err_rows(got[b:b + 1], r.h_out[b:b + 1])[0] < tol, (l, b)
            after = npf(bk.act)
            taken = set(r.slots)
            for j in range(cfg.n_bank):
                if j in r.refreshed or j in taken:
                    assert rel_err_rows(after[j:j + 1], np.asarray(ob.act[j:j + 1]))[0] < tol, (l, j)
                else:
                    assert torch.equal(bk.act[j], act_before[l][j]), (l, j)
            if flags & L.INSERT_ON_MISS:
                assert gate.slots.cpu().tolist()[:int(cnt[L.CNT_MISS])] == r.slots
            if l == 0:
                # tick 4 samples rows 0, 2, 4, 6: rows 4 and 6 both matched the drifted entry 3 and row 4 decides;
                # tick 5 samples the hit rows 1, 3, 5: entries 1 and 5 drifted, entry 3 was replaced one tick earlier
                assert sorted(r.refreshed) == ([3] if tick == 4 else [1, 5])
        say(f"  tick {tick}: layer-0 recomputed rows {res_rows(st, L)}, replaced {int(st.gate[0].counters[L.CNT_DIVERGED])}")
    st.close()


def res_rows(st, L):
    c = st.gate[0].counters.cpu().numpy()
    return int(c[L.CNT_REVALIDATED])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_compressed_values_against_oracle(L, dtype):
    """Banks that store coefficients on a basis: what insertion stores (C = h U^T) and what a hit returns (C U),
    both against the oracle, through the gated layer and through llmc_gather_hits."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"compressed cached values {dtype}: rank 64 basis, build by insertion, hits return reconstructions")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=8, n_bank=24) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=2, B=8, S=40, n_bank=24)
    tol, r = TOL[dtype], 64
    g = np.random.Generator(np.random.PCG64(51))
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    bases = []
    for l in range(cfg.n_layers):
        Q, _ = np.linalg.qr(g.standard_normal((cfg.d, r)))
        bases.append(torch.from_numpy(Q.T.astype(np.float32)).to(cfg.torch_dtype).contiguous())
    st = GatedStack(cfg, ws, Ps, bases=bases)
    obanks = [O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, dtype, basis=npf(bases[l])) for l in range(cfg.n_layers)]
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    src = W.make_sources(cfg, 16, seed=1)
    for tick, s0 in ((1, 0), (2, 8)):
        h0 = W.embed(torch.from_numpy(src[s0:s0 + 8]), tok, pos, cfg.torch_dtype).cuda()
        outs = st.forward(h0, tau=2.0, flags=L.INSERT_ON_MISS, tick=tick, keep_all=True)
        torch.cuda.synchronize()
        for l in range(cfg.n_layers):
            h_prev = h0 if l == 0 else outs[l - 1]
            rr = O.gated_layer(npf(h_prev), obanks[l], Pnp[l], None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu,
                               2.0, flags=O.FLAG_INSERT_ON_MISS, tick=tick, out_dtype=dtype)
            assert st.gate[l].slots.cpu().tolist() == rr.slots
            # stored coefficients of the rows just inserted, teacher-forced: the oracle encodes the GPU's own outputs
            want = obanks[l].encode(npf(outs[l]))
            got = npf(st.banks[l].act)[rr.slots]
            assert rel_err_rows(got, want).max() < tol, (l, rel_err_rows(got, want).max())
            obanks[l].act[rr.slots] = got                 # continue from the GPU's stored coefficients
    assert st.banks[0].act.shape == (cfg.n_bank, cfg.S, r)
    # resubmitted sources plus fresh rows: hits return C U
    ids = np.concatenate([src[[0, 5, 9, 15]], W.make_sources(cfg, 4, seed=9)], axis=0)
    h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    outs = st.forward(h0, tau=0.9, keep_all=True)
    torch.cuda.synchronize()
    for l in range(cfg.n_layers):
        h_prev = h0 if l == 0 else outs[l - 1]
        rr = O.gated_layer(npf(h_prev), obanks[l], Pnp[l], None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu,
                           f32(0.9))
        hit = st.gate[l].hit.cpu().numpy().astype(bool)
        assert not (np.abs(rr.sim - f32(0.9)) < 1e-3).any()
        assert np.array_equal(hit, rr.hit) and np.array_equal(st.gate[l].idx.cpu().numpy()[hit], rr.idx[hit])
        assert hit.sum() >= 4 if l == 0 else True
        err = rel_err_rows(npf(outs[l]), rr.h_out)
        assert err.max() < tol, (l, err)
        say(f"  layer {l}: {int(hit.sum())} hits, max rel err of reconstructed / computed rows {err.max():.2e}")
    # the gather entry point alone, rows listed out of order, with a device count
    bank, ob = st.banks[0], obanks[0]
    idx = torch.tensor([3, 0, 7, 11, 2, 5, 1, 9], dtype=torch.int32, device="cuda")
    rows = torch.tensor([6, 1, 4, 0, 7], dtype=torch.int32, device="cuda")
    n = torch.tensor([3], dtype=torch.int32, device="cuda")
    out = torch.zeros((8, cfg.S, cfg.d), dtype=cfg.torch_dtype, device="cuda")
    L.llmc_gather_hits(bank, idx, rows, n, 5, out)
    torch.cuda.synchronize()
    for b in (6, 1, 4):
        want = ob.value(int(idx[b]))
        assert rel_err_rows(npf(out[b:b + 1]), want[None])[0] < tol
    assert torch.all(out[[0, 2, 3, 5, 7]] == 0)
    st.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_carried_token_means_change_nothing(L, dtype):
    """Banks that keep the token mean of every cached output hand it to the next layer for reused rows, which is then
    not pooled again.  Keys, decisions, similarities and outputs must be the same bits as without the carry, the
    stored means must be what the pooling arithmetic gives for the stored outputs, and the flags must follow the hits."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"carried token means {dtype}: stack with and without the carry, bit for bit")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=3, B=8, n_bank=24) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=3, B=8, S=70, n_bank=24)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    stacks = [GatedStack(cfg, ws, Ps, keep_means=km, keep_next_keys=kk)
              for km, kk in ((False, False), (True, False), (True, True))]
    final = []
    src = W.make_sources(cfg, 16, seed=1)
    fresh = W.make_sources(cfg, 8, seed=9)
    batches = [(src[0:8], 2.0, L.INSERT_ON_MISS), (src[8:16], 2.0, L.INSERT_ON_MISS),
               (np.concatenate([src[[0, 5, 9, 15]], fresh[:4]]), 0.9, 0),
               (np.concatenate([src[[3, 3, 12]], fresh[3:8]]), 0.9, L.INSERT_ON_MISS | L.UPDATE_LRU),   # evicts
               (np.concatenate([fresh[4:8], src[[1, 2, 14, 7]]]), 0.9, L.UPDATE_LRU)]
    for tick, (ids, tau, flags) in enumerate(batches, start=1):
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
        outs = [st.forward(h0, tau=tau, flags=flags, tick=tick, keep_all=True) for st in stacks]
        torch.cuda.synchronize()
        if not (flags & L.INSERT_ON_MISS):
            # the same batch once more without keeping every layer: reused rows travel as references (deferred
            # copies) through the stack with stored keys; final output, decisions and slots must be the same bits
            y_plain = stacks[0].forward(h0, tau=tau, flags=flags, tick=tick).clone()
            hits_plain = [g.hit.clone() for g in stacks[0].gate]
            idx_plain = [g.idx.clone() for g in stacks[0].gate]
            y_defer = stacks[2].forward(h0, tau=tau, flags=flags, tick=tick).clone()
            torch.cuda.synchronize()
            assert torch.equal(y_plain, y_defer), tick
            for l in range(cfg.n_layers):
                assert torch.equal(hits_plain[l], stacks[2].gate[l].hit) and torch.equal(idx_plain[l], stacks[2].gate[l].idx)
            refs = [int((g.ref >= 0).sum()) for g in stacks[2].gate]
            final.append(refs)
            y_off = stacks[2].forward(h0, tau=tau, flags=flags, tick=tick, defer=False).clone()
            torch.cuda.synchronize()
            assert torch.equal(y_plain, y_off)
        for l in range(cfg.n_layers):
          for other in (1, 2):
            a, b = stacks[0].gate[l], stacks[other].gate[l]
            assert torch.equal(a.hit, b.hit) and torch.equal(a.idx, b.idx) and torch.equal(a.sim, b.sim), (tick, l)
            assert torch.equal(a.counters, b.counters)
            assert torch.equal(outs[0][l], outs[other][l]), (tick, l)
            # reused rows carry their stored mean (flag 1); computed rows of a post-LayerNorm block were pooled by its
            # last LayerNorm on the way out (flag 2)
            assert torch.equal(b.pooled_valid, torch.where(b.hit.bool(), 1, 2).to(torch.uint8))
            assert torch.equal(stacks[0].banks[l].act, stacks[other].banks[l].act)
            assert torch.equal(stacks[0].banks[l].fp, stacks[other].banks[l].fp)
            hit_rows = torch.nonzero(b.hit).flatten()
            if len(hit_rows):
                want = stacks[other].banks[l].act_pool[b.idx[hit_rows].long()]
                assert torch.equal(b.pooled[hit_rows], want)
                if b.key is not None:
                    assert torch.equal(b.key[hit_rows], stacks[other].banks[l].next_fp[b.idx[hit_rows].long()])
        say(f"  batch {tick}: hits per layer {[int(g.hit.sum()) for g in stacks[1].gate]}")
    # stored means = the pooling arithmetic on the stored outputs (recomputed by the library), and = the plain mean
    bk = stacks[1].banks[1]
    stored = bk.act_pool.clone()
    bk.act_pool.zero_()
    L.llmc_bank_pool_values(bk)
    torch.cuda.synchronize()
    v = bk.valid.bool()
    assert torch.equal(bk.act_pool[v], stored[v])
    ref = npf(bk.act)[v.cpu().numpy()].astype(np.float64).mean(axis=1)
    np.testing.assert_allclose(npf(bk.act_pool[v]), ref, rtol=0, atol=1e-5 * max(1.0, np.abs(ref).max()))
    # a row that is a reference and then has to be computed: free two entries of layer 2's banks, so that rows which
    # hit at layer 1 miss at layer 2 (their input is copied from layer 1's bank just in time) and hit again at layer 3
    ids, tau, _ = batches[2]
    h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    stacks[0].forward(h0, tau=tau)
    torch.cuda.synchronize()
    gone = stacks[0].gate[1].idx[:2].long().cpu()
    for st in stacks:
        st.banks[1].valid[gone.cuda()] = 0
        st.banks[1].refresh()
    y_plain = stacks[0].forward(h0, tau=tau).clone()
    pattern = [int(g.hit.sum()) for g in stacks[0].gate]
    y_defer = stacks[2].forward(h0, tau=tau).clone()
    torch.cuda.synchronize()
    assert pattern[1] <= pattern[0] - 2 and pattern[2] >= pattern[1], pattern      # some references had to be computed
    assert torch.equal(y_plain, y_defer)
    for l in range(cfg.n_layers):
        assert torch.equal(stacks[0].gate[l].hit, stacks[2].gate[l].hit)
    say(f"  with two entries of layer 2 freed: hits per layer {pattern}, deferred run equal")
    say(f"  rows left as references per layer in the deferred runs: {final}")
    assert any(sum(r) > 0 for r in final)
    # stored next-layer keys = the fingerprint of the stored outputs under the next layer's map, bit for bit,
    # both as written at insertion and as recomputed by llmc_bank_pool_values
    bk = stacks[2].banks[0]
    assert bk.next_fp is not None and stacks[2].banks[cfg.n_layers - 1].next_fp is None
    v = bk.valid.bool()
    acts = bk.act[v].contiguous()
    n = acts.shape[0]
    fp = torch.empty((n, cfg.k), dtype=cfg.torch_dtype, device="cuda")
    inv = torch.empty((n,), dtype=torch.float32, device="cuda")
    wsf = torch.empty((L.llmc_fingerprint_workspace_bytes(n, cfg.S, cfg.d),), dtype=torch.uint8, device="cuda")
    L.llmc_fingerprint(acts, stacks[2].proj[1], None, fp, inv, wsf)
    torch.cuda.synchronize()
    assert torch.equal(bk.next_fp[v], fp) and torch.equal(bk.next_inv[v], inv)
    bk.next_fp.zero_()
    bk.next_inv.zero_()
    L.llmc_bank_pool_values(bk)
    torch.cuda.synchronize()
    assert torch.equal(bk.next_fp[v], fp) and torch.equal(bk.next_inv[v], inv)
    for st in stacks:
        st.close()


@pytest.mark.parametrize("lsh", [False, True], ids=["full", "bucketed"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gated_stack_with_sign_bit_banks(L, dtype, lsh):
    """Banks of sign-bit keys inside the gated layer: keys, matched slots, distances' cosines, decisions, slots taken
    and outputs against the oracle, layer by layer with the GPU's own layer inputs and bank arrays.  "bucketed": the
    lookup goes through the bank's band buckets, which the library rebuilds after every batch that stored or
    replaced keys (insertions into free slots, then evictions)."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"gated stack with sign-bit banks {dtype} lsh={lsh}: build by insertion, resubmissions, near-duplicates, eviction")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=8, n_bank=20) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=2, B=8, S=48, n_bank=20)
    tol = TOL[dtype]
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, key_bits=True, keep_means=True, lsh=lsh)
    look = L.LOOKUP_LSH if lsh else 0
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    src = W.make_sources(cfg, 16, seed=1)
    near, _ = W.make_substitution_queries(W.scaled(cfg, B=4), src, n_dup=4, n_subst=1, seed=5)
    fresh = W.make_sources(cfg, 8, seed=9)
    batches = [(src[0:8], 0.9, L.INSERT_ON_MISS), (src[8:16], 0.9, L.INSERT_ON_MISS),
               (np.concatenate([src[[0, 5, 9, 15]], near]), 0.9, L.UPDATE_LRU),
               (np.concatenate([src[[2, 2]], fresh[:6]]), 0.9, L.INSERT_ON_MISS | L.UPDATE_LRU),      # evicts
               (np.concatenate([fresh[:4], src[[1, 3, 7, 11]]]), 1.0, 0)]                             # tau 1: nothing hits
    total_hits = 0
    for tick, (ids, tau, flags) in enumerate(batches, start=1):
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
        pre = []
        for b in st.banks:
            ob = O.Bank(b.n_slots, b.k, b.S, b.d, dtype, key_bits=True)
            ob.fp = b.fp.cpu().numpy().view(np.uint32).copy()
            ob.act = npf(b.act)
            ob.valid = b.valid.cpu().numpy().copy()
            ob.last_used = b.last_used.cpu().numpy().astype(np.uint64)
            ob.hits = b.hits.cpu().numpy().astype(np.uint32)
            pre.append(ob)
        outs = st.forward(h0, tau=tau, flags=flags | look, tick=tick, keep_all=True)
        torch.cuda.synchronize()
        oflags = (O.FLAG_UPDATE_LRU if flags & L.UPDATE_LRU else 0) | (O.FLAG_INSERT_ON_MISS if flags & L.INSERT_ON_MISS else 0) \
            | (O.FLAG_LOOKUP_LSH if lsh else 0)
        for l in range(cfg.n_layers):
            h_prev = npf(h0 if l == 0 else outs[l - 1])
            ob = pre[l]
            # the sign of a projection within 1e-5 of the vector's scale of zero may be decided differently in fp32
            v = O.simhash_projection(h_prev, Pnp[l], None)
            shaky = (np.abs(v) < 1e-5 * np.sqrt((v * v).mean(axis=1, keepdims=True))).any(axis=1)
            r = O.gated_layer(h_prev, ob, Pnp[l], None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu, f32(tau),
                              flags=oflags, tick=tick, out_dtype=dtype)
            assert not shaky.any()
            g, bk = st.gate[l], st.banks[l]
            hit = g.hit.cpu().numpy().astype(bool)
            assert np.array_equal(hit, r.hit), (tick, l)
            assert np.array_equal(g.idx.cpu().numpy(), r.idx), (tick, l)
            np.testing.assert_allclose(npf(g.sim), r.sim, atol=1e-6)
            n_miss = int((~hit).sum())
            if flags & L.INSERT_ON_MISS:
                assert g.slots.cpu().tolist()[:n_miss] == r.slots
                assert np.array_equal(bk.fp.cpu().numpy().view(np.uint32)[r.slots], r.q[~hit])
            assert np.array_equal(bk.valid.cpu().numpy(), ob.valid)
            vmask = ob.valid.astype(bool)
            assert np.array_equal(bk.last_used.cpu().numpy().astype(np.uint64)[vmask], ob.last_used[vmask])
            assert np.array_equal(bk.hits.cpu().numpy().astype(np.uint32)[vmask], ob.hits[vmask])
            got = npf(outs[l])
            for b in range(cfg.B):
                if hit[b]:
                    assert torch.equal(outs[l][b], torch.from_numpy(np.asarray(r.h_out[b], dtype=np.float32)).to(cfg.torch_dtype).cuda())
                else:
                    assert rel_err_rows(got[b:b + 1], r.h_out[b:b + 1])[0] < tol, (tick, l, b)
            total_hits += int(hit.sum())
        say(f"  batch {tick} (tau {tau}): hits per layer {[int(x.hit.sum()) for x in st.gate]}")
    assert total_hits > 0
    st.close()


def test_forward_can_be_captured_in_a_graph_and_replayed(L):
    """The per-layer call only enqueues kernels (no allocation, no memset, no host read-back), so a whole forward can
    be recorded in a HIP graph.  Every replay, with eager work and synchronisations in between, must give the eager
    result bit for bit, also after the input buffer's contents changed."""
    from paper_2512_16843_amd.engine import GatedStack
    say("graph capture of a 3-layer gated forward (carried means and keys): three replays against eager")
    cfg = W.scaled(W.BERT_BASE, n_layers=3, B=8, S=64, n_bank=32)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, keep_means=True, keep_next_keys=True)
    src = W.make_sources(cfg, 16, seed=1)
    for s0 in (0, 8):
        st.forward(W.embed(torch.from_numpy(src[s0:s0 + 8]), tok, pos, cfg.torch_dtype).cuda(), tau=2.0,
                   flags=L.INSERT_ON_MISS, tick=1)
    fresh = W.make_sources(cfg, 8, seed=9)
    inputs = [np.concatenate([src[[0, 3, 9, 12]], fresh[:4]]), np.concatenate([fresh[4:8], src[[1, 2, 14, 15]]]),
              src[8:16]]
    h_static = torch.empty((cfg.B, cfg.S, cfg.d), dtype=cfg.torch_dtype, device="cuda")
    h_static.copy_(W.embed(torch.from_numpy(inputs[0]), tok, pos, cfg.torch_dtype))
    st.forward(h_static, tau=0.9)                       # warm-up outside the capture (first-use settings)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out_static = st.forward(h_static, tau=0.9)
    torch.cuda.synchronize()
    for ids in inputs:
        h = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
        eager = st.forward(h, tau=0.9).clone()
        eager_hits = torch.stack([g.hit.clone() for g in st.gate])
        torch.cuda.synchronize()
        junk = torch.randn(1 << 20, device="cuda").sum()          # unrelated eager work between replays
        h_static.copy_(h)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_static, eager)
        assert torch.equal(torch.stack([g.hit for g in st.gate]), eager_hits)
        del junk
    st.close()


def test_insert_without_eviction_drops_and_counts(L):
    say("insert into a full bank with policy NONE")
    g = np.random.Generator(np.random.PCG64(13))
    bank = L.Bank(6, 32, 1, 64, torch.float32, "cuda", policy=L.EVICT_NONE)
    keys = torch.from_numpy(unit_rows(g, 8, 32).astype(np.float32)).cuda()
    inv = torch.empty((8,), dtype=torch.float32, device="cuda")
    L.llmc_inv_norm(keys, inv)
    acts = torch.zeros((8, 1, 64), dtype=torch.float32, device="cuda")
    slots = torch.empty((8,), dtype=torch.int32, device="cuda")
    counters = torch.zeros((L.CNT_WORDS,), dtype=torch.int32, device="cuda")
    L.llmc_bank_insert(bank, keys, inv, acts, None, None, 8, 1, slots, counters)
    torch.cuda.synchronize()
    assert slots.cpu().tolist() == [0, 1, 2, 3, 4, 5, -1, -1]
    assert int(counters[L.CNT_INSERTED]) == 6 and int(counters[L.CNT_DROPPED]) == 2 and int(counters[L.CNT_EVICTED]) == 0
    bank.close()


def test_gated_stream_with_insertion_and_lru_eviction(L):
    say("stream of batches with INSERT_ON_MISS | UPDATE_LRU on a small bank (eviction fires), fp32")
    from paper_2512_16843_amd.engine import GatedStack
    cfg = W.scaled(W.TINY_ENCODER, n_layers=1, n_bank=20, B=8)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, torch.float32, seed=3, n_layers=1)
    pool = W.make_sources(cfg, 30, seed=1)
    st = GatedStack(cfg, ws, Ps)
    wnp = [{k: npf(v) for k, v in w.items()} for w in ws]
    ob = O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, "f32")
    g = np.random.Generator(np.random.PCG64(21))
    flags = L.INSERT_ON_MISS | L.UPDATE_LRU
    tau = 0.999
    total_evicted = 0
    for tick in range(1, 13):
        # recurring sequences from a pool of 30: exact repeats hit, others miss and insert
        pick = g.integers(0, 30, cfg.B)
        h0 = W.embed(torch.from_numpy(pool[pick]), tok, pos, torch.float32)
        out = st.forward(h0.cuda(), tau=tau, flags=flags, tick=tick).clone()
        torch.cuda.synchronize()
        r = O.gated_layer(h0.numpy(), ob, npf(Ps[0]), None, wnp[0], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu,
                          f32(tau), flags=O.FLAG_INSERT_ON_MISS | O.FLAG_UPDATE_LRU, tick=tick, out_dtype="f32")
        gt = st.gate[0]
        assert np.array_equal(gt.hit.cpu().numpy().astype(bool), r.hit)
        assert np.array_equal(gt.idx.cpu().numpy(), r.idx)
        n_miss = int((~r.hit).sum())
        assert gt.slots.cpu().tolist()[:n_miss] == r.slots
        cnt = st.hit_counts()[0]
        assert cnt[L.CNT_INSERTED] == n_miss and cnt[L.CNT_EVICTED] == r.n_evicted
        total_evicted += r.n_evicted
        b = st.banks[0]
        assert np.array_equal(b.valid.cpu().numpy(), ob.valid)
        v = ob.valid.astype(bool)
        assert np.array_equal(b.last_used.cpu().numpy().astype(np.uint64)[v], ob.last_used[v])
        assert np.array_equal(b.hits.cpu().numpy().astype(np.uint32)[v], ob.hits[v])
        assert rel_err_rows(npf(out), r.h_out).max() < TOL["f32"]
        assert rel_err_rows(npf(b.act)[v], ob.act[v]).max() < TOL["f32"]
        # keep the two banks' stored values identical so later hits copy the same numbers
        ob.act[v] = npf(b.act)[v]
        ob.fp[v] = npf(b.fp)[v]
        ob.inv_norm[v] = npf(b.inv_norm)[v]
    assert total_evicted > 10
    st.close()


# ---------------------------------------------------------------------------
# bf16, model-sized rows, teacher-forced per layer
# ---------------------------------------------------------------------------

def bf16_steps(a, b):
    """Distance between two arrays of bf16 values (held in float32) in steps of the bf16 number line."""
    def ordinal(x):
        bits = (np.ascontiguousarray(x, dtype=np.float32).view(np.uint32) >> 16).astype(np.int64)
        mag = bits & 0x7FFF
        return np.where(bits & 0x8000, -mag, mag)
    return np.abs(ordinal(a) - ordinal(b))


def key_codes_close(q_gpu, q_oracle):
    """The GPU pools and projects in fp32 (fixed order), the oracle in fp64, and both round the normalised vector to
    bf16: an element's code may land one bf16 step apart.  For elements near zero a bf16 step is smaller than the
    fp32 noise of the sums they come from (about 1e-6 of the largest term, more after a centring offset has
    cancelled the common component), so there the bound is absolute: 1e-5 of the unit vector."""
    return bool(((bf16_steps(q_gpu, q_oracle) <= 1) | (np.abs(q_gpu - q_oracle) <= 1e-5)).all())


def teacher_forced_check(L, st, cfg, ws, Ps, h0, tau, dtype="bf16"):
    """Layer by layer with the GPU's own layer inputs and bank arrays.  The GPU's keys (fp32 accumulation) may differ
    from the oracle's by one bf16 step in a few elements: the codes are bounded separately, and the oracle's match is
    fed the GPU's keys, so that similarities are compared at 1e-5 and slots exactly."""
    outs = st.forward(h0, tau=tau, keep_all=True)
    torch.cuda.synchronize()
    stats = []
    h_prev = h0
    tau32 = f32(tau)
    for l in range(cfg.n_layers):
        wnp = {k: npf(v) for k, v in ws[l].items()}
        ob = oracle_bank_from_gpu(st.banks[l], dtype)
        g = st.gate[l]
        q_o, _ = O.fingerprint(npf(h_prev), npf(Ps[l]), None, dtype)
        q_g, qinv_g = npf(g.fp_used), npf(g.inv_used)
        steps = bf16_steps(q_g, q_o)
        assert key_codes_close(q_g, q_o), (steps.max(), np.abs(q_g - q_o).max())
        r = O.gated_layer(npf(h_prev), ob, None, None, wnp, cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu, tau32,
                          fp_override=(q_g, qinv_g))
        hit = g.hit.cpu().numpy().astype(bool)
        idx = g.idx.cpu().numpy()
        near = np.abs(r.sim - tau32) < 1e-3
        ties = O.near_tie_sets(q_g, qinv_g, ob.fp, ob.inv_norm, ob.valid)
        multi = np.array([len(t) > 1 for t in ties])
        assert np.array_equal(hit[~near], r.hit[~near]), (l, hit, r.hit, r.sim)
        assert np.array_equal(idx[~multi], r.idx[~multi]), (l, idx, r.idx)
        for b in np.nonzero(multi)[0]:
            assert idx[b] in ties[b]
        np.testing.assert_allclose(npf(g.sim), r.sim, rtol=0, atol=1e-5)
        got = npf(outs[l])
        for b in range(h0.shape[0]):
            if hit[b]:
                assert np.array_equal(got[b], ob.act[ob.act_slot[idx[b]]])
        miss = ~hit & ~r.hit
        err = rel_err_rows(got[miss], r.h_out[miss]) if miss.any() else np.zeros(1)
        assert err.max() < TOL[dtype], (l, err)
        stats.append(dict(layer=l, hits=int(hit.sum()), near_tau=int(near.sum()), near_tie=int(multi.sum()),
                          key_codes_off_by_one=int((steps > 0).sum()), max_err=float(err.max())))
        h_prev = outs[l]
    return stats


@pytest.mark.parametrize("which", ["encoder", "decoder"])
def test_model_sized_rows_bf16_teacher_forced(L, which):
    from paper_2512_16843_amd.engine import GatedStack
    if which == "encoder":
        cfg = W.scaled(W.BERT_BASE, n_layers=2, B=6, n_bank=192)
    else:
        cfg = W.scaled(W.GPT2_SMALL, n_layers=2, B=3, S=320, n_bank=96)
    say(f"{cfg.name} slice bf16: L=2 B={cfg.B} S={cfg.S} bank {cfg.n_bank}, teacher-forced")
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, torch.bfloat16, seed=3, n_layers=cfg.n_layers)
    src = W.make_sources(cfg, cfg.n_bank, seed=1)
    st = GatedStack(cfg, ws, Ps, expose_keys=True)
    h_src = W.embed(torch.from_numpy(src), tok, pos, torch.bfloat16).cuda()
    build_banks_gpu(L, st, h_src)
    assert all(torch.all(b.valid == 1) for b in st.banks)
    if which == "encoder":
        ids, _ = W.make_substitution_queries(cfg, src, n_dup=4, n_subst=12, seed=2)
    else:
        ids, _, _ = W.make_prefix_queries(cfg, src, seed=2)
    h0 = W.embed(torch.from_numpy(ids), tok, pos, torch.bfloat16).cuda()
    for tau in (0.98, 1.5):
        stats = teacher_forced_check(L, st, cfg, ws, Ps, h0, tau)
        for s in stats:
            say(f"  tau={tau} {s}")
    st.close()


# ---------------------------------------------------------------------------
# the cost hint with carried AND uncarried rows; Algorithm 1's single fingerprint
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("deferred", [False, True])
def test_cost_hint_with_carried_and_uncarried_rows(L, dtype, deferred):
    """LLMC_HINT_MOSTLY_CARRIED passed through the C ABI on a batch in which some rows arrive with a carried mean /
    key (or as references to the producing bank) and some do not: the uncarried rows are then pooled inside the
    projection's workgroups.  Keys against the oracle's fingerprint of the layer input, and every result against
    the same call without the hint, bit for bit.  S is not a multiple of the 64-token pooling chunk."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"cost hint with mixed rows, {dtype}, deferred copies {deferred}")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=3, B=8, S=70, n_bank=24) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=3, B=8, S=150, n_bank=24)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, keep_means=True, keep_next_keys=True, expose_keys=True)
    src = W.make_sources(cfg, 16, seed=1)
    fresh = W.make_sources(cfg, 8, seed=9)
    for s0 in (0, 8):
        st.forward(W.embed(torch.from_numpy(src[s0:s0 + 8]), tok, pos, cfg.torch_dtype).cuda(), tau=2.0,
                   flags=L.INSERT_ON_MISS, tick=1)
    ids = np.concatenate([src[[0, 5]], fresh[:3], src[[9, 15]], fresh[3:4]])       # 4 rows hit, 4 rows are computed
    h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    results = {}
    for hint in (False, True):
        st._stat_event = None                      # the engine's own hint logic stays out of the way
        st.auto_hint = False
        st._hint = [hint] * cfg.n_layers
        if deferred:
            y = st.forward(h0, tau=0.9).clone()
            outs = None
        else:
            outs = st.forward(h0, tau=0.9, keep_all=True)
            y = outs[-1].clone()
        torch.cuda.synchronize()
        assert any(st._deferred) == deferred
        results[hint] = (y, [dict(idx=g.idx.clone(), sim=g.sim.clone(), hit=g.hit.clone(), key=g.fp_used.clone(),
                                  inv=g.inv_used.clone()) for g in st.gate], outs)
    y0, g0, outs0 = results[False]
    y1, g1, _ = results[True]
    assert torch.equal(y0, y1)
    for l in range(cfg.n_layers):
        for k_ in g0[l]:
            assert torch.equal(g0[l][k_], g1[l][k_]), (l, k_)
        n_hit = int(g1[l]["hit"].sum())
        assert 0 < n_hit < cfg.B                   # carried and uncarried rows in every layer
    if outs0 is not None:
        # keys of the hinted run against the oracle's fingerprint of each layer's input
        for l in range(cfg.n_layers):
            h_prev = h0 if l == 0 else outs0[l - 1]
            q_o, qinv_o = O.fingerprint(npf(h_prev), npf(Ps[l]), None, dtype)
            q_g = npf(g1[l]["key"])
            if dtype == "bf16":
                assert key_codes_close(q_g, q_o)
            else:
                assert np.abs(q_g - q_o).max() < 1e-6
            np.testing.assert_allclose(npf(g1[l]["inv"]), O.inv_norm(q_g), rtol=3e-7, atol=0)
    st.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gated_decoder_with_prefix_attention_keys(L, dtype):
    """A causal decoder stack looked up under keys that include the prefix attention statistics (Section IV-B):
    banks are built from sources, queries share a prefix (a quarter to three quarters of the tokens) with a source and
    continue with fresh tokens.  Per layer, teacher-forced on the GPU's layer inputs: the keys against the oracle's,
    then decisions, matched slots, similarities and outputs against the oracle fed those keys.  The feature does what
    it is for: under these keys a query is closer to its source than under the token average alone."""
    from paper_2512_16843_amd.engine import GatedStack
    n_p = 16
    say(f"gated decoder with prefix attention keys {dtype}: first {n_p} tokens, prefix-sharing queries")
    if dtype == "f32":
        cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=8, S=64, n_bank=24, arch=1, gelu=1, ln_eps=1e-5)
    else:
        cfg = W.scaled(W.GPT2_SMALL, n_layers=2, B=8, S=64, n_bank=24)
    tol = TOL[dtype]
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    Pa = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=13, n_layers=cfg.n_layers)
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    src = W.make_sources(cfg, 16, seed=1)
    qids, qsrc, plen = W.make_prefix_queries(cfg, src, seed=2)
    assert plen.min() >= n_p
    # weigh the attention feature like the token average: scale its map by the ratio of the two features' lengths
    h_src = W.embed(torch.from_numpy(src[:8]), tok, pos, cfg.torch_dtype)
    a0 = O.prefix_attention_mean(npf(h_src), wnp[0], cfg.arch, cfg.n_heads, cfg.ln_eps, n_p)
    ratio = float(np.linalg.norm(npf(h_src).astype(np.float64).mean(axis=1)) / np.linalg.norm(a0))
    P2 = [torch.cat([Ps[l].float(), Pa[l].float() * (2.0 * ratio)]).to(cfg.torch_dtype) for l in range(cfg.n_layers)]
    st = GatedStack(cfg, ws, Ps, prefix_tokens=n_p, proj2=P2)
    obanks = [O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, dtype) for _ in range(cfg.n_layers)]
    batches = [(src[0:8], 2.0, L.INSERT_ON_MISS), (src[8:16], 2.0, L.INSERT_ON_MISS), (qids, 0.8, L.UPDATE_LRU)]
    for tick, (ids, tau, flags) in enumerate(batches, start=1):
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype)
        outs = st.forward(h0.cuda(), tau=tau, flags=flags, tick=tick, keep_all=True)
        torch.cuda.synchronize()
        oflags = (O.FLAG_UPDATE_LRU if flags & L.UPDATE_LRU else 0) | (O.FLAG_INSERT_ON_MISS if flags & L.INSERT_ON_MISS else 0)
        for l in range(cfg.n_layers):
            h_prev = npf(h0 if l == 0 else outs[l - 1])
            q_g, qinv_g = npf(st.pfx_fp[l]), npf(st.pfx_inv[l])
            q_o, _ = O.fingerprint_prefix(h_prev, npf(P2[l]), None, dtype, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, n_p)
            err = np.abs(q_g - q_o).max()
            assert err < (1e-5 if dtype == "f32" else 1.5e-3), (tick, l, err)
            ob = obanks[l]
            pre_fp, pre_inv, pre_valid = ob.fp.copy(), ob.inv_norm.copy(), ob.valid.copy()
            r = O.gated_layer(h_prev, ob, None, None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu, f32(tau),
                              flags=oflags, tick=tick, out_dtype=dtype, fp_override=(q_g, qinv_g))
            g, bk = st.gate[l], st.banks[l]
            hit = g.hit.cpu().numpy().astype(bool)
            assert not (np.abs(r.sim - f32(tau)) < 1e-3).any()
            assert np.array_equal(hit, r.hit), (tick, l)
            gi = g.idx.cpu().numpy()
            if pre_valid.any():
                ties = O.near_tie_sets(q_g, qinv_g, pre_fp, pre_inv, pre_valid)
                for b in range(cfg.B):
                    assert gi[b] == r.idx[b] or gi[b] in ties[b], (tick, l, b)
                np.testing.assert_allclose(npf(g.sim), r.sim, rtol=0, atol=1e-5)
            assert np.array_equal(bk.valid.cpu().numpy(), ob.valid)
            if flags & L.INSERT_ON_MISS:
                assert np.array_equal(npf(bk.fp)[r.slots], q_g[~hit])
            got = npf(outs[l])
            for b in range(cfg.B):
                if hit[b]:
                    assert np.array_equal(got[b], npf(bk.act[int(gi[b])]))
                else:
                    assert rel_err_rows(got[b:b + 1], r.h_out[b:b + 1])[0] < tol, (tick, l, b)
            if tick == 3 and l == 0:
                # first layer, queries against their own sources: similarity under both kinds of key
                s_pfx = O.similarities(q_g, qinv_g, pre_fp, pre_inv)[np.arange(cfg.B), qsrc]
                q_pl, qi_pl = O.fingerprint(h_prev, npf(Ps[0]), None, dtype)
                k_pl, ki_pl = O.fingerprint(npf(W.embed(torch.from_numpy(src), tok, pos, cfg.torch_dtype)), npf(Ps[0]), None, dtype)
                s_plain = O.similarities(q_pl, qi_pl, k_pl, ki_pl)[np.arange(cfg.B), qsrc]
                say(f"  similarity to the own source: prefix keys {s_pfx.mean():.4f}, token average alone {s_plain.mean():.4f}; "
                    f"hits {int(hit.sum())} of {cfg.B}")
                assert s_pfx.mean() > s_plain.mean()
    st.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_single_fingerprint_mode_against_oracle(L, dtype):
    """Algorithm 1 as printed: one fingerprint of the input, reused by every layer (d_fp_given of the C ABI)."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"single-fingerprint mode {dtype}: banks built and queried with the key of h_0 at every layer")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=3, B=8, n_bank=24) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=3, B=8, S=48, n_bank=24)
    tol = TOL[dtype]
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps)
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    Pnp = [npf(p) for p in Ps]
    obanks = [O.Bank(cfg.n_bank, cfg.k, cfg.S, cfg.d, dtype) for _ in range(cfg.n_layers)]
    src = W.make_sources(cfg, 16, seed=1)
    near, _ = W.make_substitution_queries(W.scaled(cfg, B=4), src, n_dup=4, n_subst=1, seed=5)
    fresh = W.make_sources(cfg, 8, seed=9)
    batches = [(src[0:8], 2.0, L.INSERT_ON_MISS), (src[8:16], 2.0, L.INSERT_ON_MISS),
               (np.concatenate([src[[0, 5, 9, 15]], fresh[:4]]), 0.9, 0),
               (np.concatenate([near, fresh[4:8]]), 0.9, L.INSERT_ON_MISS | L.UPDATE_LRU)]
    for tick, (ids, tau, flags) in enumerate(batches, start=1):
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype)
        outs = st.forward(h0.cuda(), tau=tau, flags=flags, tick=tick, keep_all=True, single_fingerprint=True)
        torch.cuda.synchronize()
        oflags = (O.FLAG_UPDATE_LRU if flags & L.UPDATE_LRU else 0) | (O.FLAG_INSERT_ON_MISS if flags & L.INSERT_ON_MISS else 0)
        # the oracle runs teacher-forced per layer on the GPU's layer inputs.  The one key of the batch: the oracle's
        # fingerprint of h_0 bounds the GPU's (one step of the storage type at most), and the GPU's key is what
        # the oracle's layers are fed, so that similarities compare at 1e-5
        q_o, _ = O.fingerprint(npf(h0), Pnp[0], None, dtype)
        q_g, qinv_g = run_fingerprint(L, h0.cuda(), Ps[0].cuda(), None)
        q_g, qinv_g = npf(q_g), npf(qinv_g)
        if dtype == "bf16":
            assert key_codes_close(q_g, q_o)
        else:
            assert np.abs(q_g - q_o).max() < 1e-6
        fp0 = (q_g, qinv_g)
        for l in range(cfg.n_layers):
            h_prev = npf(h0 if l == 0 else outs[l - 1])
            ob = obanks[l]
            pre_fp, pre_inv, pre_valid = ob.fp.copy(), ob.inv_norm.copy(), ob.valid.copy()
            r = O.gated_layer(h_prev, ob, None, None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu, f32(tau),
                              flags=oflags, tick=tick, out_dtype=dtype, fp_override=fp0)
            g, bk = st.gate[l], st.banks[l]
            hit = g.hit.cpu().numpy().astype(bool)
            near_tau = np.abs(r.sim - f32(tau)) < 1e-3
            assert not near_tau.any()
            assert np.array_equal(hit, r.hit), (tick, l)
            ties = O.near_tie_sets(fp0[0], fp0[1], pre_fp, pre_inv, pre_valid) if pre_valid.any() else None
            gi = g.idx.cpu().numpy()
            for b in range(cfg.B):
                assert gi[b] == r.idx[b] or (ties is not None and gi[b] in ties[b]), (tick, l, b)
            if pre_valid.any():
                np.testing.assert_allclose(npf(g.sim), r.sim, rtol=0, atol=1e-5)
            n_miss = int((~hit).sum())
            if flags & L.INSERT_ON_MISS:
                assert g.slots.cpu().tolist()[:n_miss] == r.slots
            assert np.array_equal(bk.valid.cpu().numpy(), ob.valid)
            got = npf(outs[l])
            for b in range(cfg.B):
                if hit[b]:
                    assert np.array_equal(got[b], npf(bk.act[int(gi[b])]))
                else:
                    assert rel_err_rows(got[b:b + 1], r.h_out[b:b + 1])[0] < tol, (tick, l, b)
            # keep the two banks' stored arrays identical, so that later hits copy the same numbers
            v = ob.valid.astype(bool)
            ob.act[v] = npf(bk.act)[v]
            ob.fp[v] = npf(bk.fp)[v]
            ob.inv_norm[v] = npf(bk.inv_norm)[v]
        say(f"  batch {tick} (tau {tau}): hits per layer {[int(x.hit.sum()) for x in st.gate]}")
    assert sum(int(x.hit.sum()) for x in st.gate) > 0
    st.close()


def test_large_batch_equals_its_halves(L):
    """Batches of more than 64 rows take the stand-alone decision and compaction kernels, smaller ones the fused
    kernel: a batch of 96 rows and the same rows as two batches of 48 must give the same bits row by row."""
    from paper_2512_16843_amd.engine import GatedStack
    say("gated stack: 96 rows at once against two batches of 48")
    cfg = W.scaled(W.BERT_BASE, n_layers=2, B=96, S=40, n_bank=160)
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    src = W.make_sources(cfg, 160, seed=1)
    fresh = W.make_sources(cfg, 48, seed=9)
    ids = np.concatenate([src[::4][:40], fresh[:30], src[1::7][:20], fresh[30:36]])
    assert ids.shape[0] == 96
    big = GatedStack(cfg, ws, Ps, expose_keys=True)
    half = GatedStack(W.scaled(cfg, B=48), ws, Ps, expose_keys=True)
    wide = GatedStack(W.scaled(cfg, B=80), ws, Ps)
    for s0 in range(0, 160, 80):                              # one set of banks, built by 80-row batches
        h = W.embed(torch.from_numpy(src[s0:s0 + 80]), tok, pos, cfg.torch_dtype).cuda()
        wide.forward(h, tau=2.0, flags=L.INSERT_ON_MISS, tick=1)
    for st in (big, half):                                    # hand the built banks' arrays to the two stacks under test
        for l in range(cfg.n_layers):
            for name in ("fp", "inv_norm", "act", "last_used", "hits", "valid"):
                getattr(st.banks[l], name).copy_(getattr(wide.banks[l], name))
            st.banks[l].refresh()
    h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
    y_big = big.forward(h0, tau=0.9).clone()
    g_big = [dict(idx=g.idx.clone(), sim=g.sim.clone(), hit=g.hit.clone(), key=g.fp_used.clone()) for g in big.gate]
    torch.cuda.synchronize()
    assert 0 < int(g_big[0]["hit"].sum()) < 96
    for part in range(2):
        rows = slice(48 * part, 48 * part + 48)
        y = half.forward(h0[rows].contiguous(), tau=0.9).clone()
        torch.cuda.synchronize()
        assert torch.equal(y, y_big[rows])
        for l in range(cfg.n_layers):
            g = half.gate[l]
            assert torch.equal(g.idx, g_big[l]["idx"][rows]) and torch.equal(g.sim, g_big[l]["sim"][rows])
            assert torch.equal(g.hit, g_big[l]["hit"][rows]) and torch.equal(g.fp_used, g_big[l]["key"][rows])
    for st in (big, half, wide):
        st.close()


@pytest.mark.parametrize("dtype,d,k,S,B", [
    ("bf16", 768, 256, 65, 1027),      # two chunks, three rows in the last workgroup
    ("bf16", 64, 64, 1, 1537),         # slices of four rows of the map, one token, one row in the last workgroup
    ("f32", 192, 128, 130, 514),       # two rows in the last workgroup, three chunks
    ("bf16", 1088, 256, 2, 1026),      # slices of 68 rows
    ("bf16", 128, 256, 577, 257),      # the first batch of 256-value keys that goes four rows to a workgroup, ten chunks
    ("f32", 64, 128, 3, 513),          # ... of 128 values
    ("bf16", 4032, 64, 1, 1536),       # ... of 64 values, at the widest rows for them
    ("bf16", 6016, 256, 1, 259),       # the widest rows whose sums fit the LDS
    ("f32", 4096, 256, 1, 258),        # the widest rows of fp32
])
def test_keys_of_many_rows_are_those_of_a_few(L, dtype, d, k, S, B):
    """Batches of many rows (more than 256 for keys of 256 values, 512 for 128, from 1536 for 64) are projected four rows to a
    workgroup: the same bits as in a small batch, for cosine keys, their norms and sign-bit keys."""
    say(f"keys of {B} rows {dtype} d={d} k={k} S={S}")
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(B)
    h = torch.randn((B, S, d), generator=g, device="cuda").to(dt)
    h[1] = 0                                                       # a zero key
    P = (torch.randn((d, k), generator=g, device="cuda") * k ** -0.5).to(dt)
    bias = torch.randn((k,), generator=g, device="cuda") * 0.1
    def keys(x, c):
        n = x.shape[0]
        fp, inv = torch.empty((n, k), dtype=dt, device="cuda"), torch.empty((n,), device="cuda")
        bits = torch.empty((n, k // 32), dtype=torch.int32, device="cuda")
        ws = torch.empty((L.llmc_fingerprint_workspace_bytes(n, S, d),), dtype=torch.uint8, device="cuda")
        L.llmc_fingerprint(x, P, c, fp, inv, ws)
        L.llmc_fingerprint_bits(x, P, c, bits, ws)
        torch.cuda.synchronize()
        return fp, inv, bits
    for c in (None, bias):
        many = keys(h, c)
        for rows in (slice(0, 9), slice(B // 2, B // 2 + 5), slice(B - 6, B)):
            few = keys(h[rows].contiguous(), c)
            assert all(torch.equal(m[rows], f) for m, f in zip(many, few)), (rows, c is None)


@pytest.mark.parametrize("dtype,d,k,n", [("bf16", 192, 256, 258), ("f32", 128, 128, 515), ("bf16", 64, 64, 1538)])
def test_next_keys_of_a_large_bank_are_those_of_a_small_one(L, dtype, d, k, n):
    """llmc_bank_pool_values projects the kept means of a large bank four rows to a workgroup: the bits of a small bank."""
    say(f"next-layer keys of {n} stored values {dtype} d={d} k={k}")
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n)
    act = torch.randn((n, 2, d), generator=g, device="cuda").to(dt)
    P = (torch.randn((d, k), generator=g, device="cuda") * k ** -0.5).to(dt)
    c = torch.randn((k,), generator=g, device="cuda") * 0.1

    def keys(rows):
        bank = L.Bank(rows.shape[0], 32, 2, d, dt, "cuda", keep_means=True, next_proj=P, next_bias=c)
        bank.act.copy_(rows)
        L.llmc_bank_pool_values(bank)
        torch.cuda.synchronize()
        out = [t.clone() for t in (bank.act_pool, bank.next_fp, bank.next_inv)]
        bank.close()
        return out
    many = keys(act)
    for rows in (slice(0, 5), slice(n - 3, n)):
        assert all(torch.equal(m[rows], f) for m, f in zip(many, keys(act[rows]))), rows


@pytest.mark.parametrize("dtype,d,S,B,n_bank,policy", [
    ("bf16", 128, 1, 5, 8, "lru"),          # one token: one chunk of one
    ("bf16", 768, 64, 3, 16, "lru"),        # whole chunks
    ("bf16", 1024, 130, 4, 6, "lru"),       # the widest row that is pooled on the way out; entries are evicted
    ("bf16", 256, 577, 3, 4, "none"),       # ten chunks, the last of one token; the second batch is dropped
    ("f32", 512, 65, 4, 8, "lru"),
    ("f32", 768, 65, 4, 8, "lru"),          # too wide for it: the rows are pooled again
])
def test_means_and_next_keys_kept_at_insertion_are_those_of_the_stored_values(L, dtype, d, S, B, n_bank, policy):
    """What a bank keeps beside the outputs that a call computes and stores (their token means and next-layer keys, formed
    from the chunk sums of the block's last LayerNorm) has the bits that llmc_bank_pool_values forms from the values."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"kept means and next keys {dtype} d={d} S={S} B={B} bank {n_bank} {policy}")
    cfg = W.scaled(small_cfg(0, dtype, d, d // 64, 2 * d, S, B), n_layers=2, n_bank=n_bank)
    ws = W.make_layer_weights(cfg, seed=4)
    Ps = W.make_projection(d, cfg.k, cfg.torch_dtype, seed=3, n_layers=2)
    st = GatedStack(cfg, ws, Ps, keep_means=True, keep_next_keys=True, policy=L.EVICT_LRU if policy == "lru" else L.EVICT_NONE)
    g = torch.Generator(device="cuda").manual_seed(S + d)
    for tick in (1, 2):
        h0 = torch.randn((B, S, d), generator=g, device="cuda").to(cfg.torch_dtype)
        st.forward(h0, tau=2.0, flags=L.INSERT_ON_MISS, tick=tick)
        torch.cuda.synchronize()
        for l in range(2):
            b = st.banks[l]
            live = b.valid.bool()
            kept = [b.act_pool[live].clone()] + ([b.next_fp[live].clone(), b.next_inv[live].clone()] if l == 0 else [])
            L.llmc_bank_pool_values(b)
            torch.cuda.synchronize()
            again = [b.act_pool[live]] + ([b.next_fp[live], b.next_inv[live]] if l == 0 else [])
            assert int(live.sum()) == min(n_bank, tick * B)
            assert all(torch.equal(x, y) for x, y in zip(kept, again)), (tick, l)
    st.close()


@pytest.mark.parametrize("arch", [0, 1])
def test_few_rows_and_many_rows_give_the_same_bits(L, arch):
    """A launch with few rows cuts the linear layers into smaller tiles with a deeper ring than a launch with many:
    a sequence must come out with the same bits whether it is computed among 64 or among 4."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"plain block arch={arch}: 64 sequences of 128 tokens at once against the first 4 and the last 3 alone")
    base = W.BERT_BASE if arch == 0 else W.GPT2_SMALL
    cfg = W.scaled(base, n_layers=2, B=64, S=128)
    ws = W.make_layer_weights(cfg, seed=5)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    g = torch.Generator(device="cuda").manual_seed(3)
    h0 = (torch.randn((64, 128, cfg.d), generator=g, device="cuda") * 0.5).to(cfg.torch_dtype)
    big = GatedStack(cfg, ws, Ps, cached_layers=[])
    y_big = big.forward(h0, tau=2.0).clone()
    torch.cuda.synchronize()
    for rows in (slice(0, 4), slice(61, 64)):
        n = rows.stop - rows.start
        few = GatedStack(W.scaled(cfg, B=n), ws, Ps, cached_layers=[])
        y = few.forward(h0[rows].contiguous(), tau=2.0).clone()
        torch.cuda.synchronize()
        assert torch.equal(y, y_big[rows])
        few.close()
    big.close()


@pytest.mark.parametrize("d,dff,S,B,tilings", gemm_rule.FEW_ROWS)
@pytest.mark.parametrize("arch", [0, 1])
def test_bf16_layer_tilings(L, arch, d, dff, S, B, tilings):
    """The bf16 block on the tilings for few rows against the oracle, and the same bits for the last sequence computed
    alone (where fewer rows may mean other tiles).  The case names the tilings that its layers take."""
    assert gemm_rule.block(d, dff, S * B) == tilings.split()
    from paper_2512_16843_amd.engine import GatedStack
    say(f"plain bf16 layer arch={arch} d={d} dff={dff} S={S} B={B}")
    cfg = small_cfg(arch, "bf16", d, d // 64, dff, S, B)
    ws = W.make_layer_weights(cfg, seed=12)
    Ps = W.make_projection(d, cfg.k, torch.bfloat16)
    g = np.random.Generator(np.random.PCG64(d + S))
    h0 = torch.from_numpy(g.standard_normal((B, S, d)).astype(np.float32)).bfloat16().cuda()
    st = GatedStack(cfg, ws, Ps, cached_layers=[])
    out = st.forward(h0, tau=0.5).clone()
    torch.cuda.synchronize()
    one = GatedStack(W.scaled(cfg, B=1), ws, Ps, cached_layers=[])
    alone = one.forward(h0[B - 1:].contiguous(), tau=0.5)
    torch.cuda.synchronize()
    assert torch.equal(alone[0], out[B - 1])
    wnp = {k: npf(v) for k, v in ws[0].items()}
    rows = [0, B - 1]
    want = np.stack([O.layer_forward(npf(h0[b]), wnp, arch, d // 64, cfg.ln_eps, cfg.gelu) for b in rows])
    assert rel_err_rows(npf(out)[rows], want).max() < TOL["bf16"]
    st.close()
    one.close()


@pytest.mark.parametrize("d,dff,S,B,tilings", gemm_rule.MANY_ROWS)
@pytest.mark.parametrize("arch", [0, 1])
def test_bf16_layer_tilings_of_many_rows(L, arch, d, dff, S, B, tilings):
    """The bf16 block on the tilings for many rows against the oracle, and the same bits for the last sequence alone."""
    test_bf16_layer_tilings(L, arch, d, dff, S, B, tilings)


@pytest.mark.parametrize("d,dff,S,B", [
    (64, 64, 1, 1),          # one token, one column tile
    (192, 320, 33, 3),       # 99 tokens: ragged against 32 and 64 rows, widths that are odd multiples of 64
    (128, 64, 145, 2),       # attention: two query blocks and a third of 17, five key tiles, the last with 17 keys
    (768, 3072, 128, 12),    # 1536 tokens: the wide outputs (2304 and 3072) take the 64 x 64 tiles, the others 32 x 32
    (768, 3072, 131, 27),    # 3537 tokens, 17 of them in the last row of tiles: 672 tiles of 64 x 64 or more in every layer
])
@pytest.mark.parametrize("arch", [0, 1])
def test_f32_layer_tilings(L, arch, d, dff, S, B):
    """The fp32 block on its tilings against the oracle, and the same bits for the last sequence computed alone."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"plain fp32 layer arch={arch} d={d} dff={dff} S={S} B={B}")
    cfg = small_cfg(arch, "f32", d, d // 64, dff, S, B)
    ws = W.make_layer_weights(cfg, seed=12)
    Ps = W.make_projection(d, cfg.k, torch.float32)
    g = np.random.Generator(np.random.PCG64(d + S))
    h0 = torch.from_numpy(g.standard_normal((B, S, d)).astype(np.float32)).cuda()
    st = GatedStack(cfg, ws, Ps, cached_layers=[])
    out = st.forward(h0, tau=0.5).clone()
    torch.cuda.synchronize()
    one = GatedStack(W.scaled(cfg, B=1), ws, Ps, cached_layers=[])
    alone = one.forward(h0[B - 1:].contiguous(), tau=0.5)
    torch.cuda.synchronize()
    assert torch.equal(alone[0], out[B - 1])
    wnp = {k: npf(v) for k, v in ws[0].items()}
    rows = [0, B - 1]
    want = np.stack([O.layer_forward(npf(h0[b]), wnp, arch, d // 64, cfg.ln_eps, cfg.gelu) for b in rows])
    # sums of at most 3072 fp32 products per element, a few layers of them: well inside 1e-5 of the row's largest value
    assert rel_err_rows(npf(out)[rows], want).max() < 1e-5
    st.close()
    one.close()


@pytest.mark.parametrize("masked,every,inf_values", [
    (32, 2, False),          # the first 32-key tile: every other query of a wavefront
    (32, 1, True),           # ... of every query, and the values there are infinite
    (65, 1, False),          # two tiles and one key of the third
])
def test_f32_attention_scores_that_overflow_in_the_first_tiles(L, masked, every, inf_values):
    """Scores of the first keys that overflow to -inf: those keys count for nothing, the later ones as usual."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"fp32 attention, the first {masked} keys of {masked + 9} masked by overflow, inf_values={inf_values}")
    S, B = masked + 9, 2
    cfg = small_cfg(0, "f32", 64, 1, 64, S, B)
    ws = W.make_layer_weights(cfg, seed=31)
    w = ws[0]
    g = np.random.Generator(np.random.PCG64(masked))
    x = g.standard_normal((B, S, 64)).astype(np.float32)
    x[:, :, 0] = 0.0
    x[:, :masked, 0] = 2.0                                    # the masked keys
    x[:, :, 1] = 0.0
    x[:, ::every, 1] = 1.0                                    # the queries that they are masked for
    # query and key 0 see these two channels alone: their product is -2e40 for a masked pair and 0 for any other
    for row, ch, v in ((0, 1, 1e20), (64, 0, -1e20)) + (((128, 0, 3e38),) if inf_values else ()):
        w["wqkv"][row] = 0.0
        w["wqkv"][row, ch] = v
        w["bqkv"][row] = 0.0
    st = GatedStack(cfg, ws, W.make_projection(64, cfg.k, torch.float32), cached_layers=[])
    out = st.forward(torch.from_numpy(x).cuda(), tau=0.5)
    torch.cuda.synchronize()
    wnp = {k: npf(v) for k, v in w.items()}
    want = np.stack([O.layer_forward(x[b], wnp, 0, 1, cfg.ln_eps, cfg.gelu) for b in range(B)])
    assert np.isfinite(npf(out)).all()
    assert rel_err_rows(npf(out), want).max() < 1e-5          # sums of at most 74 fp32 products
    st.close()


@pytest.mark.parametrize("carry", [False, True], ids=["plain", "carried"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_within_batch_reuse_against_oracle(L, dtype, carry):
    """LLMC_DEDUP: rows of a batch that miss the bank follow an earlier, similar row of the same batch instead of
    being computed and stored again (Algorithm 1 applied to the rows in order).  Leaders, followers, slots, counters,
    bank metadata and outputs against the oracle, layer by layer with the GPU's own layer inputs, keys and bank
    arrays, over batches that fill the banks and then evict.  "carried": the banks also store token means and
    next-layer keys, so rows reach the second layer carried (hits), pooled by the block (leaders) or neither
    (followers, whose rows are written after the block ran)."""
    from paper_2512_16843_amd.engine import GatedStack
    say(f"within-batch reuse {dtype} carry={carry}: duplicates and near-duplicates inside batches, insertion + LRU, eviction")
    cfg = W.scaled(W.TINY_ENCODER, n_layers=2, B=8, n_bank=12) if dtype == "f32" else \
        W.scaled(W.BERT_BASE, n_layers=2, B=8, S=48, n_bank=12)
    tol = TOL[dtype]
    ws = W.make_layer_weights(cfg, seed=0)
    tok, pos = W.make_embeddings(cfg, seed=0)
    Ps = W.make_projection(cfg.d, cfg.k, cfg.torch_dtype, seed=3, n_layers=cfg.n_layers)
    st = GatedStack(cfg, ws, Ps, expose_keys=True, keep_means=carry, keep_next_keys=carry)
    wnp = [{k_: npf(v) for k_, v in w.items()} for w in ws]
    src = W.make_sources(cfg, 16, seed=1)
    near, _ = W.make_substitution_queries(W.scaled(cfg, B=4), src[:4], n_dup=4, n_subst=1, seed=5)
    fresh = W.make_sources(cfg, 12, seed=9)
    tau = 0.97 if dtype == "f32" else 0.995
    flags = L.INSERT_ON_MISS | L.UPDATE_LRU | L.DEDUP
    oflags = O.FLAG_INSERT_ON_MISS | O.FLAG_UPDATE_LRU | O.FLAG_DEDUP
    batches = [np.stack([src[0], src[0], fresh[0], near[0], fresh[1], fresh[0], src[5], src[5]]),
               np.stack([src[0], fresh[2], fresh[2], src[5], near[1], near[1], fresh[0], fresh[3]]),
               np.stack([fresh[4], fresh[5], fresh[4], fresh[6], fresh[7], fresh[5], fresh[8], fresh[4]])]      # evicts
    total_followers = 0
    for tick, ids in enumerate(batches, start=1):
        h0 = W.embed(torch.from_numpy(ids), tok, pos, cfg.torch_dtype).cuda()
        pre = [oracle_bank_from_gpu(b, dtype) for b in st.banks]
        outs = st.forward(h0, tau=tau, flags=flags, tick=tick, keep_all=True)
        torch.cuda.synchronize()
        for l in range(cfg.n_layers):
            h_prev = npf(h0 if l == 0 else outs[l - 1])
            ob, g, bk = pre[l], st.gate[l], st.banks[l]
            q_g, qinv_g = npf(g.fp_used), npf(g.inv_used)
            q_o, _ = O.fingerprint(h_prev, npf(Ps[l]), None, dtype)
            assert key_codes_close(q_g, q_o) if dtype == "bf16" else np.abs(q_g - q_o).max() < 1e-6
            r = O.gated_layer(h_prev, ob, None, None, wnp[l], cfg.arch, cfg.n_heads, cfg.ln_eps, cfg.gelu, f32(tau),
                              flags=oflags, tick=tick, out_dtype=dtype, fp_override=(q_g, qinv_g))
            # no similarity (to the bank or between rows of the batch) sits within 1e-3 of the threshold here
            pair = O.similarities(q_g, qinv_g, q_g, qinv_g)
            assert not (np.abs(pair - f32(tau)) < 1e-3).any() and not (np.abs(r.sim - f32(tau)) < 1e-3).any()
            hit = g.hit.cpu().numpy().astype(bool)
            assert np.array_equal(hit, r.hit), (tick, l, hit, r.hit)
            assert np.array_equal(g.idx.cpu().numpy()[hit], r.idx[hit]), (tick, l)
            np.testing.assert_allclose(npf(g.sim)[hit], r.sim[hit], rtol=0, atol=1e-5)
            cnt = g.counters.cpu().numpy()
            n_fol, n_lead = len(r.follower_of), len(r.slots)
            assert cnt[L.CNT_DEDUP] == n_fol and cnt[L.CNT_MISS] == n_lead and cnt[L.CNT_COMPUTED] == n_lead
            assert cnt[L.CNT_HIT] == int(hit.sum()) and cnt[L.CNT_INSERTED] == n_lead and cnt[L.CNT_EVICTED] == r.n_evicted
            assert g.slots.cpu().tolist()[:n_lead] == r.slots
            assert np.array_equal(bk.valid.cpu().numpy(), ob.valid)
            v = ob.valid.astype(bool)
            assert np.array_equal(bk.last_used.cpu().numpy().astype(np.uint64)[v], ob.last_used[v])
            assert np.array_equal(bk.hits.cpu().numpy().astype(np.uint32)[v], ob.hits[v])
            got = npf(outs[l])
            for b in range(cfg.B):
                if b in r.follower_of:
                    assert torch.equal(outs[l][b], outs[l][r.follower_of[b]])          # the leader's row, bit for bit
                    assert torch.equal(outs[l][b], bk.act[int(r.idx[b])])
                elif hit[b]:
                    assert np.array_equal(got[b], npf(bk.act[int(r.idx[b])]))
                else:
                    assert rel_err_rows(got[b:b + 1], r.h_out[b:b + 1])[0] < tol, (tick, l, b)
            total_followers += n_fol
        say(f"  batch {tick}: hits per layer {[int(x.hit.sum()) for x in st.gate]}, "
            f"followers per layer {[int(x.counters[L.CNT_DEDUP]) for x in st.gate]}")
    assert total_followers >= 8
    st.close()
